// Bus admittance matrix assembly on the device (pi-model branches, Sec. 2.1).
//
// Pipeline (one thread per branch or per row; rows have a handful of entries):
//   1. validate branches, count incident branches per bus (integer atomics)
//   2. exclusive scan of (1 + degree)            -> slot offsets
//   3. scatter (neighbour, branch) slots per row  (slot 0 of each row = diagonal)
//      (1 to 3 in one workgroup up to kYbusSmallBuses buses)
//   4. per row: count distinct columns; scan the counts within each workgroup
//   5. scan of the workgroups' totals (in step 6 while they are few)
//   6. per row: order slots by branch, sum the diagonal in branch order, stable-order by
//      column, emit row_ptr and merged entries; parallel branches are summed in branch
//      order
// A bad branch makes every later step leave at once; the host reads the flag, the number
// of entries and the longest row back once, at the end.
// Products are not contracted into FMAs here, so every entry is the same
// correctly-rounded sequence as a plain sequential assembly.
#pragma once

#include "common.hpp"

namespace dpf {

__global__ void ybus_count_kernel(int32_t n_bus, int32_t n_branch, const int32_t *__restrict__ from,
                                  const int32_t *__restrict__ to, const double *__restrict__ r,
                                  const double *__restrict__ x, int32_t *__restrict__ deg,
                                  int32_t *__restrict__ err) {
    int32_t e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n_branch) return;
    int32_t f = from[e], t = to[e];
    bool bad = f < 0 || f >= n_bus || t < 0 || t >= n_bus || f == t || (r[e] == 0.0 && x[e] == 0.0);
    if (bad) {
        atomicOr(err, 1);
        return;
    }
    atomicAdd(&deg[f], 1);
    atomicAdd(&deg[t], 1);
}

// Exclusive scan of in[i] + add for i < n into out[0..n] by one workgroup of 1024
// threads, in tiles of 4096 with the next tile's loads in flight (one thread per
// contiguous chunk instead reads uncoalesced: 37 us for 5300 values, this 4).
__global__ __launch_bounds__(1024) void scan_kernel(int32_t n, const int32_t *__restrict__ in, int32_t add,
                                                   int32_t *__restrict__ out) {
    __shared__ int32_t part[2][1024 / kWave];
    const int32_t tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wv = tid / kWave;
    int32_t v[4], next[4];
    auto load = [&](int64_t base, int32_t *x) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t i = base + tid * 4 + u;
            x[u] = i < n ? in[i] + add : 0;
        }
    };
    load(0, next);
    int32_t run = 0;
    int flip = 0;
    for (int64_t base = 0; base < n; base += 4096, flip ^= 1) {
        int32_t s = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            v[u] = next[u];
            s += v[u];
        }
        load(base + 4096, next);
        int32_t incl = s;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int32_t y = __shfl_up(incl, o, kWave);
            if (lane >= o) incl += y;
        }
        if (lane == kWave - 1) part[flip][wv] = incl;
        __syncthreads();
        int32_t o = run + incl - s;
        for (int k = 0; k < 1024 / kWave; ++k) {
            o += k < wv ? part[flip][k] : 0;
            run += part[flip][k];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t i = base + tid * 4 + u;
            if (i < n) out[i] = o;
            o += v[u];
        }
    }
    if (tid == 0) out[n] = run;
}

__global__ void ybus_scatter_kernel(int32_t n_bus, int32_t n_branch, const int32_t *__restrict__ from,
                                    const int32_t *__restrict__ to, const int32_t *__restrict__ soff,
                                    int32_t *__restrict__ fill, int2 *__restrict__ slot,
                                    const int32_t *__restrict__ err) {
    int32_t k = blockIdx.x * blockDim.x + threadIdx.x;
    if (*err) return;
    if (k < n_bus) slot[soff[k]] = make_int2(k, -1);  // diagonal
    if (k >= n_branch) return;
    int32_t f = from[k], t = to[k];
    int32_t pf = atomicAdd(&fill[f], 1);
    int32_t pt = atomicAdd(&fill[t], 1);
    slot[soff[f] + 1 + pf] = make_int2(t, k);
    slot[soff[t] + 1 + pt] = make_int2(f, k);
}

__device__ __forceinline__ double2 series_admittance_rn(double r, double x) {
    double d = __dadd_rn(__dmul_rn(r, r), __dmul_rn(x, x));
    return make_double2(__ddiv_rn(r, d), __ddiv_rn(-x, d));
}

// Steps 1 to 3 for grids of at most kYbusSmallBuses buses in one workgroup, the
// counters in LDS: three launches fewer, and no atomics in memory.
constexpr int kYbusSmallBuses = 4096;  // 9241 buses: 38 us here, 15 us in four launches
__global__ __launch_bounds__(1024) void ybus_slots_small_kernel(
    int32_t n_bus, int32_t n_branch, const int32_t *__restrict__ from, const int32_t *__restrict__ to,
    const double *__restrict__ r, const double *__restrict__ x, int32_t *__restrict__ soff, int2 *__restrict__ slot,
    int32_t *__restrict__ err) {
    extern __shared__ int32_t at[];  // [n_bus] degree, then the next free slot of the row
    __shared__ int32_t part[1024 / kWave];
    __shared__ int bad;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    for (int32_t i = tid; i < n_bus; i += 1024) at[i] = 0;
    if (tid == 0) bad = 0;
    __syncthreads();
    for (int32_t e = tid; e < n_branch; e += 1024) {
        const int32_t f = from[e], t = to[e];
        if (f < 0 || f >= n_bus || t < 0 || t >= n_bus || f == t || (r[e] == 0.0 && x[e] == 0.0)) {
            atomicOr(&bad, 1);
        } else {
            atomicAdd(&at[f], 1);
            atomicAdd(&at[t], 1);
        }
    }
    __syncthreads();
    if (tid == 0) {
        err[0] = bad;
        err[1] = 0;  // longest row
    }
    if (bad) return;
    // exclusive scan of 1 + degree: each thread its contiguous rows
    const int32_t per = (n_bus + 1023) / 1024;
    const int32_t lo = min(tid * per, n_bus), hi = min(lo + per, n_bus);
    int32_t s = 0;
    for (int32_t i = lo; i < hi; ++i) s += at[i] + 1;
    int32_t incl = s;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int32_t y = __shfl_up(incl, o, kWave);
        if (lane >= o) incl += y;
    }
    if (lane == kWave - 1) part[wv] = incl;
    __syncthreads();
    int32_t run = incl - s;
    for (int k = 0; k < wv; ++k) run += part[k];
    for (int32_t i = lo; i < hi; ++i) {
        const int32_t d = at[i] + 1;
        soff[i] = run;
        slot[run] = make_int2(i, -1);  // diagonal
        at[i] = run + 1;
        run += d;
    }
    if (tid == 1023) soff[n_bus] = run;
    __syncthreads();
    for (int32_t e = tid; e < n_branch; e += 1024) {
        const int32_t f = from[e], t = to[e];
        slot[atomicAdd(&at[f], 1)] = make_int2(t, e);
        slot[atomicAdd(&at[t], 1)] = make_int2(f, e);
    }
}

// Rows of up to kYbusLocal slots are handled in registers and LDS (one column of it per
// thread), longer ones are sorted in place in memory.
constexpr int kYbusRows = 128;   // rows (threads) per workgroup of steps 4 and 6
constexpr int kYbusLocal = 16;

// insertion sort of slots [1, n) of a row (slot 0 is its diagonal) by key
template <typename Row, typename Key>
__device__ __forceinline__ void sort_slots(Row row, int32_t first, int32_t n, Key key) {
    for (int32_t p = first + 1; p < n; ++p) {
        const int2 v = row(p);
        int32_t q = p - 1;
        while (q >= first && key(row(q)) > key(v)) {
            row(q + 1) = row(q);
            --q;
        }
        row(q + 1) = v;
    }
}

// sum of the incident branches' diagonal terms, slots 1..n-1 in branch order
template <typename Row>
__device__ __forceinline__ double2 diag_sum(Row row, int32_t n, const double *__restrict__ r,
                                            const double *__restrict__ x, const double *__restrict__ b) {
    double2 acc = make_double2(0.0, 0.0);
    for (int32_t p = 1; p < n; ++p) {
        const int32_t e = row(p).y;
        const double2 y = series_admittance_rn(r[e], x[e]);
        acc.x = __dadd_rn(acc.x, y.x);
        acc.y = __dadd_rn(acc.y, __dadd_rn(y.y, __dmul_rn(b[e], 0.5)));
    }
    return acc;
}

// Step 4: distinct columns of every row, their exclusive scan within the workgroup's
// rows (uoff) and the workgroup's total, and the longest row (err[1]).  A long row is
// also brought into its final order here (by branch for the diagonal, which is summed
// in branch order, then stably by column).
__global__ __launch_bounds__(kYbusRows) void ybus_row_count_kernel(
    int32_t n_bus, const int32_t *__restrict__ soff, int2 *__restrict__ slot, const double *__restrict__ r,
    const double *__restrict__ x, const double *__restrict__ b, double2 *__restrict__ diag,
    int32_t *__restrict__ uoff, int32_t *__restrict__ total, int32_t *__restrict__ err) {
    __shared__ int32_t col[kYbusLocal][kYbusRows];
    __shared__ int32_t part[kYbusRows / kWave];
    if (err[0]) return;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int32_t i = blockIdx.x * kYbusRows + tid;
    int32_t u = 0;
    if (i < n_bus) {
        const int32_t lo = soff[i], n = soff[i + 1] - lo;
        if (n <= kYbusLocal) {
            for (int32_t p = 0; p < n; ++p) {
                const int32_t c = slot[lo + p].x;
                bool seen = false;
                for (int32_t q = 0; q < p; ++q) seen |= col[q][tid] == c;
                col[p][tid] = c;
                u += seen ? 0 : 1;
            }
        } else {
            auto row = [&](int32_t p) -> int2 & { return slot[lo + p]; };
            sort_slots(row, 0, n, [](int2 v) { return v.y; });  // by branch (diagonal slot has -1)
            diag[i] = diag_sum(row, n, r, x, b);
            sort_slots(row, 0, n, [](int2 v) { return v.x; });  // stable by column
            for (int32_t p = 0; p < n; ++p) u += p == 0 || row(p).x != row(p - 1).x ? 1 : 0;
        }
    }
    int32_t incl = u, mx = u;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int32_t y = __shfl_up(incl, o, kWave);
        if (lane >= o) incl += y;
        mx = max(mx, __shfl_xor(mx, o, kWave));
    }
    if (lane == kWave - 1) part[wv] = incl;
    if (lane == 0) atomicMax(&err[1], mx);
    __syncthreads();
    int32_t before = 0, sum = 0;
    for (int k = 0; k < kYbusRows / kWave; ++k) {
        before += k < wv ? part[k] : 0;
        sum += part[k];
    }
    if (i < n_bus) uoff[i] = before + incl - u;
    if (tid == 0) total[blockIdx.x] = sum;
}

// A row of n <= L slots, ranked in registers by branch and by (column, branch), its
// branch data all in flight at once: writes the merged entries from q on.  ly, lc: L
// LDS values of this thread, kYbusRows apart.
template <int L>
__device__ __forceinline__ void emit_short_row(int32_t i, int32_t lo, int32_t n, const int2 *__restrict__ slot,
                                               const double *__restrict__ r, const double *__restrict__ x,
                                               const double *__restrict__ b, double2 *ly, int32_t *lc, int32_t q,
                                               int32_t *__restrict__ col_idx, double2 *__restrict__ val) {
    int32_t c[L], e[L];
#pragma unroll
    for (int p = 0; p < L; ++p) {
        const int2 v = slot[lo + (p < n ? p : 0)];
        c[p] = p < n ? v.x : INT32_MAX;
        e[p] = p < n ? v.y : INT32_MAX;
    }
    double2 y[L];
    double bb[L];
    y[0] = make_double2(0.0, 0.0);
    if (n > 1) {
        double rr[L], xx[L];
#pragma unroll
        for (int p = 1; p < L; ++p) {
            const int32_t k = p < n ? e[p] : e[1];
            rr[p] = r[k];
            xx[p] = x[k];
            bb[p] = b[k];
        }
#pragma unroll
        for (int p = 1; p < L; ++p) y[p] = series_admittance_rn(rr[p], xx[p]);
    }
    // the diagonal: terms summed in branch order
#pragma unroll
    for (int p = 1; p < L; ++p) {
        int32_t rank = 0;
#pragma unroll
        for (int k = 0; k < L; ++k) rank += e[k] < e[p] ? 1 : 0;
        if (p < n) ly[rank * kYbusRows] = make_double2(y[p].x, __dadd_rn(y[p].y, __dmul_rn(bb[p], 0.5)));
    }
    double2 d = make_double2(0.0, 0.0);
    for (int32_t p = 1; p < n; ++p) {
        const double2 t = ly[p * kYbusRows];
        d.x = __dadd_rn(d.x, t.x);
        d.y = __dadd_rn(d.y, t.y);
    }
    y[0] = d;
    // entries by column, parallel branches in branch order
#pragma unroll
    for (int p = 0; p < L; ++p) {
        int32_t rank = 0;
#pragma unroll
        for (int k = 0; k < L; ++k) rank += c[k] < c[p] || (c[k] == c[p] && e[k] < e[p]) ? 1 : 0;
        if (p < n) {
            ly[rank * kYbusRows] = y[p];
            lc[rank * kYbusRows] = c[p];
        }
    }
    double2 acc = make_double2(0.0, 0.0);
    int32_t cur = -1;
    for (int32_t p = 0; p < n; ++p) {
        const int32_t cp = lc[p * kYbusRows];
        const double2 t = ly[p * kYbusRows];
        if (cp != cur) {
            if (cur >= 0) {
                col_idx[q] = cur;
                val[q] = acc;
                ++q;
            }
            cur = cp;
            acc = make_double2(0.0, 0.0);
        }
        if (cp == i) {
            acc = t;
        } else {
            acc.x = __dadd_rn(acc.x, -t.x);
            acc.y = __dadd_rn(acc.y, -t.y);
        }
    }
    col_idx[q] = cur;
    val[q] = acc;
}

// Step 6: per row, emit merged entries; parallel branches are summed in branch order.
// first: null, or the scanned workgroup totals; without it every workgroup adds up the
// totals before its own (up to kYbusSumTotals of them).  Bad flag, longest row and number
// of entries go to result; when the entries do not fit nnz_cap none is written.
constexpr int kYbusSumTotals = 2048;
__global__ __launch_bounds__(kYbusRows) void ybus_emit_kernel(
    int32_t n_bus, const int32_t *__restrict__ soff, const int2 *__restrict__ slot, const double *__restrict__ r,
    const double *__restrict__ x, const double *__restrict__ b, const double2 *__restrict__ diag,
    const int32_t *__restrict__ uoff, const int32_t *__restrict__ total, const int32_t *__restrict__ first,
    int32_t nnz_cap, int32_t *__restrict__ row_ptr, int32_t *__restrict__ col_idx, double2 *__restrict__ val,
    const int32_t *__restrict__ err, int32_t *__restrict__ result) {
    __shared__ double2 ly[kYbusLocal][kYbusRows];
    __shared__ int32_t lc[kYbusLocal][kYbusRows];
    __shared__ int32_t part[2][kYbusRows / kWave];
    if (err[0]) {
        if (blockIdx.x == 0 && threadIdx.x == 0) result[0] = 1;
        return;
    }
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int nblk = gridDim.x;
    int32_t before = 0, nnz = 0;
    if (first) {
        before = first[blockIdx.x];
        nnz = first[nblk];
    } else {
        for (int k = tid; k < nblk; k += kYbusRows) {
            const int32_t t = total[k];
            nnz += t;
            before += k < (int)blockIdx.x ? t : 0;
        }
        before = wave_isum(before);
        nnz = wave_isum(nnz);
        if (lane == 0) {
            part[0][wv] = before;
            part[1][wv] = nnz;
        }
        __syncthreads();
        before = nnz = 0;
        for (int k = 0; k < kYbusRows / kWave; ++k) {
            before += part[0][k];
            nnz += part[1][k];
        }
    }
    const int32_t i = blockIdx.x * kYbusRows + tid;
    if (blockIdx.x == 0 && tid == 0) {
        result[0] = 0;
        result[1] = err[1];
        result[2] = nnz;
        row_ptr[n_bus] = nnz;
    }
    if (i >= n_bus) return;
    int32_t q = before + uoff[i];
    row_ptr[i] = q;
    if (nnz > nnz_cap) return;
    const int32_t lo = soff[i], n = soff[i + 1] - lo;
    if (n <= kYbusLocal) {
        if (__ballot(n > kYbusLocal / 2) == 0)  // uniform: no row of the wave needs the wider form
            emit_short_row<kYbusLocal / 2>(i, lo, n, slot, r, x, b, &ly[0][tid], &lc[0][tid], q, col_idx, val);
        else
            emit_short_row<kYbusLocal>(i, lo, n, slot, r, x, b, &ly[0][tid], &lc[0][tid], q, col_idx, val);
        return;
    }
    for (int32_t p = 0; p < n;) {  // sorted by step 4
        const int32_t c = slot[lo + p].x;
        double2 acc = make_double2(0.0, 0.0);
        if (c == i) {
            acc = diag[i];
            while (p < n && slot[lo + p].x == c) ++p;
        } else {
            for (; p < n && slot[lo + p].x == c; ++p) {
                const int32_t e = slot[lo + p].y;
                const double2 y = series_admittance_rn(r[e], x[e]);
                acc.x = __dadd_rn(acc.x, -y.x);
                acc.y = __dadd_rn(acc.y, -y.y);
            }
        }
        col_idx[q] = c;
        val[q] = acc;
        ++q;
    }
}

}  // namespace dpf
