// Persistent DPF solve: one workgroup owns one work item (a case of a sub-grid)
// and runs the whole Adam iteration of Algorithm 1 for it inside the kernel.
//
// Why this shape on gfx950: a solve needs two grid-wide exchanges per
// iteration (the adjoint product needs every neighbour's residual seed, the next
// forward product needs every neighbour's updated voltage).  Keeping one item
// inside one workgroup turns both into LDS traffic plus workgroup barriers: the
// complex exchange vector X (16 B per bus) lives in LDS, so a sub-grid of up to
// ~10k buses fits in the 160 KB of one CU.  Converged items simply leave the
// kernel; the hardware dispatcher then starts the next item on that CU.
//
// Per iteration, for every bus i owned by the thread (i = lo + tid + k*NT):
//   A: I_i = sum_j Y_ij X_j (X = V) [- outage block];  dS_i = V_i conj(I_i) - S_i
//      r^P = [PV|PQ] Re dS, r^Q = [PQ] Im dS; loss and max|r| (workgroup reduce)
//      a_i = (2/m)(r^P + j r^Q); w_i = a_i conj(V_i); keep a_i I_i (the banded kernels
//      only Im(V_i conj(I_i)), see gradient_of_row)
//   stop test on max|r| (before the update, as the loop's convergence check)
//   B: h_i = sum_j Y_ij X_j (X = w; Y^T = Y) [- outage block]
//      G_i = a_i I_i + conj(h_i); g_vm = Re(conj(G) V)/vm at PQ; g_va = Im(G conj V)
//      Adam on the learnable entries; V_i = vm e^{j va}
// Where the state (vm, va, the moments) lives between iterations:
//   kReg        : in registers; up to 2048 buses with the matrix in LDS where it fits
//                 (team_solve_reg_kernel), 2049 to 4096 with the matrix read from L2
//                 (team_solve_resident_kernel)
//   kGlobal     : in the caller's arrays, streamed once per iteration (any size)
//   kBandStream : the same, with w in place over V in LDS (small bandwidths)
//   kPair       : as kBandStream, the state as three 16-byte pairs (pair.hpp)
// The register and resident kernels keep V and w in two LDS arrays (2 barriers per
// iteration); the others exchange through one.
#pragma once

#include "../../include/dpf.h"
#include "common.hpp"
#include "eval.hpp"
#include "sell.hpp"

#include <algorithm>

namespace dpf {

enum StoreMode {
    kReg = 0,         // state in registers (register and resident kernels)
    kGlobal = 1,      // streaming: state in global memory
    kBandStream = 2,  // banded, barrier-free gradient sweep
    kWide = 3,        // the multi-workgroup path for a whole call
    kPair = 4         // banded, state kept as (|V|, theta) and moment pairs
};
__host__ __device__ constexpr bool is_banded(int mode) { return mode == kBandStream || mode == kPair; }

constexpr int kSchedWords = 6;  // per-item schedule state, see SolveArgs::sched

struct SolveArgs {
    const int32_t *rp;
    const int32_t *ci;
    const double2 *yv;
    const int8_t *bt;
    const double2 *s_spec;
    int64_t s_ld;
    OutageView ov;
    double *vm;
    double *va;
    int64_t ld;
    double *st;          // Adam moments [4][B][ld]
    int64_t st_stride;   // B * ld
    int32_t st_fresh;    // moments start at zero
    double2 *scratch;    // streaming: [3][B][ld] complex (V, a*I, w)
    double *sched;       // [items][6] (t, lr, best, bad + cooldown * 2^20, b1^t, b2^t) or null
    const int32_t *sub_off;  // device [n_sub + 1] or null
    SellView sell;           // sliced-ELL copy of Y (local columns)
    const int32_t *sub_bw;   // [n_sub] largest |row - col| of the sub-grid's matrix (local indices)
    int32_t band_nt;         // > 0: sub-grids with sub_bw <= band_nt belong to the banded kernel
    int32_t team_cap;        // items above this size belong to the multi-workgroup path
    const int32_t *bad_grid; // set when a row exceeded the declared width bound
    int32_t handoff;         // > 0: tail handoff threshold in unfinished items (see handoff_due)
    int32_t total_items;     // items of the call
    int32_t *done_count;     // items finished so far (handoff only), cleared per call
    const int32_t *order;    // [items] item taken by workgroup k, or null: workgroup k takes item k
    int32_t n_bus;
    int32_t n_sub;
    int32_t B;
    int32_t lds_cap;     // complex entries available in dynamic LDS
    double lr, b1, b2, eps, tol;
    int32_t opt;  // DPF_OPT_*
    int32_t max_iter;
    int32_t sch;
    double factor;
    int32_t patience;
    double threshold;
    int32_t cooldown;
    double min_lr;
    double sched_eps;
    int32_t *iters;
    int32_t *status;
    double *mu_out;
    double *loss_out;
    int64_t *done_ns;         // per item: ns from the call's start stamp to completion, or null
    double *trace;            // per item [trace_len]: max|r| every trace_every iterations, or null
    int32_t trace_every, trace_len;
    const int64_t *stamp;     // wall clock at the start of the call
    double ns_per_tick;
};

// The kernel's SolveArgs (the first argument of every solve kernel) read from the
// kernel-argument segment where they are needed.  What an iteration uses once
// (optimizer, schedule, trace, stop test) is read this way: as ordinary arguments
// the compiler keeps all of them in scalar registers across the loops, spills 100 to
// 200 of those to vector lanes, and the FP64 constants end up in vector registers.
// (The one-row register kernels, whose iteration is one latency chain, take them as
// ordinary arguments: a 14-bus iteration is 6% longer otherwise.)
typedef const __attribute__((address_space(4))) SolveArgs ColdArgs;
__device__ __forceinline__ ColdArgs *cold_args() {
    ColdArgs *p = (ColdArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

template <int NT>
__device__ __forceinline__ void block_reduce2(double &s, double &m, double (*red)[NT / kWave]) {
    wave_last_sum_max(s, m);
    const int wv = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == kWave - 1) {
        red[0][wv] = s;
        red[1][wv] = m;
    }
}

template <int NT>
__device__ __forceinline__ void block_reduce2_finish(double &s, double &m, double (*red)[NT / kWave]) {
    s = 0.0;
    m = 0.0;
#pragma unroll
    for (int k = 0; k < NT / kWave; ++k) {
        s += red[0][k];
        m = fmax(m, red[1][k]);
    }
    s = uniform(s);  // every lane read the same partials
    m = uniform(m);
}

// Per-item step count and learning-rate schedule, kept across calls in
// SolveArgs::sched as {t, lr, best, bad + cooldown * 2^20, b1^t, b2^t}.
struct ItemSched {
    double t_step, lr, best, b1t, b2t;
    int bad, cool;
};

__device__ __forceinline__ ItemSched load_item_sched(const SolveArgs &a, int out_idx) {
    ItemSched s{0.0, a.lr, __longlong_as_double(0x7ff0000000000000LL), 1.0, 1.0, 0, 0};
    if (a.sched) {
        const double *ss = a.sched + kSchedWords * (int64_t)out_idx;
        s.t_step = ss[0];
        s.lr = ss[1];
        s.best = ss[2];
        const int packed = (int)ss[3];
        s.bad = packed & 0xFFFFF;
        s.cool = packed >> 20;
        s.b1t = ss[4];
        s.b2t = ss[5];
    }
    return s;
}

// scheduler step after an optimizer step (uniform across the workgroup; s.t_step
// already counts that step): PyTorch's reduce-on-plateau (mode min, relative
// threshold) or StepLR.  StepLR decays after every `patience`-th update of the
// item's persistent step count, so a call resumed from its schedule state keeps
// the phase of the decay (PyTorch's StepLR counts scheduler steps across epochs
// the same way).
template <typename A>
__device__ __forceinline__ void sched_step(A *p, ItemSched &s, double loss) {
    if (p->sch == DPF_SCHED_PLATEAU) {
        if (loss < s.best * (1.0 - p->threshold)) {
            s.best = loss;
            s.bad = 0;
        } else {
            s.bad += 1;
        }
        if (s.cool > 0) {
            s.cool -= 1;
            s.bad = 0;
        }
        if (s.bad > p->patience) {
            double nl = s.lr * p->factor;
            if (nl < p->min_lr) nl = p->min_lr;
            if (s.lr - nl > p->sched_eps) s.lr = nl;
            s.cool = p->cooldown;
            s.bad = 0;
        }
    } else if (p->sch == DPF_SCHED_STEP) {
        if (p->patience > 0 && ((int64_t)s.t_step % p->patience) == 0) s.lr = s.lr * p->factor;
    }
}

// the stop test of Algorithm 1, before an update: the item's status, or -1 to go on
template <typename A>
__device__ __forceinline__ int stop_status(A *p, double loss, double mu, int it) {
    if (!(isfinite(loss) && isfinite(mu))) return DPF_NONFINITE;
    if (mu < p->tol) return DPF_CONVERGED;
    return it >= p->max_iter ? DPF_MAX_ITER : -1;
}

// one more update: the step count and beta powers, and the update's scalars
template <typename A>
__device__ __forceinline__ OptStep begin_update(A *p, ItemSched &s) {
    s.t_step += 1.0;
    s.b1t *= p->b1;
    s.b2t *= p->b2;
    return opt_step(p->opt, s.lr, p->b1, p->b2, p->eps, 1.0 - s.b1t, 1.0 - s.b2t);
}

// Tail handoff.  Early retirement leaves the last items of a batch alone on
// their CUs, one workgroup each; once at most a.handoff items of the call are
// unfinished, the per-item kernels stop them (status kPaused, state in global
// memory, schedule in a.sched) and the host finishes them on the multi-workgroup
// path, which spreads every item over many CUs.  Checked every 32 iterations;
// thread 0 reads the counter and the decision reaches the workgroup through LDS.
__device__ __forceinline__ bool handoff_due(int it, int *flag) {
    ColdArgs *p = cold_args();
    if (p->handoff <= 0 || it == 0 || (it & 31) != 0) return false;
    if (threadIdx.x == 0)
        *flag = p->total_items - __hip_atomic_load(p->done_count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <=
                p->handoff;
    __syncthreads();
    return *flag != 0;
}

// optional trace of the stop-test quantity: max|r| of iteration `it` of this call
// (tested before its update) goes to slot it / trace_every when it is a multiple
// of trace_every and the slot exists; one thread writes (thread 0 of `writer`)
template <typename A>
__device__ __forceinline__ void trace_mu(A *p, bool writer, int out_idx, int it, double mu) {
    if (p->trace_len > 0 && writer && threadIdx.x == 0 && it % p->trace_every == 0 && it / p->trace_every < p->trace_len)
        p->trace[(int64_t)out_idx * p->trace_len + it / p->trace_every] = mu;
}

// per-item results and the schedule state, written by one thread
__device__ __forceinline__ void finish_item(int out_idx, int it, int stat, double mu, double loss,
                                            const ItemSched &s) {
    ColdArgs *p = cold_args();
    if (p->handoff > 0 && stat != kPaused) atomicAdd(p->done_count, 1);
    p->iters[out_idx] = it;
    p->status[out_idx] = stat;
    p->mu_out[out_idx] = mu;
    p->loss_out[out_idx] = loss;
    if (p->done_ns) p->done_ns[out_idx] = (int64_t)((double)(wall_clock64() - *p->stamp) * p->ns_per_tick);
    if (p->sched) {
        double *ss = p->sched + kSchedWords * (int64_t)out_idx;
        ss[0] = s.t_step;
        ss[1] = s.lr;
        ss[2] = s.best;
        ss[3] = (double)(s.bad + (s.cool << 20));
        ss[4] = s.b1t;
        ss[5] = s.b2t;
    }
}

// residual count m = n_pv + 2 n_pq of buses [lo, hi) (workgroup reduction)
template <int NT>
__device__ __forceinline__ double residual_count(const int8_t *__restrict__ bt, int lo, int hi,
                                                 double (*red)[NT / kWave]) {
    double cnt = 0.0, dummy = 0.0;
    for (int i = lo + (int)threadIdx.x; i < hi; i += NT) {
        const int8_t t = bt[i];
        cnt += t == kPQ ? 2.0 : (t == kPV ? 1.0 : 0.0);
    }
    block_reduce2<NT>(cnt, dummy, red);
    __syncthreads();
    block_reduce2_finish<NT>(cnt, dummy, red);
    __syncthreads();
    return cnt;
}

// the N-1 branch of case c as local bus indices and its pi-model blocks
// (of = ot = -1 when the case has no outage inside [lo, hi)); bad: the index is
// neither -1 nor a branch index, and the kernels leave the case alone (the call's
// prologue, outage_check_kernel, reports it)
struct Rank2 {
    int of, ot;
    double2 oy, oyd;
    bool bad;
};

__device__ __forceinline__ Rank2 outage_of_case(const OutageView &ov, int c, int lo, int hi) {
    Rank2 r{-1, -1, make_double2(0.0, 0.0), make_double2(0.0, 0.0), false};
    if (ov.outage) {
        const int32_t k = ov.outage[c];
        r.bad = outage_index_bad(k, ov.n_branch);
        if ((uint32_t)k < (uint32_t)ov.n_branch) {
            const int32_t f = ov.from[k], t = ov.to[k];
            if (f >= lo && f < hi && t >= lo && t < hi && f != t) {
                r.of = f - lo;
                r.ot = t - lo;
                double2 ysh;
                branch_admittance(ov.r[k], ov.x[k], ov.b[k], r.oy, ysh);
                r.oyd = cadd(r.oy, ysh);
            }
        }
    }
    return r;
}

// an index whose address arithmetic is re-derived where it is used instead of being
// hoisted out of the iterations and kept live
__device__ __forceinline__ uint32_t opaque_index(uint32_t i) {
    asm volatile("" : "+v"(i));
    return i;
}

// Register-resident kernel: a thread owns rows tid + k*NT, k < K, and keeps their
// whole state in registers for the solve; V and w are separate LDS arrays, two
// barriers per iteration.
//
// What bounds it: with one row per thread (small grids) the latency of one
// iteration's dependent chain, with more the FP64 issue of the one CU that runs the
// item.  Both are served by the same choices:
//  - the item's matrix entries sit in LDS behind V and w (values 16 B, columns as
//    16-bit LDS offsets; the offsets of a row's first kRegCols entries even in
//    registers), so a row product is one round trip to LDS instead of a chain of
//    scalar load, L1/L2 load and LDS gather.  A matrix that does not fit is read
//    from the sliced-ELL copy in global memory (the host asks for at most
//    kRegLdsPerThread bytes per thread, the share that leaves room for as many
//    workgroups as the registers allow);
//  - cos and sin of a row's angle stay in registers, so V, w and both gradients need
//    no second sincos and no division by |V|;
//  - the stop test does not stand between the two products: the reduction's partials
//    are read after the gradient sweep has formed every gradient, and only the update
//    waits for the decision;
//  - the updates of |V| and theta run side by side (coordinates that are not
//    learnable keep their value by a select), their two division chains overlapped.
//  - a single grid's rows are sorted by length (sell_sort_rows), so slices carry next
//    to no padding in any numbering.
// Measured on an MI355X, us per iteration (the difference of calls of 50 and 250), the
// form before (matrix from L2, updates one after the other behind the stop test) -> this
// one: 14 buses x 1 case 2.3 -> 1.3; 118 x 2048 6.7 -> 4.1; 250 x 1024 6.6 -> 4.2;
// 900 x 512 12.7 -> 7.0; 1354 x 64 7.6 -> 5.1 (8.8 -> 5.1 in an arbitrary numbering);
// 1950 x 64 11.5 -> 8.0.
// At three rows per thread the columns and injections are re-read instead of kept
// (both kept: 94 spilled registers and no gain); at four the matrix stays in global memory
// (V, w and a 2048-row matrix exceed the LDS).  1024 threads with two rows each spill
// 150 registers (twice the time for 1354 x 64).
constexpr int kRegCols = 8;           // columns of a row kept in registers
constexpr int kRegLdsRows = 3;        // rows per thread up to which the matrix goes to LDS
constexpr int kRegLdsPerThread = 320; // bytes: 160 KB over the 512 threads two waves per SIMD make

// dynamic LDS of one register-kernel workgroup in 16-byte units: V and w of n_max rows
// and room for `entries` matrix entries (18 B each, whole slices), at most the share
// of its threads
inline int32_t reg_lds_units(int nt, int32_t n_max, int64_t entries, int32_t lds_units) {
    const int64_t share = std::max<int64_t>(2 * (int64_t)n_max, (int64_t)nt * kRegLdsPerThread / 16 - 32);
    return (int32_t)std::max<int64_t>(
        1, std::min<int64_t>(2 * (int64_t)n_max + (entries * 9 + 7) / 8, std::min<int64_t>(share, lds_units)));
}

//
// MANY: calls of many sub-grids well below the largest.  The row loops skip what a wave
// has no row for (a scalar branch per row); without that an item of one row per thread
// pays the updates of all K.  us of 40 iterations, plain -> skipping: the largest of 2000
// buses and 199 of up to 500, 4 cases 901 -> 592; 1500 and up to 375 716 -> 478; 300 and up
// to 75, 300 grids 404 -> 331.  Where every item has all rows, or the call ends with its
// largest item, the branches cost: 2000 buses and 99 to 399 of 100, 100 iterations
// 1030..1051 -> 1077..1092 (599 of them 1516 -> 1112); 1000 and 299 of 1000, 2 cases
// 2493 -> 2534 (of 700 1212 -> 1117).  The line lies at two items per CU and a mean size of
// three quarters of the largest (2000 and 299 of 1500: 4422 -> 4365, 500 and 399 of 400:
// 878 -> 901).
template <int NT, int K, bool MANY = false>
__global__ __launch_bounds__(NT) void team_solve_reg_kernel(SolveArgs a) {
    extern __shared__ double2 X[];
    __shared__ double red[2][NT / kWave];
    constexpr int NW = NT / kWave;
    auto args = [&]() {
        if constexpr (K == 1) return &a;
        else return cold_args();
    };

    const int tid = threadIdx.x;
    const int item = a.order ? a.order[blockIdx.x] : (int)blockIdx.x;
    const int sidx = item / a.B;
    const int c = item - sidx * a.B;
    const int lo = a.sub_off ? a.sub_off[sidx] : 0;
    const int hi = a.sub_off ? a.sub_off[sidx + 1] : a.n_bus;
    const int n = hi - lo;
    const int out_idx = c * a.n_sub + sidx;
    if (n > a.team_cap) return;  // handled by the multi-workgroup path
    if (a.band_nt > 0 && a.sub_bw[sidx] <= a.band_nt) return;  // handled by the banded kernel
    if (n < 0 || n > NT * K || 2 * n > a.lds_cap || *a.bad_grid) {  // see DPF_BAD_GRID
        if (tid == 0) {
            a.status[out_idx] = DPF_BAD_GRID;
            a.iters[out_idx] = 0;
        }
        return;
    }
    const int lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int slice0 = a.sell.slice_off[sidx];
    const int ns = (n + kWave - 1) / kWave;

    // step count and schedule (a resumed solve continues them)
    ItemSched sc = load_item_sched(a, out_idx);

    const double m_res = residual_count<NT>(a.bt, lo, hi, red);
    const double two_over_m = m_res > 0.0 ? 2.0 / m_res : 0.0;

    // N-1 outage of this case (only meaningful for a single sub-grid)
    const Rank2 r2 = outage_of_case(a.ov, c, lo, hi);
    if (r2.bad) return;  // reported by the call's prologue
    // LDS and slices go by slot, the caller's arrays by row
    const int of = r2.of >= 0 && a.sell.slot ? a.sell.slot[r2.of] : r2.of;
    const int ot = r2.ot >= 0 && a.sell.slot ? a.sell.slot[r2.ot] : r2.ot;
    const double2 oy = r2.oy, oyd = r2.oyd;

    const int64_t cb = (int64_t)c * a.ld + lo;
    const int64_t sb = (int64_t)c * a.s_ld + lo;
    double *vm_c = a.vm + cb;
    double *va_c = a.va + cb;
    double *mv_c = a.st + cb;
    double *ma_c = a.st + a.st_stride + cb;
    double *sv_c = a.st + 2 * a.st_stride + cb;
    double *sa_c = a.st + 3 * a.st_stride + cb;

    // LDS: V [n], w [n], matrix values [cap], matrix columns [cap] (byte offsets, 16 bit)
    char *lds = reinterpret_cast<char *>(X);
    double2 *Xv = X;
    const int wofs = n * 16;  // byte offset of w
    double2 *MV = X + 2 * n;
    const int cap = ((a.lds_cap - 2 * n) * 8 / 9) & ~(kWave - 1);
    uint16_t *MC = reinterpret_cast<uint16_t *>(MV + cap);
    const int e0 = a.sell.start[slice0];  // units of 64 entries
    const int64_t base0 = (int64_t)e0 * kWave;
    if constexpr (K <= kRegLdsRows) {
        const int tot = min((a.sell.start[slice0 + ns] - e0) * kWave, cap);
        for (int e = tid; e < tot; e += NT) {
            MV[e] = a.sell.val[base0 + e];
            MC[e] = (uint16_t)(a.sell.col[base0 + e] * 16);
        }
    }

    // the rows of this thread: slot tid + k*NT is lane `lane` of slice wv + k*NW
    int row[K];
    int wd[K], mo[K];  // slice width (0: no such slice) and first entry
    constexpr bool SREG = K <= 2;  // else the injections are re-read (L2) each iteration
    double2 S[SREG ? K : 1], aI[K];
    double vm[K], va[K], mv[K], ma[K], sv[K], sa[K], cs[K], sn[K];
    uint32_t pq = 0, fre = 0;  // bit k: row k is PQ / not the slack
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int j = wv + k * NW;
        const int il = tid + k * NT;
        row[k] = il < n && a.sell.row ? a.sell.row[il] : il;
        wd[k] = j < ns ? a.sell.width[slice0 + j] : 0;
        mo[k] = j < ns ? (a.sell.start[slice0 + j] - e0) * kWave : 0;
        if constexpr (SREG) S[k] = make_double2(0.0, 0.0);
        aI[k] = make_double2(0.0, 0.0);
        vm[k] = va[k] = mv[k] = ma[k] = sv[k] = sa[k] = sn[k] = 0.0;
        cs[k] = 1.0;
        if (il < n) {
            const int8_t t = a.bt[lo + row[k]];
            pq |= (t == kPQ ? 1u : 0u) << k;
            fre |= (t != kSlack ? 1u : 0u) << k;
            vm[k] = vm_c[row[k]];
            va[k] = va_c[row[k]];
            if constexpr (SREG) S[k] = a.s_spec[sb + row[k]];
            if (!a.st_fresh) {
                mv[k] = mv_c[row[k]];
                ma[k] = ma_c[row[k]];
                sv[k] = sv_c[row[k]];
                sa[k] = sa_c[row[k]];
            }
        }
    }
    // cos and sin of every row's angle and V to LDS: near zero for all rows at once, then
    // the rows of other angles, if the wave has any, one at a time in one rolled loop (the
    // general reduction inlined once instead of once per row)
    auto has_row = [&](int k) { return wv * kWave + k * NT < n; };  // this wave, MANY
    auto publish = [&]() {
        bool far = false;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if constexpr (MANY)
                if constexpr (MANY)
                    if (!has_row(k)) break;
            near_sincos(va[k], sn[k], cs[k]);
            far |= !angle_is_near(va[k]);
        }
        if (__ballot(far) != 0) {
#pragma unroll 1
            for (int r = 0; r < K; ++r) {
                double x = va[0], s1, c1;
#pragma unroll
                for (int k = 1; k < K; ++k) x = r == k ? va[k] : x;
                fast_sincos(x, s1, c1);
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    sn[k] = r == k ? s1 : sn[k];
                    cs[k] = r == k ? c1 : cs[k];
                }
            }
        }
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (tid + k * NT < n) Xv[tid + k * NT] = make_double2(vm[k] * cs[k], vm[k] * sn[k]);
    };
    publish();
    __syncthreads();

    int it = 0, stat = DPF_MAX_ITER;
    double mu = 0.0, loss = 0.0;
    // the iterations, with the matrix in LDS or read from the sliced-ELL copy
    auto iterate = [&](auto in_lds) {
        constexpr bool LDSM = decltype(in_lds)::value;
        constexpr int COLS = K <= 2 ? kRegCols : 0;
        uint32_t ccol[K][LDSM && COLS > 0 ? COLS / 2 : 1];
        if constexpr (LDSM && COLS > 0) {
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int q = 0; q < COLS; q += 2) {
                    const uint32_t c0 = q < wd[k] ? (uint32_t)MC[mo[k] + q * kWave + lane] : 0u;
                    const uint32_t c1 = q + 1 < wd[k] ? (uint32_t)MC[mo[k] + (q + 1) * kWave + lane] : 0u;
                    ccol[k][q / 2] = c0 | (c1 << 16);
                }
        }
        auto at = [&](int ofs) -> double2 { return *reinterpret_cast<const double2 *>(lds + ofs); };
        // row k of Y z, z at byte offset zo of the LDS
        auto product = [&](int k, int zo) {
            double2 acc = make_double2(0.0, 0.0);
            const int w = wd[k];
            if constexpr (LDSM) {
                // entries Q .. Q+N-1 at once; N is the whole row where one row per thread
                // leaves the registers, else 4
                constexpr int G = K == 1 ? kRegCols : 4;
                const double2 *mvp = MV + mo[k] + lane;
                auto group = [&](auto first, auto count) {
                    constexpr int Q = decltype(first)::value, N = decltype(count)::value;
                    double2 v[N], z[N];
#pragma unroll
                    for (int u = 0; u < N; ++u) {
                        v[u] = mvp[(Q + u) * kWave];
                        if constexpr (COLS > 0) {
                            const uint32_t pk = ccol[k][(Q + u) / 2];
                            z[u] = at(zo + (int)(((Q + u) & 1) ? pk >> 16 : pk & 0xffffu));
                        } else {
                            z[u] = at(zo + MC[mo[k] + (Q + u) * kWave + lane]);
                        }
                    }
#pragma unroll
                    for (int u = 0; u < N; ++u) acc = cfma(v[u], z[u], acc);
                };
                auto groups = [&](auto first, int left) {
#define DPF_GROUP(N) \
    case N: group(first, std::integral_constant<int, N>{}); break;
                    switch (min(left, G)) {
                        DPF_GROUP(1) DPF_GROUP(2) DPF_GROUP(3) DPF_GROUP(4)
                        default:
                            if constexpr (G > 4) {
                                switch (min(left, G)) {
                                    DPF_GROUP(5) DPF_GROUP(6) DPF_GROUP(7) DPF_GROUP(8)
                                    default: break;
                                }
                            }
                    }
#undef DPF_GROUP
                };
                groups(std::integral_constant<int, 0>{}, w);
                if constexpr (G < kRegCols)
                    if (w > G) groups(std::integral_constant<int, G < kRegCols ? G : 0>{}, w - G);
#pragma unroll 1
                for (int q = kRegCols; q < w; ++q)
                    acc = cfma(mvp[q * kWave], at(zo + MC[mo[k] + q * kWave + lane]), acc);
            } else {
                const int own = max(min(tid + k * NT, n - 1), 0);
                acc = sell_row<4, true>(a.sell.val + base0, a.sell.col + base0, mo[k] + lane, w, own,
                                        [&](int j) { return at(zo + j * 16); }, acc);
            }
            if (of >= 0) {
                const int il = tid + k * NT;
                const double2 zf = at(zo + of * 16), zt = at(zo + ot * 16);
                if (il == of) acc = csub(acc, csub(cmul(oyd, zf), cmul(oy, zt)));
                else if (il == ot) acc = csub(acc, csub(cmul(oyd, zt), cmul(oy, zf)));
            }
            return acc;
        };

        for (;; ++it) {
            // this iteration's optimizer scalars, off the chain of the products
            ItemSched nx = sc;
            const OptStep os = begin_update(args(), nx);

            // ---------------- A: forward product, residual, loss, seed
            double lsum = 0.0, lmax = 0.0;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int il = tid + k * NT;
                if constexpr (MANY)
                    if (!has_row(k)) break;
                double2 sp = make_double2(0.0, 0.0);
                if constexpr (SREG) sp = S[k];
                else if (il < n) sp = a.s_spec[sb + opaque_index(row[k])];
                const double2 acc = product(k, 0);
                const double2 v = make_double2(vm[k] * cs[k], vm[k] * sn[k]);
                const double2 d = csub(cmulc(v, acc), sp);
                const double rP = (fre >> k) & 1u ? d.x : 0.0;
                const double rQ = (pq >> k) & 1u ? d.y : 0.0;
                lsum += rP * rP + rQ * rQ;
                lmax = fmax(lmax, fmax(fabs(rP), fabs(rQ)));
                const double2 av = make_double2(two_over_m * rP, two_over_m * rQ);
                aI[k] = cmul(av, acc);
                // w = av conj(v), scaled after the product: the same cost as before it, another
                // rounding.  The step at which a solve of thousands of steps meets its tolerance
                // hangs on such roundings (the oracle's own does, under 1e-16 changes of its
                // inputs), so the order stays as the tests of such solves were run with
                if (il < n) *reinterpret_cast<double2 *>(lds + wofs + il * 16) = cscale(two_over_m, cmulc(make_double2(rP, rQ), v));
            }
            if constexpr (NW > 1) block_reduce2<NT>(lsum, lmax, red);
            __syncthreads();
            if constexpr (NW == 1) {  // one wave: its last lane holds the item's sums
                wave_last_sum_max(lsum, lmax);
                lsum = read_lane(lsum, kWave - 1);
                lmax = read_lane(lmax, kWave - 1);
            }

            // ---------------- B: adjoint product and gradients (they change no state yet)
            double gv[K], ga[K];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if constexpr (MANY)
                    if (!has_row(k)) break;
                const double2 h = product(k, wofs);
                const double2 G = make_double2(aI[k].x + h.x, aI[k].y - h.y);
                gv[k] = grad_vm(G, cs[k], sn[k], vm[k]);
                ga[k] = vm[k] * (G.y * cs[k] - G.x * sn[k]);
            }
            if constexpr (NW > 1) block_reduce2_finish<NT>(lsum, lmax, red);
            loss = m_res > 0.0 ? lsum / m_res : 0.0;
            mu = isnan(lsum) ? lsum : lmax;
            trace_mu(args(), true, out_idx, it, mu);
            const int stop = stop_status(args(), loss, mu, it);
            if (stop >= 0) {
                stat = stop;
                break;
            }

            // ---------------- update; the moments of a coordinate that is not learnable are
            // never written back
            sc = nx;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if constexpr (MANY)
                    if (!has_row(k)) break;
                double vmn = vm[k], van = va[k];
                opt_update2(os, vmn, gv[k], mv[k], sv[k], van, ga[k], ma[k], sa[k]);
                vm[k] = (pq >> k) & 1u ? vmn : vm[k];
                va[k] = (fre >> k) & 1u ? van : va[k];
            }
            publish();
            sched_step(args(), sc, loss);
            __syncthreads();
        }
    };
    if (K <= kRegLdsRows && (a.sell.start[slice0 + ns] - e0) * kWave <= cap) iterate(std::bool_constant<(K <= kRegLdsRows)>{});
    else iterate(std::false_type{});

    // ---------------- write back
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if ((pq >> k) & 1u) {
            vm_c[row[k]] = vm[k];
            if (!a.st_fresh) {
                mv_c[row[k]] = mv[k];
                sv_c[row[k]] = sv[k];
            }
        }
        if ((fre >> k) & 1u) {
            va_c[row[k]] = va[k];
            if (!a.st_fresh) {
                ma_c[row[k]] = ma[k];
                sa_c[row[k]] = sa[k];
            }
        }
    }
    if (tid == 0) finish_item(out_idx, it, stat, mu, loss, sc);
}

// Resident kernel for sub-grids of 2049 to 4096 buses: the state of every row (|V|,
// theta and the four moments) and a*I stay in registers as in the register kernel, V
// and w are separate LDS arrays, and everything else is read where it is needed: the
// matrix (rows sorted by length) and the injections from L2, a row's own V from LDS.
// The streaming kernel moves 176 B of state per bus and iteration through L2 and the
// Infinity Cache (5.4 TB/s at 256 cases of 3000 buses, its bound); this one moves none
// and is bound by the latency of its row products (two waves per SIMD, about half of
// the FP64 issue used).  us per iteration, streaming -> this, 256 cases in an arbitrary
// numbering: 2500 buses 19.5 -> 12.0, 3000 23.4 -> 13.0, 4000 30.9 -> 19.8 (8 rows per
// thread; a*I in global memory).  Calls of 60 iterations of 256 x 3000, us per iteration
// with the call's fixed cost: 14.6; 1024 threads, which spill 30 to 120 registers, 15.0 at
// best; gathers of a group of four one at a time 17.1 instead of together; groups of 6 or 8
// 16.1, 17.5.
template <int NT, int K>
__global__ __launch_bounds__(NT) void team_solve_resident_kernel(SolveArgs a) {
    extern __shared__ double2 X[];
    __shared__ double red[2][NT / kWave];
    constexpr int NW = NT / kWave;

    const int tid = threadIdx.x;
    const int item = a.order ? a.order[blockIdx.x] : (int)blockIdx.x;
    const int sidx = item / a.B;
    const int c = item - sidx * a.B;
    const int lo = a.sub_off ? a.sub_off[sidx] : 0;
    const int hi = a.sub_off ? a.sub_off[sidx + 1] : a.n_bus;
    const int n = hi - lo;
    const int out_idx = c * a.n_sub + sidx;
    if (n > a.team_cap) return;  // handled by the multi-workgroup path
    if (a.band_nt > 0 && a.sub_bw[sidx] <= a.band_nt) return;  // handled by the banded kernel
    if (n < 0 || n > NT * K || 2 * n > a.lds_cap || *a.bad_grid) {  // see DPF_BAD_GRID
        if (tid == 0) {
            a.status[out_idx] = DPF_BAD_GRID;
            a.iters[out_idx] = 0;
        }
        return;
    }
    const int lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int slice0 = a.sell.slice_off[sidx];
    const int ns = (n + kWave - 1) / kWave;
    ItemSched sc = load_item_sched(a, out_idx);
    const double m_res = residual_count<NT>(a.bt, lo, hi, red);
    const double two_over_m = m_res > 0.0 ? 2.0 / m_res : 0.0;
    const Rank2 r2 = outage_of_case(a.ov, c, lo, hi);
    if (r2.bad) return;  // reported by the call's prologue
    // LDS and slices go by slot, the caller's arrays by row
    const int of = r2.of >= 0 && a.sell.slot ? a.sell.slot[r2.of] : r2.of;
    const int ot = r2.ot >= 0 && a.sell.slot ? a.sell.slot[r2.ot] : r2.ot;
    const double2 oy = r2.oy, oyd = r2.oyd;

    const int64_t cb = (int64_t)c * a.ld + lo;
    double *__restrict__ vm_c = a.vm + cb;
    double *__restrict__ va_c = a.va + cb;
    double *__restrict__ st_c = a.st + cb;
    const int64_t stride = a.st_stride;
    const double2 *__restrict__ Sc = a.s_spec + (int64_t)c * a.s_ld + lo;
    const double2 *__restrict__ sval = a.sell.val;
    const int32_t *__restrict__ scol = a.sell.col;
    double2 *Xv = X, *Xw = X + n;
    // a*I between the sweeps: a third LDS array where it fits, else the scratch
    const bool aI_lds = 3 * n <= a.lds_cap;
    double2 *Xa = X + 2 * n;
    double2 *__restrict__ aIg = a.scratch + cb;

    double vm[K], va[K], mv[K], ma[K], sv[K], sa[K];
    uint32_t pq = 0, fre = 0;  // bit k: row k is PQ / not the slack
    int row[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int il = tid + k * NT;
        row[k] = il < n && a.sell.row ? a.sell.row[il] : il;
        vm[k] = va[k] = mv[k] = ma[k] = sv[k] = sa[k] = 0.0;
        if (il < n) {
            const int r = row[k];
            const int8_t t = a.bt[lo + r];
            pq |= (t == kPQ ? 1u : 0u) << k;
            fre |= (t != kSlack ? 1u : 0u) << k;
            vm[k] = vm_c[r];
            va[k] = va_c[r];
            if (!a.st_fresh) {
                mv[k] = st_c[r];
                ma[k] = st_c[stride + r];
                sv[k] = st_c[2 * stride + r];
                sa[k] = st_c[3 * stride + r];
            }
        }
    }
    // V of row k to LDS, right for angles near zero; the rows of other angles, if the wave
    // has any, follow one at a time in one rolled loop (see the register kernel)
    bool far = false;
    auto publish = [&](int k, int il) {
        double sn, cs;
        near_sincos(va[k], sn, cs);
        far |= !angle_is_near(va[k]);
        if (il < n) Xv[il] = make_double2(vm[k] * cs, vm[k] * sn);
    };
    auto publish_far = [&]() {
        if (__ballot(far) != 0) {
#pragma unroll 1
            for (int r = 0; r < K; ++r) {
                double x = va[0], m = vm[0], sn, cs;
#pragma unroll
                for (int k = 1; k < K; ++k) {
                    x = r == k ? va[k] : x;
                    m = r == k ? vm[k] : m;
                }
                fast_sincos(x, sn, cs);
                if (tid + r * NT < n) Xv[tid + r * NT] = make_double2(m * cs, m * sn);
            }
        }
        far = false;
    };
#pragma unroll
    for (int k = 0; k < K; ++k) publish(k, tid + k * NT);
    publish_far();
    __syncthreads();

    // row of slot il (slice j = wv + k*NW of the sub-grid, 0 entries past the last one)
    auto product = [&](int k, int il, const double2 *Z) {
        const int j = wv + k * NW;
        double2 acc = make_double2(0.0, 0.0);
        if (j < ns)
            acc = sell_row<4, true>(sval, scol, a.sell.start[slice0 + j] * kWave + lane, a.sell.width[slice0 + j],
                                    min(il, n - 1), [&](int q) { return Z[q]; }, acc);
        if (of >= 0) {
            if (il == of) acc = csub(acc, csub(cmul(oyd, Z[of]), cmul(oy, Z[ot])));
            else if (il == ot) acc = csub(acc, csub(cmul(oyd, Z[ot]), cmul(oy, Z[of])));
        }
        return acc;
    };

    int it = 0, stat = DPF_MAX_ITER;
    double mu = 0.0, loss = 0.0;
    for (;; ++it) {
        // ---------------- A
        double lsum = 0.0, lmax = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int il = (int)opaque_index(tid + k * NT);
            double2 sp = make_double2(0.0, 0.0), v = make_double2(0.0, 0.0);
            if (il < n) {
                sp = Sc[opaque_index(row[k])];
                v = Xv[il];
            }
            const double2 acc = product(k, il, Xv);
            const double2 d = csub(cmulc(v, acc), sp);
            const double rP = (fre >> k) & 1u ? d.x : 0.0;
            const double rQ = (pq >> k) & 1u ? d.y : 0.0;
            lsum += rP * rP + rQ * rQ;
            lmax = fmax(lmax, fmax(fabs(rP), fabs(rQ)));
            const double2 av = make_double2(two_over_m * rP, two_over_m * rQ);
            const double2 ai = cmul(av, acc);
            if (il < n) {
                Xw[il] = cmulc(av, v);
                if (aI_lds) Xa[il] = ai;
                else aIg[il] = ai;
            }
        }
        block_reduce2<NT>(lsum, lmax, red);
        __syncthreads();
        block_reduce2_finish<NT>(lsum, lmax, red);
        loss = m_res > 0.0 ? lsum / m_res : 0.0;
        mu = isnan(lsum) ? lsum : lmax;
        trace_mu(cold_args(), true, out_idx, it, mu);
        const int stop = stop_status(cold_args(), loss, mu, it);
        if (stop >= 0) {
            stat = stop;
            break;
        }

        // ---------------- B
        const OptStep os = begin_update(cold_args(), sc);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int il = (int)opaque_index(tid + k * NT);
            double2 ai = make_double2(0.0, 0.0), v = make_double2(0.0, 0.0);
            if (il < n) {
                v = Xv[il];
                if (aI_lds) ai = Xa[il];
                else ai = aIg[il];
            }
            const double2 h = product(k, il, Xw);
            const double2 G = make_double2(ai.x + h.x, ai.y - h.y);
            const double gv = (G.x * v.x + G.y * v.y) / vm[k];
            const double ga = G.y * v.x - G.x * v.y;
            const double vmn = opt_update(os, vm[k], gv, mv[k], sv[k]);
            asm volatile("" ::: "memory");  // one update after the other: 26 spilled registers fewer
            const double van = opt_update(os, va[k], ga, ma[k], sa[k]);
            vm[k] = (pq >> k) & 1u ? vmn : vm[k];
            va[k] = (fre >> k) & 1u ? van : va[k];
            publish(k, il);
        }
        publish_far();
        sched_step(cold_args(), sc, loss);
        __syncthreads();
    }

    // ---------------- write back (the moments of learnable coordinates only)
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int r = row[k];
        if ((pq >> k) & 1u) {
            vm_c[r] = vm[k];
            if (!a.st_fresh) {
                st_c[r] = mv[k];
                st_c[2 * stride + r] = sv[k];
            }
        }
        if ((fre >> k) & 1u) {
            va_c[r] = va[k];
            if (!a.st_fresh) {
                st_c[stride + r] = ma[k];
                st_c[3 * stride + r] = sa[k];
            }
        }
    }
    if (tid == 0) finish_item(out_idx, it, stat, mu, loss, sc);
}

// Streaming variant for large sub-grids.  Every per-bus value lives in global
// memory (the caller's vm/va/Adam arrays and the scratch arrays a*I and w) and
// is streamed once per iteration, with a runtime loop over any number of buses
// per thread.  With the single-buffered LDS exchange, w goes through the scratch
// array W and the new V is rebuilt from |V| and theta (both L2-resident), which
// keeps the register count low enough for 1024-thread workgroups; the per-bus
// address arithmetic is re-derived inside the iteration (opaque_index) instead
// of being kept live.
template <int NT>
__global__ __launch_bounds__(NT) void team_solve_stream_kernel(SolveArgs a) {
    extern __shared__ double2 X[];
    __shared__ double red[2][NT / kWave];

    const int tid = threadIdx.x;
    const int item = a.order ? a.order[blockIdx.x] : (int)blockIdx.x;
    const int sidx = item / a.B;
    const int c = item - sidx * a.B;
    const int lo = a.sub_off ? a.sub_off[sidx] : 0;
    const int hi = a.sub_off ? a.sub_off[sidx + 1] : a.n_bus;
    const int n = hi - lo;
    const int out_idx = c * a.n_sub + sidx;
    if (n > a.team_cap) return;  // handled by the multi-workgroup path
    if (a.band_nt > 0 && a.sub_bw[sidx] <= a.band_nt) return;  // handled by the banded kernel
    if (n < 0 || n > a.lds_cap || *a.bad_grid) {  // see DPF_BAD_GRID
        if (tid == 0) {
            a.status[out_idx] = DPF_BAD_GRID;
            a.iters[out_idx] = 0;
        }
        return;
    }
    const int slice0 = a.sell.slice_off[sidx];
    const int lane = tid & (kWave - 1);
    const bool dbl = 2 * n <= a.lds_cap;
    double2 *Xv = X;
    double2 *Xw = dbl ? X + n : X;

    // step count and schedule (a resumed solve continues them)
    ItemSched sc = load_item_sched(a, out_idx);

    const double m_res = residual_count<NT>(a.bt, lo, hi, red);
    const double two_over_m = m_res > 0.0 ? 2.0 / m_res : 0.0;

    // N-1 outage of this case (only meaningful for a single sub-grid)
    const Rank2 r2 = outage_of_case(a.ov, c, lo, hi);
    if (r2.bad) return;  // reported by the call's prologue
    const int of = r2.of, ot = r2.ot;
    const double2 oy = r2.oy, oyd = r2.oyd;

    const int64_t cb = (int64_t)c * a.ld;
    const int64_t sb = (int64_t)c * a.s_ld;
    double2 *__restrict__ Wg = a.scratch + 2 * a.st_stride + cb;
    double *__restrict__ vm_c = a.vm + cb;
    double *__restrict__ va_c = a.va + cb;
    double *__restrict__ mv_c = a.st + cb;
    double *__restrict__ ma_c = a.st + a.st_stride + cb;
    double *__restrict__ sv_c = a.st + 2 * a.st_stride + cb;
    double *__restrict__ sa_c = a.st + 3 * a.st_stride + cb;
    double2 *__restrict__ aIg = a.scratch + a.st_stride + cb;
    const double2 *__restrict__ Sc = a.s_spec + sb;
    const int32_t *__restrict__ swidth = a.sell.width;
    const int32_t *__restrict__ sstart = a.sell.start;
    const int32_t *__restrict__ scol = a.sell.col;
    const double2 *__restrict__ sval = a.sell.val;
    const int8_t *__restrict__ btp = a.bt;

    for (int i = lo + tid; i < hi; i += NT) {
        double sn, cs;
        const double vmi = vm_c[i];
        fast_sincos(va_c[i], sn, cs);
        const double2 v = make_double2(vmi * cs, vmi * sn);
        Xv[i - lo] = v;
        if (a.st_fresh) {
            mv_c[i] = 0.0;
            ma_c[i] = 0.0;
            sv_c[i] = 0.0;
            sa_c[i] = 0.0;
        }
    }
    __syncthreads();

    // bus loop of one phase
#define DPF_BUS_LOOP_BEGIN                                               \
    for (int kk = 0;; ++kk) {                                            \
        const uint32_t i = opaque_index((uint32_t)(lo + tid + kk * NT)); \
        if ((int)i >= hi) break;                                         \
        {
#define DPF_BUS_LOOP_END \
    }                    \
    }

    int it = 0, stat = DPF_MAX_ITER;
    double mu = 0.0, loss = 0.0;
    __shared__ int pause_flag;
    for (;; ++it) {
        if (handoff_due(it, &pause_flag)) {
            stat = kPaused;
            break;
        }
        // ---------------- phase A
        double lsum = 0.0, lmax = 0.0;
        DPF_BUS_LOOP_BEGIN
                const int il = (int)i - lo;
                // global loads of this bus first, so that they overlap the gather below
                const int8_t tk = btp[i];
                const double2 sp = Sc[i];
                const int gsl = __builtin_amdgcn_readfirstlane(slice0 + (il >> 6));
                const int wdt = swidth[gsl];
                const int base = sstart[gsl] * kWave + lane;
                double2 acc = make_double2(0.0, 0.0);
                acc = sell_row<4, false>(sval, scol, base, wdt, il, [&](int j) { return Xv[j]; }, acc);
                if (il == of) acc = csub(acc, csub(cmul(oyd, Xv[of]), cmul(oy, Xv[ot])));
                else if (il == ot) acc = csub(acc, csub(cmul(oyd, Xv[ot]), cmul(oy, Xv[of])));
                const double2 v = Xv[il];
                const double2 d = csub(cmulc(v, acc), sp);
                const double rP = tk != kSlack ? d.x : 0.0;
                const double rQ = tk == kPQ ? d.y : 0.0;
                lsum += rP * rP + rQ * rQ;
                lmax = fmax(lmax, fmax(fabs(rP), fabs(rQ)));
                const double2 av = make_double2(two_over_m * rP, two_over_m * rQ);
                aIg[i] = cmul(av, acc);
                const double2 w = cmulc(av, v);
                if (dbl) Xw[il] = w;
                else Wg[i] = w;
        DPF_BUS_LOOP_END
        block_reduce2<NT>(lsum, lmax, red);
        __syncthreads();
        if (!dbl)
            for (int i = lo + tid; i < hi; i += NT) Xw[i - lo] = Wg[i];
        block_reduce2_finish<NT>(lsum, lmax, red);
        loss = m_res > 0.0 ? lsum / m_res : 0.0;
        mu = isnan(lsum) ? lsum : lmax;
        trace_mu(cold_args(), true, out_idx, it, mu);
        if (!dbl) __syncthreads();
        const int stop = stop_status(cold_args(), loss, mu, it);
        if (stop >= 0) {
            stat = stop;
            break;
        }

        // ---------------- phase B
        const OptStep os = begin_update(cold_args(), sc);
        DPF_BUS_LOOP_BEGIN
                const int il = (int)i - lo;
                // every global load of this bus first, so that they overlap the gather
                const int8_t tk = btp[i];
                const double2 ai = aIg[i];
                double vmi = vm_c[i], vai = va_c[i];
                const double mv0 = mv_c[i], sv0 = sv_c[i], ma0 = ma_c[i], sa0 = sa_c[i];
                const int gsl = __builtin_amdgcn_readfirstlane(slice0 + (il >> 6));
                const int wdt = swidth[gsl];
                const int base = sstart[gsl] * kWave + lane;
                double2 h = make_double2(0.0, 0.0);
                h = sell_row<4, false>(sval, scol, base, wdt, il, [&](int j) { return Xw[j]; }, h);
                if (il == of) h = csub(h, csub(cmul(oyd, Xw[of]), cmul(oy, Xw[ot])));
                else if (il == ot) h = csub(h, csub(cmul(oyd, Xw[ot]), cmul(oy, Xw[of])));
                const double2 G = make_double2(ai.x + h.x, ai.y - h.y);
                double sn0, cs0;
                fast_sincos(vai, sn0, cs0);
                const double2 v = make_double2(vmi * cs0, vmi * sn0);
                if (tk == kPQ) {
                    const double g = grad_vm(G, cs0, sn0, vmi);
                    double mv = mv0, sv = sv0;
                    vmi = opt_update(os, vmi, g, mv, sv);
                    vm_c[i] = vmi;
                    mv_c[i] = mv;
                    sv_c[i] = sv;
                }
                if (tk != kSlack) {
                    const double g = G.y * v.x - G.x * v.y;
                    double ma = ma0, sa = sa0;
                    vai = opt_update(os, vai, g, ma, sa);
                    va_c[i] = vai;
                    ma_c[i] = ma;
                    sa_c[i] = sa;
                }
                if (dbl) {
                    double sn, cs;
                    fast_sincos(vai, sn, cs);
                    Xv[il] = make_double2(vmi * cs, vmi * sn);
                }
        DPF_BUS_LOOP_END
        sched_step(cold_args(), sc, loss);
        if (!dbl) {
            __syncthreads();
            for (int i = lo + tid; i < hi; i += NT) {
                double sn, cs;
                const double vmi = vm_c[i];
                fast_sincos(va_c[i], sn, cs);
                Xv[i - lo] = make_double2(vmi * cs, vmi * sn);
            }
        }
        __syncthreads();
    }
#undef DPF_BUS_LOOP_BEGIN
#undef DPF_BUS_LOOP_END

    if (tid == 0) finish_item(out_idx, it, stat, mu, loss, sc);
}

// V conj(I) - S with S inside the chain of multiply-adds: its rounding then differs from
// that of any S formed as a product before, and a start at such an S (an outage from the
// base case's own injections, evaluated by this library) takes about the steps that the
// same start takes with injections from anywhere else.  With the product formed first, as in
// the other solve kernels and in these ones before, the residual is exactly zero at most
// buses and Adam takes another path: on 1024 outages of 9241 buses 264 instead of 50 steps
// at the median to max|r| < 1e-3 and 4% more to 1e-6; at other settings fewer (300 to 9241
// buses, lr 1e-4, eps 1e-14: 250..330 instead of 470..690) or none that converge within
// 2000 (lr 1e-3, eps 1e-8, where this form takes 83..90 up to 3000 buses).  qv, which keeps the product
// alive beside the residual, would undo a contraction left to the compiler.
__device__ __forceinline__ double2 residual_of_row(double2 v, double2 i, double2 s) {
    return make_double2(fma(v.x, i.x, fma(v.y, i.y, -s.x)), fma(v.y, i.x, fma(-v.x, i.y, -s.y)));
}

// Where an item whose rows begin at lo keeps one double per row in its case's part of a
// complex scratch array, indexed by row: in the first half of its own rows' entries, so
// that items of one call that run on different kernels at the same time never share
// memory, however each of them uses its entries (indexed from 0 over the case's 8-byte
// words, the values would reach into the entries of other items).
__device__ __forceinline__ double *kept_values(double2 *scratch, int lo) {
    return reinterpret_cast<double *>(scratch) + lo;
}

// The gradient of one row from w = a conj(V) and h = (Y w), without I.  With
// conj(G) V = conj(a) s + h V, s = V conj(I): at a PQ row the seed a holds the whole
// residual, s = S_spec + (m/2) a; at a PV row a is real and only Im s = qv is needed,
// 8 B kept between the sweeps where I was 16 (the paired kernel keeps it in LDS, for the
// PV rows only).  a = w V / |V|^2; a PV row held at |V| = 0 has w = 0 and no angle to
// move, and gets 0 instead of 0 / 0 (a PQ row there has no direction: NaN, see grad_vm).
struct SeedTerm {
    double vm, va;
};
__device__ __forceinline__ SeedTerm gradient_of_row(double2 w, double2 h, double vm, double cs, double sn, double2 sp,
                                                    double qv, double half_m, bool pq) {
    double iv = 1.0 / vm;
    if (!pq && isinf(iv)) iv = 0.0;
    const double2 e = make_double2(cs, sn);
    double2 a = cscale(iv, cmul(w, e));
    if (!pq) a.y = 0.0;
    const double2 s = make_double2(sp.x + half_m * a.x, pq ? sp.y + half_m * a.y : qv);
    const double2 t = cmulc(s, a);
    const double2 hv = cscale(vm, cmul(h, e));
    return SeedTerm{(t.x + hv.x) * iv, -(t.y + hv.y)};
}

// Banded variant, for sub-grids numbered with a small bandwidth: every entry of
// the matrix has |row - col| <= NT*J in local indices (a reverse Cuthill-McKee
// numbering gives ~80 on a 9241-bus meshed grid).  Buses are processed in blocks
// of BLK = NT*J consecutive buses, thread tid owning buses s*BLK + j*NT + tid of
// block s.  The rows of block s then read the exchange vector only in blocks
// s-1, s and s+1, so the single LDS array X can go from V to w to the new V
// block by block, with one block of values held in registers instead of the
// whole sub-grid:
//   A/W sweep, step s: rows of block s gather V, form dS, the loss terms and
//       w = a conj(V); Im(V conj(I)) goes to scratch for the second sweep.  After a barrier
//       the w of block s-1 replaces V there (its readers, blocks s-2..s, are done).
//   stop test on the reduced max|r|
//   gradient sweep, one pass without barriers (w stays in X throughout): rows
//       gather w, form the gradient (gradient_of_row) and apply the optimizer step; then X is refilled with the new V from |V| and theta.
// Per bus and iteration this moves |V|, theta and the four moments once each way,
// Im(V conj(I)) (8 B written, 8 B read) and the refill's |V| and theta (16 B read); there is
// no w round trip through memory.  (A pipelined gradient sweep that overwrote w
// block by block with the new V moved 16 B less but, with a barrier per block,
// ran slower: the lockstep waves stopped overlapping loads and arithmetic.)
template <int NT, int J>
__global__ __launch_bounds__(NT) void team_solve_band_kernel(SolveArgs a) {
    constexpr int BLK = NT * J;
    extern __shared__ double2 X[];
    __shared__ double red[2][NT / kWave];

    const int tid = threadIdx.x;
    const int item = a.order ? a.order[blockIdx.x] : (int)blockIdx.x;
    const int sidx = item / a.B;
    const int c = item - sidx * a.B;
    const int lo = a.sub_off ? a.sub_off[sidx] : 0;
    const int hi = a.sub_off ? a.sub_off[sidx + 1] : a.n_bus;
    const int n = hi - lo;
    const int out_idx = c * a.n_sub + sidx;
    if (n > a.team_cap) return;        // handled by the multi-workgroup path
    if (a.sub_bw[sidx] > BLK) return;  // bandwidth too large: the general kernel takes it
    if (n < 0 || n > a.lds_cap || *a.bad_grid) {  // see DPF_BAD_GRID
        if (tid == 0) {
            a.status[out_idx] = DPF_BAD_GRID;
            a.iters[out_idx] = 0;
        }
        return;
    }
    const int slice0 = a.sell.slice_off[sidx];
    const int lane = tid & (kWave - 1);

    // step count and schedule (a resumed solve continues them)
    ItemSched sc = load_item_sched(a, out_idx);

    const double m_res = residual_count<NT>(a.bt, lo, hi, red);
    const double two_over_m = m_res > 0.0 ? 2.0 / m_res : 0.0;
    const double half_m = 0.5 * m_res;

    // N-1 outage of this case (only meaningful for a single sub-grid)
    const Rank2 r2 = outage_of_case(a.ov, c, lo, hi);
    if (r2.bad) return;  // reported by the call's prologue
    const int of = r2.of, ot = r2.ot;
    const double2 oy = r2.oy, oyd = r2.oyd;

    const int64_t cb = (int64_t)c * a.ld;
    const int64_t sb = (int64_t)c * a.s_ld;
    double *__restrict__ vm_c = a.vm + cb;
    double *__restrict__ va_c = a.va + cb;
    double *__restrict__ mv_c = a.st + cb;
    double *__restrict__ ma_c = a.st + a.st_stride + cb;
    double *__restrict__ sv_c = a.st + 2 * a.st_stride + cb;
    double *__restrict__ sa_c = a.st + 3 * a.st_stride + cb;
    double *__restrict__ Qg = kept_values(a.scratch + cb, lo);  // Im(V conj(I)) of the A/W sweep
    const double2 *__restrict__ Sc = a.s_spec + sb;
    const int32_t *__restrict__ swidth = a.sell.width;
    const int32_t *__restrict__ sstart = a.sell.start;
    const int32_t *__restrict__ scol = a.sell.col;
    const double2 *__restrict__ sval = a.sell.val;
    const int8_t *__restrict__ btp = a.bt;

    for (int i = lo + tid; i < hi; i += NT) {
        double sn, cs;
        const double vmi = vm_c[i];
        fast_sincos(va_c[i], sn, cs);
        X[i - lo] = make_double2(vmi * cs, vmi * sn);
        if (a.st_fresh) {
            mv_c[i] = 0.0;
            ma_c[i] = 0.0;
            sv_c[i] = 0.0;
            sa_c[i] = 0.0;
        }
    }
    __syncthreads();

    const int nb = (n + BLK - 1) / BLK;
    int it = 0, stat = DPF_MAX_ITER;
    double mu = 0.0, loss = 0.0;
    __shared__ int pause_flag;
    for (;; ++it) {
        if (handoff_due(it, &pause_flag)) {
            stat = kPaused;
            break;
        }
        // ---------------- A/W sweep
        double lsum = 0.0, lmax = 0.0;
        double2 hold[J];
#pragma unroll
        for (int j = 0; j < J; ++j) hold[j] = make_double2(0.0, 0.0);
        for (int s = 0; s <= nb; ++s) {
            double2 w[J];
#pragma unroll
            for (int j = 0; j < J; ++j) {
                w[j] = make_double2(0.0, 0.0);
                const int il = s * BLK + j * NT + tid;
                if (s < nb && il < n) {
                    const int i = lo + il;
                    const int8_t tk = btp[i];
                    const double2 sp = Sc[i];
                    const int gsl = __builtin_amdgcn_readfirstlane(slice0 + (il >> 6));
                    const int wdt = swidth[gsl];
                    const int base = sstart[gsl] * kWave + lane;
                    double2 acc = make_double2(0.0, 0.0);
                    acc = sell_row<4, false>(sval, scol, base, wdt, il, [&](int j) { return X[j]; }, acc);
                    if (il == of) acc = csub(acc, csub(cmul(oyd, X[of]), cmul(oy, X[ot])));
                    else if (il == ot) acc = csub(acc, csub(cmul(oyd, X[ot]), cmul(oy, X[of])));
                    const double2 v = X[il];
                    const double2 d = residual_of_row(v, acc, sp);
                    const double qv = fma(v.y, acc.x, -(v.x * acc.y));
                    const double rP = tk != kSlack ? d.x : 0.0;
                    const double rQ = tk == kPQ ? d.y : 0.0;
                    lsum += rP * rP + rQ * rQ;
                    lmax = fmax(lmax, fmax(fabs(rP), fabs(rQ)));
                    const double2 av = make_double2(two_over_m * rP, two_over_m * rQ);
                    Qg[i] = qv;
                    w[j] = cmulc(av, v);
                }
            }
            __syncthreads();
            if (s > 0) {
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    const int il = (s - 1) * BLK + j * NT + tid;
                    if (il < n) X[il] = hold[j];
                }
            }
#pragma unroll
            for (int j = 0; j < J; ++j) hold[j] = w[j];
        }
        block_reduce2<NT>(lsum, lmax, red);
        __syncthreads();
        block_reduce2_finish<NT>(lsum, lmax, red);
        loss = m_res > 0.0 ? lsum / m_res : 0.0;
        mu = isnan(lsum) ? lsum : lmax;
        trace_mu(cold_args(), true, out_idx, it, mu);
        const int stop = stop_status(cold_args(), loss, mu, it);
        if (stop >= 0) {
            stat = stop;
            break;
        }

        // ---------------- B/U sweep
        const OptStep os = begin_update(cold_args(), sc);
        // one barrier-free pass (w stays in X throughout), then the new V is
        // rebuilt from |V| and theta in a refill pass
        for (int s = 0; s < nb; ++s) {
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int il = s * BLK + j * NT + tid;
                if (il < n) {
                    const int i = lo + il;
                    // every global load of this bus first, so that they overlap the gather
                    const int8_t tk = btp[i];
                    const double qv = Qg[i];
                    const double2 sp = Sc[i];
                    double vmi = vm_c[i], vai = va_c[i];
                    const double mv0 = mv_c[i], sv0 = sv_c[i], ma0 = ma_c[i], sa0 = sa_c[i];
                    const int gsl = __builtin_amdgcn_readfirstlane(slice0 + (il >> 6));
                    const int wdt = swidth[gsl];
                    const int base = sstart[gsl] * kWave + lane;
                    double2 h = make_double2(0.0, 0.0);
                    h = sell_row<4, false>(sval, scol, base, wdt, il, [&](int j) { return X[j]; }, h);
                    if (il == of) h = csub(h, csub(cmul(oyd, X[of]), cmul(oy, X[ot])));
                    else if (il == ot) h = csub(h, csub(cmul(oyd, X[ot]), cmul(oy, X[of])));
                    double sn0, cs0;
                    fast_sincos(vai, sn0, cs0);
                    const SeedTerm g = gradient_of_row(X[il], h, vmi, cs0, sn0, sp, qv, half_m, tk == kPQ);
                    if (tk == kPQ) {
                        double mv = mv0, sv = sv0;
                        vmi = opt_update(os, vmi, g.vm, mv, sv);
                        vm_c[i] = vmi;
                        mv_c[i] = mv;
                        sv_c[i] = sv;
                    }
                    if (tk != kSlack) {
                        double ma = ma0, sa = sa0;
                        vai = opt_update(os, vai, g.va, ma, sa);
                        va_c[i] = vai;
                        ma_c[i] = ma;
                        sa_c[i] = sa;
                    }
                }
            }
        }
        __syncthreads();
        for (int i = lo + tid; i < hi; i += NT) {
            double sn, cs;
            const double vmi = vm_c[i];
            fast_sincos(va_c[i], sn, cs);
            X[i - lo] = make_double2(vmi * cs, vmi * sn);
        }
        sched_step(cold_args(), sc, loss);
        __syncthreads();
    }

    if (tid == 0) finish_item(out_idx, it, stat, mu, loss, sc);
}

// start point of every step of a time-series window: rows [0, gridDim.y) of dst
// receive the source voltages
__global__ void row_broadcast_kernel(int32_t n, const double *__restrict__ src_m, const double *__restrict__ src_a,
                                     double *__restrict__ dst_m, double *__restrict__ dst_a, int64_t ld) {
    int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double m = src_m[i], v = src_a[i];
    dst_m[blockIdx.y * ld + i] = m;
    dst_a[blockIdx.y * ld + i] = v;
}

// default schedule state {t, lr, best, bad + cooldown * 2^20, b1^t, b2^t} of B items
__global__ void sched_init_kernel(int32_t B, double lr, double *__restrict__ sched) {
    const int32_t c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= B) return;
    double *ss = sched + kSchedWords * (int64_t)c;
    ss[0] = 0.0;
    ss[1] = lr;
    ss[2] = __longlong_as_double(0x7ff0000000000000LL);
    ss[3] = 0.0;
    ss[4] = 1.0;
    ss[5] = 1.0;
}

// indices of the paused items (one workgroup; the order of the list is free)
__global__ __launch_bounds__(1024) void collect_paused_kernel(int32_t n_items, const int32_t *__restrict__ status,
                                                              int32_t *__restrict__ list, int32_t *__restrict__ count) {
    __shared__ int n;
    if (threadIdx.x == 0) n = 0;
    __syncthreads();
    for (int32_t i = threadIdx.x; i < n_items; i += blockDim.x)
        if (status[i] == kPaused) list[atomicAdd(&n, 1)] = i;
    __syncthreads();
    if (threadIdx.x == 0) *count = n;
}

// Call prologue with an outage list: a case whose index is neither -1 nor a
// branch index is reported (status DPF_BAD_OUTAGE, no updates, NaN mismatch and
// loss) and counted as finished for the tail handoff; the kernels skip it.
__global__ void outage_check_kernel(int32_t B, OutageView ov, int32_t *__restrict__ status,
                                    int32_t *__restrict__ iters, double *__restrict__ mu,
                                    double *__restrict__ loss, int32_t *__restrict__ done_count) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= B || !outage_index_bad(ov.outage[c], ov.n_branch)) return;
    status[c] = DPF_BAD_OUTAGE;
    iters[c] = 0;
    mu[c] = __longlong_as_double(0x7ff8000000000000LL);
    loss[c] = __longlong_as_double(0x7ff8000000000000LL);
    atomicAdd(done_count, 1);
}

// Case order of a call: descending initial max|r| (NaN first, ties by index), so
// that the cases likely to run longest start first.  order[rank] = case; one
// thread per case counts the cases ahead of it (B is small enough for O(B^2)).
__global__ void rank_desc_kernel(int32_t B, const double *__restrict__ key, int32_t *__restrict__ order) {
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= B) return;
    auto k = [&](int32_t j) {
        const double x = key[j];
        return isnan(x) ? __longlong_as_double(0x7ff0000000000000LL) : x;
    };
    const double ki = k(i);
    int32_t rank = 0;
    for (int32_t j = 0; j < B; ++j) {
        const double kj = k(j);
        rank += (kj > ki || (kj == ki && j < i)) ? 1 : 0;
    }
    order[rank] = i;
}

}  // namespace dpf
