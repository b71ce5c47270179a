// DC power flow on the device: the linear approximation that the paper lists as
// a screening method (Sec. 3, direct methods) and that Algorithm 2 uses to
// initialise Newton-Raphson.  With |V| = 1, no losses and small angle
// differences, the active injections satisfy  L theta = P,  where L is the
// branch-susceptance Laplacian (weights 1/x) and the slack angle is fixed.
//
// L comes from an admittance matrix built with r = 0 and b = 0 (the "DC grid"):
// there Y = -j L, so L_ij = -Im(Y_ij).  One workgroup per case solves the
// grounded system by conjugate gradients with a Jacobi preconditioner.  Up to 8192
// buses everything but the exchanged search direction stays in registers
// (dc_cg_kernel); above that the search direction lives in LDS (8 B per bus), the
// other vectors in the workspace (dc_pcg_kernel).  An N-1 outage removes the branch's 1/x (rank-1, on the fly).
#pragma once

#include "../../include/dpf.h"
#include "common.hpp"
#include "eval.hpp"

namespace dpf {

struct DcArgs {
    const int32_t *rp;
    const int32_t *ci;
    const double2 *yv;  // admittance matrix of the DC grid (r = 0, b = 0)
    const int8_t *bt;
    const double2 *s_spec;
    int64_t s_ld;
    OutageView ov;
    double *va;  // [B][ld] in: start (slack angle fixed), out: DC angles
    int64_t ld;
    double *r;   // [B][n] residual
    double *z;   // [B][n] preconditioned residual
    double *dg;  // [B][n] diagonal of L (after the outage)
    int32_t n;
    double tol;
    int32_t max_iter;
    int32_t *iters;    // [B] or null
    double *res_out;   // [B] relative residual ||r|| / ||P||, or null
};

template <int NT>
__device__ __forceinline__ void block_sum2(double &a, double &b, double (*red)[NT / kWave]) {
    a = wave_sum(a);
    b = wave_sum(b);
    const int wv = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0) {
        red[0][wv] = a;
        red[1][wv] = b;
    }
    __syncthreads();
    a = 0.0;
    b = 0.0;
#pragma unroll
    for (int k = 0; k < NT / kWave; ++k) {
        a += red[0][k];
        b += red[1][k];
    }
    a = uniform(a);
    b = uniform(b);
    __syncthreads();
}

// (L p)_i for a real vector p held in LDS; the outaged branch's block removed
__device__ __forceinline__ double dc_row(const DcArgs &a, int i, const double *p, int of, int ot, double oyi) {
    double acc = 0.0;
    for (int q = a.rp[i]; q < a.rp[i + 1]; ++q) {
        const int j = a.ci[q];
        if ((unsigned)j < (unsigned)a.n) acc += a.yv[q].y * p[j];
    }
    double v = -acc;  // L = -Im(Y)
    // outage: L loses (1/x)(e_f - e_t)(e_f - e_t)^T; Im(y) = -1/x for y = 1/(jx)
    if (i == of) v += oyi * (p[of] - p[ot]);
    else if (i == ot) v += oyi * (p[ot] - p[of]);
    return v;
}

template <int NT>
__global__ __launch_bounds__(NT) void dc_pcg_kernel(DcArgs a) {
    extern __shared__ double P[];
    __shared__ double red[2][NT / kWave];
    const int c = blockIdx.x;
    const int n = a.n;
    double *va = a.va + (int64_t)c * a.ld;
    double *r = a.r + (int64_t)c * n;
    double *z = a.z + (int64_t)c * n;
    double *dg = a.dg + (int64_t)c * n;
    const double2 *S = a.s_spec + (int64_t)c * a.s_ld;

    int of = -1, ot = -1;
    double oyi = 0.0;  // Im of the outaged branch's series admittance (= -1/x)
    if (a.ov.outage) {
        const int k = a.ov.outage[c];
        if (outage_index_bad(k, a.ov.n_branch)) {  // neither -1 nor a branch: va untouched
            if (threadIdx.x == 0) {
                if (a.iters) a.iters[c] = 0;
                if (a.res_out) a.res_out[c] = __longlong_as_double(0x7ff8000000000000LL);
            }
            return;
        }
        if ((unsigned)k < (unsigned)a.ov.n_branch) {
            const int f = a.ov.from[k], t = a.ov.to[k];
            if ((unsigned)f < (unsigned)n && (unsigned)t < (unsigned)n && f != t) {
                of = f;
                ot = t;
                double2 y, ysh;
                branch_admittance(a.ov.r[k], a.ov.x[k], a.ov.b[k], y, ysh);
                oyi = y.y;
            }
        }
    }

    // start: theta in LDS (slack entry fixed), diagonal, r = P - L theta, z = r / diag
    for (int i = threadIdx.x; i < n; i += NT) P[i] = va[i];
    __syncthreads();
    double bb = 0.0, rz = 0.0;
    for (int i = threadIdx.x; i < n; i += NT) {
        double d = 0.0;
        for (int q = a.rp[i]; q < a.rp[i + 1]; ++q)
            if (a.ci[q] == i) d = -a.yv[q].y;
        if (i == of || i == ot) d += oyi;
        const bool free = a.bt[i] != kSlack;
        const double b = free ? S[i].x : 0.0;
        const double ri = free ? b - dc_row(a, i, P, of, ot, oyi) : 0.0;
        const double zi = free && d > 0.0 ? ri / d : 0.0;
        dg[i] = d;
        r[i] = ri;
        z[i] = zi;
        bb += b * b;
        rz += ri * zi;
    }
    block_sum2<NT>(bb, rz, red);  // ends with a barrier: every read of theta in P is done
    const double bnorm = sqrt(bb);
    // search direction p = z (the slack entry stays 0)
    for (int i = threadIdx.x; i < n; i += NT) P[i] = z[i];
    double rr = 0.0, dummy = 0.0;
    for (int i = threadIdx.x; i < n; i += NT) rr += r[i] * r[i];
    block_sum2<NT>(rr, dummy, red);
    int it = 0;
    while (it < a.max_iter && !(sqrt(rr) <= a.tol * bnorm)) {
        // q = L p; alpha = rz / (p . q)
        double pq = 0.0, unused = 0.0;
        for (int i = threadIdx.x; i < n; i += NT) {
            const double qi = a.bt[i] != kSlack ? dc_row(a, i, P, of, ot, oyi) : 0.0;
            z[i] = qi;  // z holds q until the update below
            pq += P[i] * qi;
        }
        block_sum2<NT>(pq, unused, red);
        const double alpha = pq != 0.0 ? rz / pq : 0.0;
        double rz_new = 0.0, rr_new = 0.0;
        for (int i = threadIdx.x; i < n; i += NT) {
            if (a.bt[i] == kSlack) continue;
            va[i] += alpha * P[i];
            const double ri = r[i] - alpha * z[i];
            const double zi = dg[i] > 0.0 ? ri / dg[i] : 0.0;
            r[i] = ri;
            z[i] = zi;
            rz_new += ri * zi;
            rr_new += ri * ri;
        }
        block_sum2<NT>(rz_new, rr_new, red);
        const double beta = rz != 0.0 ? rz_new / rz : 0.0;
        rz = rz_new;
        rr = rr_new;
        for (int i = threadIdx.x; i < n; i += NT) P[i] = z[i] + beta * P[i];
        __syncthreads();
        ++it;
    }
    if (threadIdx.x == 0) {
        if (a.iters) a.iters[c] = it;
        if (a.res_out) a.res_out[c] = bnorm > 0.0 ? sqrt(rr) / bnorm : sqrt(rr);
    }
}

// Sum of two values over the workgroup, the same in every lane: DPP within the waves,
// one LDS round for the wave sums, DPP again over at most 16 of them.  `red` must not be
// rewritten before every wave has read it (the callers alternate two of them).
template <int NT>
__device__ __forceinline__ void fast_sum2(double &a, double &b, double2 *red) {
    constexpr int kShr = 0x110, kBcast15 = 0x142, kBcast31 = 0x143, NW = NT / kWave;
    auto rows = [&]() {
        a += dpp_or_zero<kShr + 1, 0xf>(a);
        b += dpp_or_zero<kShr + 1, 0xf>(b);
        a += dpp_or_zero<kShr + 2, 0xf>(a);
        b += dpp_or_zero<kShr + 2, 0xf>(b);
        a += dpp_or_zero<kShr + 4, 0xf>(a);
        b += dpp_or_zero<kShr + 4, 0xf>(b);
        a += dpp_or_zero<kShr + 8, 0xf>(a);
        b += dpp_or_zero<kShr + 8, 0xf>(b);
    };
    rows();
    a += dpp_or_zero<kBcast15, 0xa>(a);
    b += dpp_or_zero<kBcast15, 0xa>(b);
    a += dpp_or_zero<kBcast31, 0xc>(a);
    b += dpp_or_zero<kBcast31, 0xc>(b);
    if constexpr (NW == 1) {
        a = read_lane(a, kWave - 1);
        b = read_lane(b, kWave - 1);
        return;
    }
    const int lane = threadIdx.x & (kWave - 1);
    if (lane == kWave - 1) red[threadIdx.x / kWave] = make_double2(a, b);
    __syncthreads();
    const double2 p = lane < NW ? red[lane] : make_double2(0.0, 0.0);
    a = p.x;
    b = p.y;
    rows();
    a = read_lane(a, 15);
    b = read_lane(b, 15);
}

// The same iteration with everything a thread owns in registers: of each of its K rows
// the angle, residual, inverse diagonal and search direction, and the first REG matrix
// entries (-Im(Y) and a packed 16-bit column).  The search direction's copy in LDS is
// what the rows read; entries past REG sit in LDS beside it, 10 B each in 64-row slices,
// or are read from the CSR when they do not fit.  Three barriers per step.
// Bound by the latency of a step (two reductions, two divisions, the gathers), where the
// form above, with its vectors in global memory, waited for about ten dependent trips to
// L2.  us per step on an MI355X, above -> this: 118 buses 3.8 -> 0.9, 500 5.1 -> 1.3,
// 1354 x 64 cases 8.6 -> 1.75, 3000 13.5 -> 3.2, 4000 16.9 -> 10.0 (4 entries of a row in
// registers; the rest of this grid's rows exceeds the LDS and comes from the CSR: 4.4 on
// one whose rows fit), 8000 31 -> 29 (no entries in registers).
// 512 threads up to 4096 buses: the registers of 1024 hold 4 rows without entries.
constexpr int kDcMaxRows = 8 * 1024;  // rows: 16-bit byte offsets, and slices of one wave scan

template <int NT, int K, int REG>
__global__ __launch_bounds__(NT) void dc_cg_kernel(DcArgs a, int32_t cap) {
    static_assert(REG % 4 == 0, "the product takes register entries in groups of four");
    extern __shared__ double P[];  // direction [n], values [cap], columns [cap] (byte offsets, 16 bit)
    __shared__ double2 red[2][NT / kWave];
    __shared__ int32_t sw[kDcMaxRows / kWave], so[kDcMaxRows / kWave + 1];
    constexpr int NW = NT / kWave;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int c = blockIdx.x;
    const int n = a.n, ns = (n + kWave - 1) / kWave;
    double *va = a.va + (int64_t)c * a.ld;
    const double2 *S = a.s_spec + (int64_t)c * a.s_ld;

    int of = -1, ot = -1;
    double oyi = 0.0;  // Im of the outaged branch's series admittance (= -1/x)
    if (a.ov.outage) {
        const int k = a.ov.outage[c];
        if (outage_index_bad(k, a.ov.n_branch)) {  // neither -1 nor a branch: va untouched
            if (tid == 0) {
                if (a.iters) a.iters[c] = 0;
                if (a.res_out) a.res_out[c] = __longlong_as_double(0x7ff8000000000000LL);
            }
            return;
        }
        if ((unsigned)k < (unsigned)a.ov.n_branch) {
            const int f = a.ov.from[k], t = a.ov.to[k];
            if ((unsigned)f < (unsigned)n && (unsigned)t < (unsigned)n && f != t) {
                of = f;
                ot = t;
                double2 y, ysh;
                branch_admittance(a.ov.r[k], a.ov.x[k], a.ov.b[k], y, ysh);
                oyi = y.y;
            }
        }
    }

    // slice widths and offsets, then the entries (if they fit)
    double *MV = P + n;
    uint16_t *MC = reinterpret_cast<uint16_t *>(MV + cap);
    int q0[K], len[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = tid + k * NT;
        q0[k] = i < n ? a.rp[i] : 0;
        len[k] = i < n ? a.rp[i + 1] - q0[k] : 0;
        int w = len[k];
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1) w = max(w, __shfl_xor(w, o, kWave));
        if (lane == 0 && wv + k * NW < ns) sw[wv + k * NW] = max(w - REG, 0);
    }
    __syncthreads();
    if (wv == 0) {
        int before = 0;
        for (int j0 = 0; j0 < ns; j0 += kWave) {
            const int w = j0 + lane < ns ? sw[j0 + lane] : 0;
            int incl = w;
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                const int y = __shfl_up(incl, o, kWave);
                if (lane >= o) incl += y;
            }
            if (j0 + lane < ns) so[j0 + lane] = before + incl - w;
            before += __shfl(incl, kWave - 1, kWave);
        }
        if (lane == 0) so[ns] = before;
    }
    __syncthreads();
    const bool fits = (int64_t)so[ns] * kWave <= cap;

    int wd[K], mo[K];  // LDS entries of the row's slice: width and first
    double x[K], r[K], di[K], p[K];
    double mv[K][REG > 0 ? REG : 1];
    uint32_t mc[K][REG > 0 ? REG / 2 : 1];
    uint32_t fre = 0;
    double bb = 0.0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = tid + k * NT, j = wv + k * NW;
        wd[k] = j < ns ? __builtin_amdgcn_readfirstlane(sw[j]) : 0;
        mo[k] = j < ns ? __builtin_amdgcn_readfirstlane(so[j]) * kWave : 0;
        double d = 0.0;
        // entry q of the row: L = -Im(Y) and its column's byte offset (0 at the own row
        // past the end and for a column out of range)
        auto entry = [&](int q, uint32_t &col) {
            double v = 0.0;
            col = (uint32_t)(i < n ? i : 0) * 8u;
            if (q < len[k]) {
                const int jc = a.ci[q0[k] + q];
                const double y = -a.yv[q0[k] + q].y;
                if ((unsigned)jc < (unsigned)n) {
                    v = y;
                    col = (uint32_t)jc * 8u;
                }
                if (jc == i) d = y;
            }
            return v;
        };
#pragma unroll
        for (int q = 0; q < REG; q += 2) {
            uint32_t c0, c1;
            mv[k][q] = entry(q, c0);
            mv[k][q + 1] = entry(q + 1, c1);
            mc[k][q / 2] = c0 | (c1 << 16);
        }
        for (int q = 0; q < wd[k]; ++q) {
            uint32_t col;
            const double v = entry(REG + q, col);
            if (fits) {
                MV[mo[k] + q * kWave + lane] = v;
                MC[mo[k] + q * kWave + lane] = (uint16_t)col;
            }
        }
        if (i == of || i == ot) d += oyi;
        di[k] = d > 0.0 ? 1.0 / d : 0.0;
        x[k] = p[k] = r[k] = 0.0;
        if (i < n) {
            fre |= (a.bt[i] != kSlack ? 1u : 0u) << k;
            x[k] = va[i];
            P[i] = x[k];
            const double b = (fre >> k) & 1u ? S[i].x : 0.0;
            r[k] = b;
            bb += b * b;
        }
    }
    // entries of the longest row of each slice that are in registers (uniform)
    int wr[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        int w = min(len[k], REG);
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1) w = max(w, __shfl_xor(w, o, kWave));
        wr[k] = __builtin_amdgcn_readfirstlane(w);
    }
    __syncthreads();

    const char *lds = reinterpret_cast<const char *>(P);
    auto at = [&](uint32_t ofs) { return *reinterpret_cast<const double *>(lds + ofs); };
    // (L p)_i for row k of this thread, p in LDS
    auto product = [&](int k) {
        const int i = tid + k * NT;
        double acc = 0.0;
        // four gathers at a time
#pragma unroll
        for (int g = 0; g < REG; g += 4) {
            if (g >= wr[k]) break;
            double z[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) z[u] = at((u & 1) ? mc[k][(g + u) / 2] >> 16 : mc[k][(g + u) / 2] & 0xffffu);
#pragma unroll
            for (int u = 0; u < 4; ++u) acc = fma(mv[k][g + u], z[u], acc);
        }
        if (fits) {
#pragma unroll 4
            for (int q = 0; q < wd[k]; ++q)
                acc = fma(MV[mo[k] + q * kWave + lane], at(MC[mo[k] + q * kWave + lane]), acc);
        } else {
            for (int q = REG; q < len[k]; ++q) {
                const int j = a.ci[q0[k] + q];
                if ((unsigned)j < (unsigned)n) acc -= a.yv[q0[k] + q].y * P[j];
            }
        }
        // outage: L loses (1/x)(e_f - e_t)(e_f - e_t)^T; Im(y) = -1/x for y = 1/(jx)
        if (of >= 0) {
            if (i == of) acc += oyi * (P[of] - P[ot]);
            else if (i == ot) acc += oyi * (P[ot] - P[of]);
        }
        return acc;
    };

    // r = P - L theta, z = r / diag, p = z (the slack entry stays 0)
    double rz = 0.0, rr = 0.0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const double q = product(k);
        r[k] = (fre >> k) & 1u ? r[k] - q : 0.0;
        p[k] = (fre >> k) & 1u ? r[k] * di[k] : 0.0;
        rz += r[k] * p[k];
        rr += r[k] * r[k];
    }
    double zero = 0.0;
    fast_sum2<NT>(bb, zero, red[0]);  // its barrier: every read of theta in P is done
    const double bnorm = sqrt(bb);
    fast_sum2<NT>(rz, rr, red[1]);
    if constexpr (NW == 1) __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (tid + k * NT < n) P[tid + k * NT] = p[k];
    __syncthreads();

    // the stop test sqrt(rr) <= tol ||P||, its root taken only near the bound (the squares
    // decide elsewhere; where they could underflow the root is always taken)
    const double stop = a.tol * bnorm, stop2 = stop * stop * (1.0 + 1e-12);
    const bool squares = stop2 > 1e-280;
    int it = 0;
    while (it < a.max_iter && ((squares && rr > stop2) || !(sqrt(rr) <= stop))) {
        // q = L p; alpha = rz / (p . q)
        double q[K];
        double pq = 0.0, unused = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            q[k] = product(k);
            q[k] = (fre >> k) & 1u ? q[k] : 0.0;
            pq += p[k] * q[k];
        }
        fast_sum2<NT>(pq, unused, red[0]);
        const double alpha = pq != 0.0 ? rz / pq : 0.0;
        double rz_new = 0.0, rr_new = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            x[k] += alpha * p[k];
            r[k] -= alpha * q[k];
            rz_new += r[k] * (r[k] * di[k]);
            rr_new += r[k] * r[k];
        }
        fast_sum2<NT>(rz_new, rr_new, red[1]);
        const double beta = rz != 0.0 ? rz_new / rz : 0.0;
        rz = rz_new;
        rr = rr_new;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            p[k] = r[k] * di[k] + beta * p[k];
            if (tid + k * NT < n) P[tid + k * NT] = p[k];
        }
        __syncthreads();
        ++it;
    }
#pragma unroll
    for (int k = 0; k < K; ++k)
        if ((fre >> k) & 1u) va[tid + k * NT] = x[k];
    if (tid == 0) {
        if (a.iters) a.iters[c] = it;
        if (a.res_out) a.res_out[c] = bnorm > 0.0 ? sqrt(rr) / bnorm : sqrt(rr);
    }
}

}  // namespace dpf
