// One forward + fused-adjoint evaluation for B cases on one grid
// (dpf_mismatch_grad).  Case-major layout, one thread per (bus, case):
//
// Large grids with few cases, one thread per (bus, case) and three launches:
//   polar    : V = vm e^{j va}, residual count                   -> ws.V
//   forward  : I = Y V (+ rank-2 outage term), dS = V conj(I) - S,
//              masked residual r, seed a = (2/m) r, w = a conj(V), aI = a I
//              per-block partial loss / max                        -> ws
//   adjoint  : h = Y^T w (Y symmetric: same CSR, + outage term),
//              G = aI + conj(h); g_vm = Re(conj(G) V)/vm, g_va = Im(G conj(V))
//              and per-case loss = sum / m and max, fixed summation order
// The others run in one launch, one workgroup per case (eval_case_kernel).
//
// The gradient follows from d loss = Re sum_k conj(G_k) dV_k with
// dV_k = e^{j va_k} dvm_k + j V_k dva_k (reverse mode through S = V conj(Y V)).
#pragma once

#include "common.hpp"

namespace dpf {

constexpr int kEvalBlock = 256;

struct OutageView {
    const int32_t *outage;  // [B] or null
    const int32_t *from;
    const int32_t *to;
    const double *r;
    const double *x;
    const double *b;
    int32_t n_branch;
};

// An outage index is -1 (no outage) or a branch index; anything else marks the
// case as bad (the solve reports DPF_BAD_OUTAGE, the evaluations return NaN).
__host__ __device__ __forceinline__ bool outage_index_bad(int32_t k, int32_t n_branch) {
    return k != -1 && (uint32_t)k >= (uint32_t)n_branch;
}

// Rank-2 correction: subtract branch k's pi-model block from row i of Y z.
// Y_k = [[y + ysh, -y], [-y, y + ysh]] on (f, t).
__device__ __forceinline__ double2 outage_term(const OutageView &ov, int32_t k, int32_t i, double2 zf, double2 zt,
                                               int32_t f, int32_t t) {
    double2 y, ysh;
    branch_admittance(ov.r[k], ov.x[k], ov.b[k], y, ysh);
    double2 yd = cadd(y, ysh);
    if (i == f) return csub(cmul(yd, zf), cmul(y, zt));
    return csub(cmul(yd, zt), cmul(y, zf));  // i == t
}

// row i of Y z from the CSR, z_j = get(j), entries in groups of four whose loads are
// issued together (a row's entries share cache lines, and most rows have at most four
// to five)
template <typename Get>
__device__ __forceinline__ double2 csr_row(const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
                                           const double2 *__restrict__ yv, int32_t i, int32_t n, Get get) {
    double2 acc = make_double2(0.0, 0.0);
    const int32_t end = rp[i + 1];
    for (int32_t q = rp[i]; q < end; q += 4) {
        int32_t j[4];
        double2 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int32_t p = q + u < end ? q + u : q;
            j[u] = ci[p];
            v[u] = yv[p];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (q + u < end && (uint32_t)j[u] < (uint32_t)n) acc = cfma(v[u], get(j[u]), acc);
    }
    return acc;
}

// V of every bus and case; one more block of the first case counts the residuals
// (m = n_pv + 2 n_pq), grid (blocks of n, + 1, B)
__global__ __launch_bounds__(kEvalBlock) void polar_kernel(int32_t n, int64_t ld, const double *__restrict__ vm,
                                                            const double *__restrict__ va,
                                                            const int8_t *__restrict__ bt, double2 *__restrict__ V,
                                                            double *__restrict__ m_out) {
    int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    int32_t c = blockIdx.y;
    if (blockIdx.x == gridDim.x - 1) {
        if (c != 0) return;
        __shared__ int part[kEvalBlock / kWave];
        int s = 0;
        for (i = threadIdx.x; i < n; i += kEvalBlock) {
            const int8_t t = bt[i];
            s += t == kPQ ? 2 : (t == kPV ? 1 : 0);
        }
        s = wave_isum(s);
        if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x / kWave] = s;
        __syncthreads();
        if (threadIdx.x == 0) {
            int tot = 0;
            for (int w = 0; w < kEvalBlock / kWave; ++w) tot += part[w];
            *m_out = (double)tot;
        }
        return;
    }
    if (i >= n) return;
    double s, co;
    fast_sincos(va[c * ld + i], s, co);
    double m = vm[c * ld + i];
    V[(int64_t)c * n + i] = make_double2(m * co, m * s);
}

__global__ __launch_bounds__(kEvalBlock) void forward_kernel(
    int32_t n, const int32_t *__restrict__ rp, const int32_t *__restrict__ ci, const double2 *__restrict__ yv,
    const int8_t *__restrict__ bt, const double2 *__restrict__ s_spec, int64_t s_ld, OutageView ov,
    const double2 *__restrict__ V, const double *__restrict__ m_res, int64_t ld, double2 *__restrict__ dS,
    double2 *__restrict__ w, double2 *__restrict__ aI, double2 *__restrict__ part, double2 *__restrict__ g_s) {
    __shared__ double red[2][kEvalBlock / kWave];
    int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    int32_t c = blockIdx.y;
    const double2 *Vc = V + (int64_t)c * n;
    double lsum = 0.0, lmax = 0.0;
    if (i < n) {
        double2 acc = csr_row(rp, ci, yv, i, n, [&](int32_t j) { return Vc[j]; });
        if (ov.outage) {
            int32_t k = ov.outage[c];
            if ((uint32_t)k < (uint32_t)ov.n_branch) {
                int32_t f = ov.from[k], t = ov.to[k];
                if ((i == f || i == t) && (uint32_t)f < (uint32_t)n && (uint32_t)t < (uint32_t)n)
                    acc = csub(acc, outage_term(ov, k, i, Vc[f], Vc[t], f, t));
            } else if (outage_index_bad(k, ov.n_branch)) {
                acc = make_double2(__longlong_as_double(0x7ff8000000000000LL), 0.0);  // NaN outputs
            }
        }
        double2 v = Vc[i];
        double2 s = s_spec[c * s_ld + i];
        double2 d = csub(cmulc(v, acc), s);
        int8_t ty = bt[i];
        double rP = ty != kSlack ? d.x : 0.0;
        double rQ = ty == kPQ ? d.y : 0.0;
        lsum = rP * rP + rQ * rQ;
        lmax = fmax(fabs(rP), fabs(rQ));
        double sc = 2.0 / *m_res;
        double2 a = make_double2(sc * rP, sc * rQ);
        int64_t o = (int64_t)c * n + i;
        w[o] = cmulc(a, v);
        aI[o] = cmul(a, acc);
        if (dS) dS[c * ld + i] = d;
        if (g_s) g_s[c * ld + i] = make_double2(-a.x, -a.y);  // d loss / d S_spec
    }
    lsum = wave_sum(lsum);
    lmax = wave_max(lmax);
    int wv = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0) {
        red[0][wv] = lsum;
        red[1][wv] = lmax;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0, m = 0.0;
        for (int k = 0; k < kEvalBlock / kWave; ++k) {
            s += red[0][k];
            m = fmax(m, red[1][k]);
        }
        part[(int64_t)c * gridDim.x + blockIdx.x] = make_double2(s, m);
    }
}

// loss and max|r| of case c from its block partials, by one wave in a fixed order
__device__ __forceinline__ void finalize_case(int32_t c, int32_t nblk, const double2 *__restrict__ part,
                                              const double *__restrict__ m_res, double *__restrict__ loss,
                                              double *__restrict__ max_mis) {
    double s = 0.0, m = 0.0;
    for (int32_t k = threadIdx.x; k < nblk; k += kWave) {
        const double2 p = part[(int64_t)c * nblk + k];
        s += p.x;
        m = fmax(m, p.y);
    }
    wave_last_sum_max(s, m);
    if (threadIdx.x != kWave - 1) return;
    const double mm = *m_res;
    loss[c] = mm > 0.0 ? s / mm : 0.0;
    // a NaN residual makes the sum NaN; report it in max_mis too
    max_mis[c] = isnan(s) ? __longlong_as_double(0x7ff8000000000000LL) : m;
}

__global__ __launch_bounds__(kEvalBlock) void adjoint_kernel(
    int32_t n, const int32_t *__restrict__ rp, const int32_t *__restrict__ ci, const double2 *__restrict__ yv,
    const int8_t *__restrict__ bt, OutageView ov, const double2 *__restrict__ V, const double *__restrict__ vm,
    int64_t ld, const double2 *__restrict__ w, const double2 *__restrict__ aI, double *__restrict__ g_vm,
    double *__restrict__ g_va, const double2 *__restrict__ part, const double *__restrict__ m_res,
    double *__restrict__ loss, double *__restrict__ max_mis) {
    int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    int32_t c = blockIdx.y;
    if (blockIdx.x == gridDim.x - 1) {  // one more block per case: its loss and max|r|
        if (threadIdx.x < kWave) finalize_case(c, (int32_t)gridDim.x - 1, part, m_res, loss, max_mis);
        return;
    }
    if (i >= n) return;
    const double2 *wc = w + (int64_t)c * n;
    double2 h = csr_row(rp, ci, yv, i, n, [&](int32_t j) { return wc[j]; });  // Y^T w with Y = Y^T
    if (ov.outage) {
        int32_t k = ov.outage[c];
        if ((uint32_t)k < (uint32_t)ov.n_branch) {
            int32_t f = ov.from[k], t = ov.to[k];
            if ((i == f || i == t) && (uint32_t)f < (uint32_t)n && (uint32_t)t < (uint32_t)n)
                h = csub(h, outage_term(ov, k, i, wc[f], wc[t], f, t));
        }
    }
    int64_t o = (int64_t)c * n + i;
    double2 G = cadd(aI[o], cconj(h));
    double2 v = V[o];
    int8_t ty = bt[i];
    // conj(G) V = (G.x v.x + G.y v.y) + j (G.x v.y - G.y v.x)
    double gv = ty == kPQ ? (G.x * v.x + G.y * v.y) / vm[c * ld + i] : 0.0;
    double ga = ty != kSlack ? (G.y * v.x - G.x * v.y) : 0.0;
    g_vm[c * ld + i] = gv;
    g_va[c * ld + i] = ga;
}

// d loss / d(r, x, b) of every branch, from V and the adjoint seed w = a conj(V)
// of the forward kernel.  With d loss = Re sum_i w_i dI_i and dI = dY V, a branch
// (f, t) with y = 1/(r + jx) and charging b contributes
//   dI_f = dy (V_f - V_t) + j (db/2) V_f,  dI_t = dy (V_t - V_f) + j (db/2) V_t,
// so with D = (w_f - w_t)(V_f - V_t) and dy = -y^2 (dr + j dx):
//   d/dr = -Re(y^2 D),  d/dx = Im(y^2 D),  d/db = -Im(w_f V_f + w_t V_t) / 2.
// The outaged branch of a case is absent from its Y: gradient 0.
template <typename GetV, typename GetW>
__device__ __forceinline__ void branch_grad(const OutageView &ov, int32_t e, int32_t n, bool out, GetV V, GetW w,
                                            double *__restrict__ g_r, double *__restrict__ g_x,
                                            double *__restrict__ g_b) {
    const int32_t f = ov.from[e], t = ov.to[e];
    double gr = 0.0, gx = 0.0, gb = 0.0;
    if (!out && f != t && (uint32_t)f < (uint32_t)n && (uint32_t)t < (uint32_t)n) {
        const double2 vf = V(f), vt = V(t), wf = w(f), wt = w(t);
        double2 y, ysh;
        branch_admittance(ov.r[e], ov.x[e], ov.b[e], y, ysh);
        const double2 D = cmul(csub(wf, wt), csub(vf, vt));
        const double2 y2D = cmul(cmul(y, y), D);
        gr = -y2D.x;
        gx = y2D.y;
        gb = -0.5 * (cmul(wf, vf).y + cmul(wt, vt).y);
    }
    g_r[e] = gr;
    g_x[e] = gx;
    g_b[e] = gb;
}

__global__ __launch_bounds__(kEvalBlock) void branch_grad_kernel(int32_t n, int32_t n_branch, OutageView ov,
                                                                  const double2 *__restrict__ V,
                                                                  const double2 *__restrict__ w, int64_t bld,
                                                                  double *__restrict__ g_r, double *__restrict__ g_x,
                                                                  double *__restrict__ g_b) {
    const int32_t e = blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t c = blockIdx.y;
    if (e >= n_branch) return;
    const int64_t o = (int64_t)c * n, q = (int64_t)c * bld;
    branch_grad(ov, e, n, ov.outage && ov.outage[c] == e, [&](int32_t i) { return V[o + i]; },
                [&](int32_t i) { return w[o + i]; }, g_r + q, g_x + q, g_b + q);
}

// What one call of the fused evaluation computes; null outputs are left out.
struct EvalArgs {
    int32_t n;
    const int32_t *rp;
    const int32_t *ci;
    const double2 *yv;
    const int8_t *bt;
    const double2 *s_spec;
    int64_t s_ld;
    OutageView ov;
    const double *vm;
    const double *va;
    int64_t ld;
    double2 *dS;    // [B][ld]
    double *loss;   // [B], with max_mis
    double *max_mis;
    double *g_vm;   // [B][ld], with g_va
    double *g_va;
    double2 *g_s;   // [B][ld]
    double *g_r;    // [B][bld], with g_x and g_b (BOTH)
    double *g_x;
    double *g_b;
    int64_t bld;
};

// The whole evaluation of one case in one workgroup: V in LDS, I of the thread's K rows
// in registers, w over V (or, BOTH, in a second array beside V, for the branch
// gradients), then the adjoint rows.  With conj(G) V = conj(a) V conj(I) + h V the
// gradient needs no a*I: a row keeps conj(a) (dS + S) instead of I.
// One launch instead of five and no V, w and a*I through memory (per bus and case 168 B
// before, 64 to 80 B here).  Bound by the chain of matrix load and LDS gather of every
// row: four lanes sharing a row, 16 rows per load and so a quarter of the cache lines
// per load, is 4 to 20% slower (1354 x 64 13.1 -> 15.7 us, 9241 x 256 81 -> 97), its
// gathers and sums being more.  A call on an MI355X, grids in an arbitrary numbering, five
// launches -> this: 118 buses x 8 cases 31 -> 15 us (host; its kernels 14 -> 6), 5000 x 256
// 124 -> 45, 9241 x 256 220 -> 76 (in a small-bandwidth numbering 185 -> 73); kernels with
// branch gradients, 1354 x 64, 21 -> 10.4.
template <int NT, int K, bool BOTH>
__global__ __launch_bounds__(NT) void eval_case_kernel(EvalArgs a) {
    extern __shared__ double2 X[];
    __shared__ double red[2][NT / kWave];
    __shared__ int cnt[NT / kWave];
    constexpr int NW = NT / kWave;
    const int tid = threadIdx.x, wv = tid / kWave;
    const int n = a.n, c = blockIdx.x;
    const int64_t cb = (int64_t)c * a.ld;
    const double *__restrict__ vm = a.vm + cb;
    const double *__restrict__ va = a.va + cb;
    const double2 *__restrict__ S = a.s_spec + (int64_t)c * a.s_ld;

    // V, and the residual count m = n_pv + 2 n_pq
    int m = 0;
    for (int i = tid; i < n; i += NT) {
        double sn, cs;
        fast_sincos(va[i], sn, cs);
        X[i] = make_double2(vm[i] * cs, vm[i] * sn);
        const int8_t t = a.bt[i];
        m += t == kPQ ? 2 : (t == kPV ? 1 : 0);
    }
    m = wave_isum(m);
    if ((tid & (kWave - 1)) == 0) cnt[wv] = m;

    // the outage: rows f and t lose the branch's pi-model block
    int of = -1, ot = -1;
    bool bad = false;
    double2 oy = make_double2(0.0, 0.0), oyd = oy;
    if (a.ov.outage) {
        const int32_t k = a.ov.outage[c];
        bad = outage_index_bad(k, a.ov.n_branch);
        if ((uint32_t)k < (uint32_t)a.ov.n_branch) {
            const int32_t f = a.ov.from[k], t = a.ov.to[k];
            if ((uint32_t)f < (uint32_t)n && (uint32_t)t < (uint32_t)n) {
                of = f;
                ot = t;
                double2 ysh;
                branch_admittance(a.ov.r[k], a.ov.x[k], a.ov.b[k], oy, ysh);
                oyd = cadd(oy, ysh);
            }
        }
    }
    auto row = [&](int i, const double2 *Z) {
        double2 acc = csr_row(a.rp, a.ci, a.yv, i, n, [&](int j) { return Z[j]; });
        if (i == of) acc = csub(acc, csub(cmul(oyd, Z[of]), cmul(oy, Z[ot])));
        else if (i == ot) acc = csub(acc, csub(cmul(oyd, Z[ot]), cmul(oy, Z[of])));
        return acc;
    };
    __syncthreads();
    m = 0;
    for (int k = 0; k < NW; ++k) m += cnt[k];
    const double scale = 2.0 / (double)m;

    // forward rows
    double2 T[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = tid + k * NT;
        T[k] = make_double2(0.0, 0.0);
        if (i < n) T[k] = bad ? make_double2(__longlong_as_double(0x7ff8000000000000LL), 0.0) : row(i, X);
    }
    if constexpr (!BOTH) __syncthreads();  // every row has read V; w takes its place
    double2 *W = BOTH ? X + n : X;
    double lsum = 0.0, lmax = 0.0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = tid + k * NT;
        if (i >= n) continue;
        const double2 v = X[i];
        const double2 p = cmulc(v, T[k]);
        const double2 d = csub(p, S[i]);
        const int8_t t = a.bt[i];
        const double rP = t != kSlack ? d.x : 0.0;
        const double rQ = t == kPQ ? d.y : 0.0;
        lsum += rP * rP + rQ * rQ;
        lmax = fmax(lmax, fmax(fabs(rP), fabs(rQ)));
        const double2 s = make_double2(scale * rP, scale * rQ);
        W[i] = cmulc(s, v);
        T[k] = cmulc(p, s);
        if (a.dS) a.dS[cb + i] = d;
        if (a.g_s) a.g_s[cb + i] = make_double2(-s.x, -s.y);  // d loss / d S_spec
    }
    wave_last_sum_max(lsum, lmax);
    if ((tid & (kWave - 1)) == kWave - 1) {
        red[0][wv] = lsum;
        red[1][wv] = lmax;
    }
    __syncthreads();
    if (a.loss && tid == 0) {
        double s = 0.0, mx = 0.0;
        for (int k = 0; k < NW; ++k) {
            s += red[0][k];
            mx = fmax(mx, red[1][k]);
        }
        a.loss[c] = m > 0 ? s / (double)m : 0.0;
        a.max_mis[c] = isnan(s) ? __longlong_as_double(0x7ff8000000000000LL) : mx;
    }
    if (a.g_vm) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int i = tid + k * NT;
            if (i >= n) continue;
            const double vmi = vm[i];
            double2 v;
            if constexpr (BOTH) {
                v = X[i];
            } else {
                double sn, cs;
                fast_sincos(va[i], sn, cs);
                v = make_double2(vmi * cs, vmi * sn);
            }
            const int8_t t = a.bt[i];
            const double2 hv = cmul(row(i, W), v);
            a.g_vm[cb + i] = t == kPQ ? (T[k].x + hv.x) / vmi : 0.0;
            a.g_va[cb + i] = t != kSlack ? -(T[k].y + hv.y) : 0.0;
        }
    }
    if constexpr (BOTH) {
        if (a.g_r) {
            const int64_t eb = (int64_t)c * a.bld;
            const int32_t out = a.ov.outage ? a.ov.outage[c] : -1;
            for (int e = tid; e < a.ov.n_branch; e += NT)
                branch_grad(a.ov, e, n, e == out, [&](int i) { return X[i]; }, [&](int i) { return W[i]; },
                            a.g_r + eb, a.g_x + eb, a.g_b + eb);
        }
    }
}

// grid (B) of one wave
__global__ __launch_bounds__(kWave) void finalize_kernel(int32_t nblk, const double2 *__restrict__ part,
                                                         const double *__restrict__ m_res, double *__restrict__ loss,
                                                         double *__restrict__ max_mis) {
    finalize_case(blockIdx.x, nblk, part, m_res, loss, max_mis);
}

}  // namespace dpf
