// learn.hip -- the learned part of the polynomial preconditioner.
//
//   * features of one system: row statistics of A, Gershgorin bounds of
//     D^-1 A, and the Ritz values of the Lanczos tridiagonal that 12
//     Jacobi-PCG iterations build (the CG-Lanczos relation; the iterations
//     run on the solve kernels, the tridiagonal's eigenvalues by Sturm-count
//     bisection, one thread per eigenvalue);
//   * the training label of one system: the smallest Ritz value lmin of its
//     full Jacobi-PCG solve (Sturm-sequence multisection on the tridiagonal
//     of all iterations), a = 3 lmin clamped to [1e-3 lmax, lmax / 2], and
//     the target p* = the Chebyshev semi-iterative polynomial on [a, lmax]
//     (its residual polynomial is the minimax one there), as the quadratic
//     form (G, h) of the loss;
//   * a 16 -> 64 -> 64 -> 9 tanh MLP in FP32: forward, loss, backward,
//     Adam, all with fixed reduction orders (deterministic).
//
// The polynomial is p(t) = sum_j c_j T_j(2 t / lmax - 1) on [0, lmax],
// lmax = the Gershgorin upper bound of D^-1 A.  Loss of one system:
//   L(c) = c'G c - 2 h'c + 1 + mu/Q sum_q max(0, eps - p(s_q))^2
// with G = G0 / kappa, h = G0 c* / kappa, kappa = c*' G0 c*,
// G0_jk = sum_q w_q t_q^2 T_j(y_q) T_k(y_q) over the 16-point Gauss-Chebyshev
// rule (t_q on [a, lmax], w_q = 1/16, y_q = 2 t_q / lmax - 1): the relative
// mean-square distance of the residual polynomial 1 - t p(t) from the
// minimax one, plus a positivity penalty on Q = 64 points s_q of [0, lmax].
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>

#include "internal.h"

namespace apcg {
namespace {

constexpr int FB = 256;   // block size of the row-statistics kernels
constexpr int MSTEPS = 12;
constexpr int NF = 16, NH = 64, NC = 9, NPARAM = 5833, QGRID = 64;
constexpr int LABEL_Q = 16;
constexpr double LABEL_SHIFT = 3.0;
constexpr double LABEL_FLOOR = 1e-3;  // keeps the target's minimum away from zero
constexpr int OFF_W1 = 0, OFF_B1 = 1024, OFF_W2 = 1088, OFF_B2 = 5184, OFF_W3 = 5248, OFF_B3 = 5824;
static_assert(OFF_B3 + NC == NPARAM, "parameter layout");

// Row statistics, pass 1 -> partials [7][G] (dev::RowStats order).
__global__ __launch_bounds__(FB) void k_feat_rows(int32_t n, const int32_t *__restrict__ rowptr,
                                                  const int32_t *__restrict__ col, const double *__restrict__ val,
                                                  double *part, int64_t per_block) {
    const dev::Chunk c = dev::block_chunk(n, per_block);
    dev::RowStats a;
    for (int64_t i = c.lo + threadIdx.x; i < c.hi; i += FB) dev::row_stats_add(a, rowptr, col, val, i);
    __shared__ double sh[7][FB];
    dev::row_stats_block<FB>(a, sh);
    if (threadIdx.x == 0) {
        const int lb = dev::xcd_block(blockIdx.x, gridDim.x);
        for (int k = 0; k < 7; ++k) part[k * gridDim.x + lb] = a.v[k];
    }
}

// One workgroup of FB: pass-1 totals -> stats[0..6] (stats[7] = mean ln d);
// thread t merges partials t, t + FB, ..., then the fixed tree.
__global__ __launch_bounds__(FB) void k_feat_rows_final(const double *part, int G, int32_t n, double *stats) {
    dev::RowStats a;
    for (int g = threadIdx.x; g < G; g += FB) {
        double b[7];
        for (int k = 0; k < 7; ++k) b[k] = part[k * G + g];
        dev::row_stats_merge(a, b);
    }
    __shared__ double sh[7][FB];
    dev::row_stats_block<FB>(a, sh);
    if (threadIdx.x != 0) return;
    for (int k = 0; k < 7; ++k) stats[k] = a.v[k];
    stats[7] = a.v[4] / (double)n;
}

// Pass 2: partials of sum (ln d_i - mean)^2 (two-pass variance).
__global__ __launch_bounds__(FB) void k_feat_rows2(int32_t n, const int32_t *__restrict__ rowptr,
                                                   const int32_t *__restrict__ col, const double *__restrict__ val,
                                                   const double *stats, double *part, int64_t per_block) {
    const dev::Chunk c = dev::block_chunk(n, per_block);
    const double mean = stats[7];
    double acc = 0.0;
    for (int64_t i = c.lo + threadIdx.x; i < c.hi; i += FB) {
        const double e = dev::row_logdiag(rowptr, col, val, i) - mean;
        acc = fma(e, e, acc);
    }
    double v[1] = {acc};
    dev::store_partials<FB, 1>(v, part, gridDim.x, dev::xcd_block(blockIdx.x, gridDim.x));
}

__device__ double cheb(int j, double y) {  // T_j(y) by the recurrence, any real y
    double t0 = 1.0, t1 = y;
    if (j == 0) return t0;
    for (int k = 2; k <= j; ++k) {
        const double t2 = 2.0 * y * t1 - t0;
        t0 = t1;
        t1 = t2;
    }
    return t1;
}

// One workgroup of 64: thread i < m finds the i-th smallest Ritz value (the
// eigenvalues of the 12-step Lanczos tridiagonal); thread 0 then forms the
// 16 features (FP32) and lmax (FP64).
__global__ __launch_bounds__(64) void k_feat_final(const double *stats, const double *var_part, int Gv,
                                                   const double *hist, int hist_cap, const apcg_solve_info *info,
                                                   int32_t n, int64_t nnz, float *feat, double *lmax_out) {
    int m = info->iterations;
    if (m > hist_cap) m = hist_cap;
    if (m > 16) m = 16;
    const double *al = hist, *be = hist + hist_cap;
    __shared__ double th[16], td[16], te2[16];
    dev::ritz_values(al, be, m, td, te2, th);
    double vs[1];
    dev::reduce_partials<64, 1>(var_part, Gv, vs);  // sum of squared deviations, fixed order
    __syncthreads();
    if (threadIdx.x != 0) return;
    if (m < 1) {  // no iteration (b = 0): lmax stands in as the only Ritz value
        th[0] = stats[1];
        m = 1;
    }
    const double var = vs[0];
    const double relres = info->ref_norm > 0.0 ? info->res_norm / info->ref_norm : 1.0;
    dev::feature_vector(stats, var, th, m, relres, n, nnz, feat);
    *lmax_out = stats[1];
}

// One workgroup of 64: the smallest eigenvalue by multisection (each round
// splits the bracket into 65 parts and keeps the one where the count first
// reaches 1), then the interval, the target's coefficients (interpolation at
// the 9 Chebyshev points, exact for a degree-8 polynomial:
// c_j = (2 - [j = 0]) / 9 sum_k p*(t(y_k)) T_j(y_k), y_k = cos(pi (k + 1/2) / 9))
// and the loss's normalised quadratic form.
__global__ __launch_bounds__(64) void k_label(const double *stats, const double *hist, int cap,
                                              const apcg_solve_info *info, float *Gout, float *hout,
                                              double *lab) {
    const double hi = stats[1];
    int m = info->iterations;
    if (m > cap) m = cap;
    const double *al = hist, *be = hist + cap;
    __shared__ double s_lo, s_hi;
    __shared__ int first;
    if (threadIdx.x == 0) {
        s_lo = -0.5 * hi;
        s_hi = 1.5 * hi;
    }
    __syncthreads();
    if (m > 0) {
        for (int round = 0; round < 10; ++round) {
            const double lo = s_lo, w = (s_hi - lo) / 65.0;
            const double x = lo + w * (threadIdx.x + 1);
            const bool hit = dev::sturm_below(al, be, m, x) >= 1;
            if (threadIdx.x == 0) first = 64;
            __syncthreads();
            if (hit) atomicMin(&first, (int)threadIdx.x);
            __syncthreads();
            if (threadIdx.x == 0) {
                const int f = first;
                s_lo = lo + w * f;  // count(lo + w f) == 0 (f = 0: the old lower end)
                if (f < 64) s_hi = lo + w * (f + 1);
            }
            __syncthreads();
        }
    }
    if (threadIdx.x != 0) return;
    const double lmin = m > 0 ? 0.5 * (s_lo + s_hi) : 0.0;
    double a = 0.5 * hi;
    if (m > 0) a = fmin(fmax(LABEL_SHIFT * lmin, LABEL_FLOOR * hi), 0.5 * hi);
    // target coefficients
    const double s0 = (hi + a) / (hi - a), T9s0 = cheb(9, s0);
    double cs[NC];
    for (int j = 0; j < NC; ++j) cs[j] = 0.0;
    for (int k = 0; k < NC; ++k) {
        const double y = cos(M_PI * (k + 0.5) / NC);
        const double t = 0.5 * (y + 1.0) * hi;
        const double pv = (1.0 - cheb(9, (hi + a - 2.0 * t) / (hi - a)) / T9s0) / t;
        for (int j = 0; j < NC; ++j) cs[j] += pv * cheb(j, y);
    }
    for (int j = 0; j < NC; ++j) cs[j] *= (j == 0 ? 1.0 : 2.0) / NC;
    // G0 over the Gauss-Chebyshev rule on [a, hi]
    double G[NC][NC];
    for (int j = 0; j < NC; ++j)
        for (int k = 0; k < NC; ++k) G[j][k] = 0.0;
    for (int q = 0; q < LABEL_Q; ++q) {
        const double t = 0.5 * (a + hi) + 0.5 * (hi - a) * cos((2 * q + 1) * M_PI / (2 * LABEL_Q));
        const double y = 2.0 * t / hi - 1.0, w = 1.0 / LABEL_Q;
        double T[NC];
        T[0] = 1.0;
        T[1] = y;
        for (int j = 2; j < NC; ++j) T[j] = 2.0 * y * T[j - 1] - T[j - 2];
        for (int j = 0; j < NC; ++j)
            for (int k = 0; k < NC; ++k) G[j][k] += w * t * t * T[j] * T[k];
    }
    double Gc[NC], kappa = 0.0;
    for (int j = 0; j < NC; ++j) {
        Gc[j] = 0.0;
        for (int k = 0; k < NC; ++k) Gc[j] += G[j][k] * cs[k];
        kappa += cs[j] * Gc[j];
    }
    for (int j = 0; j < NC; ++j) {
        hout[j] = (float)(Gc[j] / kappa);
        for (int k = 0; k < NC; ++k) Gout[j * NC + k] = (float)(G[j][k] / kappa);
    }
    lab[0] = lmin;
    lab[1] = a;
    lab[2] = hi;
}

// ----------------------------------------------------------------- MLP
__global__ void k_phi_grid(float *phi) {
    const int q = threadIdx.x;  // Q = 64 threads
    if (q >= QGRID) return;
    const double y = -1.0 + 2.0 * q / (QGRID - 1);
    for (int j = 0; j < NC; ++j) phi[q * NC + j] = (float)cheb(j, y);
}

// One workgroup of 64 threads per sample.
__global__ __launch_bounds__(64) void k_mlp_fwd(const float *__restrict__ P, const float *__restrict__ X, int B,
                                                float *__restrict__ C) {
    const int b = blockIdx.x, j = threadIdx.x;
    if (b >= B) return;
    __shared__ float x[NF], h1[NH], h2[NH];
    if (j < NF) x[j] = X[b * NF + j];
    __syncthreads();
    float a = P[OFF_B1 + j];
    for (int k = 0; k < NF; ++k) a = fmaf(P[OFF_W1 + j * NF + k], x[k], a);
    const float t1 = tanhf(a);
    h1[j] = t1;
    __syncthreads();
    a = P[OFF_B2 + j];
    for (int k = 0; k < NH; ++k) a = fmaf(P[OFF_W2 + j * NH + k], h1[k], a);
    const float t2 = tanhf(a);
    h2[j] = t2;
    __syncthreads();
    if (j < NC) {
        a = P[OFF_B3 + j];
        for (int k = 0; k < NH; ++k) a = fmaf(P[OFF_W3 + j * NH + k], h2[k], a);
        C[b * NC + j] = a;
    }
}

// Everything of a training step that belongs to one sample, one wavefront
// each, four to a workgroup that brings the weights through LDS once: the
// network, the loss, dL/dc (divided by B for the mean loss) and the
// back-propagated activation gradients dA2 = (dC W3) (1 - h2^2), dA1 =
// (dA2 W2) (1 - h1^2).  What bounds it is latency: as three kernels of one
// wavefront a workgroup, each reading its weights row by row from the caches,
// 11 us for 128 samples; 7.7 here (13 with the loads of one table waiting for
// those of the last).
constexpr int SPW = 4;  // samples (wavefronts) per workgroup
__global__ __launch_bounds__(64 * SPW) void k_mlp_sample(const float *__restrict__ P, const float *__restrict__ X,
                                                         const float *__restrict__ G, const float *__restrict__ h,
                                                         const float *__restrict__ phi_in, int B, float mu, float eps,
                                                         float *__restrict__ H1, float *__restrict__ H2,
                                                         float *__restrict__ dC, float *__restrict__ dA1,
                                                         float *__restrict__ dA2, float *__restrict__ loss_b) {
    // rows an odd number of words apart: lanes reading a column hit different banks
    __shared__ float w1[NH][NF + 1], w2[NH][NH + 1], w3[NC][NH + 1], b1[NH], b2[NH], b3[NC], phi[QGRID * NC];
    struct Sample {
        float x[NF], h1[NH], h2[NH], da2[NH], viol[QGRID], g[NC * NC], h[NC], c[NC], dc[NC], gc[NC];
    };
    __shared__ Sample all[SPW];
    const int tid = threadIdx.x, wave = tid >> 6, j = tid & 63, b = blockIdx.x * SPW + wave;
    Sample &s = all[wave];
    // everything this thread brings, all of it in flight before the first use
    constexpr int NT = 64 * SPW, N3 = (NC * NH + NT - 1) / NT, NP = (QGRID * NC + NT - 1) / NT, NG = (NC * NC + 63) / 64;
    static_assert(NH * NF % NT == 0 && NH * NH % NT == 0 && 2 * NH + NC <= NT, "shares of a thread");
    const int bs = min(b, B - 1);
    float v1[NH * NF / NT], v2[NH * NH / NT], v3[N3], vp[NP], vg[NG];
    const float vx = X[bs * NF + j % NF], vh = h[bs * NC + j % NC];
#pragma unroll
    for (int q = 0; q < NG; ++q) vg[q] = G[bs * NC * NC + min(q * 64 + j, NC * NC - 1)];
#pragma unroll
    for (int q = 0; q < NH * NF / NT; ++q) v1[q] = P[OFF_W1 + q * NT + tid];
#pragma unroll
    for (int q = 0; q < NH * NH / NT; ++q) v2[q] = P[OFF_W2 + q * NT + tid];
#pragma unroll
    for (int q = 0; q < N3; ++q) v3[q] = P[OFF_W3 + min(q * NT + tid, NC * NH - 1)];
#pragma unroll
    for (int q = 0; q < NP; ++q) vp[q] = phi_in[min(q * NT + tid, QGRID * NC - 1)];
    const float vb = P[tid < NH ? OFF_B1 + tid : tid < 2 * NH ? OFF_B2 + tid - NH : OFF_B3 + min(tid - 2 * NH, NC - 1)];
    __builtin_amdgcn_sched_barrier(0);
    if (j < NF) s.x[j] = vx;
    if (j < NC) s.h[j] = vh;
#pragma unroll
    for (int q = 0; q < NG; ++q)
        if (q * 64 + j < NC * NC) s.g[q * 64 + j] = vg[q];
#pragma unroll
    for (int q = 0; q < NH * NF / NT; ++q) w1[(q * NT + tid) / NF][tid % NF] = v1[q];
#pragma unroll
    for (int q = 0; q < NH * NH / NT; ++q) w2[(q * NT + tid) / NH][tid % NH] = v2[q];
#pragma unroll
    for (int q = 0; q < N3; ++q)
        if (q * NT + tid < NC * NH) w3[(q * NT + tid) / NH][tid % NH] = v3[q];
#pragma unroll
    for (int q = 0; q < NP; ++q)
        if (q * NT + tid < QGRID * NC) phi[q * NT + tid] = vp[q];
    if (tid < NH) b1[tid] = vb;
    else if (tid < 2 * NH) b2[tid - NH] = vb;
    else if (tid < 2 * NH + NC) b3[tid - 2 * NH] = vb;
    __syncthreads();
    if (b >= B) return;
    float a = b1[j];
#pragma unroll
    for (int k = 0; k < NF; ++k) a = fmaf(w1[j][k], s.x[k], a);
    const float h1 = tanhf(a);
    s.h1[j] = h1;
    dev::wave_lds_fence();
    a = b2[j];
#pragma unroll
    for (int k = 0; k < NH; ++k) a = fmaf(w2[j][k], s.h1[k], a);
    const float h2 = tanhf(a);
    s.h2[j] = h2;
    dev::wave_lds_fence();
    if (j < NC) {
        a = b3[j];
#pragma unroll
        for (int k = 0; k < NH; ++k) a = fmaf(w3[j][k], s.h2[k], a);
        s.c[j] = a;
    }
    dev::wave_lds_fence();
    float q = 0.f;
#pragma unroll
    for (int k = 0; k < NC; ++k) q = fmaf(phi[j * NC + k], s.c[k], q);
    s.viol[j] = fmaxf(0.f, eps - q);
    dev::wave_lds_fence();
    const float scale = mu / (float)QGRID;
    if (j < NC) {
        float g = -2.f * s.h[j], gc = 0.f, pen = 0.f;
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            g = fmaf(2.f * s.g[j * NC + k], s.c[k], g);
            gc = fmaf(s.g[j * NC + k], s.c[k], gc);
        }
#pragma unroll
        for (int k = 0; k < QGRID; ++k) pen = fmaf(s.viol[k], phi[k * NC + j], pen);
        g = fmaf(-2.f * scale, pen, g);
        s.dc[j] = g / (float)B;
        s.gc[j] = gc;
        dC[b * NC + j] = s.dc[j];
    }
    dev::wave_lds_fence();
    a = 0.f;
#pragma unroll
    for (int o = 0; o < NC; ++o) a = fmaf(s.dc[o], w3[o][j], a);
    const float d2 = a * (1.f - h2 * h2);
    s.da2[j] = d2;
    dev::wave_lds_fence();
    a = 0.f;
#pragma unroll
    for (int k = 0; k < NH; ++k) a = fmaf(s.da2[k], w2[k][j], a);
    H1[b * NH + j] = h1;
    H2[b * NH + j] = h2;
    dA2[b * NH + j] = d2;
    dA1[b * NH + j] = a * (1.f - h1 * h1);
    if (j == 0) {
        float L = 1.f, pen = 0.f;
#pragma unroll
        for (int k = 0; k < NC; ++k) L = fmaf(s.c[k], s.gc[k] - 2.f * s.h[k], L);
#pragma unroll
        for (int k = 0; k < QGRID; ++k) pen = fmaf(s.viol[k], s.viol[k], pen);
        loss_b[b] = fmaf(scale, pen, L);
    }
}

struct Adam {
    float *P, *m, *v;  // P == nullptr: no step
    int t;
    float lr, b1, b2, eps;
};

__device__ __forceinline__ void adam_step(const Adam &o, int p, float gi) {
    const float mi = o.b1 * o.m[p] + (1.f - o.b1) * gi;
    const float vi = o.b2 * o.v[p] + (1.f - o.b2) * gi * gi;
    o.m[p] = mi;
    o.v[p] = vi;
    const float mh = mi / (1.f - powf(o.b1, (float)o.t));
    const float vh = vi / (1.f - powf(o.b2, (float)o.t));
    o.P[p] -= o.lr * mh / (sqrtf(vh) + o.eps);
}

// Parameter gradients, one thread per parameter, the sum over samples in
// order, and the Adam step on them; the last workgroup forms the mean loss.
// Each layer's gradient is the product of two activation arrays over the
// samples: a workgroup takes 16 x 16 of its entries and brings GCH samples of
// both arrays through LDS at a time, the next ones in flight (a thread per
// parameter reading both for every sample waited for the caches: 33 us at 128
// samples, and 7 and 4 for the loss and the step in kernels of their own;
// 5.3 in all here).
constexpr int GCH = 128;
constexpr int GRAD_TILES = NH / 16 + (NH / 16) * (NH / 16) + NH / 16;
__global__ __launch_bounds__(256) void k_mlp_grad(const float *__restrict__ X, const float *__restrict__ H1,
                                                  const float *__restrict__ H2, const float *__restrict__ dC,
                                                  const float *__restrict__ dA1, const float *__restrict__ dA2, int B,
                                                  const float *__restrict__ loss_b, float *__restrict__ loss,
                                                  float *__restrict__ grad, Adam adam) {
    __shared__ float sa[GCH][16], sb[GCH][16];
    const int tid = threadIdx.x;
    if (blockIdx.x == GRAD_TILES) {
        double s = 0.0;
        float *l = sa[0];
        for (int c0 = 0; c0 < B; c0 += GCH * 16) {
            const int cnt = min(GCH * 16, B - c0);
            __syncthreads();
#pragma unroll
            for (int q = 0; q < GCH * 16 / 256; ++q)
                if (q * 256 + tid < cnt) l[q * 256 + tid] = loss_b[c0 + q * 256 + tid];
            __syncthreads();
            if (tid == 0) {
#pragma unroll 8
                for (int k = 0; k < cnt; ++k) s += l[k];
            }
        }
        if (tid == 0) *loss = (float)(s / B);
        return;
    }
    // entries (row, k) of dA1 x X, dA2 x H1 or dC x H2: rows and columns of
    // this tile, and where W and the bias of the layer lie
    const float *ra, *rb;
    int na, nb, row0, k0, off_w, off_b;
    const int t = blockIdx.x;
    if (t < NH / 16) {
        ra = dA1, rb = X, na = NH, nb = NF, row0 = 16 * t, k0 = 0, off_w = OFF_W1, off_b = OFF_B1;
    } else if (t < NH / 16 + NH / 16 * (NH / 16)) {
        const int u = t - NH / 16;
        ra = dA2, rb = H1, na = NH, nb = NH, row0 = 16 * (u / (NH / 16)), k0 = 16 * (u % (NH / 16));
        off_w = OFF_W2, off_b = OFF_B2;
    } else {
        ra = dC, rb = H2, na = NC, nb = NH, row0 = 0, k0 = 16 * (t - NH / 16 - NH / 16 * (NH / 16));
        off_w = OFF_W3, off_b = OFF_B3;
    }
    const int r = tid / 16, k = tid % 16;
    constexpr int PT = GCH * 16 / 256;  // staged entries of either array per thread
    const int ca = row0 + k < na ? row0 + k : 0;  // (the output layer has 9 rows)
    float va[PT], vb[PT];
    auto fetch = [&](int c0) {
#pragma unroll
        for (int q = 0; q < PT; ++q) {
            const int b = min(c0 + q * 16 + r, B - 1);
            va[q] = ra[b * na + ca];
            vb[q] = rb[b * nb + k0 + k];
        }
    };
    float g = 0.f, gb = 0.f;
    fetch(0);
    for (int c0 = 0; c0 < B; c0 += GCH) {
        const int cnt = min(GCH, B - c0);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PT; ++q) {
            sa[q * 16 + r][k] = va[q];
            sb[q * 16 + r][k] = vb[q];
        }
        __syncthreads();
        if (c0 + GCH < B) fetch(c0 + GCH);
#pragma unroll 16
        for (int b = 0; b < cnt; ++b) {
            g = fmaf(sa[b][r], sb[b][k], g);
            gb += sa[b][r];
        }
    }
    if (row0 + r >= na) return;
    const int p = off_w + (row0 + r) * nb + k0 + k, pb = off_b + row0 + r;
    const bool bias = k0 == 0 && k == 0;
    if (grad) {
        grad[p] = g;
        if (bias) grad[pb] = gb;
    }
    if (adam.P) {
        adam_step(adam, p, g);
        if (bias) adam_step(adam, pb, gb);
    }
}

// Column statistics (two-pass) and in-place standardisation of X [B, 16].
__global__ void k_standardize(float *X, int B, float *mean, float *stdv, int compute) {
    const int f = threadIdx.x;
    if (f >= NF) return;
    if (compute) {
        double s = 0.0;
        for (int b = 0; b < B; ++b) s += X[b * NF + f];
        const double mu = s / B;
        double q = 0.0;
        for (int b = 0; b < B; ++b) {
            const double e = X[b * NF + f] - mu;
            q += e * e;
        }
        const double sd = sqrt(q / B);
        mean[f] = (float)mu;
        stdv[f] = (float)(sd > 1e-12 ? sd : 1.0);
    }
    const float mu = mean[f], sd = stdv[f];
    for (int b = 0; b < B; ++b) X[b * NF + f] = (X[b * NF + f] - mu) / sd;
}

// Per-context MLP scratch (activations and gradients for up to cap samples).
struct MlpScratch {
    int device = 0;
    int64_t cap = 0;
    float *buf = nullptr;  // H1, H2, dA1, dA2, dC, loss_b, phi
    float *H1() const { return buf; }
    float *H2() const { return buf + cap * NH; }
    float *dA1() const { return buf + 2 * cap * NH; }
    float *dA2() const { return buf + 3 * cap * NH; }
    float *dC() const { return buf + 4 * cap * NH; }
    float *loss_b() const { return dC() + cap * NC; }
    float *phi() const { return loss_b() + cap; }
    static size_t floats(int64_t cap) { return (size_t)(4 * cap * NH + cap * NC + cap + QGRID * NC); }
};

struct FeatScratch {
    int device = 0;
    int64_t cap = 0;
    double *x = nullptr;      // n doubles
    double *stats = nullptr;  // 8 + partials
    double *hist = nullptr;   // 2 * MSTEPS
    double *lhist = nullptr;  // 2 * lhist_cap: alpha, beta of a full solve
    int64_t lhist_cap = 0;
    float *fbuf = nullptr;    // learned solve: features [16], coefficients [9]
    double *dbuf = nullptr;   // learned solve: lmax
    apcg_info info = nullptr;
};

}  // namespace

static std::mutex g_learn_mu;
static std::vector<std::pair<uint64_t, MlpScratch *>> g_mlp;
static std::vector<std::pair<uint64_t, FeatScratch *>> g_feat;

static MlpScratch *mlp_scratch(apcg_ctx c) {
    std::lock_guard<std::mutex> lk(g_learn_mu);
    for (auto &p : g_mlp)
        if (p.first == c->id) return p.second;
    MlpScratch *s = new MlpScratch();
    s->device = c->device;
    g_mlp.emplace_back(c->id, s);
    return s;
}

static FeatScratch *feat_scratch(apcg_ctx c) {
    std::lock_guard<std::mutex> lk(g_learn_mu);
    for (auto &p : g_feat)
        if (p.first == c->id) return p.second;
    FeatScratch *s = new FeatScratch();
    s->device = c->device;
    g_feat.emplace_back(c->id, s);
    return s;
}

void learn_cache_release(uint64_t ctx_id, int device) {
    MlpScratch *m = nullptr;
    FeatScratch *f = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_learn_mu);
        for (auto it = g_mlp.begin(); it != g_mlp.end(); ++it)
            if (it->first == ctx_id) {
                m = it->second;
                g_mlp.erase(it);
                break;
            }
        for (auto it = g_feat.begin(); it != g_feat.end(); ++it)
            if (it->first == ctx_id) {
                f = it->second;
                g_feat.erase(it);
                break;
            }
    }
    hipSetDevice(device);
    if (m) {
        hipFree(m->buf);
        delete m;
    }
    if (f) {
        hipFree(f->x);
        hipFree(f->stats);
        hipFree(f->hist);
        hipFree(f->lhist);
        hipFree(f->fbuf);
        hipFree(f->dbuf);
        if (f->info) apcg_info_destroy(f->info);
        delete f;
    }
}

static apcg_status ensure_mlp(apcg_ctx c, MlpScratch *s, int64_t B) {
    if (s->buf && s->cap >= B) return APCG_SUCCESS;
    if (s->buf) {
        EventRef ev = event_get(c->device);
        if (!ev) return set_error(APCG_ERR_HIP, "event creation failed");
        APCG_HIP(event_record(ev, c->stream));
        float *old = s->buf;
        const int dev = c->device;
        defer_release({ev}, [old, dev]() {
            hipSetDevice(dev);
            hipFree(old);
        });
        s->buf = nullptr;
    }
    const int64_t cap = std::max<int64_t>(B, 256);
    APCG_HIP(hipMalloc((void **)&s->buf, sizeof(float) * MlpScratch::floats(cap)));
    s->cap = cap;
    hipLaunchKernelGGL(k_phi_grid, dim3(1), dim3(64), 0, c->stream, s->phi());
    APCG_CHECK_LAUNCH("k_phi_grid");
    return APCG_SUCCESS;
}

apcg_status mlp_infer(apcg_ctx ctx, const float *params, const float *mean, const float *std, float *X, int32_t B,
                      float *C) {
    if (B < 1) return APCG_SUCCESS;
    hipLaunchKernelGGL(k_standardize, dim3(1), dim3(64), 0, ctx->stream, X, B, (float *)mean, (float *)std, 0);
    APCG_CHECK_LAUNCH("k_standardize");
    hipLaunchKernelGGL(k_mlp_fwd, dim3(B), dim3(64), 0, ctx->stream, params, (const float *)X, B, C);
    APCG_CHECK_LAUNCH("k_mlp_fwd");
    return APCG_SUCCESS;
}

// Allocates the per-context feature scratch for n rows (ordered after the
// context's pending work when it grows).
static apcg_status feat_prepare(apcg_ctx ctx, FeatScratch *fs, int64_t n) {
    apcg_status s;
    if (!fs->stats) {
        APCG_HIP(hipMalloc((void **)&fs->stats, sizeof(double) * (8 + 8 * (int64_t)kMaxBlocks)));
        APCG_HIP(hipMalloc((void **)&fs->hist, sizeof(double) * 2 * MSTEPS));
        APCG_HIP(hipMalloc((void **)&fs->fbuf, sizeof(float) * 32));
        APCG_HIP(hipMalloc((void **)&fs->dbuf, sizeof(double) * 4));
        if ((s = apcg_info_create(ctx->device, 1, &fs->info))) return s;
    }
    if (fs->cap < n) {
        if (fs->x) {
            EventRef ev = event_get(ctx->device);
            if (!ev) return set_error(APCG_ERR_HIP, "event creation failed");
            APCG_HIP(event_record(ev, ctx->stream));
            double *old = fs->x;
            const int dev = ctx->device;
            defer_release({ev}, [old, dev]() {
                hipSetDevice(dev);
                hipFree(old);
            });
            fs->x = nullptr;
        }
        APCG_HIP(hipMalloc((void **)&fs->x, sizeof(double) * n));
        fs->cap = n;
    }
    return APCG_SUCCESS;
}

// Row statistics (both passes) into fs->stats; partials after the first 8.
static apcg_status feat_rows(apcg_ctx ctx, apcg_mat A, FeatScratch *fs, int *G_out) {
    hipStream_t st = ctx->stream;
    int G;
    int64_t pb;
    elementwise_grid(A->n, &G, &pb);
    double *part = fs->stats + 8;
    hipLaunchKernelGGL(k_feat_rows, dim3(G), dim3(FB), 0, st, A->n, A->rowptr, A->col, A->val, part, pb);
    APCG_CHECK_LAUNCH("k_feat_rows");
    hipLaunchKernelGGL(k_feat_rows_final, dim3(1), dim3(FB), 0, st, (const double *)part, G, A->n, fs->stats);
    APCG_CHECK_LAUNCH("k_feat_rows_final");
    hipLaunchKernelGGL(k_feat_rows2, dim3(G), dim3(FB), 0, st, A->n, A->rowptr, A->col, A->val,
                       (const double *)fs->stats, part, pb);
    APCG_CHECK_LAUNCH("k_feat_rows2");
    *G_out = G;
    return APCG_SUCCESS;
}

static apcg_status check_system(apcg_ctx ctx, apcg_mat A, apcg_vec b) {
    if (!ctx || !A || !b) return set_error(APCG_ERR_INVALID_ARG, "NULL argument");
    if (b->n != A->n || A->n < 1) return set_error(APCG_ERR_INVALID_ARG, "dimension mismatch or empty system");
    if (ctx->device != A->device || b->device != A->device)
        return set_error(APCG_ERR_INVALID_ARG, "operands on different devices");
    return APCG_SUCCESS;
}

// Features into dev_feat[16] / dev_lmax[1] (device pointers), on ctx.
static apcg_status features_into(apcg_ctx ctx, apcg_mat A, apcg_vec b, float *dev_feat, double *dev_lmax) {
    FeatScratch *fs = feat_scratch(ctx);
    apcg_status s;
    APCG_HIP(hipSetDevice(ctx->device));
    if ((s = feat_prepare(ctx, fs, A->n))) return s;
    // 12 Jacobi-PCG steps from x0 = 0 with rtol = 0 record alpha and beta
    apcg_vec_s xv;
    xv.device = ctx->device;
    xv.d = fs->x;
    xv.n = A->n;
    apcg_solve_opts o;
    apcg_solve_opts_default(&o);
    o.x0_is_zero = 1;
    o.iters_per_graph = MSTEPS;  // one captured period, cached per matrix like the solve's
    if ((s = pcg_solve_marked(ctx, A, b, &xv, 0.0, MSTEPS, &o, fs->info, 0, fs->hist, MSTEPS))) return s;
    Acc acc[2] = {{&A->rec, ACC_R}, {&b->rec, ACC_R}};
    if ((s = op_begin(ctx, acc, 2))) return s;
    int G;
    if ((s = feat_rows(ctx, A, fs, &G))) return s;
    hipLaunchKernelGGL(k_feat_final, dim3(1), dim3(64), 0, ctx->stream, (const double *)fs->stats,
                       (const double *)(fs->stats + 8), G, (const double *)fs->hist, MSTEPS,
                       (const apcg_solve_info *)fs->info->d, A->n, A->nnz, dev_feat, dev_lmax);
    APCG_CHECK_LAUNCH("k_feat_final");
    return op_end(ctx, acc, 2);
}

}  // namespace apcg

using namespace apcg;

extern "C" {

apcg_status apcg_pc_features(apcg_ctx ctx, apcg_mat A, apcg_vec b, float *dev_feat, double *dev_lmax) {
    try {
        apcg_status s;
        if ((s = check_system(ctx, A, b))) return s;
        if (!dev_feat || !dev_lmax) return set_error(APCG_ERR_INVALID_ARG, "NULL argument");
        return features_into(ctx, A, b, dev_feat, dev_lmax);
    } catch (const std::bad_alloc &) {
        return set_error(APCG_ERR_OUT_OF_MEMORY, "host allocation failed");
    }
}

apcg_status apcg_pc_label(apcg_ctx ctx, apcg_mat A, apcg_vec b, double rtol, int32_t maxit, float *dev_G,
                          float *dev_h, double *dev_label) {
    try {
        apcg_status s;
        if ((s = check_system(ctx, A, b))) return s;
        if (!dev_G || !dev_h || !dev_label) return set_error(APCG_ERR_INVALID_ARG, "NULL argument");
        if (maxit < 1) return set_error(APCG_ERR_INVALID_ARG, "maxit must be >= 1");
        FeatScratch *fs = feat_scratch(ctx);
        APCG_HIP(hipSetDevice(ctx->device));
        if ((s = feat_prepare(ctx, fs, A->n))) return s;
        if (fs->lhist_cap < maxit) {
            if (fs->lhist) {
                EventRef ev = event_get(ctx->device);
                if (!ev) return set_error(APCG_ERR_HIP, "event creation failed");
                APCG_HIP(event_record(ev, ctx->stream));
                double *old = fs->lhist;
                const int dev = ctx->device;
                defer_release({ev}, [old, dev]() {
                    hipSetDevice(dev);
                    hipFree(old);
                });
                fs->lhist = nullptr;
            }
            APCG_HIP(hipMalloc((void **)&fs->lhist, sizeof(double) * 2 * (int64_t)maxit));
            fs->lhist_cap = maxit;
        }
        const int cap = (int)fs->lhist_cap;
        apcg_vec_s xv;
        xv.device = ctx->device;
        xv.d = fs->x;
        xv.n = A->n;
        apcg_solve_opts o;
        apcg_solve_opts_default(&o);
        o.x0_is_zero = 1;
        if ((s = pcg_solve_marked(ctx, A, b, &xv, rtol, maxit, &o, fs->info, 0, fs->lhist, cap))) return s;
        Acc acc[2] = {{&A->rec, ACC_R}, {&b->rec, ACC_R}};
        if ((s = op_begin(ctx, acc, 2))) return s;
        int G;
        if ((s = feat_rows(ctx, A, fs, &G))) return s;
        hipLaunchKernelGGL(k_label, dim3(1), dim3(64), 0, ctx->stream, (const double *)fs->stats,
                           (const double *)fs->lhist, cap, (const apcg_solve_info *)fs->info->d, dev_G, dev_h,
                           dev_label);
        APCG_CHECK_LAUNCH("k_label");
        return op_end(ctx, acc, 2);
    } catch (const std::bad_alloc &) {
        return set_error(APCG_ERR_OUT_OF_MEMORY, "host allocation failed");
    }
}

apcg_status apcg_ksp_solve_learned(apcg_ctx ctx, apcg_mat A, apcg_vec b, apcg_vec x, double rtol, int32_t maxit,
                                   const float *dev_params, const float *dev_mean, const float *dev_std,
                                   const apcg_solve_opts *opts, const apcg_fcg_opts *fopts, apcg_info info,
                                   int32_t info_index) {
    try {
        apcg_status s;
        if ((s = check_system(ctx, A, b))) return s;
        if (!dev_params || !dev_mean || !dev_std) return set_error(APCG_ERR_INVALID_ARG, "NULL network argument");
        FeatScratch *fs = feat_scratch(ctx);
        APCG_HIP(hipSetDevice(ctx->device));
        if ((s = feat_prepare(ctx, fs, A->n))) return s;
        float *feat = fs->fbuf, *coef = fs->fbuf + NF;
        if ((s = features_into(ctx, A, b, feat, fs->dbuf))) return s;
        hipLaunchKernelGGL(k_standardize, dim3(1), dim3(64), 0, ctx->stream, feat, 1, (float *)dev_mean,
                           (float *)dev_std, 0);
        APCG_CHECK_LAUNCH("k_standardize");
        hipLaunchKernelGGL(k_mlp_fwd, dim3(1), dim3(64), 0, ctx->stream, dev_params, (const float *)feat, 1, coef);
        APCG_CHECK_LAUNCH("k_mlp_fwd");
        apcg_solve_opts o;
        if (opts) o = *opts;
        else apcg_solve_opts_default(&o);
        if (o.x0_is_zero) {
            // Warm start: the feature run's Jacobi-PCG steps from x0 = 0 left
            // their iterate in the scratch x; the flexible solve continues
            // from it instead of discarding it.
            if (!x || x->n != A->n || x->device != A->device)
                return set_error(APCG_ERR_INVALID_ARG, "x does not match the system");
            Acc acc[1] = {{&x->rec, ACC_W}};
            if ((s = op_begin(ctx, acc, 1))) return s;
            APCG_HIP(hipMemcpyAsync(x->d, fs->x, sizeof(double) * (size_t)A->n, hipMemcpyDeviceToDevice,
                                    ctx->stream));
            if ((s = op_end(ctx, acc, 1))) return s;
            o.x0_is_zero = 0;
        }
        return apcg_ksp_solve_fcg_poly(ctx, A, b, x, rtol, maxit, coef, fs->dbuf, &o, fopts, info, info_index);
    } catch (const std::bad_alloc &) {
        return set_error(APCG_ERR_OUT_OF_MEMORY, "host allocation failed");
    }
}

apcg_status apcg_mlp_standardize(apcg_ctx ctx, float *dev_X, int32_t B, float *dev_mean, float *dev_std,
                                 int32_t compute_stats) {
    if (!ctx || !dev_X || !dev_mean || !dev_std || B < 1) return set_error(APCG_ERR_INVALID_ARG, "bad arguments");
    if (apcg_status gs = ctx_end_group(ctx)) return gs;
    hipLaunchKernelGGL(k_standardize, dim3(1), dim3(64), 0, ctx->stream, dev_X, B, dev_mean, dev_std,
                       compute_stats ? 1 : 0);
    APCG_CHECK_LAUNCH("k_standardize");
    if (ctx->type == APCG_STREAM_GLOBAL_BLOCKING) APCG_HIP(hipStreamSynchronize(ctx->stream));
    return APCG_SUCCESS;
}

apcg_status apcg_mlp_forward(apcg_ctx ctx, const float *dev_params, const float *dev_X, int32_t B, float *dev_C) {
    if (!ctx || !dev_params || !dev_X || !dev_C || B < 1) return set_error(APCG_ERR_INVALID_ARG, "bad arguments");
    if (apcg_status gs = ctx_end_group(ctx)) return gs;
    hipLaunchKernelGGL(k_mlp_fwd, dim3(B), dim3(64), 0, ctx->stream, dev_params, dev_X, B, dev_C);
    APCG_CHECK_LAUNCH("k_mlp_fwd");
    if (ctx->type == APCG_STREAM_GLOBAL_BLOCKING) APCG_HIP(hipStreamSynchronize(ctx->stream));
    return APCG_SUCCESS;
}

// Loss, gradients (dev_grad, may be NULL) and, with adam.P, the Adam step.
static apcg_status mlp_step(apcg_ctx ctx, const float *dev_params, const float *dev_X, const float *dev_G,
                            const float *dev_h, int32_t B, float mu, float eps, float *dev_loss, float *dev_grad,
                            const Adam &adam) {
    if (apcg_status gs = ctx_end_group(ctx)) return gs;
    MlpScratch *ms = mlp_scratch(ctx);
    apcg_status s;
    if ((s = ensure_mlp(ctx, ms, B))) return s;
    hipStream_t st = ctx->stream;
    hipLaunchKernelGGL(k_mlp_sample, dim3((B + SPW - 1) / SPW), dim3(64 * SPW), 0, st, dev_params, dev_X, dev_G, dev_h,
                       (const float *)ms->phi(), B, mu, eps, ms->H1(), ms->H2(), ms->dC(), ms->dA1(), ms->dA2(),
                       ms->loss_b());
    APCG_CHECK_LAUNCH("k_mlp_sample");
    hipLaunchKernelGGL(k_mlp_grad, dim3(GRAD_TILES + 1), dim3(256), 0, st, dev_X, (const float *)ms->H1(),
                       (const float *)ms->H2(), (const float *)ms->dC(), (const float *)ms->dA1(),
                       (const float *)ms->dA2(), B, (const float *)ms->loss_b(), dev_loss, dev_grad, adam);
    APCG_CHECK_LAUNCH("k_mlp_grad");
    if (ctx->type == APCG_STREAM_GLOBAL_BLOCKING) APCG_HIP(hipStreamSynchronize(ctx->stream));
    return APCG_SUCCESS;
}

apcg_status apcg_mlp_loss_grad(apcg_ctx ctx, const float *dev_params, const float *dev_X, const float *dev_G,
                               const float *dev_h, int32_t B, float mu, float eps, float *dev_loss,
                               float *dev_grad) {
    if (!ctx || !dev_params || !dev_X || !dev_G || !dev_h || !dev_loss || !dev_grad || B < 1)
        return set_error(APCG_ERR_INVALID_ARG, "bad arguments");
    return mlp_step(ctx, dev_params, dev_X, dev_G, dev_h, B, mu, eps, dev_loss, dev_grad, Adam{});
}

apcg_status apcg_mlp_train_step(apcg_ctx ctx, float *dev_params, float *dev_adam_m, float *dev_adam_v, int32_t t,
                                float lr, const float *dev_X, const float *dev_G, const float *dev_h, int32_t B,
                                float mu, float eps, float *dev_loss) {
    if (!dev_adam_m || !dev_adam_v || t < 1) return set_error(APCG_ERR_INVALID_ARG, "bad Adam state");
    if (!ctx || !dev_params || !dev_X || !dev_G || !dev_h || !dev_loss || B < 1)
        return set_error(APCG_ERR_INVALID_ARG, "bad arguments");
    return mlp_step(ctx, dev_params, dev_X, dev_G, dev_h, B, mu, eps, dev_loss, nullptr,
                    Adam{dev_params, dev_adam_m, dev_adam_v, t, lr, 0.9f, 0.999f, 1e-8f});
}

}  // extern "C"
