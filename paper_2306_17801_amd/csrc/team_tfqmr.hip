// team_tfqmr.hip -- TFQMR (tfqmr.hip) of a system that fits the chip, held by
// a team of workgroups (team.h) in one launch.
//
// What bounds the kernels it stands in for: four launches an iteration, each
// with a reduction, and twelve passes over vectors.  Here a member keeps its
// rows' entries and vectors in registers and an iteration is two meetings:
// r0.v for alpha, and then both half-steps at once -- neither w after the
// first half-step nor r0.w after the second depends on a norm, so ||w||^2 of
// both and r0.w travel together.  v and w of the border rows go with the two
// meetings: a reader keeps the border of y and takes the same steps as the
// owner.
// Twenty iterations on 354,000 rows of 7 entries: 768 us by kernels, 345 here
// (about 12 us an iteration, and 100 to load the matrix and finish).
//
// The values travel with tags that count on from launch to launch
// (team_fcg.hip) through two buffers in turn; a buffer is written again two
// meetings later, when all its readers have taken the values before.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "team.h"
#include "team_host.h"

namespace apcg {
namespace {

using namespace team;

constexpr int R = 4;  // slices per wavefront

struct TeamTqPlan {
    const int32_t *rowptr, *col;
    const double *val, *b;
    double *x;
    uint64_t *swap;      // two buffers of 2 n tagged words
    uint8_t *need;       // n marks: the row is another member's border column
    uint64_t *words;     // kStride per group: messages of the setup (8 words), r0.v (2, at 8), the half-steps (8, at 16)
    apcg_solve_info *info;
    uint32_t *head, *verdict;
    TeamWait wait;
    int32_t n, T, border;
    double rtol;
    int32_t maxit, x0_zero, pc;
    uint32_t tag;        // tag of the first exchange
};

template <int L>
__device__ __forceinline__ void team_tfqmr(const TeamTqPlan &P, Member &M, double *win, double *red, int *area) {
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int n = M.n;
    const double rtol = P.rtol;
    const int maxit = P.maxit, x0_zero = P.x0_zero, pc = P.pc, border_max = P.border;
    const uint32_t tag0 = P.tag;
    const gptr<const int32_t> rowptr = uniform(P.rowptr), col = uniform(P.col);
    const gptr<const double> val = uniform(P.val), b = uniform(P.b);
    const gptr<double> sx = uniform(P.x);
    const gptr<uint64_t> w_init = uniform(P.words), w_sigma = w_init + 8, w_half = w_init + 16;
    const gptr<uint64_t> swap = uniform(P.swap);
    const gptr<uint8_t> need = uniform(P.need);
    Rows<R, L> A;
    const int row0 = M.m * kOwn<R>, row1 = min(n, row0 + kOwn<R>);
    // LDS: the window of y, the border's columns
    const int wsize = window_size(R, border_max);
    double *own = win + kPad + wave * 64 + lane, *border = win + kPad + kOwn<R>;
    uint16_t *list = (uint16_t *)(win + wsize);
    double r0[R], bd[R], x[R];

    uint64_t lens;
    const bool fits = load_rows<R, L>(A, rowptr, col, val, n, row0, lens, [&](int q, int i, bool in, int len,
                                      const int32_t (&cj)[L], double diag, bool found) {
        double ax = 0.0;
        if (!x0_zero) {
#pragma unroll
            for (int t = 0; t < L; ++t)
                if (t < len) ax = fma(A.a[q][t], sx[cj[t]], ax);
        }
        r0[q] = bd[q] = x[q] = 0.0;
        double v[4] = {0.0, 0.0, 0.0, 0.0};  // ||r0||^2, unusable diagonals
        if (in) {
            const bool ok = pc == APCG_PC_NONE || (found && diag != 0.0 && isfinite(diag));
            bd[q] = pc == APCG_PC_NONE ? 1.0 : (ok ? 1.0 / diag : 0.0);
            r0[q] = bd[q] * (x0_zero ? b[i] : b[i] - ax);
            if (!x0_zero) x[q] = sx[i];
            v[0] = r0[q] * r0[q];
            v[1] = ok ? 0.0 : 1.0;
        }
        slices_put<R, 4, 1>(red, q, v);
    });
    if (!__syncthreads_and(fits)) return refuse(M, kUnfit);
    const int nb = make_border<R, L>(A, lens, row1 - row0, (uint32_t *)win, list, border_max, area);
    if (nb > border_max) return refuse(M, kUnfit);
    for (int i = tid; i < wsize; i += TT) win[i] = 0.0;
    auto column = [&](int c) { return (uint32_t)(row0 + (int)list[c] - kBias); };
    for (int c = tid; c < nb; c += TT) store_shared<uint8_t>(need, column(c), 1);
    const auto none = [](int, int) { return true; };
    double t4[4];
    if (!team_meet<R, 4>(M, red, w_init, 1u, true, t4, none)) return;

    unsigned share = 0;  // bit q: this row of slice q is named by another member
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int i = row0 + (q * TW + wave) * 64 + lane;
        if (i < n && load_shared<uint8_t>(need, (uint32_t)i)) share |= 1u << q;
    }
    uint32_t ex = 0;  // exchanges so far
    auto buffer = [&](uint32_t e) { return swap + (e & 1u) * 2u * (uint32_t)n; };
    auto send = [&](int q, double v) __attribute__((always_inline)) {
        if (share & (1u << q))
            post(buffer(ex), (uint32_t)(row0 + (q * TW + wave) * 64 + lane) * 2, v, tag0 + ex);
    };
    // Four values of exchange e, border places c, c + nt, ... (past the
    // border's end: place c again).
    auto take4 = [&](uint32_t e, int c, int nt, double (&out)[kSide]) __attribute__((always_inline)) {
        static_assert(kSide == 4, "load_pairs");
        uint32_t place[kSide];
#pragma unroll
        for (int u = 0; u < kSide; ++u) place[u] = column(c + u * nt < nb ? c + u * nt : c) * 2;
        const gptr<uint64_t> buf = buffer(e);
        const uint32_t tag = tag0 + e;
        long long since = 0;
        for (int spin = 0;; ++spin) {
            uint64_t w[kSide][2];
            load_pairs(buf, place, w);
            bool all = true;
#pragma unroll
            for (int u = 0; u < kSide; ++u) {
                all = all && (uint32_t)(w[u][0] >> 32) == tag && (uint32_t)(w[u][1] >> 32) == tag;
                out[u] = unpack(w[u][0], w[u][1]);
            }
            if (all) return true;
            if (!keep_waiting(M, spin, since)) return false;
        }
    };
    // A short border is fetched during the meeting by the wavefronts that
    // collect no messages, a longer one by all of them when it is used.
    const int first = tid - M.mw * 64, others = TT - M.mw * 64;
    const bool small = nb <= kSide * others;
    double fetched[kSide];
    auto fetch = [&](uint32_t e) {
        return [&, e](int t, int nt) {
            if (!small || t >= nb) return true;
            return take4(e, t, nt, fetched);
        };
    };
    // border = step(border, value) with the values of exchange e
    auto apply = [&](uint32_t e, auto step) __attribute__((always_inline)) {
        if (small) {
            if (wave >= M.mw) {
#pragma unroll
                for (int u = 0; u < kSide; ++u) {
                    const int c = first + u * others;
                    if (c < nb) border[c] = step(border[c], fetched[u]);
                }
            }
            return;
        }
        for (int c = tid; c < nb; c += kSide * TT) {
            double v[kSide];
            if (!take4(e, c, TT, v)) {
                M.out->ok[1] = 0;
                return;
            }
#pragma unroll
            for (int u = 0; u < kSide; ++u)
                if (c + u * TT < nb) border[c + u * TT] = step(border[c + u * TT], v[u]);
        }
    };

    const double ref = sqrt(t4[0]);
    double rho = t4[0], tau = ref, theta = 0.0, eta = 0.0, bound = ref;
    int status = 0, its = 0, half = 0;
    if (t4[1] > 0.0) status = APCG_SOLVE_SETUP_ERROR;
    else if (!isfinite(ref)) status = APCG_SOLVE_NAN;
    else if (ref == 0.0) {
        status = APCG_SOLVE_CONVERGED;
        bound = 0.0;
    } else if (maxit <= 0) status = APCG_SOLVE_MAXIT;

    double w[R], d[R], v[R], u[R];
    double beta = 0.0;
    for (int k = 0; !status; ++k) {
        // y1 = w + beta y2 (r0 at first), u1 = B A y1, v = u1 + beta (u2 + beta v)
        A.keep_packed();
        asm volatile("" : "+v"(share));
        if (k == 0) {
#pragma unroll
            for (int q = 0; q < R; ++q) {
                w[q] = own[q * TT] = r0[q];
                d[q] = v[q] = u[q] = 0.0;
                send(q, r0[q]);
            }
            if (small && wave >= M.mw && !fetch(ex)(first, others)) M.out->ok[1] = 0;
        } else {
#pragma unroll
            for (int q = 0; q < R; ++q) own[q * TT] = fma(beta, own[q * TT], w[q]);
        }
        apply(ex, [&](double y, double value) { return fma(beta, y, value); });  // (the border starts as zeros)
        ++ex;
        __syncthreads();
        if (!M.out->ok[1]) return;
        {
            double s[R];
#pragma unroll
            for (int q = 0; q < R; ++q) {
                const double u1 = bd[q] * A.dot(q, win);
                v[q] = k == 0 ? u1 : fma(beta, fma(beta, v[q], u[q]), u1);
                u[q] = u1;
                send(q, v[q]);
                s[q] = r0[q] * v[q];
            }
            slices_put<R, 1, R>(red + 4 * R * TW, 0, s);
        }
        double t1[1];
        if (!team_meet<R, 1>(M, red + 4 * R * TW, w_sigma, (uint32_t)k + 1u, false, t1, fetch(ex))) return;
        const double sigma = t1[0];
        if (!isfinite(sigma)) status = APCG_SOLVE_NAN;
        else if (sigma == 0.0) status = APCG_SOLVE_BREAKDOWN_PAP;
        if (status) break;
        // both half-steps: y2 = y1 - alpha v, u2 = B A y2, w -= alpha u1, w -= alpha u2
        A.keep_packed();
        const double alpha = rho / sigma;
        its = k + 1;
        {
            const double f = theta * theta * eta / alpha;
            apply(ex, [&](double y, double value) { return fma(-alpha, value, y); });
            ++ex;
            double s[4 * R];
#pragma unroll
            for (int q = 0; q < R; ++q) {
                const double y1 = own[q * TT];
                d[q] = fma(f, d[q], y1);
                own[q * TT] = fma(-alpha, v[q], y1);
                w[q] = fma(-alpha, u[q], w[q]);
                s[4 * q] = w[q] * w[q];
            }
            __syncthreads();
            if (!M.out->ok[1]) return;
#pragma unroll
            for (int q = 0; q < R; ++q) {
                u[q] = bd[q] * A.dot(q, win);
                w[q] = fma(-alpha, u[q], w[q]);
                send(q, w[q]);
                s[4 * q + 1] = w[q] * w[q];
                s[4 * q + 2] = r0[q] * w[q];
                s[4 * q + 3] = 0.0;
            }
            slices_put<R, 4, R>(red, 0, s);
        }
        if (!team_meet<R, 4>(M, red, w_half, (uint32_t)k + 1u, false, t4, fetch(ex))) return;
        // theta, c, tau, eta of half-step m and its test
        auto half_step = [&](double ww, int m) __attribute__((always_inline)) {
            theta = sqrt(ww) / tau;
            const double cc = 1.0 / sqrt(1.0 + theta * theta);
            tau = tau * theta * cc;
            eta = cc * cc * alpha;
            bound = tau * sqrt((double)m + 1.0);
            half = m;
            if (!isfinite(bound)) status = APCG_SOLVE_NAN;
            else if (bound <= rtol * ref) status = APCG_SOLVE_CONVERGED;
        };
        half_step(t4[0], 2 * its - 1);
#pragma unroll
        for (int q = 0; q < R; ++q) x[q] = fma(eta, d[q], x[q]);
        if (status) break;
        const double f = theta * theta * eta / alpha;
        half_step(t4[1], 2 * its);
        if (!status && its >= maxit) status = APCG_SOLVE_MAXIT;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            d[q] = fma(f, d[q], own[q * TT]);
            x[q] = fma(eta, d[q], x[q]);
        }
        if (status) break;
        const double rho_new = t4[2];
        if (!isfinite(rho_new)) status = APCG_SOLVE_NAN;
        else if (rho_new == 0.0) status = APCG_SOLVE_BREAKDOWN_RZ;
        beta = rho_new / rho;
        rho = rho_new;
    }
    if (!finish(M)) return;
    // x leaves the registers once (every member read its x0 entries before
    // the setup meeting)
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int i = row0 + (q * TW + wave) * 64 + lane;
        if (i < n) sx[i] = x[q];
    }
    if (M.m == 0 && tid == 0) {
        P.info->iterations = its;
        P.info->status = status;
        P.info->fcg_iterations = 0;
        P.info->half_steps = half;
        P.info->res_norm = bound;
        P.info->ref_norm = ref;
    }
}

template <int L>
__global__ __launch_bounds__(TT, 2) void k_team_tfqmr(TeamTqPlan P) {
    extern __shared__ double lds[];
    // sums of the setup or the half-steps (4), and of r0.v (1)
    __shared__ double red[5 * R * TW], tot[16];
    __shared__ int area[2 * TW], member;
    __shared__ Exit out;
    if (threadIdx.x == 0) member = next_ticket(P.head, P.T, false);  // in the order the workgroups start
    __syncthreads();
    const int m = __builtin_amdgcn_readfirstlane(member);
    if (m >= P.T) return;
    const int ngr = (P.n + kGroupRows - 1) / kGroupRows;
    set_exit(out, P.head, P.verdict, P.wait.ticks, P.T);
    Member M{P.T, m, P.n, ngr, min((ngr + 63) / 64, kTree / 64), P.wait.look, tot, &out};
    team_tfqmr<L>(P, M, lds, red, area);
}

}  // namespace

apcg_status team_tfqmr_solve(apcg_ctx c, apcg_mat A, apcg_vec b, apcg_vec x, double rtol, int32_t maxit,
                             const apcg_solve_opts &opts, const TeamFit &fit, apcg_solve_info *info,
                             std::vector<int32_t> *left) {
    left->clear();
    TeamCache *t = team_cache(c);
    hipStream_t st = c->stream;
    const int32_t n = A->n, T = (n + TT * R - 1) / (TT * R);  // (n > kTeamMinRows: several members)
    const int64_t swap = ((int64_t)n * 4 + 7) / 8 * 8, marks = ((int64_t)n + 63) / 64 * 64;
    const int64_t words = ((int64_t)n + kGroupRows - 1) / kGroupRows * kStride;
    apcg_status s;
    uint32_t tag;
    if ((s = team_swap(t, st, swap, 2 * ((int64_t)maxit + 2), &tag))) return s;
    // cleared area: the head, the verdict, messages, marks
    const int64_t head = team_head_bytes(1);
    const int64_t sync_bytes = head + 8 * words + marks;
    t->desc_hash = 0;  // the buffer is laid out anew
    if ((s = team_memory(t, st, 0, sync_bytes, 0))) return s;
    uint32_t *head_p = reinterpret_cast<uint32_t *>(t->d_sync);
    TeamTqPlan P{};
    P.rowptr = A->rowptr;
    P.col = A->col;
    P.val = A->val;
    P.b = b->d;
    P.x = x->d;
    P.swap = t->d_swap;
    P.words = reinterpret_cast<uint64_t *>(t->d_sync + head);
    P.need = reinterpret_cast<uint8_t *>(t->d_sync + head + 8 * words);
    P.info = info;
    P.head = head_p;
    P.verdict = head_p + kHeadWords;
    P.wait = t->wait;
    P.n = n;
    P.T = T;
    P.border = fit.border[0];
    P.rtol = rtol;
    P.maxit = maxit;
    P.x0_zero = opts.x0_is_zero ? 1 : 0;
    P.pc = opts.pc;
    P.tag = tag;
    void (*fn)(TeamTqPlan) = A->sell_maxw <= 5 ? k_team_tfqmr<5> : k_team_tfqmr<7>;
    const size_t lds = (size_t)team_lds(R, P.border, 1, false);
    APCG_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                 (int)kLdsBytes));
    if ((s = team_clear(st, reinterpret_cast<uint64_t *>(t->d_sync), (sync_bytes + 7) / 8))) return s;
    s = team_launch(t->device, st, T, t->cus, [&]() -> apcg_status {
        hipLaunchKernelGGL(fn, dim3(T), dim3(TT), lds, st, P);
        APCG_CHECK_LAUNCH("k_team_tfqmr");
        return APCG_SUCCESS;
    });
    if (s) return s;
    return team_finish(c, t, 1, &A, left);
}

}  // namespace apcg
