// team_fcg.hip -- FCG(1) with each system's own degree-8 polynomial
// preconditioner (batched_fcg.hip) for systems that fit the chip, each held by
// a team of workgroups (team.h) in one launch.
//
// What bounds the kernels it stands in for: 13 launches an iteration, nine of
// them a product whose vectors and matrix go through the caches again.  Here
// an iteration is three meetings (delta, the residual, r.z with z.w) and
// eight exchanges of border values.  An exchange is no meeting: a member waits
// for the members whose rows it names and for nobody else.  Every value
// travels with the tag of its exchange, in one of two buffers in turn: a
// member overwrites the values of exchange e in e + 2, which it can only reach
// after everyone it reads has sent e + 1 and so has taken e -- if those are
// the members that read it, which the setup checks.  The tags go on counting
// from launch to launch, so the buffers are not cleared.
// An iteration with 64^3 rows: 75 us by kernels, 42 here; 48 mixed systems of
// 1e3 to 1e5 rows in one call: 52.2 ms on tiles, 9.7 here.  Four border
// values in flight per thread: with eight 42 registers spill (49.4 for 48.9 us
// at 64^3, 66.3 for 62.2 at 78^3), five and six make no difference.  All 256
// registers are taken as it is, with 104 bytes of scratch a lane (128, and 8
// registers spilled, with rows of seven entries).  What is left is the latency
// of eight dependent exchanges, 2 to 4 us each.
//
// The states, the operations and the order of every sum are those of
// batched_fcg.hip, so the two give the same bits.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "team.h"
#include "team_host.h"

namespace apcg {
namespace {

using namespace team;

constexpr int R = 4;      // slices per wavefront
constexpr int DEG = 8;
constexpr int MODE_FLEX = 0, MODE_JACOBI = 1;

struct TeamFcgSys {
    const int32_t *rowptr, *col;
    const double *val, *b;
    double *x;
    uint64_t *swap;      // two buffers of 2 n tagged words: the exchanges
    uint8_t *need;       // n marks: the row is another member's border column
    uint8_t *reads;      // [T][T] marks: member column reads rows of member row
    uint64_t *words;     // kStride per group: messages of the setup (8 words), delta (2, at 8), residual (2, at 10),
                         // r.z and z.w (4, at 12 and 16 in turn)
    apcg_solve_info *info;
    uint32_t *verdict;
    const float *coef;   // 9
    const double *lmax;  // 1
    int32_t n, T;
};

struct TeamFcgPlan {
    const TeamFcgSys *sys;
    const int2 *ticket;
    uint32_t *head;  // kHeadWords words
    TeamWait wait;
    int32_t tickets, border;
    double rtol, stall_frac;
    int32_t maxit, x0_zero, stall_min, fallback;
    uint32_t tag;  // tag of the first exchange
};

template <int L>
__device__ __forceinline__ void team_fcg(const TeamFcgPlan &P, const TeamFcgSys &S, Member &M, double *win, double *red,
                                         int *area, double *cc) {
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int n = M.n;
    // the plan's values in registers of their own (captured as a whole by the
    // lambdas below, the plan would lie in scratch memory)
    const double rtol = P.rtol, stall_frac = P.stall_frac;
    const int maxit = P.maxit, x0_zero = P.x0_zero, stall_min = P.stall_min, fallback = P.fallback;
    const int border = P.border;
    const uint32_t tag0 = P.tag;
    const gptr<const int32_t> rowptr = uniform(S.rowptr), col = uniform(S.col);
    const gptr<const double> val = uniform(S.val), b = uniform(S.b);
    const gptr<double> sx = uniform(S.x);
    const gptr<uint64_t> w_init = uniform(S.words), w_delta = w_init + 8, w_res = w_init + 10;
    const gptr<uint64_t> swap = uniform(S.swap);
    const gptr<uint8_t> need = uniform(S.need), reads = uniform(S.reads);
    Rows<R, L> A;
    const int row0 = M.m * kOwn<R>, row1 = min(n, row0 + kOwn<R>);
    // LDS: the window of p, the window of what the polynomial multiplies, the
    // border's columns
    const int wsize = window_size(R, border);
    double *pw = win, *uw = win + wsize;
    double *p_own = pw + kPad + wave * 64 + lane, *u_own = uw + kPad + wave * 64 + lane;
    double *p_border = pw + kPad + kOwn<R>, *u_border = uw + kPad + kOwn<R>;
    uint16_t *list = (uint16_t *)(win + 2 * wsize);
    double r[R], d[R], x[R], w[R];

    uint64_t lens;
    const bool fits = load_rows<R, L>(A, rowptr, col, val, n, row0, lens, [&](int q, int i, bool in, int len,
                                      const int32_t (&cj)[L], double diag, bool found) {
        double ax = 0.0;
        if (!x0_zero) {
#pragma unroll
            for (int t = 0; t < L; ++t)
                if (t < len) ax = fma(A.a[q][t], sx[cj[t]], ax);
        }
        r[q] = d[q] = x[q] = w[q] = 0.0;
        double v[4] = {0.0, 0.0, 0.0, 0.0};  // ||b||^2, ||r||^2, bad diagonals
        if (in) {
            const bool ok = found && diag > 0.0;
            const double bi = b[i], ri = x0_zero ? bi : bi - ax;
            if (!x0_zero) x[q] = sx[i];
            r[q] = ri;
            d[q] = ok ? 1.0 / diag : 0.0;
            v[0] = bi * bi;
            v[1] = ri * ri;
            v[2] = ok ? 0.0 : 1.0;
        }
        slices_put<R, 4, 1>(red, q, v);
    });
    if (!__syncthreads_and(fits)) return refuse(M, kUnfit);
    const int nb = make_border<R, L>(A, lens, row1 - row0, (uint32_t *)win, list, border, area);
    if (nb > border) return refuse(M, kUnfit);
    for (int i = tid; i < 2 * wsize; i += TT) win[i] = 0.0;
    auto column = [&](int c) { return (uint32_t)(row0 + (int)list[c] - kBias); };
    for (int c = tid; c < nb; c += TT) {
        const uint32_t j = column(c);
        store_shared<uint8_t>(need, j, 1);
        store_shared<uint8_t>(reads, j / kOwn<R> * M.T + M.m, 1);
    }
    if (tid <= DEG) cc[tid] = (double)S.coef[tid];
    __syncthreads();
    const double lm = *S.lmax;
    bool positive = true;
    for (int q = tid; q < 1024; q += TT) positive = positive && dev::poly_at<DEG>(cc, lm * q / 1023.0, lm) > 0.0;
    positive = __syncthreads_and(positive);
    const auto none = [](int, int) { return true; };
    double t4[4];
    if (!team_meet<R, 4>(M, red, w_init, 1u, true, t4, none)) return;

    unsigned share = 0;  // bit q: this row of slice q is named by another member
    bool mutual = true;
    if (M.T > 1) {
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int i = row0 + (q * TW + wave) * 64 + lane;
            if (i < n && load_shared<uint8_t>(need, (uint32_t)i)) share |= 1u << q;
        }
        for (int o = tid; o < M.T; o += TT)
            mutual = mutual && (load_shared<uint8_t>(reads, (uint32_t)(o * M.T + M.m)) != 0) ==
                                   (load_shared<uint8_t>(reads, (uint32_t)(M.m * M.T + o)) != 0);
    }
    mutual = __syncthreads_and(mutual);

    uint32_t ex = 0;  // exchanges so far
    auto buffer = [&](uint32_t e) { return swap + (e & 1u) * 2u * (uint32_t)n; };
    // sends this thread's row of slice q in exchange ex
    auto send = [&](int q, double v) __attribute__((always_inline)) {
        if (share & (1u << q))
            post(buffer(ex), (uint32_t)(row0 + (q * TW + wave) * 64 + lane) * 2, v, tag0 + ex);
    };
    // takes the border of exchange e into the border of window u
    auto take = [&](uint32_t e) __attribute__((always_inline)) {
        return [&, e](int t, int nt) __attribute__((always_inline)) {
            const gptr<uint64_t> buf = buffer(e);
            const uint32_t tag = tag0 + e;
            for (int c0 = t; c0 < nb; c0 += kSide * nt) {
                uint32_t place[kSide];  // past the border's end: the round's first column again
#pragma unroll
                for (int u = 0; u < kSide; ++u) place[u] = column(c0 + u * nt < nb ? c0 + u * nt : c0) * 2;
                long long t0 = 0;
                for (int spin = 0;; ++spin) {
                    uint64_t v[kSide][2];
                    load_pairs(buf, place, v);
                    bool all = true;
#pragma unroll
                    for (int u = 0; u < kSide; ++u)
                        all = all && (uint32_t)(v[u][0] >> 32) == tag && (uint32_t)(v[u][1] >> 32) == tag;
                    if (all) {
#pragma unroll
                        for (int u = 0; u < kSide; ++u)
                            if (c0 + u * nt < nb) u_border[c0 + u * nt] = unpack(v[u][0], v[u][1]);
                        break;
                    }
                    if (!keep_waiting(M, spin, t0)) return false;
                }
            }
            return true;
        };
    };
    // the exchange of the values just sent and stored in window u, on its own
    auto exchange = [&]() __attribute__((always_inline)) {
        const bool good = take(ex)(tid, TT);
        ++ex;
        if (!good) M.out->ok[1] = 0;
        __syncthreads();
        return M.out->ok[1] != 0;
    };

    const double ref = sqrt(t4[0]);
    double res = sqrt(t4[1]), best_res = res, rho = 0.0, delta = 0.0, beta = 0.0;
    int its = 0, fcg_its = 0, best_its = 0, mode = MODE_FLEX, reason = 0, status = 0;
    bool restart = true, stopped = false, zero_x = false;  // restart: the first application of the preconditioner
    if (t4[2] > 0.0) status = APCG_SOLVE_SETUP_ERROR;
    else if (ref == 0.0) {
        status = APCG_SOLVE_CONVERGED;
        zero_x = true;
        res = 0.0;
    } else if (!isfinite(res) || !isfinite(ref)) status = APCG_SOLVE_NAN;
    else if (res <= rtol * ref) status = APCG_SOLVE_CONVERGED;
    else if (maxit <= 0) status = APCG_SOLVE_MAXIT;
    stopped = status != 0;
    if (!stopped && (!positive || !(lm > 0.0) || !isfinite(lm))) {  // the preconditioner would not be SPD
        if (fallback) {
            mode = MODE_JACOBI;
            reason = APCG_SOLVE_BREAKDOWN_RZ;
        } else {
            status = APCG_SOLVE_BREAKDOWN_RZ;
            stopped = true;
        }
    }
    if (!stopped && !mutual) return refuse(M, kOneSided);  // (an end without exchanges needs no readers)
    auto stop = [&](int why) __attribute__((always_inline)) {
        status = mode == MODE_JACOBI ? why | APCG_SOLVE_FALLBACK | reason : why;
        stopped = true;
    };
    // over to Jacobi-PCG from the current x, or the end when that is not possible
    auto hand_over = [&](int why) __attribute__((always_inline)) {
        if (mode == MODE_FLEX && fallback) {
            mode = MODE_JACOBI;
            reason = why;
            restart = true;
        } else {
            stop(why);
        }
    };

    double z[R];
#pragma unroll
    for (int q = 0; q < R; ++q) z[q] = 0.0;
    for (uint32_t step = 1; !stopped; ++step) {
        A.keep_packed();
        asm volatile("" : "+v"(share));
        bool sent = false;  // v = D^-1 r has been exchanged
        if (restart) {
            // a meeting of one member ends without a barrier: r.z of the last
            // step has been read before this step's sums take its place
            __syncthreads();
        } else {
            for (int c = tid; c < nb; c += TT) p_border[c] = fma(beta, p_border[c], u_border[c]);
#pragma unroll
            for (int q = 0; q < R; ++q) p_own[q * TT] = fma(beta, p_own[q * TT], z[q]);
            __syncthreads();
            {
                double v[R];
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    w[q] = A.dot(q, pw);
                    v[q] = p_own[q * TT] * w[q];
                }
                slices_put<R, 1, R>(red + 4 * R * TW, 0, v);
            }
            double t1[1];
            if (!team_meet<R, 1>(M, red + 4 * R * TW, w_delta, step, false, t1, none)) return;
            delta = t1[0];
            if (!(delta > 0.0)) {
                if (!isfinite(delta)) stop(APCG_SOLVE_NAN);
                else hand_over(APCG_SOLVE_BREAKDOWN_PAP);
            } else {
                const double alpha = rho / delta;
                double v[R];
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    r[q] = fma(-alpha, w[q], r[q]);
                    v[q] = r[q] * r[q];
                    if (mode == MODE_FLEX) {
                        const double vi = d[q] * r[q];
                        u_own[q * TT] = vi;
                        send(q, vi);
                    }
                }
#pragma unroll
                for (int q = 0; q < R; ++q) x[q] = fma(alpha, p_own[q * TT], x[q]);
                slices_put<R, 1, R>(red, 0, v);
                if (mode == MODE_FLEX) {
                    if (!team_meet<R, 1>(M, red, w_res, step, false, t1, take(ex))) return;
                    ++ex;
                    sent = true;
                } else if (!team_meet<R, 1>(M, red, w_res, step, false, t1, none)) {
                    return;
                }
                res = sqrt(t1[0]);
                ++its;
                if (mode == MODE_FLEX) fcg_its = its;
                if (!isfinite(res)) stop(APCG_SOLVE_NAN);
                else if (res <= rtol * ref) stop(APCG_SOLVE_CONVERGED);
                else {
                    if (mode == MODE_FLEX) {
                        if (res < best_res) {
                            best_res = res;
                            best_its = its;
                        } else {
                            double window = stall_frac * (double)its;
                            if (window < (double)stall_min) window = (double)stall_min;
                            if ((double)(its - best_its) >= window) hand_over(APCG_SOLVE_STALL);
                        }
                    }
                    if (!stopped && its >= maxit) stop(APCG_SOLVE_MAXIT);
                }
            }
        }
        if (stopped) break;
        // z = p(D^-1 A) D^-1 r by Clenshaw's recurrence, or D^-1 r
        if (mode == MODE_JACOBI) {
#pragma unroll
            for (int q = 0; q < R; ++q) z[q] = d[q] * r[q];
        } else {
#pragma clang fp contract(off)
            if (!sent) {
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    const double vi = d[q] * r[q];
                    u_own[q * TT] = vi;
                    send(q, vi);
                }
                if (!exchange()) return;
            }
            const double s2 = 2.0 / lm, cd = cc[DEG];
            double b1[R], b2[R];
            {
                const double cj = cc[DEG - 1];
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    const double au = A.dot(q, uw), vi = d[q] * r[q];
                    b1[q] = fma(2.0 * cd, s2 * d[q] * au - vi, cj * vi);
                    b2[q] = cd * vi;
                }
            }
            for (int j = DEG - 2; j >= 0; --j) {
                A.keep_packed();
                __syncthreads();  // every gather from window u is done
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    u_own[q * TT] = b1[q];
                    send(q, b1[q]);
                }
                if (!exchange()) return;
                const double cj = cc[j];
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    const double au = A.dot(q, uw), vi = d[q] * r[q];
                    const double yu = s2 * d[q] * au - b1[q];
                    const double b0 = j > 0 ? fma(2.0, yu, cj * vi) - b2[q] : cj * vi + yu - b2[q];
                    b2[q] = b1[q];
                    b1[q] = b0;
                }
            }
#pragma unroll
            for (int q = 0; q < R; ++q) z[q] = b1[q];
        }
        {
            double v[2 * R];
#pragma unroll
            for (int q = 0; q < R; ++q) {
                send(q, z[q]);
                v[2 * q] = r[q] * z[q];
                v[2 * q + 1] = z[q] * w[q];
            }
            slices_put<R, 2, R>(red + 2 * R * TW, 0, v);  // (beside the residual's, which may still be read)
        }
        // two message areas in turn: after a hand-over this meeting follows the
        // last of its kind with no other between them
        double t2[2];
        if (!team_meet<R, 2>(M, red + 2 * R * TW, w_init + 12 + 4 * (step & 1u), step, false, t2, take(ex))) return;
        ++ex;
        const double rz = t2[0], zw = t2[1];
        if (restart) {  // a fresh recurrence from the current x
            if (!isfinite(rz)) stop(APCG_SOLVE_NAN);
            else if (!(rz > 0.0)) hand_over(APCG_SOLVE_BREAKDOWN_RZ);  // stays in restart when handing over
            else {
                rho = rz;
                beta = 0.0;
                restart = false;
            }
        } else if (!isfinite(rz) || !isfinite(zw)) {
            stop(APCG_SOLVE_NAN);
        } else if (!(rz > 0.0)) {
            hand_over(APCG_SOLVE_BREAKDOWN_RZ);
        } else {
            beta = mode == MODE_FLEX ? -zw / delta : rz / rho;
            rho = rz;
        }
    }
    if (!finish(M)) return;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int i = row0 + (q * TW + wave) * 64 + lane;
        if (i < n) sx[i] = zero_x ? 0.0 : x[q];
    }
    if (M.m == 0 && tid == 0) {
        S.info->iterations = its;
        S.info->status = status;
        S.info->fcg_iterations = fcg_its;
        S.info->half_steps = 0;
        S.info->res_norm = res;
        S.info->ref_norm = ref;
    }
}

template <int L>
__global__ __launch_bounds__(TT, 2) void k_team_fcg(TeamFcgPlan P) {
    extern __shared__ double lds[];
    // sums of the setup (4) or the residual (1) and r.z with z.w (2, from the third on), and of delta (1)
    __shared__ double red[5 * R * TW], tot[16], cc[DEG + 1];
    __shared__ int area[2 * TW], next;
    __shared__ Exit out;
    for (bool through = false;; through = true) {
        __syncthreads();  // the previous ticket is finished in every thread
        if (threadIdx.x == 0) next = next_ticket(P.head, P.tickets, through);
        __syncthreads();
        const int t = next;
        if (t >= P.tickets) return;
        const int2 tk = P.ticket[t];
        const int sys = __builtin_amdgcn_readfirstlane(tk.x), m = __builtin_amdgcn_readfirstlane(tk.y);
        const TeamFcgSys S = P.sys[sys];
        const int n = __builtin_amdgcn_readfirstlane(S.n);
        const int ngr = (n + kGroupRows - 1) / kGroupRows;
        const int T = __builtin_amdgcn_readfirstlane(S.T);
        set_exit(out, P.head, S.verdict, P.wait.ticks, t - m + T);
        Member M{T, m, n, ngr, min((ngr + 63) / 64, kTree / 64), P.wait.look, tot, &out};
        team_fcg<L>(P, S, M, lds, red, area, cc);
    }
}

}  // namespace

apcg_status team_fcg_solve(apcg_ctx c, int32_t nsys, const apcg_mat *A, const apcg_vec *b, const apcg_vec *x,
                           const std::vector<int32_t> &order, double rtol, int32_t maxit, const apcg_solve_opts &opts,
                           const apcg_fcg_opts &fo, const TeamFit &fit, const float *coeffs, const double *lmax,
                           apcg_solve_info *info, std::vector<int32_t> *left) {
    left->clear();
    TeamCache *t = team_cache(c);
    hipStream_t st = c->stream;
    int maxrow = 1, border = 0;
    int64_t swap = 0, marks = 0, words = 0, tickets = 0;
    std::vector<TeamFcgSys> sys(nsys);
    for (int32_t i = 0; i < nsys; ++i) {
        TeamFcgSys &s = sys[i];
        s.rowptr = A[i]->rowptr;
        s.col = A[i]->col;
        s.val = A[i]->val;
        s.b = b[i]->d;
        s.x = x[i]->d;
        s.n = A[i]->n;
        s.T = (int32_t)std::max<int64_t>(1, ((int64_t)s.n + TT * R - 1) / (TT * R));
        s.info = info + i;
        s.coef = coeffs + (int64_t)i * (DEG + 1);
        s.lmax = lmax + i;
        maxrow = std::max(maxrow, A[i]->sell_maxw);
        if (s.T > 1) border = std::max(border, fit.border[i]);
        s.swap = reinterpret_cast<uint64_t *>(swap);
        s.need = reinterpret_cast<uint8_t *>(marks);
        s.reads = reinterpret_cast<uint8_t *>(marks + ((int64_t)s.n + 63) / 64 * 64);
        s.words = reinterpret_cast<uint64_t *>(words);
        if (s.T > 1) {
            swap += ((int64_t)s.n * 4 + 7) / 8 * 8;
            marks += ((int64_t)s.n + 63) / 64 * 64 + ((int64_t)s.T * s.T + 63) / 64 * 64;
            words += ((int64_t)s.n + kGroupRows - 1) / kGroupRows * kStride;
        }
        tickets += s.T;
    }
    apcg_status s;
    // tags of this launch: at most nine exchanges for every iteration and
    // every restart, one restart a system and one more for its start
    const int64_t tags = 9 * ((int64_t)maxit + 4);
    uint32_t tag;
    if ((s = team_swap(t, st, swap, tags, &tag))) return s;
    const int64_t head = team_head_bytes(nsys);
    const int64_t sync_bytes = head + 8 * words + marks;
    if ((s = team_memory(t, st, team_desc_bytes((int64_t)sizeof(TeamFcgSys) * nsys, tickets), sync_bytes, 0))) return s;
    uint32_t *head_p = reinterpret_cast<uint32_t *>(t->d_sync);
    for (int32_t i = 0; i < nsys; ++i) {
        TeamFcgSys &q = sys[i];
        q.swap = t->d_swap + reinterpret_cast<int64_t>(q.swap);
        q.words = reinterpret_cast<uint64_t *>(t->d_sync + head) + reinterpret_cast<int64_t>(q.words);
        q.need = reinterpret_cast<uint8_t *>(t->d_sync + head + 8 * words) + reinterpret_cast<int64_t>(q.need);
        q.reads = reinterpret_cast<uint8_t *>(t->d_sync + head + 8 * words) + reinterpret_cast<int64_t>(q.reads);
        q.verdict = head_p + kHeadWords + i;
    }
    std::vector<int32_t> members(nsys);
    for (int32_t i = 0; i < nsys; ++i) members[i] = sys[i].T;
    const char *d_sys;
    const int2 *d_tickets;
    if ((s = team_upload(t, st, sys.data(), (int64_t)sizeof(TeamFcgSys) * nsys, order, members, &d_sys, &d_tickets)))
        return s;
    TeamFcgPlan P{};
    P.sys = reinterpret_cast<const TeamFcgSys *>(d_sys);
    P.ticket = d_tickets;
    P.head = head_p;
    P.wait = t->wait;
    P.tickets = (int32_t)tickets;
    P.border = border;
    P.rtol = rtol;
    P.stall_frac = fo.stall_frac;
    P.maxit = maxit;
    P.x0_zero = opts.x0_is_zero ? 1 : 0;
    P.stall_min = fo.stall_min;
    P.fallback = fo.fallback ? 1 : 0;
    P.tag = tag;
    void (*fn)(TeamFcgPlan) = maxrow <= 5 ? k_team_fcg<5> : k_team_fcg<7>;
    const size_t lds = (size_t)team_lds(R, border, 2, false);
    APCG_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                 (int)kLdsBytes));
    const int grid = (int)std::min<int64_t>(tickets, t->cus);
    if ((s = team_clear(st, reinterpret_cast<uint64_t *>(t->d_sync), (sync_bytes + 7) / 8))) return s;
    s = team_launch(t->device, st, grid, t->cus, [&]() -> apcg_status {
        hipLaunchKernelGGL(fn, dim3(grid), dim3(TT), lds, st, P);
        APCG_CHECK_LAUNCH("k_team_fcg");
        return APCG_SUCCESS;
    });
    if (s) return s;
    return team_finish(c, t, nsys, A, left);
}

}  // namespace apcg
