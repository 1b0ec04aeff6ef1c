// team.hip -- Jacobi-PCG of one or many systems that fit the chip, each held
// by a team of workgroups (team.h): the whole solve is one launch.
//
// What bounds it: the multi-kernel iteration of a system of 8e3 to 6e5 rows
// is bound by its kernel boundaries and, in the segmented batch, by streaming
// every vector and the matrix through the caches again in every kernel.  Here
// nothing but D^-1 r of the rows at the members' borders leaves the compute
// units between two iterations, and an iteration is bound by its two meetings
// (1.2 to 1.8 us each).  Microseconds per iteration, before and after:
//   2D, 30k rows   10.0   4.6        3D, 64^3 (262k rows)   15.8   8.0
//   2D, 250k rows  15     6.4
// and 256 2D systems of 1e3 to 6.5e4 rows in one call: 192 ms, now 28.5.  The direction of the border columns is kept
// and updated by every member that reads it (p = z + beta p, the same
// operation on the same values), so only z travels.
//
// One iteration k of a member:
//   p = z + beta p for its rows and its window's border columns (LDS);
//   w = A p from registers and LDS, delta = p.w                    (meeting 1)
//   x += alpha p, r -= alpha w, z = D^-1 r, border rows of z stored for the
//   other members, z.r and the stopping norm                       (meeting 2)
//   the tests, beta.
// The operations and the order of every sum are those of the segmented
// schedule (batched.hip), so the two give the same bits.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <vector>

#include "team.h"
#include "team_host.h"

namespace apcg {
namespace {

using namespace team;

struct TeamSys {
    const int32_t *rowptr, *col;
    const double *val, *b;
    double *x;
    uint64_t *z;         // D^-1 r of the rows other members read: n doubles, or 2 n tagged words
    uint8_t *need;       // n marks: the row is another member's border column
    uint64_t *words;     // kStride per group: messages of the setup (8 words), delta (2, at 8), residual (4, at 12)
    apcg_solve_info *info;
    uint32_t *done;      // members that have finished
    int32_t n, T;
    int32_t tagged;      // z travels as tagged words (few border columns)
};

struct TeamPlan {
    const TeamSys *sys;
    const int2 *ticket;   // (system, member), a system's members in a row
    uint32_t *next;       // next ticket to hand out
    uint32_t *stop;
    int32_t tickets, window;  // window: capacity in columns
    double rtol;
    int32_t maxit, x0_zero, pc, norm_pre;
    double *hist;         // one system only: alpha, beta of the first hist_cap iterations
    int32_t hist_cap;
};

// Eight slices a wavefront leave no registers for x and D^-1 beside the
// entries, r and w: they lie in LDS behind the window then (kept in registers
// they spilled, and a member of 4096 rows took 7.6 us an iteration instead of
// 5.5).
constexpr bool rows_in_lds(int R) { return R == 8; }

template <int R, int L>
__device__ __forceinline__ void team_pcg(const TeamPlan &P, const TeamSys &S, Member &M, double *win, double *red, int *area) {
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int n = M.n;
    const gptr<const int32_t> rowptr = uniform(S.rowptr), col = uniform(S.col);
    const gptr<const double> val = uniform(S.val), b = uniform(S.b);
    const gptr<double> sx = uniform(S.x);
    const gptr<uint64_t> w_init = uniform(S.words), w_delta = w_init + 8, w_res = w_init + 12;
    const gptr<uint64_t> z_w = uniform(S.z);
    const gptr<double> z_sh = (gptr<double>)z_w;
    const bool tagged = R <= 4 && __builtin_amdgcn_readfirstlane(S.tagged) != 0;
    const gptr<uint8_t> need = uniform(S.need);
    Rows<R, L> A;
    const int row0 = M.m * (TT * R), row1 = min(n, row0 + TT * R);
    double r[R], dreg[R], xreg[R];
    // D^-1 and x of this thread's row of slice q
    double *dl = win + P.window + wave * 64 + lane, *xl = dl + TT * R;
    auto d = [&](int q) -> double & {
        if constexpr (rows_in_lds(R)) return dl[q * TT];
        else return dreg[q];
    };
    auto x = [&](int q) -> double & {
        if constexpr (rows_in_lds(R)) return xl[q * TT];
        else return xreg[q];
    };
    unsigned share = 0;  // bit q: this row of slice q is stored for the other members
    uint64_t lens = 0;   // row lengths, four bits each

    // ---- setup: entries, window, D^-1, r0, z0 and the four setup sums
    int lo = row0, hi = max(row1 - 1, row0);
    bool fits = true;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int i = row0 + (q * TW + wave) * 64 + lane;
        const bool in = i < n;
        const int s = in ? rowptr[i] : 0, len = in ? rowptr[i + 1] - s : 0;
        fits = fits && len <= L;
        int32_t cj[L];
#pragma unroll
        for (int t = 0; t < L; ++t) {
            const bool has = t < len;
            cj[t] = has ? col[s + t] : row0;
            A.a[q][t] = has ? val[s + t] : 0.0;
            lo = min(lo, cj[t]);
            hi = max(hi, cj[t]);
        }
#pragma unroll
        for (int t = 0; t < L; t += 2) {
            const uint32_t even = (uint32_t)(cj[t] - row0 + kBias) & 0xffffu;
            const uint32_t odd = t + 1 < L ? (uint32_t)(cj[t + 1] - row0 + kBias) & 0xffffu : 0u;
            A.j[q][t >> 1] = even | odd << 16;
        }
        lens |= (uint64_t)(uint32_t)min(len, 15) << (4 * q);
        double diag = 0.0, ax = 0.0;
        bool found = false;
#pragma unroll
        for (int t = 0; t < L; ++t)
            if (t < len) {
                if (cj[t] == i) {
                    diag = A.a[q][t];
                    found = true;
                }
                if (!P.x0_zero) ax = fma(A.a[q][t], sx[cj[t]], ax);
            }
        r[q] = d(q) = x(q) = 0.0;
        double v4[4] = {0.0, 0.0, 0.0, 0.0};
        if (in) {
            double di = 1.0;
            if (P.pc == APCG_PC_JACOBI) {
                const bool ok = found && diag > 0.0;
                v4[3] = ok ? 0.0 : 1.0;
                di = ok ? 1.0 / diag : 0.0;
            }
            const double bi = b[i];
            const double ri = P.x0_zero ? bi : bi - ax;
            if (!P.x0_zero) x(q) = sx[i];
            r[q] = ri;
            d(q) = di;
            const double zi = di * ri;
            v4[0] = zi * ri;
            if (P.norm_pre) {
                const double zb = di * bi;
                v4[1] = zi * zi;
                v4[2] = zb * zb;
            } else {
                v4[1] = ri * ri;
                v4[2] = bi * bi;
            }
            if (M.T > 1) {
                if (tagged) post(z_w, (uint32_t)i * 2, zi, 1u);
                else store_shared<double>(z_sh, (uint32_t)i, zi);
            }
        }
        slices_put<R, 4, 1>(red, q, v4);
        __builtin_amdgcn_sched_barrier(0);  // one slice at a time: the loads of all would not fit the registers
    }
    block_minmax(lo, hi, area);
    lo &= ~63;
    hi += 1;
    fits = fits && lo >= 0 && hi <= max(n, 1) && hi - lo <= P.window;
    // a row longer than the registers hold or a window wider than the LDS:
    // the pattern is not the one this schedule was chosen for
    if (!__syncthreads_and(fits)) {
        if (tid == 0) {
            store_shared<uint32_t>(M.stop, 0, 2u);
            *M.ok = 0;
        }
        __syncthreads();
        return;
    }
    for (int i = tid; i < max(hi - lo, row0 - lo + TT * R) + kZero; i += TT) win[i - kZero] = 0.0;
    const int below = row0 - lo, border = below + max(0, hi - row1);
    // the window place of border column h
    auto place = [&](int h) { return h < below ? h : row1 - lo + h - below; };
    // Which border columns some row names (a member of half a grid plane has
    // two whole planes in its window and names half of each): bit u of want
    // for column tid + u TT, of side for the thread's columns in fetch.  Their
    // owners are told to keep storing z of these rows.
    uint32_t want = 0, side = 0;
    if (M.T > 1) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < R; ++q)
#pragma unroll
            for (int t = 0; t < L; ++t)
                if (t < ((int)(lens >> (4 * q)) & 15)) win[A.rel(q, t) - kBias + below] = 1.0;
        __syncthreads();
        for (int u = 0; tid + u * TT < border; ++u) {
            const int pl = place(tid + u * TT);
            if (win[pl] != 0.0) {
                want |= 1u << u;
                store_shared<uint8_t>(need, (uint32_t)(lo + pl), 1);
            }
        }
        if (tagged && wave >= M.mw)
            for (int u = 0; u < kSide; ++u) {
                const int h = tid - M.mw * 64 + u * (TT - M.mw * 64);
                if (h < border && win[place(h)] != 0.0) side |= 1u << u;
            }
        __syncthreads();
        for (int i = tid; i < hi - lo; i += TT) win[i] = 0.0;
    }
    const double *base = win + (row0 - lo) - kBias;
    const uint32_t zero = (uint32_t)(kBias - (row0 - lo) - 1);
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int len = (int)(lens >> (4 * q)) & 15;
#pragma unroll
        for (int t = 0; t < L; ++t)
            if (t >= len) A.j[q][t >> 1] = (A.j[q][t >> 1] & ~(0xffffu << (16 * (t & 1)))) | zero << (16 * (t & 1));
    }
    // A short border's z is fetched during the meeting, by the wavefronts that
    // collect no messages, as its tags arrive: neither an acknowledged store
    // before the message nor a round trip after it.
    double zb[kSide];
    auto fetch = [&](uint32_t tag) {
        return [&, tag](int t, int nt) {
#pragma unroll
            for (int u = 0; u < kSide; ++u) zb[u] = 0.0;
            if (!tagged) return true;
            static_assert(kSide == 4, "load_pairs");
            uint32_t at4[kSide];  // an unnamed column's place is taken by the first named one's
#pragma unroll
            for (int u = 0; u < kSide; ++u)
                at4[u] = (uint32_t)(lo + place(t + (side & (1u << u) ? u : max(__ffs(side) - 1, 0)) * nt)) * 2;
            if (!side) return true;
            long long t0 = 0;
            for (int spin = 0;; ++spin) {
                uint64_t w[kSide][2];
                load_pairs(z_w, at4, w);
                bool all = true;
#pragma unroll
                for (int u = 0; u < kSide; ++u) {
                    all = all && (uint32_t)(w[u][0] >> 32) == tag && (uint32_t)(w[u][1] >> 32) == tag;
                    zb[u] = unpack(w[u][0], w[u][1]);
                }
                if (all) return true;
                if (!keep_waiting(M, spin, t0)) return false;
            }
        };
    };
    double t4[4];
    const auto none = [](int, int) { return true; };
    if (!team_meet<R, 4>(M, red, w_init, 1u, true, t4, none)) return;
    // every row's z carries tag 1 now, whatever an earlier solve left there
    if (wave >= M.mw && !fetch(1u)(tid - M.mw * 64, TT - M.mw * 64)) *M.ok = 0;
    double rho = t4[0], res = sqrt(t4[1]);
    const double ref = sqrt(t4[2]);
    int status = 0, its = 0;
    bool zero_x = false;
    if (t4[3] > 0.0) status = APCG_SOLVE_SETUP_ERROR;
    else if (ref == 0.0) {
        status = APCG_SOLVE_CONVERGED;
        zero_x = true;
        res = 0.0;
    } else if (!isfinite(res) || !isfinite(ref)) status = APCG_SOLVE_NAN;
    else if (res <= P.rtol * ref) status = APCG_SOLVE_CONVERGED;
    else if (!(rho > 0.0)) status = isfinite(rho) ? APCG_SOLVE_BREAKDOWN_RZ : APCG_SOLVE_NAN;
    else if (P.maxit <= 0) status = APCG_SOLVE_MAXIT;

    if (M.T > 1) {
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int i = row0 + (q * TW + wave) * 64 + lane;
            if (i < n && load_shared<uint8_t>(need, (uint32_t)i)) share |= 1u << q;
        }
    }
    // this thread's row of slice 0; the places of rows past the last one (of
    // the last member only, whose window ends with its rows) hold zeros
    double *own = win + (row0 - lo) + wave * 64 + lane;
    double beta = 0.0;
    for (int k = 1; !status; ++k) {
        A.keep_packed();
        asm volatile("" : "+v"(share));
        // the border columns' direction
        int first = tid;
        asm volatile("" : "+v"(first));  // the places are worked out here, not kept in registers
        if (tagged) {
            if (wave >= M.mw) {
#pragma unroll
                for (int u = 0; u < kSide; ++u) {
                    const int pl = place(first - M.mw * 64 + u * (TT - M.mw * 64));
                    if (side & (1u << u)) win[pl] = fma(beta, win[pl], zb[u]);
                }
            }
        } else {
            constexpr int UB = R <= 4 ? 8 : 4;  // loads in flight
            for (int u0 = 0; first + u0 * TT < border; u0 += UB) {
                const uint32_t mask = want >> u0;
                if (!__any(mask & ((1u << UB) - 1u))) continue;
                double z[UB];
#pragma unroll
                for (int u = 0; u < UB; ++u)
                    z[u] = mask & (1u << u) ? load_shared<double>(z_sh, (uint32_t)(lo + place(first + (u0 + u) * TT)))
                                            : 0.0;
#pragma unroll
                for (int u = 0; u < UB; ++u)
                    if (mask & (1u << u)) {
                        const int pl = place(first + (u0 + u) * TT);
                        win[pl] = fma(beta, win[pl], z[u]);
                    }
            }
        }
        constexpr bool kKeep = R <= 4;  // p stays in registers
        constexpr int H = 4;  // slices whose sums are formed together
        double p[R], w[R];
#pragma unroll
        for (int q = 0; q < R; ++q) {
            p[q] = fma(beta, own[q * TT], d(q) * r[q]);
            own[q * TT] = p[q];
        }
        __syncthreads();
#pragma unroll
        for (int h = 0; h < R; h += H) {
            double v[H];
#pragma unroll
            for (int q = 0; q < H; ++q) {
                w[h + q] = A.dot(h + q, base);
                v[q] = (kKeep ? p[h + q] : own[(h + q) * TT]) * w[h + q];
            }
            slices_put<R, 1, H>(red + 4 * R * TW, h, v);
        }
        double t1[1];
        if (!team_meet<R, 1>(M, red + 4 * R * TW, w_delta, (uint32_t)k, false, t1, none)) return;
        const double delta = t1[0];
        if (!(delta > 0.0)) {
            status = isfinite(delta) ? APCG_SOLVE_BREAKDOWN_PAP : APCG_SOLVE_NAN;
            break;
        }
        const double alpha = rho / delta;
#pragma unroll
        for (int h = 0; h < R; h += H) {
            double v[2 * H];
#pragma unroll
            for (int u = 0; u < H; ++u) {
                const int q = h + u;
                r[q] = fma(-alpha, w[q], r[q]);
                const double zi = d(q) * r[q];
                if (share & (1u << q)) {
                    const uint32_t i = (uint32_t)(row0 + (q * TW + wave) * 64 + lane);
                    if (tagged) post(z_w, i * 2, zi, (uint32_t)k + 1u);
                    else store_shared<double>(z_sh, i, zi);
                }
                v[2 * u] = zi * r[q];
                v[2 * u + 1] = P.norm_pre ? zi * zi : r[q] * r[q];
            }
            slices_put<R, 2, H>(red, h, v);
        }
#pragma unroll
        for (int q = 0; q < R; ++q) x(q) = fma(alpha, kKeep ? p[q] : own[q * TT], x(q));
        double t2[2];
        if (!team_meet<R, 2>(M, red, w_res, (uint32_t)k, !tagged, t2, fetch((uint32_t)k + 1u))) return;
        const double rho_new = t2[0];
        res = sqrt(t2[1]);
        its = k;
        if (!isfinite(res) || !isfinite(rho_new)) status = APCG_SOLVE_NAN;
        else if (res <= P.rtol * ref) status = APCG_SOLVE_CONVERGED;
        else if (!(rho_new > 0.0)) status = APCG_SOLVE_BREAKDOWN_RZ;
        else if (k >= P.maxit) status = APCG_SOLVE_MAXIT;
        if (P.hist && M.m == 0 && tid == 0 && k <= P.hist_cap) {
            P.hist[k - 1] = alpha;
            if (!status) P.hist[P.hist_cap + k - 1] = rho_new / rho;
        }
        if (!status) {
            beta = rho_new / rho;
            rho = rho_new;
        }
    }
    // x leaves the registers once (every member read its x0 entries before
    // the setup meeting)
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int i = row0 + (q * TW + wave) * 64 + lane;
        if (i < n) sx[i] = zero_x ? 0.0 : x(q);
    }
    if (M.m == 0 && tid == 0) {
        S.info->iterations = its;
        S.info->status = status;
        S.info->fcg_iterations = 0;
        S.info->half_steps = 0;
        S.info->res_norm = res;
        S.info->ref_norm = ref;
    }
    if (tid == 0) atomicAdd(S.done, 1u);
}

// Persistent members: each takes the next ticket until none is left.  Tickets
// are handed out in order, so at most one system is partly staffed at any
// time and the members it waits for are the next to come free; a workgroup
// that has not started holds no ticket.
template <int R, int L>
__global__ __launch_bounds__(TT, 2) void k_team_pcg(TeamPlan P) {
    extern __shared__ double lds[];
    double *win = lds + kZero;
    // sums of the setup or the residual (4), and of delta (1)
    __shared__ double red[5 * R * TW], tot[16];
    __shared__ int area[2 * TW], ok, next;
    if (threadIdx.x == 0) ok = 1;
    for (;;) {
        __syncthreads();  // the previous ticket is finished in every thread
        if (threadIdx.x == 0)
            next = __hip_atomic_load(P.stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                       ? P.tickets
                       : (int)min(atomicAdd(P.next, 1u), (uint32_t)P.tickets);
        __syncthreads();
        const int t = next;
        if (t >= P.tickets || !ok) return;
        const int2 tk = P.ticket[t];
        const int sys = __builtin_amdgcn_readfirstlane(tk.x), m = __builtin_amdgcn_readfirstlane(tk.y);
        const TeamSys S = P.sys[sys];
        const int n = __builtin_amdgcn_readfirstlane(S.n);
        const int ngr = (n + kGroupRows - 1) / kGroupRows;
        Member M{__builtin_amdgcn_readfirstlane(S.T), m, n, ngr, min((ngr + 63) / 64, kTree / 64), uniform(P.stop),
                 tot, &ok};
        team_pcg<R, L>(P, S, M, win, red, area);
    }
}

__global__ __launch_bounds__(256) void k_team_clear(uint64_t *w, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) w[i] = 0;
}

// Largest distance of a column below and above its row, over a set of
// matrices (block b strides over matrix blockIdx.y's rows).
struct BandItem {
    const int32_t *rowptr, *col;
    int32_t n, pad;
};
__global__ __launch_bounds__(256) void k_band(const BandItem *it, int32_t *out) {
    const BandItem B = it[blockIdx.y];
    int below = 0, above = 0;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < B.n; i += gridDim.x * 256)
        for (int e = B.rowptr[i]; e < B.rowptr[i + 1]; ++e) {
            below = max(below, i - B.col[e]);
            above = max(above, B.col[e] - i);
        }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        below = max(below, __shfl_xor(below, o, 64));
        above = max(above, __shfl_xor(above, o, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        if (below) atomicMax(out + 2 * blockIdx.y, below);
        if (above) atomicMax(out + 2 * blockIdx.y + 1, above);
    }
}

using TeamFn = void (*)(TeamPlan);

template <int L>
TeamFn team_fn_r(int R) {
    switch (R) {
        case 4: return k_team_pcg<4, L>;
        case 8: return L <= 5 ? k_team_pcg<8, 5> : nullptr;  // seven entries a row do not fit the registers
        default: return nullptr;
    }
}
TeamFn team_fn(int R, int L) { return L <= 5 ? team_fn_r<5>(R) : team_fn_r<7>(R); }
}  // namespace

// ------------------------------------------------------------------- host

// Team launches in flight on a device: a member waits for the other members
// of its team, so the workgroups of all team launches that may run at the
// same time must fit the chip together (one per compute unit).  A launch that
// would not fit is queued behind the ones in flight.
struct TeamFlight {
    EventRef ev;
    int wgs;
    hipStream_t stream;
};
static std::mutex g_flight_mu;
static std::vector<TeamFlight> g_flight[64];

// Queues launch() (wgs workgroups) on stream st; cus: what fits side by side.
template <class F>
static apcg_status team_launch(int device, hipStream_t st, int wgs, int cus, F launch) {
    EventRef ev = event_get(device);
    if (!ev) return set_error(APCG_ERR_HIP, "event creation failed");
    std::lock_guard<std::mutex> lk(g_flight_mu);  // admitted and counted in one step
    auto &fl = g_flight[device & 63];
    fl.erase(std::remove_if(fl.begin(), fl.end(),
                            [](const TeamFlight &f) { return hipEventQuery(f.ev->e) == hipSuccess; }),
             fl.end());
    (void)hipGetLastError();  // hipErrorNotReady of the queries
    int sum = wgs;
    for (const auto &f : fl)
        if (f.stream != st) sum += f.wgs;  // launches of this stream run one after the other
    if (sum > cus)
        for (const auto &f : fl)
            if (f.stream != st) {
                g_counters.stream_waits++;
                APCG_HIP(hipStreamWaitEvent(st, f.ev->e, 0));
            }
    apcg_status s = launch();
    if (s) return s;
    APCG_HIP(hipEventRecord(ev->e, st));
    fl.push_back({ev, wgs, st});
    return APCG_SUCCESS;
}

// Per-context buffers of the team solves.
struct TeamCache {
    int device = 0;
    int cus = 0;
    char *d_desc = nullptr;  // TeamSys[], int2 tickets[]
    int64_t desc_cap = 0;
    uint64_t desc_hash = 0;
    char *d_sync = nullptr;  // cleared before every launch: next, stop, done[], words, need marks
    int64_t sync_cap = 0;
    double *d_z = nullptr;
    int64_t z_cap = 0;
    uint32_t *pinned = nullptr;
    int64_t pinned_cap = 0;
    EventRef ev;
};
static std::mutex g_team_mu;
static std::vector<std::pair<uint64_t, TeamCache *>> g_team;

static TeamCache *team_cache(apcg_ctx c) {
    std::lock_guard<std::mutex> lk(g_team_mu);
    for (auto &p : g_team)
        if (p.first == c->id) return p.second;
    TeamCache *t = new TeamCache();
    t->device = c->device;
    g_team.emplace_back(c->id, t);
    return t;
}

void team_cache_release(uint64_t ctx_id, int device) {
    TeamCache *t = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_team_mu);
        for (auto it = g_team.begin(); it != g_team.end(); ++it)
            if (it->first == ctx_id) {
                t = it->second;
                g_team.erase(it);
                break;
            }
    }
    if (!t) return;
    hipSetDevice(device);
    hipFree(t->d_desc);
    hipFree(t->d_sync);
    hipFree(t->d_z);
    if (t->pinned) hipHostFree(t->pinned);
    delete t;
}

// Grows a device buffer; the old one may still be used by queued work.
template <typename T>
static apcg_status grow(T **p, int64_t *cap, int64_t need, int device, hipStream_t st) {
    if (*p && *cap >= need) return APCG_SUCCESS;
    if (*p) {
        EventRef ev = event_get(device);
        if (!ev) return set_error(APCG_ERR_HIP, "event creation failed");
        APCG_HIP(hipEventRecord(ev->e, st));
        T *old = *p;
        defer_release({ev}, [old, device]() {
            hipSetDevice(device);
            hipFree(old);
        });
        *p = nullptr;
        *cap = 0;
    }
    APCG_HIP(hipMalloc((void **)p, sizeof(T) * need));
    *cap = need;
    return APCG_SUCCESS;
}

// Window capacity in columns: 8 bytes each of the 160 KiB of LDS, less the
// kernel's own areas, and at most 32 border columns a thread beside the own
// rows (the bits of want).
constexpr int kWindowMax = 32 * TT + 4 * TT;

// LDS taken by x and D^-1 where a member's registers do not hold them.
static int own_columns(int R) { return rows_in_lds(R) ? 2 * TT * R : 0; }

static int team_width(int maxrow) { return maxrow <= 5 ? 5 : maxrow <= 7 ? 7 : 0; }

// The band of every matrix that does not know it yet, in one launch and one
// readback (once per matrix; a solve checks on the device that the pattern
// still fits).
static apcg_status team_bands(apcg_ctx c, int32_t nsys, const apcg_mat *A) {
    std::vector<BandItem> items;
    std::vector<apcg_mat> mats;
    int32_t nmax = 0;
    for (int32_t i = 0; i < nsys; ++i)
        if (A[i]->band_below < 0) {
            items.push_back({A[i]->rowptr, A[i]->col, A[i]->n, 0});
            mats.push_back(A[i]);
            nmax = std::max(nmax, A[i]->n);
        }
    if (items.empty()) return APCG_SUCCESS;
    const size_t ni = items.size();
    TeamCache *t = team_cache(c);
    apcg_status s;
    const int64_t bytes = (int64_t)(sizeof(BandItem) * ni + sizeof(int32_t) * 2 * ni);
    t->desc_hash = 0;  // the descriptor buffer is used as scratch
    if ((s = grow(&t->d_desc, &t->desc_cap, std::max<int64_t>(bytes, 4096), c->device, c->stream))) return s;
    int32_t *out = reinterpret_cast<int32_t *>(t->d_desc + sizeof(BandItem) * ni);
    std::vector<int32_t> h(2 * ni, 0);
    g_counters.h2d_copies += 2;
    APCG_HIP(hipMemcpyAsync(t->d_desc, items.data(), sizeof(BandItem) * ni, hipMemcpyHostToDevice, c->stream));
    APCG_HIP(hipMemcpyAsync(out, h.data(), sizeof(int32_t) * 2 * ni, hipMemcpyHostToDevice, c->stream));
    const unsigned gx = (unsigned)std::max<int64_t>(1, std::min<int64_t>((nmax + 255) / 256, 256));
    for (size_t i0 = 0; i0 < ni; i0 += 32768) {  // grid.y is limited
        const unsigned gy = (unsigned)std::min<size_t>(32768, ni - i0);
        hipLaunchKernelGGL(k_band, dim3(gx, gy), dim3(256), 0, c->stream,
                           reinterpret_cast<const BandItem *>(t->d_desc) + i0, out + 2 * i0);
        APCG_CHECK_LAUNCH("k_band");
    }
    g_counters.d2h_copies++;
    APCG_HIP(hipMemcpyAsync(h.data(), out, sizeof(int32_t) * 2 * ni, hipMemcpyDeviceToHost, c->stream));
    if (!t->ev && !(t->ev = event_get(c->device))) return set_error(APCG_ERR_HIP, "event creation failed");
    APCG_HIP(hipEventRecord(t->ev->e, c->stream));
    g_counters.host_polls++;
    APCG_HIP(hipEventSynchronize(t->ev->e));
    for (size_t i = 0; i < ni; ++i) {
        mats[i]->band_below = h[2 * i];
        mats[i]->band_above = h[2 * i + 1];
    }
    return APCG_SUCCESS;
}

// Slices per wavefront (R) for systems of these sizes: four while all members
// run side by side, else eight (of five-entry rows): a member of 4096 rows
// takes an iteration about 1.25 times as long as one of 2048, so a batch that
// queues for the compute units finishes sooner.  0: some system does not fit.
static int team_rows(int32_t nsys, const apcg_mat *A, int cus, int width) {
    int best = 0;
    for (int R : {4, 8}) {
        if (R == 8 && width > 5) break;
        int64_t total = 0;
        bool ok = true;
        for (int32_t i = 0; i < nsys && ok; ++i) {
            const int64_t T = std::max<int64_t>(1, ((int64_t)A[i]->n + TT * R - 1) / (TT * R));
            const int64_t window = (T == 1 ? 0 : (int64_t)A[i]->band_below + A[i]->band_above) + TT * R + 64;
            ok = T <= cus && window <= kWindowMax - own_columns(R);
            total += T;
        }
        if (!ok) continue;
        best = R;
        if (total <= cus) break;
    }
    return best;
}

apcg_status team_eligible(apcg_ctx c, int32_t nsys, const apcg_mat *A, int *rows) {
    *rows = 0;
    if (c->type == APCG_STREAM_GLOBAL_BLOCKING) return APCG_SUCCESS;
    int maxrow = 1;
    for (int32_t i = 0; i < nsys; ++i) {
        maxrow = std::max(maxrow, A[i]->sell_maxw);
        if (!team_width(maxrow) || A[i]->n > 256 * TT * kMaxRows) return APCG_SUCCESS;
    }
    TeamCache *t = team_cache(c);
    if (!t->cus) APCG_HIP(hipDeviceGetAttribute(&t->cus, hipDeviceAttributeMultiprocessorCount, c->device));
    apcg_status s;
    if ((s = team_bands(c, nsys, A))) return s;
    *rows = team_rows(nsys, A, t->cus, team_width(maxrow));
    return APCG_SUCCESS;
}

apcg_status team_pcg_solve(apcg_ctx c, int32_t nsys, const apcg_mat *A, const apcg_vec *b, const apcg_vec *x,
                           const std::vector<int32_t> &order, double rtol, int32_t maxit, const apcg_solve_opts &opts,
                           int rows, apcg_solve_info *info, double *hist, int32_t hist_cap,
                           std::vector<int32_t> *left) {
    left->clear();
    TeamCache *t = team_cache(c);
    hipStream_t st = c->stream;
    const int R = rows;
    int maxrow = 1, window = 0;
    int64_t zn = 0, marks = 0, words = 0, tickets = 0;
    std::vector<TeamSys> sys(nsys);
    for (int32_t i = 0; i < nsys; ++i) {
        TeamSys &s = sys[i];
        s.rowptr = A[i]->rowptr;
        s.col = A[i]->col;
        s.val = A[i]->val;
        s.b = b[i]->d;
        s.x = x[i]->d;
        s.n = A[i]->n;
        s.T = (int32_t)std::max<int64_t>(1, ((int64_t)s.n + TT * R - 1) / (TT * R));
        s.info = info + i;
        maxrow = std::max(maxrow, A[i]->sell_maxw);
        const int64_t border = s.T == 1 ? 0 : (int64_t)A[i]->band_below + A[i]->band_above + 64;
        window = std::max<int>(window, (int)std::min<int64_t>(kWindowMax - own_columns(R), TT * R + border));
        const int64_t ngr = ((int64_t)s.n + kGroupRows - 1) / kGroupRows;
        // what the wavefronts beside at most four that collect messages fetch at once
        s.tagged = R <= 4 && border <= kSide * (TT - kTree) ? 1 : 0;
        s.z = reinterpret_cast<uint64_t *>(zn);
        s.need = reinterpret_cast<uint8_t *>(marks);
        s.words = reinterpret_cast<uint64_t *>(words);
        if (s.T > 1) {
            zn += ((int64_t)s.n + 63) / 64 * 64 * (s.tagged ? 2 : 1);
            marks += ((int64_t)s.n + 63) / 64 * 64;
            words += ngr * kStride;
        }
        tickets += s.T;
    }
    std::vector<int2> tk;
    tk.reserve(tickets);
    for (int32_t i : order)
        for (int m = 0; m < sys[i].T; ++m) tk.push_back(make_int2(i, m));
    // cleared area: next, stop, done counts, messages, marks
    const int64_t head = (8 + (int64_t)nsys * 4 + 63) / 64 * 64;
    const int64_t sync_bytes = head + 8 * words + marks;
    apcg_status s;
    if ((s = grow(&t->d_sync, &t->sync_cap, sync_bytes, t->device, st))) return s;
    if ((s = grow(&t->d_z, &t->z_cap, std::max<int64_t>(zn, 64), t->device, st))) return s;
    uint32_t *head_p = reinterpret_cast<uint32_t *>(t->d_sync);
    for (int32_t i = 0; i < nsys; ++i) {
        TeamSys &q = sys[i];
        q.z = reinterpret_cast<uint64_t *>(t->d_z) + reinterpret_cast<int64_t>(q.z);
        q.words = reinterpret_cast<uint64_t *>(t->d_sync + head) + reinterpret_cast<int64_t>(q.words);
        q.need = reinterpret_cast<uint8_t *>(t->d_sync + head + 8 * words) + reinterpret_cast<int64_t>(q.need);
        q.done = head_p + 2 + i;
    }
    const int64_t sys_bytes = (int64_t)sizeof(TeamSys) * nsys, tk_bytes = (int64_t)sizeof(int2) * tickets;
    if ((s = grow(&t->d_desc, &t->desc_cap, std::max<int64_t>(sys_bytes + tk_bytes, 4096), t->device, st))) return s;
    std::vector<char> desc((size_t)(sys_bytes + tk_bytes));
    memcpy(desc.data(), sys.data(), sys_bytes);
    memcpy(desc.data() + sys_bytes, tk.data(), tk_bytes);
    uint64_t h = 1469598103934665603ull ^ (uint64_t)(uintptr_t)t->d_desc;
    for (char ch : desc) h = (h ^ (unsigned char)ch) * 1099511628211ull;
    if (h == 0) h = 1;

    if (h != t->desc_hash) {
        g_counters.h2d_copies++;
        APCG_HIP(hipMemcpyAsync(t->d_desc, desc.data(), desc.size(), hipMemcpyHostToDevice, st));
        t->desc_hash = h;

    }
    if (t->pinned_cap < nsys + 2) {
        if (t->pinned) hipHostFree(t->pinned);
        t->pinned = nullptr;
        t->pinned_cap = 0;
        APCG_HIP(hipHostMalloc((void **)&t->pinned, sizeof(uint32_t) * (nsys + 2), hipHostMallocDefault));
        t->pinned_cap = nsys + 2;
    }
    TeamPlan P{};
    P.sys = reinterpret_cast<const TeamSys *>(t->d_desc);
    P.ticket = reinterpret_cast<const int2 *>(t->d_desc + sys_bytes);
    P.next = head_p;
    P.stop = head_p + 1;
    P.tickets = (int32_t)tickets;
    P.window = window;
    P.rtol = rtol;
    P.maxit = maxit;
    P.x0_zero = opts.x0_is_zero ? 1 : 0;
    P.pc = opts.pc;
    P.norm_pre = opts.norm_type == APCG_NORM_PRECONDITIONED;
    P.hist = hist;
    P.hist_cap = hist ? hist_cap : 0;
    const TeamFn fn = team_fn(R, team_width(maxrow));
    const size_t lds = sizeof(double) * (size_t)(window + kZero + own_columns(R));
    if (lds > 65536 - 4096)
        APCG_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)(sizeof(double) * (kWindowMax + kZero))));
    const int grid = (int)std::min<int64_t>(tickets, t->cus);
    const int64_t cw = (sync_bytes + 7) / 8;
    hipLaunchKernelGGL(k_team_clear, dim3((unsigned)std::min<int64_t>(1024, (cw + 255) / 256)), dim3(256), 0, st,
                       reinterpret_cast<uint64_t *>(t->d_sync), cw);
    APCG_CHECK_LAUNCH("k_team_clear");
    s = team_launch(t->device, st, grid, t->cus, [&]() -> apcg_status {
        hipLaunchKernelGGL(fn, dim3(grid), dim3(TT), lds, st, P);
        APCG_CHECK_LAUNCH("k_team_pcg");
        return APCG_SUCCESS;
    });
    if (s) return s;
    // the members that finished, observed through an event like the other
    // schedules' stop flags
    g_counters.d2h_copies++;
    APCG_HIP(hipMemcpyAsync(t->pinned, head_p, sizeof(uint32_t) * (nsys + 2), hipMemcpyDeviceToHost, st));
    if (!t->ev && !(t->ev = event_get(t->device))) return set_error(APCG_ERR_HIP, "event creation failed");
    APCG_HIP(hipEventRecord(t->ev->e, st));
    g_counters.host_polls++;
    APCG_HIP(hipEventSynchronize(t->ev->e));

    for (int32_t i = 0; i < nsys; ++i)
        if (t->pinned[2 + i] != (uint32_t)sys[i].T) left->push_back(i);
    if (t->pinned[1] == 2)  // a pattern changed in place: measured again next time
        for (int32_t i : *left) A[i]->band_below = A[i]->band_above = -1;
    return APCG_SUCCESS;
}

}  // namespace apcg
