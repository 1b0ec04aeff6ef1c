// team.hip -- Jacobi-PCG of one or many systems that fit the chip, each held
// by a team of workgroups (team.h): the whole solve is one launch.
//
// What bounds it: the multi-kernel iteration of a system of 8e3 to 6e5 rows
// is bound by its kernel boundaries and, in the segmented batch, by streaming
// every vector and the matrix through the caches again in every kernel.  Here
// nothing but D^-1 r of the rows at the members' borders leaves the compute
// units between two iterations, and an iteration is bound by its two meetings
// (1.2 to 1.8 us each).  Microseconds per iteration, before and after:
//   2D, 30k rows   10.0   4.6        3D, 64^3 (262k rows)   15.8   7.0
//   2D, 250k rows  15     5.7
// and 256 2D systems of 1e3 to 6.5e4 rows in one call: 192 ms, now 28.6.  The
// direction of the border columns is kept and updated by every member that
// reads it (p = z + beta p, the same operation on the same values), so only z
// travels.
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

#define TEAM_ASK __attribute__((noinline))  // (see there)
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
    uint32_t *verdict;
    int32_t n, T;
    int32_t tagged;      // z travels as tagged words (few border columns)
    int32_t limit;       // border columns a member may have: there is room for more, but no plan
};

struct TeamPlan {
    const TeamSys *sys;
    const int2 *ticket;   // (system, member), a system's members in a row
    uint32_t *head;       // kHeadWords words
    TeamWait wait;
    int32_t tickets;
    double rtol;
    int32_t maxit, x0_zero, pc, norm_pre;
    double *hist;         // one system only: alpha, beta of the first hist_cap iterations
    int32_t hist_cap;
};

// Eight slices a wavefront leave no registers for x and D^-1 beside the
// entries, r and w: they lie in LDS behind the window then (kept in registers
// they spilled, and a member of 4096 rows took 7.6 us an iteration instead of
// 5.5).  Seven registers still spill, 32 bytes a lane; four slices spill none
// (233 registers of five-entry rows, 253 of seven).
constexpr bool rows_in_lds(int R) { return R == 8; }

template <int R, int L>
__device__ __forceinline__ void team_pcg(const TeamPlan &P, const TeamSys &S, Member &M, double *win, double *red,
                                         int *area) {
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
    const int row0 = M.m * kOwn<R>, row1 = min(n, row0 + kOwn<R>);
    // LDS: the window (of p), D^-1 and x where the registers do not hold them,
    // the border's columns
    const int limit = __builtin_amdgcn_readfirstlane(S.limit), wsize = window_size(R, limit);
    double *own = win + kPad + wave * 64 + lane;  // this thread's row of slice 0; rows past the last hold zeros
    double *dl = win + wsize + wave * 64 + lane, *xl = dl + kOwn<R>;
    uint16_t *list = (uint16_t *)(win + wsize + (rows_in_lds(R) ? 2 * kOwn<R> : 0));
    double r[R], dreg[R], xreg[R];
    // D^-1 and x of this thread's row of slice q
    auto d = [&](int q) -> double & {
        if constexpr (rows_in_lds(R)) return dl[q * TT];
        else return dreg[q];
    };
    auto x = [&](int q) -> double & {
        if constexpr (rows_in_lds(R)) return xl[q * TT];
        else return xreg[q];
    };
    unsigned share = 0;  // bit q: this row of slice q is stored for the other members

    // ---- setup: entries, D^-1, r0, z0 and the four setup sums
    uint64_t lens;
    const bool fits = load_rows<R, L>(A, rowptr, col, val, n, row0, lens, [&](int q, int i, bool in, int len,
                                      const int32_t (&cj)[L], double diag, bool found) {
        double ax = 0.0;
        if (!P.x0_zero) {
#pragma unroll
            for (int t = 0; t < L; ++t)
                if (t < len) ax = fma(A.a[q][t], sx[cj[t]], ax);
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
    });
    if (!__syncthreads_and(fits)) return refuse(M, kUnfit);
    const int nb = make_border<R, L>(A, lens, row1 - row0, (uint32_t *)win, list, limit, area);
    if (nb > limit) return refuse(M, kUnfit);
    for (int i = tid; i < wsize; i += TT) win[i] = 0.0;
    // the column of border place c; the owners keep storing z of these rows
    auto column = [&](int c) { return (uint32_t)(row0 + (int)list[c] - kBias); };
    for (int c = tid; c < nb; c += TT) store_shared<uint8_t>(need, column(c), 1);
    // A short border's z is fetched during the meeting, by the wavefronts that
    // collect no messages, as its tags arrive: neither an acknowledged store
    // before the message nor a round trip after it.
    double zb[kSide];
    auto fetch = [&](uint32_t tag) {
        return [&, tag](int t, int nt) {
            static_assert(kSide == 4, "load_pairs");
#pragma unroll
            for (int u = 0; u < kSide; ++u) zb[u] = 0.0;
            if (!tagged || t >= nb) return true;
            uint32_t at4[kSide];  // past the border's end: its first column again
#pragma unroll
            for (int u = 0; u < kSide; ++u) at4[u] = column(t + u * nt < nb ? t + u * nt : t) * 2;
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
    if (wave >= M.mw && !fetch(1u)(tid - M.mw * 64, TT - M.mw * 64)) M.out->ok[1] = 0;
    __syncthreads();
    if (!M.out->ok[1]) return;
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
    double beta = 0.0;
    for (int k = 1; !status; ++k) {
        A.keep_packed();
        asm volatile("" : "+v"(share));
        // the border columns' direction
        double *border = win + kPad + kOwn<R>;
        if (tagged) {
            if (wave >= M.mw) {
#pragma unroll
                for (int u = 0; u < kSide; ++u) {
                    const int c = tid - M.mw * 64 + u * (TT - M.mw * 64);
                    if (c < nb) border[c] = fma(beta, border[c], zb[u]);
                }
            }
        } else {
            // Loads in flight: nine are the best at every 3D size (48^3 4, 6, 8,
            // 9 and 12 in flight: 6.43, 6.28, 6.27, 6.04 and 6.11 us an
            // iteration, 64^3 7.36, 7.25, 7.18, 7.00 and 7.10, 78^3 10.1, 9.9,
            // 9.9, 9.6 and 9.9); eight slices leave registers for four.
            constexpr int UB = R <= 4 ? 9 : 4;
            for (int c0 = tid; c0 < nb; c0 += UB * TT) {
                double z[UB];
#pragma unroll
                for (int u = 0; u < UB; ++u)
                    z[u] = c0 + u * TT < nb ? load_shared<double>(z_sh, column(c0 + u * TT)) : 0.0;
#pragma unroll
                for (int u = 0; u < UB; ++u) {
                    const int c = c0 + u * TT;
                    if (c < nb) border[c] = fma(beta, border[c], z[u]);
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
                w[h + q] = A.dot(h + q, win);
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
    if (!finish(M)) return;
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
}

// Persistent members: each takes the next ticket until none is left.  Tickets
// are handed out in order, so at most one system is partly staffed at any
// time and the members it waits for are the next to come free; a workgroup
// that has not started holds no ticket.
template <int R, int L>
__global__ __launch_bounds__(TT, 2) void k_team_pcg(TeamPlan P) {
    extern __shared__ double lds[];
    double *win = lds;
    // sums of the setup or the residual (4), and of delta (1)
    __shared__ double red[5 * R * TW], tot[16];
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
        const TeamSys S = P.sys[sys];
        const int n = __builtin_amdgcn_readfirstlane(S.n);
        const int ngr = (n + kGroupRows - 1) / kGroupRows;
        const int T = __builtin_amdgcn_readfirstlane(S.T);
        set_exit(out, P.head, S.verdict, P.wait.ticks, t - m + T);
        Member M{T, m, n, ngr, min((ngr + 63) / 64, kTree / 64), P.wait.look, tot, &out};
        team_pcg<R, L>(P, S, M, win, red, area);
    }
}

__global__ __launch_bounds__(256) void k_team_clear(uint64_t *w, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) w[i] = 0;
}

// The most border columns of any member, for members of 2048 and 4096 rows
// (out[2 y], out[2 y + 1] of matrix blockIdx.y; blockIdx.z: which).  A column
// outside the 16-bit range counts as more than any border.
struct BorderItem {
    const int32_t *rowptr, *col;
    int32_t n, pad;
};
__global__ __launch_bounds__(256) void k_border(const BorderItem *it, int32_t *out) {
    const BorderItem B = it[blockIdx.y];
    const int rows = blockIdx.z ? kOwn<8> : kOwn<4>;
    __shared__ uint32_t marks[kMarkWords];
    __shared__ int far;
    for (int row0 = blockIdx.x * rows; row0 < B.n; row0 += gridDim.x * rows) {
        const int row1 = min(B.n, row0 + rows);
        for (int i = threadIdx.x; i < kMarkWords; i += 256) marks[i] = 0u;
        if (threadIdx.x == 0) far = 0;
        __syncthreads();
        const int e1 = B.rowptr[row1];
        for (int e = B.rowptr[row0] + (int)threadIdx.x; e < e1; e += 256) {
            const int c = B.col[e], rel = c - row0 + kBias;
            if (c >= row0 && c < row1) continue;
            if (rel < 0 || rel >= 65536) far = 1;
            else atomicOr(&marks[rel >> 5], 1u << (rel & 31));
        }
        __syncthreads();
        int cnt = 0;
        for (int i = threadIdx.x; i < kMarkWords; i += 256) cnt += __popc(marks[i]);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
        __shared__ int part[4];
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = cnt;
        __syncthreads();
        if (threadIdx.x == 0)
            atomicMax(out + 2 * blockIdx.y + blockIdx.z, far ? 1 << 24 : part[0] + part[1] + part[2] + part[3]);
        __syncthreads();
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

std::mutex g_flight_mu;
std::vector<TeamFlight> *const g_flight = new std::vector<TeamFlight>[64];  // (not taken down at exit)

static std::mutex g_team_mu;
static std::vector<std::pair<uint64_t, TeamCache *>> g_team;

TeamCache *team_cache(apcg_ctx c) {
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
    hipFree(t->mem);
    hipFree(t->d_swap);
    if (t->pinned) hipHostFree(t->pinned);
    if (t->reports) hipHostFree(t->reports);
    delete t;
}

apcg_status LeftRecords::open(apcg_ctx ctx, int32_t n) {
    char *p = nullptr;
    APCG_HIP(hipMalloc((void **)&p, (sizeof(apcg_solve_info) + sizeof(double) + 9 * sizeof(float)) * n));
    ctx_ = ctx;
    info = reinterpret_cast<apcg_solve_info *>(p);
    lmax = reinterpret_cast<double *>(info + n);
    coeffs = reinterpret_cast<float *>(lmax + n);
    return APCG_SUCCESS;
}

apcg_status LeftRecords::copy_polynomials(const std::vector<int32_t> &left, const float *all_coeffs,
                                          const double *all_lmax) {
    hipStream_t st = ctx_->stream;
    for (size_t k = 0; k < left.size(); ++k) {
        APCG_HIP(hipMemcpyAsync(coeffs + 9 * k, all_coeffs + 9 * (size_t)left[k], 9 * sizeof(float),
                                hipMemcpyDeviceToDevice, st));
        APCG_HIP(hipMemcpyAsync(lmax + k, all_lmax + left[k], sizeof(double), hipMemcpyDeviceToDevice, st));
    }
    return APCG_SUCCESS;
}

apcg_status LeftRecords::copy_back(const std::vector<int32_t> &left, apcg_solve_info *all) {
    for (size_t k = 0; k < left.size(); ++k)
        APCG_HIP(hipMemcpyAsync(all + left[k], info + k, sizeof(apcg_solve_info), hipMemcpyDeviceToDevice,
                                ctx_->stream));
    return APCG_SUCCESS;
}

LeftRecords::~LeftRecords() {
    if (!info) return;
    EventRef ev = event_get(ctx_->device);
    if (!ev || event_record(ev, ctx_->stream) != hipSuccess) return;
    const int dev = ctx_->device;
    apcg_solve_info *p = info;
    defer_release({ev}, [p, dev]() {
        hipSetDevice(dev);
        hipFree(p);
    });
}

int64_t team_lds(int R, int nb, int windows, bool own_vectors) {
    const int64_t doubles = (int64_t)windows * window_size(R, nb) + (own_vectors ? 2 * TT * R : 0);
    return std::max<int64_t>(8 * doubles, 8 * kMarkWords) + (2 * (int64_t)nb + 15) / 8 * 8;
}

apcg_status team_memory(TeamCache *t, hipStream_t st, int64_t desc, int64_t sync, int64_t z) {
    auto up = [](int64_t b) { return (b + 255) / 256 * 256; };
    const int64_t need = up(desc) + up(sync) + up(z);
    if (need > t->mem_cap) {
        apcg_status s = grow(&t->mem, &t->mem_cap, std::max<int64_t>(need, 1 << 20), t->device, st);
        if (s) return s;
    }
    t->d_desc = t->mem;
    t->d_sync = t->mem + up(desc);
    t->d_z = reinterpret_cast<uint64_t *>(t->d_sync + up(sync));
    return APCG_SUCCESS;
}

apcg_status team_clear(hipStream_t st, uint64_t *words, int64_t n) {
    if (n <= 0) return APCG_SUCCESS;
    hipLaunchKernelGGL(k_team_clear, dim3((unsigned)std::min<int64_t>(1024, (n + 255) / 256)), dim3(256), 0, st, words,
                       n);
    APCG_CHECK_LAUNCH("k_team_clear");
    return APCG_SUCCESS;
}

apcg_status team_swap(TeamCache *t, hipStream_t st, int64_t words, int64_t tags, uint32_t *tag) {
    if (t->swap_cap < words || t->tag + tags > (int64_t)1 << 32) {
        apcg_status s;
        if ((s = grow(&t->d_swap, &t->swap_cap, std::max<int64_t>(words, 64), t->device, st))) return s;
        if ((s = team_clear(st, t->d_swap, t->swap_cap))) return s;
        t->tag = 1;
    }
    *tag = (uint32_t)t->tag;
    t->tag += tags;
    return APCG_SUCCESS;
}

apcg_status team_upload(TeamCache *t, hipStream_t st, const void *sys, int64_t sys_bytes,
                        const std::vector<int32_t> &order, const std::vector<int32_t> &members, const char **d_sys,
                        const int2 **d_tickets) {
    int64_t tickets = 0;
    for (int32_t m : members) tickets += m;
    std::vector<int2> tk;
    tk.reserve((size_t)tickets);
    for (int32_t i : order)
        for (int m = 0; m < members[i]; ++m) tk.push_back(make_int2(i, m));
    const int64_t tk_bytes = (int64_t)sizeof(int2) * tickets;
    auto desc = std::make_shared<std::vector<char>>((size_t)(sys_bytes + tk_bytes));
    memcpy(desc->data(), sys, (size_t)sys_bytes);
    memcpy(desc->data() + sys_bytes, tk.data(), (size_t)tk_bytes);
    uint64_t h = 1469598103934665603ull ^ (uint64_t)(uintptr_t)t->d_desc;
    for (char ch : *desc) h = (h ^ (unsigned char)ch) * 1099511628211ull;
    if (h == 0) h = 1;
    if (h != t->desc_hash) {
        g_counters.h2d_copies++;
        APCG_HIP(hipMemcpyAsync(t->d_desc, desc->data(), desc->size(), hipMemcpyHostToDevice, st));
        t->desc_hash = h;
        EventRef ev = event_get(t->device);
        if (!ev) return set_error(APCG_ERR_HIP, "event creation failed");
        APCG_HIP(event_record(ev, st));
        defer_release({ev}, [desc]() {});  // the host's copy lives until it has been read
    }
    *d_sys = t->d_desc;
    *d_tickets = reinterpret_cast<const int2 *>(t->d_desc + sys_bytes);
    return APCG_SUCCESS;
}

// What a verdict other than done says about the matrix (may be null) and the chip.
static void team_left(TeamCache *t, TeamState *m, uint32_t verdict) {
    if (verdict == kUnfit) {  // (changed in place)
        if (!m) return;
        ++m->unfit;
        m->reread = true;
    } else if (verdict == kOneSided) {
        if (m) m->one_sided = true;
    } else {
        t->rest = 256;  // a wait ran out: the chip is shared, no teams for a while
    }
}

// Numbers a launch that nobody waits for.
static apcg_status team_later(TeamCache *t, int32_t nsys, const apcg_mat *A, TeamLater *later) {
    if (!t->reports) {
        APCG_HIP(hipHostMalloc((void **)&t->reports, sizeof(uint64_t) * kReports, hipHostMallocDefault));
        memset(t->reports, 0, sizeof(uint64_t) * kReports);
    }
    const uint64_t k = ++t->launches;
    auto &mats = t->reported[k % kReports];
    mats.clear();
    for (int32_t i = 0; i < nsys; ++i) mats.push_back(A[i]->team);
    later->verdicts = reinterpret_cast<const uint32_t *>(t->d_sync) + kHeadWords;
    later->report = t->reports + k % kReports;
    later->launch = k << 40;
    return APCG_SUCCESS;
}

// Reads what those launches have reported (the last of a launch's systems).
static void team_reports(TeamCache *t) {
    if (!t->reports) return;
    for (int q = 0; q < kReports; ++q) {
        volatile uint64_t *word = t->reports + q;
        const uint64_t w = *word;
        if (!w) continue;
        *word = 0;
        const uint64_t now = t->launches - (t->launches - (uint64_t)q) % kReports;  // the launch this word is for now
        const size_t i = (size_t)((w >> 8 & 0xffffffffull) - 1);
        const auto &mats = t->reported[q];
        const bool known = (w >> 40) == (now & 0xffffffull) && i < mats.size();
        team_left(t, known ? mats[i].lock().get() : nullptr, (uint32_t)(w & 255));
    }
}

apcg_status team_finish(apcg_ctx ctx, TeamCache *t, int32_t nsys, const apcg_mat *A, std::vector<int32_t> *left) {
    hipStream_t st = ctx->stream;
    // a few verdicts fit the words the context's polls use (pinning memory
    // takes longer than a small solve)
    uint32_t *host = reinterpret_cast<uint32_t *>(ctx->pinned_flags);
    if (nsys > kMaxLookahead) {
        if (t->pinned_cap < nsys) {
            if (t->pinned) hipHostFree(t->pinned);
            t->pinned = nullptr;
            t->pinned_cap = 0;
            APCG_HIP(hipHostMalloc((void **)&t->pinned, sizeof(uint32_t) * nsys, hipHostMallocDefault));
            t->pinned_cap = nsys;
        }
        host = t->pinned;
    }
    // observed through an event, like the other schedules' stop flags
    g_counters.d2h_copies++;
    APCG_HIP(hipMemcpyAsync(host, t->d_sync + 4 * kHeadWords, sizeof(uint32_t) * nsys, hipMemcpyDeviceToHost, st));
    if (!t->ev && !(t->ev = event_get(t->device))) return set_error(APCG_ERR_HIP, "event creation failed");
    APCG_HIP(event_record(t->ev, st));
    g_counters.host_polls++;
    APCG_HIP(hipEventSynchronize(t->ev->e));
    for (int32_t i = 0; i < nsys; ++i) {
        if (host[i] == kDone) continue;
        left->push_back(i);
        team_left(t, A[i]->team.get(), host[i]);
    }
    return APCG_SUCCESS;
}

static int team_width(int maxrow) { return maxrow <= 5 ? 5 : maxrow <= 7 ? 7 : 0; }

// The border of every matrix that does not know it yet, in one launch and one
// readback (once per matrix; a solve checks on the device that the pattern
// still fits).
// border[w][i]: of system i's members of 2048 (w = 0) and 4096 rows.
static apcg_status team_borders(apcg_ctx c, int32_t nsys, const apcg_mat *A, std::vector<int32_t> (&border)[2]) {
    std::vector<BorderItem> items;
    std::vector<int32_t> which;
    int32_t nmax = 0;
    TeamCache *t = team_cache(c);
    for (auto &b : border) b.assign(nsys, 0);
    for (int32_t i = 0; i < nsys; ++i) {
        TeamState &m = *A[i]->team;
        for (int w = 0; w < 2; ++w) border[w][i] = m.reread ? -1 : m.border[w].load();
        if (border[0][i] < 0 || border[1][i] < 0) {
            items.push_back({A[i]->rowptr, A[i]->col, A[i]->n, 0});
            which.push_back(i);
            nmax = std::max(nmax, A[i]->n);
        }
    }
    if (items.empty()) return APCG_SUCCESS;
    const size_t ni = items.size();
    apcg_status s;
    const int64_t bytes = (int64_t)(sizeof(BorderItem) * ni + sizeof(int32_t) * 2 * ni);
    t->desc_hash = 0;  // the descriptor buffer is used as scratch
    if ((s = team_memory(t, c->stream, bytes, 0, 0))) return s;
    int32_t *out = reinterpret_cast<int32_t *>(t->d_desc + sizeof(BorderItem) * ni);
    std::vector<int32_t> h(2 * ni, 0);
    g_counters.h2d_copies += 2;
    APCG_HIP(hipMemcpyAsync(t->d_desc, items.data(), sizeof(BorderItem) * ni, hipMemcpyHostToDevice, c->stream));
    APCG_HIP(hipMemcpyAsync(out, h.data(), sizeof(int32_t) * 2 * ni, hipMemcpyHostToDevice, c->stream));
    const unsigned gx = (unsigned)std::max<int64_t>(1, std::min<int64_t>(((int64_t)nmax + 2047) / 2048, 512));
    for (size_t i0 = 0; i0 < ni; i0 += 32768) {  // grid.y is limited
        const unsigned gy = (unsigned)std::min<size_t>(32768, ni - i0);
        hipLaunchKernelGGL(k_border, dim3(gx, gy, 2), dim3(256), 0, c->stream,
                           reinterpret_cast<const BorderItem *>(t->d_desc) + i0, out + 2 * i0);
        APCG_CHECK_LAUNCH("k_border");
    }
    g_counters.d2h_copies++;
    APCG_HIP(hipMemcpyAsync(h.data(), out, sizeof(int32_t) * 2 * ni, hipMemcpyDeviceToHost, c->stream));
    if (!t->ev && !(t->ev = event_get(c->device))) return set_error(APCG_ERR_HIP, "event creation failed");
    APCG_HIP(event_record(t->ev, c->stream));
    g_counters.host_polls++;
    APCG_HIP(hipEventSynchronize(t->ev->e));
    for (size_t i = 0; i < ni; ++i) {
        TeamState &m = *A[which[i]]->team;
        if (m.reread.exchange(false) && (m.border[0] != h[2 * i] || m.border[1] != h[2 * i + 1])) m.unfit = 0;
        for (int w = 0; w < 2; ++w) m.border[w] = border[w][which[i]] = h[2 * i + w];
    }
    return APCG_SUCCESS;
}

// Slices per wavefront (R) for systems of these sizes: four while all members
// run side by side, else eight (of five-entry rows): a member of 4096 rows
// takes an iteration about 1.25 times as long as one of 2048, so a batch that
// queues for the compute units finishes sooner.  0: some system does not fit.
static int team_rows(int32_t nsys, const apcg_mat *A, const std::vector<int32_t> (&border)[2], int cus, int width,
                     int windows) {
    int best = 0;
    for (int R : {4, 8}) {
        if (R == 8 && (width > 5 || windows > 1)) break;
        int64_t total = 0;
        bool ok = true;
        for (int32_t i = 0; i < nsys && ok; ++i) {
            const int64_t T = std::max<int64_t>(1, ((int64_t)A[i]->n + TT * R - 1) / (TT * R));
            const int nb = border[R == 8][i];
            ok = T <= cus && nb >= 0 && nb < 1 << 20 && team_lds(R, nb, windows, rows_in_lds(R)) <= kLdsBytes;
            total += T;
        }
        if (!ok) continue;
        best = R;
        if (total <= cus) break;
    }
    return best;
}

apcg_status team_eligible(apcg_ctx c, int32_t nsys, const apcg_mat *A, int windows, TeamFit *fit) {
    fit->rows = 0;
    if (c->type == APCG_STREAM_GLOBAL_BLOCKING) return APCG_SUCCESS;
    int maxrow = 1;
    for (int32_t i = 0; i < nsys; ++i) {
        maxrow = std::max(maxrow, A[i]->sell_maxw);
        if (!team_width(maxrow) || A[i]->n > 256 * TT * kMaxRows) return APCG_SUCCESS;
        if (A[i]->team->unfit > 1 || (windows > 1 && A[i]->team->one_sided)) return APCG_SUCCESS;
    }
    TeamCache *t = team_cache(c);
    team_reports(t);
    if (t->rest > 0) {
        --t->rest;
        return APCG_SUCCESS;
    }
    if (!t->cus) APCG_HIP(hipDeviceGetAttribute(&t->cus, hipDeviceAttributeMultiprocessorCount, c->device));
    apcg_status s;
    std::vector<int32_t> border[2];
    if ((s = team_borders(c, nsys, A, border))) return s;
    fit->rows = team_rows(nsys, A, border, t->cus, team_width(maxrow), windows);
    fit->border = std::move(border[fit->rows == 8]);
    return APCG_SUCCESS;
}

apcg_status team_pcg_solve(apcg_ctx c, int32_t nsys, const apcg_mat *A, const apcg_vec *b, const apcg_vec *x,
                           const std::vector<int32_t> &order, double rtol, int32_t maxit, const apcg_solve_opts &opts,
                           const TeamFit &fit, apcg_solve_info *info, double *hist, int32_t hist_cap,
                           std::vector<int32_t> *left, TeamLater *later) {
    TeamCache *t = team_cache(c);
    hipStream_t st = c->stream;
    const int R = fit.rows;
    int maxrow = 1, border = 0;
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
        const int nb = s.T == 1 ? 0 : fit.border[i];
        border = std::max(border, nb);
        const int64_t ngr = ((int64_t)s.n + kGroupRows - 1) / kGroupRows;
        // what the wavefronts beside at most four that collect messages fetch at once
        s.tagged = R <= 4 && nb <= kSide * (TT - kTree) ? 1 : 0;
        s.limit = s.tagged ? kSide * (TT - kTree) : INT32_MAX;  // (and that of the widest, for which there is room)
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
    // cleared area: the head, verdicts, messages, marks
    const int64_t head = team_head_bytes(nsys);
    const int64_t sync_bytes = head + 8 * words + marks;
    apcg_status s;
    if ((s = team_memory(t, st, team_desc_bytes((int64_t)sizeof(TeamSys) * nsys, tickets), sync_bytes, 8 * zn))) return s;
    uint32_t *head_p = reinterpret_cast<uint32_t *>(t->d_sync);
    for (int32_t i = 0; i < nsys; ++i) {
        TeamSys &q = sys[i];
        q.z = t->d_z + reinterpret_cast<int64_t>(q.z);
        q.words = reinterpret_cast<uint64_t *>(t->d_sync + head) + reinterpret_cast<int64_t>(q.words);
        q.need = reinterpret_cast<uint8_t *>(t->d_sync + head + 8 * words) + reinterpret_cast<int64_t>(q.need);
        q.verdict = head_p + kHeadWords + i;
    }
    std::vector<int32_t> members(nsys);
    for (int32_t i = 0; i < nsys; ++i) {
        members[i] = sys[i].T;
        sys[i].limit = std::min(sys[i].limit, border);
    }
    const char *d_sys;
    const int2 *d_tickets;
    if ((s = team_upload(t, st, sys.data(), (int64_t)sizeof(TeamSys) * nsys, order, members, &d_sys, &d_tickets)))
        return s;
    TeamPlan P{};
    P.sys = reinterpret_cast<const TeamSys *>(d_sys);
    P.ticket = d_tickets;
    P.head = head_p;
    P.wait = t->wait;
    P.tickets = (int32_t)tickets;
    P.rtol = rtol;
    P.maxit = maxit;
    P.x0_zero = opts.x0_is_zero ? 1 : 0;
    P.pc = opts.pc;
    P.norm_pre = opts.norm_type == APCG_NORM_PRECONDITIONED;
    P.hist = hist;
    P.hist_cap = hist ? hist_cap : 0;
    const TeamFn fn = team_fn(R, team_width(maxrow));
    const size_t lds = (size_t)team_lds(R, border, 1, rows_in_lds(R));
    APCG_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                 (int)kLdsBytes));
    const int grid = (int)std::min<int64_t>(tickets, t->cus);
    if ((s = team_clear(st, reinterpret_cast<uint64_t *>(t->d_sync), (sync_bytes + 7) / 8))) return s;
    s = team_launch(t->device, st, grid, t->cus, [&]() -> apcg_status {
        hipLaunchKernelGGL(fn, dim3(grid), dim3(TT), lds, st, P);
        APCG_CHECK_LAUNCH("k_team_pcg");
        return APCG_SUCCESS;
    });
    if (s) return s;
    return left ? team_finish(c, t, nsys, A, left) : team_later(t, nsys, A, later);
}

}  // namespace apcg

// For tests, not part of the interface: the waits of ctx's team launches from
// now on (TeamWait).
extern "C" void apcg_internal_set_team_wait(apcg_ctx ctx, int64_t ticks, int32_t look) {
    apcg::team_cache(ctx)->wait = apcg::TeamWait{ticks, look};
}
