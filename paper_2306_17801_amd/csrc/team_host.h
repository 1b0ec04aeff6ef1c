// team_host.h -- host side of the team solves (team.hip, team_fcg.hip,
// team_tfqmr.hip).
#pragma once

#include <algorithm>
#include <mutex>
#include <vector>

#include "internal.h"

namespace apcg {

// Single solves take the team schedule above this many rows.
constexpr int32_t kTeamMinRows = 8192;

// Longest wait for one message (ticks of the 100 MHz clock; 2 s): far beyond
// any solve's step; then other work, another process's team say, holds the
// compute units of members that are due: no more tickets are handed out, and
// what is left is solved by the other schedules.  Not counted is the time in
// which the first members of a system wait in the setup for workgroups that
// solve the systems before it, however long that takes.
constexpr long long kWaitTicks = 200000000ll;
struct TeamWait {
    long long ticks;
    int32_t look;  // the clock is read at every look + 1 unsuccessful looks (a power of two less one)
};

// The words before the verdicts: the next ticket to hand out; nonzero once a
// wait has run out, after which no tickets are handed out; tickets that are
// through.
constexpr int kHeadNext = 0, kHeadStop = 1, kHeadThrough = 2, kHeadWords = 4;
// A system's verdict: nobody has seen its end or left it; x is solved; a wait
// has run out; its rows or their border do not fit; one member reads another
// that does not read it (flexible solve).  The last three: x as it was.
constexpr uint32_t kOpen = 0, kDone = 1, kLeft = 2, kUnfit = 3, kOneSided = 4;

// Team launches in flight on a device, by stream: a member waits for the other
// members of its team, so the workgroups of all team launches that may run at
// the same time must fit the chip together (one per compute unit).  A launch
// that would not fit is queued behind the ones in flight.
struct TeamFlight {
    EventRef ev;         // of the stream's last launch (it keeps the stream, so no other has its name)
    int wgs;             // of its largest since it had none
    hipStream_t stream;
};
extern std::mutex g_flight_mu;
extern std::vector<TeamFlight> *const g_flight;  // one for each device

// Queues launch() (wgs workgroups) on stream st; cus: what fits side by side.
template <class F>
apcg_status team_launch(int device, hipStream_t st, int wgs, int cus, F launch) {
    EventRef ev = event_get(device);
    if (!ev) return set_error(APCG_ERR_HIP, "event creation failed");
    std::lock_guard<std::mutex> lk(g_flight_mu);  // admitted and counted in one step
    auto &fl = g_flight[device & 63];
    fl.erase(std::remove_if(fl.begin(), fl.end(),
                            [](const TeamFlight &f) { return hipEventQuery(f.ev->e) == hipSuccess; }),
             fl.end());
    (void)hipGetLastError();  // hipErrorNotReady of the queries
    int sum = wgs;
    TeamFlight *own = nullptr;
    for (auto &f : fl)
        if (f.stream != st) sum += f.wgs;  // (launches of one stream run one after the other)
        else own = &f;
    if (sum > cus)
        for (const auto &f : fl)
            if (f.stream != st) {
                g_counters.stream_waits++;
                APCG_HIP(hipStreamWaitEvent(st, f.ev->e, 0));
            }
    apcg_status s = launch();
    if (s) return s;
    APCG_HIP(event_record(ev, st));
    if (own) *own = {ev, std::max(own->wgs, wgs), st};
    else fl.push_back({ev, wgs, st});
    return APCG_SUCCESS;
}

// A launch nobody waits for: what it leaves is solved by a kernel queued behind
// it (k_pcg_left), which reports each such system to the host: where the
// verdicts lie, and what to write where (pinned memory).
struct TeamLater {
    const uint32_t *verdicts = nullptr;
    uint64_t *report = nullptr;
    uint64_t launch = 0;  // its number, in the upper 24 bits
};
// Its report of system i: the launch, i + 1 (32 bits), the verdict (8 bits).
constexpr int kReports = 64;  // launches whose reports the host can still tell apart

// Records of the systems that teams have left, by their place among them: the
// results, and the flexible solve's polynomials.  Given back once ctx's work
// queued until then has run.
struct LeftRecords {
    apcg_solve_info *info = nullptr;
    double *lmax = nullptr;
    float *coeffs = nullptr;
    apcg_status open(apcg_ctx ctx, int32_t n);
    apcg_status copy_polynomials(const std::vector<int32_t> &left, const float *all_coeffs, const double *all_lmax);
    apcg_status copy_back(const std::vector<int32_t> &left, apcg_solve_info *all);
    ~LeftRecords();

private:
    apcg_ctx ctx_ = nullptr;
};

// Per-context buffers of the team solves.
struct TeamCache {
    int device = 0;
    int cus = 0;
    TeamWait wait{kWaitTicks, 255};
    uint64_t launches = 0;   // that nobody waits for
    uint64_t *reports = nullptr;  // pinned, kReports words: of launch k in word k modulo kReports
    std::vector<std::weak_ptr<TeamState>> reported[kReports];  // the matrices of those launches
    int rest = 0;            // solves to leave to the other schedules after a wait that ran out
    char *mem = nullptr;     // one buffer for the three below (an allocation costs as much as a small solve)
    int64_t mem_cap = 0;
    char *d_desc = nullptr;  // the systems, int2 tickets[]
    uint64_t desc_hash = 0;
    char *d_sync = nullptr;  // cleared before every launch: the head, verdicts, words, marks
    uint64_t *d_z = nullptr; // border values
    uint64_t *d_swap = nullptr;  // border exchanges of the flexible solve; tags below tag are used up
    int64_t swap_cap = 0, tag = 1;
    uint32_t *pinned = nullptr;
    int64_t pinned_cap = 0;
    EventRef ev;
};
TeamCache *team_cache(apcg_ctx c);

// Grows a device buffer; the old one may still be used by queued work.
template <typename T>
apcg_status grow(T **p, int64_t *cap, int64_t need, int device, hipStream_t st) {
    if (*p && *cap >= need) return APCG_SUCCESS;
    if (*p) {
        EventRef ev = event_get(device);
        if (!ev) return set_error(APCG_ERR_HIP, "event creation failed");
        APCG_HIP(event_record(ev, st));
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

// LDS a member may take (160 KiB less the kernels' fixed areas), and what
// `windows` windows take with nb border columns.
constexpr int64_t kLdsBytes = 163840 - 4096;
int64_t team_lds(int R, int nb, int windows, bool own_vectors);

// Makes room for so many bytes of descriptors, cleared memory and border
// values of the next launch.
apcg_status team_memory(TeamCache *t, hipStream_t st, int64_t desc, int64_t sync, int64_t z);
inline int64_t team_desc_bytes(int64_t sys_bytes, int64_t tickets) { return sys_bytes + tickets * (int64_t)sizeof(int2); }

// Clears n words on stream st (a kernel: a launch may be captured).
apcg_status team_clear(hipStream_t st, uint64_t *words, int64_t n);

// Makes room for so many words of border exchanges and sets tags aside that
// no word there carries; *tag is the first.
apcg_status team_swap(TeamCache *t, hipStream_t st, int64_t words, int64_t tags, uint32_t *tag);

// Uploads the systems' descriptors and the tickets (members[i] of system i,
// systems in `order`) unless the device holds them already.
apcg_status team_upload(TeamCache *t, hipStream_t st, const void *sys, int64_t sys_bytes,
                        const std::vector<int32_t> &order, const std::vector<int32_t> &members, const char **d_sys,
                        const int2 **d_tickets);

// Bytes of the head and the verdicts at the start of d_sync.
inline int64_t team_head_bytes(int32_t nsys) { return (4 * (kHeadWords + (int64_t)nsys) + 63) / 64 * 64; }

// Waits for the launch and lists the systems that are not done.
apcg_status team_finish(apcg_ctx ctx, TeamCache *t, int32_t nsys, const apcg_mat *A, std::vector<int32_t> *left);

// How teams would solve some systems.
struct TeamFit {
    int rows = 0;                 // 64-row slices per wavefront, 0: not by teams
    std::vector<int32_t> border;  // most border columns of a member, by system
};

// Whether every system can be solved by teams on ctx's device: rows of at
// most 7 entries, `windows` windows that fit the LDS (1: PCG, 2: the flexible
// solve), no system larger than the chip, none that members have refused.
// Reads the matrices' borders back, and waits for them, once per matrix.
apcg_status team_eligible(apcg_ctx ctx, int32_t nsys, const apcg_mat *A, int windows, TeamFit *fit);

// Jacobi-PCG (or CG) of the systems, started in `order` (largest cost
// first), results in info[i]; hist as in pcg_solve_marked (one system).
// Returns once the launch has finished; *left holds the systems it did not
// solve (their x untouched), which the caller solves with another schedule.
// Without left, returns at once, and the caller queues what solves the systems
// whose verdict is not done (*later).
apcg_status team_pcg_solve(apcg_ctx ctx, int32_t nsys, const apcg_mat *A, const apcg_vec *b, const apcg_vec *x,
                           const std::vector<int32_t> &order, double rtol, int32_t maxit, const apcg_solve_opts &opts,
                           const TeamFit &fit, apcg_solve_info *info, double *hist, int32_t hist_cap,
                           std::vector<int32_t> *left, TeamLater *later = nullptr);

// FCG(1) of the systems with their polynomials coeffs[i][9], lmax[i] (device),
// as apcg_ksp_solve_batched_fcg_poly; otherwise as team_pcg_solve.
apcg_status team_fcg_solve(apcg_ctx ctx, int32_t nsys, const apcg_mat *A, const apcg_vec *b, const apcg_vec *x,
                           const std::vector<int32_t> &order, double rtol, int32_t maxit, const apcg_solve_opts &opts,
                           const apcg_fcg_opts &fo, const TeamFit &fit, const float *coeffs, const double *lmax,
                           apcg_solve_info *info, std::vector<int32_t> *left);
// TFQMR of one system with members of 2048 rows (team_eligible: rows == 4),
// as apcg_ksp_solve_tfqmr; otherwise as team_pcg_solve.
apcg_status team_tfqmr_solve(apcg_ctx ctx, apcg_mat A, apcg_vec b, apcg_vec x, double rtol, int32_t maxit,
                             const apcg_solve_opts &opts, const TeamFit &fit, apcg_solve_info *info,
                             std::vector<int32_t> *left);
// The tags one flexible launch may use are limited (see team_fcg.hip).
constexpr int32_t kTeamFcgMaxIts = 100000000;

// When nobody waits for a launch, one workgroup per system solves what is left:
// up to so many rows times iterations (about a second).
constexpr int64_t kLeftWork = (int64_t)1 << 25;
}  // namespace apcg
