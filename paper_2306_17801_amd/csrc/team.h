// team.h -- device side of the team solves: a system held on the chip by a
// team of workgroups that exchange only what crosses their borders.
//
// A team of T workgroups owns one system for its whole solve.  Member m owns
// rows [512 R m, 512 R (m + 1)): its eight wavefronts take the 64-row slices
// 8 q + wave (q < R) of that range, one row per lane, and keep the matrix
// entries and every vector of those rows in registers.  The members meet
// twice per Krylov step, at the two inner products.  A meeting is one
// message per group of 32 slices, and every member waits for all groups'
// messages, so it is the grid-wide barrier and the reduction in one: measured
// on an idle MI355X at 1.2 us (8 members), 1.6 us (64) and 2.4 us (256),
// where a kernel boundary costs about 4 us once its first loads have
// arrived.
//
// Messages carry their own arrival mark: a double travels as two 64-bit
// words, each holding half of it and the 32-bit tag of the step, so no flag
// has to follow the data and be ordered after it.  All traffic between
// members goes through agent-scope relaxed atomics, which neither stay in an
// XCD's L2 (stores) nor are served from it (loads).  Vector entries the
// other members read are stored the same way, and every wavefront waits for
// its own stores (s_waitcnt vmcnt(0)) before the barrier behind which the
// message that announces them leaves.  An agent-scope release fence does the
// same ordering but writes back the whole L2: 58-76 us a meeting at 256
// members.
//
// Members never wait for a workgroup that has not started: work is handed
// out by ticket (see TeamPlan), so every workgroup that a member waits for
// is running or is the next to start.  Every wait is bounded all the same,
// and a member whose wait runs out, or whose rows are not what the schedule
// was chosen for, leaves its system.
//
// x is written by all members of a system or by none.  A system's verdict is
// open until member 0, when it has seen the system's end, sets it to done, or
// one that leaves sets it to something else, whichever is first; the others
// wait for it.  Member 0 has every member's last message then, so every member
// has sent it and can only be waiting for the others', which are on their way:
// a member that wants to leave a system that is done goes on waiting instead
// and finds them.
#pragma once

#include "internal.h"
#include "team_host.h"

namespace apcg {
namespace team {

// Threads of a member: eight wavefronts with 256 registers each.  (Sixteen
// with 128 spill from two slices on: 4096 rows took 9.2 us an iteration.)
constexpr int TT = 512;
constexpr int TW = TT / 64;      // its wavefronts
constexpr int kGroup = 32;       // 64-row slices per message: the rows of a member at R = 4
constexpr int kGroupRows = 64 * kGroup;
constexpr int kMaxRows = 8;      // slices per wavefront (R): 4 or 8
// Words from one group's messages to the next: 256 bytes, so that neighbours
// lie in different memory channels.  Every member reads every message, and
// packed messages share a few channels: 123 members on 2.5e5 rows took 9.4 us
// an iteration packed, 7.3 at 64 bytes apart and 6.7 at 256.
constexpr int kStride = 32;
constexpr int kTree = 256;       // threads of the reduction tree over groups
constexpr int kSide = 4;         // border entries a thread may fetch during a meeting


// Global pointers the compiler keeps in scalar registers: the values read
// from a device table are the same in every lane, which it cannot see.
template <class T>
using gptr = dev::glob_t<T> *;
template <class T>
__device__ __forceinline__ gptr<T> uniform(T *p) {
    const uint64_t b = (uint64_t)p;
    const uint32_t l = __builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    const uint32_t h = __builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
    return (gptr<T>)((uint64_t)h << 32 | l);
}

// Entry i of a table with a scalar base and an offset below 4 GiB: one 32-bit
// register of address per access instead of two.
template <class T>
__device__ __forceinline__ gptr<T> at(gptr<T> p, uint32_t i) {
    return (gptr<T>)((gptr<char>)p + i * (uint32_t)sizeof(T));
}
template <class T>
__device__ __forceinline__ const dev::glob_t<T> *at(const dev::glob_t<T> *p, uint32_t i) {
    return (const dev::glob_t<T> *)((const dev::glob_t<char> *)p + i * (uint32_t)sizeof(T));
}

template <class T>
__device__ __forceinline__ T load_shared(gptr<T> p, uint32_t i) {
    return __hip_atomic_load(at(p, i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ void store_shared(gptr<T> p, uint32_t i, T v) {
    __hip_atomic_store(at(p, i), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Every store this wavefront has issued has reached the device's point of
// coherence (stores count in vmcnt on this architecture).
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// What a member needs when it waits long or leaves, in LDS: in registers it
// would push some of the matrix out.
struct Exit {
    uint32_t *head;     // the launch's kHeadWords words
    uint32_t *verdict;  // the system's
    long long ticks;    // TeamWait
    uint32_t last;      // one more than the system's last ticket
    int ok[2];          // 0 once a wait has failed: in a meeting, between meetings
};

// A member's place in its team, the same in all its threads.
struct Member {
    int T, m;        // members, this one's index
    int n;           // rows of the system
    int ngr;         // groups of the system
    int mw;          // wavefronts that collect messages (the others are free for a side job)
    int look;        // TeamWait
    double *tot;     // LDS: 4 * 4 tree sums
    Exit *out;       // LDS
};

__device__ __forceinline__ uint32_t exchange_if(gptr<uint32_t> p, uint32_t from, uint32_t to) {
    __hip_atomic_compare_exchange_strong(p, &from, to, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return from;  // what was there
}

// The rare part of keep_waiting: the time from which the wait counts (t0: since
// when it did, 0 at first), or -1 when the member leaves its system.  A call in
// the PCG kernels, where it cost 3 to 8% of an iteration with 240 members to
// have it in every loop that waits (700 x 700: 8.7 us, 8.0 as a call); the
// flexible solve and TFQMR are 1% to 4% better off without calls.
#ifndef TEAM_ASK
#define TEAM_ASK __forceinline__
#endif
__device__ TEAM_ASK long long ask(const Exit *E, int T, long long t0) {
    const gptr<uint32_t> head = (gptr<uint32_t>)E->head, verdict = (gptr<uint32_t>)E->verdict;
    const long long now = wall_clock64();
    if (t0 == 0) t0 = now;
    const uint32_t v = load_shared<uint32_t>(verdict, 0);
    if (v == kDone) return now - t0 <= E->ticks + kWaitTicks ? t0 : -1;  // the messages are on their way
    if (v != kOpen) return -1;                                          // a team mate has left
    // the system lacks members: they come when tickets before its own are through
    const bool lacks = load_shared<uint32_t>(head, kHeadNext) < E->last;
    if (lacks && load_shared<uint32_t>(head, kHeadThrough) < E->last - (uint32_t)T) t0 = now;
    const bool late = now - t0 > E->ticks;
    if (late) store_shared<uint32_t>(head, kHeadStop, 1u);
    else if (!lacks || !load_shared<uint32_t>(head, kHeadStop)) return t0;
    return exchange_if(verdict, kOpen, kLeft) == kDone ? t0 : -1;
}

// Whether to look at a message again after so many unsuccessful looks (counted
// by the caller, in a scalar register); every now and then that is a question
// of the clock and of the others.  t0: 0 at first.
__device__ __forceinline__ bool keep_waiting(const Member &M, int spin, long long &t0) {
    if (__builtin_expect((spin & M.look) != M.look, 1)) return true;
    t0 = ask(M.out, M.T, t0);
    return t0 >= 0;
}

// A ticket's exit; thread 0 sets it up while the others wait for the setup's
// first barrier.
__device__ __forceinline__ void set_exit(Exit &E, uint32_t *head, uint32_t *verdict, long long ticks, int last) {
    if (threadIdx.x != 0) return;
    E.head = head;
    E.verdict = verdict;
    E.ticks = ticks;
    E.last = (uint32_t)last;
    E.ok[0] = E.ok[1] = 1;
}

// The next ticket (through: the last one is); `tickets` when there is none, or
// none are handed out any more.
__device__ __forceinline__ int next_ticket(uint32_t *head, int tickets, bool through) {
    if (through) __hip_atomic_fetch_add(head + kHeadThrough, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__hip_atomic_load(head + kHeadStop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return tickets;
    return (int)min(atomicAdd(head + kHeadNext, 1u), (uint32_t)tickets);
}

// At the end of a system, in all threads of a member: whether the member may
// write its x.
__device__ __forceinline__ bool finish(const Member &M) {
    if (M.T == 1) {
        if (threadIdx.x == 0) *M.out->verdict = kDone;
        return true;
    }
    __syncthreads();  // nobody looks at ok any more
    if (threadIdx.x == 0) {
        const gptr<uint32_t> verdict = (gptr<uint32_t>)M.out->verdict;
        // one member says so, the others wait for it (an exchange by each of 240 takes 10 us)
        uint32_t v = M.m == 0 ? exchange_if(verdict, kOpen, kDone) : kOpen;
        if (M.m == 0 && v == kOpen) v = kDone;
        long long t0 = 0;
        for (int spin = 0; v == kOpen && keep_waiting(M, spin, t0); ++spin) v = load_shared<uint32_t>(verdict, 0);
        if (v != kDone) M.out->ok[0] = 0;
    }
    __syncthreads();
    return M.out->ok[0] != 0;
}

__device__ __forceinline__ double unpack(uint64_t lo, uint64_t hi) {
    return __longlong_as_double((long long)((lo & 0xffffffffull) | (hi << 32)));
}

// Sends v as the two words at words + i (16-byte aligned), in one 16-byte
// store that does not stay in the L2 (store_shared twice would write every
// other 8 bytes of a line, and then the rest).  The s_nop keeps the vector
// unit off the data registers until the store has read them.
__device__ __forceinline__ void post(gptr<uint64_t> words, uint32_t i, double v, uint32_t tag) {
    typedef uint32_t v4 __attribute__((ext_vector_type(4)));
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const v4 d = {(uint32_t)b, tag, (uint32_t)(b >> 32), tag};
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 2" : : "v"(at(words, i)), "v"(d) : "memory");
}

// The NW words (a multiple of two, 16-byte aligned) at words + i, by 16-byte
// loads that miss the L2 like load_shared (each word carries its own tag, so
// nothing is assumed of the two words together).  Half the requests of
// single words: what the members' looks cost is requests at the channel that
// holds a message.
template <int NW>
__device__ __forceinline__ void load_message(gptr<uint64_t> words, uint32_t i, uint64_t (&w)[NW]) {
    static_assert(NW == 2 || NW == 4 || NW == 8, "message sizes");
    typedef uint32_t v4 __attribute__((ext_vector_type(4)));
    const gptr<uint64_t> p = at(words, i);
    v4 a, b, c, d;
    if constexpr (NW == 2)
        asm volatile("global_load_dwordx4 %0, %1, off sc1\n\ts_waitcnt vmcnt(0)" : "=&v"(a) : "v"(p) : "memory");
    if constexpr (NW == 4)
        asm volatile("global_load_dwordx4 %0, %2, off sc1\n\tglobal_load_dwordx4 %1, %2, off offset:16 sc1\n\t"
                     "s_waitcnt vmcnt(0)" : "=&v"(a), "=&v"(b) : "v"(p) : "memory");
    if constexpr (NW == 8)
        asm volatile("global_load_dwordx4 %0, %4, off sc1\n\tglobal_load_dwordx4 %1, %4, off offset:16 sc1\n\t"
                     "global_load_dwordx4 %2, %4, off offset:32 sc1\n\tglobal_load_dwordx4 %3, %4, off offset:48 sc1\n\t"
                     "s_waitcnt vmcnt(0)" : "=&v"(a), "=&v"(b), "=&v"(c), "=&v"(d) : "v"(p) : "memory");
    auto put = [&](int k, const v4 &x) {
        w[k] = (uint64_t)x[1] << 32 | x[0];
        w[k + 1] = (uint64_t)x[3] << 32 | x[2];
    };
    put(0, a);
    if constexpr (NW >= 4) put(2, b);
    if constexpr (NW == 8) {
        put(4, c);
        put(6, d);
    }
}

// Four pairs of words at once, one from each place i of the buffer.
// (Addresses in vector registers: a scalar base written by the vector unit
// just before would need wait states that the compiler does not put before an
// asm block.)
__device__ __forceinline__ void load_pairs(gptr<uint64_t> words, const uint32_t (&i)[4], uint64_t (&w)[4][2]) {
    typedef uint32_t v4 __attribute__((ext_vector_type(4)));
    v4 a[4];
    asm volatile("global_load_dwordx4 %0, %4, off sc1\n\tglobal_load_dwordx4 %1, %5, off sc1\n\t"
                 "global_load_dwordx4 %2, %6, off sc1\n\tglobal_load_dwordx4 %3, %7, off sc1\n\t"
                 "s_waitcnt vmcnt(0)"
                 : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3])
                 : "v"(at(words, i[0])), "v"(at(words, i[1])), "v"(at(words, i[2])), "v"(at(words, i[3]))
                 : "memory");
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        w[k][0] = (uint64_t)a[k][1] << 32 | a[k][0];
        w[k][1] = (uint64_t)a[k][3] << 32 | a[k][2];
    }
}

// Adds the NV doubles of group g's message to acc once it carries `tag`;
// false when the member leaves its system.
template <int NV>
__device__ __forceinline__ bool collect(const Member &M, gptr<uint64_t> words, int g, uint32_t tag,
                                        double (&acc)[NV]) {
    long long t0 = 0;
    for (int spin = 0;; ++spin) {
        uint64_t w[2 * NV];
        load_message<2 * NV>(words, (uint32_t)(g * kStride), w);
        bool all = true;
#pragma unroll
        for (int k = 0; k < 2 * NV; ++k) all = all && (uint32_t)(w[k] >> 32) == tag;
        if (all) {
#pragma unroll
            for (int k = 0; k < NV; ++k) acc[k] += unpack(w[2 * k], w[2 * k + 1]);
            return true;
        }
        if (!keep_waiting(M, spin, t0)) return false;
    }
}

// a + b of the two vectors a half-wave or row swap of (x, y) leaves: lanes of
// the first half (row) hold x's pair sums, those of the second y's.
__device__ __forceinline__ double swap_add32(double x, double y) {
    const uint64_t a = (uint64_t)__double_as_longlong(x), b = (uint64_t)__double_as_longlong(y);
    const auto l = __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)b, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
    return __longlong_as_double((long long)((uint64_t)h[0] << 32 | l[0])) +
           __longlong_as_double((long long)((uint64_t)h[1] << 32 | l[1]));
}
__device__ __forceinline__ double swap_add16(double x, double y) {
    const uint64_t a = (uint64_t)__double_as_longlong(x), b = (uint64_t)__double_as_longlong(y);
    const auto l = __builtin_amdgcn_permlane16_swap((uint32_t)a, (uint32_t)b, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
    return __longlong_as_double((long long)((uint64_t)h[0] << 32 | l[0])) +
           __longlong_as_double((long long)((uint64_t)h[1] << 32 | l[1]));
}

// Wavefront sums of N values (N a power of two), each added in the pairs of
// dev::wave_sum and so to the same bits, four values to a register: the first
// two steps of four butterflies are three additions instead of eight, and
// the remaining four steps serve four values at once.  Value i's sum goes to
// *out(i).
template <int N, class Out>
__device__ __forceinline__ void wave_sums(const double (&v)[N], Out out) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < N; i += 4) {
        const double a = v[i], b = v[i + (N > 1 ? 1 : 0)], c = v[i + (N > 2 ? 2 : 0)], d = v[i + (N > 2 ? 3 : 0)];
        const double ab = swap_add32(a, b);  // lanes 0..31: a, 32..63: b
        const double cd = N > 2 ? swap_add32(c, d) : ab;
        double s = swap_add16(ab, cd);       // rows of 16 lanes: a, c, b, d
        s += dev::dpp_row<0x128>(s);
        s += dev::dpp_row<0x124>(s);
        s += dev::dpp_row<0x122>(s);
        s += dev::dpp_row<0x121>(s);
        if ((lane & 15) == 0) {
            const int row = lane >> 4;
            const int id = N > 2 ? i + ((row & 1) << 1 | row >> 1) : N > 1 ? row >> 1 : 0;
            *out(id) = s;  // fewer than four values: rows of equal sums
        }
    }
}

// The sums over the system's rows of NV values per row, in two steps: every
// wavefront puts the sums of its slices (slices_put), then the team meets
// (team_meet) and every thread of every member holds the totals.  The order
// is that of the segmented schedule (sys_sum in batched.hip): the 64 rows of
// a slice and the 32 slices of a group by butterflies, groups l, l + 256, ...
// by thread l of a 256-thread tree.  It does not depend on T or R.
// red: NV areas of 8 R slice sums, one for each value.
// v[q * NV + k]: value k of this thread's row of slice q0 + q.
template <int R, int NV, int NQ>
__device__ __forceinline__ void slices_put(double *red, int q0, const double (&v)[NQ * NV]) {
    double *mine = red + q0 * TW + (threadIdx.x >> 6);
    wave_sums<NQ * NV>(v, [=](int i) { return mine + i % NV * (R * TW) + i / NV * TW; });
}

// words: group 0's message of this meeting (2 NV words, kStride from group to
// group), tag: its step.
// ack: wait for this wavefront's shared stores before the message leaves, so
// that they are visible to whoever has received it.
// Between its own message and the others' the wavefronts that collect no
// messages run side(thread, threads) -> bool.  red is free again after the
// next meeting's (other) red has been put.  A team of one does not end the
// meeting with a barrier: the caller puts the next sums into another area, or
// passes a barrier first.
// Returns false when the member leaves its system.
template <int R, int NV, class Side>
__device__ __forceinline__ bool team_meet(const Member &M, const double *red, gptr<uint64_t> words, uint32_t tag,
                                          bool ack, double (&total)[NV], Side side) {
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    if (M.T == 1) {  // the whole system is here, in one or two groups: the tree in every wavefront
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const double g = dev::half_sum(lane < R * TW ? red[k * (R * TW) + lane] : 0.0);
            total[k] = swap_add32(g, g);
        }
        return true;
    }
    if (ack) wait_stores();
    __syncthreads();
    if (tid < R * TW * NV) {  // half wavefront (q, k): value k of the member's group q
        const int q = tid / (32 * NV), k = tid / 32 % NV, g = M.m * (R * TW / kGroup) + q;
        const double t = dev::half_sum(red[k * (R * TW) + q * kGroup + (tid & 31)]);
        if ((tid & 31) == 0 && g < M.ngr) post(words, (uint32_t)(g * kStride + k * 2), t, tag);
    }
    bool good = true;
    double acc[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) acc[k] = 0.0;
    if (wave < M.mw) {
        for (int g = tid; good && g < M.ngr; g += kTree) good = collect<NV>(M, words, g, tag, acc);
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const double t = dev::wave_sum(acc[k]);
            if (lane == 0) M.tot[k * (kTree / 64) + wave] = t;
        }
    } else {
        good = side(tid - M.mw * 64, TT - M.mw * 64);
    }
    if (!good) M.out->ok[0] = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        double t = M.tot[k * (kTree / 64)];
        for (int w = 1; w < M.mw; ++w) t += M.tot[k * (kTree / 64) + w];  // the other wavefronts' sums are zeros
        total[k] = t;
    }
    return M.out->ok[0] != 0;
}

// The rows of a member: matrix entries in registers, the columns as places in
// the member's window.  A window is the LDS copy of one vector where the
// member needs it: place 0 holds 0 (the column of absent entries), places
// kPad on its own rows, then the border -- the columns of other members that
// some own row names, in column order.
constexpr int kPad = 8;
constexpr int kBias = 32768;       // columns relative to the first own row, as 16-bit col - row0 + kBias
constexpr int kMarkWords = 65536 / 32;  // one bit for each of those
template <int R>
constexpr int kOwn = TT * R;       // own places
// Doubles of LDS of one window with nb border columns.
constexpr int window_size(int R, int nb) { return (kPad + TT * R + nb + 7) / 8 * 8; }

template <int R, int L>
struct Rows {
    double a[R][L];
    uint32_t j[R][(L + 1) / 2];  // two 16-bit places a word

    __device__ __forceinline__ int place(int q, int t) const { return (int)((j[q][t >> 1] >> (16 * (t & 1))) & 0xffffu); }
    __device__ __forceinline__ void set(int q, int t, int v) {
        j[q][t >> 1] = (j[q][t >> 1] & ~(0xffffu << (16 * (t & 1)))) | (uint32_t)v << (16 * (t & 1));
    }

    // The packed places are unpacked where they are used: without this the
    // compiler keeps every unpacked place in a register of its own across
    // the iterations, and spills.
    __device__ __forceinline__ void keep_packed() {
#pragma unroll
        for (int q = 0; q < R; ++q)
#pragma unroll
            for (int t = 0; t < (L + 1) / 2; ++t) asm volatile("" : "+v"(j[q][t]));
    }

    // sum_t a_t win[j_t] in storage order, one FMA per entry (an absent one
    // adds 0 * 0)
    __device__ __forceinline__ double dot(int q, const double *win) const {
        double g[L];
#pragma unroll
        for (int t = 0; t < L; ++t) g[t] = win[place(q, t)];
        double sum = 0.0;
#pragma unroll
        for (int t = 0; t < L; ++t) sum = fma(a[q][t], g[t], sum);
        return sum;
    }
};

// Loads the member's rows: entries and relative columns; lens: row lengths,
// four bits each.  row(q, i, in, len, cj, diag, found) does the rest of a
// row's setup.  False in some thread when an entry does not fit (a row longer
// than L, a column outside the matrix or too far away): the pattern is not
// the one this schedule was chosen for.
template <int R, int L, class Row>
__device__ __forceinline__ bool load_rows(Rows<R, L> &A, gptr<const int32_t> rowptr, gptr<const int32_t> col,
                                          gptr<const double> val, int n, int row0, uint64_t &lens, Row row) {
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    bool fits = true;
    lens = 0;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int i = row0 + (q * TW + wave) * 64 + lane;
        const bool in = i < n;
        const int s = in ? rowptr[i] : 0, len = in ? rowptr[i + 1] - s : 0;
        fits = fits && len <= L;
        int32_t cj[L];
        double diag = 0.0;
        bool found = false;
#pragma unroll
        for (int t = 0; t < (L + 1) / 2; ++t) A.j[q][t] = 0;
#pragma unroll
        for (int t = 0; t < L; ++t) {
            const bool has = t < len;
            cj[t] = has ? col[s + t] : row0;
            A.a[q][t] = has ? val[s + t] : 0.0;
            const int rel = cj[t] - row0 + kBias;
            fits = fits && cj[t] >= 0 && cj[t] < (has ? n : 0x7fffffff) && rel >= 0 && rel < 65536;
            A.set(q, t, rel & 0xffff);
            if (has && cj[t] == i) {
                diag = A.a[q][t];
                found = true;
            }
        }
        lens |= (uint64_t)(uint32_t)min(len, 15) << (4 * q);
        row(q, i, in, len, cj, diag, found);
        __builtin_amdgcn_sched_barrier(0);  // one slice at a time: the loads of all would not fit the registers
    }
    return fits;
}

// Turns the relative columns into places and lists the border: list[c] is the
// relative column of border place c.  scratch: kMarkWords uint32 of marks and
// as many of ranks (LDS, overwritten); area: 8 ints of LDS.  Returns the
// border's length (more than cap: nothing was listed).  Ends with a barrier.
template <int R, int L>
__device__ __forceinline__ int make_border(Rows<R, L> &A, uint64_t lens, int own, uint32_t *scratch, uint16_t *list,
                                           int cap, int *area) {
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    constexpr int PER = kMarkWords / TT;
    uint32_t *marks = scratch, *rank = scratch + kMarkWords;
    for (int i = tid; i < kMarkWords; i += TT) marks[i] = 0u;
    __syncthreads();
    auto mine = [&](int rel) { return rel >= kBias && rel < kBias + own; };
#pragma unroll
    for (int q = 0; q < R; ++q)
#pragma unroll
        for (int t = 0; t < L; ++t) {
            const int rel = A.place(q, t);
            if (t < ((int)(lens >> (4 * q)) & 15) && !mine(rel)) atomicOr(&marks[rel >> 5], 1u << (rel & 31));
        }
    __syncthreads();
    int cnt = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) cnt += __popc(marks[tid * PER + i]);
    int scan = cnt;  // inclusive over the wavefront
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int up = __shfl_up(scan, o, 64);
        if (lane >= o) scan += up;
    }
    if (lane == 63) area[wave] = scan;
    __syncthreads();
    int first = scan - cnt, nb = 0;
#pragma unroll
    for (int w = 0; w < TW; ++w) {
        if (w < wave) first += area[w];
        nb += area[w];
    }
    for (int i = 0; i < PER; ++i) {
        const int word = tid * PER + i;
        rank[word] = (uint32_t)first;
        uint32_t m = marks[word];
        while (m) {
            const int bit = __ffs(m) - 1;
            if (first < cap) list[first] = (uint16_t)(word * 32 + bit);
            ++first;
            m &= m - 1;
        }
    }
    __syncthreads();
    if (nb <= cap) {
#pragma unroll
        for (int q = 0; q < R; ++q)
#pragma unroll
            for (int t = 0; t < L; ++t) {
                const int rel = A.place(q, t);
                const int border = (int)rank[rel >> 5] + __popc(marks[rel >> 5] & ((1u << (rel & 31)) - 1u));
                A.set(q, t, t < ((int)(lens >> (4 * q)) & 15)
                                ? (mine(rel) ? kPad + rel - kBias : kPad + kOwn<R> + border)
                                : 0);
            }
    }
    __syncthreads();
    return nb;
}

// Leaves the system, whose pattern is not the one the schedule was chosen for
// (why: kUnfit or kOneSided).  Nobody can have seen the system's end: it takes
// messages that this member has not sent.
__device__ __forceinline__ void refuse(const Member &M, uint32_t why) {
    if (threadIdx.x == 0) __hip_atomic_fetch_max(M.out->verdict, why, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace team
}  // namespace apcg
