// Pieces shared by the 32-bit planner kernels: the LDS row entry, the per-stage constants, scalar
// helpers, the LDS-only barrier, and the workspace layout the pre-pass and the DP kernels agree on.
#pragma once

#include "harp_internal.h"

namespace harp {
namespace fastdp {

constexpr uint32_t kInf32 = 0xFFFFFFFFu;
constexpr int kPad = 4;
constexpr int kFastThreads = 256;
constexpr uint32_t kRowMask = (1u << 27) - 1u;
constexpr uint32_t kDeadStatusShift = 30;   // dead-list entry: candidate | status << 30

struct alignas(8) Pair {
    uint32_t d;   // previous DP row
    uint32_t p;   // fused time row of the stage's slot
};

// Workgroup barrier that orders LDS traffic only.  Global loads and stores stay in flight across
// it (the stage loop never communicates through global memory), which keeps the round trips of the
// back-pointer stores and of the next stage's table rows off the per-stage critical path.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// wavefront-scope ordering of LDS traffic: one wavefront's LDS operations execute in order, so
// this only keeps the compiler from moving accesses across the phases of a stage
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ uint32_t umax3(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t m = a > b ? a : b;
    return m > c ? m : c;
}

// Cross-lane steps on the DPP path of the vector unit, one instruction where a shuffle goes through LDS and
// back (a score takes some forty of them, half of them in a chain; k2_fast some thirty per candidate: 262,144
// candidates of 512 operators 4.69 -> 4.53 ms a step).
// Lanes a step has no source for read 0, so 0 has to be the neutral value.
template <int kCtrl, int kRows>
__device__ __forceinline__ uint32_t dpp0(uint32_t v) {
    return uint32_t(__builtin_amdgcn_update_dpp(0, int(v), kCtrl, kRows, 0xF, false));
}
constexpr int kRowShr = 0x110, kWaveShl1 = 0x130, kWaveShr1 = 0x138, kRowBcast15 = 0x142, kRowBcast31 = 0x143;

// lane l: f over lanes 0 .. l; lane 63 holds the whole wavefront's
template <typename F>
__device__ __forceinline__ uint32_t wave_scan(uint32_t v, F f) {
    v = f(v, dpp0<kRowShr + 1, 0xF>(v));
    v = f(v, dpp0<kRowShr + 2, 0xF>(v));
    v = f(v, dpp0<kRowShr + 4, 0xF>(v));
    v = f(v, dpp0<kRowShr + 8, 0xF>(v));
    v = f(v, dpp0<kRowBcast15, 0xA>(v));
    v = f(v, dpp0<kRowBcast31, 0xC>(v));
    return v;
}
template <typename F>
__device__ __forceinline__ uint32_t wave_all(uint32_t v, F f) {
    return uint32_t(__builtin_amdgcn_readlane(int(wave_scan(v, f)), 63));
}
__device__ __forceinline__ uint32_t sum2(uint32_t a, uint32_t b) { return a + b; }
__device__ __forceinline__ uint32_t max2(uint32_t a, uint32_t b) { return a > b ? a : b; }
// (the least value is the complement of the largest complement: 0 is neutral there)
__device__ __forceinline__ uint32_t wave_least(uint32_t v) { return ~wave_all(~v, max2); }
// sum of values from 0 to 2^40
__device__ __forceinline__ int64_t wave_sum(int64_t v) {
    const uint32_t lo = wave_all(uint32_t(v) & 0xFFFFFFu, sum2), hi = wave_all(uint32_t(v >> 24), sum2);
    return (int64_t(hi) << 24) + lo;
}

// A value every lane of the wave holds, moved to a scalar register.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uniform64(int64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
// A kernel argument in scalar registers of its own.  Arguments come in loads of up to sixteen registers, and where
// scalars run out such a load is kept, and fetched back, as a whole: sixteen moves from a vector register's lanes for
// one pointer (k2_fast: one stage in eight instructions).
template <typename T>
__device__ __forceinline__ T own_scalar(T v) {
    static_assert(sizeof(T) == 4 || sizeof(T) == 8, "one or two registers");
    T own;
    if constexpr (sizeof(T) == 8) asm("s_mov_b64 %0, %1" : "=s"(own) : "s"(v));
    else asm("s_mov_b32 %0, %1" : "=s"(own) : "s"(v));
    return own;
}
// A pointer out of an asm has no address space, and its loads would be flat ones, which count on the LDS counter as
// well: a stage's requests for the next one would be waited for with the first LDS read behind them (262,144 candidates
// of 512 operators, flat 4.50 ms a step, global 4.40; exact search, 65,536 of 160: 3.40, 3.33).
template <typename T>
__device__ __forceinline__ T *own_scalar(T *p) {
    using Global = __attribute__((address_space(1))) T;
    Global *own;
    asm("s_mov_b64 %0, %1" : "=s"(own) : "s"((Global *)p));
    return (T *)own;
}
template <typename T>
__device__ __forceinline__ const T *uniform_ptr(const T *p) {
    return reinterpret_cast<const T *>(uniform64(reinterpret_cast<int64_t>(p)));
}

// Per-slot constants of the candidate in flight, computed once per candidate so that the stage
// loop starts from LDS and never waits on a chain of dependent global loads.
// Rows are named by element offsets from the table bases, not by pointers: a pointer read back
// from LDS has no known address space and would turn every table access into a flat load.
struct alignas(16) StageConst {
    int64_t cap;            // tp * device memory of the slot's GPU type
    uint32_t p_row;         // element offset of the slot's fused time row in P32
    uint32_t cm_row_shift;  // element offset of the link's cut-time row in CM (low 27 bits) | log2 tp << 27
};
static_assert(sizeof(StageConst) == 16, "one 16-byte LDS read per stage");
static_assert(kFastCutTableLimit / 4 <= (size_t(1) << 27), "cut-table offsets must fit 27 bits");

__device__ __forceinline__ int band_lo(uint32_t w) { return int(w & 0xFFFFu); }
__device__ __forceinline__ int band_hi(uint32_t w) { return int(w >> 16); }

// How a stage time follows from a difference of its fused row.  `code`: log2 of the degree, or (kOdd: some
// degree is no power of two) the degree's index.  The multiply takes four issue slots where the shift takes
// one, so tables of powers of two keep the shift.
template <bool kOdd>
__device__ __forceinline__ TpDiv tp_div(const TablesDev &tb, uint32_t code) {
    if (kOdd) return tb.tp_div[code];
    return TpDiv{(1u << code) - 1u, 0u, int32_t(code)};
}
template <bool kOdd>
__device__ __forceinline__ uint32_t tp_quot(uint32_t x, const TpDiv &d) {       // x: difference + d.add
    return kOdd ? __umulhi(x, d.mul) >> d.shift : x >> d.shift;
}
template <bool kOdd>
__device__ __forceinline__ uint32_t tp_times(const TablesDev &tb, uint32_t x, uint32_t code) {   // x: below 2^32 / degree
    return kOdd ? x * uint32_t(tb.tp[code]) : x << code;
}
// The largest difference of a fused row whose time is at most t.
template <bool kOdd>
__device__ __forceinline__ uint32_t cap_reach(const TablesDev &tb, uint32_t t, uint32_t code) {
    const uint64_t far = kOdd ? uint64_t(t) * uint32_t(tb.tp[code]) : uint64_t(t) << code;
    return far < 0xFFFFFFFFull ? uint32_t(far) : 0xFFFFFFFFu;
}
template <bool kOdd>
__device__ __forceinline__ uint32_t tp_code(const TablesDev &tb, int k) {
    return uint32_t(kOdd ? k : tb.tp_shift[k]);
}

__device__ __forceinline__ int tp_index(const TablesDev &tb, int tp) {
    int k = -1;
    for (int q = 0; q < tb.n_tp; ++q)
        if (tb.tp[q] == tp) k = q;
    return k;
}

inline int fast_row_len(int L) { return (L + 1 + kPad + 7) / 8 * 8; }

inline size_t fast_lds_bytes(int L, int S_max) {
    size_t b = size_t(fast_row_len(L)) * 32 + size_t(S_max) * sizeof(StageConst) +
               size_t(S_max + 2) * 4 + size_t(S_max) * 3;
    return (b + 15) & ~size_t(15);
}

// Which candidate a wavefront takes next, in the kernels that work one per wavefront.  One counter for all
// would serialise them: an addition to a word that every XCD adds to takes 11.4 ns, whoever asks, so 16,384
// draws cost 190 us where the candidates themselves take 60.  Hence the first candidate of a wavefront is
// the one of its own number, and the others are dealt into 64 shares with a counter each, on a line of its
// own, which only workgroups of one XCD draw from (consecutive workgroups go to the 8 XCDs in turn): 64
// counters 14 ns apart each.  A wavefront whose share is used up reads all counters at once, a lane each,
// and goes on with the next share that has candidates left.  Ends: a counter only rises, and every round
// either returns a candidate or finds its share used up.
constexpr int kShares = 64;
constexpr int kShareInts = int(kTicketBytes / kShares / sizeof(int));
constexpr int kWideBands = 12;          // counter: candidates listed with wide bands
constexpr uint32_t kWideFlag = 1u << 30;    // on a live-list entry: the candidate is one of them, its bands are in `tight`
__device__ __forceinline__ int listed(int32_t entry) { return int(uint32_t(entry) & (kWideFlag - 1u)); }
constexpr int kTicketFast = 0, kTicketFastWide = 1, kTicketExact = 2, kTicketH1f1b = 3;   // word of a line
constexpr int kLongRows = 4;            // another: candidates whose narrowed bands are too wide for a wavefront's share
// Bands of listed candidates are narrowed (k2_narrow) where at least a quarter of the live ones are listed.
__device__ __forceinline__ bool bands_narrowed(const int *counts) { return 4 * int64_t(counts[kWideBands]) >= counts[0]; }
struct Draw {
    int *word;               // this kernel's word of the first share's line
    int n_items, n_waves, home;
    bool first;
    __device__ __forceinline__ Draw(int *tickets, int which, int items, int waves)
        : word(tickets + which), n_items(items), n_waves(waves), home(blockIdx.x & (kShares - 1)), first(true) {}
    // All lanes of the wavefront: the next item, or -1.
    __device__ __forceinline__ int next(int wave_id) {
        if (first) {
            first = false;
            if (wave_id < n_items) return wave_id;
        }
        if (n_items <= n_waves) return -1;
        for (;;) {
            // (a lane number of its own: the compiler must not join this branch with another on lane 0 around it,
            // or the other lanes reach the broadcast without lane 0's ticket)
            int lane = threadIdx.x & 63;
            asm volatile("" : "+v"(lane));
            int t = 0;
            if (lane == 0) t = atomicAdd(word + home * kShareInts, 1);
            wave_sync();
            const int n = n_waves + home + kShares * uniform(t);
            if (n < n_items) return n;
            const int seen = __hip_atomic_load(word + lane * kShareInts, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const unsigned long long left = __ballot(n_waves + lane + kShares * seen < n_items);
            if (left == 0) return -1;
            const int from = (home + 1) & (kShares - 1);
            const unsigned long long turned = from == 0 ? left : (left >> from) | (left << (64 - from));
            home = uniform((from + __ffsll((long long)turned) - 1) & (kShares - 1));
        }
    }
};

// Back-pointer slice of one wavefront (k2_fast) or workgroup (the kernels built on it): a 16-bit
// entry per DP cell, followed by the one-byte entries k2_fast uses for cells whose back-pointers
// leave LDS (distance to the previous cut; the 16-bit entry holds the cut itself when the distance
// does not fit a byte).
inline size_t fast_arg_u16_bytes(int L, int S_max) {
    size_t b = size_t(S_max) * fast_row_len(L) * sizeof(uint16_t);
    return (b + 255) & ~size_t(255);
}
inline size_t fast_arg_per_group(int L, int S_max) {
    size_t b = size_t(S_max) * fast_row_len(L);
    return fast_arg_u16_bytes(L, S_max) + ((b + 255) & ~size_t(255));
}

// Rows of the feasibility index (see k2_fast.hip): one per in-flight count n = 1 .. n_max, GPU type and
// degree index.  Two tables of that many rows, one after the other: entry i of a row of the first
// is the lowest previous cut j such that operators [j, i) fit, entry j of a row of the second the
// highest cut i such that they do.
inline int lo_n_max(int L, int S_max, int M) {
    int n = S_max < M ? S_max : M;
    return n < L ? n : L;
}
inline size_t lo_pitch(int L) { return (size_t(L) + 1 + 31) & ~size_t(31); }
inline size_t lo_table_bytes(int L, int S_max, int M, int T, int n_tp) {
    return 2 * size_t(lo_n_max(L, S_max, M)) * size_t(T) * size_t(n_tp) * lo_pitch(L) * sizeof(uint16_t);
}

// Workspace: counters | tickets | live list [C] | dead list [C] | bands [C][S_max+1] | feasibility index |
// list of wide candidates [C] | their bands under a cap [C][S_max+1] (both only where bands are narrowed) |
// back-pointer slices (one per resident wavefront of k2_fast, one per workgroup of the other kernels).
struct FastWorkspace {
    int *counts;
    int *tickets;            // [kShares] lines
    int32_t *live_list;
    uint32_t *dead_list;
    uint32_t *bands;
    uint16_t *lo_tab;
    int32_t *wide_list;      // [C] candidates with wide memory bands
    uint32_t *tight;         // [C][S_max+1] their bands under a cap
    unsigned char *arg;
    size_t total;
};

struct FastShape {
    int L, S_max, C, M, T, n_tp;
    bool narrow;             // bands under a cap where memory bands are wide (k2_narrow.hip, exact search)
};

inline FastShape fast_shape(const TablesDev &tb, const CandDev &cd, bool narrow) {
    return FastShape{tb.L, cd.S_max, cd.C, tb.M, tb.T, tb.n_tp, narrow};
}

inline FastWorkspace carve(void *ws, const FastShape &f, int n_slices) {
    auto up = [](size_t x) { return (x + 255) & ~size_t(255); };
    unsigned char *base = static_cast<unsigned char *>(ws);
    FastWorkspace w;
    size_t off = 0;
    w.counts = reinterpret_cast<int *>(base + off); off += 256;
    w.tickets = reinterpret_cast<int *>(base + off); off += kTicketBytes;
    w.live_list = reinterpret_cast<int32_t *>(base + off); off += up(size_t(f.C) * 4);
    w.dead_list = reinterpret_cast<uint32_t *>(base + off); off += up(size_t(f.C) * 4);
    w.bands = reinterpret_cast<uint32_t *>(base + off); off += up(size_t(f.C) * (f.S_max + 1) * 4);
    w.lo_tab = reinterpret_cast<uint16_t *>(base + off); off += up(lo_table_bytes(f.L, f.S_max, f.M, f.T, f.n_tp));
    w.wide_list = nullptr;
    w.tight = nullptr;
    if (f.narrow) {
        w.wide_list = reinterpret_cast<int32_t *>(base + off); off += up(size_t(f.C) * 4);
        w.tight = reinterpret_cast<uint32_t *>(base + off); off += up(size_t(f.C) * (f.S_max + 1) * 4);
    }
    w.arg = base + off; off += size_t(n_slices) * fast_arg_per_group(f.L, f.S_max);
    w.total = off;
    return w;
}

}  // namespace fastdp
}  // namespace harp
