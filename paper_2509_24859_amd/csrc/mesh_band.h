// Band-limited passes of the submesh planner on the 32-bit rows (paper section 5.2.3, eq. dp_general
// with its device index).  Device functions called by all threads of a workgroup, one ordering of
// device groups at a time; k2_mesh.hip drives them.
//
// The state is (s, i, d): s stages hold the first i operators and use exactly the first d devices of
// the ordering.  Under a cap t on every stage and transfer time, and the memory constraint, the cuts
// i that matter for a given (s, d) form a narrow range [B, F]:
//   F[s+1][d'] = max over degrees q, d = d' - tp_q inside the group of d', of
//                the highest cut that a stage started at F[s][d] reaches with time <= t, in memory,
//                lowered to a cut whose transfer time is at most t;
//   B[s][d]    = the same from the end: the lowest cut from which stage s reaches B[s+1][d + tp_q].
// Both reaches never decrease with the cut they start from, so F bounds every cut some plan under t
// can have after s stages on d devices, and B every cut from which one can be completed; cells
// outside the range are on no plan under t.  Leaving them out changes no cell on such a plan: its
// value, and the lowest previous cut that attains it, come from cells on plans under t as well.
// For the capped (least-sum) and H-1F1B passes t is the cap (H-1F1B's counts are never below the
// classic ones the ranges are worked out with).  For the min-max pass any t >= the optimum will do: a
// guess from the groups' speeds (guess), and where F does not reach (S, L, all devices) under it, a t little
// above the smallest at which it does, found by a search over chains (bracket).  A
// chain can leave a stage without operators, so where some device's memory holds no operator alone the
// pass may find no plan under that t; it is then repeated under a higher one, and at last
// without a cap on the times.  On orderings of 82 operators and 64 devices the ranges hold between
// 0.1% and 25% of the (i, d) cells, the wide ones where a slow link decides the bottleneck.
//
// Two chains are worked at once, F and B of one t or F of two, a lane per column d and a wavefront per 64 of
// them.  A pass keeps its value rows in LDS (cells of a row packed one column after the other), all of
// them where they fit, else the last two with every row written to the workgroup's slice of the workspace,
// and where not even two fit it works from the slice.  Only the H-1F1B pass keeps back-pointers: the plans of the
// others are found from the value rows, per stage one step for all degrees and cuts at once.  That leaves a minimum
// per transition (a subtraction, a shift, a three-way maximum) where back-pointers cost a 64-bit key.  Rows of the fused stage times sit in LDS, one set per
// distinct (GPU type, own link) of the ordering; memory limits come from the feasibility index
// (k2_index), one 16-bit load per cell and degree.
#pragma once

#include "fast_common.h"
#include "harp_internal.h"
#include "plan_common.h"

namespace harp {
namespace meshband {

using fastdp::lds_barrier;
using fastdp::uniform;
using fastdp::wave_sync;

constexpr uint32_t kNoCut = 0xFFFFu;
constexpr uint32_t kInfSum = 0x80000000u;        // least sums stay below this (largest_cap)
constexpr uint32_t kTopCap = 0x7FFFFFFFu;        // no time on these tables is larger
constexpr int kRowPad = 4;                       // a window of four entries may overrun a row
constexpr int kReachRun = 8;                     // entries of a reach table that a thread works at most
constexpr int kTeams = 2;                        // chains worked at once

// LDS layout of a launch (byte offsets into dynamic LDS) and its capacities.
struct BandShape {
    int W, NW;                   // cuts (L + 1), 64-bit words of a mask of cuts
    int cols;                    // columns: devices + 1
    int K_cap, set_cap;          // groups of an ordering, sets of time rows
    int S_cap;                   // min(S_max, L)
    int idx_pitch;               // feasibility index
    uint32_t o_offs, o_order, o_type, o_row_at, o_group_at, o_cut_at, o_use, o_mem, o_ok, o_col, o_small, o_prow,
        o_set_of, total;
};

constexpr int kMaxDevices = 2048;                // columns sit in LDS, 24 bytes each
// LDS of a CU, less what the band kernels hold statically (272 to 288 bytes: the ordering drawn, a score, and the
// scratch of __syncthreads_or), which counts against the same limit
constexpr size_t kBandLds = (size_t(160) << 10) - 1024;
// forms of a launch: what the value rows hold
constexpr int kFormMinMax = 0, kFormSum = 1, kFormH1 = 2, kFormSweep = 3;
bool band_shape(const TablesDev &tb, int S_max, int G_max, int64_t total_devices, int form, size_t budget,
                BandShape &sh);

// What the band kernels of a launch share: LDS shape, feasibility index, slices, and counters [0] ticket,
// [1] orderings handed over to the whole-table kernels, [2] .. tickets of those.
struct BandArgs {
    BandShape sh;
    const uint16_t *lo_tab, *hi_tab;
    unsigned char *slices;
    size_t per_group;
    int *counters;
    int *redo;
};

// Workspace of a launch: counters | orderings handed over [C] | feasibility index | slices.
struct MeshWorkspace {
    int *counters, *redo;
    uint16_t *index;
    size_t index_bytes;
    unsigned char *slices;
    size_t before_slices;
};
MeshWorkspace mesh_carve(const TablesDev &tb, int S_max, int C, void *ws);
// Threads and LDS of the band kernels for a batch, given how many workgroups have a slice; false when the batch
// is for the whole-table kernels.
bool band_launch(const TablesDev &tb, const OrdDev &od, int64_t total_devices, int form, int n_cu, int n_groups,
                 int &threads, BandShape &sh);

// Per workgroup, in the workspace slice: F, B [S_cap + 1][cols] uint16, first cell index less lowest
// cut [S_cap + 1][cols] int32, value rows (uint32) or, H-1F1B, back-pointers (uint16).
struct BandSlice {
    uint16_t *F, *B;
    int32_t *off;
    uint32_t *hist;
    uint32_t *spare_h;           // two rows of sums and two of counts, for H-1F1B rows that do not fit in LDS
    uint16_t *spare_n;
    int64_t row;                 // cells of a spare row
};
__device__ __forceinline__ BandSlice band_slice(unsigned char *mine, const BandShape &sh) {
    BandSlice b;
    const size_t n = size_t(sh.S_cap + 1) * sh.cols;
    b.off = reinterpret_cast<int32_t *>(mine);
    b.F = reinterpret_cast<uint16_t *>(b.off + n);
    b.B = b.F + n;
    b.row = int64_t(sh.cols) * sh.W + kRowPad;
    b.spare_h = reinterpret_cast<uint32_t *>(mine + ((n * 8 + 255) & ~size_t(255)));
    b.spare_n = reinterpret_cast<uint16_t *>(b.spare_h + 2 * b.row);
    b.hist = b.spare_h + 3 * b.row;
    return b;
}
inline size_t band_slice_bytes(int L, int S_max, int64_t total_devices) {
    const size_t S_cap = size_t(S_max < L ? S_max : L), cols = size_t(total_devices + 1);
    const size_t row = cols * size_t(L + 1) + kRowPad;
    return (((S_cap + 1) * cols * 8 + 255) & ~size_t(255)) + (((S_cap + 4) * row * 4 + 255) & ~size_t(255));
}

struct Band {
    static constexpr bool kChoosesSlicing = true, kGuesses = true, kSpreads = false;
    static constexpr int kMaxClimb = 8;       // see k2_sweep.hip
    const TablesDev &tb;
    const BandShape &sh;
    const uint16_t *lo_tab, *hi_tab;
    BandSlice sl;
    // LDS
    int32_t *offs;               // [K + 1] first device offset of every group
    uint16_t *order, *type, *group_at;
    uint32_t *prow_at, *index_at;   // [K] first entry of a group's time rows (and reach rows), of its type's index rows
    uint32_t *link_at;           // [2 K] first entry of a link's row in the cut table: K links inside groups, K - 1 to the next
    uint32_t *cut_at;            // [cols] the same for the link behind a stage that ends at device d
    uint32_t *use;               // [sets] largest group of a set: its degrees up to that size are candidate stages
    uint32_t *prow;              // [sets][n_tp][W]
    uint16_t *reach;             // [2][sets][n_tp][W] reach of a stage under a cap
    int64_t *mem;                // PP [W], PS [W] (H-1F1B form)
    uint16_t *chain;             // [kTeams][2][cols + 1], where the columns of the passes go
    unsigned long long *ok;      // [kTeams][2 K][NW]
    uint2 *col;                  // [2][cols] lowest and highest cut of a column | index of its first cell less its lowest cut
    uint32_t *col_min;           // [2][cols] least value of a column (min-max form)
    int32_t *tot, *base;         // [S_cap + 1] cells of a row, first cell of a row in hist
    int32_t *cuts;               // [S_cap + 1]
    int32_t *slot_first;         // [S_cap]
    int32_t *warmup;             // [S_cap] counts of the plan (H-1F1B form)
    uint16_t *slot_g;            // [S_cap]
    uint8_t *slot_k;             // [S_cap]
    uint32_t *scal;              // [8]
    uint16_t *set_of;            // [K] first group with the same time rows, while an ordering is loaded: in the room of the rows
    uint32_t *rows;              // rows of a pass, [n][pitch], behind the sets the ordering has
    uint16_t *counts;            // [2][pitch] (H-1F1B form)
    uint16_t *map;               // [pitch] column of a cell
    uint32_t room;               // bytes for rows, counts and map
    int pitch;                   // cells of a row that fit, and a window
    bool ranges_in_lds;          // the last prepared cap: F, B and off sit in LDS, not in the slice
    bool whole;                  // the last pass: all its rows are in LDS, none in the slice
    uint32_t *rows_all, *ring;   // rows of the whole pass; rows it keeps the last ones of
    uint32_t pass_room;          // what the ranges leave of the room
    uint32_t *pass_at;
    bool chains_in_lds;
    int all_cells;               // of all rows of the last prepared cap
    bool reached;                // the last prepared cap: its chains get from end to end
    bool unlikely;               // no plan is expected under the first cap: the next pass is taken for one that found none
    int most_cells;              // of a row of the last prepared cap
    int map_shift;               // load_columns
    int nthreads, wave;
    int K, S, D, L, n_sets;
    int least_cut;               // the cut behind the operator of least output (operators but the last)
    int run_len, runs;           // entries of a reach table that a thread works, such runs in a row of it
    uint32_t runs_inv;           // x / runs is the high half of x * runs_inv for x below 2^32 / runs (runs above 1)
    bool keys_fit;               // sums times a degree fit 32 bits under the cap of the next pass for the least sum
    int64_t count_cap;           // the cap H-1F1B's counts are worked out with: the pass's own, or above any time

    __device__ __forceinline__ Band(const TablesDev &t, const BandShape &s, unsigned char *lds, const uint16_t *lo,
                                    const uint16_t *hi, const BandSlice &slice)
        : tb(t), sh(s), lo_tab(lo), hi_tab(hi), sl(slice) {
        offs = reinterpret_cast<int32_t *>(lds + sh.o_offs);
        order = reinterpret_cast<uint16_t *>(lds + sh.o_order);
        type = reinterpret_cast<uint16_t *>(lds + sh.o_type);
        prow_at = reinterpret_cast<uint32_t *>(lds + sh.o_row_at);
        index_at = prow_at + sh.K_cap;
        link_at = index_at + sh.K_cap;
        cut_at = reinterpret_cast<uint32_t *>(lds + sh.o_cut_at);
        group_at = reinterpret_cast<uint16_t *>(lds + sh.o_group_at);
        use = reinterpret_cast<uint32_t *>(lds + sh.o_use);
        prow = reinterpret_cast<uint32_t *>(lds + sh.o_prow);
        set_of = reinterpret_cast<uint16_t *>(lds + sh.o_set_of);
        mem = reinterpret_cast<int64_t *>(lds + sh.o_mem);
        chain = reinterpret_cast<uint16_t *>(lds + sh.o_col);
        ok = reinterpret_cast<unsigned long long *>(lds + sh.o_ok);
        col = reinterpret_cast<uint2 *>(lds + sh.o_col);
        col_min = reinterpret_cast<uint32_t *>(col + 2 * sh.cols);
        scal = reinterpret_cast<uint32_t *>(lds + sh.o_small);
        tot = reinterpret_cast<int32_t *>(scal + 8);
        base = tot + (sh.S_cap + 1);
        cuts = base + (sh.S_cap + 1);
        slot_first = cuts + (sh.S_cap + 1);
        warmup = slot_first + sh.S_cap;
        slot_g = reinterpret_cast<uint16_t *>(warmup + sh.S_cap);
        slot_k = reinterpret_cast<uint8_t *>(slot_g + sh.S_cap);
        find_room(0);
        nthreads = blockDim.x; wave = uniform(int(threadIdx.x) >> 6);
        L = tb.L;
        K = S = D = n_sets = 0;
        pitch = most_cells = map_shift = 0;
        reached = unlikely = false;
        run_len = runs = 1;
        runs_inv = 0;
        keys_fit = true;
        ranges_in_lds = chains_in_lds = whole = false;
        all_cells = 0;
        least_cut = 1;
        count_cap = 0;
    }

    // What the sets of an ordering leave of the LDS holds the rows of its passes: a fixed share for the most sets an
    // ordering may have, cut for the widest form of a row, left values of 160 operators and 128 devices room for 2,900
    // cells where 12,000 fit (256 orderings, exact form: two of three least-sum passes worked from the workspace).
    static constexpr int kValueBytes = 10, kCountBytes = 14;       // of a cell: two rows of values (and of counts), and the map
    __device__ __forceinline__ int keys_bytes() const { return 4 * (1 + tb.n_tp) + 2; }
    __device__ __forceinline__ void find_room(int sets) {
        const uint32_t per_table = uint32_t(sets) * uint32_t(tb.n_tp) * uint32_t(sh.W);      // entries
        reach = reinterpret_cast<uint16_t *>(prow + per_table + 4);                          // (a window may overrun the last row)
        const uint32_t from = (sh.o_prow + 16u + per_table * 8u + 15u) & ~15u;
        rows = prow + (from - sh.o_prow) / 4u;
        room = sh.total - from - 256u;                     // (256: what windows may overrun)
    }

    // The thread's index, new to the compiler at every use: what a phase derives from it (LDS addresses,
    // mostly) must not be hoisted out of the phase and kept in registers through all the others.
    static __device__ __forceinline__ int thread_id() {
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));
        return t;
    }

    // All threads, once per kernel: the cheapest cut of the sequence on any link.
    __device__ __forceinline__ void find_least_cut() {
        const int tid = thread_id();
        const int lane = tid & 63;
        unsigned long long key = ~0ull;
        for (int i = 1 + tid; i < L; i += nthreads) {
            const unsigned long long a = (unsigned long long)tb.act_bytes[i - 1];
            if (a < key) key = a;
        }
#pragma unroll
        for (int x = 32; x >= 1; x >>= 1) {
            const unsigned long long o = __shfl_xor(key, x, 64);
            key = o < key ? o : key;
        }
        unsigned long long *part = ok;                     // free until the first ordering
        if (lane == 0) part[wave & 1] = ~0ull;
        __syncthreads();
        if (lane == 0) atomicMin(&part[0], key);
        __syncthreads();
        key = part[0];
        if (tid == 0) scal[0] = 1;
        __syncthreads();
        for (int i = 1 + tid; i < L; i += nthreads)
            if ((unsigned long long)tb.act_bytes[i - 1] == key) scal[0] = uint32_t(i);      // any of them
        __syncthreads();
        least_cut = int(scal[0]);
        __syncthreads();
    }

    __device__ __forceinline__ int shift_of(int q) const { return tb.tp_shift[q]; }
    __device__ __forceinline__ int tp_of(int q) const { return tb.tp[q]; }
    __device__ __forceinline__ int in_flight(int s) const { return (S - s) < tb.M ? (S - s) : tb.M; }
    // feasibility index of a stage with n micro-batches in flight: entry of degree q of group k at
    // index_n(n) + index_at[k] + q * idx_pitch (the index and the cut table have fewer than 2^28 entries)
    __device__ __forceinline__ uint32_t index_n(int n) const {
        return uint32_t(n - 1) * uint32_t(tb.T) * uint32_t(tb.n_tp) * uint32_t(sh.idx_pitch);
    }
    // link behind a stage that ends at device d (1 <= d < D) as a mask index
    __device__ __forceinline__ int link_of(int d) const {
        const int k = group_at[d - 1];
        return d == offs[k + 1] && k + 1 < K ? K + k : k;
    }

    // The ordering og[0 .. K): groups in range, distinct; offsets; time rows.  Returns 0, or 1 when the
    // ordering is malformed (bad), 2 when no plan can exist, 3 when it does not fit this launch's LDS.
    __device__ __forceinline__ int load(int S_, int K_, const int32_t *og, int S_max, int G_max) {
        const int tid = thread_id();
        S = uniform(S_); K = uniform(K_);
        // (more groups than the problem has cannot be distinct)
        int bad = (S < 1 || S > S_max || K < 1 || K > G_max || K > sh.K_cap) ? 1 : 0;
        if (!bad)
            for (int k = tid; k < K; k += nthreads) {
                const int g = og[k];
                if (g < 0 || g >= tb.G) { bad = 1; continue; }
                for (int q = 0; q < k; ++q)
                    if (og[q] == g) bad = 1;
                order[k] = uint16_t(g);
                type[k] = uint16_t(tb.group_type[g]);
            }
        if (__syncthreads_or(bad)) return 1;
        if (tid == 0) {
            int64_t o = 0;
            offs[0] = 0;
            for (int k = 0; k < K; ++k) { o += tb.group_ndev[order[k]]; offs[k + 1] = int32_t(o); }
        }
        // the set of time rows of a group: that of the first group with its type and own link
        for (int k = tid; k < K; k += nthreads) {
            const int g = order[k];
            const int64_t link = tb.bw[int64_t(g) * tb.G + g];
            int q = 0;
            while (q < k && !(type[q] == type[k] && tb.bw[int64_t(order[q]) * tb.G + order[q]] == link)) ++q;
            set_of[k] = uint16_t(q);
            index_at[k] = uint32_t(type[k]) * uint32_t(tb.n_tp) * uint32_t(sh.idx_pitch);
            link_at[k] = uint32_t(g * tb.G + g) * uint32_t(tb.pitch32);
            if (k + 1 < K) link_at[K + k] = uint32_t(g * tb.G + order[k + 1]) * uint32_t(tb.pitch32);
        }
        __syncthreads();
        D = uniform(offs[K]);
        if (S > L || S < K || S > D) return 2;
        n_sets = 0;
        for (int k = 0; k < K; ++k) n_sets += set_of[k] == k ? 1 : 0;
        n_sets = uniform(n_sets);
        if (n_sets > sh.set_cap) return 3;
        find_room(n_sets);
        run_len = (n_sets * tb.n_tp * sh.W + nthreads - 1) / nthreads;
        run_len = uniform(run_len < kReachRun ? run_len : kReachRun);
        runs = (sh.W + run_len - 1) / run_len;
        runs_inv = uint32_t(uniform(int(0xFFFFFFFFu / uint32_t(runs) + 1u)));
        map_shift = 0;
        while (map_shift < 3 && (D << (map_shift + 1)) <= nthreads) ++map_shift;
        for (int k = 0, set = 0; k < K; ++k) {
            if (set_of[k] != k) continue;
            const uint32_t *from = tb.P32 + int64_t(order[k]) * tb.n_tp * tb.pitch32;
            uint32_t *to = prow + set * tb.n_tp * sh.W;
            for (int q = 0; q < tb.n_tp; ++q)
                for (int i = tid; i <= L; i += nthreads) to[q * sh.W + i] = from[int64_t(q) * tb.pitch32 + i];
            ++set;
        }
        for (int k = 0; k < K; ++k)
            for (int d = offs[k] + tid; d < offs[k + 1]; d += nthreads) group_at[d] = uint16_t(k);
        // sets are numbered in the order of their first groups
        for (int k = tid; k < K; k += nthreads) {
            uint32_t set = 0;
            for (int q = 0; q < set_of[k]; ++q) set += set_of[q] == q ? 1u : 0u;
            prow_at[k] = set * uint32_t(tb.n_tp) * uint32_t(sh.W);
        }
        for (int x = tid; x < n_sets; x += nthreads) use[x] = 0;
        __syncthreads();
        for (int k = tid; k < K; k += nthreads)
            atomicMax(&use[prow_at[k] / uint32_t(tb.n_tp * sh.W)], uint32_t(offs[k + 1] - offs[k]));
        for (int d = tid; d <= D; d += nthreads) cut_at[d] = link_at[d == 0 ? 0 : d == D ? K - 1 : link_of(d)];
        __syncthreads();
        return 0;
    }
    __device__ __forceinline__ const uint32_t *time_row(int k) const { return prow + prow_at[k]; }   // degree q at q * W
    __device__ __forceinline__ uint16_t *reach_row(int side, int k) const {
        return reach + side * n_sets * tb.n_tp * sh.W + prow_at[k];
    }
    __device__ __forceinline__ unsigned long long *masks(int team) const { return ok + size_t(team) * 2 * sh.K_cap * sh.NW; }

    // All threads: cuts whose transfer time is at most t[w], one mask per link, for n values of t at once
    // (the cut tables come from L2: four words are requested before the first is used).
    __device__ __forceinline__ void cut_masks(int n, uint32_t ta, uint32_t tb_) {
        const int lane = thread_id() & 63;
        const int words = (2 * K - 1) * sh.NW, step = nthreads >> 6;
        unsigned long long *ma = masks(0), *mb = masks(n - 1);
        for (int x0 = wave; x0 < words; x0 += 4 * step) {
            uint32_t cut[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int x = x0 + u * step, l = x / sh.NW, i = (x - l * sh.NW) * 64 + lane;
                cut[u] = 0xFFFFFFFFu;
                if (x < words && i >= 1 && i <= L) cut[u] = tb.CM[link_at[l] + uint32_t(i)];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int x = x0 + u * step;
                const unsigned long long a = __ballot(cut[u] <= ta), b = __ballot(cut[u] <= tb_);
                if (x < words && lane == 0) {
                    ma[x] = a;
                    if (n > 1) mb[x] = b;
                }
            }
        }
    }
    // All threads: how far a stage gets under t on every (set, degree), into table `side`.  Upwards: entry j = the
    // highest cut i with time(j, i) <= t; downwards: entry i = the lowest cut j with time(j, i) <= t.  Neither falls from
    // one entry to the next, so a thread finds the first of a run of entries by bisection and goes on from there:
    // a cut or so per entry, where a bisection each takes seven or eight steps (4,096 orderings of 82 operators and 64
    // devices: of an ordering's 145 us the tables took 31, now 19).  Runs are as long as the workgroup's threads leave entries
    // to each, up to kReachRun: a run is a chain of LDS reads, and with runs of eight for 104 entries (12 operators) the
    // tables of a cap took 5 us, 1.5 with one entry a thread.
    template <bool kUp>
    __device__ __forceinline__ void reach_table(uint32_t t, int side) {
        uint16_t *to = reach + side * n_sets * tb.n_tp * sh.W;
        const int top_step = 1 << (31 - __clz(L));
        for (int x = thread_id(); x < n_sets * tb.n_tp * runs; x += nthreads) {
            const int r = runs == 1 ? x : int(__umulhi(uint32_t(x), runs_inv)), e0 = (x - r * runs) * run_len, end = e0 + run_len < sh.W ? e0 + run_len : sh.W;
            const uint64_t far = uint64_t(t) * uint32_t(tb.tp[r % tb.n_tp]);
            const uint32_t reach_of = far > 0xFFFFFFFFull ? 0xFFFFFFFFu : uint32_t(far);
            const uint32_t *p = prow + r * sh.W;
            uint16_t *out = to + r * sh.W;
            int pos = e0;
            for (int e = e0; e < end; ++e) {
                const uint32_t pe = p[e];
                const uint32_t target = kUp ? (pe > 0xFFFFFFFFu - reach_of ? 0xFFFFFFFFu : pe + reach_of) : (pe > reach_of ? pe - reach_of : 0u);
                if (e == e0) {
                    for (int step = top_step; step > 0; step >>= 1) {
                        const int nx = kUp ? pos + step : pos - step;
                        if (kUp) pos = nx <= L && p[nx <= L ? nx : L] <= target ? nx : pos;
                        else pos = nx >= 0 && p[nx >= 0 ? nx : 0] >= target ? nx : pos;
                    }
                } else if (kUp) {
                    while (pos < L && p[pos + 1] <= target) ++pos;
                } else {
                    while (p[pos] < target) ++pos;                     // (p[e] is no less)
                }
                out[e] = uint16_t(pos);
            }
        }
    }
    // highest cut <= i in a mask, -1 when there is none; lowest cut >= i, > L when there is none
    __device__ __forceinline__ int mask_down(const unsigned long long *m, int i) const {
        int w = i >> 6;
        unsigned long long b = m[w] & (~0ull >> (63 - (i & 63)));
        while (b == 0 && w > 0) b = m[--w];
        return b == 0 ? -1 : w * 64 + 63 - __clzll((long long)b);
    }
    __device__ __forceinline__ int mask_up(const unsigned long long *m, int i) const {
        int w = i >> 6;
        unsigned long long b = m[w] & (~0ull << (i & 63));
        while (b == 0 && w + 1 < sh.NW) b = m[++w];
        return b == 0 ? L + 1 : w * 64 + __ffsll((long long)b) - 1;
    }

    // A chain step, a lane per column: F of the columns d after stage s (forwards, from the upward reach table),
    // or B of those in front of it (backwards).  What a column's lane needs of its group does not change from stage to
    // stage (chain_lane).
    struct ChainLane { int d, edge; uint32_t index, far, link; };
    template <bool kBack>
    __device__ __forceinline__ ChainLane chain_lane(int c) const {
        ChainLane l;
        l.d = c * 64 + (thread_id() & 63) + (kBack ? 0 : 1);       // forwards columns 1 .. D, backwards 0 .. D - 1
        const int stage_on = kBack ? (l.d < D ? l.d : D - 1) : (l.d <= D ? l.d : D) - 1, k = group_at[stage_on];
        // (a lane behind column D has no column to come from: its offsets would lie behind the row, and what it read there
        // would be taken for a cut of the index in memory)
        l.edge = kBack ? offs[k + 1] : l.d <= D ? offs[k] : INT32_MAX;
        l.index = index_at[k];
        l.far = prow_at[k];
        const int cut_on = kBack ? stage_on : stage_on + 1;
        l.link = uint32_t(cut_on > 0 ? link_of(cut_on) : 0) * uint32_t(sh.NW);
        return l;
    }
    template <bool kBack>
    __device__ __forceinline__ void chain_step(const ChainLane &l, int c, int s, int side, const unsigned long long *m,
                                               const uint16_t *from, uint16_t *to, bool keep) const {
        const uint16_t *far = reach + side * n_sets * tb.n_tp * sh.W;
        const uint16_t *fits = (kBack ? lo_tab : hi_tab) + index_n(in_flight(s));
        int best = kBack ? INT32_MAX : -1;
        for (int q0 = 0; q0 < tb.n_tp; q0 += 4) {
            // (no branches around the loads: the four degrees' are in flight together)
            uint32_t v[4];
            int a[4], b[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int q = q0 + u < tb.n_tp ? q0 + u : tb.n_tp - 1;
                const int d = kBack ? l.d + tp_of(q) : l.d - tp_of(q);
                v[u] = from[(kBack ? d <= l.edge : d >= l.edge) ? d : sh.cols];      // [cols]: no cut
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int q = q0 + u < tb.n_tp ? q0 + u : tb.n_tp - 1;
                const uint32_t e = v[u] != kNoCut ? v[u] : 0u;
                a[u] = far[l.far + uint32_t(q * sh.W) + e];
                b[u] = fits[l.index + uint32_t(q * sh.idx_pitch) + e];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (kBack) {
                    const int j = a[u] > b[u] ? a[u] : b[u];
                    best = v[u] != kNoCut && j < best ? j : best;
                } else {
                    const int i = a[u] < b[u] ? a[u] : b[u];
                    best = v[u] != kNoCut && i > best ? i : best;
                }
            }
        }
        if (kBack) {
            const int d_hi = s == 0 ? 0 : D - (S - s);
            best = best > s ? best : s;
            if (s > 0 && best <= L) best = mask_up(m + l.link, best);
            if (best > L - (S - s) || (s == 0 && best != 0) || l.d > d_hi) best = -1;
        } else {
            const int top = L - (S - 1 - s), d_hi = D - (S - 1 - s);
            const bool last = s == S - 1;
            best = best < top ? best : top;
            if (best >= 0 && !last) best = mask_down(m + l.link, best);
            if (best < s + 1 || l.d > d_hi || (last && l.d != D)) best = -1;
        }
        const int outside = kBack ? D : 0;                         // the column that only the first row has
        const uint32_t row = uint32_t(kBack ? s : s + 1) * uint32_t(sh.cols);
        const uint16_t v = best < 0 ? uint16_t(kNoCut) : uint16_t(best);
        if (kBack ? l.d < D : l.d <= D) {
            to[l.d] = v;
            if (keep) put_range<kBack>(row + l.d, v);
        }
        if (c == 0 && (threadIdx.x & 63) == 0) {
            to[outside] = uint16_t(kNoCut);
            if (keep) put_range<kBack>(row + outside, uint16_t(kNoCut));
        }
    }
    template <bool kBack>
    __device__ __forceinline__ void put_range(uint32_t at, uint16_t v) const {
        if (chains_in_lds) reinterpret_cast<uint16_t *>(rows)[at + (kBack ? n_ranges() : 0u)] = v;
        else if (kBack) sl.B[at] = v;
        else sl.F[at] = v;
    }
    // Ranges in LDS, in front of the rows: F, B, off, of n_ranges entries each.  (Kept as pointers beside those of the slice
    // they would be chosen between by name, and the whole object stays in memory.)
    __device__ __forceinline__ uint32_t n_ranges() const { return uint32_t(S + 1) * uint32_t(sh.cols); }
    // All threads: two chains at once, the one of team 0 forwards, that of team 1 forwards or (kBack) backwards, a
    // wavefront for every 64 columns where there are as many, and a barrier per stage that waits for LDS only.  Backwards: F and
    // B are kept, in the room of the rows where they fit, else in the slice.  Verdict: (S, D) reaches L, or (0, 0) is reached.
    template <bool kBack>
    __device__ __forceinline__ void run_chains(bool &good0, bool &good1) {
        const int chunks = (D + 63) >> 6, half = nthreads >> 7, waves = chunks < half ? chunks : half;
        const int team = wave < waves ? 0 : wave < 2 * waves ? 1 : 2, first = team == 1 ? wave - waves : wave;
        const int pitch16 = sh.cols + 1;
        uint16_t *buf = chain + (team == 1 ? 2 : 0) * pitch16;
        for (int x = thread_id(); x < 4 * pitch16; x += nthreads) {
            const int b = x / pitch16, d = x - b * pitch16;
            uint16_t v = uint16_t(kNoCut);
            if (kBack && b == 2) v = d == D ? uint16_t(L) : v;
            else if (b == 0 || b == 2) v = d == 0 ? uint16_t(0) : v;
            chain[x] = v;
            if (kBack && b == 0 && d <= D) put_range<false>(uint32_t(d), v);
            if (kBack && b == 2 && d <= D) put_range<true>(uint32_t(S * sh.cols + d), v);
        }
        __syncthreads();
        const bool back = kBack && team == 1;
        const unsigned long long *m = masks(kBack ? 0 : team == 1 ? 1 : 0);
        ChainLane l = back ? chain_lane<true>(first) : chain_lane<false>(first);
        for (int n = 0; n < S; ++n) {
            const uint16_t *from = buf + (n & 1) * pitch16;
            uint16_t *to = buf + ((n & 1) ^ 1) * pitch16;
            if (team < 2)
                for (int c = first; c < chunks; c += waves) {
                    if (back) {
                        if (chunks > waves) l = chain_lane<true>(c);
                        chain_step<true>(l, c, S - 1 - n, 1, m, from, to, true);
                    } else {
                        if (chunks > waves) l = chain_lane<false>(c);
                        chain_step<false>(l, c, n, team, m, from, to, kBack);
                    }
                }
            lds_barrier();
        }
        if (kBack && !chains_in_lds) __syncthreads();
        const int at = (S & 1) * pitch16;
        good0 = uniform(chain[at + D]) == L;
        good1 = kBack ? uniform(chain[2 * pitch16 + at]) == 0 : uniform(chain[2 * pitch16 + at + D]) == L;
    }

    // All threads: the ranges under t, cell numbering of every row.  False: no plan under t.
    __device__ __forceinline__ bool prepare(uint32_t t) {
        const int tid = thread_id();
        const int lane = tid & 63;
        __syncthreads();                                   // earlier use of rows, chains and ranges is over
        cut_masks(1, t, t);
        reach_table<true>(t, 0);
        reach_table<false>(t, 1);
        bool good0, good1;
        chains_in_lds = n_ranges() * 4u <= room;
        run_chains<true>(good0, good1);                    // (its first barrier stands behind the tables)
        reached = good0 && good1;
        if (!reached) return false;
        // cells of every row: columns one after the other (column 0 has one in row 0), a wavefront per row
        for (int s = wave; s <= S; s += nthreads >> 6) {
            const int n = number_row(s, false);
            if (lane == 0) tot[s] = n;
        }
        __syncthreads();
        int most = 0, sum = 0, least = INT32_MAX;
        for (int s = 0; s <= S; ++s) {
            const int n = tot[s];
            if (tid == 0) base[s] = sum;
            sum += n;
            most = n > most ? n : most;
            least = n < least ? n : least;
        }
        all_cells = uniform(sum);
        most = uniform(most);
        // F, B and the numbering stay in LDS where the rows of the whole pass fit beside them (with room for any form), else
        // they go to the slice: rows that leave LDS for them cost more
        const uint32_t bytes = (n_ranges() * 8u + 15u) & ~15u;
        ranges_in_lds = chains_in_lds && bytes + uint32_t(all_cells) * 4u + uint32_t(most) * 16u + 256u <= room;
        pass_at = rows + (ranges_in_lds ? bytes / 4u : 0u);
        pass_room = room - (ranges_in_lds ? bytes : 0u);
        for (int s = wave; s <= S; s += nthreads >> 6) number_row(s, true);
        most_cells = most;
        __syncthreads();
        return least > 0;
    }

    // One wavefront: the cells of row s; their numbering goes to LDS or to the slice (keep).
    __device__ __forceinline__ int number_row(int s, bool keep) const {
        const int lane = thread_id() & 63;
        int total = s == 0 ? 1 : 0;
        const uint32_t row = uint32_t(s) * uint32_t(sh.cols);
        for (int d = 1 + lane; d - lane <= D; d += 64) {
            uint32_t f = kNoCut, b = kNoCut;
            if (d <= D) {
                if (chains_in_lds) { const uint16_t *f_lds = reinterpret_cast<const uint16_t *>(rows) + row + d; f = f_lds[0]; b = f_lds[n_ranges()]; }
                else { f = sl.F[row + d]; b = sl.B[row + d]; }
            }
            const bool has = f != kNoCut && b != kNoCut && b <= f;
            const int w = has ? int(f - b) + 1 : 0, inc = int(fastdp::wave_scan(uint32_t(w), fastdp::sum2));
            if (keep && d <= D) put_column(row + d, has ? b : 1u, has ? f : 0u, total + inc - w - (has ? int(b) : 0));
            total += __builtin_amdgcn_readlane(inc, 63);
        }
        if (keep && lane == 0) put_column(row, s > 0 ? 1u : 0u, 0u, 0);
        return total;
    }
    __device__ __forceinline__ void put_column(uint32_t at, uint32_t lo, uint32_t hi, int off) const {
        if (ranges_in_lds) {
            uint16_t *f = reinterpret_cast<uint16_t *>(rows) + at;
            f[0] = uint16_t(hi);
            f[n_ranges()] = uint16_t(lo);
            reinterpret_cast<int32_t *>(rows)[n_ranges() + at] = off;
        } else { sl.F[at] = uint16_t(hi); sl.B[at] = uint16_t(lo); sl.off[at] = off; }
    }
    struct Column { int lo, hi, off; };
    __device__ __forceinline__ Column column(uint32_t at) const {
        Column c;
        if (ranges_in_lds) {
            const uint16_t *f = reinterpret_cast<const uint16_t *>(rows) + at;
            c.hi = f[0];
            c.lo = f[n_ranges()];
            c.off = reinterpret_cast<const int32_t *>(rows)[n_ranges() + at];
        } else { c.lo = sl.B[at]; c.hi = sl.F[at]; c.off = sl.off[at]; }
        return c;
    }
    // Range and numbering of row s into column buffer b, and the column of every cell; a thread's first
    // column is requested ahead (request_column) and waits in a register.  2^map_shift threads share a column: they
    // write its part of the map together.  Column 0 has a cell in row 0 only.
    __device__ __forceinline__ Column request_column(int s) const {
        const int d = 1 + (thread_id() >> map_shift);
        Column c{1, 0, 0};
        if (d <= D) c = column(uint32_t(s * sh.cols + d));
        return c;
    }
    __device__ __forceinline__ void store_column(int d, const Column &c, int b, bool with_map) {
        const int part = thread_id() & ((1 << map_shift) - 1);
        if (part == 0) {
            col[b * sh.cols + d] = uint2{uint32_t(c.lo) | (uint32_t(c.hi) << 16), uint32_t(c.off)};
            col_min[b * sh.cols + d] = 0xFFFFFFFFu;
        }
        if (with_map)
            for (int i = c.lo + part; i <= c.hi; i += 1 << map_shift) map[c.off + i] = uint16_t(d);
    }
    __device__ __forceinline__ void load_columns(int s, const Column &first, int b, bool with_map) {
        const int tid = thread_id();
        const int d0 = 1 + (tid >> map_shift);
        if (d0 <= D) store_column(d0, first, b, with_map);
        for (int d = d0 + (nthreads >> map_shift); d <= D; d += nthreads >> map_shift)
            store_column(d, column(uint32_t(s * sh.cols + d)), b, with_map);
        if (tid == 0) {
            col[b * sh.cols] = uint2{s == 0 ? 0u : 1u, 0u};
            col_min[b * sh.cols] = 0xFFFFFFFFu;
            if (s == 0 && with_map) map[0] = 0;
        }
    }
    __device__ __forceinline__ static int col_lo(const uint2 &c) { return int(c.x & 0xFFFFu); }
    __device__ __forceinline__ static int col_hi(const uint2 &c) { return int(c.x >> 16); }
    // column of cell x when there is no map: the last column that starts at or before x
    __device__ __forceinline__ int find_column(int b, int x) const {
        const uint2 *cols = col + b * sh.cols;
        int lo = 0, hi = D;                                // first cells rise with d; empty columns share theirs
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            const uint2 c = cols[mid];
            const int first = int(c.y) + (col_lo(c) <= col_hi(c) ? col_lo(c) : 0);
            if (first <= x) lo = mid; else hi = mid - 1;
        }
        while (col_lo(cols[lo]) > col_hi(cols[lo])) --lo;
        return lo;
    }

    // Rows of a pass in what the sets and the ranges of an ordering leave of the LDS: n rows of values of which a pass
    // keeps the last ones, two of counts (H-1F1B), the map.
    __device__ __forceinline__ int cells_that_fit(int bytes_per_cell) const { return int(pass_room / uint32_t(bytes_per_cell)) & ~7; }
    // All rows one after the other where they fit (whole; cell_bytes: of what a cell leaves behind, ring_bytes: of the
    // rest): nothing of the pass is stored to the slice then, and the plan is found from LDS.  Else the last rows, cut for
    // as many cells as fit.
    __device__ __forceinline__ void place_rows(int n, int n_counts, int cell_bytes, int ring_bytes, int bytes_per_cell) {
        const uint32_t most = (uint32_t(most_cells) + 7u) & ~7u, all = (uint32_t(all_cells) * uint32_t(cell_bytes) + 31u) & ~15u;
        whole = all + most * uint32_t(ring_bytes) <= pass_room;
        rows_all = pass_at;
        ring = whole ? pass_at + all / 4u : pass_at;
        pitch = (whole ? int(most) : cells_that_fit(bytes_per_cell)) + kRowPad;
        counts = reinterpret_cast<uint16_t *>(ring + n * pitch);
        map = counts + n_counts * pitch;
    }

    // One pass over all stages in the ranges of the last prepare.  Min-max: values above `t` count as
    // unreachable.  Otherwise: least sum of (t + 2c) over stage and transfer times of at most t.  Returns the value of
    // (S, L, D), or kInf.
    //
    // Min-max cells scan windows of four cuts downwards and stop when the stage time alone exceeds the
    // best value, or when nothing below the column's least value or the cell's transfer time is left to
    // gain (where a slow link decides, most columns hold one value throughout).
    // Least sums: D[j] + floor((P[i] + tp - 1 - P[j]) / tp) is floor((D[j] tp - P[j] + P[i] + tp - 1) / tp),
    // and the minimum can be taken inside the floor.  A row that fits LDS n_tp times over is turned into D[j] tp - P[j] per
    // degree once (key rows), and a cell is the minimum over a run of consecutive words; where only the values fit, the
    // product and the difference are formed on the way (two rows to read and two instructions more per cut); from the
    // workspace, and where the products do not fit 32 bits, a cut takes its whole time.
    enum { kPassMinMax, kPassSum, kPassKeys };
    struct StageCtx {
        int s, cur, nxt, total;
        bool last;
        const uint32_t *prev;
        uint32_t *next, *out;
        const int32_t *keys;
        const uint32_t *cut_tab;
        const uint16_t *fits_tab;
        uint32_t t, none;
    };
    template <int kPass, bool kLds>
    __device__ __forceinline__ void degree_best(const StageCtx &c, int q, int shift, int d2, int i, uint32_t cut, int from,
                                                int in_memory, int within, const uint32_t *p_k, uint32_t &best) const {
        const int tp = 1 << shift, d = d2 - tp;
        if (d < from) return;
        uint32_t floor_v = cut;
        if (kPass == kPassMinMax) {
            const uint32_t m = col_min[c.cur * sh.cols + d];
            floor_v = m > cut ? m : cut;
            if (floor_v >= best) return;
        }
        // previous cuts: in the column's range, in memory, within t
        const uint2 w = col[c.cur * sh.cols + d];
        int jl = in_memory > within ? in_memory : within;
        jl = jl > col_lo(w) ? jl : col_lo(w);
        const int jh = (i - 1) < col_hi(w) ? (i - 1) : col_hi(w);
        if (jl > jh) return;
        const uint32_t *p = p_k + q * sh.W;
        const uint32_t xi = p[i] + uint32_t(tp) - 1u;
        const int off = int(w.y);
        if (kPass == kPassKeys || (kPass == kPassSum && kLds)) {
            constexpr int32_t kNoKey = INT32_MAX;
            const int32_t *e = c.keys + q * pitch + off;
            const uint32_t *r = c.prev + off;
            auto key = [&](int j) -> int32_t { return kPass == kPassKeys ? e[j] : int32_t((r[j] << shift) - p[j]); };
            // the first window may reach beyond jh (what it reads there does not count), the others are pushed down
            // against it: cuts seen twice do not matter to a minimum
            int j = jl;
            const int32_t e0 = key(j);
            int32_t e1 = key(j + 1), e2 = key(j + 2), e3 = key(j + 3);
            e1 = j + 1 <= jh ? e1 : kNoKey;
            e2 = j + 2 <= jh ? e2 : kNoKey;
            e3 = j + 3 <= jh ? e3 : kNoKey;
            int32_t m = least(least(e0, e1), least(e2, e3));
            while (j + 3 < jh) {
                j = j + 4 < jh - 3 ? j + 4 : jh - 3;
                const int32_t f0 = key(j), f1 = key(j + 1), f2 = key(j + 2), f3 = key(j + 3);
                m = least(least(least(f0, f1), m), least(f2, f3));
            }
            if (kPass == kPassSum || m != kNoKey) best = least(best, (xi + uint32_t(m)) >> shift);
        } else {
            constexpr bool kCapped = kPass == kPassSum;
            const uint32_t *r = c.prev + off;
            // the first window may be cut short at its upper end, the last is pushed up
            // against jl (cuts seen twice do not matter to a minimum)
            int j = jh - 3 > jl ? jh - 3 : jl;
            uint32_t t0;
            {
                const uint32_t p0 = p[j], p1 = p[j + 1], p2 = p[j + 2], p3 = p[j + 3];
                const uint32_t r0 = r[j], r1 = r[j + 1], r2 = r[j + 2], r3 = r[j + 3];
                t0 = (xi - p0) >> shift;
                const uint32_t t1 = (xi - p1) >> shift, t2 = (xi - p2) >> shift, t3 = (xi - p3) >> shift;
                const uint32_t v0 = value<kCapped>(r0, t0, cut);
                const uint32_t v1 = j + 1 <= jh ? value<kCapped>(r1, t1, cut) : c.none;
                const uint32_t v2 = j + 2 <= jh ? value<kCapped>(r2, t2, cut) : c.none;
                const uint32_t v3 = j + 3 <= jh ? value<kCapped>(r3, t3, cut) : c.none;
                best = least(best, least(least(v0, v1), least(v2, v3)));
            }
            while (j > jl && (kCapped || (t0 <= best && best > floor_v))) {
                j = j - 4 > jl ? j - 4 : jl;
                const uint32_t p0 = p[j], p1 = p[j + 1], p2 = p[j + 2], p3 = p[j + 3];
                const uint32_t r0 = r[j], r1 = r[j + 1], r2 = r[j + 2], r3 = r[j + 3];
                t0 = (xi - p0) >> shift;
                const uint32_t t1 = (xi - p1) >> shift, t2 = (xi - p2) >> shift, t3 = (xi - p3) >> shift;
                const uint32_t v0 = value<kCapped>(r0, t0, cut), v1 = value<kCapped>(r1, t1, cut);
                const uint32_t v2 = value<kCapped>(r2, t2, cut), v3 = value<kCapped>(r3, t3, cut);
                best = least(best, least(least(v0, v1), least(v2, v3)));
            }
        }
    }
    // The cells of a row.  kSplit: four lanes share a cell, a degree each (at most four degrees, my_*: the lane's own):
    // a row of few cells is bound by the chain of one cell's degrees.
    template <int kPass, bool kLds, bool kSplit>
    __device__ __forceinline__ void row_cells(const StageCtx &c, int my_q, int my_shift) {
        const int tid = thread_id();
        const int part = kSplit ? tid & 3 : 0, step = kSplit ? nthreads >> 2 : nthreads;
        int x = kSplit ? tid >> 2 : tid;
        for (; x < c.total; x += step) {
            const int d2 = kLds ? int(map[x]) : find_column(c.nxt, x);
            const int i = x - int(col[c.nxt * sh.cols + d2].y);
            const int k = group_at[d2 - 1];
            uint32_t cut = c.cut_tab[cut_at[d2] + uint32_t(i)];        // (read behind the last stage too: no branch to wait in)
            uint32_t best = c.none;
            const uint32_t *p_k = time_row(k);
            const int from = offs[k] > c.s ? offs[k] : c.s;
            const uint16_t *fits = c.fits_tab + (index_at[k] + uint32_t(i)), *far = reach_row(1, k) + i;
            if (kSplit) {
                const int in_memory = fits[my_q * sh.idx_pitch], within = far[my_q * sh.W];
                cut = c.last ? 0u : cut;
                if (cut <= c.t && my_shift >= 0)
                    degree_best<kPass, kLds>(c, my_q, my_shift, d2, i, cut, from, in_memory, within, p_k, best);
                best = least(best, uint32_t(__builtin_amdgcn_update_dpp(int(best), int(best), 0xB1, 0xF, 0xF, false)));   // lanes 1 and 2 apart
                best = least(best, uint32_t(__builtin_amdgcn_update_dpp(int(best), int(best), 0x4E, 0xF, 0xF, false)));
                if (part != 0) continue;
            } else {
                // degrees from the largest down, four at a time: the first values found are then the best ones,
                // and a degree whose column holds nothing below the best value is passed over
                for (int q0 = (tb.n_tp - 1) & ~3; q0 >= 0; q0 -= 4) {
                    int in_memory[4], within[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int q = q0 + u < tb.n_tp ? q0 + u : q0;
                        in_memory[u] = fits[q * sh.idx_pitch];
                        within[u] = far[q * sh.W];
                    }
                    // (requested together: a load that the compiler moves into a branch is waited for there)
                    asm volatile("" : "+v"(in_memory[0]), "+v"(in_memory[1]), "+v"(in_memory[2]), "+v"(in_memory[3]));
                    cut = c.last ? 0u : cut;
                    if (cut > c.t) break;
#pragma unroll
                    for (int u = 3; u >= 0; --u)
                        if (q0 + u < tb.n_tp)
                            degree_best<kPass, kLds>(c, q0 + u, shift_of(q0 + u), d2, i, cut, from, in_memory[u], within[u], p_k, best);
                }
            }
            if (kPass != kPassMinMax) best = best < c.none ? best + 2u * cut : c.none;
            if (kLds) c.next[x] = best;
            // (lanes of a wavefront mostly share a column: the read in front spares the serialised atomics)
            if (kPass == kPassMinMax && best < col_min[c.nxt * sh.cols + d2]) atomicMin(&col_min[c.nxt * sh.cols + d2], best);
            if (!kLds || c.out) c.out[x] = best;
        }
    }
    template <int kPass, bool kLds>
    __device__ __forceinline__ int64_t value_pass_in(uint32_t t) {
        const int tid = thread_id();
        constexpr bool kKeys = kPass == kPassKeys;
        constexpr int32_t kNoKey = INT32_MAX;
        // sums are below 2^31, and where keys are formed below 2^31 / degree, less one (largest_cap)
        const uint32_t none = kPass == kPassMinMax ? t + 1u : kPass == kPassSum && kLds ? key_limit() - 1u : kInfSum;
        // kept for the plan: the rows of values; for the next stage: key rows, the map
        if (kLds) place_rows(kKeys ? tb.n_tp : 0, 0, 4, kKeys ? 4 * tb.n_tp + 2 : 2, kKeys ? keys_bytes() : kValueBytes);
        else whole = false;
        // (not whole: the one row of values, or the two, behind the key rows)
        int32_t *keys = reinterpret_cast<int32_t *>(ring);                 // [n_tp][pitch] (kKeys)
        uint32_t *values = ring + (kKeys ? tb.n_tp * pitch : 0);
        if (kLds && !whole) map = reinterpret_cast<uint16_t *>(values + (kKeys ? 1 : 2) * pitch);
        int my_q = 0, my_shift = -1;                                       // (no degree: no stage)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if ((tid & 3) == q && q < tb.n_tp) { my_q = q; my_shift = shift_of(q); }
        int cur = 0;
        load_columns(0, request_column(0), 0, false);
        Column ahead = request_column(1);
        if (tid == 0) {                                    // row 0: no operators on no devices
            if (!kLds) sl.hist[0] = 0;
            else if (whole) rows_all[0] = 0;
            else values[0] = sl.hist[0] = 0;
            col_min[0] = 0;
            if (kKeys)
                for (int q = 0; q < tb.n_tp; ++q) keys[q * pitch] = 0;
        }
        for (int s = 0; s < S; ++s) {
            const int nxt = cur ^ 1;
            load_columns(s + 1, ahead, nxt, kLds);
            pass_barrier<kLds>();                          // row s, its columns and those of row s + 1 are in place
            if (s + 1 < S) ahead = request_column(s + 2);
            StageCtx c;
            c.s = s; c.cur = cur; c.nxt = nxt; c.t = t; c.none = none;
            c.last = s == S - 1;
            c.total = uniform(tot[s + 1]);
            const int at = uniform(base[s]), at_next = uniform(base[s + 1]);
            c.prev = kLds ? (whole ? rows_all + at : values + cur * pitch) : sl.hist + at;
            c.next = whole ? rows_all + at_next : kKeys ? values : values + nxt * pitch;
            c.out = whole ? nullptr : sl.hist + at_next;
            c.keys = keys;
            c.cut_tab = tb.CM;
            c.fits_tab = lo_tab + index_n(in_flight(s));
            if (kLds && tb.n_tp > 1 && tb.n_tp <= 4 && 2 * c.total <= nthreads) row_cells<kPass, kLds, true>(c, my_q, my_shift);
            else row_cells<kPass, kLds, false>(c, my_q, my_shift);
            pass_barrier<kLds>();                          // row s + 1 is complete
            if (kKeys && !c.last) {
                // the row as stage s + 1 reads it: a stage that starts at device d runs on the group of d
                for (int x = tid; x < c.total; x += nthreads) {
                    const int d = map[x], i = x - int(col[nxt * sh.cols + d].y), k = group_at[d];
                    const uint32_t v = c.next[x], *p = time_row(k) + i;
                    for (int q = 0; q < tb.n_tp; ++q)
                        keys[q * pitch + x] = v < kInfSum ? int32_t((v << shift_of(q)) - p[q * sh.W]) : kNoKey;
                }
                lds_barrier();
            }
            cur = nxt;
        }
        if (kLds && !whole) __syncthreads();               // (the slice's rows, for the plan)
        const int end = uniform(base[S]);
        const uint32_t v = !kLds ? sl.hist[end] : whole ? rows_all[end] : values[kKeys ? 0 : cur * pitch];
        return v >= none ? kInf : int64_t(v);
    }
    template <bool kLds>
    __device__ __forceinline__ void pass_barrier() const {
        if (kLds) lds_barrier();
        else __syncthreads();
    }
    template <bool kCapped>
    __device__ __forceinline__ uint32_t value(uint32_t before, uint32_t time, uint32_t cut) const {
        if (kCapped) return before + time;
        return fastdp::umax3(before, time, cut);
    }
    __device__ __forceinline__ int32_t least(int32_t a, int32_t b) const { return a < b ? a : b; }
    __device__ __forceinline__ uint32_t least(uint32_t a, uint32_t b) const { return a < b ? a : b; }
    // All threads: the plan of the last value pass, value `v`, from the value rows: per stage the lowest
    // previous cut, then the smallest degree, that attain the cell's value (lanes over degrees and cuts).
    __device__ __forceinline__ void find_plan(bool capped, uint32_t v, uint32_t cap) {
        const int lane = thread_id() & 63;
        if (wave == 0) {
            const int per = tb.n_tp <= 1 ? 64 : tb.n_tp <= 2 ? 32 : tb.n_tp <= 4 ? 16 : 8;   // lanes per degree
            const int q = lane / per, jj = lane - q * per;
            const int tp = q < tb.n_tp ? tp_of(q) : 0, shift = q < tb.n_tp ? shift_of(q) : 0;
            int d2 = D, i = L;
            if (lane == 0) cuts[S] = L;
            for (int s = S - 1; s >= 0; --s) {
                const int k = group_at[d2 - 1], n = in_flight(s), d = d2 - tp;
                uint32_t want = v;
                if (capped && s < S - 1) want = v - 2u * tb.CM[cut_at[d2] + uint32_t(i)];
                const bool in = q < tb.n_tp && d >= offs[k] && d >= s;
                int jl = 1, jh = 0, off = 0;
                if (in) {
                    const int fits = lo_tab[index_n(n) + index_at[k] + uint32_t(q * sh.idx_pitch + i)];
                    const Column w = column(uint32_t(s * sh.cols + d));
                    off = w.off;
                    jl = fits > w.lo ? fits : w.lo;
                    jh = (i - 1) < w.hi ? (i - 1) : w.hi;
                }
                const uint32_t *p = time_row(k) + (in ? q : 0) * sh.W;
                const uint32_t xi = p[i] + uint32_t(tp) - 1u;
                uint32_t key = 0xFFFFFFFFu, val = 0;
                for (int j = jl + jj; __any(in && j <= jh && key == 0xFFFFFFFFu); j += per) {
                    if (in && j <= jh && key == 0xFFFFFFFFu) {
                        const uint32_t time = (xi - p[j]) >> shift;
                        if (time <= (capped ? cap : want)) {
                            const int at = base[s] + off + j;
                            uint32_t before;
                            if (whole) before = rows_all[at]; else before = sl.hist[at];
                            const bool hit = capped ? before < kInfSum && before + time == want : before <= want;
                            if (hit) { key = (uint32_t(j) << 3) | uint32_t(q); val = before; }
                        }
                    }
                }
                const uint32_t low = fastdp::wave_least(key);
                const unsigned long long who = __ballot(key == low);
                v = __builtin_amdgcn_readlane(val, __ffsll((long long)who) - 1);
                // a reached cell always has one; the clamps keep the indices inside the rows whatever happens
                const int jn = int((low >> 3) & 0xFFFFu), qn = int(low & 7u);
                i = jn < i ? jn : i - 1;
                i = i > 0 ? i : 0;
                d2 -= tp_of(qn < tb.n_tp ? qn : 0);
                d2 = d2 > 0 ? d2 : 0;
                if (lane == 0) {
                    cuts[s] = i;
                    slot_g[s] = order[k];
                    slot_k[s] = uint8_t(qn < tb.n_tp ? qn : 0);
                    slot_first[s] = tb.group_base[order[k]] + (d2 - offs[k]);
                }
                if (s > 0 && d2 == 0) d2 = 1;
            }
        }
        __syncthreads();
    }

    // All threads: the first cap to try the min-max pass under.  Every group takes work in proportion to its speed; and
    // every plan cuts somewhere on every link from a group to the next, no cheaper than at the operator of least output.
    // Where a link decides, the optimum mostly lies there: the ranges under this cap are worked out at once, and
    // only where they do not meet is a higher one looked for (82 operators and 64 devices: two reach tables and one
    // round of chains where a search in front of the ranges takes four and two).  Where the speeds decide, no plan spreads the
    // work that evenly: there the search comes first, and a round of chains that fails is spared (us with it tried at once /
    // with the search first: 4,096 orderings of 82 operators 725 / 714; search over the cap, 16 of 29 operators and 4 stages 142 /
    // 137).
    __device__ __forceinline__ uint32_t guess() {
        const int lane = thread_id() & 63;
        if (wave == 0) {
            float share = 0.f;
            uint32_t bound = 0;
            for (int k = lane; k < K; k += 64) {
                const float whole = float(tb.PF(type[k])[L]);
                share += float(offs[k + 1] - offs[k]) / (whole > 1.f ? whole : 1.f);
                if (k + 1 < K) {
                    const uint32_t c = tb.CM[link_at[K + k] + uint32_t(least_cut)];
                    bound = c > bound ? c : bound;
                }
            }
#pragma unroll
            for (int x = 32; x >= 1; x >>= 1) {
                share += __shfl_xor(share, x, 64);
                const uint32_t o = __shfl_xor(bound, x, 64);
                bound = o > bound ? o : bound;
            }
            const float guess = 1.f / share;
            if (lane == 0) { scal[5] = guess < 1.f ? 1u : guess > 1e9f ? 1000000000u : uint32_t(guess); scal[6] = bound; }
        }
        __syncthreads();
        const uint32_t g = scal[5] > scal[6] ? scal[5] : scal[6];
        unlikely = scal[5] > scal[6] && g < kTopCap;
        return g < kTopCap ? g : kTopCap;
    }
    // All threads: the next cap to try when the ranges under the first, g, did not meet; -1 when no plan exists under any.
    __device__ __forceinline__ int64_t bracket(int64_t g) {
        int64_t bad = g, good = -1;                        // largest t known to have no plan, smallest t whose chain succeeds
        // until the two are within 1/12 of each other: below that the rows hardly get shorter than a workgroup
        for (int round = 0; good < 0 || good - bad > good / 12 + 1; ++round) {
            int64_t at[kTeams];
            for (int w = 0; w < kTeams; ++w) {
                // where the optimum did not lie at the guess it lay within a fifth above on most
                const int step = round * kTeams + w + 1;
                int64_t t;
                if (good >= 0) t = bad + (good - bad) * (w + 1) / (kTeams + 1);
                else t = step == 1 ? g + g * 7 / 32 + 1 : step == 2 ? g + g * 5 / 8 + 1 : step == 3 ? 5 * g / 2 + 1
                         : step == 4 ? 8 * g + 1 : step == 5 ? 64 * g + 1 : int64_t(kTopCap);
                at[w] = t < int64_t(kTopCap) ? t : int64_t(kTopCap);
            }
            __syncthreads();
            cut_masks(kTeams, uint32_t(at[0]), uint32_t(at[1]));
            for (int w = 0; w < kTeams; ++w) reach_table<true>(uint32_t(at[w]), w);
            bool fine[kTeams];
            run_chains<false>(fine[0], fine[1]);
            for (int w = kTeams - 1; w >= 0; --w)
                if (fine[w]) good = at[w];
            for (int w = 0; w < kTeams; ++w)
                if (!fine[w] && at[w] > bad) bad = at[w];
            if (good < 0 && bad >= int64_t(kTopCap)) return -1;           // no plan under any cap
        }
        return good;
    }

    // The cap after one under which the min-max pass found no plan: an eighth above, then a quarter, where an optimum
    // that the chains missed lies as a rule, then none.  With no / one / both steps, us: 1,024 orderings of 82
    // operators and 64 devices, each with a plan, 567 / 478 / 473; 160 operators and 128 devices 4,860 / 6,130 /
    // 4,340; 120 operators, 60 stages on 64 devices, none with a plan, 618 / 746 / 870 (2,650 with steps that grow
    // up to 2^31, some twenty passes).
    static __device__ __forceinline__ uint32_t raised(uint32_t t, int tries) {
        return tries < 2 && t < kTopCap / 2 ? t + (t >> (3 - tries)) + 1u : kTopCap;
    }

    // The recurrence with H-1F1B warm-up counts (eq. dp_ni) in the ranges of the last prepare, suffix
    // direction: cell (s, d, i) = stages s .. S-1 hold the operators from i on, on the devices from d on.
    // A row is stored ready for the stage in front of it: sum plus twice the transfer time of the cut
    // at i (kInfSum beyond the cap) and the count that stage would have.  Ties: lowest end cut, then
    // smallest degree.  The memory test runs only for a cut that would be taken.  Returns the value of
    // (0, 0, 0) or kInf; back-pointers (cut | degree index << 13) go to the slice.
    //
    // kCount: the least count of the first stage instead of the least sum (every row: the least count the
    // stage in front could have).  A smaller count never hurts - it weakens every memory test in front of
    // it - so this decides whether ANY plan exists under the cap, and it is monotone in the cap.
    template <bool kCount, bool kLds>
    __device__ __forceinline__ int64_t h1_pass_in(uint32_t cap) {
        constexpr uint32_t kNoCount = 0xFFFFu;
        const int tid = thread_id();
        const uint64_t e6 = uint64_t(count_cap) >> 6, x1 = e6 >> 1, x2 = (uint64_t(count_cap) + e6) >> 1;
        const uint32_t th1 = uint32_t(x1 < kTopCap ? x1 : kTopCap), th2 = uint32_t(x2 < kTopCap ? x2 : kTopCap);   // 2c - e > 0; > cap
        const uint32_t m_cap = uint32_t(tb.M);
        const int64_t *PP = mem, *PS = mem + sh.W;
        if (kLds) place_rows(2, 2, 2, kCountBytes, kCountBytes);
        else whole = false;
        uint16_t *back = reinterpret_cast<uint16_t *>(sl.hist), *back_lds = reinterpret_cast<uint16_t *>(rows_all);
        auto row_h = [&](int b) -> uint32_t * { return kLds ? ring + b * pitch : sl.spare_h + b * sl.row; };
        auto row_n = [&](int b) -> uint16_t * { return kLds ? counts + b * pitch : sl.spare_n + b * sl.row; };
        int cur = 0;
        load_columns(S, request_column(S), 0, false);
        Column ahead = request_column(S - 1);
        if (tid == 0) { row_h(0)[0] = 0; row_n(0)[0] = 1; }    // behind the last stage: it launches one
        for (int s = S - 1; s >= 0; --s) {
            const uint32_t index_at_n = index_n(in_flight(s));
            const int nxt = cur ^ 1;
            load_columns(s, ahead, nxt, kLds);
            pass_barrier<kLds>();
            if (s > 0) ahead = request_column(s - 1);
            const uint32_t *prev_h = row_h(cur);
            const uint16_t *prev_n = row_n(cur);
            uint32_t *next_h = row_h(nxt);
            uint16_t *next_n = row_n(nxt);
            const int total = tot[s], at = base[s];
            for (int x = tid; x < total; x += nthreads) {
                const int d = kLds ? int(map[x]) : find_column(nxt, x);
                const int i = x - int(col[nxt * sh.cols + d].y);
                const int k = group_at[d], end = offs[k + 1];
                const int64_t mem_dev = tb.type_mem[type[k]];
                uint32_t cut = tb.CM[cut_at[d] + uint32_t(i)];             // (read in front of the first stage too: no branch to wait in)
                const uint16_t *fits = hi_tab + (index_at_n + index_at[k] + uint32_t(i)), *far = reach_row(0, k) + i;
                const uint32_t *p_k = time_row(k);
                const int64_t ppi = PP[i], psi = PS[i];
                cut = s > 0 ? cut : 0u;
                uint32_t best = kInfSum, best_n = kCount ? kNoCount : 0u;
                int best_j = 0, best_q = 0;
                for (int q0 = 0; q0 < tb.n_tp; q0 += 4) {
                    int in_memory[4];                          // requested together, no branches in between
#pragma unroll
                    for (int u = 0; u < 4; ++u) in_memory[u] = fits[(q0 + u < tb.n_tp ? q0 + u : q0) * sh.idx_pitch];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        if (q0 + u >= tb.n_tp) continue;
                        const int q = q0 + u, shift = shift_of(q), tp = 1 << shift, d1 = d + tp;
                        if (d1 > end) continue;
                        const uint2 w = col[cur * sh.cols + d1];
                        const int lo = col_lo(w), hi = col_hi(w);
                        const int within = far[q * sh.W];
                        const int jl = (i + 1) > lo ? (i + 1) : lo;
                        int jh = in_memory[u] < within ? in_memory[u] : within;
                        jh = jh < hi ? jh : hi;
                        const uint32_t *p = p_k + q * sh.W;
                        const int off = int(w.y);
                        const uint32_t xi = p[i] - uint32_t(tp) + 1u;
                        const int64_t capm = int64_t(tp) * mem_dev;
                        for (int j = jl; j <= jh; ++j) {
                            if (kCount) {
                                const uint32_t cnt = prev_n[off + j];
                                if (cnt < best_n && (PP[j] - ppi) + int64_t(cnt) * (PS[j] - psi) <= capm) best_n = cnt;
                            } else {
                                const uint32_t v = prev_h[off + j] + ((p[j] - xi) >> shift);
                                if (v < best || (v == best && j < best_j)) {
                                    const uint32_t cnt = prev_n[off + j];
                                    if ((PP[j] - ppi) + int64_t(cnt) * (PS[j] - psi) <= capm) {
                                        best = v; best_j = j; best_q = q; best_n = cnt;
                                    }
                                }
                            }
                        }
                    }
                }
                if (!kCount) {
                    const uint16_t to = uint16_t(uint32_t(best_j) | (uint32_t(best_q) << 13));
                    if (whole) back_lds[at + x] = to; else back[at + x] = to;
                }
                if (s > 0) {
                    const uint32_t cnt = 1u + (cut > th1 ? 1u : 0u) + (cut > th2 ? 1u : 0u) + best_n;
                    const uint32_t cnt_m = cnt < m_cap ? cnt : m_cap;
                    if (kCount) {
                        next_n[x] = uint16_t(best_n != kNoCount && cut <= cap ? cnt_m : kNoCount);
                    } else {
                        const uint32_t h = best < kInfSum && cut <= cap ? best + 2u * cut : kInfSum;
                        next_h[x] = h < kInfSum ? h : kInfSum;
                        next_n[x] = uint16_t(cnt_m);
                    }
                } else {
                    scal[4] = kCount ? (best_n != kNoCount ? 0u : kInfSum) : best;
                }
            }
            pass_barrier<kLds>();
            cur = nxt;
        }
        if (kLds && !kCount && !whole) __syncthreads();    // (the slice's back-pointers, for the plan)
        const uint32_t v = scal[4];
        return v >= kInfSum ? kInf : int64_t(v);
    }
    // One pass under the cap t in one of the four forms: the min-max value, the least sum, the least sum with
    // H-1F1B's counts, or 0 when those admit a plan at all; kInf without one.  kForms: the forms a kernel
    // uses, as a mask.  Called at one place of a kernel: every inlined copy of the passes costs registers
    // everywhere else.
    static constexpr int kMinMax = 1, kSum = 2, kH1 = 4, kAny = 8;
    template <int kForms>
    __device__ __forceinline__ int64_t run(int form, uint32_t t) {
        if (unlikely) { unlikely = reached = false; return kInf; }
        if (!prepare(t)) return kInf;
        if ((kForms & (kMinMax | kSum)) && (form == kMinMax || form == kSum)) {
            const bool values_fit = most_cells <= cells_that_fit(kValueBytes);
            if ((kForms & kMinMax) && form == kMinMax)
                return values_fit ? value_pass_in<kPassMinMax, true>(t) : value_pass_in<kPassMinMax, false>(t);
            if (keys_fit && most_cells <= cells_that_fit(keys_bytes())) return value_pass_in<kPassKeys, true>(t);
            return keys_fit && values_fit ? value_pass_in<kPassSum, true>(t) : value_pass_in<kPassSum, false>(t);
        }
        const bool rows_fit = most_cells <= cells_that_fit(kCountBytes);
        if ((kForms & kH1) && form == kH1) return rows_fit ? h1_pass_in<false, true>(t) : h1_pass_in<false, false>(t);
        if (kForms & kAny) return rows_fit ? h1_pass_in<true, true>(t) : h1_pass_in<true, false>(t);
        return kInf;
    }
    // All threads: PP and PS into LDS, once per kernel
    __device__ __forceinline__ void load_memory_sums() {
        const int tid = thread_id();
        const int64_t *PP = tb.PP(), *PS = tb.PS();
        for (int j = tid; j <= L; j += nthreads) { mem[j] = PP[j]; mem[sh.W + j] = PS[j]; }
        __syncthreads();
    }
    // All threads, once per kernel of the search over the cap (walk: no bracket in it), and its item c.
    __device__ __forceinline__ void start(bool walk) {
        load_memory_sums();
        if (!walk) find_least_cut();
    }
    __device__ __forceinline__ int load_item(const OrdDev &od, int c) {
        return load(od.ord_S[c], od.ord_G[c], od.ord_group + int64_t(c) * od.G_max, od.S_max, od.G_max);
    }
    // All threads: the plan of the last H-1F1B pass, with its counts by eq. Ni.
    __device__ __forceinline__ void find_h1_plan() {
        const int lane = thread_id() & 63;
        if (wave == 0) {
            const uint16_t *back = reinterpret_cast<const uint16_t *>(sl.hist), *back_lds = reinterpret_cast<const uint16_t *>(rows_all);
            int d = 0, i = 0;
            for (int s = 0; s < S; ++s) {
                const int k = group_at[d];
                const Column w = column(uint32_t(s * sh.cols + d));
                const int ic = i < w.lo ? w.lo : (i > w.hi ? w.hi : i);       // a finite sum only chains through cells
                const int at = base[s] + w.off + ic;
                uint32_t a;
                if (whole) a = back_lds[at]; else a = back[at];
                const int q = int(a >> 13) & 7;
                if (lane == 0) {
                    cuts[s] = i;
                    slot_g[s] = order[k];
                    slot_k[s] = uint8_t(q < tb.n_tp ? q : 0);
                    slot_first[s] = tb.group_base[order[k]] + (d - offs[k]);
                }
                i = int(a & 0x1FFFu);
                d += tb.tp[q < tb.n_tp ? q : 0];
                d = d < D ? d : (s + 1 < S ? D - 1 : D);
            }
            if (lane == 0) cuts[S] = L;
            wave_sync();
            const uint64_t e6 = uint64_t(count_cap) >> 6;
            for (int s = lane; s < S; s += 64) {
                uint32_t cut = 0;
                if (s < S - 1) cut = tb.CM[(int64_t(slot_g[s]) * tb.G + slot_g[s + 1]) * tb.pitch32 + cuts[s + 1]];
                warmup[s] = 1 + (2ull * cut > e6 ? 1 : 0) + (2ull * cut > uint64_t(count_cap) + e6 ? 1 : 0);
            }
            wave_sync();
            if (lane == 0) {
                int run = 0;
                for (int s = S - 1; s >= 0; --s) {
                    run += warmup[s];
                    run = run < tb.M ? run : tb.M;
                    warmup[s] = run;
                }
            }
        }
        __syncthreads();
    }

    // Candidate caps of the ordering (section 5.2.4 (2)): every stage time of a listed group, a degree not
    // above its size and an operator range; every transfer time of an inner cut inside a listed group
    // or to the group after it.  All threads: visit(v) for every one in (a, b], repetitions included; a
    // thread's `beyond` becomes the least value above b it has seen.
    template <typename VisitFn>
    __device__ __forceinline__ void visit_values(uint32_t a, uint32_t b, uint32_t &beyond, VisitFn visit) const {
        const int tid = thread_id();
        const int n = n_sets * tb.n_tp * L, top_step = 1 << (31 - __clz(L));
        for (int x = tid; x < n; x += nthreads) {
            const int r = x / L, j = x - r * L, set = r / tb.n_tp, q = r - set * tb.n_tp;
            const uint32_t tp = uint32_t(tb.tp[q]);
            if (tp > use[set]) continue;
            const int shift = tb.tp_shift[q];
            const uint32_t *p = prow + r * sh.W;
            const uint32_t pj = p[j];
            const uint64_t far = uint64_t(a) * tp + pj;        // time(j, i) <= a
            const uint32_t target = far > 0xFFFFFFFFull ? 0xFFFFFFFFu : uint32_t(far);
            int i = j;
            for (int step = top_step; step > 0; step >>= 1) {
                const int nx = i + step;
                i = nx <= L && p[nx <= L ? nx : L] <= target ? nx : i;
            }
            for (++i; i <= L; ++i) {
                const uint32_t v = (p[i] - pj + tp - 1u) >> shift;
                if (v > b) { beyond = v < beyond ? v : beyond; break; }
                visit(v);
            }
        }
        if (L < 2) return;
        const int links = 2 * K - 1;
        for (int x = tid; x < links * (L - 1); x += nthreads) {
            const int l = x / (L - 1), i = 1 + x - l * (L - 1);
            const uint32_t v = tb.CM[link_at[l] + uint32_t(i)];
            if (v > b) beyond = v < beyond ? v : beyond;
            else if (v > a) visit(v);
        }
    }
    // All threads: a workgroup-wide minimum / sum through LDS
    __device__ __forceinline__ uint32_t group_min(uint32_t v) {
        const int tid = thread_id();
#pragma unroll
        for (int x = 32; x >= 1; x >>= 1) {
            const uint32_t o = __shfl_xor(v, x, 64);
            v = o < v ? o : v;
        }
        __syncthreads();
        if (tid == 0) scal[7] = 0xFFFFFFFFu;
        __syncthreads();
        if ((tid & 63) == 0) atomicMin(&scal[7], v);
        __syncthreads();
        return scal[7];
    }
    // The highest cap up to which the last pass, under the cap t, is known to come out the same.
    __device__ __forceinline__ uint32_t same_up_to(uint32_t t) const { return t; }
    // All threads: the smallest candidate cap above a; 0xFFFFFFFF when there is none.
    __device__ __forceinline__ uint32_t next_value(uint32_t a) {
        uint32_t beyond = 0xFFFFFFFFu;
        visit_values(a, a, beyond, [](uint32_t) {});
        return group_min(beyond);
    }
    // All threads: the largest candidate cap.
    __device__ __forceinline__ uint32_t largest_value() {
        const int tid = thread_id();
        uint32_t most = 0;
        for (int r = tid; r < n_sets * tb.n_tp; r += nthreads) {
            const int set = r / tb.n_tp, q = r - set * tb.n_tp;
            const uint32_t tp = uint32_t(tb.tp[q]);
            const uint32_t v = (prow[r * sh.W + L] + tp - 1u) >> tb.tp_shift[q];
            most = tp <= use[set] && v > most ? v : most;
        }
        const int links = L < 2 ? 0 : 2 * K - 1;
        for (int x = tid; x < links * (L - 1); x += nthreads) {
            const int l = x / (L - 1), i = 1 + x - l * (L - 1);
            const uint32_t v = tb.CM[link_at[l] + uint32_t(i)];
            most = v > most ? v : most;
        }
        return ~group_min(~most);
    }
    // All threads: how many distinct candidate caps lie in (a, b], counted up to `limit`; `last` becomes the
    // limit-th of them when there are that many.  A bitmap over a window of values in LDS (the value rows,
    // which no pass needs meanwhile) no longer than the values left, window after window, each starting at the next value there is.
    __device__ __forceinline__ uint32_t count_values(uint32_t a, uint32_t b, uint32_t limit, uint32_t &last) {
        const int tid = thread_id();
        const uint32_t most = (room / 4u) & ~63u;
        uint32_t *bits = rows;
        uint32_t found = 0, from = a + 1u;
        while (from <= b && found < limit) {
            const uint32_t left = ((b - from) / 2048u + 1u) * 64u, words = left < most ? left : most, span = words * 32u;
            const uint32_t to = b - from < span ? b : from + (span - 1u);
            __syncthreads();
            for (uint32_t w = tid; w < words; w += nthreads) bits[w] = 0;
            __syncthreads();
            uint32_t beyond = 0xFFFFFFFFu;
            visit_values(from - 1u, to, beyond, [&](uint32_t v) {
                const uint32_t at = v - from;
                atomicOr(&bits[at >> 5], 1u << (at & 31u));
            });
            const uint32_t next = group_min(beyond);       // (its barriers complete the bitmap)
            uint32_t mine = 0;
            for (uint32_t w = tid; w < words; w += nthreads) mine += __popc(bits[w]);
#pragma unroll
            for (int x = 32; x >= 1; x >>= 1) mine += __shfl_xor(mine, x, 64);
            __syncthreads();
            if (tid == 0) scal[7] = 0;
            __syncthreads();
            if ((tid & 63) == 0) atomicAdd(&scal[7], mine);
            __syncthreads();
            const uint32_t here = scal[7];
            if (found + here >= limit) {
                // the limit-th value: the words of the bitmap in order (rare, one wavefront)
                __syncthreads();
                if (tid < 64) {
                    uint32_t rank = limit - found;
                    for (uint32_t w0 = 0; w0 < words; w0 += 64) {
                        const uint32_t v = bits[w0 + tid];
                        uint32_t inc = __popc(v);
#pragma unroll
                        for (int x = 1; x < 64; x <<= 1) {
                            const uint32_t o = __shfl_up(inc, x, 64);
                            if (tid >= x) inc += o;
                        }
                        const uint32_t all = __shfl(inc, 63, 64);
                        if (rank > all) { rank -= all; continue; }
                        const uint32_t before = inc - __popc(v);
                        if (before < rank && rank <= inc) {
                            uint32_t rest = v;
                            for (uint32_t n = rank - before; n > 1; --n) rest &= rest - 1u;
                            scal[7] = from + (w0 + tid) * 32u + uint32_t(__ffs((int)rest) - 1);
                        }
                        break;
                    }
                }
                __syncthreads();
                last = scal[7];
                return limit;
            }
            found += here;
            if (next == 0xFFFFFFFFu || next > b) break;
            from = next;
        }
        return found;
    }

    // All threads: the plan in cuts / slot_* to the outputs of ordering c.
    __device__ __forceinline__ void write_slots(const PlansDev &out, int c, int S_max, int32_t *sg, int32_t *stp) const {
        const int tid = thread_id();
        int32_t *sp = out.splits + int64_t(c) * (S_max + 1), *df = out.dev_first + int64_t(c) * S_max;
        for (int s = tid; s <= S_max; s += nthreads) sp[s] = s <= S ? cuts[s] : -1;
        for (int s = tid; s < S_max; s += nthreads) {
            sg[s] = s < S ? int32_t(slot_g[s]) : -1;
            stp[s] = s < S ? tb.tp[slot_k[s]] : -1;
            df[s] = s < S ? slot_first[s] : -1;
        }
    }
    // All threads: bottleneck and iteration time of the plan in cuts / slot_* (scored: LDS, two entries).
    __device__ __forceinline__ void score(int64_t *scored, int64_t &bott, int64_t &total) const {
        const int lane = thread_id() & 63;
        if (wave == 0) {
            int64_t x, y;
            wave_score_partition(tb, S, slot_g, slot_k, cuts, lane, x, y);
            if (lane == 0) { scored[0] = x; scored[1] = y; }
        }
        __syncthreads();
        bott = scored[0];
        total = scored[1];
    }

    // All threads: what no plan of this ordering exceeds in sum, whatever its cap: every operator in the slowest
    // way the ordering has for it (a stage's time, rounded up once, is at most the sum of its operators', each
    // rounded up), every cut at the largest output over the slowest link.
    __device__ __forceinline__ uint64_t most_sum() {
        const int tid = thread_id();
        uint64_t sum = 0;
        for (int i = tid; i < L; i += nthreads) {
            uint32_t worst = 0;
            for (int r = 0; r < n_sets * tb.n_tp; ++r) {
                const int set = r / tb.n_tp, q = r - set * tb.n_tp;
                const uint32_t tp = uint32_t(tb.tp[q]), *p = prow + r * sh.W + i;
                const uint32_t time = (p[1] - p[0] + tp - 1u) >> tb.tp_shift[q];
                worst = tp <= use[set] && time > worst ? time : worst;
            }
            sum += worst;
        }
        uint32_t cut = 0;                                  // below 2^31 on these tables
        for (int l = tid; l < 2 * K - 1; l += nthreads) {
            const int g = order[l < K ? l : l - K], h = l < K ? g : order[l - K + 1];
            const uint64_t link = uint64_t(tb.bw[int64_t(g) * tb.G + h]);
            const uint32_t c = uint32_t((tb.header->max_act + link - 1u) / link);
            cut = c > cut ? c : cut;
        }
        cut = ~group_min(~cut);
#pragma unroll
        for (int x = 32; x >= 1; x >>= 1) sum += __shfl_xor((unsigned long long)sum, x, 64);
        if (tid == 0) ok[0] = 0;                           // (the masks are made anew for every pass)
        __syncthreads();
        if ((tid & 63) == 0) atomicAdd(&ok[0], (unsigned long long)sum);
        __syncthreads();
        return ok[0] + 2ull * uint64_t(S - 1) * cut;
    }
    // 2^31 over the largest degree that a group has devices for.
    __device__ __forceinline__ uint32_t key_limit() const {
        uint32_t devices = 1;
        int degree = 1;
        for (int x = 0; x < n_sets; ++x) devices = use[x] > devices ? use[x] : devices;
        for (int q = 1; q < tb.n_tp; ++q) degree = uint32_t(tb.tp[q]) <= devices ? tb.tp[q] : degree;
        return uint32_t(uniform(int(kInfSum / uint32_t(degree))));
    }
    // The largest cap under which sums stay below 2^31: S stage and twice S transfer times of at most the cap, or
    // any cap when `most` (most_sum) does.  Key rows hold sums times a degree that a group has devices for; a pass
    // whose sums fit but not those products works from the workspace's value rows, as one does whose rows leave LDS.
    __device__ __forceinline__ int64_t largest_cap(uint64_t most, bool keys) const {
        const int64_t limit = keys ? int64_t(key_limit()) : int64_t(kInfSum);
        return most < uint64_t(limit) - 1u ? INT64_MAX : limit / (3ll * S) - 1;
    }
};

}  // namespace meshband
}  // namespace harp
