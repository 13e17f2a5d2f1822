// Passes over a fixed slicing (every stage's group and degree given by a candidate) in the ranges of cuts
// that matter under a cap, for the search over the cap of harp_plan_h1f1b_sweep_batch; k2_sweep.hip drives
// them.  Device functions called by all threads of a workgroup, one candidate at a time.
//
// It is mesh_band.h without the device index: a stage has one device offset and one degree, so the ranges
// [B, F] of the cuts behind s stages are two chains of S steps (same argument as there), and a row of the
// recurrence has one cell per cut.  All forms run in the suffix direction of the H-1F1B recurrence
// (eq. dp_ni): cell (s, i) = stages s .. S-1 hold the operators from i on.  A row is stored ready for the
// stage in front of it, as in mesh_band.h.
//
// A pass is a chain of S stages of a few dozen transitions each, so what bounds it is the latency of LDS
// and of a barrier per stage (1.5 us a stage, the ranges' chains included).  Hence: rows of the stage and transfer times in LDS where they fit
// (kResident), no feasibility index (the memory test runs on the sums in LDS: a chain would wait for a
// global load per stage), a chain step is one comparison per lane and a ballot, and kPart lanes share a
// cell's end cuts.
#pragma once

#include "fast_common.h"
#include "harp_internal.h"
#include "plan_common.h"

namespace harp {
namespace slotdp {

using fastdp::uniform;
using fastdp::wave_sync;

// 64 candidates of 82 operators and 8 to 16 stages, ms: 256 threads 1.20, 512 0.94, 1,024 0.97; 4 of those 0.63, 0.60,
// 0.63; 16 of 12 operators 0.087, 0.092, 0.103; 16 of 300 operators and up to 32 stages 12.6, 8.2, 6.3; 8 of 512 8.4, 6.4, 6.0.
constexpr int kThreads = 512;
constexpr int kTeams = kThreads / 64;            // chains worked at once, by one wavefront each
constexpr int kPart = 8;                         // lanes per cell
constexpr uint32_t kInfSum = 0x80000000u;        // values stay below this (largest_cap)
constexpr uint32_t kTopCap = 0x7FFFFFFFu;        // no time on these tables is larger
constexpr uint32_t kBitWords = 8192;             // bitmap of cap values: 262,144 of them at once
// Rows in LDS up to this many bytes of a workgroup (two workgroups per CU), else read from L2.
constexpr size_t kResidentLds = size_t(76) << 10;

struct SlotShape {
    int W, S_cap;                                // cuts (L + 1), min(S_max, L)
    uint32_t o_cap, o_stage, o_small, o_rows, o_back, o_time, o_cut, o_bits, total;
    bool resident;
};
inline SlotShape slot_shape(int L, int S_max) {
    SlotShape s;
    s.W = L + 1;
    s.S_cap = S_max < L ? S_max : L;
    const size_t W = size_t(s.W), S = size_t(s.S_cap);
    size_t at = 0;
    auto take = [&at](size_t bytes) { const size_t o = at; at += (bytes + 15) & ~size_t(15); return uint32_t(o); };
    take(2 * W * 8);                             // PP, PS
    s.o_cap = take(S * 8);
    s.o_stage = take(S * 16);
    s.o_small = take((4 * (S + 1) + 3 * S + 16) * 4 + 4 * (S + 1));
    s.o_rows = take(2 * W * 4 + 2 * W * 2);
    s.o_bits = take(size_t(kBitWords) * 4);
    const size_t without = at;
    s.o_back = take(S * W * 2);
    s.o_time = take(S * W * 4);
    s.o_cut = take(S * W * 4);
    s.resident = at <= kResidentLds;
    s.total = uint32_t(s.resident ? at : without);
    return s;
}

template <bool kResident>
struct Slots {
    static constexpr bool kChoosesSlicing = false, kGuesses = false, kSpreads = true;
    // see k2_sweep.hip; a climb passes over the values that change nothing and takes 1 to 3 passes, so kMaxClimb is a
    // bound for constructed inputs, where each of many operators of a few microseconds changes something
    static constexpr int kMaxClimb = 256;
    struct alignas(16) Stage { uint32_t row_at, cut_at; int32_t tp, shift; };
    const TablesDev &tb;
    const SlotShape &sh;
    const int32_t *cand_group, *cand_tp;
    SlotInfo &info;
    uint16_t *back_global;
    // LDS
    int64_t *mem, *capm;                         // PP [W], PS [W]; memory of a stage's submesh
    Stage *stage;
    uint16_t *F, *B;                             // [S_cap + 1]
    int32_t *cuts, *warmup, *slot_first;
    uint16_t *slot_g;
    uint8_t *slot_k;
    uint16_t *rows_of, *links_of;                // stages with a row (a link) of their own: candidate values come from these
    uint32_t *scal;
    uint32_t *h;                                 // [2][W]
    uint16_t *n;                                 // [2][W]
    uint16_t *back_lds;                          // [S_cap][W]
    uint32_t *time_lds, *cut_lds, *bits;
    int nthreads, wave;
    int S, L, n_rows, n_links;
    bool keys_fit;
    static constexpr bool reached = true;        // (guess() has looked)
    __device__ __forceinline__ int64_t bracket(int64_t) const { return -1; }
    int64_t count_cap;                           // as in mesh_band.h

    __device__ __forceinline__ Slots(const TablesDev &t, const SlotShape &s, unsigned char *lds, SlotInfo &si,
                                     const int32_t *cg, const int32_t *ct, unsigned char *slice)
        : tb(t), sh(s), cand_group(cg), cand_tp(ct), info(si), back_global(reinterpret_cast<uint16_t *>(slice)) {
        mem = reinterpret_cast<int64_t *>(lds);
        capm = reinterpret_cast<int64_t *>(lds + sh.o_cap);
        stage = reinterpret_cast<Stage *>(lds + sh.o_stage);
        scal = reinterpret_cast<uint32_t *>(lds + sh.o_small);
        cuts = reinterpret_cast<int32_t *>(scal + 16);
        warmup = cuts + (sh.S_cap + 1);
        F = reinterpret_cast<uint16_t *>(warmup + sh.S_cap);
        B = F + (sh.S_cap + 1);
        rows_of = B + (sh.S_cap + 1);
        links_of = rows_of + sh.S_cap;
        h = reinterpret_cast<uint32_t *>(lds + sh.o_rows);
        n = reinterpret_cast<uint16_t *>(h + 2 * sh.W);
        bits = reinterpret_cast<uint32_t *>(lds + sh.o_bits);
        back_lds = reinterpret_cast<uint16_t *>(lds + sh.o_back);
        time_lds = reinterpret_cast<uint32_t *>(lds + sh.o_time);
        cut_lds = reinterpret_cast<uint32_t *>(lds + sh.o_cut);
        slot_first = info.dev_first;
        slot_g = info.g;
        slot_k = info.k;
        nthreads = kThreads;
        wave = uniform(int(threadIdx.x) >> 6);
        L = tb.L;
        S = n_rows = n_links = 0;
        keys_fit = true;
        count_cap = 0;
    }
    static __device__ __forceinline__ int thread_id() { return threadIdx.x; }
    __device__ __forceinline__ int in_flight(int s) const { return (S - s) < tb.M ? (S - s) : tb.M; }
    __device__ __forceinline__ const uint32_t *time_row(int s) const {
        if constexpr (kResident) return time_lds + s * sh.W;
        else return tb.P32 + stage[s].row_at;
    }
    __device__ __forceinline__ const uint32_t *cut_row(int s) const {     // transfer times behind stage s
        if constexpr (kResident) return cut_lds + s * sh.W;
        else return tb.CM + stage[s].cut_at;
    }
    __device__ __forceinline__ uint16_t *back_row(int s) const {
        if constexpr (kResident) return back_lds + s * sh.W;
        else return back_global + size_t(s) * sh.W;
    }

    // All threads, once per kernel.
    __device__ __forceinline__ void start(bool) {
        const int64_t *PP = tb.PP(), *PS = tb.PS();
        for (int j = threadIdx.x; j <= L; j += kThreads) { mem[j] = PP[j]; mem[sh.W + j] = PS[j]; }
        __syncthreads();
    }

    // All threads: candidate c.  0; 1 when the slot list is malformed, 2 when no plan can exist.
    __device__ __forceinline__ int load_item(const OrdDev &od, int c) {
        const int tid = threadIdx.x;
        S = od.ord_S[c];
        const int64_t at = int64_t(c) * od.S_max;
        if (load_and_check_slots(tb, S, od.S_max, cand_group + at, cand_tp + at, info) != HARP_CAND_OK) return 1;
        if (S > L) return 2;
        for (int s = tid; s < S; s += kThreads) {
            const int g = slot_g[s], k = slot_k[s], to = slot_g[s + 1 < S ? s + 1 : s];
            stage[s].row_at = uint32_t((g * tb.n_tp + k) * int(tb.pitch32));
            stage[s].cut_at = uint32_t(g * tb.G + to) * uint32_t(tb.pitch32);
            stage[s].tp = tb.tp[k];
            stage[s].shift = tb.tp_shift[k];
            capm[s] = int64_t(tb.tp[k]) * tb.type_mem[tb.group_type[g]];
        }
        if (wave == 0) {
            // a row is listed once per group and degree, a link once: the slots of a group are adjacent
            int rows = 0, links = 0;
            for (int s0 = 0; s0 < S; s0 += 64) {
                const int s = s0 + tid;
                bool row = s < S, link = s + 1 < S;
                if (row)
                    for (int q = s - 1; q >= 0 && slot_g[q] == slot_g[s]; --q) row = row && slot_k[q] != slot_k[s];
                if (link && s > 0) link = !(slot_g[s - 1] == slot_g[s] && slot_g[s + 1] == slot_g[s]);
                const unsigned long long a = __ballot(row), b = __ballot(link), below = (1ull << tid) - 1ull;
                if (row) rows_of[rows + __popcll(a & below)] = uint16_t(s);
                if (link) links_of[links + __popcll(b & below)] = uint16_t(s);
                rows += __popcll(a);
                links += __popcll(b);
            }
            if (tid == 0) { scal[8] = uint32_t(rows); scal[9] = uint32_t(links); }
        }
        __syncthreads();
        n_rows = int(scal[8]);
        n_links = L < 2 ? 0 : int(scal[9]);
        if constexpr (kResident) {
            for (int s = wave; s < S; s += kTeams) {
                const uint32_t *p = tb.P32 + stage[s].row_at, *c2 = tb.CM + stage[s].cut_at;
                for (int i = tid & 63; i <= L; i += 64) {
                    time_lds[s * sh.W + i] = p[i];
                    cut_lds[s * sh.W + i] = c2[i];
                }
            }
        }
        __syncthreads();
        return 0;
    }

    // What a pass under t finds holds for every cap up to the next event: the least cap at which a comparison it
    // made with the cap comes out differently - a stage or transfer time above t that is in memory, or a
    // transfer time whose delta (eq. dp_ni) falls.  Chains and H-1F1B passes leave it in scal[12]; the values of
    // the cap below it have the same sum, so the search goes on at the first value from there on.
    __device__ __forceinline__ void note_event(uint32_t ev) const {
#pragma unroll
        for (int x = 32; x >= 1; x >>= 1) {
            const uint32_t o = __shfl_xor(ev, x, 64);
            ev = o < ev ? o : ev;
        }
        if ((threadIdx.x & 63) == 0) atomicMin(&scal[12], ev);
    }
    // The highest cap up to which the last pass, under the cap t, comes out the same.
    __device__ __forceinline__ uint32_t same_up_to(uint32_t t) const { return scal[12] > t ? scal[12] - 1u : t; }

    // One wavefront: the highest cut behind every stage that some plan under t can have; true when the last
    // stage reaches L.  Fs null: the verdict only.
    __device__ __forceinline__ bool forward_chain(uint32_t t, uint16_t *Fs, uint32_t &ev) const {
        const int lane = threadIdx.x & 63;
        const int64_t *PP = mem, *PS = mem + sh.W;
        int at = 0;
        if (Fs && lane == 0) Fs[0] = 0;
        for (int s = 0; s < S; ++s) {
            const int64_t nf = in_flight(s);
            const uint32_t *p = time_row(s);
            const uint64_t far = uint64_t(p[at]) + uint64_t(t) * uint32_t(stage[s].tp);
            const int64_t held = PP[at] + nf * PS[at], room = capm[s];
            int from = at;
            for (;;) {
                const int i = from + 1 + lane, ii = i <= L ? i : L;
                const bool ok = i <= L && uint64_t(p[ii]) <= far && PP[ii] + nf * PS[ii] - held <= room;
                const unsigned long long m = __ballot(ok);
                from += __popcll(m);
                if (m != ~0ull) break;
            }
            const int top = L - (S - 1 - s);
            if (Fs && from < top && PP[from + 1] + nf * PS[from + 1] - held <= room) {
                const uint32_t time = (p[from + 1] + uint32_t(stage[s].tp) - 1u - p[at]) >> stage[s].shift;
                ev = time < ev ? time : ev;
            }
            at = from < top ? from : top;
            if (s < S - 1) {
                // lowered to a cut whose transfer time is at most t
                const uint32_t *cut = cut_row(s);
                int found = -1;
                for (int r = at; r >= s + 1; r -= 64) {
                    const int i = r - lane;
                    const uint32_t c = cut[i >= 0 ? i : 0];
                    const unsigned long long m = __ballot(i >= s + 1 && c <= t);
                    if (m != 0) found = r - (__ffsll((long long)m) - 1);
                    if (i >= s + 1 && i > found && c < ev) ev = c;
                    if (m != 0) break;
                }
                if (found < 0) return false;
                at = found;
            }
            if (Fs && lane == 0) Fs[s + 1] = uint16_t(at);
        }
        return at == L;
    }
    // One wavefront: the lowest cut in front of every stage from which a plan under t can be completed.
    __device__ __forceinline__ bool backward_chain(uint32_t t, uint16_t *Bs, uint32_t &ev) const {
        const int lane = threadIdx.x & 63;
        const int64_t *PP = mem, *PS = mem + sh.W;
        int at = L;
        if (lane == 0) Bs[S] = uint16_t(L);
        for (int s = S - 1; s >= 0; --s) {
            const int64_t nf = in_flight(s);
            const uint32_t *p = time_row(s);
            const uint64_t far = uint64_t(t) * uint32_t(stage[s].tp);
            const uint32_t pe = p[at];
            const int64_t need = PP[at] + nf * PS[at] - capm[s];
            int from = at;
            for (;;) {
                const int j = from - 1 - lane, jj = j >= 0 ? j : 0;
                const bool ok = j >= 0 && uint64_t(pe - p[jj]) <= far && PP[jj] + nf * PS[jj] >= need;
                const unsigned long long m = __ballot(ok);
                from -= __popcll(m);
                if (m != ~0ull) break;
            }
            if (from > s && PP[from - 1] + nf * PS[from - 1] >= need) {
                const uint32_t time = (pe + uint32_t(stage[s].tp) - 1u - p[from - 1]) >> stage[s].shift;
                ev = time < ev ? time : ev;
            }
            at = from > s ? from : s;
            if (s > 0) {
                const uint32_t *cut = cut_row(s - 1);
                const int top = L - (S - s);
                int found = -1;
                for (int r = at; r <= top; r += 64) {
                    const int j = r + lane;
                    const uint32_t c = cut[j <= L ? j : L];
                    const unsigned long long m = __ballot(j <= top && c <= t);
                    if (m != 0) found = r + (__ffsll((long long)m) - 1);
                    if (j <= top && (found < 0 || j < found) && c < ev) ev = c;
                    if (m != 0) break;
                }
                if (found < 0) return false;
                at = found;
            }
            if (lane == 0) Bs[s] = uint16_t(at);
        }
        return at == 0;
    }
    // All threads: the ranges under t.  False: no plan under t.
    __device__ __forceinline__ bool prepare(uint32_t t) {
        const int lane = threadIdx.x & 63;
        __syncthreads();
        if (threadIdx.x == 0) scal[12] = 0xFFFFFFFFu;
        __syncthreads();
        uint32_t ev = 0xFFFFFFFFu;
        if (wave == 0) {
            const bool good = forward_chain(t, F, ev);
            if (lane == 0) scal[0] = good ? 1u : 0u;
            note_event(ev);
        } else if (wave == 1) {
            const bool good = backward_chain(t, B, ev);
            if (lane == 0) scal[1] = good ? 1u : 0u;
            note_event(ev);
        }
        __syncthreads();
        if (scal[0] == 0 || scal[1] == 0) return false;
        int empty = 0;
        for (int s = threadIdx.x; s <= S; s += kThreads) empty |= F[s] < B[s] ? 1 : 0;
        return !__syncthreads_or(empty);
    }

    template <int kCtrl>
    static __device__ __forceinline__ unsigned long long least_with(unsigned long long v) {
        const uint32_t lo = uint32_t(__builtin_amdgcn_update_dpp(int(uint32_t(v)), int(uint32_t(v)), kCtrl, 0xF, 0xF, false));
        const uint32_t hi = uint32_t(__builtin_amdgcn_update_dpp(int(uint32_t(v >> 32)), int(uint32_t(v >> 32)), kCtrl, 0xF, 0xF, false));
        const unsigned long long o = ((unsigned long long)hi << 32) | lo;
        return o < v ? o : v;
    }

    // The recurrence in the ranges of the last prepare under the cap t, in one of the forms below.  A cell's
    // best is one key, value << 32 | end cut << 16 | count of the stage: the least value, the lowest end cut
    // among equal ones.
    static constexpr int kMinMax = 1, kSum = 2, kH1 = 4, kAny = 0;       // (whether any plan exists: least_cap)
    template <int kForm>
    __device__ __forceinline__ int64_t pass(uint32_t t) {
        constexpr unsigned long long kNone = ~0ull;
        constexpr bool kCounts = kForm == kH1;
        const int tid = threadIdx.x, part = tid & (kPart - 1);
        const uint64_t e6 = uint64_t(count_cap) >> 6, x1 = e6 >> 1, x2 = (uint64_t(count_cap) + e6) >> 1;
        const uint32_t th1 = uint32_t(x1 < kTopCap ? x1 : kTopCap), th2 = uint32_t(x2 < kTopCap ? x2 : kTopCap);   // 2c - e > 0; > cap
        const uint32_t m_cap = uint32_t(tb.M);
        const int64_t *PP = mem, *PS = mem + sh.W;
        uint32_t ev = 0xFFFFFFFFu;
        int cur = 0;
        if (tid == 0) { h[L] = 0; n[L] = 1; }          // behind the last stage: it launches one
        for (int s = S - 1; s >= 0; --s) {
            __syncthreads();                           // row s + 1 is complete
            const int jl = B[s + 1], jh = F[s + 1], il = B[s], ih = F[s];
            const uint32_t *prev_h = h + cur * sh.W;
            const uint16_t *prev_n = n + cur * sh.W;
            uint32_t *next_h = h + (cur ^ 1) * sh.W;
            uint16_t *next_n = n + (cur ^ 1) * sh.W;
            const uint32_t *p = time_row(s);
            const uint32_t tp = uint32_t(stage[s].tp);
            const int shift = stage[s].shift;
            const int64_t room = capm[s];
            const uint32_t classic = uint32_t(in_flight(s));
            const uint32_t *cut_s = cut_row(s > 0 ? s - 1 : 0);
            uint16_t *back = back_row(s);
            for (int i0 = il; i0 <= ih; i0 += kThreads / kPart) {
                const int i = i0 + tid / kPart;
                if (i > ih) continue;                  // (all lanes of a cell together)
                const uint32_t cut = s > 0 ? cut_s[i] : 0u;
                const uint32_t xi = p[i] - tp + 1u;
                const int64_t ppi = PP[i], psi = PS[i];
                unsigned long long best = kNone;
                for (int j = (i + 1 > jl ? i + 1 : jl) + part; j <= jh; j += kPart) {
                    const uint32_t time = (p[j] - xi) >> shift;
                    if (time > t) {                    // constraint (i); grows with j
                        // (H-1F1B's counts are never below the classic one)
                        if (kCounts && (PP[j] - ppi) + int64_t(classic) * (PS[j] - psi) <= room) ev = time < ev ? time : ev;
                        break;
                    }
                    const uint32_t before = prev_h[j];
                    const uint32_t cnt = kCounts ? uint32_t(prev_n[j]) : classic;
                    const int64_t need = (PP[j] - ppi) + int64_t(cnt) * (PS[j] - psi);
                    uint32_t v;
                    if (kForm == kMinMax) v = before > time ? before : time;
                    else v = before + time;
                    const bool out = before >= kInfSum;
                    const unsigned long long key = ((unsigned long long)v << 32) | (uint32_t(j) << 16) | (kCounts ? cnt : 0u);
                    if (!out && need <= room && key < best) best = key;
                }
                best = least_with<0xB1>(best);         // lanes 1, 2 and 4 apart
                best = least_with<0x4E>(best);
                best = least_with<0x141>(best);
                if (part != 0) continue;
                const bool has = best != kNone;
                const uint32_t v = uint32_t(best >> 32), cnt0 = uint32_t(best) & 0xFFFFu;
                if (kForm != kMinMax) back[i] = uint16_t(uint32_t(best) >> 16);
                if (s > 0) {
                    const bool in = has && cut <= t;   // constraint (ii)
                    const uint32_t w = kForm == kMinMax ? (v > cut ? v : cut) : v + 2u * cut;
                    next_h[i] = in && w < kInfSum ? w : kInfSum;
                    if (kCounts) {
                        const uint32_t cnt = 1u + (cut > th1 ? 1u : 0u) + (cut > th2 ? 1u : 0u) + cnt0;   // eq. dp_ni
                        next_n[i] = uint16_t(cnt < m_cap ? cnt : m_cap);
                    }
                    if (kCounts && has) {
                        // the cap that admits the cut, or at which its delta falls: 2c - e <= 0 from 128 c on,
                        // 2c - e <= cap no earlier than at 128 c / 65
                        uint64_t at = ~0ull;
                        if (cut > t) at = cut;
                        else if (cut > th2) at = 128ull * cut / 65u;
                        else if (cut > th1) at = 128ull * cut;
                        at = at > t ? at : t + 1u;
                        ev = at < ev ? uint32_t(at) : ev;
                    }
                } else {
                    scal[4] = has ? v : kInfSum;
                }
            }
            cur ^= 1;
        }
        if (kCounts) note_event(ev);
        __syncthreads();
        const uint32_t v = scal[4];
        return v >= kInfSum ? kInf : int64_t(v);
    }
    // The least-count pass under the cap t on one wavefront, ranges included, in `mine` (team_words words of LDS): whether any
    // plan exists under t (a smaller count weakens every memory test in front of it).  ev: as for the passes of the workgroup.
    __device__ __forceinline__ uint32_t team_words() const { return (uint32_t(2 * sh.W) + uint32_t(2 * (sh.S_cap + 1)) + 3u) / 2u + 1u; }
    __device__ __forceinline__ bool any_plan(uint32_t t, uint32_t *mine, uint32_t &ev) const {
        const int lane = threadIdx.x & 63, part = lane & (kPart - 1);
        uint16_t *rows = reinterpret_cast<uint16_t *>(mine + 1), *Fs = rows + 2 * sh.W, *Bs = Fs + (sh.S_cap + 1);
        ev = 0xFFFFFFFFu;
        if (!forward_chain(t, Fs, ev) || !backward_chain(t, Bs, ev)) return false;
        wave_sync();
        const uint64_t e6 = uint64_t(t) >> 6, x1 = e6 >> 1, x2 = (uint64_t(t) + e6) >> 1;
        const uint32_t th1 = uint32_t(x1 < kTopCap ? x1 : kTopCap), th2 = uint32_t(x2 < kTopCap ? x2 : kTopCap);
        const uint32_t m_cap = uint32_t(tb.M);
        const int64_t *PP = mem, *PS = mem + sh.W;
        bool found = false;
        int cur = 0;
        if (lane == 0) rows[L] = 1;
        for (int s = S - 1; s >= 0; --s) {
            wave_sync();
            const int jl = uniform(Bs[s + 1]), jh = uniform(Fs[s + 1]), il = uniform(Bs[s]), ih = uniform(Fs[s]);
            if (jl > jh || il > ih) return false;
            const uint16_t *prev = rows + cur * sh.W;
            uint16_t *next = rows + (cur ^ 1) * sh.W;
            const uint32_t *p = time_row(s), *cut_s = cut_row(s > 0 ? s - 1 : 0);
            const uint32_t tp = uint32_t(stage[s].tp), classic = uint32_t(in_flight(s));
            const int shift = stage[s].shift;
            const int64_t room = capm[s];
            for (int i0 = il; i0 <= ih; i0 += 64 / kPart) {
                const int i = i0 + lane / kPart;
                if (i > ih) continue;                  // (all lanes of a cell together)
                const uint32_t cut = s > 0 ? cut_s[i] : 0u;
                const uint32_t xi = p[i] - tp + 1u;
                const int64_t ppi = PP[i], psi = PS[i];
                uint32_t best = 0xFFFFu;
                for (int j = (i + 1 > jl ? i + 1 : jl) + part; j <= jh; j += kPart) {
                    const uint32_t time = (p[j] - xi) >> shift;
                    const int64_t held = PP[j] - ppi, stash = PS[j] - psi;
                    if (time > t) {
                        if (held + int64_t(classic) * stash <= room) ev = time < ev ? time : ev;
                        break;
                    }
                    const uint32_t cnt = prev[j];      // (0xFFFF: no plan from there)
                    if (cnt < best && held + int64_t(cnt) * stash <= room) best = cnt;
                }
                best = least32<0xB1>(best);            // lanes 1, 2 and 4 apart
                best = least32<0x4E>(best);
                best = least32<0x141>(best);
                if (part != 0) continue;
                const bool has = best != 0xFFFFu;
                if (s == 0) { found = has; continue; }
                const uint32_t cnt = 1u + (cut > th1 ? 1u : 0u) + (cut > th2 ? 1u : 0u) + best, capped = cnt < m_cap ? cnt : m_cap;
                next[i] = uint16_t(has && cut <= t ? capped : 0xFFFFu);
                if (has) {
                    uint64_t at = ~0ull;
                    if (cut > t) at = cut;
                    else if (cut > th2) at = 128ull * cut / 65u;
                    else if (cut > th1) at = 128ull * cut;
                    at = at > t ? at : t + 1u;
                    ev = at < ev ? uint32_t(at) : ev;
                }
            }
            cur ^= 1;
        }
        return __any(found);
    }
    template <int kCtrl>
    static __device__ __forceinline__ uint32_t least32(uint32_t v) {
        const uint32_t o = uint32_t(__builtin_amdgcn_update_dpp(int(v), int(v), kCtrl, 0xF, 0xF, false));
        return o < v ? o : v;
    }
    // All threads: whether any cap up to `top` has a plan; if so the lowest that can have one lies above lo and not above hi,
    // which come within 1/4,096 of each other.  lo: no plan up to there.  Every wavefront tries a cap of its own, at
    // distances that grow by four first, evenly spread then: a pass is as long as its stages are one after the other, whoever
    // works it.  One cap after the other on the whole workgroup took up to twenty passes: 64 candidates of 40 operators
    // 884 -> 793 us, 64 of 82 with tight memory 588 -> 471, 16 of 12 operators 188 -> 127.
    __device__ __forceinline__ bool least_cap(uint32_t top, uint32_t &lo, uint32_t &hi) {
        // (six at least: sequences of up to 1,024 operators and 256 stages come here)
        const int fit = int(kBitWords / team_words()), lane = threadIdx.x & 63, n = fit < kTeams ? fit : kTeams;
        uint32_t *mine = bits + uint32_t(wave < n ? wave : 0) * team_words();
        const uint64_t step = (lo >> 4) + 1u;
        hi = 0;                                        // (none known)
        for (bool first = true; first || (lo < hi && hi - lo > 1u + (hi >> 12)); first = false) {
            auto cap_of = [&](int w) -> uint32_t {
                if (first) {
                    const uint64_t t = lo + (step << (2 * w));
                    return w == n - 1 || t > top ? top : uint32_t(t);
                }
                return lo + uint32_t(uint64_t(hi - lo) * uint32_t(w + 1) / uint32_t(n + 1));
            };
            __syncthreads();
            if (wave < n) {
                uint32_t ev;
                const bool found = any_plan(cap_of(wave), mine, ev);
                ev = fastdp::wave_least(ev);
                if (lane == 0) { scal[wave] = found ? 1u : 0u; mine[0] = ev; }
            }
            __syncthreads();
            // the verdict never changes back as the cap grows
            int w = 0;
            while (w < n && scal[w] == 0) ++w;
            if (first && w == n) return false;
            uint32_t low = lo;
            if (w > 0) {
                const uint32_t t = cap_of(w - 1), e = bits[uint32_t(w - 1) * team_words()];
                low = e > t ? e - 1u : t;
            }
            if (w < n) hi = cap_of(w);
            lo = low > lo ? low : lo;
        }
        return true;
    }

    // One pass under the cap t; kInf without a plan.  kForms: the forms a kernel uses, as a mask.
    template <int kForms>
    __device__ __forceinline__ int64_t run(int form, uint32_t t) {
        if (!prepare(t)) return kInf;
        if ((kForms & kMinMax) && form == kMinMax) return pass<kMinMax>(t);
        if ((kForms & kSum) && form == kSum) return pass<kSum>(t);
        if (kForms & kH1) return pass<kH1>(t);
        return kInf;
    }

    // All threads: the cuts of the last least-sum pass, along its back-pointers.
    __device__ __forceinline__ void find_plan(bool, uint32_t, uint32_t) {
        if (threadIdx.x == 0) {
            int i = 0;
            for (int s = 0; s < S; ++s) {
                cuts[s] = i;
                const int j = back_row(s)[i];
                i = j <= L ? j : L;                    // a finite sum only chains through cells
            }
            cuts[S] = L;
        }
        __syncthreads();
    }
    // All threads: the plan of the last H-1F1B pass, with its counts by eq. Ni.
    __device__ __forceinline__ void find_h1_plan() {
        find_plan(true, 0, 0);
        if (wave == 0) {
            const uint64_t e6 = uint64_t(count_cap) >> 6;
            for (int s = threadIdx.x; s < S; s += 64) {
                const uint32_t cut = s < S - 1 ? cut_row(s)[cuts[s + 1]] : 0u;
                warmup[s] = 1 + (2ull * cut > e6 ? 1 : 0) + (2ull * cut > uint64_t(count_cap) + e6 ? 1 : 0);
            }
            wave_sync();
            if (threadIdx.x == 0) {
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
    // All threads: bottleneck of the plan in cuts (scored: LDS).
    __device__ __forceinline__ void score(int64_t *scored, int64_t &bott, int64_t &) const {
        if (wave == 0) {
            uint32_t worst = 0;
            for (int s = threadIdx.x; s < S; s += 64) {
                const int j = cuts[s], i = cuts[s + 1];
                const uint32_t *p = time_row(s);
                const uint32_t time = (p[i] + uint32_t(stage[s].tp) - 1u - p[j]) >> stage[s].shift;
                const uint32_t cut = s < S - 1 ? cut_row(s)[i] : 0u;
                worst = time > worst ? time : worst;
                worst = cut > worst ? cut : worst;
            }
#pragma unroll
            for (int x = 32; x >= 1; x >>= 1) {
                const uint32_t o = __shfl_xor(worst, x, 64);
                worst = o > worst ? o : worst;
            }
            if (threadIdx.x == 0) scored[0] = int64_t(worst);
        }
        __syncthreads();
        bott = scored[0];
    }
    __device__ __forceinline__ void write_slots(const PlansDev &out, int c, int S_max, int32_t *, int32_t *) const {
        int32_t *sp = out.splits + int64_t(c) * (S_max + 1), *df = out.dev_first + int64_t(c) * S_max;
        for (int s = threadIdx.x; s <= S_max; s += kThreads) sp[s] = s <= S ? cuts[s] : -1;
        for (int s = threadIdx.x; s < S_max; s += kThreads) df[s] = s < S ? slot_first[s] : -1;
    }

    // All threads: the first cap to try the min-max pass under; -1 when no plan exists under any.  As in
    // mesh_band.h, with kTeams caps at once: the speeds of the stages give a first guess, the cheapest cut on
    // every link a bound from below.
    __device__ __forceinline__ int64_t guess() {
        const int tid = threadIdx.x, lane = tid & 63;
        if (tid == 0) scal[6] = 0;
        __syncthreads();
        for (int s = wave; s + 1 < S; s += kTeams) {
            const uint32_t *cut = cut_row(s);
            uint32_t low = kTopCap;
            for (int i = 1 + lane; i < L; i += 64) low = cut[i] < low ? cut[i] : low;
#pragma unroll
            for (int x = 32; x >= 1; x >>= 1) {
                const uint32_t o = __shfl_xor(low, x, 64);
                low = o < low ? o : low;
            }
            if (lane == 0) atomicMax(&scal[6], low);
        }
        if (wave == 0) {
            float share = 0.f;
            for (int s = lane; s < S; s += 64) {
                const float whole = float(time_row(s)[L]) / float(stage[s].tp);
                share += 1.f / (whole > 1.f ? whole : 1.f);
            }
#pragma unroll
            for (int x = 32; x >= 1; x >>= 1) share += __shfl_xor(share, x, 64);
            const float guess = 1.f / share;
            if (lane == 0) scal[5] = guess < 1.f ? 1u : guess > 1e9f ? 1000000000u : uint32_t(guess);
        }
        __syncthreads();
        const int64_t bound = scal[6], g = int64_t(scal[5]) > bound ? int64_t(scal[5]) : bound;
        int64_t bad = bound - 1, good = -1;                // largest t known to have no plan, smallest t whose chain succeeds
        for (int round = 0; good < 0 || good - bad > good / 12 + 1; ++round) {
            int64_t at[kTeams];
#pragma unroll
            for (int w = 0; w < kTeams; ++w) {
                const int step = round * kTeams + w;
                int64_t t;
                if (good >= 0) t = bad + (good - bad) * (w + 1) / (kTeams + 1);
                else t = step == 0 ? g : step == 1 ? g + g * 7 / 32 + 1 : step == 2 ? g + g * 5 / 8 + 1 : step == 3 ? 5 * g / 2 + 1
                         : step == 4 ? 8 * g + 1 : step == 5 ? 64 * g + 1 : int64_t(kTopCap);
                at[w] = t < int64_t(kTopCap) ? t : int64_t(kTopCap);
            }
            __syncthreads();
            int64_t mine = at[0];
#pragma unroll
            for (int w = 1; w < kTeams; ++w) mine = wave == w ? at[w] : mine;
            uint32_t unused = 0xFFFFFFFFu;
            const bool fine = forward_chain(uint32_t(mine), nullptr, unused);
            if (lane == 0) scal[wave] = fine ? 1u : 0u;
            __syncthreads();
#pragma unroll
            for (int w = kTeams - 1; w >= 0; --w)
                if (scal[w] != 0) good = at[w];
#pragma unroll
            for (int w = 0; w < kTeams; ++w)
                if (scal[w] == 0 && at[w] > bad) bad = at[w];
            __syncthreads();
            if (good < 0 && bad >= int64_t(kTopCap)) return -1;           // no plan under any cap
            if (good == g) break;                                          // near enough
        }
        return good;
    }
    // Steps as in mesh_band.h.
    static __device__ __forceinline__ uint32_t raised(uint32_t t, int tries) {
        return tries < 2 && t < kTopCap / 2 ? t + (t >> (3 - tries)) + 1u : kTopCap;
    }

    // Candidate caps of the candidate (section 5.2.4 (2)): every stage time of a slot over any operator range,
    // every transfer time of an inner cut between consecutive slots.  All threads: visit(v) for every one in
    // (a, b], repetitions included; a thread's `beyond` becomes the least value above b it has seen.
    template <typename VisitFn>
    __device__ __forceinline__ void visit_values(uint32_t a, uint32_t b, uint32_t &beyond, VisitFn visit) const {
        const int tid = threadIdx.x;
        const int top_step = 1 << (31 - __clz(L));
        for (int x = tid; x < n_rows * L; x += kThreads) {
            const int r = x / L, j = x - r * L, s = rows_of[r];
            const uint32_t tp = uint32_t(stage[s].tp);
            const int shift = stage[s].shift;
            const uint32_t *p = time_row(s);
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
        for (int x = tid; x < n_links * (L - 1); x += kThreads) {
            const int l = x / (L - 1), i = 1 + x - l * (L - 1);
            const uint32_t v = cut_row(links_of[l])[i];
            if (v > b) beyond = v < beyond ? v : beyond;
            else if (v > a) visit(v);
        }
    }
    // All threads: a workgroup-wide minimum through LDS
    __device__ __forceinline__ uint32_t group_min(uint32_t v) {
        const int tid = threadIdx.x;
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
    // All threads: the smallest candidate cap above a; 0xFFFFFFFF when there is none.
    __device__ __forceinline__ uint32_t next_value(uint32_t a) {
        uint32_t beyond = 0xFFFFFFFFu;
        visit_values(a, a, beyond, [](uint32_t) {});
        return group_min(beyond);
    }
    // All threads: the largest candidate cap.
    __device__ __forceinline__ uint32_t largest_value() {
        uint32_t most = 0;
        for (int r = threadIdx.x; r < n_rows; r += kThreads) {
            const int s = rows_of[r];
            const uint32_t v = (time_row(s)[L] + uint32_t(stage[s].tp) - 1u) >> stage[s].shift;
            most = v > most ? v : most;
        }
        for (int x = threadIdx.x; x < n_links * (L - 1); x += kThreads) {
            const int l = x / (L - 1), i = 1 + x - l * (L - 1);
            const uint32_t v = cut_row(links_of[l])[i];
            most = v > most ? v : most;
        }
        return ~group_min(~most);
    }
    // All threads: how many distinct candidate caps lie in (a, b], counted up to `limit`; `last` becomes the
    // limit-th of them when there are that many.  A bitmap over a window of values, window after window, each
    // starting at the next value there is.
    __device__ __forceinline__ uint32_t count_values(uint32_t a, uint32_t b, uint32_t limit, uint32_t &last) {
        const int tid = threadIdx.x;
        constexpr uint32_t span = kBitWords * 32u;
        uint32_t found = 0, from = a + 1u;
        while (from <= b && found < limit) {
            const uint32_t to = b - from < span ? b : from + (span - 1u);
            __syncthreads();
            for (uint32_t w = tid; w < kBitWords; w += kThreads) bits[w] = 0;
            __syncthreads();
            uint32_t beyond = 0xFFFFFFFFu;
            visit_values(from - 1u, to, beyond, [&](uint32_t v) {
                const uint32_t at = v - from;
                atomicOr(&bits[at >> 5], 1u << (at & 31u));
            });
            const uint32_t next = group_min(beyond);       // (its barriers complete the bitmap)
            uint32_t mine = 0;
            for (uint32_t w = tid; w < kBitWords; w += kThreads) mine += __popc(bits[w]);
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
                    uint32_t left = limit - found;
                    for (uint32_t w0 = 0; w0 < kBitWords; w0 += 64) {
                        const uint32_t v = bits[w0 + tid];
                        uint32_t inc = __popc(v);
#pragma unroll
                        for (int x = 1; x < 64; x <<= 1) {
                            const uint32_t o = __shfl_up(inc, x, 64);
                            if (tid >= x) inc += o;
                        }
                        const uint32_t all = __shfl(inc, 63, 64);
                        if (left > all) { left -= all; continue; }
                        const uint32_t before = inc - __popc(v);
                        if (before < left && left <= inc) {
                            uint32_t rest = v;
                            for (uint32_t k = left - before; k > 1; --k) rest &= rest - 1u;
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

    // All threads: what no plan of this candidate exceeds in sum, whatever its cap: every operator on its
    // slowest stage, every cut at its link's dearest.
    __device__ __forceinline__ uint64_t most_sum() {
        const int tid = threadIdx.x;
        uint64_t sum = 0;
        for (int i = tid; i < L; i += kThreads) {
            uint32_t worst = 0;
            for (int r = 0; r < n_rows; ++r) {
                const int s = rows_of[r];
                const uint32_t *p = time_row(s) + i;
                const uint32_t time = (p[1] - p[0] + uint32_t(stage[s].tp) - 1u) >> stage[s].shift;
                worst = time > worst ? time : worst;
            }
            sum += worst;
        }
        uint32_t cut = 0;
        for (int x = tid; x < n_links * (L - 1); x += kThreads) {
            const int l = x / (L - 1), i = 1 + x - l * (L - 1);
            const uint32_t c = cut_row(links_of[l])[i];
            cut = c > cut ? c : cut;
        }
        cut = ~group_min(~cut);
#pragma unroll
        for (int x = 32; x >= 1; x >>= 1) sum += __shfl_xor((unsigned long long)sum, x, 64);
        unsigned long long *total = reinterpret_cast<unsigned long long *>(scal + 10);
        if (tid == 0) *total = 0;
        __syncthreads();
        if ((tid & 63) == 0) atomicAdd(total, (unsigned long long)sum);
        __syncthreads();
        const uint64_t most = *total + 2ull * uint64_t(S - 1) * cut;
        __syncthreads();
        return most;
    }
    // The largest cap under which sums stay below 2^31: S stage and twice S transfer times of at most the cap,
    // or any cap when `most` (most_sum) does.
    __device__ __forceinline__ int64_t largest_cap(uint64_t most, bool) const {
        return most < uint64_t(kInfSum) - 1u ? INT64_MAX : int64_t(kInfSum) / (3ll * S) - 1;
    }
};

}  // namespace slotdp
}  // namespace harp
