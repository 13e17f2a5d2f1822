// The capped recurrence with H-1F1B warm-up counts (paper sections 4.1 and 5.2.3), 32-bit path.
//
// Under H-1F1B the last stage launches one forward microbatch during warm-up and every earlier
// stage launches delta more than the stage after it (eq. Ni), with delta in {1, 2, 3} growing with
// the transfer time of the cut between them relative to the cap t_max (eq. dp_ni; integer form:
// slack = t_max / 64 rounded down, delta = 1 if 2c <= slack, 2 if 2c - slack <= t_max, else 3).
// A stage's memory need depends on its count (eq. mem_cons), and the count depends on everything
// behind the stage, so the recurrence runs in the paper's own suffix direction (eq. dp_general):
// the state "the last stages, from slot sigma on, start at operator i" holds the least sum of
// (t + 2c) under the cap and carries the warm-up count of its first stage as determined by the
// continuation that attained the least sum.  Counts never exceed the number of microbatches.
//
// Mapping: one wavefront per live candidate at a time (64-thread workgroups), one lane per cell
// of the current slot's reachability band (the bands of the pre-pass were computed with the classic
// 1F1B counts, which are never larger than H-1F1B's, so they remain outer bounds), rows in LDS that
// hold the cuts one slot touches; a candidate whose widest slot does not fit the wavefront's LDS
// share is queued for a second launch with one 256-thread workgroup per candidate and rows over the
// whole sequence, which is also the form the 64-bit instantiation has.
// The row handed from slot sigma+1 to slot sigma is stored ready for use: entry j holds the
// suffix sum plus twice the transfer time of the cut at j (infinity when that transfer exceeds the
// cap) and the count the stage in front of j would have, so a transition is one stage time, one
// memory test and one add.  Scans run upwards in j with a strict comparison, which keeps the lowest j
// among equal sums; the stage time grows with j and stops the scan at the cap, and the scan ends at
// the highest end cut that fits with the slot's classic count (from the pre-pass's feasibility
// index: a larger count cannot fit where the classic one does not).
//
// Sums are 32-bit while they stay below 2^31 - 1 - cap, so that a stored sum plus any admissible
// stage time cannot reach infinity (2^31); a candidate for which some cell would exceed that is
// queued and redone by the instantiation with 64-bit sums.
#include <type_traits>

#include "fast_common.h"
#include "harp_internal.h"
#include "plan_common.h"

namespace harp {

using namespace fastdp;

namespace {

constexpr size_t kLdsGranule = 1280;     // LDS is allocated in units of this many bytes
constexpr int kTail = 4;     // spare entries behind a row: a group of four may overrun the band

template <typename SumT> struct H1Traits;
template <> struct H1Traits<uint32_t> {
    static constexpr uint32_t inf = 0x80000000u;
    struct alignas(8) Entry { uint32_t h; float nn; };
};
template <> struct H1Traits<uint64_t> {
    static constexpr uint64_t inf = uint64_t(1) << 62;
    struct alignas(16) Entry { uint64_t h; float nn; uint32_t unused; };
};

// The memory test of a transition, eq. mem_cons, is a 64-bit sum with a 64 x 32 multiply, half of what a
// transition costs in 64-bit integers.  It runs in float on running sums rounded to float (counts, at most
// 3 S, are exact in float): the need comes out within a bound E of the true one, so a need of at most
// cap - E fits and one above cap + E does not.  A transition is taken up to cap + E, and where the need of the one a cell
// ends with is above cap - E the cell is worked again in 64 bits, on the sums in global memory (any other transition is
// either refused for certain or no better, whether it fits or not).  512 operators, 65,536 candidates, loose
// memory: 18.1 -> 14.1 ms, 160 operators 1.60 -> 1.47.
// What end cut j puts into the need, P[j] + n Q[j] with n the count of its entry, is worked out once when the entry is
// made and sits in a row of its own; cut i adds P[i] to the limits and n Q[i] in one fused operation: 9 vector
// instructions a transition for 14 (us a call: 160 operators, 65,536 candidates 1,452 -> 1,249; 512 operators, 65,536, loose
// memory 15,107 -> 13,374, tight 1,995 -> 1,736; 307 operators, degrees 1 2 3 6, 1,531 -> 1,241; the scans are bound by the
// issue of vector instructions).  Measured and left: the least of four first and its place found after the scan (1,279
// for 1,250), the reach requested a slot ahead (1,260 for 1,250).  With u = 2^-24, P
// and Q the whole sums of parameter and stash bytes and n the largest count: rounding two sums each (sum_f), 6 u P and
// 6 u n Q; the two fused operations, 2 u (P + n Q); the limits with P[i], u P; the cap, 3 u cap.
// E = 16 u (P + n Q) + 4 u cap.
struct alignas(8) MemPair { float pp, ps; };
// 0 <= v < 2^63 as a float, off by less than 3 u v: the halves (either is rounded to 24 bits) and their sum
__device__ __forceinline__ float sum_f(int64_t v) {
    return fmaf(float(uint32_t(uint64_t(v) >> 32)), 4294967296.f, float(uint32_t(v)));
}

// c <= cap, so the quotient of eq. dp_ni is 0, 1 or 2 and needs no division.
__device__ __forceinline__ uint32_t h1f1b_delta(uint32_t c, int64_t cap) {
    const int64_t x = 2 * int64_t(c) - (cap >> 6);
    return 1u + (x > 0 ? 1u : 0u) + (x > cap ? 1u : 0u);
}

// LDS in front of the rows: per-slot constants, two scalars, band and trial cuts, two flags, the
// wavefronts' ranges of finite sums, index-row offsets, the plan's deltas
__host__ __device__ inline size_t h1f1b_small_bytes(int S_max) {
    const size_t b = size_t(S_max) * sizeof(StageConst) + 16 + size_t(S_max + 1) * 8 + 8 + 64 + size_t(S_max) * 8;
    return (b + 15) & ~size_t(15);
}
// bytes per cut of the rows in LDS when every row is sized for one slot: two rows of entries, two of needs, one of times
__host__ __device__ inline size_t h1f1b_cut_bytes(size_t entry) { return 2 * entry + 2 * sizeof(float) + 4; }

// counts: [0] live, [1] dead, [2] queued for 64-bit sums, [7] ticket of the 64-bit kernel, [10] candidates queued for rows over the whole sequence, [11] next item of that list.
// Both queues sit in the unused tail of the dead list, the 64-bit one from its front, the other from
// its back.
//
// kMode 0: a workgroup per candidate, LDS rows with an entry for every cut.  kMode 1: a wavefront
// per candidate (64-thread workgroups), LDS rows that hold the cuts one slot touches (a slot's cells
// and continuations: B[slot] .. F[slot+1]), sized for the candidate's widest slot; a candidate that
// does not fit is queued.  kMode 2: as 0, on the candidates queued by 1.
template <typename SumT, int kMode, bool kOdd>
__device__ __forceinline__ void h1f1b_body(const TablesDev &tb, const CandDev &cd, const int64_t *t_max,
                                           const PlansDev &out, int32_t *warmup, int *counts, int *tickets,
                                           const int32_t *live_list, uint32_t *dead_list,
                                           const uint32_t *bands, const uint16_t *hi_tab, int idx_pitch,
                                           unsigned char *arg_base, size_t arg_per_group, int row_len,
                                           int arg_pitch) {
    using Entry = typename H1Traits<SumT>::Entry;
    constexpr SumT kInfSum = H1Traits<SumT>::inf;
    constexpr bool kWide = sizeof(SumT) == 8;
    constexpr bool kBandRows = kMode == 1;
    extern __shared__ __align__(16) unsigned char lds_raw[];

    const int L = tb.L, S_max = cd.S_max;
    const int tid = threadIdx.x, lane = tid & 63, nthreads = blockDim.x;
    const int wave = uniform(tid >> 6);
    StageConst *sc = reinterpret_cast<StageConst *>(lds_raw);                          // [S_max]
    uint64_t *scal = reinterpret_cast<uint64_t *>(sc + S_max);                         // [2]
    uint32_t *band = reinterpret_cast<uint32_t *>(scal + 2);                           // [S_max + 1]
    int32_t *trial = reinterpret_cast<int32_t *>(band + S_max + 1);                    // [S_max + 1]
    uint32_t *flags = reinterpret_cast<uint32_t *>(trial + S_max + 1);                 // [2]: ticket, overflow
    // element offset of each slot's row of the feasibility index: the highest end cut that fits with the
    // classic count of the slot, an outer bound for H-1F1B's (its counts are never below the classic ones)
    int32_t *fin_w = reinterpret_cast<int32_t *>(flags + 2);                           // [2][4][2]: per slot parity and wavefront, lowest and highest cell with a finite sum
    uint32_t *hi_off = reinterpret_cast<uint32_t *>(fin_w + 16);                       // [S_max]
    uint32_t *deltas = hi_off + S_max;                                                 // [S_max]
    // Rows of row_len entries.  Whole-sequence form: two rows of entries, two of needs, two of times;
    // entry x of a row is cut x.  Slot-sized form: a row's entry 0 is the lowest cut of the
    // slot it serves, and the times of the slot in front take the place of this
    // slot's once its cells are done (one wavefront: its LDS operations execute in order).
    Entry *rows0 = reinterpret_cast<Entry *>(lds_raw + h1f1b_small_bytes(S_max));
    Entry *rows1 = rows0 + row_len;
    float *needs0 = reinterpret_cast<float *>(rows1 + row_len), *needs1 = needs0 + row_len;
    uint32_t *prow0 = reinterpret_cast<uint32_t *>(needs1 + row_len);
    uint32_t *prow1 = kBandRows ? prow0 : prow0 + row_len;
    uint16_t *arg = reinterpret_cast<uint16_t *>(arg_base + size_t(blockIdx.x) * arg_per_group);
    const int n_dead = counts[1];
    const int n_items = kWide ? counts[2] : kMode == 2 ? counts[10] : counts[0];
    int *next_item = counts + (kWide ? 7 : 11);
    Draw items(tickets, kTicketH1f1b, n_items, int(gridDim.x));
    if (!kBandRows && int(blockIdx.x) >= n_items) return;      // mostly nothing is queued: no ticket to draw (25 us)
    const int64_t m_cap = tb.M;
    const int64_t *PP = tb.PP(), *PS = tb.PS();

    auto sums_at = [&](int x) { return MemPair{sum_f(PP[x]), sum_f(PS[x])}; };
    if (!kBandRows)
        for (int j = L + 1 + tid; j < row_len; j += nthreads) { prow0[j] = 0; prow1[j] = 0; }

    for (;;) {
        __syncthreads();   // the previous candidate's tail has finished with LDS
        int n;
        if constexpr (kBandRows) {
            n = items.next(int(blockIdx.x));
            if (n < 0) break;
            if (tid == 0) flags[1] = 0;
        } else {
            if (tid == 0) { flags[0] = (uint32_t)atomicAdd(next_item, 1); flags[1] = 0; }
            __syncthreads();
            n = uniform((int)flags[0]);
            if (n >= n_items) break;
        }
        const int c = kWide ? int(dead_list[n_dead + n]) : kMode == 2 ? int(dead_list[cd.C - 1 - n]) : live_list[n];
        const int S = cd.cand_S[c];
        const int64_t cap64 = t_max[c];
        int32_t *sp = out.splits + int64_t(c) * (S_max + 1);
        int32_t *df = out.dev_first + int64_t(c) * S_max;
        int32_t *wu = warmup + int64_t(c) * S_max;
        if (cap64 < 0 || cap_out_of_range(tb, cap64)) {   // no time fits under a negative cap; too large a cap is refused
            write_failed(out, c, S_max, cap64 < 0 ? HARP_CAND_INFEASIBLE : HARP_CAND_INVALID);
            for (int s = tid; s < S_max; s += nthreads) wu[s] = -1;
            continue;
        }
        const uint32_t tcap = (uint32_t)(cap64 > 0x7FFFFFFFll ? 0x7FFFFFFFll : cap64);   // no time here is larger
        {
            const int32_t *grp = cd.cand_group + int64_t(c) * S_max;
            const int32_t *tpv = cd.cand_tp + int64_t(c) * S_max;
            for (int s = tid; s < S; s += nthreads) {
                const int g = grp[s], k = tp_index(tb, tpv[s]);
                const int g_next = s + 1 < S ? grp[s + 1] : g;
                sc[s].cap = int64_t(tb.tp[k]) * tb.type_mem[tb.group_type[g]];
                sc[s].p_row = uint32_t((int64_t(g) * tb.n_tp + k) * tb.pitch32);
                sc[s].cm_row_shift = uint32_t((int64_t(g) * tb.G + g_next) * tb.pitch32) |
                                     (tp_code<kOdd>(tb, k) << 27);
                int32_t first = tb.group_base[g];
                for (int q = s - 1; q >= 0 && grp[q] == g; --q) first += tpv[q];
                df[s] = first;
                const int n_classic = int((S - s) < m_cap ? (S - s) : m_cap);
                hi_off[s] = uint32_t((int64_t(n_classic - 1) * tb.T * tb.n_tp + int64_t(tb.group_type[g]) * tb.n_tp + k) *
                                     idx_pitch);
            }
            for (int s = S + tid; s < S_max; s += nthreads) df[s] = -1;
            for (int s = tid; s <= S; s += nthreads) band[s] = bands[int64_t(c) * (S_max + 1) + s];
        }
        const int64_t most_n = m_cap < 3 * int64_t(S) ? m_cap : 3 * int64_t(S);
        const float need_err = (float(PP[L]) + float(most_n) * float(PS[L])) * (16.f / 16777216.f);
        // stored sums stay this small, so that adding an admissible stage time cannot reach infinity
        const uint64_t limit = kWide ? uint64_t(kInfSum) - 1 : uint64_t(kInfSum) - 1 - tcap;
        __syncthreads();          // slot constants and bands are in LDS
        if (kBandRows) {
            // a slot touches its cells and its continuations, B[slot] .. F[slot+1], and up to kTail
            // entries behind them
            int span = 0;
            for (int s = tid; s < S; s += nthreads) {
                const int w = band_hi(band[s + 1]) - (s == 0 ? 0 : band_lo(band[s])) + 1;
                span = w > span ? w : span;
            }
            span = int(wave_all(uint32_t(span), max2));
            if (span + kTail > row_len) {
                if (tid == 0) dead_list[cd.C - 1 - atomicAdd(&counts[10], 1)] = uint32_t(c);
                continue;
            }
        }
        // prologue: behind the last stage no operators are left and nothing is launched yet (the last
        // stage itself adds delta(0) = 1); the fused time row of the last slot over its cells and its
        // single continuation
        MemPair sums_n{0.f, 0.f};            // memory sums at this lane's first cell of the slot to come
        {
            const int il0 = (S == 1) ? 0 : band_lo((uint32_t)uniform((int)band[S - 1]));
            Entry *row_S = rows0 - (kBandRows ? L : 0);
            if (tid == 0) {
                const MemPair all = sums_at(L);
                row_S[L].h = 0;
                row_S[L].nn = 1.f;
                (needs0 - (kBandRows ? L : 0))[L] = all.pp + all.ps;
            }
            if (tid >= 1 && tid <= kTail) row_S[L + tid].h = kInfSum;
            const uint32_t *p32 = tb.P32 + (uint32_t)uniform((int)sc[S - 1].p_row);
            uint32_t *pr = prow0 - (kBandRows ? il0 : 0);
            for (int x = il0 + tid; x <= L; x += nthreads) pr[x] = p32[x];
            if (il0 + tid <= L) sums_n = sums_at(il0 + tid);
        }
        lds_barrier();
        int cur = 0, pcur = 0;
        const int wave_first = wave * 64;
        // Continuations with a finite sum lie in [fin_lo, fin_hi]: scans are clamped to that range,
        // which changes no value, and a row without a finite sum ends the candidate - no plan - at
        // once.  Every wavefront keeps the range of its own cells (one ballot per round of cells); a
        // workgroup's wavefronts exchange theirs through LDS at the barrier that ends a slot.
        int fin_lo = L, fin_hi = L;
        auto end_of_slot = [&](int slot, int new_lo, int new_hi) -> bool {      // true: no continuation is left
            if (!kBandRows && lane == 0) {
                fin_w[((slot & 1) * 4 + wave) * 2] = new_lo;
                fin_w[((slot & 1) * 4 + wave) * 2 + 1] = new_hi;
            }
            lds_barrier();
            if (slot == 0) return false;
            if (kBandRows) {
                // lane 0 has a cell in every round that any lane has one in: its copy is complete
                fin_lo = uniform(new_lo);
                fin_hi = uniform(new_hi);
            } else {
                int lo = INT32_MAX, hi = -1;
                for (int w = 0; w < int(nthreads >> 6); ++w) {
                    const int wl = fin_w[((slot & 1) * 4 + w) * 2], wh = fin_w[((slot & 1) * 4 + w) * 2 + 1];
                    lo = wl < lo ? wl : lo;
                    hi = wh > hi ? wh : hi;
                }
                fin_lo = uniform(lo);
                fin_hi = uniform(hi);
            }
            if (fin_hi < 0 && tid == 0) scal[0] = uint64_t(kInfSum);
            return fin_hi < 0;
        };
        for (int slot = S - 1; slot >= 0; --slot) {
            const uint32_t b0 = (uint32_t)uniform((int)band[slot]);
            const uint32_t b1 = (uint32_t)uniform((int)band[slot + 1]);
            const int il = slot == 0 ? 0 : band_lo(b0), ih = slot == 0 ? 0 : band_hi(b0);   // cells
            const int jl = band_lo(b1), jh = band_hi(b1);                                     // continuations
            const int jl_f = fin_lo > jl ? fin_lo : jl;
            const int jh_f = fin_hi < jh ? fin_hi : jh;
            int new_lo = INT32_MAX, new_hi = -1;        // this wavefront's cells with a finite sum
            // what the slot in front will read of its own time row: its cells and this slot's cells
            const int nl = slot >= 2 ? band_lo((uint32_t)uniform((int)band[slot - 1])) : 0;
            const bool stage_next = slot >= 1;
            // a wave whose lanes own neither a cell nor a staged entry only keeps the barrier
            if (il + wave_first > ih && (!stage_next || nl + wave_first > ih)) {
                if (end_of_slot(slot, INT32_MAX, -1)) break;
                cur ^= 1;
                pcur ^= 1;
                continue;
            }
            const uint32_t rsv = (uint32_t)uniform((int)sc[slot].cm_row_shift);
            const TpDiv div = tp_div<kOdd>(tb, rsv >> 27);
            const int64_t capm = uniform64(sc[slot].cap);
            const float cap_f = float(capm), err = need_err + cap_f * (4.f / 16777216.f);
            const float fits_up_to = cap_f - err, none_above = cap_f + err;
            const uint16_t *hi_row = hi_tab + (uint32_t)uniform((int)hi_off[slot]);
            // rows of this slot start at its lowest cell il, the row of continuations at jl, the rows
            // staged for the slot in front at nl
            const uint32_t *pr_cur = (pcur ? prow1 : prow0) - (kBandRows ? il : 0);
            uint32_t *pr_next = (pcur ? prow0 : prow1) - (kBandRows ? nl : 0);
            const Entry *prev = (cur ? rows1 : rows0) - (kBandRows ? jl : 0);
            Entry *next = (cur ? rows0 : rows1) - (kBandRows ? il : 0);
            const float *needs = (cur ? needs1 : needs0) - (kBandRows ? jl : 0);
            float *needs_next = (cur ? needs0 : needs1) - (kBandRows ? il : 0);
            // the cut in front of this slot's stage (between slot - 1 and slot)
            const uint32_t *cm_front = stage_next ? tb.CM + ((uint32_t)uniform((int)sc[slot - 1].cm_row_shift) & kRowMask)
                                                  : nullptr;
            const uint32_t *p32_n = stage_next ? tb.P32 + (uint32_t)uniform((int)sc[slot - 1].p_row) : nullptr;
            // requests for the slot in front: entry xn of its time row and the memory sums there, and this lane's own cut time
            const int xn = nl + tid;
            uint32_t p_n = 0, cf_first = 0;
            int64_t pp_n = 0, ps_n = 0;
            if (stage_next && xn <= ih) { p_n = p32_n[xn]; pp_n = PP[xn]; ps_n = PS[xn]; }
            if (stage_next && il + tid <= ih) cf_first = cm_front[il + tid];

            bool first_trip = true;
            for (int i = il + tid; i <= ih; i += nthreads) {
                const MemPair mi = first_trip ? sums_n : sums_at(i);
                const float fits = fits_up_to + mi.pp, none = none_above + mi.pp;
                const uint32_t xi = pr_cur[i], add = div.add - xi;
                SumT best = kInfSum;
                int best_j = jl;
                const int first = (i + 1) > jl_f ? (i + 1) : jl_f;
                int j = first;
                // end cuts beyond the classic count's reach cannot fit with a larger count either
                const int reach = hi_row[i];
                const int end = reach < jh_f ? reach : jh_f;
                bool more = j <= end;
                while (more) {
                    uint32_t tj = 0;
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        // end cuts behind jh_f (up to kTail behind L) hold an infinite sum, whatever the other
                        // rows hold there; those behind `reach` need more memory than there is with any count
                        const float need = fmaf(-prev[j + u].nn, mi.ps, needs[j + u]);
                        tj = tp_quot<kOdd>(pr_cur[j + u] + add, div);
                        const SumT v = prev[j + u].h + tj;
                        const bool upd = (need <= none) & (tj <= tcap) & (v < best);
                        best = upd ? v : best;
                        best_j = upd ? (j + u) : best_j;
                    }
                    more = ((j + 4) <= end) & (tj <= tcap);
                    j += 4;
                }
                if (best < kInfSum && !(fmaf(-prev[best_j].nn, mi.ps, needs[best_j]) <= fits)) {
                    // rare: the cell again, in 64 bits
                    best = kInfSum;
                    best_j = jl;
                    for (j = first; j <= end; ++j) {
                        const Entry e = prev[j];
                        const uint32_t time = tp_quot<kOdd>(pr_cur[j] + add, div);
                        if (time > tcap) break;
                        const SumT v = e.h + time;
                        const int64_t dpp = PP[j] - PP[i], dps = PS[j] - PS[i];
                        if (v < best && dpp + int64_t(e.nn) * dps <= capm) { best = v; best_j = j; }
                    }
                }
                arg[slot * arg_pitch + i] = (uint16_t)best_j;
                if (stage_next) {
                    const uint32_t cf = first_trip ? cf_first : cm_front[i];
                    const uint64_t total = uint64_t(best) + 2ull * cf;
                    const bool reach = (best < kInfSum) & (cf <= tcap);
                    if (reach & (total > limit)) flags[1] = 1;        // needs 64-bit sums
                    const bool finite = reach & (total <= limit);
                    next[i].h = finite ? SumT(total) : kInfSum;
                    {
                        // lanes hold consecutive cells from i - lane on: the lowest and the highest lane with
                        // a finite sum bound this round's cells
                        const unsigned long long fm = __ballot(finite);
                        if (fm != 0) {
                            const int base = uniform(i - lane);
                            const int lo_r = base + __ffsll((long long)fm) - 1, hi_r = base + 63 - __clzll((long long)fm);
                            new_lo = lo_r < new_lo ? lo_r : new_lo;
                            new_hi = hi_r > new_hi ? hi_r : new_hi;
                        }
                    }
                    const uint32_t nn = h1f1b_delta(cf, cap64) + uint32_t(prev[best_j].nn);
                    const float n_f = float(nn < uint32_t(m_cap) ? nn : uint32_t(m_cap));
                    next[i].nn = n_f;
                    needs_next[i] = fmaf(n_f, mi.ps, mi.pp);
                } else {
                    scal[0] = uint64_t(best);
                }
                first_trip = false;
            }
            if (stage_next) {
                if (tid < kTail) next[ih + 1 + tid].h = kInfSum;     // behind the band
                if (xn <= ih) pr_next[xn] = p_n;
                for (int x = xn + nthreads; x <= ih; x += nthreads) pr_next[x] = p32_n[x];
                sums_n = MemPair{sum_f(pp_n), sum_f(ps_n)};
            }
            if (end_of_slot(slot, new_lo, new_hi)) break;
            cur ^= 1;
            pcur ^= 1;
        }
        __syncthreads();
        if (!kWide && uniform((int)flags[1]) != 0) {
            if (tid == 0) dead_list[n_dead + atomicAdd(&counts[2], 1)] = uint32_t(c);
            continue;
        }
        const uint64_t sum = (uint64_t)uniform64((int64_t)scal[0]);
        if (sum >= uint64_t(kInfSum)) {
            write_failed(out, c, S_max, HARP_CAND_INFEASIBLE);
            for (int s = tid; s < S_max; s += nthreads) wu[s] = -1;
            continue;
        }
        // the cuts, from the first slot on: the cut in a scalar, a lane per slot for the cuts found
        if (wave == 0) {
            int b = 0;
            for (int s0 = 0; s0 < S; s0 += 64) {
                const int n = S - s0 < 64 ? S - s0 : 64;
                int found = 0;
                for (int s = 0; s < n; ++s) {
                    found = lane == s ? b : found;
                    b = uniform(arg[(s0 + s) * arg_pitch + b]);
                    b = b <= L ? b : L;      // a finite sum only chains through cuts inside the row
                }
                if (lane < n) trial[s0 + lane] = found;
            }
            if (lane == 0) trial[S] = b;
        }
        __syncthreads();
        // one lane per stage: the plan's own bottleneck, and the counts by eq. Ni along the plan
        if (wave == 0) {
            uint32_t w = 0;
            for (int s = lane; s < S; s += 64) {
                const int j = trial[s], i = trial[s + 1];
                const uint32_t rsl = sc[s].cm_row_shift;
                const TpDiv div = tp_div<kOdd>(tb, rsl >> 27);
                const uint32_t *p = tb.P32 + sc[s].p_row;
                const uint32_t t = tp_quot<kOdd>(p[i] + div.add - p[j], div);
                const uint32_t cu = s < S - 1 ? tb.CM[(rsl & kRowMask) + uint32_t(i)] : 0u;
                const uint32_t m = t > cu ? t : cu;
                w = w > m ? w : m;
                deltas[s] = s < S - 1 ? h1f1b_delta(cu, cap64) : 1u;
            }
            w = wave_all(w, max2);
            if (lane == 0) {
                out.bottleneck[c] = int64_t(w);
                out.iter_time[c] = int64_t(sum) + (m_cap - 1) * cap64;
                out.status[c] = HARP_CAND_OK;
            }
        }
        __syncthreads();
        // N of a stage = the growths from it to the last one, at most M: a running sum from the end
        if (wave == 0) {
            uint32_t behind = 0;
            for (int s0 = (S - 1) & ~63; s0 >= 0; s0 -= 64) {
                const int s = s0 + 63 - lane;
                const uint32_t n = wave_scan(s < S ? uint32_t(deltas[s]) : 0u, sum2) + behind;
                if (s < S) wu[s] = int32_t(n < uint32_t(m_cap) ? n : uint32_t(m_cap));
                behind = uint32_t(__builtin_amdgcn_readlane(int(n), 63));
            }
        }
        for (int s = tid; s <= S_max; s += nthreads) sp[s] = s <= S ? trial[s] : -1;
        for (int s = S + tid; s < S_max; s += nthreads) wu[s] = -1;
    }
    // candidates the pre-pass rejected: no plan to report
    if (!kWide && kMode != 2) {
        for (int n = blockIdx.x; n < n_dead; n += gridDim.x) {
            const uint32_t e = dead_list[n];
            const int c = int(e & ((1u << kDeadStatusShift) - 1u));
            const int st = cap_out_of_range(tb, t_max[c]) ? HARP_CAND_INVALID : int(e >> kDeadStatusShift);
            write_failed(out, c, S_max, st);
            for (int s = tid; s < S_max; s += nthreads) warmup[int64_t(c) * S_max + s] = -1;
        }
    }
}

#define HARP_H1F1B_KERNEL(NAME, BOUNDS, SUM, MODE)                                                                  \
    template <bool kOdd>                                                                                           \
    __global__ BOUNDS void NAME(TablesDev tb, CandDev cd, const int64_t *t_max, PlansDev out, int32_t *warmup,     \
                                int *counts, int *tickets, const int32_t *live_list, uint32_t *dead_list,          \
                                const uint32_t *bands,                                                             \
                                const uint16_t *hi_tab, int idx_pitch, unsigned char *arg_base,                    \
                                size_t arg_per_group, int row_len, int arg_pitch) {                                \
        h1f1b_body<SUM, MODE, kOdd>(tb, cd, t_max, out, warmup, counts, tickets, live_list, dead_list, bands, hi_tab, idx_pitch, \
                              arg_base, arg_per_group, row_len, arg_pitch);                                        \
    }
HARP_H1F1B_KERNEL(k2_h1f1b, __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(6, 6))), uint32_t, 1)
HARP_H1F1B_KERNEL(k2_h1f1b_rows, __launch_bounds__(kFastThreads) __attribute__((amdgpu_waves_per_eu(8, 8))), uint32_t, 2)
HARP_H1F1B_KERNEL(k2_h1f1b_wide, __launch_bounds__(kFastThreads), uint64_t, 0)
#undef HARP_H1F1B_KERNEL

int h1f1b_row_len(int L) { return (L + 1 + kTail + 7) / 8 * 8; }

// whole-sequence rows: two of entries, two of needs, two of times
size_t h1f1b_lds_bytes(int L, int S_max, size_t entry) {
    return h1f1b_small_bytes(S_max) + size_t(h1f1b_row_len(L)) * (2 * entry + 2 * sizeof(float) + 8);
}

}  // namespace

// Runs the pre-pass itself (launch_plan_fast's first two kernels are shared through
// launch_plan_prepass) and then the three instantiations.  n_groups: resident 256-thread workgroups;
// n_slices: back-pointer slices in the workspace (the wavefront-per-candidate launch runs at most
// that many).
void launch_plan_h1f1b(const TablesDev &tb, const CandDev &cd, const int64_t *t_max, const PlansDev &out,
                       int32_t *warmup, void *ws, int n_groups, int n_slices, int n_cu, hipStream_t st) {
    const FastWorkspace w = carve(ws, fast_shape(tb, cd, false), n_groups);
    launch_plan_prepass(tb, cd, ws, n_groups, false, st);
    const int row_len = h1f1b_row_len(tb.L);
    const int idx_pitch = int(lo_pitch(tb.L));
    const uint16_t *hi_tab = w.lo_tab + (long long)lo_n_max(tb.L, cd.S_max, tb.M) * tb.T * tb.n_tp * idx_pitch;
    const size_t per_group = fast_arg_per_group(tb.L, cd.S_max);
    const int arg_pitch = fast_row_len(tb.L);
    // Wavefronts per CU of the first launch and the row entries their LDS share leaves.  LDS is allocated in units, so a share
    // is as many units as hold the widest slot of a candidate with a stage on every group (S stages: L - S + 2 cuts), or rows for
    // the sequence up to one cut in forty that hardly any slot needs, and there are as many wavefronts as such shares fit, between
    // 14 and 24 (six per SIMD, held to 80 registers with 5 of them spilled; fewer hide less of the latency: 160 operators, five per SIMD 1.61 ms, six 1.47, seven 1.54 with
    // more spills).  The smaller the share, the more candidates leave for the second launch: 300 operators, 14 per
    // CU 3.7 ms, 17 3.7, 20 4.9; 512 operators, tight memory 1.90, 1.88, 1.92, loose memory 14.1 for all.  Counted in bytes, a number of
    // wavefronts left part of a unit to each and rows that just do not fit: 20,000 candidates of up to 32 stages, us by
    // bytes / by units: 200 operators 759 / 669, 230 792 / 781, 245 897 / 848, 280 921 / 901, 330 1,145 / 1,107.  Rows
    // for the whole sequence where candidates have a stage on each of many groups take more than their slots need: 278 operators on 32
    // groups, 12,000 candidates 727 -> 694 with shares for the widest slot, 209 on 30, 42,385 candidates 1,767 -> 1,641.
    const size_t small = h1f1b_small_bytes(cd.S_max), units = (size_t(160) << 10) / kLdsGranule;
    auto held = [&](size_t n) -> int {
        const size_t share = n * kLdsGranule;
        return share > small + h1f1b_cut_bytes(8) * 16 ? int((share - small) / h1f1b_cut_bytes(8)) & ~1 : 16;
    };
    size_t n_units = units / 24;
    const int stages = tb.G < cd.S_max ? tb.G : cd.S_max, widest = tb.L - stages + 2 + kTail, nearly = (tb.L + 1) - (tb.L + 1) / 40;
    while (n_units < units / 14 && held(n_units) < (widest < nearly ? widest : nearly)) ++n_units;
    const int per_cu = units / n_units < 24 ? int(units / n_units) : 24;
    const int entries = held(n_units) < row_len ? held(n_units) : row_len;
    int n_waves = per_cu * n_cu;
    if (n_waves > n_slices) n_waves = n_slices;
    if (n_waves > cd.C) n_waves = cd.C;
    if (n_waves < 1) n_waves = 1;
    auto launch = [&](auto odd_t) {
        constexpr bool odd = decltype(odd_t)::value;
        hipLaunchKernelGGL(k2_h1f1b<odd>, dim3(n_waves), dim3(64), small + size_t(entries) * h1f1b_cut_bytes(8), st, tb, cd,
                           t_max, out, warmup, w.counts, w.tickets, w.live_list, w.dead_list, w.bands, hi_tab, idx_pitch, w.arg,
                           per_group, entries, arg_pitch);
        if (entries < row_len)
            hipLaunchKernelGGL(k2_h1f1b_rows<odd>, dim3(n_groups), dim3(kFastThreads), h1f1b_lds_bytes(tb.L, cd.S_max, 8),
                               st, tb, cd, t_max, out, warmup, w.counts, w.tickets, w.live_list, w.dead_list, w.bands, hi_tab,
                               idx_pitch, w.arg, per_group, row_len, arg_pitch);
        hipLaunchKernelGGL(k2_h1f1b_wide<odd>, dim3(n_groups), dim3(kFastThreads), h1f1b_lds_bytes(tb.L, cd.S_max, 16), st,
                           tb, cd, t_max, out, warmup, w.counts, w.tickets, w.live_list, w.dead_list, w.bands, hi_tab, idx_pitch,
                           w.arg, per_group, row_len, arg_pitch);
    };
    if (tb.odd_degrees()) launch(std::true_type());
    else launch(std::false_type());
}

}  // namespace harp
