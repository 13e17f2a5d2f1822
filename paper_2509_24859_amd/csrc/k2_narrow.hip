// Bands under a cap for the 32-bit planner kernels.
//
// k2_band bounds the cuts of a candidate by the memory constraint alone.  With a cap t on every stage and
// transfer time the two chains get tighter:
//   F[s+1] = the highest cut that a stage started at F[s] reaches in memory with time <= t, lowered to a cut
//            whose transfer time is at most t;
//   B[s]   = the same from the end.
// A chain must not leave a stage without operators: where no such cut lies above F[s], any cut behind stage s
// that some plan has lies at or below the one found, so the cut in front of it lies below that: F[s] becomes the
// next lower cut that the link in front allows, and the step is repeated.  Every partial plan under t has its
// cuts at or below F, every completable one at or above B (both reaches never decrease with the cut they start
// from), so cells outside [B, F] are on no plan under t, and leaving them out changes no cell on such a plan.
// The planner kernels rely on ranges that rise with the stage (their rows in LDS start at B[s] and hold the cells
// of row s + 1), which a value corrected later would break; a stage holds an operator at least, so F[s] is
// lowered to F[s + 1] - 1 and B[s + 1] raised to B[s] + 1 at the end.
//
// The exact search uses it for the candidates whose memory bands are wide (k2_band lists them): no cap of its
// walk is above t_E = ceil(T(t_S) / B), T(t_S) the min-max plan's total.
//
// Four lanes work a candidate, 16 to a wavefront; a lane looks at four consecutive cuts (16 bytes of the time row
// and of the cut row), so that a step is one round trip to L2 for a window of 16 cuts.  A chain of S dependent
// steps is bound by their latency; fewer lanes per candidate put more candidates in flight.
// 65,536 candidates of 160 operators, 16 to 32 stages: 78 cuts a row -> about 50; this launch takes 0.13 ms and
// takes k2_exact from 3.11 to 2.62 ms; 131,072 of 512 operators, up to 64 stages, tight memory: the call 8.6 -> 7.6 ms.
// Not used for the min-max planner, where the cap has to be searched for
// (1.5 to 4 chains a candidate, as many as the slowest of 16 needs: 0.29 to 2.2 ms for 0.13 to 0.27 ms less in
// k2_fast), nor for H-1F1B under a given cap (0.13 ms for 0.10).
#include "fast_common.h"
#include "harp_internal.h"
#include "plan_common.h"

namespace harp {

using namespace fastdp;

namespace {

constexpr int kCands = 16;                       // candidates per wavefront, one wavefront per workgroup
constexpr uint32_t kTop = 0x7FFFFFFFu;           // no time on these tables is larger
constexpr uint32_t kRowBits = 29;                // time rows: below 65,535 x 4,112 entries

template <int kCtrl>
__device__ __forceinline__ int from_lane(int v) { return __builtin_amdgcn_update_dpp(v, v, kCtrl, 0xF, 0xF, false); }
__device__ __forceinline__ int quad_max(int v) {
    int o = from_lane<0xB1>(v);
    v = o > v ? o : v;
    o = from_lane<0x4E>(v);
    return o > v ? o : v;
}
__device__ __forceinline__ int quad_min(int v) {
    int o = from_lane<0xB1>(v);
    v = o < v ? o : v;
    o = from_lane<0x4E>(v);
    return o < v ? o : v;
}
struct alignas(4) Four { uint32_t v[4]; };

// One candidate; the four lanes of a quad hold the same values but for r, the lane within the quad.
struct Chains {
    const TablesDev &tb;
    const uint16_t *lo_tab, *hi_tab;
    // LDS, [stage][candidate]: row of times (degree index above kRowBits), of transfer times, of the index
    const uint32_t *p_row, *cm_row, *ix_row, *tp;
    uint16_t *F, *B;                             // [S_max + 1][kCands]
    int q, r, S, L, pitch;

    __device__ __forceinline__ const uint32_t *times(int s, uint32_t &degree) const {
        const uint32_t w = p_row[s * kCands + q];
        degree = tp[w >> kRowBits];
        return tb.P32 + (w & ((1u << kRowBits) - 1u));
    }
    __device__ __forceinline__ const uint32_t *cuts(int s) const { return tb.CM + cm_row[s * kCands + q]; }
    static __device__ __forceinline__ uint32_t reach(uint32_t t, uint32_t degree) {
        const uint64_t far = uint64_t(t) * degree;
        return far < kTop ? uint32_t(far) : kTop;
    }
    // highest cut in [least, x] that the link behind stage s allows; -1 when there is none
    __device__ __forceinline__ int allowed_down(int s, int x, int least, uint32_t t) const {
        const uint32_t *cm = cuts(s);
        for (; x >= least; x -= 4) {
            const int i = x - r;
            const int best = quad_max(i >= least && cm[i] <= t ? i : -1);
            if (best >= 0) return best;
        }
        return -1;
    }
    // lowest cut in [x, most]; L + 1 when there is none
    __device__ __forceinline__ int allowed_up(int s, int x, int most, uint32_t t) const {
        const uint32_t *cm = cuts(s);
        for (; x <= most; x += 4) {
            const int i = x + r;
            const int best = quad_min(i <= most && cm[i] <= t ? i : L + 1);
            if (best <= L) return best;
        }
        return L + 1;
    }
    __device__ __forceinline__ bool forward(uint32_t t) const {
        int at = 0;
        if (r == 0) F[q] = 0;
        for (int s = 0; s < S; ++s) {
            const bool last = s == S - 1;
            const int top = L - (S - 1 - s);
            uint32_t degree;
            const uint32_t *p = times(s, degree), *cm = cuts(s);
            const uint16_t *fits = hi_tab + ix_row[s * kCands + q];
            const uint32_t far = reach(t, degree);
            int best = -1;
            for (;;) {
                const uint32_t pa = p[at];
                const int fit = fits[at], lim = fit < top ? fit : top;
                bool more = true;
                for (int base = at; more; base += 16) {
                    const int idx = base + 4 * r < pitch - 4 ? base + 4 * r : pitch - 4;
                    const Four pw = *reinterpret_cast<const Four *>(p + idx), cw = *reinterpret_cast<const Four *>(cm + idx);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int i = idx + e;
                        const bool ok = (i > at) & (i <= lim) & (pw.v[e] - pa <= far) & (last | (cw.v[e] <= t));
                        best = ok && i > best ? i : best;
                    }
                    // another window when the last cut of this one is in time and memory and more are
                    more = quad_max(r == 3 && idx + 3 < lim && pw.v[3] - pa <= far ? 1 : 0) != 0;
                }
                best = quad_max(best);
                if (best > at) break;
                if (s == 0) return false;
                const int most = last ? -1 : allowed_down(s, at, s + 1, t);
                if (most < 0) return false;
                at = allowed_down(s - 1, most - 1, s, t);
                if (at < 0) return false;
                if (r == 0) F[s * kCands + q] = uint16_t(at);
            }
            at = best;
            if (r == 0) F[(s + 1) * kCands + q] = uint16_t(at);
        }
        return at == L;
    }
    __device__ __forceinline__ bool backward(uint32_t t) const {
        int at = L;
        if (r == 0) B[S * kCands + q] = uint16_t(L);
        for (int s = S - 1; s >= 0; --s) {
            uint32_t degree;
            const uint32_t *p = times(s, degree), *cm = cuts(s > 0 ? s - 1 : 0);
            const uint16_t *fits = lo_tab + ix_row[s * kCands + q];
            const uint32_t far = reach(t, degree);
            int best = L + 1;
            for (;;) {
                const uint32_t pa = p[at];
                const int fit = fits[at], lim = fit > s ? fit : s;
                bool more = true;
                for (int base = at; more; base -= 16) {
                    const int idx = base - 4 * r - 4 > 0 ? base - 4 * r - 4 : 0;
                    const Four pw = *reinterpret_cast<const Four *>(p + idx), cw = *reinterpret_cast<const Four *>(cm + idx);
#pragma unroll
                    for (int e = 3; e >= 0; --e) {
                        const int i = idx + e;
                        const bool ok = (i < at) & (i >= lim) & (pa - pw.v[e] <= far) & (s == 0 || cw.v[e] <= t);
                        best = ok && i < best ? i : best;
                    }
                    more = quad_max(r == 3 && idx > lim && pa - pw.v[0] <= far ? 1 : 0) != 0;
                }
                best = quad_min(best);
                if (best < at) break;
                if (s == 0 || s == S - 1) return false;
                const int least = allowed_up(s - 1, at, L - (S - s), t);
                if (least > L) return false;
                at = allowed_up(s, least + 1, L - (S - s - 1), t);
                if (at > L) return false;
                if (r == 0) B[(s + 1) * kCands + q] = uint16_t(at);
            }
            at = best;
            if (r == 0) B[s * kCands + q] = uint16_t(at);
        }
        return at == 0;
    }
    // Rising ranges to `row`, and the cuts of the widest stage; false, and nothing written, when a range is empty.
    __device__ __forceinline__ bool ranges(uint32_t *row, int &span) const {
        int f = L + 1;
        for (int s = S; s >= 0; --s) {
            const int own = F[s * kCands + q];
            f = own < f - 1 ? own : f - 1;
            if (r == 0) F[s * kCands + q] = uint16_t(f > 0 ? f : 0);
        }
        wave_sync();
        int b = -1;
        bool empty = f < 0;
        for (int s = 0; s <= S; ++s) {
            const int own = B[s * kCands + q], top = F[s * kCands + q];
            b = own > b + 1 ? own : b + 1;
            empty = empty || b > top;
            if (r == 0) B[s * kCands + q] = uint16_t(b);
        }
        if (empty) return false;
        wave_sync();
        for (int s = r; s <= S; s += 4) {
            const int lo = B[s * kCands + q], hi = F[s * kCands + q];
            row[s] = uint32_t(lo) | (uint32_t(hi) << 16);
            if (s < S) {
                const int w = F[(s + 1) * kCands + q] - lo + 1;
                span = w > span ? w : span;
            }
        }
        span = quad_max(span);
        return true;
    }
};

size_t narrow_lds_bytes(int S_max) {
    return size_t(S_max) * kCands * 12 + 8 * 4 + 2 * ((size_t(S_max + 1) * kCands * 2 + 15) & ~size_t(15));
}

__global__ __launch_bounds__(64) void k2_narrow(TablesDev tb, CandDev cd, PlansDev out, const int *counts,
                                                int *tickets, int row_entries, const int32_t *wide_list, const uint32_t *bands, uint32_t *tight,
                                                const uint16_t *lo_tab, const uint16_t *hi_tab, int idx_pitch) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int S_max = cd.S_max, L = tb.L;
    uint32_t *p_row = reinterpret_cast<uint32_t *>(lds_raw), *cm_row = p_row + S_max * kCands, *ix_row = cm_row + S_max * kCands;
    uint32_t *tp = ix_row + S_max * kCands;
    uint16_t *F = reinterpret_cast<uint16_t *>(tp + 8), *B = F + (S_max + 1) * kCands;
    const int n_items = counts[kWideBands];
    if (!bands_narrowed(counts)) return;
    int too_wide = 0;
    const int lane = threadIdx.x, q = lane >> 2, r = lane & 3;
    if (lane < 8) tp[lane] = lane < tb.n_tp ? uint32_t(tb.tp[lane]) : 1u;
    for (int base = blockIdx.x * kCands; base < n_items; base += gridDim.x * kCands) {
        wave_sync();
        const bool active = base + q < n_items;
        const int c = active ? wide_list[base + q] : 0;
        Chains ch{tb, lo_tab, hi_tab, p_row, cm_row, ix_row, tp, F, B, q, r, active ? cd.cand_S[c] : 0, L, int(tb.pitch32)};
        const int32_t *grp = cd.cand_group + int64_t(c) * S_max, *deg = cd.cand_tp + int64_t(c) * S_max;
        for (int s = r; s < ch.S; s += 4) {
            const int g = grp[s], k = tp_index(tb, deg[s]), to = grp[s + 1 < ch.S ? s + 1 : s];
            const int n = (ch.S - s) < tb.M ? (ch.S - s) : tb.M;
            p_row[s * kCands + q] = uint32_t((g * tb.n_tp + k) * int(tb.pitch32)) | (uint32_t(k) << kRowBits);
            cm_row[s * kCands + q] = uint32_t(g * tb.G + to) * uint32_t(tb.pitch32);
            ix_row[s * kCands + q] = uint32_t(((n - 1) * tb.T + tb.group_type[g]) * tb.n_tp + k) * uint32_t(idx_pitch);
        }
        wave_sync();
        // (the exact search passes candidates without a min-max plan by)
        if (!active || out.status[c] != HARP_CAND_OK) continue;
        const int64_t t_E = (out.iter_time[c] + tb.M - 1) / tb.M;
        const uint32_t cap = t_E < int64_t(kTop) ? uint32_t(t_E) : kTop;
        uint32_t *row = tight + int64_t(c) * (S_max + 1);
        bool through = ch.forward(cap);
        through = through && ch.backward(cap);
        wave_sync();                 // both chains are in LDS
        int span = 0;
        if (through && ch.ranges(row, span)) {
            if (r == 0 && span + kPad > row_entries) ++too_wide;
            continue;
        }
        // (cannot happen: the min-max plan is a plan under t_E)
        const uint32_t *wide = bands + int64_t(c) * (S_max + 1);
        for (int s = r; s <= ch.S; s += 4) row[s] = wide[s];
    }
    too_wide = int(wave_all(uint32_t(too_wide), sum2));
    if (too_wide != 0 && lane == 0) atomicAdd(tickets + (blockIdx.x & (kShares - 1)) * kShareInts + kLongRows, too_wide);
}

}  // namespace

// Narrowing costs a chain of some 3 to 5 us a stage whatever the batch, and gains where a stage has cuts to lose.
// Exact search without / with it: 128 operators, up to 16 stages, 4,096 candidates 0.42 / 0.46 ms; 160 operators, up to
// 32 stages, 32,768 candidates 2.71 / 2.52; 300 operators, up to 128 stages, 4,096 candidates 2.4 / 3.0: five operators
// a stage divide the last two.  A batch that the chip works in one round has the whole chain to bear: 512 candidates
// of 160 operators and up to 32 stages 0.49 / 0.57.
bool exact_narrows(int L, int S_max, int C, int n_cu) {
    return L >= 144 && L >= (C > 8 * n_cu ? 5 : 6) * S_max;
}

// Behind launch_plan_fast, on its workspace and results.  row_entries: candidates with a stage that spans more are counted.
void launch_plan_narrow(const TablesDev &tb, const CandDev &cd, const PlansDev &out, void *ws, int n_slices, int n_cu,
                        int row_entries, hipStream_t st) {
    const FastWorkspace w = carve(ws, fast_shape(tb, cd, true), n_slices);
    const size_t lds = narrow_lds_bytes(cd.S_max);
    int per_cu = int((size_t(160) << 10) / (lds + 128));
    per_cu = per_cu > 32 ? 32 : per_cu;
    long long grid = ((long long)cd.C + kCands - 1) / kCands;
    if (grid > (long long)per_cu * n_cu) grid = (long long)per_cu * n_cu;
    const long long idx_rows = (long long)lo_n_max(tb.L, cd.S_max, tb.M) * tb.T * tb.n_tp;
    const int idx_pitch = int(lo_pitch(tb.L));
    hipLaunchKernelGGL(k2_narrow, dim3(unsigned(grid)), dim3(64), lds, st, tb, cd, out, w.counts, w.tickets, row_entries,
                       w.wide_list, w.bands, w.tight, w.lo_tab, w.lo_tab + idx_rows * idx_pitch, idx_pitch);
}

}  // namespace harp
