// Submesh choice inside the recurrence (paper section 5.2.3, eq. dp_general's third index).
//
// A candidate is an order of device groups and a stage count S.  With O_k = devices of the first k
// groups of the order, the state (s, i, d) means: the first s stages hold the first i operators and
// use exactly the first d devices.  A stage placed at device offset d runs on the group k with
// O_k <= d < O_{k+1} and takes tp of its devices (an allowed degree, d + tp <= O_{k+1}); when that
// exhausts the group, the next stage is on the next group and the cut crosses the inter-group
// link, otherwise the intra-group link.  All devices of all listed groups are used: the answer is
// the state (S, L, O_K).  Min-max form with the classic 1F1B counts, as on the hot path:
//   D[s+1][i][d + tp] = min over (j, tp) of max(D[s][j][d], time, comm),
// ties resolved by the lowest previous cut j, then the smallest degree.
//
// Two forms.  k2_mesh_band and k2_mesh_band_h1f1b run on the fused 32-bit rows, on the ranges of cuts
// that some plan under the bottleneck (or cap) in question can have (mesh_band.h); k2_mesh and
// k2_mesh_h1f1b fill the whole table, one lane per target cell (i, d'), rows and back-pointers in the
// workspace, with the passes of mesh_passes.h on the fused 32-bit rows (kFast) or on the int64 rows (any
// degrees, any time width).  The int64 passes serve tables without 32-bit rows and more than 1,024
// operators; the whole table on the 32-bit rows serves problems so small that finding the ranges costs more
// than they save (whole_table), more than 2,048 devices, and the orderings the band form hands over
// because their sets of time rows do not fit its LDS or their sums could reach 2^31.
#include <math.h>

#include "mesh_band.h"
#include "mesh_passes.h"

namespace harp {

using namespace meshdp;
using meshband::Band;
using meshband::BandArgs;
using meshband::BandShape;
using meshband::MeshWorkspace;
using meshband::mesh_carve;

namespace {

// Orderings a kernel works on: all of the batch, or those a band kernel handed over.
struct MeshItems {
    int *ticket;
    const int *list;         // null: all
    const int *n_list;
};
// Workgroups beyond the orderings handed over leave without drawing from the ticket (2,048 of them drawing
// one after the other take 29 us).
__device__ __forceinline__ bool no_item(const MeshItems &it) { return it.list && int(blockIdx.x) >= *it.n_list; }
__device__ __forceinline__ int next_item(const MeshItems &it, int C) {
    const int n = atomicAdd(it.ticket, 1);
    if (!it.list) return n < C ? n : -1;
    return n < *it.n_list ? it.list[n] : -1;
}

// kExact = false: the min-max plan of every ordering.  kExact = true: the optimum of the
// iteration-time model (section 5.2.2) over every slicing and partition: the capped least-sum
// table is walked over the caps exactly as the exact search of the hot path walks them (first at
// t_S, then down from ceil(T / B), skipping caps that the sums rule out; equal totals keep the lower
// cap), which returns what the increasing sweep over every distinct stage cost returns.
template <bool kExact, bool kFast>
__device__ __forceinline__ void mesh_body(const TablesDev &tb, const OrdDev &od, const PlansDev &out,
                                          int32_t *stage_group, int32_t *stage_tp, int32_t *n_passes,
                                          unsigned char *ws, size_t per_group, int64_t n_dev, const MeshItems &items) {
    __shared__ int32_t offs[kMaxOrderGroups + 1];     // O_0 .. O_K
    __shared__ uint16_t order[kMaxOrderGroups];      // group ids are below 4096
    __shared__ uint16_t group_at[kMeshGroupTable];    // group index (in the order) of every device offset
    __shared__ int32_t cuts[kMaxStages + 1], kept_cuts[kMaxStages + 1];
    __shared__ uint16_t slot_g[kMaxStages], kept_g[kMaxStages];
    __shared__ uint8_t slot_k[kMaxStages], kept_k[kMaxStages];
    __shared__ int32_t slot_first[kMaxStages], kept_first[kMaxStages];
    __shared__ int64_t scored[2];
    __shared__ int shared_int[2];
    const int L = tb.L, S_max = od.S_max;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nthreads = blockDim.x;
    const MeshSlice m = mesh_slice(ws, per_group, L, n_dev);
    const int64_t m_cap = tb.M;
    if (no_item(items)) return;

    // all threads: thread 0 backtracks into cuts/slot_*, the first wave scores them
    auto backtrack_and_score = [&](int K, int S, int64_t &bott, int64_t &total) {
        if (tid == 0) mesh_backtrack<kFast>(tb, m, offs, order, K, S, n_dev, cuts, slot_g, slot_k, slot_first);
        __syncthreads();
        if (wave == 0) {
            int64_t b, t;
            wave_score_partition(tb, S, slot_g, slot_k, cuts, lane, b, t);
            if (lane == 0) { scored[0] = b; scored[1] = t; }
        }
        __syncthreads();
        bott = scored[0];
        total = scored[1];
    };
    extern __shared__ __align__(16) unsigned char mesh_lds[];      // kFast: a row of memory sums
    int64_t *Q = reinterpret_cast<int64_t *>(mesh_lds);
    auto run_pass = [&](auto capped, int K, int S, int64_t cap) -> int64_t {
        constexpr bool kCapped = decltype(capped)::value;
        if constexpr (kFast) return mesh_pass_fast<kCapped>(tb, m, offs, order, group_at, Q, K, S, n_dev, cap);
        else return mesh_pass<kCapped>(tb, m, offs, order, group_at, K, S, n_dev, cap);
    };
    auto keep = [&](int S) {
        for (int s = tid; s <= S; s += nthreads) kept_cuts[s] = cuts[s];
        for (int s = tid; s < S; s += nthreads) {
            kept_g[s] = slot_g[s]; kept_k[s] = slot_k[s]; kept_first[s] = slot_first[s];
        }
    };

    for (;;) {
        __syncthreads();
        if (tid == 0) shared_int[0] = next_item(items, od.C);
        __syncthreads();
        const int c = shared_int[0];
        if (c < 0) break;
        const int S = od.ord_S[c], K = od.ord_G[c];
        const int32_t *og = od.ord_group + int64_t(c) * od.G_max;
        int32_t *sg = stage_group + int64_t(c) * S_max, *stp = stage_tp + int64_t(c) * S_max;
        auto fail = [&](int status) {
            write_failed(out, c, S_max, status);
            for (int s = tid; s < S_max; s += nthreads) { sg[s] = -1; stp[s] = -1; }
            if (tid == 0 && n_passes) n_passes[c] = 0;
        };
        // the ordering itself: counts in range, group ids in range and distinct
        int bad = (S < 1 || S > S_max || K < 1 || K > od.G_max) ? 1 : 0;
        if (!bad)
            for (int k = tid; k < K; k += nthreads) {
                const int g = og[k];
                if (g < 0 || g >= tb.G) { bad = 1; continue; }
                for (int q = 0; q < k; ++q)
                    if (og[q] == g) bad = 1;
                order[k] = uint16_t(g);
            }
        if (__syncthreads_or(bad)) { fail(HARP_CAND_INVALID); continue; }
        if (tid == 0) {
            int64_t o = 0;
            offs[0] = 0;
            for (int k = 0; k < K; ++k) { o += tb.group_ndev[order[k]]; offs[k + 1] = int32_t(o); }
        }
        __syncthreads();
        const int Dtot = offs[K];
        if (S > L || S < K || S > Dtot) { fail(HARP_CAND_INFEASIBLE); continue; }
        if (Dtot <= kMeshGroupTable) {
            for (int k = 0; k < K; ++k)
                for (int d = offs[k] + tid; d < offs[k + 1]; d += nthreads) group_at[d] = uint16_t(k);
        }

        if (run_pass(std::false_type(), K, S, 0) == kInf) { fail(HARP_CAND_INFEASIBLE); continue; }
        int64_t t_S, best_T;
        backtrack_and_score(K, S, t_S, best_T);
        int64_t best_b = t_S;
        keep(S);
        int passes = 0;
        if (kExact) {
            int64_t cap = t_S;
            while (S >= 2) {
                const int64_t sum = run_pass(std::true_type(), K, S, cap);
                if (sum == kInf) break;              // cannot happen at or above t_S
                int64_t b, T;
                backtrack_and_score(K, S, b, T);
                ++passes;
                if (T < best_T || (T == best_T && b <= best_b)) {   // equal totals: the lower cap; equal caps: the capped plan
                    best_T = T;
                    best_b = b;
                    keep(S);
                }
                if (passes >= (1 << 20) || b > cap) break;           // cannot happen: the cap falls with every pass
                int64_t next_cap;
                if (passes == 1) {
                    next_cap = (best_T + m_cap - 1) / m_cap;
                } else {
                    next_cap = b - 1;
                    if (m_cap > 1) {
                        const int64_t bound = (best_T - sum) / (m_cap - 1);
                        next_cap = next_cap < bound ? next_cap : bound;
                    }
                }
                if (next_cap <= t_S) break;
                cap = next_cap;
            }
        }
        __syncthreads();
        int32_t *sp = out.splits + int64_t(c) * (S_max + 1);
        int32_t *df = out.dev_first + int64_t(c) * S_max;
        for (int s = tid; s <= S_max; s += nthreads) sp[s] = s <= S ? kept_cuts[s] : -1;
        for (int s = tid; s < S_max; s += nthreads) {
            sg[s] = s < S ? int32_t(kept_g[s]) : -1;
            stp[s] = s < S ? tb.tp[kept_k[s]] : -1;
            df[s] = s < S ? kept_first[s] : -1;
        }
        if (tid == 0) {
            out.bottleneck[c] = best_b;
            out.iter_time[c] = best_T;
            out.status[c] = HARP_CAND_OK;
            if (n_passes) n_passes[c] = passes;
        }
    }
}

template <bool kExact, bool kFast>
__global__ __launch_bounds__(kMeshMaxThreads) void k2_mesh(TablesDev tb, OrdDev od, PlansDev out,
                                                           int32_t *stage_group, int32_t *stage_tp,
                                                           int32_t *n_passes, unsigned char *ws,
                                                           size_t per_group, int64_t n_dev, MeshItems items) {
    mesh_body<kExact, kFast>(tb, od, out, stage_group, stage_tp, n_passes, ws, per_group, n_dev, items);
}

template <bool kFast>
__device__ __forceinline__ void mesh_h1_body(const TablesDev &tb, const OrdDev &od, const int64_t *t_max,
                                             const PlansDev &out, int32_t *stage_group, int32_t *stage_tp,
                                             int32_t *warmup, unsigned char *ws, size_t per_group, int64_t n_dev,
                                             const MeshItems &items) {
    __shared__ int32_t offs[kMaxOrderGroups + 1];
    __shared__ uint16_t order[kMaxOrderGroups];
    __shared__ uint16_t group_at[kMeshGroupTable];
    __shared__ int32_t cuts[kMaxStages + 1], count[kMaxStages];
    __shared__ uint16_t slot_g[kMaxStages];
    __shared__ uint8_t slot_k[kMaxStages];
    __shared__ int32_t slot_first[kMaxStages];
    __shared__ int shared_int[2];
    extern __shared__ __align__(16) unsigned char mesh_lds[];      // kFast: PP and PS, L + 1 entries each
    int64_t *sums_lds = reinterpret_cast<int64_t *>(mesh_lds);
    const int L = tb.L, S_max = od.S_max;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nthreads = blockDim.x;
    const MeshSlice m = mesh_slice(ws, per_group, L, n_dev);
    const int64_t m_cap = tb.M;
    if (no_item(items)) return;

    for (;;) {
        __syncthreads();
        if (tid == 0) shared_int[0] = next_item(items, od.C);
        __syncthreads();
        const int c = shared_int[0];
        if (c < 0) break;
        const int S = od.ord_S[c], K = od.ord_G[c];
        const int64_t cap = t_max[c];
        const int32_t *og = od.ord_group + int64_t(c) * od.G_max;
        int32_t *sg = stage_group + int64_t(c) * S_max, *stp = stage_tp + int64_t(c) * S_max;
        int32_t *wu = warmup + int64_t(c) * S_max;
        auto fail = [&](int status) {
            write_failed(out, c, S_max, status);
            for (int s = tid; s < S_max; s += nthreads) { sg[s] = -1; stp[s] = -1; wu[s] = -1; }
        };
        int bad = (S < 1 || S > S_max || K < 1 || K > od.G_max) ? 1 : 0;
        if (!bad)
            for (int k = tid; k < K; k += nthreads) {
                const int g = og[k];
                if (g < 0 || g >= tb.G) { bad = 1; continue; }
                for (int q = 0; q < k; ++q)
                    if (og[q] == g) bad = 1;
                order[k] = uint16_t(g);
            }
        if (__syncthreads_or(bad)) { fail(HARP_CAND_INVALID); continue; }
        if (cap_out_of_range(tb, cap)) { fail(HARP_CAND_INVALID); continue; }
        if (tid == 0) {
            int64_t o = 0;
            offs[0] = 0;
            for (int k = 0; k < K; ++k) { o += tb.group_ndev[order[k]]; offs[k + 1] = int32_t(o); }
        }
        __syncthreads();
        const int Dtot = offs[K];
        if (S > L || S < K || S > Dtot || cap < 0) { fail(HARP_CAND_INFEASIBLE); continue; }
        if (Dtot <= kMeshGroupTable) {
            for (int k = 0; k < K; ++k)
                for (int d = offs[k] + tid; d < offs[k + 1]; d += nthreads) group_at[d] = uint16_t(k);
        }
        int64_t sum;
        if constexpr (kFast) sum = mesh_h1_pass_fast(tb, m, offs, order, group_at, sums_lds, K, S, n_dev, cap);
        else sum = mesh_h1_pass(tb, m, offs, order, group_at, K, S, n_dev, cap);
        if (sum == kInf) { fail(HARP_CAND_INFEASIBLE); continue; }
        if (tid == 0) mesh_h1_backtrack<kFast>(tb, m, offs, order, K, S, n_dev, cap, cuts, slot_g, slot_k, slot_first, count);
        __syncthreads();
        int32_t *sp = out.splits + int64_t(c) * (S_max + 1);
        int32_t *df = out.dev_first + int64_t(c) * S_max;
        for (int s = tid; s <= S_max; s += nthreads) sp[s] = s <= S ? cuts[s] : -1;
        for (int s = tid; s < S_max; s += nthreads) {
            sg[s] = s < S ? int32_t(slot_g[s]) : -1;
            stp[s] = s < S ? tb.tp[slot_k[s]] : -1;
            df[s] = s < S ? slot_first[s] : -1;
            wu[s] = s < S ? count[s] : -1;
        }
        if (wave == 0) {
            int64_t bott, iter;
            wave_score_partition(tb, S, slot_g, slot_k, cuts, lane, bott, iter);   // the plan's own bottleneck
            if (lane == 0) {
                out.bottleneck[c] = bott;
                out.iter_time[c] = sum + (m_cap - 1) * cap;
                out.status[c] = HARP_CAND_OK;
            }
        }
    }
}

template <bool kFast>
__global__ __launch_bounds__(kMeshMaxThreads) void k2_mesh_h1f1b(TablesDev tb, OrdDev od, const int64_t *t_max,
                                                                 PlansDev out, int32_t *stage_group,
                                                                 int32_t *stage_tp, int32_t *warmup,
                                                                 unsigned char *ws, size_t per_group,
                                                                 int64_t n_dev, MeshItems items) {
    mesh_h1_body<kFast>(tb, od, t_max, out, stage_group, stage_tp, warmup, ws, per_group, n_dev, items);
}

// ------------------------------------------------------------------------------------ band form

// Bound by latency where rows are short - stages one after the other, a barrier or two each, serial parts on a wavefront
// or two (chains, plan recovery) - and by vector issue where they are long, which few orderings have and all wait for.
// Measured against the whole-table form on 32-bit rows it replaces: 4,096 orderings of 82 operators and 64 devices 3.57 ->
// 0.58-0.80 ms (of an ordering's 128 us 44% the value pass, 24% the chains, 13% the reach tables, 13% plan and score); exact
// form, 256 orderings of 160 operators and 128 devices, 15-19 -> 2.2-3.1 ms (of an ordering's 1.1 ms 54% the least-sum
// passes, 16% the min-max pass, 10% the chains, 15% plans and scores; the longest takes twice that).  Tried in vain: five
// workgroups of 256 threads on a CU (680 -> 705 us), a cell requested while the one before it is worked (exact form 10% slower).
// The exact form walks the caps as k2_mesh does: first at t_S, then down from ceil(T / B).  A plan that
// is not kept costs nothing but its score: the outputs are written whenever a better one is found.
template <bool kExact>
__global__ __launch_bounds__(1024) void k2_mesh_band(TablesDev tb, OrdDev od, PlansDev out, int32_t *stage_group,
                                                    int32_t *stage_tp, int32_t *n_passes, BandArgs ba) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    __shared__ int64_t scored[2];
    __shared__ int item;
    Band b(tb, ba.sh, lds_raw, ba.lo_tab, ba.hi_tab,
           meshband::band_slice(ba.slices + size_t(blockIdx.x) * ba.per_group, ba.sh));
    const int S_max = od.S_max, tid = threadIdx.x;
    const int64_t m_cap = tb.M;
    b.find_least_cut();
    for (;;) {
        __syncthreads();
        if (tid == 0) item = atomicAdd(&ba.counters[0], 1);
        __syncthreads();
        const int c = item;
        if (c >= od.C) break;
        int32_t *sg = stage_group + int64_t(c) * S_max, *stp = stage_tp + int64_t(c) * S_max;
        auto fail = [&](int status) {
            write_failed(out, c, S_max, status);
            for (int s = tid; s < S_max; s += b.nthreads) { sg[s] = -1; stp[s] = -1; }
            if (tid == 0 && n_passes) n_passes[c] = 0;
        };
        const int verdict = b.load(od.ord_S[c], od.ord_G[c], od.ord_group + int64_t(c) * od.G_max, S_max, od.G_max);
        if (verdict == 1) { fail(HARP_CAND_INVALID); continue; }
        if (verdict == 2) { fail(HARP_CAND_INFEASIBLE); continue; }
        auto hand_over = [&]() { if (tid == 0) ba.redo[atomicAdd(&ba.counters[1], 1)] = c; };
        if (verdict == 3) { hand_over(); continue; }
        int form = Band::kMinMax, tries = 0, passes = 0;
        uint32_t cap = b.guess();
        bool guessed = true;
        int64_t t_S = 0, best_T = kInf, best_b = kInf;
        bool keys_fit = true;
        bool over = false;
        for (;;) {
            b.keys_fit = keys_fit;
            const int64_t v = b.template run<kExact ? Band::kMinMax | Band::kSum : Band::kMinMax>(form, cap);
            if (v == kInf) {
                if (form == Band::kSum || cap >= meshband::kTopCap) break;     // (a sum cannot fail at or above t_S)
                if (guessed && !b.reached) {
                    const int64_t next = b.bracket(cap);
                    if (next < 0) break;
                    cap = uint32_t(next);
                } else {
                    cap = Band::raised(cap, tries++);
                }
                guessed = false;
                continue;
            }
            b.find_plan(form == Band::kSum, uint32_t(v), cap);
            int64_t bn, T;
            b.score(scored, bn, T);
            if (form == Band::kMinMax) t_S = bn;
            else ++passes;
            if (T < best_T || (T == best_T && bn <= best_b)) {       // equal totals: the lower cap; equal caps: the capped plan
                best_T = T;
                best_b = bn;
                b.write_slots(out, c, S_max, sg, stp);
            }
            if (!kExact || b.S < 2) break;
            int64_t next_cap;
            if (form == Band::kMinMax) {
                // every cap of the walk is at most T / B rounded up; up to the first bound it needs no look at the operators
                const int64_t t_E = (best_T + m_cap - 1) / m_cap;
                if (t_E > b.largest_cap(meshband::kInfSum, true)) {
                    const uint64_t most = b.most_sum();
                    keys_fit = t_E <= b.largest_cap(most, true);
                    over = t_E > b.largest_cap(most, false);
                    if (over) break;
                }
                form = Band::kSum;
                next_cap = t_S;
            } else {
                if (passes >= (1 << 20) || bn > int64_t(cap)) break;  // cannot happen: the cap falls with every pass
                if (passes == 1) {
                    next_cap = (best_T + m_cap - 1) / m_cap;
                } else {
                    next_cap = bn - 1;
                    if (m_cap > 1) {
                        const int64_t bound = (best_T - v) / (m_cap - 1);
                        next_cap = next_cap < bound ? next_cap : bound;
                    }
                }
                if (next_cap <= t_S) break;
            }
            cap = next_cap < int64_t(meshband::kTopCap) ? uint32_t(next_cap) : meshband::kTopCap;
        }
        if (over) { hand_over(); continue; }
        if (best_T == kInf) { fail(HARP_CAND_INFEASIBLE); continue; }
        if (tid == 0) {
            out.bottleneck[c] = best_b;
            out.iter_time[c] = best_T;
            out.status[c] = HARP_CAND_OK;
            if (n_passes) n_passes[c] = passes;
        }
    }
}

__global__ __launch_bounds__(1024) void k2_mesh_band_h1f1b(TablesDev tb, OrdDev od, const int64_t *t_max, PlansDev out,
                                                          int32_t *stage_group, int32_t *stage_tp, int32_t *warmup,
                                                          BandArgs ba) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    __shared__ int item;
    Band b(tb, ba.sh, lds_raw, ba.lo_tab, ba.hi_tab,
           meshband::band_slice(ba.slices + size_t(blockIdx.x) * ba.per_group, ba.sh));
    const int S_max = od.S_max, tid = threadIdx.x;
    b.load_memory_sums();
    for (;;) {
        __syncthreads();
        if (tid == 0) item = atomicAdd(&ba.counters[0], 1);
        __syncthreads();
        const int c = item;
        if (c >= od.C) break;
        const int64_t cap = t_max[c];
        int32_t *sg = stage_group + int64_t(c) * S_max, *stp = stage_tp + int64_t(c) * S_max;
        int32_t *wu = warmup + int64_t(c) * S_max;
        auto fail = [&](int status) {
            write_failed(out, c, S_max, status);
            for (int s = tid; s < S_max; s += b.nthreads) { sg[s] = -1; stp[s] = -1; wu[s] = -1; }
        };
        const int verdict = b.load(od.ord_S[c], od.ord_G[c], od.ord_group + int64_t(c) * od.G_max, S_max, od.G_max);
        if (verdict == 1 || cap_out_of_range(tb, cap)) { fail(HARP_CAND_INVALID); continue; }
        if (verdict == 2 || cap < 0) { fail(HARP_CAND_INFEASIBLE); continue; }
        // (caps up to the first bound need no look at the operators)
        if (verdict == 3 || (cap > b.largest_cap(meshband::kInfSum, false) && cap > b.largest_cap(b.most_sum(), false))) {
            if (tid == 0) ba.redo[atomicAdd(&ba.counters[1], 1)] = c;
            continue;
        }
        b.count_cap = cap;
        const int64_t sum = b.run<Band::kH1>(Band::kH1, cap < int64_t(meshband::kTopCap) ? uint32_t(cap) : meshband::kTopCap);
        if (sum == kInf) { fail(HARP_CAND_INFEASIBLE); continue; }
        b.find_h1_plan();
        b.write_slots(out, c, S_max, sg, stp);
        for (int s = tid; s < S_max; s += b.nthreads) wu[s] = s < b.S ? b.warmup[s] : -1;
        if (b.wave == 0) {
            int64_t bott, iter;
            wave_score_partition(tb, b.S, b.slot_g, b.slot_k, b.cuts, tid & 63, bott, iter);   // the plan's own bottleneck
            if ((tid & 63) == 0) {
                out.bottleneck[c] = bott;
                out.iter_time[c] = sum + (int64_t(tb.M) - 1) * cap;
                out.status[c] = HARP_CAND_OK;
            }
        }
    }
}

__global__ void k2_mesh_clear(int *counters) {
    if (threadIdx.x < 8) counters[threadIdx.x] = 0;
}

}  // namespace

MeshWorkspace meshband::mesh_carve(const TablesDev &tb, int S_max, int C, void *ws) {
    auto up = [](size_t x) { return (x + 255) & ~size_t(255); };
    unsigned char *p = static_cast<unsigned char *>(ws);
    MeshWorkspace w;
    // no index: sequences too long for the band kernels, or an index too large
    w.index_bytes = tb.L <= kFastRowsMaxL ? fastdp::lo_table_bytes(tb.L, S_max, tb.M, tb.T, tb.n_tp) : 0;
    if (w.index_bytes > kFastIndexLimit) w.index_bytes = 0;
    size_t off = 0;
    w.counters = reinterpret_cast<int *>(p); off += 256;
    w.redo = reinterpret_cast<int *>(p + off); off += up(size_t(C) * sizeof(int));
    w.index = reinterpret_cast<uint16_t *>(p + off); off += up(w.index_bytes);
    w.slices = p + off;
    w.before_slices = off;
    return w;
}

// LDS of a band workgroup: `budget` bytes, more when the time rows need it; false when they do not fit
// the CU.
bool meshband::band_shape(const TablesDev &tb, int S_max, int G_max, int64_t total_devices, int form, size_t budget,
                          BandShape &sh) {
    if (total_devices > kMaxDevices) return false;
    sh.W = tb.L + 1;
    sh.NW = (sh.W + 63) / 64;
    sh.cols = int(total_devices) + 1;
    sh.K_cap = G_max < tb.G ? G_max : tb.G;
    sh.S_cap = S_max < tb.L ? S_max : tb.L;
    sh.idx_pitch = int(fastdp::lo_pitch(tb.L));
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t at = off; off = (off + bytes + 15) & ~size_t(15); return uint32_t(at); };
    sh.o_offs = take(size_t(sh.K_cap + 1) * 4);
    sh.o_order = take(size_t(sh.K_cap) * 2);
    sh.o_type = take(size_t(sh.K_cap) * 2);
    sh.o_row_at = take(size_t(sh.K_cap) * 16);
    sh.o_cut_at = take(size_t(sh.cols) * 4);
    sh.o_group_at = take(size_t(sh.cols) * 2);
    const bool sums = form == kFormSum || form == kFormSweep, h1 = form == kFormH1 || form == kFormSweep;
    sh.o_mem = take(h1 ? size_t(sh.W) * 16 : 0);
    sh.o_ok = take(size_t(kTeams) * 2 * sh.K_cap * sh.NW * 8);
    // (the chains of a cap are over before its first pass loads columns; with LDS of their own, large problems at the edge of what
    // fits went to the whole-table form: 32 orderings of 170 operators, 16 groups of 32 devices, a type each 55 -> 1.3 ms)
    const size_t chains = size_t(kTeams) * 2 * (sh.cols + 1) * 2, columns = size_t(sh.cols) * 24;
    sh.o_col = take(chains > columns ? chains : columns);
    sh.o_small = take(32 + size_t(sh.S_cap + 1) * 12 + size_t(sh.S_cap) * 11);
    // time rows: of every group when they fit half the budget, else of as many sets as do, at least one per type
    // (a set: its time rows and its two reach tables)
    const size_t per_set = size_t(tb.n_tp) * sh.W * 8;
    size_t sets = budget / 2 / per_set;
    const size_t least = size_t(tb.T < sh.K_cap ? tb.T : sh.K_cap);
    sets = sets < least ? least : sets;
    sh.set_cap = int(sets < size_t(sh.K_cap) ? sets : size_t(sh.K_cap));
    sh.o_use = take(size_t(sh.set_cap) * 4);
    sh.o_prow = take(16 + size_t(sh.set_cap) * per_set);
    // the rest of the budget holds rows (Band::place_rows), at least 1,024 cells in the widest form of a pass - two rows of
    // values, or one and the key rows, counts, the map - and the numbering of an ordering's sets
    const size_t value_rows = sums && tb.n_tp > 1 ? size_t(1 + tb.n_tp) : 2, cell = value_rows * 4 + (h1 ? 4 : 0) + 2;
    const size_t want = 1024 * cell + 256, numbering = size_t(sh.K_cap) * 2;
    const size_t room = want > numbering ? want : numbering;
    sh.o_set_of = uint32_t(off);
    sh.total = uint32_t(off + room > budget ? off + room : budget & ~size_t(15));
    return sh.total <= kBandLds;
}

// Workgroups of the band kernels: a batch of at most one ordering per CU gets the whole CU's LDS and
// 1,024 threads each; beyond that two workgroups of 512 threads share a CU (the key rows of the exact form
// and the rows of the H-1F1B form want the room), or four of 256 in the min-max form where there are slices for
// four: large tables have two per CU, and there, on 160 operators and 128 devices, 600 / 1,024 / 4,096 orderings
// take 1.45 / 2.01 / 5.47 ms with two workgroups of 512, 2.24 / 2.37 / 5.40 ms with four of 256.
bool meshband::band_launch(const TablesDev &tb, const OrdDev &od, int64_t total_devices, int form, int n_cu, int n_groups,
                           int &threads, BandShape &sh) {
    const int want = od.C < 4 * n_cu ? od.C : 4 * n_cu;
    threads = od.C <= n_cu ? 1024 : (form != kFormMinMax || od.C <= 2 * n_cu || n_groups < want) ? 512 : 256;
    const size_t budget = threads == 1024 ? (size_t(156) << 10) : threads == 512 ? (size_t(79) << 10) : (size_t(39) << 10);
    return band_shape(tb, od.S_max, od.G_max, total_devices, form, budget, sh);
}

// Threads of a whole-table workgroup: a stage has up to L x devices target cells, so small tables get many
// small workgroups (more orderings in flight), large ones few large workgroups (more lanes per ordering).
int plan_mesh_threads(int L, int64_t total_devices, int C, int n_cu) {
    if (int64_t(L + 1) * (total_devices + 1) >= 16384) return kMeshMaxThreads;
    // a batch too small to fill the chip with 256-thread workgroups gets more lanes per ordering
    if (C <= 2 * n_cu) return kMeshMaxThreads;
    if (C <= 4 * n_cu) return 512;
    return 256;
}

// Per-workgroup slice: two rows of the table, the back-pointers; or the ranges and value rows of the band form.
size_t plan_mesh_ws_per_group(int L, int S_max, int64_t total_devices) {
    const size_t row = size_t(total_devices + 1) * size_t(L + 1);
    size_t b = 2 * row * sizeof(int64_t) + 2 * row * sizeof(int32_t) + size_t(S_max) * row * sizeof(uint32_t);
    const size_t band = meshband::band_slice_bytes(L, S_max, total_devices);
    b = b > band ? b : band;
    return (b + 255) & ~size_t(255);
}

size_t plan_mesh_ws_fixed(const TablesDev &tb, int S_max, int C) {
    return mesh_carve(tb, S_max, C, nullptr).before_slices;
}

namespace {

// Problems whose whole tables are worked faster than the ranges of their cuts are found.  A stage of the whole
// table costs about (cuts) x (device offsets) x (degrees) x (cuts scanned).  With S stages it can end at most at
// L - S + 1 cuts and devices - S + 1 offsets (every stage takes one of each); the H-1F1B form scans all L + 1.  The
// ranges cost a few serial steps per stage whatever the size: a workgroup's lanes make the product cheap, and many
// orderings share the lanes.  The orderings' own stage counts are not known here, so S is the largest.
// Measured on 260 random problems of 10 to 160 operators, up to 80 devices and 4,096 orderings, product: whole
// table / ranges, us.  Min-max: 1,680 (49 operators, 47 stages on 80 devices): 228 / 552; 106,090: 74 / 60; 145,800:
// 190 / 157; 165,375: 55 / 91; 53,792 with 2,767 orderings: 1,468 / 910.  Exact: 44,944: 127 / 92; 61,952: 1,335 /
// 1,668; 77,976: 608 / 531; 92,256: 5,600 / 3,406.  H-1F1B: 22,050: 69 / 86; 27,378: 290 / 246; 51,076: 48 / 66; 59,168: 238 / 202; 102,966: 151 / 79.
// The form chosen takes 1.017 x the faster one's time on average and 1.9 x at most; the whole table always 1.15 x and
// 6.8 x, the ranges always 1.7 x and 7.9 x.
bool whole_table(const TablesDev &tb, const OrdDev &od, int64_t total_devices, int form, int n_cu) {
    const int64_t most = total_devices < tb.L ? total_devices : tb.L, stages = od.S_max < most ? od.S_max : most;
    const int64_t cuts = form == meshband::kFormH1 ? tb.L + 1 : tb.L - stages + 2;
    if (cuts > 1024) return false;
    const double per_cu = od.C > n_cu && form != meshband::kFormH1 ? sqrt(double(od.C) / n_cu) : 1.0;
    const double limit = form == meshband::kFormH1 ? 20e3 : form == meshband::kFormSum ? 70e3 : 160e3;
    return double(cuts * cuts * (total_devices - stages + 2) * tb.n_tp) * per_cu <= limit;
}

// The band launch of a batch and, behind it, the whole-table launch over what it handed over.  band(sh, ...)
// and whole(fast, items, ...) launch the two kernels.  The status of the first launch is read before the second
// can replace it: without the first the second has nothing to take over.
template <typename BandFn, typename WholeFn>
hipError_t mesh_launch(const TablesDev &tb, const OrdDev &od, bool fast32, int form, void *ws, int n_groups, int threads,
                 int64_t total_devices, int n_cu, hipStream_t st, BandFn band, WholeFn whole) {
    const MeshWorkspace w = mesh_carve(tb, od.S_max, od.C, ws);
    const size_t per_group = plan_mesh_ws_per_group(tb.L, od.S_max, total_devices);
    hipLaunchKernelGGL(k2_mesh_clear, dim3(1), dim3(64), 0, st, w.counters);
    BandArgs ba;
    int band_threads = 0;
    const bool fast = fast32 && tb.L <= kMeshFastMaxL;       // (sums of memory in LDS)
    // whole-table workgroups: as many as are resident, also behind the band kernel, which can hand over the whole
    // batch (4,096 orderings of 82 operators and 64 devices in the H-1F1B form, all handed over: 16.6 ms on one
    // workgroup per CU, 7.4 ms on eight)
    const long long resident = (long long)n_cu * (2048 / threads);
    const dim3 grid(unsigned(n_groups < resident ? n_groups : resident));
    if (fast32 && w.index_bytes != 0 && !whole_table(tb, od, total_devices, form, n_cu) &&
        meshband::band_launch(tb, od, total_devices, form, n_cu, n_groups, band_threads, ba.sh)) {
        launch_plan_index(tb, od.S_max, w.index, st);
        ba.lo_tab = w.index;
        ba.hi_tab = w.index + w.index_bytes / 4;
        ba.slices = w.slices;
        ba.per_group = per_group;
        ba.counters = w.counters;
        ba.redo = w.redo;
        const int band_resident = n_cu * (1024 / band_threads);
        band(dim3(n_groups < band_resident ? n_groups : band_resident), dim3(band_threads), size_t(ba.sh.total), ba);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        whole(fast, grid, dim3(threads), MeshItems{w.counters + 2, w.redo, w.counters + 1}, w.slices, per_group);
    } else {
        whole(fast, grid, dim3(threads), MeshItems{w.counters, nullptr, nullptr}, w.slices, per_group);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_plan_mesh(const TablesDev &tb, const OrdDev &od, const PlansDev &out, int32_t *stage_group,
                      int32_t *stage_tp, int32_t *n_passes, bool exact, bool fast32, void *ws, int n_groups,
                      int threads, int64_t total_devices, int n_cu, hipStream_t st) {
    return mesh_launch(tb, od, fast32, exact ? meshband::kFormSum : meshband::kFormMinMax, ws, n_groups, threads, total_devices, n_cu, st,
                [&](dim3 grid, dim3 block, size_t lds, const BandArgs &ba) {
                    if (exact)
                        hipLaunchKernelGGL(k2_mesh_band<true>, grid, block, lds, st, tb, od, out, stage_group, stage_tp,
                                           n_passes, ba);
                    else
                        hipLaunchKernelGGL(k2_mesh_band<false>, grid, block, lds, st, tb, od, out, stage_group, stage_tp,
                                           n_passes, ba);
                },
                [&](bool fast, dim3 grid, dim3 block, const MeshItems &items, unsigned char *slices, size_t per_group) {
                    const size_t lds = fast ? size_t(tb.L + 1) * sizeof(int64_t) : 0;
#define HARP_MESH_LAUNCH(E, F)                                                                                     \
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k2_mesh<E, F>), grid, block, lds, st, tb, od, out, stage_group, stage_tp,   \
                       n_passes, slices, per_group, total_devices, items)
                    if (exact && fast) HARP_MESH_LAUNCH(true, true);
                    else if (exact) HARP_MESH_LAUNCH(true, false);
                    else if (fast) HARP_MESH_LAUNCH(false, true);
                    else HARP_MESH_LAUNCH(false, false);
#undef HARP_MESH_LAUNCH
                });
}

hipError_t launch_plan_mesh_h1f1b(const TablesDev &tb, const OrdDev &od, const int64_t *t_max, const PlansDev &out,
                            int32_t *stage_group, int32_t *stage_tp, int32_t *warmup, bool fast32, void *ws,
                            int n_groups, int threads, int64_t total_devices, int n_cu, hipStream_t st) {
    return mesh_launch(tb, od, fast32, meshband::kFormH1, ws, n_groups, threads, total_devices, n_cu, st,
                [&](dim3 grid, dim3 block, size_t lds, const BandArgs &ba) {
                    hipLaunchKernelGGL(k2_mesh_band_h1f1b, grid, block, lds, st, tb, od, t_max, out, stage_group,
                                       stage_tp, warmup, ba);
                },
                [&](bool fast, dim3 grid, dim3 block, const MeshItems &items, unsigned char *slices, size_t per_group) {
                    const size_t lds = fast ? 2 * size_t(tb.L + 1) * sizeof(int64_t) : 0;
                    if (fast)
                        hipLaunchKernelGGL(k2_mesh_h1f1b<true>, grid, block, lds, st, tb, od, t_max, out, stage_group,
                                           stage_tp, warmup, slices, per_group, total_devices, items);
                    else
                        hipLaunchKernelGGL(k2_mesh_h1f1b<false>, grid, block, lds, st, tb, od, t_max, out, stage_group,
                                           stage_tp, warmup, slices, per_group, total_devices, items);
                });
}

}  // namespace harp
