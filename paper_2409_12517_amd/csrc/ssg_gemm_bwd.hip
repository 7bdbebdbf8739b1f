// FP8 MFMA GEMMs of the backward pass for gfx950: the single-launch forms (dH with the SwiGLU derivative fused,
// the input gradient as a sum of two products) and the grouped launches, in which the tiles of several
// independent GEMMs share one grid.
//
// Why grouped: every GEMM of the block at the Llama2-7B shape has a tile count that is not a multiple of the 256
// compute units (688 tiles = 2.69 rounds), so each launch ends with a partly empty round; and within one GEMM all
// workgroups reach their epilogue at the same moment, so its global traffic (U, G reads and dU, dG writes of dH;
// 64 MB of fp32 per round of a weight gradient) hits memory in bursts while the matrix cores idle.  In a grouped
// launch the workgroups of the next GEMM follow those of the previous one in dispatch order, so its first tiles
// start on the compute units the previous GEMM's last round leaves idle.  (Alternating the members' workgroups
// instead -- so that tiles of different lengths drift out of phase -- measured 10 % slower for {dH, dW3}: two
// working sets share each XCD's L2 and every member's patch of concurrent tiles is half as large.)
#include <algorithm>
#include <functional>
#include <vector>

#include "ssg_gemm_tile.h"
#include "ssg_scaling.h"

namespace ssg {

// Up to four GEMMs in one grid, one of them perhaps as two members, one after the other in dispatch order, all in the same
// tile (gemm_wave_blocks).
// Workgroups are dealt in sets of 8 large tiles (see set_of: one per XCD, so that vblock % 8 stays the XCD inside each
// GEMM and map_tile's per-XCD patches survive); member i runs sets [first[i], first[i] + sets[i]) of its GEMM -- a GEMM
// may be split between two launches at a set boundary.
// (second group: dX is member 0, or, where its products have tiles of their own, members 0 and 1; dW1, dW2, dW3 are 2 to 4)
struct GroupParams {
    GemmParams p[5];
    int sets[5];
    int first[5];
    int tile_blocks;        // workgroups of all sets
};

// dH (with the SwiGLU derivative; EPI = EPI_SWIGLU_BWD or EPI_SWIGLU_BWD_Q), then the first part of dW3: both read dY^.
template <int WB, int EPI>
__global__ void __launch_bounds__(kThreads, waves_per_simd(WB)) gemm_group_dh_dw3_kernel(GroupParams g) {
    __shared__ __attribute__((aligned(1024))) uint8_t smem[smem_bytes(WB)];
    const int G = set_of<WB>((int)blockIdx.x), x = (int)(blockIdx.x & 7), q = quarter_of<WB>((int)blockIdx.x);
    if (G < g.sets[0]) {
        const int vb = G * 8 + x;
        if (vb < g.p[0].tiles_m * g.p[0].tiles_n) gemm_tile<WB, EPI, kE5M2, 0, 1>(g.p[0], vb, q, smem);
    } else {
        const int vb = (G - g.sets[0] + g.first[1]) * 8 + x;
        if (vb < g.p[1].tiles_m * g.p[1].tiles_n) gemm_tile<WB, EPI_STORE, kE5M2, 0, 2>(g.p[1], vb, q, smem);
    }
}

// dX (PART = 3: the sum of two products in one tile; 4: the products in tiles of their own.  The long tiles, dealt first),
// then dW1, dW2 and the rest of dW3.
template <int WB, int PART>
__global__ void __launch_bounds__(kThreads, waves_per_simd(WB)) gemm_group_dx_dw_kernel(GroupParams g, ScalingUpdate update) {
    __shared__ __attribute__((aligned(1024))) uint8_t smem[smem_bytes(WB)];
    int G = set_of<WB>((int)blockIdx.x);
    const int x = (int)(blockIdx.x & 7), q = quarter_of<WB>((int)blockIdx.x);
    const int dx_sets = g.sets[0] + (PART == 4 ? g.sets[1] : 0);
    if (G < dx_sets) {
        const int half = PART == 4 && G >= g.sets[0] ? 1 : 0;
        const int vb = (G - half * g.sets[0]) * 8 + x;
        if (vb < g.p[0].tiles_m * g.p[0].tiles_n) gemm_tile<WB, EPI_STORE, kE5M2, PART, 1>(g.p[half], vb, q, smem);
        return;
    }
    G -= dx_sets;
    int m = 2;
    if (G >= g.sets[2]) { G -= g.sets[2]; m = 3; if (G >= g.sets[3]) { G -= g.sets[3]; m = 4; } }
    if (m == 4 && G >= g.sets[4]) {
        // the workgroups after the last tile: the ranges of dY, dU, dG are complete and nothing here reads the state
        const int k = (int)blockIdx.x - g.tile_blocks;
        if (k < update.count && threadIdx.x < 64) scaling_update_wave(update, k, (int)threadIdx.x);
        return;
    }
    const GemmParams &p = g.p[m];
    const int vb = (G + g.first[m]) * 8 + x;
    if (vb < p.tiles_m * p.tiles_n) gemm_tile<WB, EPI_STORE, kE5M2, 0, 2>(p, vb, q, smem);
}

int gemm_tile_sets(const GemmArgs &a) { return sets_of(make_gemm_params(a)); }

static bool is_wgrad(const GemmArgs &a) { return a.epilogue == EPI_STORE && a.part == 0 && a.layout == 2 && a.a_fmt == kE5M2; }

bool gemm_group_ok(const GemmArgs *const *list, int n) {
    if (n < 2 || n > 4) return false;
    for (int i = 0; i < n; ++i)
        if (!list[i] || !gemm_args_ok(*list[i])) return false;
    if (n == 2) {
        const GemmArgs &a = *list[0];
        return (a.epilogue == EPI_SWIGLU_BWD || a.epilogue == EPI_SWIGLU_BWD_Q) && a.a_fmt == kE5M2 && is_wgrad(*list[1]);
    }
    for (int i = 1; i < n; ++i)
        if (!is_wgrad(*list[i])) return false;
    return list[0]->epilogue == EPI_STORE && list[0]->part >= 3;
}

// ---- where to split a weight gradient between the two grouped launches of the backward ------------------------
// Workgroups are dispatched in order to whichever compute unit is free, and a tile's time is known well enough
// from its K steps and its epilogue, so the end of a launch can be predicted by replaying that dispatch.  A launch
// whose last tiles start a round of their own pays a whole tile time for them; moving sets of the weight gradient
// from the first launch to the second (or back) shifts work between the two launches' last rounds.
static double replay_dispatch(const double *cost, const int *tiles, int n, int units, std::vector<double> &free_at) {
    // free_at: a min-heap of the times at which the compute units become free
    free_at.assign((size_t)units, 0.0);
    double end = 0.0;
    for (int i = 0; i < n; ++i)
        for (int t = 0; t < tiles[i]; ++t) {
            std::pop_heap(free_at.begin(), free_at.end(), std::greater<double>());
            const double done = free_at.back() + cost[i];
            free_at.back() = done;
            std::push_heap(free_at.begin(), free_at.end(), std::greater<double>());
            end = done > end ? done : end;
        }
    return end;
}

int gemm_group_split_sets(const GemmArgs &dh, const GemmArgs &dw_split, const GemmArgs *const *second, int n_second,
                          int units) {
    const int all = gemm_tile_sets(dw_split);
    if (units <= 0 || n_second < 1 || n_second > 3) return all;
    const GemmParams ph = make_gemm_params(dh), pw = make_gemm_params(dw_split);
    const int tiles_w = pw.tiles_m * pw.tiles_n;
    double cost_b[4]; int tiles_b[4];
    // (where dX runs in halves, its tiles are short and the stores weigh more: 7.5 fp32, 4.5 bf16, 8 where the halves meet)
    const bool halves = second[0]->part == 4;
    auto cost_of = [&](const GemmArgs &a) {
        return gemm_tile_cost(a, 4) + (!halves ? 0.0 : (a.c_f32 ? -2.5 : -1.5) + (a.part == 4 ? 8.0 : 0.0));
    };
    for (int i = 0; i < n_second; ++i) {
        const GemmParams p = make_gemm_params(*second[i]);
        cost_b[i] = cost_of(*second[i]); tiles_b[i] = p.tiles_m * p.tiles_n * (second[i]->part == 4 ? 2 : 1);
    }
    cost_b[n_second] = cost_of(dw_split);
    const double cost_a[2] = {gemm_tile_cost(dh, 4), cost_of(dw_split)};
    std::vector<double> heap;
    // the predicted time is a step function of the split.  Of the longest run of equally good splits take a point a
    // quarter of the run below its upper end: measured, the second launch behaves like a fluid (its tiles have
    // drifted out of step, so every set moved there costs its share of time) while the first shows the predicted
    // step, so the best split moves as few sets as make the step, with a margin for tile times that differ a little
    // from the estimates
    std::vector<double> t((size_t)all + 1);
    double best = 0.0;
    for (int s = 0; s <= all; ++s) {
        const int in_a = s * 8 < tiles_w ? s * 8 : tiles_w;
        const int ta[2] = {ph.tiles_m * ph.tiles_n, in_a};
        tiles_b[n_second] = tiles_w - in_a;
        t[(size_t)s] = replay_dispatch(cost_a, ta, 2, units, heap) + replay_dispatch(cost_b, tiles_b, n_second + 1, units, heap);
        if (s == 0 || t[(size_t)s] < best) best = t[(size_t)s];
    }
    if (t[(size_t)all] <= best + 1e-9) return all;             // nothing to gain: dW3 stays whole in the first launch
    int best_lo = all, best_len = 0;
    for (int s = 0; s <= all;) {
        if (t[(size_t)s] > best + 1e-9) { ++s; continue; }
        int e = s;
        while (e + 1 <= all && t[(size_t)(e + 1)] <= best + 1e-9) ++e;
        if (e - s + 1 >= best_len) { best_len = e - s + 1; best_lo = s; }     // of equal runs, the one that moves least
        s = e + 1;
    }
    return best_lo + (best_len - 1) - (best_len - 1) / 4;
}

template <int WB>
static void launch_group_wb(const GroupParams &g, int part, int epilogue, dim3 grid, const ScalingUpdate &update, hipStream_t st) {
    const dim3 with_update(grid.x + (unsigned)update.count);
    if (part == 4) hipLaunchKernelGGL((gemm_group_dx_dw_kernel<WB, 4>), with_update, dim3(kThreads), 0, st, g, update);
    else if (part == 3) hipLaunchKernelGGL((gemm_group_dx_dw_kernel<WB, 3>), with_update, dim3(kThreads), 0, st, g, update);
    else if (epilogue == EPI_SWIGLU_BWD) hipLaunchKernelGGL((gemm_group_dh_dw3_kernel<WB, EPI_SWIGLU_BWD>), grid, dim3(kThreads), 0, st, g);
    else hipLaunchKernelGGL((gemm_group_dh_dw3_kernel<WB, EPI_SWIGLU_BWD_Q>), grid, dim3(kThreads), 0, st, g);
}
static bool launch_group(GroupParams &g, int wb, int part, int epilogue, int tag, double flops, const ScalingUpdate &update, hipStream_t st) {
    int sets = 0;
    for (int m = 0; m < 5; ++m) sets += g.sets[m];
    if (sets == 0) return true;
    const dim3 grid((unsigned)sets * set_workgroups(wb));
    g.tile_blocks = (int)grid.x;
    profile_before(tag, st, flops);
    if (wb == 4) launch_group_wb<4>(g, part, epilogue, grid, update, st);
    else launch_group_wb<2>(g, part, epilogue, grid, update, st);
    profile_after(st);
    return true;
}

// The split member is the last one of either group: the first launch runs its sets [0, split), the second the rest.
static int last_member_sets(int n, int split_sets, int all) {
    const int cut = split_sets < all ? split_sets : all;
    return split_sets < 0 || n == 3 ? all : n == 2 ? cut : all - cut;
}

int gemm_group_wave_blocks(const GemmArgs *const *list, int n, int split_sets) {
    const int all = gemm_tile_sets(*list[n - 1]);
    return gemm_wave_blocks(list, n, (double)last_member_sets(n, split_sets, all) / (double)all);
}

// The member that list[i] is (the second group keeps member 1 for the second product of dX).
static int member_of(int part, int i) { return part && i > 0 ? i + 1 : i; }

bool launch_gemm_group(const GemmArgs *const *list, int n, int split_sets, hipStream_t st, const ScalingUpdate &update) {
    if (!gemm_group_ok(list, n)) return false;
    const int part = list[0]->part;
    GroupParams g;
    double flops = 0.0;
    for (int m = 0; m < 5; ++m) { g.p[m] = make_gemm_params(*list[0]); g.sets[m] = 0; g.first[m] = 0; }
    for (int i = 0; i < n; ++i) {
        const int m = member_of(part, i);
        g.p[m] = make_gemm_params(*list[i]);
        g.sets[m] = sets_of(g.p[m]);
    }
    const int last = member_of(part, n - 1), all = g.sets[last];
    g.sets[last] = last_member_sets(n, split_sets, all);
    if (n == 4) g.first[last] = all - g.sets[last];
    // The fp32 weight gradients of the second launch go out through non-temporal stores: nothing reads them before
    // the optimizer, and kept out of the caches they leave in place what the passes after this launch read (measured
    // at the Llama2-7B shape: -10 us per step, in the launches that follow, not in this one).  In the first launch,
    // beside dH's epilogue traffic, the same stores cost 3-7 us: left as they are.
    for (int m = 2; m < 5; ++m) g.p[m].nt_store = part != 0;
    for (int i = 0; i < n; ++i) {
        // flops of the tiles this launch runs (a last set may be partly beyond the GEMM's tile count)
        const int m = member_of(part, i), tiles = g.p[m].tiles_m * g.p[m].tiles_n;
        const int hi = std::min((g.first[m] + g.sets[m]) * 8, tiles), lo = std::min(g.first[m] * 8, tiles);
        flops += gemm_flops(*list[i]) * (double)(hi - lo) / (double)tiles;
    }
    if (part == 4) { g.p[1] = make_gemm_params(*list[0], 1); g.sets[1] = g.sets[0]; }
    return launch_group(g, gemm_group_wave_blocks(list, n, split_sets), part, list[0]->epilogue, n == 2 ? 16 : 17, flops, update, st);
}

// The backward forms launched on their own (a.part != 0, or one of the SwiGLU-backward epilogues); the
// argument set has passed gemm_args_ok.
template <int WB>
static void launch_bwd_wb(const GemmArgs &a, hipStream_t st) {
    const GemmParams p = make_gemm_params(a);
    const dim3 grid((unsigned)sets_of(p) * set_workgroups(WB));
    if (a.epilogue == EPI_SWIGLU_BWD) hipLaunchKernelGGL((gemm_kernel<WB, EPI_SWIGLU_BWD, kE5M2, 0, 1>), grid, dim3(kThreads), 0, st, p);
    else if (a.epilogue == EPI_SWIGLU_BWD_Q) hipLaunchKernelGGL((gemm_kernel<WB, EPI_SWIGLU_BWD_Q, kE5M2, 0, 1>), grid, dim3(kThreads), 0, st, p);
    else hipLaunchKernelGGL((gemm_kernel<WB, EPI_STORE, kE5M2, 3, 1>), grid, dim3(kThreads), 0, st, p);
}

bool launch_gemm_bwd(const GemmArgs &a, hipStream_t st) {
    const GemmParams p = make_gemm_params(a);
    const dim3 grid((unsigned)sets_of(p) * set_workgroups(4));
    const GemmArgs *one = &a;
    if (a.part == 4) {                                   // the second group without its weight gradients
        GroupParams g;
        for (int m = 0; m < 5; ++m) { g.p[m] = make_gemm_params(a, m == 1); g.sets[m] = m < 2 ? sets_of(p) : 0; g.first[m] = 0; }
        return launch_group(g, gemm_wave_blocks(&one, 1), 4, a.epilogue, gemm_profile_tag(a), gemm_flops(a), {}, st);
    }
    profile_before(gemm_profile_tag(a), st, gemm_flops(a));
    if (a.epilogue == EPI_SWIGLU_BWD && a.a_fmt == kBF16)
        hipLaunchKernelGGL((gemm_kernel<4, EPI_SWIGLU_BWD, kBF16, 0, 0>), grid, dim3(kThreads), 0, st, p);
    else if (a.part == 1) hipLaunchKernelGGL((gemm_kernel<4, EPI_STORE, kE5M2, 1, 1>), grid, dim3(kThreads), 0, st, p);
    else if (a.part == 2) hipLaunchKernelGGL((gemm_kernel<4, EPI_STORE, kE5M2, 2, 1>), grid, dim3(kThreads), 0, st, p);
    else if (gemm_wave_blocks(&one, 1) == 4) launch_bwd_wb<4>(a, st);
    else launch_bwd_wb<2>(a, st);
    profile_after(st);
    return true;
}

}  // namespace ssg
