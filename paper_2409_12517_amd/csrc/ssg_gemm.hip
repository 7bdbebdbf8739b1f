// FP8 MFMA GEMMs for gfx950, one GEMM per launch: the plain store forms of every operand layout (the public
// contraction entry points; y of the block) and the two forward forms with the fused SwiGLU epilogues.
// The backward forms and the grouped launches are instantiated in ssg_gemm_bwd.hip.
#include <algorithm>

#include "ssg_col_range.h"
#include "ssg_gemm_tile.h"

namespace ssg {

// The gate/up GEMM with an independent streaming pass in its grid.  1376 tiles on 256 compute units are 5.4
// rounds: during the last one 160 units would idle.  The workgroups after the last tile take the per-channel range
// of w3 (Section 4.4; it depends on no result of this GEMM and is needed only after it), so that pass costs little time
// of its own.  A workgroup of this kernel owns a whole compute unit (registers, LDS) with large tiles and shares it with one
// other with small ones, hence 16 loads in flight per lane.
struct ColRangeParams {
    const uint16_t *src;
    int64_t rows, cols;
    uint32_t *camax_bits;
    int blocks_x;
};
template <int WB>
__global__ void __launch_bounds__(kThreads, waves_per_simd(WB)) gemm_swiglu_col_range_kernel(GemmParams p, ColRangeParams r) {
    __shared__ __attribute__((aligned(1024))) uint8_t smem[smem_bytes(WB)];
    const int tiles = p.tiles_m * p.tiles_n, gemm_blocks = p.sets * (WB == 4 ? 8 : 32);
    if ((int)blockIdx.x < gemm_blocks) {
        const int b = (int)blockIdx.x, vb = (p.first_set + set_of<WB>(b)) * 8 + (b & 7);
        if (vb < tiles) gemm_tile<WB, EPI_SWIGLU, kE4M3, 0, 0>(p, vb, quarter_of<WB>(b), smem);
    } else {
        const int b = (int)blockIdx.x - gemm_blocks;
        col_range_bf16_block<16>(r.src, r.rows, r.cols, r.camax_bits, b % r.blocks_x, b / r.blocks_x,
                                 reinterpret_cast<uint32_t *>(smem));
    }
}

static bool is_dual(const GemmArgs &a) { return a.epilogue == EPI_SWIGLU || a.epilogue == EPI_SWIGLU_Q; }

bool gemm_args_ok(const GemmArgs &a) {
    if (a.epilogue < EPI_STORE || a.epilogue > EPI_SWIGLU_BWD_Q) return false;
    if (!a.A || !a.B || !a.C || a.M <= 0 || a.N <= 0 || a.K <= 0) return false;
    if (a.a_fmt != kE4M3 && a.a_fmt != kE5M2 && a.a_fmt != kBF16) return false;
    // bf16 operands: the two forms the unquantized last layer needs, K-contiguous operands only
    if (a.a_fmt == kBF16 && (a.layout != 0 || a.part != 0 || (a.epilogue != EPI_STORE && a.epilogue != EPI_SWIGLU_BWD))) return false;
    const bool dual = is_dual(a);
    if (dual && (!a.B2 || a.a_fmt != kE4M3 || a.layout != 0)) return false;
    if (a.epilogue == EPI_SWIGLU && (!a.C2 || !a.camax_bits)) return false;
    if (a.tail_src && (a.epilogue != EPI_SWIGLU || !a.tail_camax_bits || a.tail_rows <= 0 || a.tail_cols <= 0 ||
                       a.tail_cols % 8 != 0 || (reinterpret_cast<uintptr_t>(a.tail_src) & 15u)))
        return false;
    if (a.part != 0 && a.epilogue != EPI_STORE) return false;
    if (a.layout < 0 || a.layout > 2) return false;
    const bool bwd = a.epilogue == EPI_SWIGLU_BWD || a.epilogue == EPI_SWIGLU_BWD_Q;
    // the backward forms are built for the block's own use: gradient operand E5M2, weight operand K-major
    if (bwd && a.a_fmt != kBF16 && (a.layout != 1 || a.a_fmt != kE5M2)) return false;
    if (a.epilogue == EPI_SWIGLU_BWD_Q && (!a.q_scale || !a.q_scale2 || !a.q_scale_out || !a.q_scale_out2)) return false;
    if (a.part < 0 || a.part > 4) return false;
    if (a.part != 0 && (a.layout != 1 || a.a_fmt != kE5M2)) return false;
    if ((a.part == 2) != (a.add != nullptr)) return false;
    if (a.part == 1 && !a.c_f32) return false;
    if (a.part == 4 && (!a.partials || !a.arrivals)) return false;
    if ((a.part >= 3) != (a.A_ph2 != nullptr) || (a.part >= 3 && (!a.B_ph2 || !a.sa || !a.sb || !a.sa_ph2 || !a.sb_ph2))) return false;
    if ((a.keep_u != nullptr) != (a.keep_g != nullptr) || (a.keep_u && a.epilogue != EPI_SWIGLU_BWD_Q)) return false;
    if (bwd && (!a.U || !a.G || !a.C2 || !a.amax_bits || !a.amax_bits2)) return false;
    return true;
}

// The large tile's form of a sum of two products has no general loop body: whole K steps only, at least two.
static bool sum_in_large_tile_ok(int64_t K) { return K % BK == 0 && K >= 2 * BK; }

// ---- which tile computes a launch --------------------------------------------------------------------------------
// The 256 x 256 tile reads half as many operand bytes per product as the 128 x 128 one and keeps the matrix cores
// about 90 % busy where it fills the chip (y at T = 4096, d = 4096, f = 11008: 123 us against 150); the small one has
// four times the workgroups, two to a compute unit, whose epilogues run under each other's main loops (y at T = 2048,
// d = 2048, f = 5504, 64 large tiles for 256 compute units: 50 us against 25).  Which wins is a matter of how many
// tiles there are, of how their rows lie to the cache lines and of what comes from HBM, so the time of a launch is
// estimated for both and the smaller one taken.  Over 1499 contractions (16 to 8192 rows, up to 28672 columns and K) the
// choice takes 1.8 % longer on average than the best route measured (large tiles, small ones, whole rounds and a rest, few
// rows); 17 are more than 3 % slower than large tiles alone, the worst 1.15 times (5504 x 2384 x 1056, both K-major).  Over 964
// GEMMs of the forward and inference forms 1.2 %, 7 and 1.20 times (y at T = 1152, d = 7168, f = 18560).

// Microseconds of one tile of a group with all compute units busy, from time stamps (large tile: 1.33 per K step, 1.45 in
// the long tiles of the one-launch sum, which all run at once; 2.5 before the first step; the epilogue: 33 with the SwiGLU
// derivative, 42 when it also casts, 10 for U, G or an fp32 store, 6 for bf16).  Small tile, two on a compute unit:
// 0.96 per K step, 3.5 before and after, a quarter of the large tile's epilogue.
// (The epilogues are priced as they were when the lines between the tiles were set; measured now: 23.5 with the derivative, 5.6 for
// an fp32 store.  The constants of all estimates below belong together with these, and the figures above are of the choice that
// they make with the present kernels.)
static double k_steps(const GemmArgs &a) {
    const int64_t kbytes = a.a_fmt == kBF16 ? 2 * a.K : a.K;
    return (double)((kbytes + BK - 1) / BK) * (a.part == 3 ? 2.0 : 1.0);
}
static double epilogue_cost(const GemmArgs &a) {
    if (a.epilogue == EPI_SWIGLU_BWD) return 33.0;
    if (a.epilogue == EPI_SWIGLU_BWD_Q) return 42.0;
    return is_dual(a) || a.c_f32 ? 10.0 : 6.0;
}
double gemm_tile_cost(const GemmArgs &a, int WB) {
    if (WB == 2) return 3.5 + 0.96 * k_steps(a) + 0.25 * epilogue_cost(a);
    return 2.5 + (a.part == 3 ? 1.45 : 1.33) * k_steps(a) + epilogue_cost(a);
}

static int64_t tile_count(const GemmArgs &a, int WB) {
    const int64_t edge = tile_edge(WB), cols = is_dual(a) ? edge / 2 : edge;
    return ((a.M + edge - 1) / edge) * ((a.N + cols - 1) / cols) * (a.part == 4 ? 2 : 1);
}

// Estimated time of `tiles` small tiles of one GEMM, each of `cost` microseconds when two share a compute unit.
static double small_tile_time(int64_t tiles, double cost) {
    // a tile that has its compute unit to itself is bound by the latency of its loads: taken as 0.44 per K step, 0.58 when
    // all compute units are at it (long K, up to 160 tiles: 0.41 with a ring of five, as in the groups, 0.30 with one of
    // nine; 0.47 and 0.41 up to 256; up to twice that where rows split cache lines).  With 257 to 512 of them the units that hold two decide, and these slow
    // each other down the more of them there are.  Beyond two rounds the tiles drift out of step and the rounds blur
    if (tiles <= kComputeUnits) return 5.5 + (cost - 5.5) * (tiles <= 160 ? 0.46 : 0.6);
    if (tiles <= 2 * kComputeUnits) return cost * (0.65 + 0.35 * (double)(tiles - kComputeUnits) / kComputeUnits);
    const double blurred = std::max(cost, cost * (double)tiles / (2.0 * kComputeUnits));
    return tiles <= 3 * kComputeUnits ? std::max(blurred, 1.65 * cost) : blurred;
}

// Operand bytes that have to come from memory once, and how many of the two operands have rows that do not start on
// 128-byte lines, so that a small tile's 128-byte pieces of them span two lines each.
static double operand_bytes(const GemmArgs &a) {
    return (double)(a.M + (is_dual(a) ? 2 : 1) * a.N) * (double)a.K * (a.a_fmt == kBF16 ? 2.0 : 1.0) * (a.part >= 3 ? 2.0 : 1.0);
}
static int split_line_operands(const GemmArgs &a) {
    return ((a.layout == 2 ? a.M : a.K) % 128 != 0) + ((a.layout >= 1 ? a.N : a.K) % 128 != 0);
}
constexpr double kHbmBytesPerUs = 4.2e6;         // what a launch of these kernels draws from HBM

// Estimated microseconds of `tiles` of the tiles of one GEMM in a launch of its own.
// Large tiles: 1.26 per K step in a round that fills the chip.  A last round that does not draws less power and runs at a
// higher clock: 0.86 per K step with few tiles, 1.06 with half of the chip, and a cheaper epilogue (2064 x 11008 x 11008,
// 1.5 rounds: 207 to 226 us in large tiles, 247 to 292 in small ones).
static double large_launch_time(const GemmArgs &a, int64_t tiles) {
    const int64_t full = tiles / kComputeUnits, rest = tiles - full * kComputeUnits;
    const double ks = k_steps(a), epilogue = 1.4 * epilogue_cost(a), share = (double)rest / kComputeUnits;
    double t = (double)full * (2.5 + 1.26 * ks + epilogue);
    if (rest) t += 2.5 + (0.86 + 0.4 * share) * ks + epilogue * (0.57 + 0.43 * share) * std::min(1.0, (double)a.M / tile_edge(4));
    return 4.0 + std::max(t, operand_bytes(a) / kHbmBytesPerUs * ((double)tiles / (double)tile_count(a, 4)));
}
// Small tiles: a fifth more per K step for each operand that splits lines (256 to 2000 tiles: 0.95, 1.17, 1.33 per step of
// a full chip with none, one, both), and half as much again for its bytes.  Where compute units hold two, a quarter of the
// smaller of the two times does not hide behind the larger.  In the training forward small tiles pay for more atomics on the
// channel maxima of U, G's product and for a range pass over w3 that a last round of large tiles would hide; both were dearer
// when this was set (gate/up at T = 4096, d = 768, f = 2048: 39 us large, 53 small; now 34 and 33), so a few long batches of small width stay in
// large tiles that small ones would take less for (3440, 256, 848: 22.5 and 17.5).
static double small_launch_time(const GemmArgs &a, int64_t tiles) {
    const int split = split_line_operands(a);
    const double cost = 3.0 + 0.96 * k_steps(a) * (1.0 + 0.2 * split) + 0.25 * epilogue_cost(a);
    const double share = (double)tiles / (double)tile_count(a, 2), run = small_tile_time(tiles, cost);
    const double hbm = std::min(1.0, share) * operand_bytes(a) / kHbmBytesPerUs * (1.0 + 0.5 * split);
    const double range = a.tail_src ? 2.0 * (double)(a.tail_rows * a.tail_cols) / kHbmBytesPerUs : 0.0;
    double t = std::max(run, hbm) + (tiles > kComputeUnits ? 0.25 * std::min(run, hbm) : 0.0);
    if (a.epilogue == EPI_SWIGLU && tiles == tile_count(a, 2)) t += 4.5e-3 * (double)a.M + 0.5 * range;
    else if (a.epilogue == EPI_SWIGLU) t += (0.6e-3 + 3e-3 * share) * (double)a.M + 0.25 * range;     // the rest of a split
    return t;
}
static double launch_time(const GemmArgs &a, int WB) {
    return WB == 2 ? small_launch_time(a, tile_count(a, 2)) : large_launch_time(a, tile_count(a, 4));
}

// Estimated time of the GEMMs of `list` in one grid; of the last one, the share `last` of its tiles.
static double grid_time(const GemmArgs *const *list, int n, int WB, double last = 1.0) {
    double sum = 0.0, longest = 0.0;
    int64_t tiles = 0;
    for (int i = 0; i < n; ++i) {
        const int64_t t = (int64_t)((double)tile_count(*list[i], WB) * (i == n - 1 ? last : 1.0));
        const double cost = gemm_tile_cost(*list[i], WB);
        tiles += t;
        sum += cost * (double)t;
        longest = std::max(longest, cost);
    }
    if (WB == 2) return tiles <= kComputeUnits ? small_tile_time(tiles, longest) : std::max(longest, sum / (2.0 * kComputeUnits));
    // one tile per compute unit: the last round of one member is filled by the others
    // where a few long tiles decide (dX of a short batch: 64 tiles of 172 K steps), the members beside them slow them
    // down (T = 1024, d = 4096, f = 11008: 305 us for 258 estimated; the step 605 us, 574 with small tiles)
    return std::max(1.15 * longest, sum / kComputeUnits);
}

// Estimated microseconds of the second backward group, dX in form `part` and two weight gradients, in either tile.  dX's tiles
// are dealt first; where there are few of them they decide, else the work does.  Large tile: a long tile beside many short
// ones that write takes longer.  Small tile: 0.89 per K step where two share a compute unit, 0.57 for one that has it to
// itself, which dX's are once the weight gradients have ended, if they end early; a quarter more for each operand that splits
// lines; gradients leave at 5.9 MB/us at most.  The constants are those with which the choice between the forms and tiles
// comes out best over 1626 measured calls of the backward (see gemm_sum_form), so what counts is how the estimates compare.
static double dx_group_time(GemmArgs dx, const GemmArgs &dw, int part, int WB) {
    dx.part = part;
    const double kx = k_steps(dx), kw = k_steps(dw), nx = (double)tile_count(dx, WB), nw = 2.0 * (double)tile_count(dw, WB);
    if (WB == 4) {
        const double cx = part == 4 ? 25.5 + 1.61 * kx : 2.0 + 1.44 * kx, cw = 9.5 + 1.44 * kw;
        return 4.0 + std::max(1.16 * cx, (nx * cx + nw * cw) / kComputeUnits + 0.65 * cw);
    }
    const double slots = 2.0 * kComputeUnits, split = 1.0 + 0.23 * split_line_operands(dx), shared = 0.89 * split, alone = 0.57 * split;
    const double end_x = part == 4 ? 7.4 : 4.0, cx = end_x + shared * kx, cw = 5.7 + shared * kw;
    const double beside = std::max(nw * cw / slots, 2.0 * (double)(dw.M * dw.N) * (dw.c_f32 ? 4.0 : 2.0) / 5.9e6);
    const double contended = std::min(kx, beside / shared);      // (steps beside another tile)
    return 6.0 + std::max(end_x + shared * contended + alone * (kx - contended), nx * cx / slots + beside + (nx + nw > slots ? 0.7 * cw : 0.0));
}

int gemm_wave_blocks(const GemmArgs *const *list, int n, double last) {
    if (list[0]->part == 4) {
        const GemmArgs &dw = *list[n > 1 ? 1 : 0];       // (alone: the tile does not change its bits; taken as with weight gradients of its own size)
        return dx_group_time(*list[0], dw, 4, 2) < dx_group_time(*list[0], dw, 4, 4) ? 2 : 4;
    }
    for (int i = 0; i < n; ++i) {
        if (list[i]->a_fmt == kBF16 || list[i]->part == 1 || list[i]->part == 2) return 4;      // not built in the small tile
        if (list[i]->part == 3 && !sum_in_large_tile_ok(list[i]->K)) return 2;
    }
    if (n == 1) return launch_time(*list[0], 2) < 0.98 * launch_time(*list[0], 4) ? 2 : 4;
    return grid_time(list, n, 2, last) < grid_time(list, n, 4, last) ? 2 : 4;
}

// Sets of large tiles that make whole rounds of the chip when the rest is worth a launch of small tiles of its own (5 us):
// a last round of large tiles that fills a third of the chip takes longer than its share.  0: the GEMM stays whole.
// (gate/up of the inference form at T = 4096, d = 4096, f = 11008, 5.4 rounds: 299 us whole, 282 as 5 rounds and 384 small
// tiles.  Gate/up of the training forward at d = 3072, f = 8208, W1, W2 cached: T = 2048, 2.03 rounds, 119 us whole, 107 in two;
// T = 2064, 2.3 rounds, 119 and 114; T = 1552, 1.8 rounds, 82 and 96.)
static int full_round_sets(const GemmArgs &a, double whole) {
    if (a.a_fmt == kBF16) return 0;
    const int64_t tiles = tile_count(a, 4), rounds = tiles / kComputeUnits, rest = tiles - rounds * kComputeUnits;
    if (rounds == 0 || rest == 0) return 0;
    const double split = large_launch_time(a, rounds * kComputeUnits) + 5.0 + small_launch_time(a, 4 * rest);
    return split < 0.98 * whole ? (int)(rounds * kComputeUnits / 8) : 0;
}

size_t gemm_arrival_words(int64_t M, int64_t N) {
    return (size_t)(4 * ((M + tile_edge(4) - 1) / tile_edge(4)) * ((N + tile_edge(4) - 1) / tile_edge(4)));
}

// Without halves.  The input gradient of a hidden width that is no multiple of 128: in one launch of small tiles together with
// the weight gradients, or as two launches of large tiles through fp32 scratch and the weight gradients each on its own
// (T = 4096, d = 4096, f = 11024, the whole step: 1945 us against 1776; T = 2048, d = 3072, f = 8208: 704 against 798).
static int sum_form_unsplit(const GemmArgs &dx, const GemmArgs &dw, double *separate_time) {
    *separate_time = 0.0;
    if (sum_in_large_tile_ok(dx.K)) return 3;
    GemmArgs sum = dx, half = dx;
    sum.part = 3; half.part = 1; half.c_f32 = 1;
    const GemmArgs *one[3] = {&sum, &dw, &dw};
    auto rounds = [](const GemmArgs &a) { return gemm_tile_cost(a, 4) * (double)((tile_count(a, 4) + kComputeUnits - 1) / kComputeUnits); };
    const double separate = 2.0 * rounds(half) + 2.0 * std::min(rounds(dw), small_tile_time(tile_count(dw, 2), gemm_tile_cost(dw, 2)));
    *separate_time = separate;
    return grid_time(one, 3, 2) < separate ? 3 : 1;
}

// Each product of dX in tiles of its own, which meet where the second of them is done: for short batches, whose few tiles of
// both products (172 K steps at d = 4096, f = 11008) are still running when the weight gradients have long ended.  Up to 80
// large tiles, twice that as halves; beyond, the tiles of dX fill the chip by themselves and the products' way through memory
// (the one, 256 KB per large tile, out and in) costs (the group at 2048, 3072, 8192, 96 tiles: 210 us whole, 219 in halves;
// 4096, 4096, 11008 559 and 590; only where f is no multiple of 128, and whole means small tiles, there would still be a gain: the
// backward at 4096, 2000, 6000 462 and 371).  Not where a tile of both products takes less than four thirds of a weight
// gradient's K steps (the backward, whole and in halves: 3072, 768, 2048 69.4 and 73.2 us; 2560, 512, 1360 57.4 and 60.2), unless all
// tiles together are few (1280, 256, 688 40.6 and 39.0); elsewhere as estimated, up to 2.5 % above whole tiles (3 % with bf16
// gradients), where the choice came out best over the calls that the estimates are fitted to.
// Measured, the whole backward in each form, 27 pairs of d and f from 256 x 688 to 8192 x 28672, T = 16 to 4096, fp32 and bf16
// gradients: over the 1626 calls with up to 128 tiles the choice takes 0.904 of the time without halves, the best of
// both for every call 0.903.  8 calls take more than 1.5 % longer than without halves, the worst 1.045 times (2048, 2560, 6912,
// fp32 gradients).  T = 1024, d = 4096, f = 11008 (fp32) 411 us whole and 356 in halves, 768 343 and 313, 512 317 and 275; 256,
// 2048, 5504 90 and 73; 656, 3072, 8192 161 and 170, left whole.
int gemm_sum_form(const GemmArgs &dx, const GemmArgs &dw) {
    double separate;
    const int whole = sum_form_unsplit(dx, dw, &separate);
    GemmArgs sum = dx;
    sum.part = 0;
    const bool few = 2 * (tile_count(sum, 2) + tile_count(dw, 2)) <= kComputeUnits / 2;
    if (tile_count(sum, 4) > kHalvesTiles || (few ? 2.0 : 1.5) * k_steps(sum) <= k_steps(dw)) return whole;
    double unsplit = separate;
    if (whole == 3) {
        sum.part = 3;
        const GemmArgs *list[3] = {&sum, &dw, &dw};
        unsplit = dx_group_time(sum, dw, 3, gemm_wave_blocks(list, 3));
    }
    return std::min(dx_group_time(sum, dw, 4, 2), dx_group_time(sum, dw, 4, 4)) < (dw.c_f32 ? 1.025 : 1.03) * unsplit ? 4 : whole;
}

int gemm_profile_tag(const GemmArgs &a) {
    // 2 * epilogue + A format; the halves of a sum of two products run as two launches get 9 and 10, the sum in
    // one launch 11; the gate/up GEMM with the column range pass in its grid 18
    if (a.part) return 8 + (a.part == 4 ? 3 : a.part);
    if (a.tail_src) return 18;
    if (a.a_fmt == kBF16) return a.epilogue == EPI_STORE ? 20 : 21;
    return 2 * (a.epilogue == EPI_SWIGLU_BWD_Q ? (int)EPI_SWIGLU_BWD : a.epilogue) + a.a_fmt;
}

template <int WB, int UNITS, int EPI, int AFMT, int LAY>
static void launch_tiles(const GemmParams &p, bool wide, unsigned blocks, hipStream_t st) {
    if constexpr (UNITS == kLongRing && EPI == EPI_STORE)
        if (wide) {
            hipLaunchKernelGGL((gemm_wide_kernel<AFMT, LAY>), dim3(blocks), dim3(kThreads), 0, st, p);
            return;
        }
    if constexpr (UNITS == kLongRing)
        hipLaunchKernelGGL((gemm_alone_kernel<EPI, AFMT, LAY>), dim3(blocks), dim3(kThreads), (unsigned)smem_bytes(2, kLongRing), st, p);
    else
        hipLaunchKernelGGL((gemm_kernel<WB, EPI, AFMT, 0, LAY>), dim3(blocks), dim3(kThreads), 0, st, p);
}
template <int WB, int UNITS, int LAY>
static void launch_store_tiles(const GemmParams &p, int a_fmt, bool wide, unsigned blocks, hipStream_t st) {
    if (a_fmt == kE4M3) launch_tiles<WB, UNITS, EPI_STORE, kE4M3, LAY>(p, wide, blocks, st);
    else launch_tiles<WB, UNITS, EPI_STORE, kE5M2, LAY>(p, wide, blocks, st);
}

template <int WB, int UNITS>
static void launch_gemm_wb(const GemmArgs &a, int first_set, int sets, hipStream_t st, bool wide = false) {
    GemmParams p = make_gemm_params(a);
    const int tiles = p.tiles_m * p.tiles_n, hi = std::min((first_set + sets) * 8, tiles);
    p.first_set = first_set;
    p.sets = sets;
    const unsigned blocks = (unsigned)sets * set_workgroups(WB);
    const bool tail = a.tail_src && hi == tiles;          // the range pass over w3 rides in the last launch of the GEMM
    profile_before(gemm_profile_tag(a), st, gemm_flops(a) * (double)(hi - first_set * 8) / (double)tiles);
    switch (a.epilogue) {
        case EPI_STORE:
            if (a.a_fmt == kBF16) hipLaunchKernelGGL((gemm_kernel<4, EPI_STORE, kBF16, 0, 0>), dim3(blocks), dim3(kThreads), 0, st, p);
            else if (a.layout == 2) launch_store_tiles<WB, UNITS, 2>(p, a.a_fmt, wide, blocks, st);
            else if (a.layout == 1) launch_store_tiles<WB, UNITS, 1>(p, a.a_fmt, wide, blocks, st);
            else launch_store_tiles<WB, UNITS, 0>(p, a.a_fmt, wide, blocks, st);
            break;
        case EPI_SWIGLU:
            if (tail) {
                ColRangeParams r{static_cast<const uint16_t *>(a.tail_src), a.tail_rows, a.tail_cols, a.tail_camax_bits,
                                 col_range_blocks_x(a.tail_cols)};
                const unsigned extra = (unsigned)(r.blocks_x * col_range_blocks_y(a.tail_rows));
                hipLaunchKernelGGL(gemm_swiglu_col_range_kernel<WB>, dim3(blocks + extra), dim3(kThreads), 0, st, p, r);
            } else {
                launch_tiles<WB, UNITS, EPI_SWIGLU, kE4M3, 0>(p, false, blocks, st);
            }
            break;
        default:   // EPI_SWIGLU_Q
            launch_tiles<WB, UNITS, EPI_SWIGLU_Q, kE4M3, 0>(p, false, blocks, st);
            break;
    }
    profile_after(st);
}

// Gate/up of the inference form: up to 64 rows beyond whole large tiles, which would fill another row of tiles to a quarter at
// most, go to the few-rows form in the grid of the others' small tiles, whose free slots its workgroups fit, where that is
// estimated shorter.  With at most one tile to a compute unit such neighbours only slow the tiles down (T = 144, d = 4096, f = 11008:
// 27.4 us in two rows of small tiles, 33.7 this way); a batch that takes whole rounds of large tiles and a rest keeps them.
// Estimates (microseconds without the launch; K steps of 128): small tiles 7 and 0.62 per step up to 256, 1.2 of two that share a
// compute unit; large ones 15 and 0.76 to 1.16 per step of a round, the fuller the more; a few-rows workgroup (16 rows; 32 where
// there are more) takes 0.2 + 0.07 per step (0.7 + 0.12) of one of 512 slots.  Their constants are those with which the choice comes
// out best over 424 measured calls, so what counts is how they compare.
// Measured, gate/up alone, 23 pairs of d and f from 256 x 1024 to 8192 x 28672, T = 256 to 2048 and 16, 32, 48 or 64 more: 0.982 of
// the time without over all, 0.962 were each call's better one known, and 4 calls more than 1.5 % slower, the worst by 0.4 us (784,
// 400, 4096 15.2 and 15.7).  16, 32, 48 and 64 rows more, in tiles and this way: T = 256, d = 4096, f = 11008 45 and 36, 45 and 39, 44 and
// 44, 44 and 45; 512, 4096, 11008 65 and 59, 66 and 59, 68 and 63, 68 and 64 (the last two stay in tiles); 1024, 1024, 4096 21 and 18, 20,
// 21, 20; 512, 2048, 5504 27 and 21, 27 and 21, 28 and 23 (these last stay).  Where they stay because it is longer: 256 and 16, 8192, 28672
// 184 and 225; 768 and 32, 2048, 5504 30 and 33; 256 and 64, 4096, 14336 50 and 56.
static int few_last_rows(const GemmArgs &a) {
    constexpr int kMost = 64;
    const int rest = (int)(a.M % tile_edge(4));
    if (a.epilogue != EPI_SWIGLU_Q || rest == 0 || rest > kMost || a.M < tile_edge(4)) return 0;
    GemmArgs main = a;
    main.M -= rest;
    const int64_t tiles = tile_count(main, 2);
    if (tiles <= kComputeUnits || tiles > 4 * kComputeUnits) return 0;
    const double ks = k_steps(a), slots = 2.0 * kComputeUnits, split = a.K % 128 != 0 ? 1.8 : 1.0;
    auto small = [&](int64_t n) {
        const double two = 1.2, one = 0.62, over = (double)(n - kComputeUnits) / kComputeUnits;
        const double step = n <= kComputeUnits ? one : n <= 2 * kComputeUnits ? one + (two - one) * over : std::max(two * (double)n / slots, 1.3 * two);
        return 7.0 + step * split * ks;
    };
    auto large = [&](int64_t n) {
        const int64_t full = n / kComputeUnits, last = n - full * kComputeUnits;
        return 15.0 + 0.76 * ks * (1.52 * (double)full + (last ? 1.0 + 0.52 * (double)last / kComputeUnits : 0.0));
    };
    const int block = few_last_block(rest);
    const double groups = (double)((rest + block - 1) / block) * (double)((a.N + 15) / 16);
    const double few = (block == 16 ? 0.2 + 0.07 * ks : 0.7 + 0.12 * ks) * split;
    const double with = std::max(small(tiles), 7.0 + (1.2 * split * ks * (double)tiles + few * groups) / slots);
    const GemmArgs *one = &a;
    const double without = gemm_wave_blocks(&one, 1) == 2 ? small(tile_count(a, 2)) : large(tile_count(a, 4));
    return with < 0.98 * without ? rest : 0;
}

GemmPlan gemm_plan(const GemmArgs &a) {
    const GemmArgs *one = &a;
    GemmPlan p;
    p.wave_blocks = gemm_wave_blocks(&one, 1);
    const double whole = launch_time(a, p.wave_blocks);
    if (gemm_skinny_time(a, &p.form) < whole) { p.wave_blocks = 0; return p; }
    p.whole_sets = full_round_sets(a, whole);
    if (p.whole_sets == 0) p.rest_rows = few_last_rows(a);
    if (p.rest_rows > 0) { p.wave_blocks = 2; return p; }
    if (p.whole_sets > 0) p.wave_blocks = 2;
    // one small tile to a compute unit, so up to 8 large tiles on an XCD of 32: the longer ring, which leaves no room
    // for a second workgroup (M = 528, N = 2048, K = 4096, 80 tiles: 27 us with five units, 21 with nine; 65 large tiles
    // give one XCD a second round: 28 and 34)
    const int64_t rest = tile_count(a, 4) - 8 * p.whole_sets;
    if (p.wave_blocks == 2 && rest <= kComputeUnits / 4) p.units = kLongRing;
    // The wide products but where power bounds these launches too: most of the chip at it, whole cache lines and enough K steps.
    // Short and wide, of the time on wide products alone (before the short form): 256 tiles, K = 4096, .97 and 1.00 (both K-major), .95 and
    // .98; 192 tiles .98 and .99, 1.02 and 1.01; K = 11008 .97 and 1.00, .99 and 1.00; 160 tiles, K = 4096, 1.00 and 1.00.  Lines split:
    // 198 tiles, K = 1040, 4112 and 11024 1.025, 1.009 and 1.001, wide 1.002, 1.001 and .997; 7 tiles, K-major, 1.06 to 1.10
    // and 1.02.  K = 1024: short .5 to 2 % longer than wide up to 256 tiles.
    const int64_t small = p.whole_sets > 0 ? 4 * rest : tile_count(a, 2);
    p.wide = a.epilogue == EPI_STORE && a.a_fmt != kBF16 && p.units == kLongRing &&
             !(small > kComputeUnits * 5 / 8 && split_line_operands(a) == 0 && a.K >= 16 * BK);
    return p;
}

bool launch_gemm(const GemmArgs &a, hipStream_t st) {
    if (!gemm_args_ok(a)) return false;
    if (a.part != 0 || a.epilogue == EPI_SWIGLU_BWD || a.epilogue == EPI_SWIGLU_BWD_Q) return launch_gemm_bwd(a, st);
    const GemmPlan plan = gemm_plan(a);
    if (plan.wave_blocks == 0) {
        profile_before(gemm_profile_tag(a), st, gemm_flops(a));
        launch_gemm_skinny(a, plan.form, st);
        profile_after(st);
        return true;
    }
    if (plan.rest_rows > 0) {
        profile_before(gemm_profile_tag(a), st, gemm_flops(a));
        launch_gemm_rest(a, plan.rest_rows, st);
        profile_after(st);
        return true;
    }
    const int full = plan.whole_sets, rest = sets_of(make_gemm_params(a)) - full;
    if (full > 0) launch_gemm_wb<4, 5>(a, 0, full, st);
    if (plan.wave_blocks == 4) launch_gemm_wb<4, 5>(a, 0, rest, st);
    else if (plan.units == kLongRing) launch_gemm_wb<2, kLongRing>(a, full, rest, st, plan.wide);
    else launch_gemm_wb<2, 5>(a, full, rest, st);
    return true;
}

}  // namespace ssg
