// Internal launch interface between the C-ABI layer and the kernels.
// Everything takes raw device pointers and a hipStream_t; nothing allocates.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

namespace ssg {

enum SrcKind { SRC_BF16 = 0, SRC_F32 = 1, SRC_SWIGLU = 2 };

// ---- elementwise / reduction passes (ssg_quant.hip) -------------------------
void launch_fill_u32(uint32_t *p, size_t n, uint32_t value, hipStream_t st);
// The range of a tensor of n > 0 elements and the scale it gives (scale_out may be null).  scratch: n bytes at least, at
// most 4 KB of them are written.
void launch_range_scale(const void *src, SrcKind kind, size_t n, uint32_t *scratch, int fmt, int pow2, float *amax_out,
                        float *scale_out, hipStream_t st);
// up to two runs of words that a kernel zeroes on the side for the kernels after it
struct ZeroWords {
    uint32_t *p[2] = {nullptr, nullptr};
    unsigned n[2] = {0, 0};
};

// Running maxima of |x| as float bits, spread over `slots` words that are kAmaxSlotStride words
// (one cache line) apart and must be zeroed by the caller: workgroup b folds into slot b % slots.
// Same-address atomics serialise in L2 (~12 ns each), so a pass that wants thousands of workgroups
// for bandwidth uses kAmaxSlots slots and the consumer takes the maximum over them; slots = 1 is
// the plain single-word form of the public entry points.
constexpr int kAmaxSlots = 64;
constexpr int kAmaxSlotStride = 32;
constexpr size_t kAmaxSlotWords = (size_t)kAmaxSlots * kAmaxSlotStride;
void launch_amax(const void *src, SrcKind kind, size_t n, uint32_t *amax_bits, int slots, hipStream_t st);
struct CastArgs {
    const void *src = nullptr;       // bf16 / f32 [rows, cols]; U for SRC_SWIGLU
    const void *src2 = nullptr;      // G for SRC_SWIGLU
    SrcKind kind = SRC_BF16;
    int64_t rows = 0, cols = 0;
    int fmt = 0;                     // kE4M3 / kE5M2
    const float *col_scale = nullptr;   // optional per-column factor applied first (one fp32 multiply)
    const float *amax = nullptr;     // per-tensor: scale = scale_from_amax(max over amax_slots slots) ...
    int amax_slots = 1;
    int range_count = 0;             // > 0: `amax` is this many packed words instead of slots
    uint32_t *range_words = nullptr; // launch_quantize_batch: kAmaxSlotWords words of scratch for the range of src
    float *amax_out = nullptr;       // where the reduced amax is recorded (may be null)
    const float *scale_in = nullptr; // ... or a given scale; both null = no per-tensor factor
    int pow2 = 0;
    float *scale_out = nullptr;      // where the per-tensor scale is recorded (may be null)
    uint32_t *record = nullptr;      // optional kAmaxSlots slotted words: max |src| seen by this pass is folded in
                                     // (bf16 source, no per-column factor, transposed copy requested)
    uint8_t *dst = nullptr;          // [rows, cols]
    uint8_t *dst_t = nullptr;        // [cols, rows] or null
    unsigned long long *counters = nullptr;   // optional (no transposed copy): [0] += elements beyond the format's
                                     // range under the scale (saturated), [1] += nonzero elements cast to +-0
};
void launch_cast(const CastArgs &a, hipStream_t st);
// up to three casts of the same form (source kind, format, optional parts) in one launch; others are launched singly
void launch_cast_batch(const CastArgs *list, int n, const ZeroWords &zero, hipStream_t st);
// Q of up to three bf16 tensors from their own ranges (rows, cols, fmt, pow2, src, dst, amax_out, scale_out, range_words
// given; one format), in one launch for small tensors, else a range and a cast launch.  Returns how many packed words of
// each range_words hold its range afterwards.
int launch_quantize_batch(CastArgs *list, int n, const ZeroWords &zero, hipStream_t st);
// Q of one tensor, any source kind but the SwiGLU product, from its own range in one launch.  polls: how often a workgroup looks
// for the others' ranges before it forms them itself, < 0: the usual number.  false: nothing launched, the tensor is too large
// or the stream is being captured.
bool launch_quantize_once(const CastArgs &a, int polls, hipStream_t st);
// camax_bits[c] = max_r |v[r,c]| as float bits (zeroed by the caller).
void launch_col_amax(const void *src, const void *src2, SrcKind kind, int64_t rows, int64_t cols,
                     uint32_t *camax_bits, hipStream_t st);

// The ranges of a call, to be entered into the history of delayed scaling
struct ScalingUpdate {
    uint32_t *slots[3] = {nullptr, nullptr, nullptr};   // slotted range words of the call just made (cleared afterwards),
    int range_count[3] = {0, 0, 0};                     // or this many packed words
    int tensor[3] = {0, 0, 0};
    int fmt[3] = {0, 0, 0};
    int count = 0;
    int pow2 = 0;
    uint32_t *state = nullptr;
};

// Per-channel factors from the per-channel maxima (Section 4.4) and the range
// of s^-1 * w3 for the folded weight.  smooth = 0: one factor for all channels.
struct ChannelFactors {
    const float *h_camax = nullptr, *w3_camax = nullptr;
    int64_t f = 0;
    int smooth = 1;
    float *s = nullptr, *sinv = nullptr;
    uint32_t *amax_w3s_bits = nullptr;      // zeroed by the caller
    uint32_t *hmax_bits = nullptr;          // plain mode: scratch, zeroed by the caller; receives the tensor's range
    const float *h_scale_given = nullptr;   // plain mode only, optional device scalar: the scale of h as the caller gives it
    ScalingUpdate update;                   // optional (count > 0): entered into the history by the same launch
};
void launch_channel_factors(const ChannelFactors &c, hipStream_t st);
// the factors, then the smooth cast of h (from bf16 U, G) and the fold + cast of w3 in one launch (two for any other pair);
// in one launch altogether for few channels
void launch_cast_h_w3(const CastArgs &h, const CastArgs &w3, const ChannelFactors &fac, hipStream_t st);

// amax_bits = max_i fl32(w3_camax[i] * sinv[i]) as float bits (zeroed by the caller).
void launch_fold_range(const float *w3_camax, const float *sinv, int64_t f, uint32_t *amax_bits, hipStream_t st);

void launch_swiglu(const void *U, const void *G, int64_t n, float *h, hipStream_t st);

// bf16 [rows, cols] -> transposed copy [cols, rows]; and the SwiGLU product of bf16 U, G [rows, cols] rounded once to
// bf16, as it stands (h) and transposed (h_t) -- the operands of the last linear layer when it is left in bf16
void launch_transpose_bf16(const void *src, int64_t rows, int64_t cols, void *dst_t, hipStream_t st);
void launch_swiglu_bf16(const void *U, const void *G, int64_t rows, int64_t cols, void *h, void *h_t, hipStream_t st);

// Q_E4M3 of a bf16 [rows, cols] matrix whose row i is first multiplied by row_scale[i]; `slots` are
// kAmaxSlots zeroed slotted range words (scratch)
void launch_rowscale_quantize(const void *w, const float *row_scale, int64_t rows, int64_t cols, uint32_t *slots,
                              int pow2, float *scale_out, float *amax_out, uint8_t *dst, hipStream_t st);

// ---- FP8 MFMA GEMM (ssg_gemm.hip) --------------------------------------------
enum Epilogue {
    EPI_STORE = 0,        // C = acc * alpha [* col_scale[n]]
    EPI_SWIGLU = 1,       // dual B: U, G bf16 stores + per-channel max of |h|
    EPI_SWIGLU_BWD = 2,   // acc -> dH; loads U, G; stores dU, dG bf16 + their amax
    EPI_SWIGLU_Q = 3,     // dual B as EPI_SWIGLU, but stores only the E4M3 cast of u * Swish(g) (C: bytes [M, N])
    EPI_SWIGLU_BWD_Q = 4  // as EPI_SWIGLU_BWD, but dU, dG leave as E5M2 codes under given scales (C, C2: bytes [M, N]):
                          // code = satcast(fl32(bf16(dU) * q_scale)); the scales are copied to q_scale_out / q_scale_out2
};

struct GemmArgs {
    int epilogue = EPI_STORE;
    int a_fmt = 0;                      // kE4M3 / kE5M2 (B is always E4M3); kBF16 = 2: A and B are bf16 (layout 0,
                                        // EPI_STORE or EPI_SWIGLU_BWD only; K counts elements)
    int64_t M = 0, N = 0, K = 0;
    const uint8_t *A = nullptr;         // [M, K]   (layout 2: stored K-major, [K, M])
    const uint8_t *B = nullptr;         // [N, K]   (layout 1, 2: stored K-major, [K, N])
    int layout = 0;                     // 0 = both K-contiguous; 1 = B K-major; 2 = A and B K-major (EPI_STORE, EPI_SWIGLU_BWD)
    const uint8_t *B2 = nullptr;        // EPI_SWIGLU, EPI_SWIGLU_Q: the second weight matrix [N, K]
    // EPI_STORE as one half of a sum of two products run as two launches:
    //   part = 1: C is the fp32 scratch [M, N] that receives this product, scaled (c_f32 = 1)
    //   part = 2: `add` (that scratch) is added to this product, scaled, before rounding into C
    //   part = 3: the whole sum in one launch: C = A B^T / (sa sb) + A_ph2 B_ph2^T / (sa_ph2 sb_ph2), the second pair of
    //             operands of the same shapes, formats and layout; all four scale pointers are required
    //   part = 4: as 3, but each product in tiles of its own, twice as many of half the length; `partials` (twice
    //             gemm_partial_floats) and `arrivals` (a word per tile, zeroed by the caller, gemm_arrival_words of them) are scratch
    // (parts are built for the input gradient: A E5M2, layout 1)
    int part = 0;
    const float *add = nullptr;
    const uint8_t *A_ph2 = nullptr, *B_ph2 = nullptr;
    const float *sa_ph2 = nullptr, *sb_ph2 = nullptr;
    float *partials = nullptr;
    uint32_t *arrivals = nullptr;
    // dequantization: alpha = 1 / (sa * sb); null pointer = 1
    const float *sa = nullptr, *sb = nullptr, *sb2 = nullptr;   // sb2: scale of B2
    const float *col_scale = nullptr;   // optional [N] factor (EPI_STORE, EPI_SWIGLU_BWD)
    void *C = nullptr;                  // EPI_STORE: [M,N];  EPI_SWIGLU: U;  EPI_SWIGLU_BWD: dU
    void *C2 = nullptr;                 // EPI_SWIGLU: G;  EPI_SWIGLU_BWD: dG
    int c_f32 = 0;                      // EPI_STORE: 1 = fp32 output, 0 = bf16
    const void *U = nullptr, *G = nullptr;      // EPI_SWIGLU_BWD inputs (bf16 [M,N])
    uint32_t *camax_bits = nullptr;     // EPI_SWIGLU: [N] running max |h| (float bits)
    uint32_t *amax_bits = nullptr;      // EPI_SWIGLU_BWD: running max |dU| (float bits), kAmaxSlots slots
    uint32_t *amax_bits2 = nullptr;     //                 same for |dG|
    const float *q_scale = nullptr, *q_scale2 = nullptr;          // EPI_SWIGLU_BWD_Q: scales of dU, dG (device)
    float *q_scale_out = nullptr, *q_scale_out2 = nullptr;        //                   where the scales used are recorded
    void *keep_u = nullptr, *keep_g = nullptr;                    //                   optional bf16 [M,N]: the rounded dU, dG
                                                                  //                   the codes were cast from (both or neither)
    // EPI_SWIGLU, optional: an independent per-column range pass over a bf16 matrix [tail_rows, tail_cols] (columns a
    // multiple of 8) run by extra workgroups at the end of the grid, where they fill the compute units that the last,
    // partly occupied round of tiles leaves idle; tail_camax_bits [tail_cols] (float bits, zeroed by the caller)
    const void *tail_src = nullptr;
    int64_t tail_rows = 0, tail_cols = 0;
    uint32_t *tail_camax_bits = nullptr;
};
// Whether the argument set is one the kernels are built for (part / add / epilogue / layout combinations).
bool gemm_args_ok(const GemmArgs &a);
// false (nothing launched): gemm_args_ok(a) is false
bool launch_gemm(const GemmArgs &a, hipStream_t st);
// How launch_gemm runs a GEMM other than the backward forms; shapes, formats and options decide, no pointer but
// tail_src and col_scale (null or not) is looked at
struct GemmPlan {
    int wave_blocks = 4;        // 4: tiles of 256 x 256, 2: tiles of 128 x 128, 0: few rows
    int units = 5;              // operand tiles of the ring
    bool wide = false;          // the long ring: the products on the wide MFMA (see gemm_tile)
    int whole_sets = 0;         // > 0: so many sets of 8 large tiles in a launch before that of the small ones
    int form = 0;               // few rows: which of its forms
    int rest_rows = 0;          // > 0: the batch's last rows, in the few-rows form in the grid of the small tiles
};
GemmPlan gemm_plan(const GemmArgs &a);
// few rows (ssg_gemm_skinny.hip): estimated microseconds of the best form, 1e30 for an argument set it is not built for
double gemm_skinny_time(const GemmArgs &a, int *form);
void launch_gemm_skinny(const GemmArgs &a, int form, hipStream_t st);
// gate/up of the inference form, the last `rows` rows of the batch in the few-rows form, `few_last_block` to a workgroup
inline int few_last_block(int rows) { return rows <= 16 ? 16 : 32; }
void launch_gemm_rest(const GemmArgs &a, int rows, hipStream_t st);
// rows and columns of the result per workgroup, steps of 128 bytes of K in a wave's ring
void gemm_skinny_extent(const GemmArgs &a, int form, int *rows, int *cols, int *steps);
bool launch_gemm_bwd(const GemmArgs &a, hipStream_t st);       // the backward forms (called by launch_gemm)
constexpr int kComputeUnits = 256;      // of an MI355X; the estimates of a launch's time are in its rounds
// Tile of a launch that runs these GEMMs in one grid: 4 (256 x 256) or 2 (128 x 128), half the 16 x 16 blocks per wave and direction
// (of the last one: the share `last` of its tiles)
int gemm_wave_blocks(const GemmArgs *const *list, int n, double last = 1.0);
double gemm_tile_cost(const GemmArgs &a, int WB);               // estimated microseconds of one tile
// how the input gradient is best run: as part = 3 or 4 (in one grid with weight gradients like `dw`), or as parts 1 and 2 (1)
int gemm_sum_form(const GemmArgs &dx, const GemmArgs &dw);
// part = 4: so many tiles of 256 x 256 at most (see gemm_sum_form); a word for every 128 x 128 tile, and 64 KB
constexpr int kHalvesTiles = 80;
size_t gemm_arrival_words(int64_t M, int64_t N);
inline size_t gemm_partial_floats(int64_t M, int64_t N) { return gemm_arrival_words(M, N) * (128 * 128); }
// The scratch of every part = 4 of N columns and at most M rows, floats of `partials` and words of `arrivals`: what a buffer
// holds that is sized before the form is chosen.  Neither falls as M grows.
inline size_t gemm_halves_floats(int64_t M, int64_t N) {
    const int64_t cols = (N + 255) / 256, rows = std::min((M + 255) / 256, kHalvesTiles / cols);
    return rows > 0 ? 2 * gemm_partial_floats(256 * rows, N) : 0;
}
constexpr size_t kHalvesWords = 4 * kHalvesTiles;
int gemm_profile_tag(const GemmArgs &a);
// Several independent GEMMs in one grid, the workgroups of one following those of the other.  Built groups:
//   { dH (EPI_SWIGLU_BWD or _Q), weight gradient (EPI_STORE, layout 2, A E5M2) }
//   { input gradient as one launch (part = 3 or 4), one to three weight gradients }
// gemm_group_ok tells whether `list` is one of them with every member valid; launch_gemm_group returns false
// (nothing launched) otherwise.  Timing tags: 16 and 17.  `update` (second group only; count > 0): workgroups at the end
// of the grid enter these ranges into the history of delayed scaling.
// split_sets >= 0 splits the LAST member (workgroups come in sets of 8 tiles, gemm_tile_sets of them per GEMM): the
// two-member group runs its sets [0, split_sets), the other group the rest, so that one weight gradient can be
// shared out between the two launches; split_sets < 0: every member whole.
// gemm_group_split_sets picks that split for {dh, dw_split} followed by {second..., rest of dw_split} on `units`
// compute units, from a replay of the in-order dispatch with per-tile times estimated from K steps and epilogues.
bool gemm_group_ok(const GemmArgs *const *list, int n);
bool launch_gemm_group(const GemmArgs *const *list, int n, int split_sets, hipStream_t st, const ScalingUpdate &update = {});
int gemm_group_wave_blocks(const GemmArgs *const *list, int n, int split_sets);      // the tile it runs in
int gemm_tile_sets(const GemmArgs &a);
int gemm_group_split_sets(const GemmArgs &dh, const GemmArgs &dw_split, const GemmArgs *const *second, int n_second, int units);

// Benchmark hook: called by the launchers before and after a kernel launch (no-ops unless enabled).  `bytes`: the
// algorithmic bytes the launch moves (elementwise passes) or its algorithmic flops (GEMMs).
void profile_before(int tag, hipStream_t st, double bytes = 0.0);
void profile_after(hipStream_t st);
// tags of the elementwise passes (the GEMM tags are listed with ssg_profile_read)
constexpr int kTagAmax = 40, kTagCast = 41, kTagCastSwiglu = 42, kTagCastColscale = 43, kTagColAmax = 44, kTagSmall = 45,
              kTagTranspose = 46, kTagCastHW3 = 47;

// ---- delayed scaling: amax history per tensor (ssg_quant.hip) ----------------------
// State words: tensor k (0..5 = x, w1, w2, dy, du, dg) owns words [32k, 32k+32): [0] the scale the next
// call uses (float), [1] position in the history ring, [2] the range seen in the last call (float),
// [8, 8+kScalingHistory) the ring of ranges.  From word kScalingHeaderWords on: four slotted range
// accumulators (x, w1, w2, dy) of kAmaxSlotWords words each, zero between calls.
constexpr int kScalingTensors = 6, kScalingHistory = 16, kScalingStride = 32;
constexpr size_t kScalingHeaderWords = 256;
constexpr size_t kScalingWords = kScalingHeaderWords + 4 * kAmaxSlotWords;
void launch_scaling_init(uint32_t *state, hipStream_t st);
void launch_scaling_update(const ScalingUpdate &u, hipStream_t st);

// ---- Adam with FP8 moments (ssg_adam.hip) ---------------------------------------
struct AdamArgs {
    const void *grad = nullptr;      // [n] fp32 or bf16
    int grad_bf16 = 0;
    float *w = nullptr;              // [n] fp32 master weights, updated in place
    void *w_bf16 = nullptr;          // optional [n] bf16 copy of the new weights
    uint8_t *m_q = nullptr, *v_q = nullptr;   // [n] E4M3 / E5M2 codes, updated in place
    uint32_t *scalars = nullptr;     // adam_scalar_words() words
    int64_t n = 0;
    int step = 1;                    // the step being taken (>= 1)
    float beta1 = 0, beta2 = 0, one_minus_beta1 = 0, one_minus_beta2 = 0, c1 = 1, c2 = 1;
    float lr = 0, eps = 0, weight_decay = 0;
    int pow2 = 0;
    int polls = -1;                  // looks at the others' ranges where the step is one launch, < 0: the usual number, the most
};
size_t adam_scalar_words();
void launch_adam_init(uint32_t *scalars, uint8_t *codes, size_t code_bytes, hipStream_t st);
void launch_adam_step(const AdamArgs &a, hipStream_t st);

}  // namespace ssg
