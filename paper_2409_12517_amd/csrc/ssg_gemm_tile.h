// FP8 MFMA GEMM for gfx950 with the block's fused epilogues: the code of one output tile (device side).
// Included by the translation units that instantiate the kernels (ssg_gemm.hip, ssg_gemm_bwd.hip).
//
//   C[m,n] = sum_k A[m,k] * B[n,k]      A [M,K], B [N,K] FP8 codes, K contiguous
//
// (the inner products of Eq. 2, the last linear layer of the display after it,
// and their gradient contractions).  fp32 accumulation on the matrix cores with
// v_mfma_f32_16x16x128_f8f6f4; its per-operand format selectors take E4M3 or E5M2.
// The chip runs these kernels at its power limit, and of the two forms with the full
// rate this one draws less per product: a loop of nothing but MFMAs on FP8 codes of
// Gaussian numbers sustains 4500 TFLOP/s with it and 4120 with v_mfma_f32_32x32x64_f8f6f4
// (4960 both on one repeated code), y at T = 4096, d = 4096, f = 11008 takes 122 us (126),
// gate/up of the inference form and y together 424 (438).
//
// The small tile with its compute unit to itself is bound by latencies and takes the other form for plain stores (WIDE, in gemm_tile).
//
// Workgroup: 256 threads = 4 waves as 2 (M) x 2 (N).  Two tile sizes, by the template parameter WB:
//   WB = 4  256 x 256 x 128, each wave owns 128 x 128 outputs = 8 x 8 MFMA blocks (256 accumulator registers, one wave
//           per SIMD).  Bound by the power that the matrix cores and the way of the operands into LDS draw: 81 % of the cycles of
//           that y are MFMA, at 1.8 GHz; without the loads into LDS it would take 106 us of 122, without the fragment reads 118.
//   WB = 2  128 x 128 x 128, 64 x 64 outputs per wave (64 accumulator registers), two workgroups per compute unit.
//           Bound by the loads into LDS, twice the bytes per product: 60 % of the cycles are MFMA, at 1.6 GHz (4096 x 2048 x 4096
//           32 us, 24 without loads), but one workgroup's prologue and epilogue run under the other's main
//           loop, and four times the tiles fill the chip where the large ones leave most of it idle.
// Operand tiles are streamed global -> LDS with 16-byte direct-to-LDS loads (no staging registers) into a ring of five
// 32 KB (16 KB) tiles, or nine of 16 KB where a small tile has its compute unit to itself.  A row of a tile is 128 bytes; the eight 16-byte chunks of a row are stored XOR-permuted by the
// row index so that the lanes that read the same logical chunk of different rows spread over all banks.
//
// Epilogues:
//   STORE       C = acc / (sa*sb) [* col_scale[n]] [+ addend], bf16 or fp32.  A sum of two
//               products (the input gradient) runs in one tile (PART = 3), as two launches: the
//               first leaves its scaled product as fp32 scratch, the second adds it before
//               rounding (PART = 1, 2), or with each product in tiles of its own: of two that
//               belong together the one that ends later adds (PART = 4).
//   SWIGLU      B tile = 128 (64) rows of W1 and the same rows of W2, so a wave
//               holds u and g of the same (t,i): stores bf16 U, G and folds
//               max_t |u * Swish(g)| into the per-channel maxima (Section 4.4).
//   SWIGLU_BWD  acc -> dH (times the channel factor s_i), reads bf16 U, G, stores
//               bf16 dU, dG and folds their amax.
//   SWIGLU_Q    as SWIGLU, but stores only the E4M3 cast of u * Swish(g) (inference form).
//   SWIGLU_BWD_Q as SWIGLU_BWD, but dU, dG leave as E5M2 codes under given scales (delayed scaling).
#pragma once
#include <type_traits>

#include "ssg_device.h"
#include "ssg_internal.h"

namespace ssg {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void *lds_void_ptr;
typedef __attribute__((address_space(1))) const void *global_void_ptr;

// The tile is square, 64 * WB rows and columns, 2 * WB blocks of 16 x 16 per wave and direction (WB = 4 or 2).
constexpr int BK = 128;
constexpr int tile_edge(int WB) { return 64 * WB; }
constexpr int unit_bytes(int WB) { return tile_edge(WB) * BK; }   // one operand tile of one K step: 32 or 16 KB
// UNITS: ring of operand tiles in LDS, an odd number.  Five large units are all 160 KB, five small ones half of them;
// nine small ones (144 KB) where a small tile has its compute unit to itself
constexpr int smem_bytes(int WB, int UNITS = 5) { return UNITS * unit_bytes(WB); }

static __device__ uint4 g_zero_chunk = {0u, 0u, 0u, 0u}; // source of the zero fill of a ragged K tail (one per translation unit)

struct GemmParams {
    const uint8_t *A, *B, *B2;
    int64_t M, N, K;
    const float *sa, *sb, *sb2, *col_scale;
    void *C, *C2;
    const uint16_t *U, *G;
    uint32_t *camax_bits, *amax_bits, *amax_bits2;
    int c_f32;
    int tiles_m, tiles_n;       // in tiles of 256 x 256, also where the small tiles compute
    int first_set, sets;        // single launches: the sets of 8 large tiles this launch computes
    float *tmp;          // fp32 [M, N] scratch for the two-launch form of a sum of two products (may be null)
    const float *add;    // gemm_kernel<.., ADD>: fp32 [M, N] added before the store
    const float *q_scale, *q_scale2;        // EPI_SWIGLU_BWD_Q: scales of dU, dG
    float *q_scale_out, *q_scale_out2;      //                   where the scales used are recorded
    uint16_t *keep_u, *keep_g;              //                   optional: the bf16 dU, dG the codes were cast from
    // PART = 3 (a sum of two products in one tile): operands and scales of the second product, same shapes
    const uint8_t *A_ph2, *B_ph2;
    const float *sa_ph2, *sb_ph2;
    // PART = 4 (one product of such a sum): where this product leaves its scaled result if it is done first, where the other
    // one did (fp32, a tile after the other), and a word per tile, zero at the start, that counts those done
    float *mine;
    const float *other;
    uint32_t *arrivals;
    int nt_store;        // EPI_STORE, fp32 output: 1 = non-temporal stores (the output is not read again soon)
};

// An LDS row holds the 128 bytes (eight 16-byte chunks, one full cache line) of one matrix row for one
// K step; two rows fill the 256-byte bank period, so the chunks of row r are XOR-ed with a permutation of r >> 1.  A fragment
// read takes 16 rows by four chunks c, c + 2, c + 4, c + 6, 16 lanes to a quarter, and goes through the banks 16 lanes at a time:
// lanes 0-3, 12-15 and 20-27, then 4-11, 16-19 and 28-31, and the same of the upper half.  Rows 0-3 and 12-15 of one chunk meet
// rows 4-11 of the next there, so 2 XOR (r >> 1) has to map each half of the rows onto itself: the two low bits of r >> 1
// are exchanged.  (With r >> 1 as it stands half of the LDS cycles were conflicts: y at 4096 x 4096 x 11008 124 us, 49 % of them.)
// WIDE: a read takes 32 rows by two chunks c, c + 2, for which r >> 1 as it stands is right.
template <bool WIDE = false> __device__ __forceinline__ int swz(int row) { return WIDE ? row >> 1 & 7 : (row >> 1 & 4) | (row & 2) | (row >> 2 & 1); }

// Direct-to-LDS loads are issued through inline assembly: the compiler would otherwise wait for
// ALL outstanding LDS-DMA loads before every ds_read (it cannot tell the two LDS stages apart),
// which serialises memory latency with the MFMA work.  M0 carries the wave-uniform LDS
// destination; lane i lands at M0 + 16*i.  The vmcnt waits are placed by hand in the main loop.
__device__ __forceinline__ void dma16(const uint8_t *g, uint32_t lds_addr) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                 :: "s"(lds_addr), "v"(g) : "memory", "m0");
#else
    (void)g; (void)lds_addr;
#endif
}

// Same with a wave-uniform 64-bit base in SGPRs and a 32-bit per-lane byte offset: no VALU work per issue.
__device__ __forceinline__ void dma16_s(const uint8_t *base_uniform, uint32_t lane_off, uint32_t lds_addr) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_addr), "v"(lane_off), "s"(base_uniform) : "memory", "m0");
#else
    (void)base_uniform; (void)lane_off; (void)lds_addr;
#endif
}

// AFMT = kE4M3 / kE5M2: the 32 bytes of a fragment are 32 FP8 codes of one row, one MFMA with K = 128 per fragment
// pair.  AFMT = kBF16 (both operands bf16, the comparison variant with the last linear layer left unquantized):
// the same 32 bytes are 16 bf16 of one row -- two 16-byte pieces of 8 elements each -- and a fragment pair feeds two
// MFMAs with K = 32 (v_mfma_f32_16x16x32_bf16), the first on the low pieces of both operands, the second on the
// high ones.  Which elements of K meet in which MFMA does not matter as long as A and B agree, and they do: both
// fragments come from the same LDS layout through the same lane arithmetic.  Per 128 bytes of K this is twice the
// MFMA instructions at half the duration each, and K in bytes is twice the element count.
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
// The weight's fragment goes first: of a 16 x 16 block a lane then holds row l & 15 and, in its four registers, the neighbouring
// columns 4 (l >> 4) .. + 3, which leave in one 16-byte (fp32) or 8-byte (bf16) access to LDS.  (With the operands the other
// way round a lane holds one column, and every register is an access of its own.)
template <int AFMT>
__device__ __forceinline__ v4f mfma(const v8i &a, const v8i &b, const v4f &c) {
    if constexpr (AFMT == kBF16) {
        const v4i a_lo = {a[0], a[1], a[2], a[3]}, a_hi = {a[4], a[5], a[6], a[7]};
        const v4i b_lo = {b[0], b[1], b[2], b[3]}, b_hi = {b[4], b[5], b[6], b[7]};
        const v4f t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, b_lo), __builtin_bit_cast(v8bf, a_lo), c, 0, 0, 0);
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, b_hi), __builtin_bit_cast(v8bf, a_hi), t, 0, 0, 0);
    } else {
        return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b, a, c, kE4M3, AFMT, 0, 0, 0, 0);
    }
}
template <int AFMT>
__device__ __forceinline__ v16f mfma_wide(const v8i &a, const v8i &b, const v16f &c) {
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(b, a, c, kE4M3, AFMT, 0, 0, 0, 0);
}

// The dequantization factor 1 / (sa * sb).  The product of two binary32 scales can leave the binary32 range
// (the scale of a gradient tensor with a tiny range reaches 1e38) and its reciprocal can fall among the
// subnormals, so it is formed in binary64 and handed out as a normal binary32 factor `a` (rounded once) times
// an exact power of two `post`, which is 1 except in those extreme cases.
struct Dequant { float a, post; };
__device__ __forceinline__ Dequant inv_scale_product(float sa, float sb) {
    const double r = 1.0 / ((double)sa * (double)sb);
    Dequant d;
    d.post = 1.0f;
    if (r < 0x1p-100) d.post = 0x1p-96f;
    else if (r > 0x1p100) d.post = 0x1p96f;
    d.a = (float)(r / (double)d.post);
    return d;
}

// Rows and columns of a tile beyond the matrix (both are multiples of 16, as are the tile's) repeat the matrix's last 16: their
// results are copies of results inside, are stored over these, equal, and change no maximum, so that no access of the
// epilogues needs a mask.
template <class T> __device__ __forceinline__ T clamp16(T at, T extent) { return at < extent ? at : extent - 16 + (at & 15); }

// Large tile number -> its place.  Consecutive workgroup ids are dealt round-robin to the 8 XCDs, each with its
// own L2, so give every XCD a contiguous range of a tile order in which any 32 consecutive tiles
// (one per CU of the XCD) form a 4 x 8 patch: 12 operand tiles fetched for 32 computed.
// `vblock` is the tile's index among the tiles of this GEMM; vblock % 8 = the XCD.
__device__ __forceinline__ void map_tile(const GemmParams &p, int vblock, int &tile_m, int &tile_n) {
    const int total = p.tiles_m * p.tiles_n;
    const int per_xcd = (total + 7) / 8;
    int t = (vblock & 7) * per_xcd + (vblock >> 3);
    if ((total & 7) != 0) {
        // ranges are uneven: fall back to the identity when the remapped id would leave the grid
        const int full = total & ~7;
        t = vblock < full ? (vblock & 7) * (full >> 3) + (vblock >> 3) : vblock;
    }
    constexpr int kGroupM = 4;
    const int group_tiles = kGroupM * p.tiles_n;
    const int gidx = t / group_tiles;
    const int first_m = gidx * kGroupM;
    const int gsize = (p.tiles_m - first_m) < kGroupM ? (p.tiles_m - first_m) : kGroupM;
    const int in_group = t - gidx * group_tiles;
    tile_m = first_m + in_group % gsize;
    tile_n = in_group / gsize;
}

// ------------------------------------------------------------------------------------------------
// 4 waves, one per SIMD and workgroup; every A and B row block is read from LDS by only two waves.  In the large tile a wave has
// no partner on its SIMD to hide stalls, so it pipelines itself: fragments are read half a K step or more before their products,
// loads go out one at a time throughout the step.  See the schedule in gemm_tile.
constexpr int kThreads = 256;
// What registers and LDS leave room for.
constexpr int waves_per_simd(int WB) { return WB == 4 ? 1 : 2; }

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
// 16 bytes that a workgroup on another XCD reads, or wrote, while the kernel runs: past this XCD's own L2 (sc1).
constexpr int kThrough = 16;
constexpr int kBufferWord3 = 0x00020000;              // of a raw buffer's descriptor: 32-bit data

template <int N> __device__ __forceinline__ void wait_dma() {       // at most N direct-to-LDS loads still in flight
    static_assert(N >= 0 && N < 64, "vmcnt has six bits");
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
#endif
}

// PART (plain store only) names the role in a sum of two products run as two launches: 1 = first half (stores
// its scaled product as fp32 scratch; the same code as 0, a separate symbol so that profiles tell it from the
// weight-gradient GEMMs), 2 = second half (the fp32 matrix p.add [M, N] is added to the scaled result before it
// is rounded and stored).  0 = an ordinary GEMM.
// LAY names how the operands lie in memory: 0 = both with the contraction index contiguous (A [M,K], B [N,K]);
// 1 = B "K-major" (stored [K,N], N contiguous); 2 = both K-major (A stored [K,M]).  A K-major tile is streamed
// into LDS as 128 rows of K x 256 (128) bytes and its MFMA fragments are read with the transposing LDS load, so the
// backward contractions read the forward's quantized tensors as they are: no transposed copies exist.
// PART = 4: one product of such a sum, the tiles of the other being elsewhere in the grid; the later of the two adds.
// PART = 3: the sum of two products in one tile -- the K loop runs twice, over (A, B) and then over (A_ph2, B_ph2)
// of the same shapes (or the other way round), and the accumulators are rescaled by the ratio of the two dequantization
// factors in between, so that one epilogue with the last factor finishes both.
//
// WIDE: the products on v_mfma_f32_32x32x64_f8f6f4, half as many of twice the length and half a K step each, 2 x 2 blocks of
// 32 x 32 per wave.  With one workgroup of one wave per SIMD no other wave fills the gaps between MFMAs: 32 cycles do not hold the reads
// and loads that go with one, 64 do.  (1040 x 2736 x 4112 23.9 us with the short form and 23.7; 48 x 896 x 10368, both K-major,
// 29.6 and 27.7; 69 drawn contractions with one small tile to a compute unit and a K-major operand 1.026 and 1.005 times what they took
// before there was the short form.)  Where the chip is full, power bounds the small tiles too: see gemm_plan.
constexpr int kLongRing = 9;                          // operand tiles of the ring of a small tile with its compute unit to itself
template <int WB, int EPI, int AFMT, int PART, int LAY, int UNITS = 5, bool WIDE = false>
__device__ __forceinline__ void gemm_tile(const GemmParams &p, const int vblock, const int sub, uint8_t *smem) {
    constexpr int BM = tile_edge(WB), BN = BM, WN = 32 * WB, kUnitBytes = unit_bytes(WB);
    constexpr int NI = 2 * WB;                         // DMA instructions of 1 KB per wave and unit
    constexpr int RB = 2 * WB;                         // blocks of 16 rows (columns) of a wave's tile; fragments of either operand
    constexpr int kUnits = UNITS, AHEAD = (UNITS - 1) / 2;   // operand tiles are issued AHEAD K steps before their use
    constexpr int kChunks = BM / 16;                   // 16-byte chunks of a K-major row
    constexpr bool HALF = PART == 4, ADD = PART == 2;
    constexpr bool TWO = PART == 3;
    constexpr bool kTwoWhole = TWO && WB == 4;         // no general loop body there (see sum_in_large_tile_ok)
    static_assert(!TWO || EPI == EPI_STORE, "a sum of two products ends in the plain store epilogue");
    constexpr bool AKM = LAY == 2, BKM = LAY >= 1;
    static_assert(!WIDE || (WB == 2 && EPI == EPI_STORE && PART == 0 && AFMT != kBF16), "plain stores of the small tile");
    constexpr bool kBwd = EPI == EPI_SWIGLU_BWD || EPI == EPI_SWIGLU_BWD_Q;     // dH -> dU, dG through the SwiGLU derivative
    static_assert(!(BKM && (EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_Q)), "the dual-B forms take K-contiguous operands");
    constexpr bool kDual = EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_Q;     // B tile = half rows of W1, half of W2
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    int l = tid & 63;            // (not const: see the note at the epilogue)
    const int wm = w >> 1, wn = w & 1;
    // the scales are read before anything else, so that nothing waits for them at the end
    const float s_a = p.sa ? *p.sa : 1.0f, s_b = p.sb ? *p.sb : 1.0f, s_b2 = kDual && p.sb2 ? *p.sb2 : 1.0f;
    const float s_a_ph2 = TWO ? *p.sa_ph2 : 1.0f, s_b_ph2 = TWO ? *p.sb_ph2 : 1.0f;
    int tile_m, tile_n;
    map_tile(p, vblock, tile_m, tile_n);
    constexpr int kTileN = kDual ? BN / 2 : BN;
    int64_t m0 = (int64_t)tile_m * tile_edge(4), n0 = (int64_t)tile_n * (kTileN * (4 / WB));
    if (WB == 2) {                                    // the sub-th quarter of the large tile
        m0 += (sub >> 1) * BM;
        n0 += (sub & 1) * kTileN;
        if (m0 >= p.M || n0 >= p.N) return;
    }

    // DMA slots: a unit is 4 * NI instructions of 1 KB, NI per wave.  K-contiguous operand: an instruction is 8 rows x
    // 128 B (rows (NI*w+j)*8 + l/8).  K-major operand: 4 rows of K x 256 B (WB = 4) or 8 x 128 B (WB = 2); the 16-byte
    // chunks of a row are permuted so that a transposing read is free of bank conflicts.  Every 32 lanes read one chunk of
    // eight consecutive K rows and of the eight that are 32 further on, which have to cover all 64 banks once.
    //   WB = 4 (a row is the 256-byte bank period): chunk c of K row k sits at position
    //     c ^ (k & 7) ^ (((c & 1) ^ (k >> 5 & 1)) << 3): the XOR with k & 7 spreads the rows over the eight positions of
    //     a half row, the chunk's own low bit picks the half.
    //   WB = 2 (two rows are the period): position c ^ ((k >> 1 & 3) << 1) ^ (k >> 5 & 1): the row's parity picks the half,
    //     the XOR spreads the four rows of one parity over four pairs of positions, k >> 5 picks the position of the pair.
    //     (WIDE: 32 lanes read two adjacent chunks of eight K rows, and k >> 5 does not enter.)
    const int lrow = l >> 3;
    const int chunk_even = (l & 7) ^ swz<WIDE>(lrow), chunk_odd = (l & 7) ^ swz<WIDE>(8 + lrow);
    // the chunk that belongs at position `pos` of K row k (the maps are their own inverses in the low three bits)
    auto kmaj_chunk = [](int k, int pos) {
        if (WB == 2) return pos ^ (((k >> 1) & 3) << 1) ^ (WIDE ? 0 : (k >> 5) & 1);
        const int low = (pos ^ k) & 7;
        return low | ((((pos >> 3) ^ (k >> 5) ^ low) & 1) << 3);
    };
    auto kmaj_row = [&](int j) { return (w * NI + j) * (64 / kChunks) + l / kChunks; };   // K row of this lane's chunk
    uint32_t a_lane[NI], b_lane[NI];
    const uint8_t *b_src = p.B;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        const int row = (w * NI + j) * 8 + lrow;
        const int ck = ((j & 1) ? chunk_odd : chunk_even) * 16;
        const int kr = kmaj_row(j);
        const int ckm = kmaj_chunk(kr, l % kChunks) * 16;               // K-major: the chunk this lane fetches
        // rows (K-major: columns) beyond the matrix are those of its last 16 again
        if (AKM) {
            int64_t gm = m0 + ckm;
            gm = clamp16(gm, p.M);
            a_lane[j] = (uint32_t)((int64_t)kr * p.M + gm);
        } else {
            int64_t gm = m0 + row;
            gm = clamp16(gm, p.M);
            a_lane[j] = (uint32_t)(gm * p.K) + ck;
        }
        if (BKM) {
            int64_t gn = n0 + ckm;
            gn = clamp16(gn, p.N);
            b_lane[j] = (uint32_t)((int64_t)kr * p.N + gn);
        } else {
            int64_t gn;
            if (kDual) gn = n0 + (row & (BN / 2 - 1));
            else gn = n0 + row;
            gn = clamp16(gn, p.N);
            b_lane[j] = (uint32_t)(gn * p.K) + ck;
        }
    }
    if (kDual && w >= 2) b_src = p.B2;      // waves 2, 3 fill the upper half of the tile rows
    const uint32_t lds_w = (uint32_t)(w * NI) * 1024u;

    // LDS byte offset of this lane's two 16-byte chunks of a fragment: row l & 15 of 16, bytes 32 (l >> 4) .. + 31 of its 128; the
    // row block of a fragment adds a wave-uniform base and a compile-time multiple of 2 KB (an instruction immediate)
    // (WIDE: row l & 31 of 32, bytes 64 kh + 32 (l >> 5) .. + 31)
    uint32_t frag_off[2], wide_off[2][2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        frag_off[e] = (uint32_t)((l & 15) * BK + ((((l >> 4) * 2 + e) ^ swz(l & 15)) << 4));
#pragma unroll
        for (int kh = 0; kh < 2; ++kh) wide_off[kh][e] = (uint32_t)((l & 31) * BK + (((kh * 4 + (l >> 5) * 2 + e) ^ swz<true>(l & 31)) << 4));
    }
    // K-major operand: lane offsets of the transposing reads.  In every group of 16 lanes the even lanes supply
    // the 8-byte words whose byte j goes to output lane j, the odd lanes those for output lane 8+j; lane p of a
    // group therefore points at K row p/2 (of eight) and at half p%2 of the 16-byte chunk that holds the 16 rows of the
    // fragment.  Four such reads (K rows +0, +8, +16, +24 from the group's 32) make one fragment.  (WIDE: two groups read the two
    // chunks of 32 rows, the other two the K rows 32 further on.)
    uint32_t tr_a[RB], tr_b[RB];
    {
        const int kg = WIDE ? l >> 5 : l >> 4, t = (l & 15) >> 1, e = l & 1;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            if (WIDE) {
                if (rb >= WB) break;
                const int ca = (wm * WB + rb) * 2 + (l >> 4 & 1), cb = (wn * WB + rb) * 2 + (l >> 4 & 1), turn = (t >> 1) << 1;
                tr_a[rb] = (uint32_t)((kg * 32 + t) * BM + ((ca ^ turn) << 4) + e * 8);
                tr_b[rb] = (uint32_t)((kg * 32 + t) * BM + ((cb ^ turn) << 4) + e * 8);
                continue;
            }
            // position of chunk c in K row k = kg * 32 + t (+ multiples of 8 below 32, which do not enter)
            auto pos = [&](int c) { return WB == 2 ? c ^ ((t >> 1) << 1) ^ (kg & 1) : ((c ^ t) & 7) | ((((c >> 3) ^ kg ^ c) & 1) << 3); };
            tr_a[rb] = (uint32_t)((kg * 32 + t) * BM + (pos(wm * RB + rb) << 4) + e * 8);
            tr_b[rb] = (uint32_t)((kg * 32 + t) * BM + (pos(wn * RB + rb) << 4) + e * 8);
        }
    }
    const uint32_t a_wave_base = (uint32_t)(wm * WN) * BK;
    const uint32_t b_wave_base = (uint32_t)(kDual ? wn * (WN / 2) : wn * WN) * BK;
    auto b_block_off = [](int nb) -> uint32_t {      // SWIGLU: the first half of the blocks from the W1 rows, the others from the W2 rows
        return (uint32_t)(kDual ? (nb / (RB / 2)) * (BN / 2) + (nb % (RB / 2)) * 16 : nb * 16) * BK;
    };

    v4f acc[RB][RB];
#pragma unroll
    for (int mb = 0; mb < RB; ++mb)
#pragma unroll
        for (int nb = 0; nb < RB; ++nb) acc[mb][nb] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    v16f wide[WB][WB];                                  // WIDE: in the place of acc
#pragma unroll
    for (int mb = 0; mb < WB; ++mb)
#pragma unroll
        for (int nb = 0; nb < WB; ++nb) wide[mb][nb] = v16f{};

    const int nk = (int)((p.K + BK - 1) / BK);
    // the staging patch of the epilogue (one 32-row slab of a wave's accumulators at a time), also used where a
    // sum of two products changes the units of its accumulators
    constexpr int kPitch = WN + 4;                       // floats; neighbouring rows are one 16-byte bank group apart
    float *stg = reinterpret_cast<float *>(smem) + w * (32 * kPitch);
    // where this lane's registers of block (r, nb) of a slab (r = 0, 1) lie in the patch
    auto stg_at = [&](int r, int nb) { return reinterpret_cast<v4f *>(stg + (r * 16 + (l & 15)) * kPitch + nb * 16 + (l >> 4) * 4); };
    // a sum of two products starts with the one whose scales are larger: its accumulators change units by a factor of
    // at most 1, so that they cannot overflow however far apart the scales are
    bool swapped = false;
    if (TWO) swapped = __builtin_amdgcn_readfirstlane((double)s_a_ph2 * (double)s_b_ph2 > (double)s_a * (double)s_b) != 0;
#pragma nounroll
    for (int phase = 0; phase < (TWO ? 2 : 1); ++phase) {
        const bool second = TWO && (phase == 1) != swapped;
        const uint8_t *a_src = second ? p.A_ph2 : p.A;
        if (TWO) b_src = second ? p.B_ph2 : p.B;
        const uint32_t smem_base = (uint32_t)(uintptr_t)(lds_void_ptr)smem;
        // general issue of unit u (unit u = A (even) / B (odd) tile of K step u/2, ring slot u % UNITS): any
        // K, zero fill of a ragged K tail
        auto issue_unit = [&](int u) {
            const int k = u >> 1;
            if (k >= nk) return;
            const uint32_t dst = smem_base + (uint32_t)(u % kUnits) * kUnitBytes + lds_w;
            const int64_t kbase = (int64_t)k * BK;
            const int64_t Kseg = p.K;
            const bool is_b = (u & 1) != 0;
            const uint8_t *base = is_b ? b_src : a_src;
            const uint8_t *zero = reinterpret_cast<const uint8_t *>(&g_zero_chunk);
            const bool kmajor = is_b ? BKM : AKM;
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                if (kmajor) {
                    const bool ok = kbase + kmaj_row(j) < Kseg;
                    dma16(ok ? base + kbase * (is_b ? p.N : p.M) + (is_b ? b_lane[j] : a_lane[j]) : zero, dst + j * 1024);
                } else {
                    const bool ok = kbase + ((j & 1) ? chunk_odd : chunk_even) * 16 < Kseg;      // K is a multiple of 16: a chunk is all in or out
                    dma16(ok ? base + kbase + (is_b ? b_lane[j] : a_lane[j]) : zero, dst + j * 1024);
                }
            }
        };
        constexpr int H = RB / 2;                            // "lo" and "hi": the first and the second half of a wave's row blocks
        constexpr int kSets = WB == 4 || WIDE ? 1 : 2;
        v8i fa[RB], fb_lo[kSets][H], fb_hi[H];
        // half e of a fragment, row block g of A (is_b: of B; lo: into `set`), out of ring slot `slot`
        auto load_half = [&](int set, bool is_b, int g, uint32_t slot, int e) {
            v8i &f = !is_b ? fa[g] : g < H ? fb_lo[set][g % H] : fb_hi[g % H];
            if (is_b ? BKM : AKM) {
                typedef int v2i_t __attribute__((ext_vector_type(2)));
                typedef __attribute__((address_space(3))) v2i_t *lds_v2i_ptr;
                const uint8_t *base = smem + slot * kUnitBytes + (is_b ? tr_b[g] : tr_a[g]) + e * 16 * BM;
                const v2i_t q0 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(base));
                const v2i_t q1 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(base + 8 * BM));
                f[4 * e] = q0.x; f[4 * e + 1] = q0.y; f[4 * e + 2] = q1.x; f[4 * e + 3] = q1.y;
            } else {
                const uint32_t ub = slot * kUnitBytes + (is_b ? b_wave_base : a_wave_base);   // uniform
                const uint32_t imm = is_b ? b_block_off(g) : (uint32_t)(g * 16 * BK);
                const uint4 q = *reinterpret_cast<const uint4 *>(smem + (frag_off[e] + ub) + imm);
                f[4 * e] = (int)q.x; f[4 * e + 1] = (int)q.y; f[4 * e + 2] = (int)q.z; f[4 * e + 3] = (int)q.w;
            }
        };
        // WIDE: fragment i of four (in the order of use) of K half kh, out of slots a and b
        v8i wa[2][WB], wb[2][WB];
        auto load_wide = [&](int kh, int i, uint32_t a, uint32_t b) {
            const bool is_b = i % 2 == 0;
            const int rb = i / 2;
            v8i f;
            if (is_b ? BKM : AKM) {
                typedef int v2i_t __attribute__((ext_vector_type(2)));
                typedef __attribute__((address_space(3))) v2i_t *lds_v2i_ptr;
                const uint8_t *base = smem + (is_b ? b : a) * kUnitBytes + (is_b ? tr_b[rb] : tr_a[rb]) + kh * 64 * BM;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const v2i_t q = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(base + k * 8 * BM));
                    f[2 * k] = q.x; f[2 * k + 1] = q.y;
                }
            } else {
                const uint32_t ub = (is_b ? b : a) * kUnitBytes + (is_b ? b_wave_base : a_wave_base);   // uniform
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const uint4 q = *reinterpret_cast<const uint4 *>(smem + (wide_off[kh][e] + ub) + rb * 32 * BK);
                    f[4 * e] = (int)q.x; f[4 * e + 1] = (int)q.y; f[4 * e + 2] = (int)q.z; f[4 * e + 3] = (int)q.w;
                }
            }
            (is_b ? wb : wa)[kh][rb] = f;
        };
        auto mul = [&](int set, int r, int c) { acc[r][c] = mfma<AFMT>(fa[r], c < H ? fb_lo[set][c % H] : fb_hi[c % H], acc[r][c]); };
        // s_waitcnt lgkmcnt(0) through the builtin (gfx9 encoding: vmcnt and expcnt fields at their
        // maxima), so that the compiler's own wait bookkeeping sees it
        auto wait_lds = [&]() { __builtin_amdgcn_s_waitcnt(0xC07F); };

        // Schedule of a K step k (units 2k, 2k+1 in ring slots sa, sb; units and steps named as with a ring of five): the quarters
        // of the wave's tile in the order (A lo, B lo), (A lo, B hi) | (A hi, B hi), (A hi, B lo), the barrier in the middle.  Each
        // wave has waited for its share of units 2k+2, 2k+3 and for its LDS reads there: step k's slots are free, step k+1 is
        // visible to all.  Before it unit 2k+4 is issued into the slot that B of step k-1 left, after it 2k+5 into that of 2k.
        // Consecutive MFMAs share a fragment, and no two stand together without what else there is to issue: an MFMA takes 32
        // cycles, eight issue slots, and nothing may follow it but what these hold.
        //   Large tile, registers for one step's fragments: B hi, A hi of step k are read before the barrier (all of them two
        //   groups of four before it), A lo and B lo of step k+1 after it, each in the place of the one whose last product is done.
        //   Small tile, bound by LDS: half a fragment after every MFMA, B hi and A hi of step k before the barrier and A lo, B lo of step
        //   k+1 after it, so that neither half has more to read or to issue than its MFMAs take.  (With B hi of step k+1 after
        //   the barrier too, three quarters of the reads in one half: K-major operands, whose fragments take twice the
        //   instructions, 48 x 896 x 10368 31.0 us and 29.5; 29 training steps in small tiles .4 % longer.)
        //   B lo is still in use when the next one is read: two sets, and steps in pairs.
        //   WIDE: the second half of step k is read before the barrier, the first half of step k+1 after it.
        constexpr int kSlots = WIDE ? WB * WB : 2 * H * H;  // MFMAs of half a step
        // the t-th MFMA of a half: by columns, in the third quarter by rows, back and forth
        auto product = [&](int set, int half, int t) {
            if constexpr (WIDE) {
                wide[t / WB][t % WB] = mfma_wide<AFMT>(wa[half][t / WB], wb[half][t % WB], wide[t / WB][t % WB]);
                return;
            }
            const int q = 2 * half + t / (H * H), g = t % (H * H) / H, i = t % H;
            const int up = g & 1 ? H - 1 - i : i, down = H - 1 - up;
            if (q == 0) mul(set, up, g);
            if (q == 1) mul(set, up, H + g);
            if (q == 2) mul(set, H + g, H + down);
            if (q == 3) mul(set, H + down, g);
        };
        // what is read after it, out of slots a and b (first half: of step k, second half: of step k+1)
        auto reads = [&](int set, int half, int t, uint32_t a, uint32_t b) {
            if constexpr (WIDE) {
                load_wide(half ^ 1, t, a, b);
                return;
            }
            if (WB == 2) {
                if (half == 0 && t < 2 * H) load_half(0, true, H + t / 2, b, t % 2);
                if (half == 0 && t >= 2 * H) load_half(0, false, H + t / 2 - H, a, t % 2);
                if (half == 1) load_half(set ^ 1, (t / 2) % 2 != 0, t / 4, (t / 2) % 2 ? b : a, t % 2);
                return;
            }
            const int g = t / H, i = t % H;
            if (half == 0) {
                const int n = 3 * g + (i == 3 ? 2 : i);     // (the third place of four is a load's)
                if (i != 2 && n < 2 * H) load_half(0, true, H + n / 2, b, n % 2);
                else if (i != 2 && n < 4 * H) load_half(0, false, n / 2, a, n % 2);
            } else if (g < H) {
                if (i < 2) load_half(0, false, g, a, i);
            } else if (i == H - 1) {
                for (int e = 0; e < 2; ++e) load_half(0, true, g - H, b, e);
            }
        };
        // which load of its unit is issued there, -1: none
        auto load_at = [](int t) { return WIDE ? t : WB == 2 ? (t % 2 ? t / 2 : -1) : (t % H == 2 ? t / H : -1); };

        const int kwhole = (int)(p.K / BK);                 // K steps with all their 128 bytes; a ragged last one is zero filled
        const int64_t a_step = AKM ? (int64_t)BK * p.M : BK, b_step = BKM ? (int64_t)BK * p.N : BK;   // bytes per K step
        if (kTwoWhole || kwhole >= AHEAD) {
            // the first UNITS - 1 units from wave-uniform bases and the lane offsets the steady state uses
#pragma unroll
            for (int u = 0; u < UNITS - 1; ++u) {
                const uint32_t dst = smem_base + (uint32_t)u * kUnitBytes + lds_w;
                const uint8_t *base = (u & 1) ? b_src + (u >> 1) * b_step : a_src + (u >> 1) * a_step;
#pragma unroll
                for (int j = 0; j < NI; ++j) dma16_s(base, (u & 1) ? b_lane[j] : a_lane[j], dst + j * 1024);
            }
        } else {
#pragma unroll
            for (int u = 0; u < UNITS - 1; ++u) issue_unit(u);
        }
        if (nk >= AHEAD) wait_dma<(UNITS - 3) * NI>();                       // units 0 and 1 have landed
        else wait_dma<0>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (WIDE) {
#pragma unroll
            for (int i = 0; i < 2 * WB; ++i) load_wide(0, i, 0, 1);
        } else {
#pragma unroll
            for (int g = 0; g < H; ++g)
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    load_half(0, false, g, 0, e);
                    load_half(0, true, g, 1, e);
                }
        }

        uint32_t sa = 0, sb = 1, sp = UNITS - 1;     // ring slots of units 2k, 2k+1 and 2k+UNITS-1
        auto next_slot = [](uint32_t s) { const uint32_t t = s + 2; return t >= (uint32_t)kUnits ? t - kUnits : t; };
        // wave-uniform sources of the units issued during step k (K step k+AHEAD): running pointers in scalar registers
        const uint8_t *ua = a_src + AHEAD * a_step, *ub = b_src + AHEAD * b_step;
        // FAST: the step's new units are whole, no per-instruction check: wave-uniform source pointers, lane offsets from
        // registers.  The last AHEAD steps, and one more before them when the last one is ragged, take the general form.
        // (a sum of two products in the large tile is launched on whole K steps, at least two, only: nothing to issue there)
        auto step = [&](auto fast, auto parity, int k) {
            constexpr bool FAST = decltype(fast)::value;
            constexpr int set = decltype(parity)::value % kSets;
            const uint32_t sa_n = next_slot(sa), sb_n = next_slot(sb);
            const uint32_t d4 = smem_base + sp * kUnitBytes + lds_w, d5 = smem_base + sa * kUnitBytes + lds_w;
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                if (!FAST && !kTwoWhole) issue_unit(2 * k + UNITS - 1 + half);
#pragma unroll
                for (int t = 0; t < kSlots; ++t) {
                    product(set, half, t);
                    __builtin_amdgcn_sched_barrier(0);
                    reads(set, half, t, half ? sa_n : sa, half ? sb_n : sb);     // (after the last step: a stale slot, never used)
                    const int j = load_at(t);
                    if (FAST && j >= 0) dma16_s(half ? ub : ua, half ? b_lane[j % NI] : a_lane[j % NI], (half ? d5 : d4) + j * 1024);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (half == 0) {
                    if (FAST || k + AHEAD < nk) wait_dma<(UNITS - 4) * NI>();    // units 2k+2, 2k+3 and all before them have landed
                    else wait_dma<0>();
                    wait_lds();
                    __builtin_amdgcn_s_barrier();
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            sp = sb; sa = sa_n; sb = sb_n;
            ua += a_step; ub += b_step;
        };
        constexpr std::integral_constant<int, 0> even{};
        constexpr std::integral_constant<int, 1> odd{};
        const int kfast = kwhole > AHEAD ? kwhole - AHEAD : 0;
        int k = 0;
        if constexpr (kSets == 1) {
            for (; k < kfast; ++k) step(std::true_type{}, even, k);
            for (; k < nk; ++k) step(std::false_type{}, even, k);
        } else {
            // An odd number of fast steps begins with the second step of a pair, B lo of the first in the other set: the last one would take
            // the general form otherwise (3 to 7 K steps in all, 84 contractions: 1.2 % on average, up to 3 %; an extra fast step
            // after the pairs costs the groups .5 % in code)
            if (kfast & 1) {
#pragma unroll
                for (int g = 0; g < H; ++g) fb_lo[kSets - 1][g] = fb_lo[0][g];
                k = -1;
            }
#pragma nounroll
            for (; k < kfast; k += 2) {
                if (k >= 0) step(std::true_type{}, even, k);
                step(std::true_type{}, odd, k + 1);
            }
            for (; k < nk; k += 2) {
                step(std::false_type{}, even, k);
                if (k + 1 < nk) step(std::false_type{}, odd, k + 1);
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (TWO && phase == 0) {
            // The accumulators hold the product done first in units of its 1 / (sa sb); the other accumulates in units
            // of its own.  They change units on a round trip through the wave's LDS patch (the ring is
            // drained here): stored from their registers, multiplied in place by ordinary vector code, loaded
            // back.  (Multiplying them in registers makes this compiler shuffle all 256 of them through the other
            // half of the register file and spill.)
            asm volatile("" : "+v"(l));      // as at the epilogue: keep this block's lane arithmetic inside the block
            const double s1 = (double)s_a * (double)s_b, s2 = (double)s_a_ph2 * (double)s_b_ph2;
            // the ratio as a normal number times an exact power of two: far below 2^-126 it still meets accumulators of 2^28
            const double ratio = swapped ? s1 / s2 : s2 / s1;
            const float post = ratio < 0x1p-100 ? 0x1p-96f : 1.0f, rho = (float)(ratio / (double)post);
#pragma unroll
            for (int slab = 0; slab < WB; ++slab) {
#pragma unroll
                for (int r = 0; r < 2; ++r)
#pragma unroll
                    for (int nb = 0; nb < RB; ++nb) *stg_at(r, nb) = acc[2 * slab + r][nb];
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int q = 0; q < 4 * WB; ++q) {
                    const int e = (q * 64 + l) * 4;
                    float4 *at = reinterpret_cast<float4 *>(stg + e / WN * kPitch + e % WN);
                    float4 v = *at;
                    v.x = v.x * rho * post; v.y = v.y * rho * post; v.z = v.z * rho * post; v.w = v.w * rho * post;
                    *at = v;
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int r = 0; r < 2; ++r)
#pragma unroll
                    for (int nb = 0; nb < RB; ++nb) {
                        acc[2 * slab + r][nb] = *stg_at(r, nb);
                        if (nb % 4 == 3) __builtin_amdgcn_sched_barrier(0);
                    }
            }
            __syncthreads();            // the patches overlap the ring slots the next product's first loads fill
        }
    }

    // ---- epilogue: a slab of 32 rows of the wave's tile at a time.  In the large tile nothing runs beside it, so it is bound
    // by its own instructions and their latencies: 16-byte accesses to the patch, all reads of a slab before their use, no
    // mask on any access (see clamp16), and one copy of the code for all slabs, in a loop (straight-line code for four would
    // be fetched once per tile and run once; dH's was 80 KB and is 15).  A slab of an fp32 weight gradient takes 1.4 us
    // (11008 x 4096 x 1024, time stamps), with one register per access and a masked store after every read 3.1; that
    // contraction 61 us (79).  dH's epilogue at T = 4096, d = 4096, f = 11008 takes 23.5 us (33): every compute unit is in it
    // at once, 134 MB of U, G, dU, dG at 5.7 TB/s.
    // (The empty statement makes the lane id opaque from here on: the compiler would compute the epilogue's lane arithmetic
    // before the main loop and spill it across.)
    asm volatile("" : "+v"(l));
    constexpr int kSlabN = kDual ? WN / 2 : WN;          // columns of the result in a wave's tile
    const int64_t wrow0 = m0 + wm * WN, wcol0 = n0 + wn * kSlabN;
    const int rows_left = wcol0 < p.N && wrow0 < p.M ? (int)(p.M - wrow0 < WN ? p.M - wrow0 : WN) : 0;
    const int cols_left = (int)(p.N - wcol0 < kSlabN ? p.N - wcol0 : kSlabN);
    const Dequant dq = TWO && !swapped ? inv_scale_product(s_a_ph2, s_b_ph2) : inv_scale_product(s_a, s_b);
    const uint32_t tile = (uint32_t)(vblock * (16 / (WB * WB)) + sub);
    f32x4 theirs[HALF ? 2 : 1][RB];                      // HALF: the other product's registers of the slab that comes next
    auto fetch_theirs = [&](int slab) {
        if constexpr (HALF) {
            const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p.other) + (size_t)tile * (BM * BN), 0, BM * BN * 4, kBufferWord3);
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int nb = 0; nb < RB; ++nb)
                    theirs[r][nb] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, tid * 16, ((slab * 2 + r) * RB + nb) * (kThreads * 16), kThrough));
        }
    };
    // the slab's accumulators, each times a factor, in ordinary registers (one block of code for each slab, which the
    // compiler must not make one that indexes them)
    auto scaled_slab = [&](int slab, float (&t)[2][RB][4], float first, float second) {
#pragma unroll
        for (int s = 0; s < WB; ++s) {
            if (slab != s) continue;
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int nb = 0; nb < RB; ++nb)
#pragma unroll
                    for (int i = 0; i < 4; ++i) t[r][nb][i] = __fmul_rn(acc[2 * s + r][nb][i], nb < RB / 2 ? first : second);
        }
    };
    auto stage_slab = [&](int slab) {
        if constexpr (HALF) {
            float t[2][RB][4];
            scaled_slab(slab, t, dq.a, dq.a);
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int nb = 0; nb < RB; ++nb) {
                    v4f v;
#pragma unroll
                    for (int k = 0; k < 4; ++k) v[k] = __fadd_rn(t[r][nb][k] * dq.post, theirs[r][nb][k]);
                    *stg_at(r, nb) = v;
                }
            if (32 * (slab + 1) < rows_left) fetch_theirs(slab + 1);
            return;
        }
#pragma unroll
        for (int s = 0; s < WB; ++s) {
            if (slab != s) continue;
            if constexpr (WIDE) {
                // a lane holds row l & 31 and, four registers at a time, columns 8 q + 4 (l >> 5) .. + 3 of a block
#pragma unroll
                for (int nb = 0; nb < WB; ++nb)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        *reinterpret_cast<v4f *>(stg + (l & 31) * kPitch + (l >> 5) * 4 + nb * 32 + q * 8) =
                            v4f{wide[s][nb][4 * q], wide[s][nb][4 * q + 1], wide[s][nb][4 * q + 2], wide[s][nb][4 * q + 3]};
            } else {
#pragma unroll
                for (int r = 0; r < 2; ++r)
#pragma unroll
                    for (int nb = 0; nb < RB; ++nb) *stg_at(r, nb) = acc[2 * s + r][nb];
            }
            asm volatile("; slab %0" :: "n"(s));         // (else the compiler makes one block of them, indexing registers in memory)
        }
    };
    // (The sum of two products runs its slabs unrolled: in a loop the compiler spills its accumulators.)
    auto for_slabs = [&](auto &&work) {
        if constexpr (TWO) {
#pragma unroll
            for (int mb = 0; mb < WB; ++mb)
                if (32 * mb < rows_left) work(32 * mb);
        } else {
#pragma nounroll
            for (int row = 0; row < rows_left; row += 32) work(row);
        }
    };
    auto pack_bf16x8 = [&](const float (&v)[8]) {
        uint32_t q[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) q[k] = pack_bf16x2(v[2 * k], v[2 * k + 1]);
        return make_uint4(q[0], q[1], q[2], q[3]);
    };
    auto unpack_bf16x8 = [&](const uint4 q, float (&v)[8]) {
        const uint32_t w4[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[2 * k] = __uint_as_float(w4[k] << 16);
            v[2 * k + 1] = __uint_as_float(w4[k] & 0xffff0000u);
        }
    };

    if (EPI == EPI_STORE || kBwd) {
        const float alpha = HALF ? 1.0f : dq.a;          // (HALF: the scales enter where the two products meet)
        const bool post = !HALF && dq.post != 1.0f;      // wave-uniform, false except for extreme scales
        // running |.| maxima of the stored dU, dG as floats: rounding to bf16 is monotone, so the
        // maximum of the rounded values is the rounded maximum (taken once, at the end); fmaxf drops NaN
        float du_maxf = 0.0f, dg_maxf = 0.0f;
        if constexpr (HALF) {
            // The product that is done first leaves its result, each lane its own registers (whole 1 KB pieces per wave, whatever
            // the tile's edges), the other adds it to its own.  Either may be the first: the sum of two numbers is the same in
            // either order.  Neither waits for the other.
            uint32_t *const arrivals = p.arrivals + tile, *const shared_word = reinterpret_cast<uint32_t *>(smem + 4 * 32 * kPitch * 4);
            if (tid == 0) *shared_word = __hip_atomic_load(arrivals, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            bool last = __builtin_amdgcn_readfirstlane(*shared_word) != 0u;
            if (!last) {
                const __amdgpu_buffer_rsrc_t mine = __builtin_amdgcn_make_buffer_rsrc(p.mine + (size_t)tile * (BM * BN), 0, BM * BN * 4, kBufferWord3);
                for_slabs([&](const int row) {
                    float t[2][RB][4];
                    scaled_slab(row >> 5, t, dq.a, dq.a);
#pragma unroll
                    for (int r = 0; r < 2; ++r)
#pragma unroll
                        for (int nb = 0; nb < RB; ++nb) {
                            f32x4 v;
#pragma unroll
                            for (int k = 0; k < 4; ++k) v[k] = t[r][nb][k] * dq.post;
                            // (No scalar offset: with one, neither the compiler nor this chip waits for the store to have read its
                            // registers, and the next vector instruction can put another piece's numbers into them, 16 lanes of one
                            // register at a time.)
                            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), mine,
                                                                   tid * 16 + (((row >> 5) * 2 + r) * RB + nb) * (kThreads * 16), 0, kThrough);
                        }
                });
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // this wave's part is where the others see it
                __syncthreads();
                if (tid == 0) *shared_word = __hip_atomic_fetch_add(arrivals, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __syncthreads();
                last = __builtin_amdgcn_readfirstlane(*shared_word) != 0u;      // the other one came in between
                if (!last) return;
            }
            asm volatile("" ::: "memory");
            if (rows_left > 0) fetch_theirs(0);
        }
        if (EPI == EPI_STORE && !ADD && p.c_f32) {
            // fp32 output: one 16-byte store per lane and pass, consecutive lanes on consecutive 16 bytes, so
            // every store instruction writes whole 512-byte (WB = 2: 256-byte) row segments
            constexpr int kLanes = WN / 4, kRows = 64 / kLanes, kPasses = 32 / kRows;
            const int lr = l / kLanes, lc = (l % kLanes) * 4, c = clamp16(lc, cols_left);
            float f[4] = {alpha, alpha, alpha, alpha};
            if (p.col_scale && rows_left > 0) {
#pragma unroll
                for (int k = 0; k < 4; ++k) f[k] = __fmul_rn(alpha, p.col_scale[wcol0 + c + k]);
            }
            float *out = reinterpret_cast<float *>(p.C) + (size_t)wrow0 * (size_t)p.N + (size_t)wcol0;
            for_slabs([&](const int row) {
                stage_slab(row >> 5);
                f32x4 v[kPasses];
#pragma unroll
                for (int pass = 0; pass < kPasses; ++pass) v[pass] = *reinterpret_cast<const f32x4 *>(stg + (pass * kRows + lr) * kPitch + lc);
#pragma unroll
                for (int pass = 0; pass < kPasses; ++pass)
#pragma unroll
                    for (int k = 0; k < 4; ++k) v[pass][k] = __fmul_rn(v[pass][k], f[k]);
                if (post) {
#pragma unroll
                    for (int pass = 0; pass < kPasses; ++pass) v[pass] *= dq.post;
                }
                f32x4 *at[kPasses];
#pragma unroll
                for (int pass = 0; pass < kPasses; ++pass)
                    at[pass] = reinterpret_cast<f32x4 *>(out + (size_t)(uint32_t)clamp16(row + pass * kRows + lr, rows_left) * (size_t)p.N + c);
                if (p.nt_store) {
                    // (the empty statements keep the compiler from making one of the two branches, which loses the hint)
                    asm volatile("; past the caches" ::: "memory");
#pragma unroll
                    for (int pass = 0; pass < kPasses; ++pass) __builtin_nontemporal_store(v[pass], at[pass]);
                    asm volatile("; past the caches" ::: "memory");
                } else {
#pragma unroll
                    for (int pass = 0; pass < kPasses; ++pass) *at[pass] = v[pass];
                }
            });
        } else {
            // a lane has eight columns of a row, the slab takes kPasses passes of kRows rows
            constexpr int kLanes = WN / 8, kRows = 64 / kLanes, kPasses = 32 / kRows, kBatch = kPasses < 4 ? kPasses : 4;
            const int lr = l / kLanes, lc = (l % kLanes) * 8, c = clamp16(lc, cols_left);
            const size_t base = (size_t)wrow0 * (size_t)p.N + (size_t)wcol0;
            auto at = [&](int row) { return base + (size_t)(uint32_t)clamp16(row + lr, rows_left) * (size_t)p.N + c; };
            // the stored U, G (or the addend) of the slab that comes next: read while this one is worked, as its registers
            // become free
            uint4 ru[kPasses], rg[kPasses];
            auto fetch = [&](int pass, int row) {
                if (ADD) {
                    ru[pass] = *reinterpret_cast<const uint4 *>(p.add + at(row));
                    rg[pass] = *reinterpret_cast<const uint4 *>(p.add + at(row) + 4);
                } else if (kBwd) {
                    ru[pass] = *reinterpret_cast<const uint4 *>(p.U + at(row));
                    rg[pass] = *reinterpret_cast<const uint4 *>(p.G + at(row));
                }
            };
            if (rows_left > 0) {
#pragma unroll
                for (int pass = 0; pass < kPasses; ++pass) fetch(pass, pass * kRows);
            }
            float f[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) f[k] = alpha;
            if (p.col_scale && rows_left > 0) {
#pragma unroll
                for (int k = 0; k < 8; ++k) f[k] = __fmul_rn(alpha, p.col_scale[wcol0 + c + k]);
            }
            float q_su = 1.0f, q_sg = 1.0f;
            if (EPI == EPI_SWIGLU_BWD_Q) {
                q_su = *p.q_scale; q_sg = *p.q_scale2;
                if (vblock == 0 && sub == 0 && tid == 0) { *p.q_scale_out = q_su; *p.q_scale_out2 = q_sg; }
            }
            for_slabs([&](const int row) {
                stage_slab(row >> 5);
                const int next = row + 32 < rows_left ? row + 32 : row;      // (the last slab's are read again, for nothing)
#pragma unroll
                for (int first = 0; first < kPasses; first += kBatch) {
                    if (kBwd) __builtin_amdgcn_sched_barrier(0);             // (the compiler would read all of the slab, and spill)
                    float v[kBatch][8];
#pragma unroll
                    for (int b = 0; b < kBatch; ++b) {
                        const float *src = stg + ((first + b) * kRows + lr) * kPitch + lc;
                        const float4 lo = *reinterpret_cast<const float4 *>(src), hi = *reinterpret_cast<const float4 *>(src + 4);
                        const float q[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
                        for (int k = 0; k < 8; ++k) v[b][k] = __fmul_rn(q[k], f[k]);
                    }
                    if (post) {
#pragma unroll
                        for (int b = 0; b < kBatch; ++b)
#pragma unroll
                            for (int k = 0; k < 8; ++k) v[b][k] *= dq.post;
                    }
#pragma unroll
                    for (int b = 0; b < kBatch; ++b) {
                        const int pass = first + b;
                        const size_t o = at(row + pass * kRows);
                        if (EPI == EPI_STORE) {
                            if (ADD) {
                                const uint32_t aw[8] = {ru[pass].x, ru[pass].y, ru[pass].z, ru[pass].w, rg[pass].x, rg[pass].y, rg[pass].z, rg[pass].w};
#pragma unroll
                                for (int k = 0; k < 8; ++k) v[b][k] = __fadd_rn(v[b][k], __uint_as_float(aw[k]));
                                fetch(pass, next + pass * kRows);
                            }
                            if (ADD && p.c_f32) {
                                float *out = reinterpret_cast<float *>(p.C) + o;
                                *reinterpret_cast<float4 *>(out) = make_float4(v[b][0], v[b][1], v[b][2], v[b][3]);
                                *reinterpret_cast<float4 *>(out + 4) = make_float4(v[b][4], v[b][5], v[b][6], v[b][7]);
                            } else {
                                *reinterpret_cast<uint4 *>(reinterpret_cast<uint16_t *>(p.C) + o) = pack_bf16x8(v[b]);
                            }
                            continue;
                        }
                        float u[8], g[8], du[8], dg[8];
                        unpack_bf16x8(ru[pass], u);
                        unpack_bf16x8(rg[pass], g);
                        fetch(pass, next + pass * kRows);
#pragma unroll
                        for (int k = 0; k < 8; ++k) {
                            swiglu_grad_f32(u[k], g[k], v[b][k], du[k], dg[k]);
                            du_maxf = fmaxf(du_maxf, fabsf(du[k]));
                            dg_maxf = fmaxf(dg_maxf, fabsf(dg[k]));
                        }
                        const uint4 qu = pack_bf16x8(du), qg = pack_bf16x8(dg);
                        if (EPI == EPI_SWIGLU_BWD_Q) {
                            // delayed scaling: the scales are known beforehand, so the bf16 values (formed only to
                            // round as the stored-tensor path does) go straight to E5M2 codes
                            unpack_bf16x8(qu, du);
                            unpack_bf16x8(qg, dg);
#pragma unroll
                            for (int k = 0; k < 8; ++k) {
                                du[k] = __fmul_rn(du[k], q_su);
                                dg[k] = __fmul_rn(dg[k], q_sg);
                            }
                            // (empty statements: what is rounded to bf16 is so before, what becomes codes does so in between)
#pragma unroll
                            for (int k = 0; k < 8; ++k) asm volatile("" : "+v"(du[k]), "+v"(dg[k]));
                            saturating_conversions();
                            uint2 cu = satcast_pk8<kE5M2>(du), cg = satcast_pk8<kE5M2>(dg);
                            asm volatile("" : "+v"(cu.x), "+v"(cu.y), "+v"(cg.x), "+v"(cg.y));
                            saturating_conversions<0>();
                            *reinterpret_cast<uint2 *>(reinterpret_cast<uint8_t *>(p.C) + o) = cu;
                            *reinterpret_cast<uint2 *>(reinterpret_cast<uint8_t *>(p.C2) + o) = cg;
                            if (p.keep_u) {
                                *reinterpret_cast<uint4 *>(p.keep_u + o) = qu;
                                *reinterpret_cast<uint4 *>(p.keep_g + o) = qg;
                            }
                        } else {
                            *reinterpret_cast<uint4 *>(reinterpret_cast<uint16_t *>(p.C) + o) = qu;
                            *reinterpret_cast<uint4 *>(reinterpret_cast<uint16_t *>(p.C2) + o) = qg;
                        }
                    }
                }
            });
        }
        // bf16 bits of the rounded maxima (an infinite maximum, 0x7f80, is kept; NaN never enters)
        uint32_t du_max = pack_bf16x2(du_maxf, 0.0f) & 0x7fffu, dg_max = pack_bf16x2(dg_maxf, 0.0f) & 0x7fffu;
        if (kBwd) {
            du_max = wave_max_u32(du_max);
            dg_max = wave_max_u32(dg_max);
            uint32_t *red = reinterpret_cast<uint32_t *>(smem + 4 * 32 * kPitch * 4);   // past the staging patches
            if (l == 0) { red[2 * w] = du_max; red[2 * w + 1] = dg_max; }
            __syncthreads();
            if (tid < 2) {
                uint32_t m = 0;
#pragma unroll
                for (int k = 0; k < 4; ++k) m = m > red[2 * k + tid] ? m : red[2 * k + tid];
                uint32_t *dst = tid == 0 ? p.amax_bits : p.amax_bits2;
                if (m) atomicMax(dst + ((vblock * (16 / (WB * WB)) + sub) % kAmaxSlots) * kAmaxSlotStride, m << 16);
            }
        }
    } else {   // EPI_SWIGLU, EPI_SWIGLU_Q: the first half of the column blocks are u, the others g of the same channels
        constexpr int kLanes = WN / 16, kRows = 64 / kLanes, kPasses = 32 / kRows;
        const int lr = l / kLanes, lc = (l % kLanes) * 8, c = clamp16(lc, cols_left);
        const Dequant dq_u = inv_scale_product(s_a, s_b), dq_g = inv_scale_product(s_a, s_b2);
        const float alpha_u = dq_u.a, alpha_g = dq_g.a;
        const bool post = dq_u.post != 1.0f || dq_g.post != 1.0f;
        // A lane holds u and g of the same elements, so the product is formed in registers; the patch only turns what is
        // stored (U and G side by side, or the codes) into whole pieces of rows.
        constexpr int NBU = RB / 2;                              // column blocks of u
        constexpr bool kCodes = EPI == EPI_SWIGLU_Q;
        constexpr int kRowBytes = kCodes ? WN / 2 + 8 : 2 * WN + 16;
        uint8_t *patch = smem + w * (32 * kRowBytes);
        const size_t base = (size_t)wrow0 * (size_t)p.N + (size_t)wcol0;
        if (kCodes) saturating_conversions();
        float hmaxf[NBU][4];                                     // fmaxf drops NaN
#pragma unroll
        for (int nb = 0; nb < NBU; ++nb)
#pragma unroll
            for (int i = 0; i < 4; ++i) hmaxf[nb][i] = 0.0f;
#pragma nounroll
        for (int row = 0; row < rows_left; row += 32) {
            float t[2][RB][4];
            scaled_slab(row >> 5, t, alpha_u, alpha_g);
            if (post) {
#pragma unroll
                for (int r = 0; r < 2; ++r)
#pragma unroll
                    for (int nb = 0; nb < RB; ++nb)
#pragma unroll
                        for (int i = 0; i < 4; ++i) t[r][nb][i] *= nb < NBU ? dq_u.post : dq_g.post;
            }
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int nb = 0; nb < NBU; nb += 2) {            // eight columns: four of two neighbouring blocks
                    float u[8], g[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) { u[k] = t[r][nb + k / 4][k % 4]; g[k] = t[r][nb + k / 4 + NBU][k % 4]; }
                    if (kCodes) {
                        // inference: the factor s_i is already inside u (folded into w1), so the product is cast as
                        // it stands; nothing else is stored
                        float h[8];
#pragma unroll
                        for (int k = 0; k < 8; ++k) h[k] = swiglu_f32(u[k], g[k]);
                        const uint2 code = satcast_pk8<kE4M3>(h);
                        uint8_t *at = patch + (r * 16 + (l & 15)) * kRowBytes + nb * 16 + (l >> 4) * 4;
                        *reinterpret_cast<uint32_t *>(at) = code.x;
                        *reinterpret_cast<uint32_t *>(at + 16) = code.y;
                        continue;
                    }
                    const uint4 qu = pack_bf16x8(u), qg = pack_bf16x8(g);
                    uint8_t *at = patch + (r * 16 + (l & 15)) * kRowBytes + nb * 32 + (l >> 4) * 8;
                    *reinterpret_cast<uint2 *>(at) = make_uint2(qu.x, qu.y);
                    *reinterpret_cast<uint2 *>(at + 32) = make_uint2(qu.z, qu.w);
                    *reinterpret_cast<uint2 *>(at + WN) = make_uint2(qg.x, qg.y);
                    *reinterpret_cast<uint2 *>(at + WN + 32) = make_uint2(qg.z, qg.w);
                    unpack_bf16x8(qu, u);
                    unpack_bf16x8(qg, g);
#pragma unroll
                    for (int k = 0; k < 8; ++k) hmaxf[nb + k / 4][k % 4] = fmaxf(hmaxf[nb + k / 4][k % 4], fabsf(swiglu_f32(u[k], g[k])));
                }
#pragma unroll
            for (int pass = 0; pass < kPasses; ++pass) {
                const uint8_t *src = patch + (pass * kRows + lr) * kRowBytes;
                const size_t o = base + (size_t)(uint32_t)clamp16(row + pass * kRows + lr, rows_left) * (size_t)p.N + c;
                if (kCodes) {
                    *reinterpret_cast<uint2 *>(reinterpret_cast<uint8_t *>(p.C) + o) = *reinterpret_cast<const uint2 *>(src + lc);
                } else {
                    *reinterpret_cast<uint4 *>(reinterpret_cast<uint16_t *>(p.C) + o) = *reinterpret_cast<const uint4 *>(src + 2 * lc);
                    *reinterpret_cast<uint4 *>(reinterpret_cast<uint16_t *>(p.C2) + o) = *reinterpret_cast<const uint4 *>(src + WN + 2 * lc);
                }
            }
        }
        if (EPI == EPI_SWIGLU) {
            // The 16 lanes of a quarter wave hold 4 NBU channels each, over a row each.  At every step a lane keeps half of its
            // channels and gives the other half to its partner, so that in the end each has the maximum of one channel:
            // one atomic instruction for all of them.  (Non-negative floats order like their bit patterns.)
            uint32_t m[4 * NBU];
#pragma unroll
            for (int nb = 0; nb < NBU; ++nb)
#pragma unroll
                for (int i = 0; i < 4; ++i) m[4 * nb + i] = __float_as_uint(hmaxf[nb][i]);
#pragma unroll
            for (int half = 2 * NBU; half > 0; half >>= 1) {
                const bool upper = (l & half) != 0;
#pragma unroll
                for (int i = 0; i < half; ++i) {
                    const uint32_t keep = upper ? m[half + i] : m[i], give = upper ? m[i] : m[half + i];
                    const uint32_t got = (uint32_t)__shfl_xor((int)give, half, 64);
                    m[i] = keep > got ? keep : got;
                }
            }
            if (NBU == 2) {
                const uint32_t o = (uint32_t)__shfl_xor((int)m[0], 8, 64);
                m[0] = m[0] > o ? m[0] : o;
            }
            const int i = l & (4 * NBU - 1);
            const int64_t channel = n0 + wn * (WN / 2) + (i >> 2) * 16 + (l >> 4) * 4 + (i & 3);
            if (channel < p.N && m[0] && (NBU == 4 || (l & 8) == 0)) atomicMax(&p.camax_bits[channel], m[0]);
        }
    }
}

// Workgroups come in sets of 8 large tiles, one per XCD: with WB = 4 a set is 8 consecutive workgroups, with WB = 2
// 32, the four quarters of a large tile on the same XCD one after the other (they share its operand panels).
template <int WB> __device__ __forceinline__ int set_of(int block) { return block >> (WB == 4 ? 3 : 5); }
template <int WB> __device__ __forceinline__ int quarter_of(int block) { return WB == 4 ? 0 : (block >> 3) & 3; }
inline unsigned set_workgroups(int WB) { return WB == 4 ? 8u : 32u; }

// One GEMM per launch.
template <int WB, int EPI, int AFMT, int PART = 0, int LAY = 0, int UNITS = 5>
__global__ void __launch_bounds__(kThreads, waves_per_simd(WB)) gemm_kernel(GemmParams p) {
    __shared__ __attribute__((aligned(1024))) uint8_t smem[smem_bytes(WB, UNITS)];
    const int b = (int)blockIdx.x, vb = (p.first_set + set_of<WB>(b)) * 8 + (b & 7);
    if (vb < p.tiles_m * p.tiles_n) gemm_tile<WB, EPI, AFMT, PART, LAY, UNITS>(p, vb, quarter_of<WB>(b), smem);
}
// The small tile with its compute unit to itself, a ring of nine.  The LDS is named at the launch: a compiler that sees 144 KB
// plans for one wave per SIMD, keeps accumulators in both halves of the register file and moves them about in the loop (116 moves
// to 32 MFMAs: 2048 x 2048 x 11008 50.6 us).  With the wide products it keeps them in one half.
extern __shared__ __attribute__((aligned(1024))) uint8_t g_long_ring[];
template <int EPI, int AFMT, int LAY>
__global__ void __launch_bounds__(kThreads, waves_per_simd(2)) gemm_alone_kernel(GemmParams p) {
    const int b = (int)blockIdx.x, vb = (p.first_set + set_of<2>(b)) * 8 + (b & 7);
    if (vb < p.tiles_m * p.tiles_n) gemm_tile<2, EPI, AFMT, 0, LAY, kLongRing>(p, vb, quarter_of<2>(b), g_long_ring);
}
template <int AFMT, int LAY>
__global__ void __launch_bounds__(kThreads, 1) gemm_wide_kernel(GemmParams p) {
    __shared__ __attribute__((aligned(1024))) uint8_t smem[smem_bytes(2, kLongRing)];
    const int b = (int)blockIdx.x, vb = (p.first_set + set_of<2>(b)) * 8 + (b & 7);
    if (vb < p.tiles_m * p.tiles_n) gemm_tile<2, EPI_STORE, AFMT, 0, LAY, kLongRing, true>(p, vb, quarter_of<2>(b), smem);
}

// Host side: algorithmic flops of the whole contraction (both weight matrices of the SwiGLU forms, both products
// of the one-launch sum)
inline double gemm_flops(const GemmArgs &a) {
    const bool dual = a.epilogue == EPI_SWIGLU || a.epilogue == EPI_SWIGLU_Q;
    return 2.0 * (double)a.M * (double)a.N * (double)a.K * (dual ? 2.0 : 1.0) * (a.part >= 3 ? 2.0 : 1.0);
}

inline int sets_of(const GemmParams &p) { return (p.tiles_m * p.tiles_n + 7) / 8; }

// Host side: the kernel's parameter block from the launch interface's argument set.
// (part = 4: of its first or second product)
inline GemmParams make_gemm_params(const GemmArgs &a, int half = 0) {
    GemmParams p;
    p.A = a.A; p.B = a.B; p.B2 = a.B2;
    p.M = a.M; p.N = a.N;
    p.K = a.a_fmt == kBF16 ? 2 * a.K : a.K;          // the kernel counts K in bytes
    p.sa = a.sa; p.sb = a.sb; p.sb2 = a.sb2; p.col_scale = a.col_scale;
    p.C = a.C; p.C2 = a.C2;
    p.U = (const uint16_t *)a.U; p.G = (const uint16_t *)a.G;
    p.camax_bits = a.camax_bits; p.amax_bits = a.amax_bits; p.amax_bits2 = a.amax_bits2;
    p.c_f32 = a.c_f32;
    p.tmp = nullptr;
    p.add = a.add;
    p.q_scale = a.q_scale; p.q_scale2 = a.q_scale2; p.q_scale_out = a.q_scale_out; p.q_scale_out2 = a.q_scale_out2;
    p.keep_u = (uint16_t *)a.keep_u; p.keep_g = (uint16_t *)a.keep_g;
    p.A_ph2 = a.A_ph2; p.B_ph2 = a.B_ph2; p.sa_ph2 = a.sa_ph2; p.sb_ph2 = a.sb_ph2;
    p.mine = nullptr; p.other = nullptr; p.arrivals = a.arrivals;
    if (a.part == 4) {
        if (half == 1) { p.A = a.A_ph2; p.B = a.B_ph2; p.sa = a.sa_ph2; p.sb = a.sb_ph2; }
        if (a.partials) {
            p.mine = a.partials + (half == 1 ? gemm_partial_floats(a.M, a.N) : 0);
            p.other = a.partials + (half == 1 ? 0 : gemm_partial_floats(a.M, a.N));
        }
    }
    p.nt_store = 0;
    constexpr int edge = tile_edge(4);
    p.tiles_m = (int)((a.M + edge - 1) / edge);
    const int n_per_tile = (a.epilogue == EPI_SWIGLU || a.epilogue == EPI_SWIGLU_Q) ? edge / 2 : edge;
    p.tiles_n = (int)((a.N + n_per_tile - 1) / n_per_tile);
    p.first_set = 0;
    p.sets = sets_of(p);
    return p;
}

}  // namespace ssg
