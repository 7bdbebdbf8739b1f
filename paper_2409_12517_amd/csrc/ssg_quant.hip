// HBM-bound passes of the FP8 Smooth-SwiGLU block for gfx950:
//   amax (Section 2: per-tensor range), the scale + saturating cast Q of Eq. 2
//   with an optional transposed copy, per-channel maxima and factors of
//   Section 4.4, and the SwiGLU product of Section 4.1 for tests.
// All loads and stores are 16-byte (8-byte for row-major code stores) vectors
// along the contiguous index; reductions use one atomic max per workgroup or
// per column on the float's bit pattern (|x| orders like an unsigned integer).
#include <type_traits>

#include "ssg_col_range.h"
#include "ssg_device.h"
#include "ssg_internal.h"
#include "ssg_meet.h"
#include "ssg_scaling.h"

namespace ssg {

// ------------------------------------------------------------------ fill
__global__ void __launch_bounds__(256) fill_u32_kernel(uint32_t *p, size_t n, uint32_t v) {
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = v;
}
void launch_fill_u32(uint32_t *p, size_t n, uint32_t value, hipStream_t st) {
    if (n == 0) return;
    profile_before(kTagSmall, st, 4.0 * (double)n);
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n, value);
    profile_after(st);
}

// Words that later kernels of the call accumulate into are zeroed on the side by its first kernel: a launch of their
// own costs 4.7 us (kernel to kernel) for a few thousand words.
__device__ __forceinline__ void zero_words(const ZeroWords &z, const unsigned first, const unsigned stride) {
#pragma unroll
    for (int k = 0; k < 2; ++k)
        for (unsigned i = first; i < z.n[k]; i += stride) z.p[k][i] = 0u;
}

// ------------------------------------------------------------------ loaders
// Each loader returns 8 consecutive elements of one row as fp32; get and widen do it in two steps, the load and the rest.
struct LoadBf16 {
    const uint16_t *p;
    typedef uint4 Raw;
    __device__ __forceinline__ Raw get(size_t off) const { return load8_raw(off); }
    // (a streaming read: the non-temporal hint keeps the source from displacing what later kernels read again)
    __device__ __forceinline__ uint4 load8_raw(size_t off) const {
        typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
        const u32x4 q = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p + off));
        return make_uint4(q[0], q[1], q[2], q[3]);
    }
    static __device__ __forceinline__ void widen(const uint4 q, float (&v)[8]) {
        uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[2 * i] = __uint_as_float(w[i] << 16);
            v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
    __device__ __forceinline__ void load8(size_t off, float (&v)[8]) const {
        uint4 q = load8_raw(off);
        uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[2 * i] = __uint_as_float(w[i] << 16);
            v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
};
struct LoadF32 {
    const float *p;
    struct Raw { float4 a, b; };
    __device__ __forceinline__ Raw get(size_t off) const {
        return Raw{*reinterpret_cast<const float4 *>(p + off), *reinterpret_cast<const float4 *>(p + off + 4)};
    }
    static __device__ __forceinline__ void widen(const Raw &q, float (&v)[8]) {
        v[0] = q.a.x; v[1] = q.a.y; v[2] = q.a.z; v[3] = q.a.w;
        v[4] = q.b.x; v[5] = q.b.y; v[6] = q.b.z; v[7] = q.b.w;
    }
    __device__ __forceinline__ void load8(size_t off, float (&v)[8]) const { widen(get(off), v); }
};
struct LoadSwiglu {          // h = u * Swish(g) from stored bf16 U, G
    const uint16_t *u, *g;
    struct Raw { uint4 u, g; };
    // plain loads: U and G were just written by the GEMM and are read again by the backward pass
    __device__ __forceinline__ Raw get(size_t off) const {
        return Raw{*reinterpret_cast<const uint4 *>(u + off), *reinterpret_cast<const uint4 *>(g + off)};
    }
    static __device__ __forceinline__ void widen(const Raw &q, float (&v)[8]) {
        float uu[8], gg[8];
        LoadBf16::widen(q.u, uu);
        LoadBf16::widen(q.g, gg);
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = swiglu_f32(uu[i], gg[i]);
    }
    __device__ __forceinline__ void load8(size_t off, float (&v)[8]) const { widen(get(off), v); }
};

// ------------------------------------------------------------------ amax
// Into one word from many workgroups: atomics on one address serialise (about 12 ns each), so where workgroups end one after
// the other those that cannot raise the maximum any more look first.  Where all end at once the look comes back stale and
// costs its latency (4096 x 4096 bf16, two runs of 16 KB per workgroup: 19.8 us with the look, 16.9 without; 256 x 1024 4.3
// and 3.9; 4096 x 11008, six runs each, 23.0 and 23.7; fp32, two units of 64 KB each, 14.3 and 17.8).
__device__ __forceinline__ void fold_max(uint32_t *word, uint32_t v, bool look) {
    if (v && (!look || v > __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) atomicMax(word, v);
}

template <class Loader, bool PACKED>
__global__ void __launch_bounds__(256) amax_kernel(Loader ld, size_t n8, uint32_t *amax_bits) {
    uint32_t m = 0;
    // work is cut into units of 2048 chunks (32 KB of bf16): 8 independent 16-byte loads per lane,
    // 4 KB apart; workgroup b takes units b, b + gridDim.x, ... (the launch picks gridDim.x so that
    // every workgroup gets the same number of units)
    const size_t units = (n8 + 2047) / 2048;
    for (size_t unit = blockIdx.x; unit < units; unit += gridDim.x) {
        const size_t i = unit * 2048 + threadIdx.x;
        float v[8][8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const size_t j = i + u * 256;
            if (j < n8) ld.load8(j * 8, v[u]);
            else {
#pragma unroll
                for (int k = 0; k < 8; ++k) v[u][k] = 0.0f;
            }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                uint32_t b = abs_bits_ignore_nan(v[u][k]);
                m = m > b ? m : b;
            }
    }
    m = wave_max_u32(m);
    __shared__ uint32_t part[4];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t r = part[0];
        for (int w = 1; w < 4; ++w) r = r > part[w] ? r : part[w];
        if (PACKED) amax_bits[blockIdx.x] = r;
        else fold_max(amax_bits, r, units > gridDim.x);
    }
}

// bf16 source: the range is taken on the raw 16-bit patterns, two per operation (biased_abs_pk, ssg_col_range.h).
// A pure streaming read: every workgroup walks contiguous runs of 4 x 256 16-byte pieces (4 independent loads per
// lane), grid-stride.  Measured on a 90 MB tensor: 13 us (6.9 TB/s) against 27-41 us for the generic kernel above
// (which widens every element to fp32 and walks 32 KB units); more loads per lane or larger workgroups are slower.
constexpr int kAmaxBf16Loads = 4;
constexpr unsigned kAmaxBlocks = 1024;
static_assert(kAmaxBlocks <= kAmaxSlotWords && kAmaxBlocks == 4 * 256, "one packed word per workgroup, four per consumer thread");
struct AmaxBatch {
    const ssg_u32x4 *src[3];
    size_t n16[3];
    uint32_t *amax_bits[3];
    ZeroWords zero;
};
// (up to three tensors per launch, blockIdx.y picks one: the ranges of x, W1, W2 share a launch)
// PACKED: workgroup b stores its maximum as word b (nothing has to be zeroed before; the consumer takes the maximum over
// all gridDim.x words); otherwise it is folded into slot b % slots.
template <bool PACKED>
__global__ void __launch_bounds__(256)
amax_bf16_kernel(const AmaxBatch batch, int slots) {
    const ssg_u32x4 *__restrict__ src = batch.src[blockIdx.y];
    const size_t n16 = batch.n16[blockIdx.y];
    uint32_t *amax_bits = batch.amax_bits[blockIdx.y];
    if (PACKED && blockIdx.y == 0) zero_words(batch.zero, blockIdx.x * 256 + threadIdx.x, gridDim.x * 256);
    ssg_i16x2 m = {0x7f, 0x7f};
    const size_t run = (size_t)kAmaxBf16Loads * 256;
    for (size_t base = (size_t)blockIdx.x * run; base < n16; base += (size_t)gridDim.x * run) {
        ssg_u32x4 v[kAmaxBf16Loads];
#pragma unroll
        for (int u = 0; u < kAmaxBf16Loads; ++u) {
            const size_t j = base + (size_t)u * 256 + threadIdx.x;
            v[u] = j < n16 ? __builtin_nontemporal_load(src + j) : ssg_u32x4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int u = 0; u < kAmaxBf16Loads; ++u)
#pragma unroll
            for (int k = 0; k < 4; ++k) m = __builtin_elementwise_max(m, biased_abs_pk(v[u][k]));
    }
    uint32_t r = wave_max_u32(unbias_max_pk(m));
    __shared__ uint32_t part[4];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = r;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w) r = r > part[w] ? r : part[w];
        r = r > part[0] ? r : part[0];
        if (PACKED) amax_bits[blockIdx.x] = r;
        else if (slots > 1) { if (r) atomicMax(amax_bits + (blockIdx.x % slots) * kAmaxSlotStride, r); }
        else fold_max(amax_bits, r, n16 > 4 * run * gridDim.x);
    }
}

static unsigned amax_blocks(size_t n16) {
    const size_t runs = (n16 + kAmaxBf16Loads * 256 - 1) / (kAmaxBf16Loads * 256);
    return (unsigned)(runs < kAmaxBlocks ? runs : kAmaxBlocks);
}

static int launch_amax_batch(const CastArgs *list, int count, const ZeroWords &zero, hipStream_t st) {
    AmaxBatch batch;
    size_t largest = 0;
    double bytes = 0.0;
    for (int i = 0; i < 3; ++i) {
        const CastArgs &c = list[i < count ? i : 0];
        const size_t n = (size_t)c.rows * (size_t)c.cols;
        batch.src[i] = (const ssg_u32x4 *)c.src; batch.n16[i] = n / 8; batch.amax_bits[i] = c.range_words;
        if (i >= count) continue;
        largest = n / 8 > largest ? n / 8 : largest;
        bytes += 2.0 * (double)n;
    }
    batch.zero = zero;
    const unsigned blocks = amax_blocks(largest);
    profile_before(kTagAmax, st, bytes);
    hipLaunchKernelGGL(amax_bf16_kernel<true>, dim3(blocks, (unsigned)count), dim3(256), 0, st, batch, 0);
    profile_after(st);
    return (int)blocks;
}

// grid of the fp32 pass: units of 2048 pieces of 8, the same number of them for every workgroup
static unsigned amax_f32_blocks(size_t n8, size_t cap) {
    const size_t units = (n8 + 2047) / 2048, per_block = (units + cap - 1) / cap;
    return (unsigned)((units + per_block - 1) / per_block);
}

void launch_amax(const void *src, SrcKind kind, size_t n, uint32_t *amax_bits, int slots, hipStream_t st) {
    size_t n8 = n / 8;      // n is a multiple of 16 at every call site (rows, cols multiples of 16)
    if (n8 == 0) return;
    profile_before(kTagAmax, st, (kind == SRC_BF16 ? 2.0 : 4.0) * (double)n);
    if (kind == SRC_BF16) {
        AmaxBatch batch;
        for (int i = 0; i < 3; ++i) { batch.src[i] = (const ssg_u32x4 *)src; batch.n16[i] = n8; batch.amax_bits[i] = amax_bits; }
        batch.zero = ZeroWords{};
        hipLaunchKernelGGL(amax_bf16_kernel<false>, dim3(amax_blocks(n8)), dim3(256), 0, st, batch, slots);
    } else {
        // (one word: the fp32 form is used by the public entry points only)
        hipLaunchKernelGGL((amax_kernel<LoadF32, false>), dim3(amax_f32_blocks(n8, 512)), dim3(256), 0, st,
                           LoadF32{(const float *)src}, n8, amax_bits);
    }
    profile_after(st);
}

// The largest of `count` packed range words, and the scale it gives.
__global__ void __launch_bounds__(256)
range_scale_kernel(const uint32_t *__restrict__ words, int count, float fmax, int pow2, float *amax_out, float *scale_out) {
    __shared__ uint32_t part[4];
    const uint32_t r = wave_max_u32(range_word_max(words, count, threadIdx.x));
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = r;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t m = part[0];
        for (int w = 1; w < 4; ++w) m = m > part[w] ? m : part[w];
        *amax_out = __uint_as_float(m);
        if (scale_out) *scale_out = scale_from_amax(__uint_as_float(m), fmax, pow2);
    }
}

void launch_range_scale(const void *src, SrcKind kind, size_t n, uint32_t *scratch, int fmt, int pow2, float *amax_out,
                        float *scale_out, hipStream_t st) {
    const size_t n8 = n / 8;
    unsigned blocks;
    profile_before(kTagAmax, st, (kind == SRC_BF16 ? 2.0 : 4.0) * (double)n);
    if (kind == SRC_BF16) {
        AmaxBatch batch;
        for (int i = 0; i < 3; ++i) { batch.src[i] = (const ssg_u32x4 *)src; batch.n16[i] = n8; batch.amax_bits[i] = scratch; }
        batch.zero = ZeroWords{};
        blocks = amax_blocks(n8);
        hipLaunchKernelGGL(amax_bf16_kernel<true>, dim3(blocks), dim3(256), 0, st, batch, 0);
    } else {
        blocks = amax_f32_blocks(n8, kAmaxBlocks);
        hipLaunchKernelGGL((amax_kernel<LoadF32, true>), dim3(blocks), dim3(256), 0, st, LoadF32{(const float *)src}, n8, scratch);
    }
    profile_after(st);
    profile_before(kTagSmall, st, 4.0 * blocks);
    hipLaunchKernelGGL(range_scale_kernel, dim3(1), dim3(256), 0, st, scratch, (int)blocks,
                       fmt == kE4M3 ? Fp8Traits<kE4M3>::fmax : Fp8Traits<kE5M2>::fmax, pow2, amax_out, scale_out);
    profile_after(st);
}

// ------------------------------------------------------------------ cast
// One workgroup converts a 128 x 128 tile.  A thread owns two 4-row x 8-column
// blocks: it loads 8 elements from each of 4 rows, scales, casts, stores the
// 8 codes of each row (8 bytes, 16 lanes cover 128 contiguous bytes), and, if
// the transposed copy is wanted, transposes its 4x4 byte blocks in registers
// and parks them in LDS as [column][row] so that the copy is written in
// 16-byte pieces that are contiguous along the source's row index.
constexpr int kTile = 128;
constexpr int kTPitchWords = 33;     // LDS pitch of one transposed column, in 32-bit words

__device__ __forceinline__ void transpose4x4_bytes(uint32_t a, uint32_t b, uint32_t c, uint32_t d,
                                                   uint32_t (&o)[4]) {
    uint32_t ab_lo = __builtin_amdgcn_perm(b, a, 0x05010400u);   // a0 b0 a1 b1
    uint32_t ab_hi = __builtin_amdgcn_perm(b, a, 0x07030602u);   // a2 b2 a3 b3
    uint32_t cd_lo = __builtin_amdgcn_perm(d, c, 0x05010400u);
    uint32_t cd_hi = __builtin_amdgcn_perm(d, c, 0x07030602u);
    o[0] = __builtin_amdgcn_perm(cd_lo, ab_lo, 0x05040100u);     // a0 b0 c0 d0
    o[1] = __builtin_amdgcn_perm(cd_lo, ab_lo, 0x07060302u);
    o[2] = __builtin_amdgcn_perm(cd_hi, ab_hi, 0x05040100u);
    o[3] = __builtin_amdgcn_perm(cd_hi, ab_hi, 0x07060302u);
}

// COUNT: also count, into counters[0] and counters[1], the elements whose scaled magnitude lies beyond the
// rounding interval of the largest finite value (only the clamp keeps them finite: overflow, Section 3) and
// the nonzero elements whose code is +-0 (underflow).
// Up to three tensors per launch (blockIdx.z picks the item; workgroups beyond an item's own tile grid leave at
// once): the casts of x, W1, W2 -- and of dU, dG -- share a launch, which saves the ramp-up and drain of two launches.
template <class Loader>
struct CastItem {
    Loader ld;
    int64_t rows, cols;
    const float *col_scale, *amax;
    int amax_slots, range_count;
    float *amax_out;
    const float *scale_in;
    float *scale_out;
    uint8_t *dst, *dst_t;
    uint32_t *record;
    unsigned long long *counters;
};
template <class Loader>
struct CastBatch {
    CastItem<Loader> item[3];
    int pow2;
    ZeroWords zero;
};
// The work of one workgroup: tile (bx, by) of item `it`, ROWS x 128.
// FACT: the per-column factor is formed here from the per-channel maxima of h that col_scale points to: s_i (kFactS) or
// s_i^-1 (kFactSinv); none otherwise.  `known`: the per-tensor scale comes from known_scale(), called by all threads, instead of
// the item.
// The first loads are under way before the scale is looked for, and small launches take tiles of 64 rows, twice as many with one round
// of loads each: there nothing but latencies counts, one after the other.
enum { kFactNone = 0, kFactS = 1, kFactSinv = 2 };
struct FromItem {};                                      // known_scale: none
template <class Loader, int FMT, bool COLSCALE, bool TRANSPOSED, bool RECORD = false, bool COUNT = false, int ROWS = kTile, int FACT = kFactNone,
          class KnownScale = FromItem>
__device__ __forceinline__ void cast_block(const CastItem<Loader> &it, const int pow2, const unsigned bx, const unsigned by,
                                           KnownScale known_scale = KnownScale{}) {
    constexpr bool KNOWN = !std::is_same<KnownScale, FromItem>::value;
    static_assert(ROWS == kTile || ((ROWS == 64 || ROWS == 16) && !TRANSPOSED), "a tile is two halves of 64 rows, or one, or 16 rows");
    constexpr int RPT = ROWS < 64 ? ROWS / 16 : 4;         // neighbouring rows of a thread
    const Loader ld = it.ld;
    const int64_t rows = it.rows, cols = it.cols;
    if ((int64_t)bx * kTile >= cols || (int64_t)by * ROWS >= rows) return;
    saturating_conversions();
    const float *__restrict__ col_scale = it.col_scale;
    const float *__restrict__ amax = it.amax;
    const int amax_slots = it.amax_slots;
    float *__restrict__ amax_out = it.amax_out;
    const float *__restrict__ scale_in = it.scale_in;
    float *__restrict__ scale_out = it.scale_out;
    uint8_t *__restrict__ dst = it.dst, *__restrict__ dst_t = it.dst_t;
    uint32_t *__restrict__ record = it.record;
    unsigned long long *__restrict__ counters = it.counters;
    __shared__ uint32_t tile[TRANSPOSED ? kTile * kTPitchWords : 1];
    uint32_t n_sat = 0, n_flush = 0;

    const int64_t row0 = (int64_t)by * ROWS;
    const int64_t col0 = (int64_t)bx * kTile;
    const int c8 = threadIdx.x & 15;       // which 8-column chunk
    const int r4 = threadIdx.x >> 4;       // which group of RPT rows (0..15) inside a half
    const int64_t col = col0 + c8 * 8;
    const bool col_ok = col < cols;

    // the four row loads of a group together: four requests in flight per lane (measured: one at a time is
    // 5-10 % slower, all eight of the lane at once is slower again)
    typename Loader::Raw raw[RPT];
    auto get = [&](int half) {
        const int64_t row = row0 + half * 64 + r4 * RPT;
        if (col_ok && row < rows)                      // rows is a multiple of 16: the group is all in or all out
#pragma unroll
            for (int r = 0; r < RPT; ++r) raw[r] = ld.get((size_t)(row + r) * (size_t)cols + (size_t)col);
    };
    get(0);

    float cs[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) cs[i] = 1.0f;
    if (COLSCALE && col_ok) {
        float4 a = *reinterpret_cast<const float4 *>(col_scale + col);
        float4 b = *reinterpret_cast<const float4 *>(col_scale + col + 4);
        cs[0] = a.x; cs[1] = a.y; cs[2] = a.z; cs[3] = a.w;
        cs[4] = b.x; cs[5] = b.y; cs[6] = b.z; cs[7] = b.w;
    }

    float sigma = 1.0f;
    bool tensor_scale = false;
    if constexpr (KNOWN) { sigma = known_scale(); tensor_scale = true; }
    else if (scale_in) { sigma = *scale_in; tensor_scale = true; }
    else if (amax) {
        // maximum over the words of the range pass, or over the slots the producers folded into: lane i of every wave
        // takes slot i (kAmaxSlots = wave size); then a wave-wide maximum
        const uint32_t *ab = reinterpret_cast<const uint32_t *>(amax);
        const int lane = threadIdx.x & 63;
        uint32_t mbits = 0u;
        if (it.range_count) {
            // one 16-byte load per thread for all of them, then across the waves: reading all words in every wave cost
            // 6 us over the casts of a step at T = 4096, d = 4096, f = 11008
            __shared__ uint32_t wave_range[4];
            mbits = wave_max_u32(range_word_max(ab, it.range_count, threadIdx.x));
            if (lane == 0) wave_range[threadIdx.x >> 6] = mbits;
            __syncthreads();
            mbits = wave_range[lane & 3];
        } else if (lane < amax_slots) {
            mbits = ab[lane * kAmaxSlotStride];
        }
        mbits = wave_max_u32(mbits);
        const float m = __uint_as_float(mbits);
        sigma = scale_from_amax(m, Fp8Traits<FMT>::fmax, pow2);
        tensor_scale = true;
        if (amax_out && bx == 0 && by == 0 && threadIdx.x == 0) *amax_out = m;
    }
    if (scale_out && bx == 0 && by == 0 && threadIdx.x == 0) *scale_out = sigma;
    if (FACT != kFactNone && col_ok) {
#pragma unroll
        for (int i = 0; i < 8; ++i) cs[i] = FACT == kFactS ? smooth_factor(cs[i]) : smooth_factor_inv(cs[i]);
    }

    ssg_i16x2 seen2 = {0x7f, 0x7f};                     // RECORD: largest (|bf16 pattern| + 0x7f) this lane met, per half
#pragma unroll
    for (int half = 0; half < (ROWS + 63) / 64; ++half) {
        const int lr = half * 64 + r4 * RPT;           // local row of the group
        uint32_t lo[RPT] = {}, hi[RPT] = {};
        if (half > 0) get(half);
        if (col_ok && row0 + lr < rows) {
            float v[RPT][8];
            if constexpr (RECORD) {
                // bf16 source: the range is taken on the raw 16-bit patterns, two per operation.  |x| + 0x7f is
                // below 0x8000 for every number and infinity and at or above it for NaN, so a signed 16-bit
                // maximum ignores NaN, as the range pass does.
#pragma unroll
                for (int r = 0; r < RPT; ++r) {
                    const uint32_t w4[4] = {raw[r].x, raw[r].y, raw[r].z, raw[r].w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const ssg_i16x2 b = __builtin_bit_cast(ssg_i16x2, (w4[i] & 0x7fff7fffu) + 0x007f007fu);
                        seen2 = __builtin_elementwise_max(seen2, b);
                    }
                }
            }
#pragma unroll
            for (int r = 0; r < RPT; ++r) Loader::widen(raw[r], v[r]);
#pragma unroll
            for (int r = 0; r < RPT; ++r) {
                const size_t off = (size_t)(row0 + lr + r) * (size_t)cols + (size_t)col;
                uint32_t nonzero = 0;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    if (COUNT) nonzero |= (v[r][i] != 0.0f ? 1u : 0u) << i;
                    if (COLSCALE) v[r][i] = __fmul_rn(v[r][i], cs[i]);
                    if (tensor_scale) v[r][i] = __fmul_rn(v[r][i], sigma);
                    if (COUNT) n_sat += fabsf(v[r][i]) > Fp8Traits<FMT>::overflow_above ? 1u : 0u;
                }
                const uint2 codes = satcast_pk8<FMT>(v[r]);
                lo[r] = codes.x;
                hi[r] = codes.y;
                if (COUNT) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const uint32_t code = ((i < 4 ? lo[r] : hi[r]) >> (8 * (i & 3))) & 0x7fu;
                        n_flush += (code == 0u && ((nonzero >> i) & 1u)) ? 1u : 0u;
                    }
                }
                *reinterpret_cast<uint2 *>(dst + off) = codes;
            }
        }
        if constexpr (TRANSPOSED) {
            uint32_t t[4];
            transpose4x4_bytes(lo[0], lo[1], lo[2], lo[3], t);
#pragma unroll
            for (int j = 0; j < 4; ++j) tile[(c8 * 8 + j) * kTPitchWords + (lr >> 2)] = t[j];
            transpose4x4_bytes(hi[0], hi[1], hi[2], hi[3], t);
#pragma unroll
            for (int j = 0; j < 4; ++j) tile[(c8 * 8 + 4 + j) * kTPitchWords + (lr >> 2)] = t[j];
        }
    }
    if (RECORD) {
        // the range this pass saw, for the history of delayed scaling: one atomic per workgroup (atomics on
        // one address from many workgroups serialise, and across XCDs they are slow: one per wave cost 20 us
        // on a 45 M element tensor)
        __shared__ uint32_t wave_seen[4];
        const uint32_t lo16 = (uint32_t)(uint16_t)seen2[0] - 0x7fu, hi16 = (uint32_t)(uint16_t)seen2[1] - 0x7fu;
        uint32_t seen = (lo16 > hi16 ? lo16 : hi16) << 16;          // bf16 pattern -> fp32 pattern of the same number
        seen = wave_max_u32(seen);
        if ((threadIdx.x & 63) == 0) wave_seen[threadIdx.x >> 6] = seen;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t m = wave_seen[0];
#pragma unroll
            for (int k = 1; k < 4; ++k) m = m > wave_seen[k] ? m : wave_seen[k];
            if (m) atomicMax(record + ((by * gridDim.x + bx) % kAmaxSlots) * kAmaxSlotStride, m);
        }
    }
    if (COUNT) {
        // one atomic per workgroup and counter, and none for a zero count
        __shared__ uint32_t wave_counts[4][2];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            n_sat += (uint32_t)__shfl_xor((int)n_sat, off, 64);
            n_flush += (uint32_t)__shfl_xor((int)n_flush, off, 64);
        }
        if ((threadIdx.x & 63) == 0) { wave_counts[threadIdx.x >> 6][0] = n_sat; wave_counts[threadIdx.x >> 6][1] = n_flush; }
        __syncthreads();
        if (threadIdx.x < 2) {
            const uint32_t c = wave_counts[0][threadIdx.x] + wave_counts[1][threadIdx.x] + wave_counts[2][threadIdx.x] +
                               wave_counts[3][threadIdx.x];
            if (c) atomicAdd(counters + threadIdx.x, (unsigned long long)c);
        }
    }
    if (TRANSPOSED) {
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int q = threadIdx.x + 256 * j;
            const int c = q >> 3;                      // local column = row of the transposed copy
            const int rc = q & 7;                      // 16-row chunk
            if (col0 + c < cols && row0 + rc * 16 < rows) {
                const uint32_t *src = &tile[c * kTPitchWords + rc * 4];
                uint4 o = make_uint4(src[0], src[1], src[2], src[3]);
                *reinterpret_cast<uint4 *>(dst_t + (size_t)(col0 + c) * (size_t)rows + (size_t)(row0 + rc * 16)) = o;
            }
        }
    }
}

template <class Loader, int FMT, bool COLSCALE, bool TRANSPOSED, bool RECORD = false, bool COUNT = false, int ROWS = kTile>
__global__ void __launch_bounds__(256)
cast_kernel(const CastBatch<Loader> batch) {
    // (the list is read where a recording cast starts a call, and not elsewhere: it costs every cast 0.15 us, 16 x 16 with a
    // given scale 2.7 and 2.55 us)
    if (RECORD && blockIdx.z == 0) zero_words(batch.zero, (blockIdx.y * gridDim.x + blockIdx.x) * 256 + threadIdx.x, gridDim.x * gridDim.y * 256);
    cast_block<Loader, FMT, COLSCALE, TRANSPOSED, RECORD, COUNT, ROWS>(batch.item[blockIdx.z], batch.pow2, blockIdx.x, blockIdx.y);
}

// The two casts between the gate/up GEMM and the last GEMM of the Smooth-SwiGLU forward in one launch: h^ =
// cast(s_i h) from bf16 U, G (Eq. 2; blockIdx.z = 0) and w3~ = Q(s^-1 w3) (the display after Eq. 2; blockIdx.z = 1).
// Both depend only on the channel factors, neither on the other.
template <bool COUNT>
__global__ void __launch_bounds__(256)
cast_h_w3_kernel(const CastItem<LoadSwiglu> h, const CastItem<LoadBf16> w3, const int pow2) {
    if (blockIdx.z == 0) cast_block<LoadSwiglu, kE4M3, true, false, false, COUNT>(h, pow2, blockIdx.x, blockIdx.y);
    else cast_block<LoadBf16, kE4M3, true, false, false, false>(w3, pow2, blockIdx.x, blockIdx.y);
}

// The same with the channel factors formed on the way: h.col_scale and w3.col_scale are the per-channel maxima of h, f.w3_camax those
// of W3.  Saves the launch of channel_factors_kernel (4.7 us; two for the plain block).  Two forms:
//   cast_h_w3_factors_kernel, Smooth-SwiGLU with few channels: every workgroup of the second cast takes the maximum of s^-1 * w3's
//     range over all channels itself, a read of 8 f bytes for each of them;
//   cast_h_w3_meet_kernel: the workgroups of the first row of tiles of h take it over their 128 channels and leave it for the
//     others (ssg_meet.h).  Their tiles are dealt first, so where there are many workgroups no one has to wait.
struct InlineFactors {
    const float *h_camax, *w3_camax;
    int64_t f;
    float *s, *sinv, *amax_w3s;
    float *hmax;                     // plain block: receives h's range
    const float *h_scale_given;      //              the scale of h as the caller gives it, or null
};
template <bool COUNT, int ROWS>
__global__ void __launch_bounds__(256)
cast_h_w3_factors_kernel(const CastItem<LoadSwiglu> h, const CastItem<LoadBf16> w3, const int pow2, const InlineFactors fac) {
    if (blockIdx.z == 0) {
        const int64_t col = (int64_t)blockIdx.x * kTile + threadIdx.x;
        if (blockIdx.y == 0 && threadIdx.x < kTile && col < fac.f) {
            const float a = fac.h_camax[col];
            fac.s[col] = smooth_factor(a);
            fac.sinv[col] = smooth_factor_inv(a);
        }
        cast_block<LoadSwiglu, kE4M3, true, false, false, COUNT, ROWS, kFactS>(h, pow2, blockIdx.x, blockIdx.y);
        return;
    }
    cast_block<LoadBf16, kE4M3, true, false, false, false, ROWS, kFactSinv>(w3, pow2, blockIdx.x, blockIdx.y, [&]() {
        uint32_t m = 0;
        for (int64_t i = threadIdx.x; i < fac.f; i += 256) {
            const uint32_t b = abs_bits_ignore_nan(__fmul_rn(fac.w3_camax[i], smooth_factor_inv(fac.h_camax[i])));
            m = m > b ? m : b;
        }
        __shared__ uint32_t wave_m[4];
        m = wave_max_u32(m);
        if ((threadIdx.x & 63) == 0) wave_m[threadIdx.x >> 6] = m;
        __syncthreads();
        m = wave_max_u32(wave_m[threadIdx.x & 3]);
        const float amax = __uint_as_float(m);
        if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *fac.amax_w3s = amax;
        return scale_from_amax(amax, Fp8Traits<kE4M3>::fmax, pow2);
    });
}

// `update`: its ranges enter the history of delayed scaling here, a workgroup each (they are complete, and no later kernel of the call
// reads the state).
template <bool COUNT, bool SMOOTH, int ROWS>
__global__ void __launch_bounds__(256)
cast_h_w3_meet_kernel(const CastItem<LoadSwiglu> h, const CastItem<LoadBf16> w3, const int pow2, const InlineFactors fac,
                      const MeetRing meeting, const ScalingUpdate update) {
    __shared__ uint32_t words[kMeetBlocks + 8];
    const int t = threadIdx.x, groups = (int)((fac.f + kTile - 1) / kTile), mine = (int)blockIdx.x;
    const unsigned salt = (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    // of channel kTile * k + t: the range of s^-1 * w3, and of h
    auto w3_range = [&](int k) {
        const int64_t i = (int64_t)k * kTile + t;
        if (t >= kTile || i >= fac.f) return 0u;
        return abs_bits_ignore_nan(SMOOTH ? __fmul_rn(fac.w3_camax[i], smooth_factor_inv(fac.h_camax[i])) : fac.w3_camax[i]);
    };
    auto h_range = [&](int k) {
        const int64_t i = (int64_t)k * kTile + t;
        return t < kTile && i < fac.f ? abs_bits_ignore_nan(fac.h_camax[i]) : 0u;
    };
    const bool first_row = blockIdx.z == 0 && blockIdx.y == 0;
    if (first_row) {
        const uint32_t a = wave_max_u32(w3_range(mine)), b = SMOOTH ? 0u : wave_max_u32(h_range(mine));
        if ((t & 63) == 0) { words[t >> 6] = a; words[4 + (t >> 6)] = b; }
        __syncthreads();
        if (t == 0) {
            meeting.leave(mine, words[0] > words[1] ? words[0] : words[1]);
            if (!SMOOTH) meeting.leave(groups + mine, words[4] > words[5] ? words[4] : words[5]);
        }
        __syncthreads();
    }
    if (blockIdx.z == 0) {
        float sigma_h = 1.0f;
        auto scale_h = [&]() {                           // plain block: one scale for the whole tensor
            const bool first = first_row && mine == 0;
            float amax = 0.0f;
            if (!fac.h_scale_given || first) amax = __uint_as_float(meet_max<256>(meeting, groups, groups, salt, words, h_range));
            if (first && t == 0) *fac.hmax = amax;
            return fac.h_scale_given ? *fac.h_scale_given : scale_from_amax(amax, 448.0f, 0);
        };
        if constexpr (SMOOTH) {
            cast_block<LoadSwiglu, kE4M3, true, false, false, COUNT, ROWS, kFactS>(h, pow2, blockIdx.x, blockIdx.y);
        } else {
            cast_block<LoadSwiglu, kE4M3, false, false, false, COUNT, ROWS>(h, pow2, blockIdx.x, blockIdx.y, [&]() { return sigma_h = scale_h(); });
        }
        if (first_row) {
            const int64_t i = (int64_t)mine * kTile + t;
            if (t < kTile && i < fac.f) {
                const float a = fac.h_camax[i];
                fac.s[i] = SMOOTH ? smooth_factor(a) : sigma_h;
                fac.sinv[i] = SMOOTH ? smooth_factor_inv(a) : 1.0f;
            }
            for (int k = mine; k < update.count; k += groups)
                if (t < 64) scaling_update_wave(update, k, t);
        }
        return;
    }
    auto scale_w3 = [&]() {
        const float amax = __uint_as_float(meet_max<256>(meeting, 0, groups, salt, words, w3_range));
        if (blockIdx.x == 0 && blockIdx.y == 0 && t == 0) *fac.amax_w3s = amax;
        return scale_from_amax(amax, Fp8Traits<kE4M3>::fmax, pow2);
    };
    if constexpr (SMOOTH) cast_block<LoadBf16, kE4M3, true, false, false, false, ROWS, kFactSinv>(w3, pow2, blockIdx.x, blockIdx.y, scale_w3);
    else cast_block<LoadBf16, kE4M3, false, false, false, false, ROWS>(w3, pow2, blockIdx.x, blockIdx.y, scale_w3);
}

// Rows of a launch's tiles, by the number of those of 128.  Small launches are bound by latencies and, where a thread has 64
// elements, by its own instructions one after the other.  A step in tiles of 128 rows, 64 and 16: 256, 256, 688 60.4 us, 56.4, 54.4;
// 1408, 256, 848 62.0, 56.3, 53.5; 384, 512, 1664 65.6, 59.8, 57.4; 1040, 1024, 2736 (396 tiles) 110.3, 108.8, 108.8; 384, 2400, 6016 (1786)
// 152, 146, 146; 2048, 2048, 5504 (1376) 290, 287; beyond 4096 tiles no difference.
static int cast_tile_rows(int64_t rows, int64_t cols, int64_t items) {
    const int64_t tiles = items * ((rows + kTile - 1) / kTile) * ((cols + kTile - 1) / kTile);
    return tiles <= 512 ? 16 : tiles <= 4096 ? 64 : kTile;
}
// f with the number as a constant
template <class F> static void with_tile_rows(int rows, F &&f) {
    if (rows == 16) f(std::integral_constant<int, 16>{});
    else if (rows == 64) f(std::integral_constant<int, 64>{});
    else f(std::integral_constant<int, kTile>{});
}

template <class Loader>
static CastItem<Loader> cast_item(const Loader &ld, const CastArgs &a) {
    return CastItem<Loader>{ld, a.rows, a.cols, a.col_scale, a.amax, a.amax_slots, a.range_count, a.amax_out, a.scale_in, a.scale_out,
                            a.dst, a.dst_t, a.record, a.counters};
}

// All items of a batch share the source kind, the format and the presence of every optional part (per-column
// factor, transposed copy, range record, counters): one kernel instantiation serves them.
static bool same_cast_form(const CastArgs &a, const CastArgs &b) {
    return a.kind == b.kind && a.fmt == b.fmt && a.pow2 == b.pow2 && (a.col_scale != nullptr) == (b.col_scale != nullptr) &&
           (a.dst_t != nullptr) == (b.dst_t != nullptr) && (a.record != nullptr) == (b.record != nullptr) &&
           (a.counters != nullptr) == (b.counters != nullptr);
}

template <class Loader, int FMT, class MakeLoader>
static void launch_cast_l(const CastArgs *list, int n, MakeLoader make, const ZeroWords &zero, hipStream_t st) {
    const CastArgs &a = list[0];
    CastBatch<Loader> batch;
    int64_t rows = 0, cols = 0;
    for (int i = 0; i < 3; ++i) {
        const CastArgs &x = list[i < n ? i : 0];
        batch.item[i] = cast_item<Loader>(make(x), x);
        if (i < n) { rows = x.rows > rows ? x.rows : rows; cols = x.cols > cols ? x.cols : cols; }
    }
    batch.pow2 = a.pow2;
    batch.zero = zero;
    const bool cs = a.col_scale != nullptr, tr = a.dst_t != nullptr;
    // (the forms of the block's own calls without a transposed copy are built for both)
    const int edge = std::is_same<Loader, LoadBf16>::value && !cs && !tr && !a.counters ? cast_tile_rows(rows, cols, n) : kTile;
    dim3 grid((unsigned)((cols + kTile - 1) / kTile), (unsigned)((rows + edge - 1) / edge), (unsigned)n);
#define SSG_CAST(...) hipLaunchKernelGGL((cast_kernel<Loader, FMT, __VA_ARGS__>), grid, dim3(256), 0, st, batch)
    if constexpr (std::is_same<Loader, LoadBf16>::value) {
        if (a.record && !cs) {
            if (tr) SSG_CAST(false, true, true);
            else with_tile_rows(edge, [&](auto r) { SSG_CAST(false, false, true, false, decltype(r)::value); });
            return;
        }
        if (edge < kTile) {
            with_tile_rows(edge, [&](auto r) { SSG_CAST(false, false, false, false, decltype(r)::value); });
            return;
        }
    }
    if (a.counters && !tr) {
        if (cs) SSG_CAST(true, false, false, true);
        else SSG_CAST(false, false, false, true);
        return;
    }
    if (cs && tr) SSG_CAST(true, true);
    else if (cs) SSG_CAST(true, false);
    else if (tr) SSG_CAST(false, true);
    else SSG_CAST(false, false);
#undef SSG_CAST
}

template <int FMT>
static void launch_cast_f(const CastArgs *list, int n, const ZeroWords &zero, hipStream_t st) {
    switch (list[0].kind) {
        case SRC_BF16:
            launch_cast_l<LoadBf16, FMT>(list, n, [](const CastArgs &x) { return LoadBf16{(const uint16_t *)x.src}; }, zero, st);
            break;
        case SRC_F32:
            launch_cast_l<LoadF32, FMT>(list, n, [](const CastArgs &x) { return LoadF32{(const float *)x.src}; }, zero, st);
            break;
        case SRC_SWIGLU:
            launch_cast_l<LoadSwiglu, FMT>(list, n, [](const CastArgs &x) {
                return LoadSwiglu{(const uint16_t *)x.src, (const uint16_t *)x.src2}; }, zero, st);
            break;
    }
}

static double cast_bytes(const CastArgs &a) {
    // algorithmic bytes: the source once (bf16 2, fp32 4, bf16 U and G 4), one code per element (two with a transposed copy)
    return ((a.kind == SRC_BF16 ? 2.0 : 4.0) + (a.dst_t ? 2.0 : 1.0)) * (double)a.rows * (double)a.cols;
}

void launch_cast_batch(const CastArgs *list, int n, const ZeroWords &zero, hipStream_t st) {
    // items that are empty or of another form than the first go on their own
    int m = 0;
    CastArgs same[3];
    for (int i = 0; i < n; ++i) {
        if (list[i].rows == 0 || list[i].cols == 0) continue;
        if (m < 3 && (m == 0 || same_cast_form(same[0], list[i]))) same[m++] = list[i];
        else launch_cast(list[i], st);
    }
    if (m == 0 || !same[0].record)                    // only a recording cast zeroes words on the side
        for (int k = 0; k < 2; ++k) launch_fill_u32(zero.p[k], zero.n[k], 0u, st);
    if (m == 0) return;
    double bytes = 0.0;
    for (int i = 0; i < m; ++i) bytes += cast_bytes(same[i]);
    const CastArgs &a = same[0];
    profile_before(a.kind == SRC_SWIGLU ? kTagCastSwiglu : a.col_scale ? kTagCastColscale : kTagCast, st, bytes);
    if (a.fmt == kE4M3) launch_cast_f<kE4M3>(same, m, zero, st);
    else launch_cast_f<kE5M2>(same, m, zero, st);
    profile_after(st);
}

void launch_cast(const CastArgs &a, hipStream_t st) { launch_cast_batch(&a, 1, ZeroWords{}, st); }

// ------------------------------------------------------------------ range and cast of small tensors in one launch
// A tensor of at most 512 KB is read whole by every workgroup (L2 serves it), which then casts its own 16 KB: no range
// words go between two launches.  Bound by the two launch latencies it replaces; a workgroup's range sweep of the 512 KB
// takes as long as the launch it saves, so the line lies there.
constexpr size_t kSmallElems = (size_t)1 << 18;
constexpr int kSmallThreads = 1024;
template <int FMT>
__global__ void __launch_bounds__(kSmallThreads) quantize_small_kernel(const CastBatch<LoadBf16> batch) {
    const CastItem<LoadBf16> &it = batch.item[blockIdx.y];
    if (blockIdx.y == 0) zero_words(batch.zero, blockIdx.x * kSmallThreads + threadIdx.x, gridDim.x * kSmallThreads);
    const unsigned n16 = (unsigned)(it.rows * it.cols / 8);
    if (blockIdx.x * kSmallThreads >= n16) return;
    const ssg_u32x4 *__restrict__ src = reinterpret_cast<const ssg_u32x4 *>(it.ld.p);
    const unsigned own = blockIdx.x * kSmallThreads + threadIdx.x;
    const ssg_u32x4 mine = own < n16 ? src[own] : ssg_u32x4{0u, 0u, 0u, 0u};
    ssg_i16x2 m = {0x7f, 0x7f};
    for (unsigned base = threadIdx.x; base < n16; base += 8 * kSmallThreads) {
        ssg_u32x4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = base + u * kSmallThreads < n16 ? src[base + u * kSmallThreads] : ssg_u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int k = 0; k < 4; ++k) m = __builtin_elementwise_max(m, biased_abs_pk(v[u][k]));
    }
    __shared__ uint32_t part[kSmallThreads / 64];
    uint32_t bits = wave_max_u32(unbias_max_pk(m));
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = bits;
    __syncthreads();
    bits = wave_max_u32(part[threadIdx.x & (kSmallThreads / 64 - 1)]);
    const float amax = __uint_as_float(bits), sigma = scale_from_amax(amax, Fp8Traits<FMT>::fmax, batch.pow2);
    if (own == 0) {
        *it.amax_out = amax; *it.scale_out = sigma;
        if (it.record) *it.record = bits;
    }
    if (own >= n16) return;
    saturating_conversions();
    float v[8];
    LoadBf16::widen(make_uint4(mine[0], mine[1], mine[2], mine[3]), v);
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = __fmul_rn(v[k], sigma);
    *reinterpret_cast<uint2 *>(it.dst + (size_t)own * 8) = satcast_pk8<FMT>(v);
}

// ------------------------------------------------------------------ range and cast of tensors that fit the registers
// Up to one workgroup per compute unit, each with up to TILES tiles of 128 x 128 in registers (100 MB on the chip) while the
// workgroups exchange their maxima (ssg_meet.h): the tensor is read once, in one launch.  Bound by HBM, and for small tensors by
// the latency of the exchange, about 2 us.  ssg_quantize with the transposed copy, in three launches before (range, scale, cast)
// and this way: 256 x 512 13.9 and 8.0 us, 1040 x 2736 13.6 and 9.7, 4096 x 4096 23.3 and 21.2, 4096 x 11008 50.4 and 41.7 (35.2 since the encode takes fewer instructions); fp32
// 2048 x 2048 15.4 and 11.0, 4096 x 5504 46.8 and 36.1.  In calls that quantize several tensors: 1040, 1024, 2736 115 and 111 us a step, the inference
// form at 272 rows, 4096, 11008 82.6 and 80.3.  Tensors of up to 2^18 elements stay with quantize_small_kernel, which has no exchange (a
// decode step of 16 rows 38.2 us, 39.0 this way).
constexpr int kHeldThreads = 512;
template <bool F32> constexpr int held_most_tiles() { return F32 ? 6 : 12; }         // 192 registers of source per lane
struct HeldItem {
    const void *src;
    int64_t rows, cols;
    uint8_t *dst, *dst_t;
    float *amax_out, *scale_out;
    uint32_t *record;                // optional: receives the range's bits
    int tiles_x, tiles;
    int first, blocks;               // workgroups (and words) of this item
};
struct HeldBatch {
    HeldItem item[3];
    int pow2;
    MeetRing meeting;
    ZeroWords zero;
};
template <bool F32, int FMT, bool TRANSPOSED, int TILES>
__global__ void __launch_bounds__(kHeldThreads, 2) quantize_held_kernel(const HeldBatch batch) {
    __shared__ uint32_t turn[TRANSPOSED ? 2 : 1][TRANSPOSED ? kTile * kTPitchWords : 1];
    __shared__ uint32_t words[kMeetBlocks + 8];
    const int b = (int)blockIdx.x, which = (b >= batch.item[1].first) + (b >= batch.item[2].first);
    const HeldItem &it = batch.item[which];
    const int own = b - it.first;
    saturating_conversions();
    zero_words(batch.zero, blockIdx.x * kHeldThreads + threadIdx.x, gridDim.x * kHeldThreads);
    // a thread has eight columns of four rows of every tile, in PER pieces of 16 bytes
    constexpr int PER = F32 ? 8 : 4;
    const int c8 = (threadIdx.x & 15) * 8, r4 = (threadIdx.x >> 4) * 4;
    auto origin = [&](int k, int t, int64_t &row0, int64_t &col0) {      // of the t-th tile of the item's workgroup k
        const int tile = k + t * it.blocks;
        row0 = (int64_t)(tile / it.tiles_x) * kTile;
        col0 = (int64_t)(tile % it.tiles_x) * kTile;
        return tile < it.tiles && row0 + r4 < it.rows && col0 + c8 < it.cols;      // (both extents are multiples of 16)
    };
    auto load = [&](int64_t row, int64_t col, ssg_u32x4 (&q)[PER]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const size_t at = (size_t)(row + r) * (size_t)it.cols + (size_t)col;
#pragma unroll
            for (int p = 0; p < PER / 4; ++p)
                q[r * (PER / 4) + p] = __builtin_nontemporal_load(reinterpret_cast<const ssg_u32x4 *>(static_cast<const uint8_t *>(it.src) + at * (F32 ? 4 : 2)) + p);
        }
    };
    struct Seen { ssg_i16x2 pk = {0x7f, 0x7f}; uint32_t bits = 0u; };
    auto see = [&](const ssg_u32x4 (&q)[PER], Seen &seen) {
#pragma unroll
        for (int p = 0; p < PER; ++p)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (F32) {
                    const uint32_t v = abs_bits_ignore_nan(__uint_as_float(q[p][k]));
                    seen.bits = seen.bits > v ? seen.bits : v;
                } else seen.pk = __builtin_elementwise_max(seen.pk, biased_abs_pk(q[p][k]));
            }
    };
    ssg_u32x4 held[TILES][PER];
    Seen seen;
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
        int64_t row0, col0;
        if (origin(own, t, row0, col0)) load(row0 + r4, col0 + c8, held[t]);
        else
#pragma unroll
            for (int p = 0; p < PER; ++p) held[t][p] = ssg_u32x4{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int t = 0; t < TILES; ++t) see(held[t], seen);
    const uint32_t mine = wave_max_u32(F32 ? seen.bits : unbias_max_pk(seen.pk));
    if ((threadIdx.x & 63) == 0) words[threadIdx.x >> 6] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t m = mine;
        for (int w = 1; w < kHeldThreads / 64; ++w) m = m > words[w] ? m : words[w];
        batch.meeting.leave(b, m);
    }
    const uint32_t bits = meet_max<kHeldThreads>(batch.meeting, it.first, it.blocks, (unsigned)own, words, [&](int k) {
        Seen s;
        for (int t = 0; k + t * it.blocks < it.tiles; ++t) {
            int64_t row0, col0;
            if (!origin(k, t, row0, col0)) continue;
            ssg_u32x4 q[PER];
            load(row0 + r4, col0 + c8, q);
            see(q, s);
        }
        return F32 ? s.bits : unbias_max_pk(s.pk);
    });
    const float amax = __uint_as_float(bits), sigma = scale_from_amax(amax, Fp8Traits<FMT>::fmax, batch.pow2);
    if (own == 0 && threadIdx.x == 0) {
        if (it.amax_out) *it.amax_out = amax;
        if (it.scale_out) *it.scale_out = sigma;
        if (it.record) *it.record = bits;
    }
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
        if (own + t * it.blocks >= it.tiles) break;
        int64_t row0, col0;
        const bool inside = origin(own, t, row0, col0);
        uint32_t code[4][2];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float v[8];
            if (F32) {
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = __uint_as_float(held[t][r * (PER / 4) + k / 4 % (PER / 4)][k % 4]);
            } else {
                const ssg_u32x4 q = held[t][r * (PER / 4)];
                LoadBf16::widen(make_uint4(q[0], q[1], q[2], q[3]), v);
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = __fmul_rn(v[k], sigma);
            const uint2 codes = satcast_pk8<FMT>(v);
            code[r][0] = codes.x;
            code[r][1] = codes.y;
            if (inside)
                *reinterpret_cast<uint2 *>(it.dst + (size_t)(row0 + r4 + r) * (size_t)it.cols + (size_t)(col0 + c8)) = codes;
        }
        if (TRANSPOSED) {
            // (two turning buffers by turns: one barrier per tile)
            uint32_t *at = turn[TRANSPOSED ? t & 1 : 0];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint32_t o[4];
                transpose4x4_bytes(code[0][h], code[1][h], code[2][h], code[3][h], o);
#pragma unroll
                for (int j = 0; j < 4; ++j) at[(c8 + 4 * h + j) * kTPitchWords + (r4 >> 2)] = o[j];
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < 1024 / kHeldThreads; ++j) {
                const int q = threadIdx.x + kHeldThreads * j, c = q >> 3, rc = q & 7;       // column of the tile, 16 rows of it
                if (col0 + c < it.cols && row0 + rc * 16 < it.rows) {
                    const uint32_t *src = &at[c * kTPitchWords + rc * 4];
                    *reinterpret_cast<uint4 *>(it.dst_t + (size_t)(col0 + c) * (size_t)it.rows + (size_t)(row0 + rc * 16)) =
                        make_uint4(src[0], src[1], src[2], src[3]);
                }
            }
        }
    }
}

// Tiles a workgroup holds so that all items' workgroups fit the chip at once; 0: they do not.
static int held_tiles(HeldItem *item, int n, bool f32) {
    int total = 0;
    for (int i = 0; i < n; ++i) {
        item[i].tiles_x = (int)((item[i].cols + kTile - 1) / kTile);
        const int64_t tiles = (int64_t)item[i].tiles_x * ((item[i].rows + kTile - 1) / kTile);
        if (tiles > kMeetBlocks * 16) return 0;
        item[i].tiles = (int)tiles;
        total += item[i].tiles;
    }
    for (int per = (total + kMeetBlocks - 1) / kMeetBlocks; per <= (f32 ? held_most_tiles<true>() : held_most_tiles<false>()); ++per) {
        int blocks = 0;
        for (int i = 0; i < n; ++i) { item[i].first = blocks; item[i].blocks = (item[i].tiles + per - 1) / per; blocks += item[i].blocks; }
        for (int i = n; i < 3; ++i) item[i].first = 1 << 30;
        if (blocks <= kMeetBlocks) return per;
    }
    return 0;
}
template <bool F32, int FMT, bool TRANSPOSED>
static void launch_held(const HeldBatch &batch, int per, unsigned blocks, hipStream_t st) {
    if (per <= 1) hipLaunchKernelGGL((quantize_held_kernel<F32, FMT, TRANSPOSED, 1>), dim3(blocks), dim3(kHeldThreads), 0, st, batch);
    else if (per <= 3) hipLaunchKernelGGL((quantize_held_kernel<F32, FMT, TRANSPOSED, 3>), dim3(blocks), dim3(kHeldThreads), 0, st, batch);
    else hipLaunchKernelGGL((quantize_held_kernel<F32, FMT, TRANSPOSED, held_most_tiles<F32>()>), dim3(blocks), dim3(kHeldThreads), 0, st, batch);
}
// false: nothing launched, the tensors do not fit or the call could be replayed
static bool launch_quantize_held(const CastArgs *list, int n, const ZeroWords &zero, int polls, hipStream_t st) {
    const bool f32 = list[0].kind == SRC_F32, tr = list[0].dst_t != nullptr;
    HeldBatch batch;
    double bytes = 0.0;
    for (int i = 0; i < 3; ++i) {
        const CastArgs &a = list[i < n ? i : 0];
        batch.item[i] = HeldItem{a.src, a.rows, a.cols, a.dst, a.dst_t, a.amax_out, a.scale_out, a.range_words, 0, 0, 0, 0};
        if (i < n) bytes += cast_bytes(a);
    }
    const int per = held_tiles(batch.item, n, f32);
    if (per == 0 || !meet_ticket(st, &batch.meeting)) return false;
    batch.meeting.polls = meet_polls(polls);
    batch.pow2 = list[0].pow2;
    batch.zero = zero;
    unsigned blocks = 0;
    for (int i = 0; i < n; ++i) blocks += (unsigned)batch.item[i].blocks;
    const int fmt = list[0].fmt;
    profile_before(kTagCast, st, bytes);
    auto go = [&](auto f, auto m, auto t) { launch_held<decltype(f)::value, decltype(m)::value, decltype(t)::value>(batch, per, blocks, st); };
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    constexpr std::integral_constant<int, kE4M3> e4{};
    constexpr std::integral_constant<int, kE5M2> e5{};
    auto pick = [&](auto f, auto t) { if (fmt == kE4M3) go(f, e4, t); else go(f, e5, t); };
    if (f32 && tr) pick(yes, yes);
    else if (f32) pick(yes, no);
    else if (tr) pick(no, yes);
    else pick(no, no);
    profile_after(st);
    return true;
}
bool launch_quantize_once(const CastArgs &a, int polls, hipStream_t st) { return launch_quantize_held(&a, 1, ZeroWords{}, polls, st); }

// Q of up to three bf16 tensors from their own ranges (Section 2).  Returns the number of packed range words each
// tensor's `range_words` holds afterwards.
int launch_quantize_batch(CastArgs *list, int n, const ZeroWords &zero, hipStream_t st) {
    size_t largest = 0;
    double bytes = 0.0;
    for (int i = 0; i < n; ++i) {
        const size_t elems = (size_t)list[i].rows * (size_t)list[i].cols;
        largest = elems > largest ? elems : largest;
        bytes += cast_bytes(list[i]);
    }
    if (largest <= kSmallElems) {
        CastBatch<LoadBf16> batch;
        for (int i = 0; i < 3; ++i) {
            const CastArgs &a = list[i < n ? i : 0];
            batch.item[i] = cast_item<LoadBf16>(LoadBf16{(const uint16_t *)a.src}, a);
            batch.item[i].record = a.range_words;
        }
        batch.pow2 = list[0].pow2;
        batch.zero = zero;
        const dim3 grid((unsigned)((largest / 8 + kSmallThreads - 1) / kSmallThreads), (unsigned)n);
        profile_before(kTagCast, st, bytes);
        if (list[0].fmt == kE4M3) hipLaunchKernelGGL(quantize_small_kernel<kE4M3>, grid, dim3(kSmallThreads), 0, st, batch);
        else hipLaunchKernelGGL(quantize_small_kernel<kE5M2>, grid, dim3(kSmallThreads), 0, st, batch);
        profile_after(st);
        return 1;
    }
    if (launch_quantize_held(list, n, zero, -1, st)) return 1;
    const int words = launch_amax_batch(list, n, zero, st);
    for (int i = 0; i < n; ++i) {
        list[i].amax = reinterpret_cast<const float *>(list[i].range_words);
        list[i].range_count = words;
    }
    launch_cast_batch(list, n, ZeroWords{}, st);
    return words;
}

bool cast_h_w3_ok(const CastArgs &h, const CastArgs &w3) {
    return h.kind == SRC_SWIGLU && w3.kind == SRC_BF16 && h.fmt == kE4M3 && w3.fmt == kE4M3 && h.col_scale && w3.col_scale &&
           !h.dst_t && !w3.dst_t && !h.record && !w3.record && !w3.counters && h.rows > 0 && w3.rows > 0 && h.cols > 0 &&
           w3.cols > 0;
}

template <bool COUNT, int ROWS>
static void launch_h_w3_factors(dim3 grid, bool smooth, const CastItem<LoadSwiglu> &h, const CastItem<LoadBf16> &w3, int pow2,
                                const InlineFactors &in, const MeetRing *meeting, const ScalingUpdate &update, hipStream_t st) {
    if (!meeting) hipLaunchKernelGGL((cast_h_w3_factors_kernel<COUNT, ROWS>), grid, dim3(256), 0, st, h, w3, pow2, in);
    else if (smooth) hipLaunchKernelGGL((cast_h_w3_meet_kernel<COUNT, true, ROWS>), grid, dim3(256), 0, st, h, w3, pow2, in, *meeting, update);
    else hipLaunchKernelGGL((cast_h_w3_meet_kernel<COUNT, false, ROWS>), grid, dim3(256), 0, st, h, w3, pow2, in, *meeting, update);
}

void launch_cast_h_w3(const CastArgs &h, const CastArgs &w3, const ChannelFactors &fac, hipStream_t st) {
    const bool pair = cast_h_w3_ok(h, w3);
    // the line between the two forms that need no launch of their own for the factors: 8 f bytes read by every workgroup of the w3 cast
    // against the exchange
    const bool few = pair && fac.smooth && fac.update.count == 0 && fac.f <= 1024;
    MeetRing meeting;
    const bool meet = pair && !few && (fac.smooth ? 1 : 2) * ((fac.f + kTile - 1) / kTile) <= kMeetBlocks && meet_ticket(st, &meeting);
    if (!few && !meet) launch_channel_factors(fac, st);
    if (!pair) {                            // not the pair this launch is built for: one after the other
        launch_cast(h, st);
        launch_cast(w3, st);
        return;
    }
    CastItem<LoadSwiglu> hi = cast_item<LoadSwiglu>(LoadSwiglu{(const uint16_t *)h.src, (const uint16_t *)h.src2}, h);
    CastItem<LoadBf16> wi = cast_item<LoadBf16>(LoadBf16{(const uint16_t *)w3.src}, w3);
    const int64_t rows = h.rows > w3.rows ? h.rows : w3.rows, cols = h.cols > w3.cols ? h.cols : w3.cols;
    const int edge = few || meet ? cast_tile_rows(rows, cols, 2) : kTile;
    const dim3 grid((unsigned)((cols + kTile - 1) / kTile), (unsigned)((rows + edge - 1) / edge), 2u);
    profile_before(kTagCastHW3, st, cast_bytes(h) + cast_bytes(w3));
    if (few || meet) {
        hi.col_scale = wi.col_scale = fac.h_camax;
        wi.amax = nullptr;
        const InlineFactors in{fac.h_camax, fac.w3_camax, fac.f, fac.s, fac.sinv, reinterpret_cast<float *>(fac.amax_w3s_bits),
                               reinterpret_cast<float *>(fac.hmax_bits), fac.h_scale_given};
        const MeetRing *m = meet ? &meeting : nullptr;
        with_tile_rows(edge, [&](auto r) {
            if (h.counters) launch_h_w3_factors<true, decltype(r)::value>(grid, fac.smooth, hi, wi, w3.pow2, in, m, fac.update, st);
            else launch_h_w3_factors<false, decltype(r)::value>(grid, fac.smooth, hi, wi, w3.pow2, in, m, fac.update, st);
        });
    } else if (h.counters) hipLaunchKernelGGL(cast_h_w3_kernel<true>, grid, dim3(256), 0, st, hi, wi, w3.pow2);
    else hipLaunchKernelGGL(cast_h_w3_kernel<false>, grid, dim3(256), 0, st, hi, wi, w3.pow2);
    profile_after(st);
}

// ------------------------------------------------------------------ per-column amax
// Grid (cols/512, rows/128).  A wave reads 1 KB of a row per load; a lane keeps 8 running column
// maxima over its wave's share of the slab's rows; the four waves of a workgroup meet in LDS and
// one atomic per column goes to memory.
constexpr int kSlabRows = 128;

template <class Loader>
__global__ void __launch_bounds__(256)
col_amax_kernel(Loader ld, int64_t rows, int64_t cols, uint32_t *__restrict__ camax_bits) {
    __shared__ uint32_t cmax[kColTile];
    cmax[threadIdx.x] = 0;
    cmax[threadIdx.x + 256] = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t col = (int64_t)blockIdx.x * kColTile + lane * 8;
    const int64_t row0 = (int64_t)blockIdx.y * kSlabRows;
    const int64_t row1 = row0 + kSlabRows < rows ? row0 + kSlabRows : rows;
    if (col < cols) {
        uint32_t m[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int64_t r = row0 + w; r < row1; r += 16) {        // four independent row loads in flight per lane
            float v[4][8];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t rr = r + 4 * u;
                if (rr < row1) ld.load8((size_t)rr * (size_t)cols + (size_t)col, v[u]);
                else {
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[u][i] = 0.0f;
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    uint32_t b = abs_bits_ignore_nan(v[u][i]);
                    m[i] = m[i] > b ? m[i] : b;
                }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (m[i]) atomicMax(&cmax[lane * 8 + i], m[i]);
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int t = threadIdx.x + 256 * h;
        const int64_t c = (int64_t)blockIdx.x * kColTile + t;
        if (c < cols && cmax[t]) atomicMax(&camax_bits[c], cmax[t]);
    }
}

// bf16 source: the workgroup's work is col_range_bf16_block (ssg_col_range.h), shared with the gate/up GEMM's grid.
__global__ void __launch_bounds__(256)
col_amax_bf16_kernel(const uint16_t *__restrict__ src, int64_t rows, int64_t cols, uint32_t *__restrict__ camax_bits) {
    __shared__ uint32_t cmax[kColTile];
    col_range_bf16_block<8>(src, rows, cols, camax_bits, (int)blockIdx.x, (int)blockIdx.y, cmax);
}

void launch_col_amax(const void *src, const void *src2, SrcKind kind, int64_t rows, int64_t cols,
                     uint32_t *camax_bits, hipStream_t st) {
    if (rows == 0 || cols == 0) return;
    dim3 grid((unsigned)((cols + kColTile - 1) / kColTile), (unsigned)((rows + kSlabRows - 1) / kSlabRows));
    profile_before(kTagColAmax, st, (double)rows * (double)cols * (kind == SRC_F32 ? 4.0 : kind == SRC_SWIGLU ? 4.0 : 2.0));
    switch (kind) {
        case SRC_BF16:
            grid.y = (unsigned)col_range_blocks_y(rows);
            hipLaunchKernelGGL(col_amax_bf16_kernel, grid, dim3(256), 0, st, (const uint16_t *)src, rows, cols, camax_bits);
            break;
        case SRC_F32:
            hipLaunchKernelGGL(col_amax_kernel<LoadF32>, grid, dim3(256), 0, st, LoadF32{(const float *)src},
                               rows, cols, camax_bits);
            break;
        case SRC_SWIGLU:
            hipLaunchKernelGGL(col_amax_kernel<LoadSwiglu>, grid, dim3(256), 0, st,
                               LoadSwiglu{(const uint16_t *)src, (const uint16_t *)src2}, rows, cols, camax_bits);
            break;
    }
    profile_after(st);
}

// ------------------------------------------------------------------ per-channel factors
// Smooth-SwiGLU (Section 4.4): s_i = fl32(448 / a_i), sinv_i = fl32(a_i / 448),
// both 1 for an all-zero channel.  The range of s^-1 * w3 needs no pass over
// W3: rounding is monotone, so max_j fl32(|w_ji| * sinv_i) = fl32(max_j |w_ji| * sinv_i).
// Workgroups after the `blocks` of the factors enter the call's ranges into the history of delayed scaling, a tensor
// each: they are complete by now and no later kernel of the call reads the state.
__global__ void __launch_bounds__(256)
channel_factors_kernel(const float *__restrict__ h_camax, const float *__restrict__ w3_camax, int64_t f,
                       int smooth, const uint32_t *__restrict__ hmax_bits, const float *__restrict__ h_scale_given,
                       float *__restrict__ s, float *__restrict__ sinv, uint32_t *__restrict__ amax_w3s_bits,
                       const unsigned blocks, const ScalingUpdate update) {
    if (blockIdx.x >= blocks) {
        if (threadIdx.x < 64) scaling_update_wave(update, (int)(blockIdx.x - blocks), (int)threadIdx.x);
        return;
    }
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    uint32_t wbits = 0;
    if (i < f) {
        float si, sv;
        if (smooth) {
            const float a = h_camax[i];
            si = smooth_factor(a);
            sv = smooth_factor_inv(a);
        } else {
            // plain block: one scale for the whole tensor, from its own range or as the caller gives it
            si = h_scale_given ? *h_scale_given : scale_from_amax(__uint_as_float(*hmax_bits), 448.0f, 0);
            sv = 1.0f;
        }
        s[i] = si;
        sinv[i] = sv;
        wbits = abs_bits_ignore_nan(__fmul_rn(w3_camax[i], sv));
    }
    wbits = wave_max_u32(wbits);
    if ((threadIdx.x & 63) == 0 && wbits) atomicMax(amax_w3s_bits, wbits);
}

__global__ void __launch_bounds__(256)
vec_max_kernel(const float *__restrict__ v, int64_t n, uint32_t *__restrict__ out_bits) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    uint32_t b = i < n ? abs_bits_ignore_nan(v[i]) : 0u;
    b = wave_max_u32(b);
    if ((threadIdx.x & 63) == 0 && b) atomicMax(out_bits, b);
}

void launch_channel_factors(const ChannelFactors &c, hipStream_t st) {
    const unsigned blocks = (unsigned)((c.f + 255) / 256);
    if (!c.smooth) {
        profile_before(kTagSmall, st, 4.0 * (double)c.f);
        hipLaunchKernelGGL(vec_max_kernel, dim3(blocks), dim3(256), 0, st, c.h_camax, c.f, c.hmax_bits);
        profile_after(st);
    }
    profile_before(kTagSmall, st, 16.0 * (double)c.f);
    hipLaunchKernelGGL(channel_factors_kernel, dim3(blocks + (unsigned)c.update.count), dim3(256), 0, st, c.h_camax, c.w3_camax, c.f,
                       c.smooth, c.hmax_bits, c.smooth ? nullptr : c.h_scale_given, c.s, c.sinv, c.amax_w3s_bits, blocks, c.update);
    profile_after(st);
}

__global__ void __launch_bounds__(256)
fold_range_kernel(const float *__restrict__ w3_camax, const float *__restrict__ sinv, int64_t f,
                  uint32_t *__restrict__ amax_bits) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    uint32_t b = i < f ? abs_bits_ignore_nan(__fmul_rn(w3_camax[i], sinv[i])) : 0u;
    b = wave_max_u32(b);
    if ((threadIdx.x & 63) == 0 && b) atomicMax(amax_bits, b);
}
void launch_fold_range(const float *w3_camax, const float *sinv, int64_t f, uint32_t *amax_bits, hipStream_t st) {
    hipLaunchKernelGGL(fold_range_kernel, dim3((unsigned)((f + 255) / 256)), dim3(256), 0, st, w3_camax, sinv, f,
                       amax_bits);
}

// ------------------------------------------------------------------ SwiGLU product (tests)
__global__ void __launch_bounds__(256)
swiglu_kernel(LoadSwiglu ld, size_t n8, float *__restrict__ h) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n8) return;
    float v[8];
    ld.load8(i * 8, v);
    *reinterpret_cast<float4 *>(h + i * 8) = make_float4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<float4 *>(h + i * 8 + 4) = make_float4(v[4], v[5], v[6], v[7]);
}
void launch_swiglu(const void *U, const void *G, int64_t n, float *h, hipStream_t st) {
    const size_t n8 = (size_t)n / 8;
    if (n8 == 0) return;
    hipLaunchKernelGGL(swiglu_kernel, dim3((unsigned)((n8 + 255) / 256)), dim3(256), 0, st,
                       LoadSwiglu{(const uint16_t *)U, (const uint16_t *)G}, n8, h);
}

// ------------------------------------------------------------------ bf16 transposes (last layer left in bf16)
// The comparison variant of Section 4.3 runs the last linear layer and its two gradient contractions on bf16
// operands; those contract over the index that is not contiguous in W3 [d,f], dY [T,d] and h [T,f], so transposed
// bf16 copies are written (64 x 64 tiles through LDS, 16-byte accesses on both sides).  SWIGLU: the source is the
// SwiGLU product of bf16 U, G, rounded once to bf16; it is written both as it stands and transposed.
template <bool SWIGLU>
__global__ void __launch_bounds__(256)
transpose_bf16_kernel(const uint16_t *__restrict__ src, const uint16_t *__restrict__ src2, int64_t rows, int64_t cols,
                      uint16_t *__restrict__ dst, uint16_t *__restrict__ dst_t) {
    __shared__ uint16_t tile[64][64 + 8];
    const int64_t row0 = (int64_t)blockIdx.y * 64, col0 = (int64_t)blockIdx.x * 64;
    const int c8 = (threadIdx.x & 7) * 8, r = threadIdx.x >> 3;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const int64_t row = row0 + r + 32 * half, col = col0 + c8;
        uint4 q = make_uint4(0u, 0u, 0u, 0u);
        if (row < rows && col < cols) {
            const size_t at = (size_t)row * (size_t)cols + (size_t)col;
            if (SWIGLU) {
                float v[8];
                LoadSwiglu{src, src2}.load8(at, v);
                q = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
                *reinterpret_cast<uint4 *>(dst + at) = q;
            } else {
                q = *reinterpret_cast<const uint4 *>(src + at);
            }
        }
        *reinterpret_cast<uint4 *>(&tile[r + 32 * half][c8]) = q;
    }
    __syncthreads();
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const int c = r + 32 * half;                          // source column = row of the transposed copy
        const int64_t col = col0 + c, row = row0 + c8;        // c8 now counts source rows
        if (col < cols && row < rows) {
            uint32_t w[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) w[k] = (uint32_t)tile[c8 + 2 * k][c] | ((uint32_t)tile[c8 + 2 * k + 1][c] << 16);
            *reinterpret_cast<uint4 *>(dst_t + (size_t)col * (size_t)rows + (size_t)row) = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
}
void launch_transpose_bf16(const void *src, int64_t rows, int64_t cols, void *dst_t, hipStream_t st) {
    if (rows == 0 || cols == 0) return;
    const dim3 grid((unsigned)((cols + 63) / 64), (unsigned)((rows + 63) / 64));
    profile_before(kTagTranspose, st, 4.0 * (double)rows * (double)cols);
    hipLaunchKernelGGL(transpose_bf16_kernel<false>, grid, dim3(256), 0, st, (const uint16_t *)src, nullptr, rows, cols,
                       nullptr, (uint16_t *)dst_t);
    profile_after(st);
}
void launch_swiglu_bf16(const void *U, const void *G, int64_t rows, int64_t cols, void *h, void *h_t, hipStream_t st) {
    if (rows == 0 || cols == 0) return;
    const dim3 grid((unsigned)((cols + 63) / 64), (unsigned)((rows + 63) / 64));
    profile_before(kTagTranspose, st, 8.0 * (double)rows * (double)cols);
    hipLaunchKernelGGL(transpose_bf16_kernel<true>, grid, dim3(256), 0, st, (const uint16_t *)U, (const uint16_t *)G, rows, cols,
                       (uint16_t *)h, (uint16_t *)h_t);
    profile_after(st);
}

// ------------------------------------------------------------------ per-row factor, then per-tensor Q
// w1~ = Q(s_i * w1_i) of the inference form (end of Section 4.4): row i of a [rows, cols] bf16 matrix is
// multiplied by rs[i] (one fp32 multiply), the result is quantized per tensor to E4M3.  Run once per
// set of weights, so two plain elementwise passes: range, then cast.  cols is a multiple of 16, so
// the 8 elements of a lane share a row.
__global__ void __launch_bounds__(256)
rowscale_amax_kernel(const uint16_t *__restrict__ w, const float *__restrict__ rs, int64_t rows, int64_t cols,
                     uint32_t *__restrict__ slots) {
    const size_t n = (size_t)rows * (size_t)cols, stride = (size_t)gridDim.x * 256 * 8;
    uint32_t m = 0;
    for (size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 8; i < n; i += stride) {
        float v[8];
        LoadBf16{w}.load8(i, v);
        const float f = rs[i / (size_t)cols];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint32_t b = abs_bits_ignore_nan(__fmul_rn(v[k], f));
            m = m > b ? m : b;
        }
    }
    m = wave_max_u32(m);
    if ((threadIdx.x & 63) == 0 && m) atomicMax(slots + (blockIdx.x % kAmaxSlots) * kAmaxSlotStride, m);
}
__global__ void __launch_bounds__(256)
rowscale_cast_kernel(const uint16_t *__restrict__ w, const float *__restrict__ rs, int64_t rows, int64_t cols,
                     const uint32_t *__restrict__ slots, int pow2, float *__restrict__ scale_out,
                     float *__restrict__ amax_out, uint8_t *__restrict__ dst) {
    const float amax = __uint_as_float(wave_max_u32(slots[(threadIdx.x & 63) * kAmaxSlotStride]));
    const float sigma = scale_from_amax(amax, Fp8Traits<kE4M3>::fmax, pow2);
    if (blockIdx.x == 0 && threadIdx.x == 0) { *scale_out = sigma; if (amax_out) *amax_out = amax; }
    const size_t n = (size_t)rows * (size_t)cols, stride = (size_t)gridDim.x * 256 * 8;
    saturating_conversions();
    for (size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 8; i < n; i += stride) {
        float v[8];
        LoadBf16{w}.load8(i, v);
        const float f = rs[i / (size_t)cols];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = __fmul_rn(__fmul_rn(v[k], f), sigma);
        *reinterpret_cast<uint2 *>(dst + i) = satcast_pk8<kE4M3>(v);
    }
}
void launch_rowscale_quantize(const void *w, const float *row_scale, int64_t rows, int64_t cols, uint32_t *slots,
                              int pow2, float *scale_out, float *amax_out, uint8_t *dst, hipStream_t st) {
    const size_t groups = ((size_t)rows * (size_t)cols / 8 + 255) / 256;
    const unsigned blocks = (unsigned)(groups < 4096 ? groups : 4096);
    hipLaunchKernelGGL(rowscale_amax_kernel, dim3(blocks), dim3(256), 0, st, (const uint16_t *)w, row_scale, rows, cols, slots);
    hipLaunchKernelGGL(rowscale_cast_kernel, dim3(blocks), dim3(256), 0, st, (const uint16_t *)w, row_scale, rows, cols,
                       slots, pow2, scale_out, amax_out, dst);
}

// ------------------------------------------------------------------ delayed scaling state
__global__ void __launch_bounds__(256) scaling_init_kernel(uint32_t *state, size_t words) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= words) return;
    const bool is_scale = i < (size_t)kScalingTensors * kScalingStride && (i % kScalingStride) == 0;
    state[i] = is_scale ? 0x3f800000u : 0u;            // empty history: scale 1
}
void launch_scaling_init(uint32_t *state, hipStream_t st) {
    hipLaunchKernelGGL(scaling_init_kernel, dim3((unsigned)((kScalingWords + 255) / 256)), dim3(256), 0, st, state,
                       kScalingWords);
}

__global__ void __launch_bounds__(64) scaling_update_kernel(ScalingUpdate u) {
    scaling_update_wave(u, (int)blockIdx.x, (int)threadIdx.x);
}
void launch_scaling_update(const ScalingUpdate &u, hipStream_t st) {
    if (u.count <= 0) return;
    profile_before(kTagSmall, st, 0.0);
    hipLaunchKernelGGL(scaling_update_kernel, dim3((unsigned)u.count), dim3(64), 0, st, u);
    profile_after(st);
}

}  // namespace ssg
