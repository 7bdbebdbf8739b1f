// Adam step with the first moment stored in E4M3 and the second in E5M2 (Section 5).
//
// Two HBM-bound passes over a flat parameter tensor (one launch for up to 4 M elements, see adam_held_kernel):
//   pass 1  new moments from the stored codes and the gradient, their ranges (max|m|, max v)
//           into 64 slotted atomics each;
//   pass 2  the same moments again (bit-identical: same inputs, same operations), the
//           bias-corrected update of the fp32 master weights (optionally a bf16 copy), and the
//           moments re-encoded with the per-tensor scales fmax / range.
// A lane takes four neighbouring elements at a time, 16 bytes of an fp32 gradient or of the weights and 4 of each code, so that
// the lanes of a wave lie side by side in every access (with 16 elements per lane a wave's load of the gradient touched 64
// pieces of 64 bytes).  Gradient and weights are read and the weights written past the caches, which leaves these to the codes:
// 45 M weights, fp32 gradient, bf16 copy: 80 + 140 us before, 83 + 138 with the narrow accesses alone, 70 + 140 with the
// gradient's reads non-temporal, 52 + 134 with the weights' reads and writes too (codes non-temporal as well: 48 + 154, the
// update pass then finds none of them); 16 M 26 + 56 and 22 + 54.
// Every arithmetic step is a single rounded fp32 operation in a fixed order (the build disables
// contraction and uses correctly rounded division and square root), so codes, scales and
// weights can be compared bit for bit with a binary32 reference.
//
// State scalars are kept twice, by step parity, so that pass 2 can read the old scales and
// range slots while workgroup 0 writes the new ones and clears the slots of the next step, and the words between them in which the
// workgroups of the one launch exchange their ranges.
#include <type_traits>

#include "ssg_device.h"
#include "ssg_internal.h"
#include "ssg_meet.h"

namespace ssg {

struct AdamParams {
    const void *grad;
    float *w;
    uint16_t *w_bf16;
    uint8_t *m_q, *v_q;
    uint32_t *scalars;          // AdamScalars layout below, as words
    int64_t n;
    float b1, b2, omb1, omb2, c1, c2, lr, eps, wd;
    int parity;                 // step & 1: the set written by this step
    int pow2;
};

// word offsets in the scalar block
constexpr int kAdamScaleM = 0, kAdamScaleV = 1, kAdamAmaxM = 2, kAdamAmaxV = 3;   // + 8 * parity
constexpr int kAdamSlotsM = 64;                                                  // + parity * 2 * kAmaxSlotWords
static_assert(kAmaxSlotStride == 32 && kMeetOwnedLines <= kAmaxSlots, "the words of the exchange lie between the slots, a run beside each moment's");
constexpr int kAdamThreads = 256;

typedef float ssg_f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int ssg_u32x2 __attribute__((ext_vector_type(2)));
// A lane takes four neighbouring elements at a time: 16 bytes of an fp32 gradient or of the weights, 4 bytes of each code, so
// that the lanes of a wave lie side by side in every access.
template <bool GRAD_BF16> using Packed = std::conditional_t<GRAD_BF16, ssg_u32x2, ssg_f32x4>;
template <bool GRAD_BF16>
__device__ __forceinline__ Packed<GRAD_BF16> load_packed4(const void *grad, size_t i) {
    return __builtin_nontemporal_load(reinterpret_cast<const Packed<GRAD_BF16> *>(static_cast<const uint8_t *>(grad) + i * (GRAD_BF16 ? 2 : 4)));
}
template <bool GRAD_BF16>
__device__ __forceinline__ void unpack4(const Packed<GRAD_BF16> &q, float (&g)[4]) {
    if constexpr (GRAD_BF16) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            g[2 * k] = __uint_as_float(q[k] << 16);
            g[2 * k + 1] = __uint_as_float(q[k] & 0xffff0000u);
        }
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) g[k] = q[k];
    }
}
template <bool GRAD_BF16>
__device__ __forceinline__ void load_grad4(const void *grad, size_t i, float (&g)[4]) {
    unpack4<GRAD_BF16>(load_packed4<GRAD_BF16>(grad, i), g);
}
// four stored moments from a word of codes each, as fp32: decode(code) * (1 / scale)
__device__ __forceinline__ void decode_moments4(uint32_t mw, uint32_t vw, float inv_sm, float inv_sv, float (&m)[4], float (&v)[4]) {
    m[0] = __fmul_rn(__builtin_amdgcn_cvt_f32_fp8((int)mw, 0), inv_sm);
    m[1] = __fmul_rn(__builtin_amdgcn_cvt_f32_fp8((int)mw, 1), inv_sm);
    m[2] = __fmul_rn(__builtin_amdgcn_cvt_f32_fp8((int)mw, 2), inv_sm);
    m[3] = __fmul_rn(__builtin_amdgcn_cvt_f32_fp8((int)mw, 3), inv_sm);
    v[0] = __fmul_rn(__builtin_amdgcn_cvt_f32_bf8((int)vw, 0), inv_sv);
    v[1] = __fmul_rn(__builtin_amdgcn_cvt_f32_bf8((int)vw, 1), inv_sv);
    v[2] = __fmul_rn(__builtin_amdgcn_cvt_f32_bf8((int)vw, 2), inv_sv);
    v[3] = __fmul_rn(__builtin_amdgcn_cvt_f32_bf8((int)vw, 3), inv_sv);
}

// the step of four elements, stored: weights, their copy, the codes of the new moments m, v under the new scales
__device__ __forceinline__ void finish4(const AdamParams &p, size_t i, const float (&m)[4], const float (&v)[4], float sm, float sv, ssg_f32x4 w) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        // bias-corrected step, decoupled decay
        const float mhat = __fmul_rn(m[k], p.c1);
        const float vhat = __fmul_rn(v[k], p.c2);
        const float denom = __fadd_rn(sqrtf(vhat), p.eps);   // sqrtf, not __fsqrt_rn: only the former is correctly rounded here
        float upd = __fdiv_rn(mhat, denom);
        upd = __fadd_rn(upd, __fmul_rn(p.wd, w[k]));
        w[k] = __fsub_rn(w[k], __fmul_rn(p.lr, upd));
    }
    __builtin_nontemporal_store(w, reinterpret_cast<ssg_f32x4 *>(p.w + i));
    if (p.w_bf16) *reinterpret_cast<ssg_u32x2 *>(p.w_bf16 + i) = ssg_u32x2{pack_bf16x2(w[0], w[1]), pack_bf16x2(w[2], w[3])};
    *reinterpret_cast<uint32_t *>(p.m_q + i) = satcast_pk4<kE4M3>(__fmul_rn(m[0], sm), __fmul_rn(m[1], sm), __fmul_rn(m[2], sm), __fmul_rn(m[3], sm));
    *reinterpret_cast<uint32_t *>(p.v_q + i) = satcast_pk4<kE5M2>(__fmul_rn(v[0], sv), __fmul_rn(v[1], sv), __fmul_rn(v[2], sv), __fmul_rn(v[3], sv));
}

// what one workgroup leaves behind for the call and for the next step: the scales and ranges, the other parity's slots and words cleared
// (they were last read by the previous step)
__device__ __forceinline__ void leave_scalars(const AdamParams &p, float sm, float sv, float amax_m, float amax_v) {
    uint32_t *cur = p.scalars + 8 * p.parity;
    if (threadIdx.x == 0) {
        cur[kAdamScaleM] = __float_as_uint(sm); cur[kAdamScaleV] = __float_as_uint(sv);
        cur[kAdamAmaxM] = __float_as_uint(amax_m); cur[kAdamAmaxV] = __float_as_uint(amax_v);
    }
    uint4 *next = reinterpret_cast<uint4 *>(p.scalars + kAdamSlotsM + (size_t)(p.parity ^ 1) * 2 * kAmaxSlotWords);
    for (unsigned i = threadIdx.x; i < 2 * kAmaxSlotWords / 4; i += blockDim.x) next[i] = make_uint4(0u, 0u, 0u, 0u);
}

// exponential moving averages of the gradient and of its square
__device__ __forceinline__ void new_moments4(const AdamParams &p, const float (&g)[4], float (&m)[4], float (&v)[4]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        m[k] = __fadd_rn(__fmul_rn(p.b1, m[k]), __fmul_rn(p.omb1, g[k]));
        v[k] = __fadd_rn(__fmul_rn(p.b2, v[k]), __fmul_rn(__fmul_rn(p.omb2, g[k]), g[k]));
    }
}

// CHUNKS groups of four per lane and trip, a workgroup's 1024 elements apart
template <bool GRAD_BF16, int CHUNKS>
__global__ void __launch_bounds__(kAdamThreads) adam_range_kernel(AdamParams p) {
    const uint32_t *old = p.scalars + 8 * (p.parity ^ 1);
    const float inv_sm = __fdiv_rn(1.0f, __uint_as_float(old[kAdamScaleM])), inv_sv = __fdiv_rn(1.0f, __uint_as_float(old[kAdamScaleV]));
    uint32_t mmax = 0, vmax = 0;
    constexpr int kChunk = 4 * kAdamThreads;
    const size_t stride = (size_t)gridDim.x * kChunk * CHUNKS;
    for (size_t i = (size_t)blockIdx.x * kChunk * CHUNKS + 4 * threadIdx.x; i < (size_t)p.n; i += stride) {
        float g[CHUNKS][4];
        uint32_t mq[CHUNKS], vq[CHUNKS];
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
            const size_t j = i + (size_t)c * kChunk;
            const size_t at = j < (size_t)p.n ? j : i;           // (a group beyond the end: this lane's first one again)
            load_grad4<GRAD_BF16>(p.grad, at, g[c]);
            mq[c] = *reinterpret_cast<const uint32_t *>(p.m_q + at);
            vq[c] = *reinterpret_cast<const uint32_t *>(p.v_q + at);
        }
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
            float m[4], v[4];
            decode_moments4(mq[c], vq[c], inv_sm, inv_sv, m, v);
            new_moments4(p, g[c], m, v);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t a = abs_bits_ignore_nan(m[k]), b = abs_bits_ignore_nan(v[k]);
                mmax = mmax > a ? mmax : a;
                vmax = vmax > b ? vmax : b;
            }
        }
    }
    mmax = wave_max_u32(mmax);
    vmax = wave_max_u32(vmax);
    __shared__ uint32_t red[2 * (kAdamThreads / 64)];
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) { red[2 * w] = mmax; red[2 * w + 1] = vmax; }
    __syncthreads();
    if (threadIdx.x < 2) {
        uint32_t r = 0;
#pragma unroll
        for (int k = 0; k < kAdamThreads / 64; ++k) r = r > red[2 * k + threadIdx.x] ? r : red[2 * k + threadIdx.x];
        uint32_t *slots = p.scalars + kAdamSlotsM + (size_t)p.parity * 2 * kAmaxSlotWords + threadIdx.x * kAmaxSlotWords;
        if (r) atomicMax(slots + (blockIdx.x % kAmaxSlots) * kAmaxSlotStride, r);
    }
}

template <bool GRAD_BF16, int CHUNKS>
__global__ void __launch_bounds__(kAdamThreads) adam_update_kernel(AdamParams p) {
    const uint32_t *old = p.scalars + 8 * (p.parity ^ 1);
    const float inv_sm = __fdiv_rn(1.0f, __uint_as_float(old[kAdamScaleM])), inv_sv = __fdiv_rn(1.0f, __uint_as_float(old[kAdamScaleV]));
    // ranges of the new moments: maximum over the slots (one slot per lane, then across the wave)
    const uint32_t *slots_m = p.scalars + kAdamSlotsM + (size_t)p.parity * 2 * kAmaxSlotWords;
    const uint32_t *slots_v = slots_m + kAmaxSlotWords;
    const int lane = threadIdx.x & 63;
    const float amax_m = __uint_as_float(wave_max_u32(slots_m[lane * kAmaxSlotStride]));
    const float amax_v = __uint_as_float(wave_max_u32(slots_v[lane * kAmaxSlotStride]));
    const float sm = scale_from_amax(amax_m, Fp8Traits<kE4M3>::fmax, p.pow2);
    const float sv = scale_from_amax(amax_v, Fp8Traits<kE5M2>::fmax, p.pow2);
    if (blockIdx.x == 0) leave_scalars(p, sm, sv, amax_m, amax_v);
    constexpr int kChunk = 4 * kAdamThreads;
    const size_t stride = (size_t)gridDim.x * kChunk * CHUNKS;
    for (size_t i = (size_t)blockIdx.x * kChunk * CHUNKS + 4 * threadIdx.x; i < (size_t)p.n; i += stride) {
        float g[CHUNKS][4];
        uint32_t mq[CHUNKS], vq[CHUNKS];
        ssg_f32x4 w[CHUNKS];
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
            const size_t j = i + (size_t)c * kChunk;
            const size_t at = j < (size_t)p.n ? j : i;
            load_grad4<GRAD_BF16>(p.grad, at, g[c]);
            mq[c] = *reinterpret_cast<const uint32_t *>(p.m_q + at);
            vq[c] = *reinterpret_cast<const uint32_t *>(p.v_q + at);
            w[c] = __builtin_nontemporal_load(reinterpret_cast<const ssg_f32x4 *>(p.w + at));
        }
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
            const size_t j = i + (size_t)c * kChunk;
            if (c > 0 && j >= (size_t)p.n) break;
            float m[4], v[4];
            decode_moments4(mq[c], vq[c], inv_sm, inv_sv, m, v);
            new_moments4(p, g[c], m, v);
            finish4(p, j, m, v, sm, sv, w[c]);
        }
    }
}

// ---- both passes in one launch
// Up to 4 M elements: every workgroup keeps its share of the gradient and the codes in registers, eight groups of four elements to a
// lane at most, while they exchange the two ranges (ssg_meet.h), then updates it.  Bound by the latency of the launch and of the exchange; the
// two passes cost 4 to 6 us more from the first's drain to the second's first load: 1 M elements 15.9 us with them, 10.4 in one
// launch, 4 M 25.9 and 19.7.  With more groups per lane it gains nothing, one workgroup per compute unit streams no faster than two launches
// that fill it: 8 M 38.4 and 38.5 (bf16 gradient 35.1 and 36.1), 16 M bf16 62.4 and 61.0.
constexpr int kHeldThreads = 512, kHeldGroups = 4, kHeldBatches = 2;
template <bool GRAD_BF16>
__global__ void __launch_bounds__(kHeldThreads, 2) adam_held_kernel(AdamParams p, MeetOwned meeting) {
    constexpr int HELD = kHeldGroups * kHeldBatches, kChunk = 4 * kHeldThreads;
    __shared__ uint32_t words[kMeetBlocks + 8];
    const uint32_t *old = p.scalars + 8 * (p.parity ^ 1);
    const float inv_sm = __fdiv_rn(1.0f, __uint_as_float(old[kAdamScaleM])), inv_sv = __fdiv_rn(1.0f, __uint_as_float(old[kAdamScaleV]));
    const int own = (int)blockIdx.x, blocks = (int)gridDim.x, t = threadIdx.x;
    // the j-th group of this thread in workgroup k's share.  One beyond the end of the tensor counts for nothing and nothing is read
    // for it: whatever other group stood in for it would belong to a workgroup that may have stored its new codes by then
    auto group_at = [&](int k, int j) { return ((size_t)j * blocks + k) * kChunk + 4 * t; };
    auto share = [&](int k) { return (int)(((size_t)p.n + kChunk - 1) / kChunk - k + blocks - 1) / blocks; };      // groups of it
    struct Group { float g[4]; uint32_t mq, vq; };
    auto load = [&](size_t i) {
        Group x;
        load_grad4<GRAD_BF16>(p.grad, i, x.g);
        x.mq = __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(p.m_q + i));
        x.vq = __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(p.v_q + i));
        return x;
    };
    auto moments = [&](const Group &x, float (&m)[4], float (&v)[4]) {
        decode_moments4(x.mq, x.vq, inv_sm, inv_sv, m, v);
        new_moments4(p, x.g, m, v);
    };
    uint32_t mmax = 0, vmax = 0;
    auto see = [&](const Group &x, uint32_t &mm, uint32_t &vm) {
        float m[4], v[4];
        moments(x, m, v);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t a = abs_bits_ignore_nan(m[k]), b = abs_bits_ignore_nan(v[k]);
            mm = mm > a ? mm : a;
            vm = vm > b ? vm : b;
        }
    };
    const int mine = share(own);
    Packed<GRAD_BF16> held_g[HELD];
    uint32_t held_m[HELD], held_v[HELD];
#pragma unroll
    for (int j = 0; j < HELD; ++j) {
        const size_t i = group_at(own, j);
        if (j < mine && i < (size_t)p.n) {
            held_g[j] = load_packed4<GRAD_BF16>(p.grad, i);
            held_m[j] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(p.m_q + i));
            held_v[j] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(p.v_q + i));
        } else {
            held_g[j] = Packed<GRAD_BF16>{};
            held_m[j] = held_v[j] = 0u;
        }
    }
    auto group_of = [&](int j) {
        Group x;
        unpack4<GRAD_BF16>(held_g[j], x.g);
        x.mq = held_m[j]; x.vq = held_v[j];
        return x;
    };
    // (groups that are not there: zero gradient and moments, no new ones)
#pragma unroll
    for (int j = 0; j < HELD; ++j)
        if (j < mine) see(group_of(j), mmax, vmax);
    // the weights of the first batch come in while the ranges are exchanged
    ssg_f32x4 w[kHeldGroups];
    auto load_w = [&](int batch) {
#pragma unroll
        for (int c = 0; c < kHeldGroups; ++c) {
            const size_t i = group_at(own, kHeldGroups * batch + c);
            w[c] = i < (size_t)p.n ? __builtin_nontemporal_load(reinterpret_cast<const ssg_f32x4 *>(p.w + i)) : ssg_f32x4{};
        }
    };
    load_w(0);
    mmax = wave_max_u32(mmax);
    vmax = wave_max_u32(vmax);
    if ((t & 63) == 0) { words[t >> 6] = mmax; words[8 + (t >> 6)] = vmax; }
    __syncthreads();
    if (t < 2) {
        uint32_t r = 0;
#pragma unroll
        for (int k = 0; k < kHeldThreads / 64; ++k) r = r > words[8 * t + k] ? r : words[8 * t + k];
        meeting.leave(t * kMeetBlocks + own, r);
    }
    __syncthreads();
    auto share_max = [&](int k, bool second) {
        uint32_t mm = 0, vm = 0;
        for (int j = 0; j < share(k); ++j)
            if (group_at(k, j) < (size_t)p.n) see(load(group_at(k, j)), mm, vm);
        return second ? vm : mm;
    };
    const float amax_m = __uint_as_float(meet_max<kHeldThreads>(meeting, 0, blocks, (unsigned)own, words, [&](int k) { return share_max(k, false); }));
    const float amax_v = __uint_as_float(meet_max<kHeldThreads>(meeting, kMeetBlocks, blocks, (unsigned)own, words, [&](int k) { return share_max(k, true); }));
    const float sm = scale_from_amax(amax_m, Fp8Traits<kE4M3>::fmax, p.pow2);
    const float sv = scale_from_amax(amax_v, Fp8Traits<kE5M2>::fmax, p.pow2);
    if (own == 0) leave_scalars(p, sm, sv, amax_m, amax_v);
#pragma nounroll
    for (int batch = 0; kHeldGroups * batch < mine; ++batch) {
        ssg_f32x4 now[kHeldGroups];
#pragma unroll
        for (int c = 0; c < kHeldGroups; ++c) now[c] = w[c];
        if (kHeldGroups * (batch + 1) < mine) load_w(batch + 1);
#pragma unroll
        for (int c = 0; c < kHeldGroups; ++c) {
            const size_t i = group_at(own, kHeldGroups * batch + c);
            float m[4], v[4];
            moments(group_of(c), m, v);
            if (i < (size_t)p.n) finish4(p, i, m, v, sm, sv, now[c]);
        }
#pragma unroll
        for (int j = 0; j + kHeldGroups < HELD; ++j) {
            held_g[j] = held_g[j + kHeldGroups]; held_m[j] = held_m[j + kHeldGroups]; held_v[j] = held_v[j + kHeldGroups];
        }
    }
}

__global__ void adam_init_kernel(uint32_t *scalars, size_t scalar_words, uint4 *codes, size_t n16) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (size_t)gridDim.x * blockDim.x;
    for (size_t k = i; k < scalar_words; k += stride) {
        // scales 1.0 in both parity sets, everything else (ranges, slots) zero
        const bool is_scale = k == kAdamScaleM || k == kAdamScaleV || k == 8 + kAdamScaleM || k == 8 + kAdamScaleV;
        scalars[k] = is_scale ? 0x3f800000u : 0u;
    }
    for (size_t k = i; k < n16; k += stride) codes[k] = make_uint4(0u, 0u, 0u, 0u);
}

size_t adam_scalar_words() { return (size_t)kAdamSlotsM + 4 * kAmaxSlotWords; }

void launch_adam_init(uint32_t *scalars, uint8_t *codes, size_t code_bytes, hipStream_t st) {
    hipLaunchKernelGGL(adam_init_kernel, dim3(1024), dim3(256), 0, st, scalars, adam_scalar_words(),
                       reinterpret_cast<uint4 *>(codes), code_bytes / 16);
}

void launch_adam_step(const AdamArgs &a, hipStream_t st) {
    AdamParams p;
    p.grad = a.grad; p.w = a.w; p.w_bf16 = (uint16_t *)a.w_bf16; p.m_q = a.m_q; p.v_q = a.v_q; p.scalars = a.scalars;
    p.n = a.n; p.b1 = a.beta1; p.b2 = a.beta2; p.omb1 = a.one_minus_beta1; p.omb2 = a.one_minus_beta2;
    p.c1 = a.c1; p.c2 = a.c2; p.lr = a.lr; p.eps = a.eps; p.wd = a.weight_decay; p.parity = a.step & 1; p.pow2 = a.pow2;
    const double gbytes = a.grad_bf16 ? 2.0 : 4.0;       // algorithmic bytes per element: gradient + two codes; update: + w in/out, bf16 copy, codes out
    const double update_bytes = gbytes + 2.0 + 4.0 + 4.0 + (a.w_bf16 ? 2.0 : 0.0) + 2.0;
    constexpr size_t kHeldChunk = 4 * kHeldThreads;
    const size_t chunks = ((size_t)a.n + kHeldChunk - 1) / kHeldChunk;
    if (chunks <= (size_t)kMeetBlocks * kHeldGroups * kHeldBatches && !launch_recorded(st)) {
        const MeetOwned meeting{p.scalars + kAdamSlotsM + (size_t)p.parity * 2 * kAmaxSlotWords, kAmaxSlots, (uint32_t)a.step, meet_polls(a.polls)};
        const dim3 grid((unsigned)(chunks < kMeetBlocks ? chunks : kMeetBlocks));
        profile_before(33, st, update_bytes * (double)a.n);
        if (a.grad_bf16) hipLaunchKernelGGL(adam_held_kernel<true>, grid, dim3(kHeldThreads), 0, st, p, meeting);
        else hipLaunchKernelGGL(adam_held_kernel<false>, grid, dim3(kHeldThreads), 0, st, p, meeting);
        profile_after(st);
        return;
    }
    // 16 elements per lane in the range pass, one trip; 8 in the update pass, 2048 looping workgroups
    constexpr int kRangeChunks = 4, kUpdateChunks = 2;
    auto grid = [&](int chunks, size_t cap) {
        const size_t per = (size_t)4 * kAdamThreads * chunks, groups = ((size_t)a.n + per - 1) / per;
        return (unsigned)(groups < cap ? groups : cap);
    };
    const unsigned grid_r = grid(kRangeChunks, (size_t)1 << 20), grid_u = grid(kUpdateChunks, 2048);
    // timing records (when enabled): tag 32 = range pass, 33 = update pass
    profile_before(32, st, (gbytes + 2.0) * (double)a.n);
    if (a.grad_bf16) hipLaunchKernelGGL((adam_range_kernel<true, kRangeChunks>), dim3(grid_r), dim3(kAdamThreads), 0, st, p);
    else hipLaunchKernelGGL((adam_range_kernel<false, kRangeChunks>), dim3(grid_r), dim3(kAdamThreads), 0, st, p);
    profile_after(st);
    profile_before(33, st, update_bytes * (double)a.n);
    if (a.grad_bf16) hipLaunchKernelGGL((adam_update_kernel<true, kUpdateChunks>), dim3(grid_u), dim3(kAdamThreads), 0, st, p);
    else hipLaunchKernelGGL((adam_update_kernel<false, kUpdateChunks>), dim3(grid_u), dim3(kAdamThreads), 0, st, p);
    profile_after(st);
}

}  // namespace ssg
