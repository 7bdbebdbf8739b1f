// Range words and the history of delayed scaling (Section 2), device side: shared by the elementwise kernels and the
// grouped GEMM launch that enters a backward call's ranges.
#pragma once
#include "ssg_device.h"
#include "ssg_internal.h"

namespace ssg {

// the largest of words 4t .. 4t+3 of `count` packed range words (the array itself is longer)
__device__ __forceinline__ uint32_t range_word_max(const uint32_t *words, int count, int t) {
    if (4 * t >= count) return 0u;
    const uint4 q = *reinterpret_cast<const uint4 *>(words + 4 * t);
    uint32_t m = q.x;
    if (4 * t + 1 < count) m = m > q.y ? m : q.y;
    if (4 * t + 2 < count) m = m > q.z ? m : q.z;
    if (4 * t + 3 < count) m = m > q.w ? m : q.w;
    return m;
}

// One wave per tensor: the range of the call just made (maximum over the packed words of the range pass, or over its
// slots, which are cleared for the next call) replaces the oldest history entry; the next call's scale is fmax over the
// largest entry (Section 2, delayed scaling).
__device__ __forceinline__ void scaling_update_wave(const ScalingUpdate &u, const int k, const int lane) {
    uint32_t *slots = u.slots[k];
    uint32_t seen = 0u;
    if (u.range_count[k]) {
        for (int q = 0; q < 4; ++q) {
            const uint32_t w = range_word_max(slots, u.range_count[k], q * 64 + lane);
            seen = seen > w ? seen : w;
        }
    } else {
        seen = slots[lane * kAmaxSlotStride];
        slots[lane * kAmaxSlotStride] = 0u;
    }
    seen = wave_max_u32(seen);
    uint32_t *w = u.state + (size_t)u.tensor[k] * kScalingStride;
    const uint32_t pos = w[1] % kScalingHistory;
    uint32_t h = lane < kScalingHistory ? w[8 + lane] : 0u;
    if (lane == (int)pos) h = seen;
    const float largest = __uint_as_float(wave_max_u32(h));
    const float fmax = u.fmt[k] == kE4M3 ? Fp8Traits<kE4M3>::fmax : Fp8Traits<kE5M2>::fmax;
    if (lane == 0) {
        w[8 + pos] = seen;
        w[1] = (pos + 1) % kScalingHistory;
        w[2] = seen;
        w[0] = __float_as_uint(scale_from_amax(largest, fmax, u.pow2));
    }
}

}  // namespace ssg
