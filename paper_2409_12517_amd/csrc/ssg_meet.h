// How the workgroups of one launch exchange a maximum each without a second launch, device and host side.
//
// Range and cast of a tensor need its range in between: as two launches the second waits for the first to drain (4.7 us from
// kernel to kernel) and reads the tensor again.  Here a workgroup keeps its share of the tensor in registers, leaves its maximum
// in a word of its own and looks at the words of the others until all are there.
//
// Nobody depends on another workgroup being on the chip: one that has looked `polls` times in vain forms the maxima that are
// missing from the tensor itself (and leaves them for the others), so every workgroup ends whatever the rest do -- when two
// such launches share the chip, when other work holds the compute units, when the words are overwritten.
//
// A word belongs to a launch by its ticket, a number that no other launch of the process has: stale words, and those of a
// launch that happens to use the same row, are told from this launch's by it, and nothing is cleared.  (64-bit accesses are
// whole; a word is a pair of them, each with half of the ticket and the maximum, which have to agree.)  A graph launches the same ticket
// every time, so calls under capture take the launches without an exchange.
//
// A workgroup may write over its share of the tensor once it has all the maxima: its own word is where the others see it before
// it looks for theirs, and one that forms a missing maximum looks for the word again after its last read of the share.  What it formed counts only if
// the word was not there then, and so nothing of the share was written yet.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

namespace ssg {

constexpr int kMeetRows = 64;                               // launches under way at once before two share a row of words
constexpr int kMeetBlocks = 256;                            // workgroups that exchange a maximum, each maybe two
constexpr int kMeetPolls = 400;                             // each takes about a microsecond

// what one launch needs to know
struct Meeting {
    uint64_t ticket;
    int polls;
};

// the words of a translation unit's launches
static __device__ uint64_t g_meet[kMeetRows][2 * kMeetBlocks][2];

__device__ __forceinline__ void meet_leave(const Meeting &m, int word, uint32_t v) {
    uint64_t *w = g_meet[m.ticket % kMeetRows][word];
    __hip_atomic_store(w, (m.ticket << 32) | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(w + 1, (m.ticket & ~(uint64_t)0xffffffffu) | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}
__device__ __forceinline__ bool meet_look(const Meeting &m, int word, uint32_t &v) {
    uint64_t *w = g_meet[m.ticket % kMeetRows][word];
    const uint64_t a = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t b = __hip_atomic_load(w + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    v = (uint32_t)a;
    return a == ((m.ticket << 32) | v) && b == ((m.ticket & ~(uint64_t)0xffffffffu) | v);
}

// The maximum over words first .. first + count - 1 (count <= kMeetBlocks <= the workgroup's threads), for all threads.  `own`:
// this workgroup's word among them; share_max(k): this thread's part of the k-th one's maximum, formed from the tensor.
// lds: kMeetBlocks + 8 words.  Called by all threads of the workgroup.
template <int THREADS, class ShareMax>
__device__ __forceinline__ uint32_t meet_max(const Meeting &m, int first, int count, int own, uint32_t *lds, ShareMax &&share_max) {
    const int t = threadIdx.x;
    constexpr uint32_t kMissing = 0xffffffffu;               // no maximum of magnitudes: above every number and infinity
    uint32_t v = 0u;
    bool have = t >= count;
    for (int n = 0; n < m.polls && !have; ++n) {
        have = meet_look(m, first + t, v);
        if (!have) __builtin_amdgcn_s_sleep(2);
    }
    if (!have) v = kMissing;
    auto over_workgroup = [&](uint32_t x) {
        x = wave_max_u32(x);
        __syncthreads();                                     // (whoever read lds before is done)
        if ((t & 63) == 0) lds[kMeetBlocks + (t >> 6)] = x;
        __syncthreads();
        uint32_t r = 0u;
#pragma unroll
        for (int w = 0; w < THREADS / 64; ++w) r = r > lds[kMeetBlocks + w] ? r : lds[kMeetBlocks + w];
        return r;
    };
    uint32_t all = over_workgroup(v);
    if (all != kMissing) return all;
    // some did not come in time: form theirs, beginning after this workgroup's own, so that several that wait share the work
    if (t < count) lds[t] = v;
    all = over_workgroup(v == kMissing ? 0u : v);
    for (int n = 1; n <= count; ++n) {
        const int k = (own + n) % count;
        if (lds[k] != kMissing) continue;
        auto look_again = [&]() {                            // by now it may have come
            uint32_t x = kMissing;
            if (t == 0 && !meet_look(m, first + k, x)) x = kMissing;
            return over_workgroup(t == 0 ? x : 0u);
        };
        uint32_t late = look_again();
        if (late == kMissing) {
            const uint32_t formed = over_workgroup(share_max(k));
            late = look_again();
            if (late == kMissing) {
                late = formed;
                if (t == 0) meet_leave(m, first + k, late);
            }
        }
        all = all > late ? all : late;
    }
    return all;
}

// Host: a ticket for a launch on `st`, or false where the launch could be replayed.
inline bool meet_ticket(hipStream_t st, Meeting *m) {
    static std::atomic<uint64_t> next{1};
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &status) != hipSuccess) {
        (void)hipGetLastError();                             // (the null stream while another one is captured)
        return false;
    }
    if (status != hipStreamCaptureStatusNone) return false;
    m->ticket = next.fetch_add(1, std::memory_order_relaxed);
    m->polls = kMeetPolls;
    return true;
}

}  // namespace ssg
