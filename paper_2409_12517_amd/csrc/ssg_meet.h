// How the workgroups of one launch exchange a maximum each without a second launch, device and host side.
//
// Range and cast of a tensor need its range in between: as two launches the second waits for the first to drain (4.7 us from
// kernel to kernel) and reads the tensor again.  Here a workgroup keeps its share of the tensor in registers, leaves its maximum
// in a word of its own and looks at the words of the others until all are there.
//
// Nobody depends on another workgroup being on the chip: one that has looked `polls` times in vain forms the maxima that are
// missing from the tensor itself and leaves them for the others, so every workgroup ends whatever the rest do -- when two
// such launches share the chip, when other work holds the compute units.  Those that wait share this work, so it comes to about
// another read of the tensor by all of them together.
//
// Two places for the words:
//   MeetRing   rows of words that all launches of a translation unit share, for launches that leave their source as it is.  A word belongs
//     to a launch by its ticket, a number that no other launch of the process has: what an earlier launch left is told from this
//     launch's by it, and nothing is cleared.  Tickets are dealt where a call is enqueued, so two launches whose tickets are
//     kMeetRows apart can be under way at once, however few there are, and write over each other's words: that costs them the wait and
//     another read of the tensor, no more, since the source still holds what the word held.
//   MeetOwned  words that nothing else writes while the launch runs, for launches that overwrite their shares.  They are
//     part of memory whose calls the caller orders, zeroed before the launch, and tagged by a number that says which call wrote them.
//
// Where a workgroup overwrites its share once it has all the maxima: its own word is where the others see it before it looks for
// theirs, and stays; one that forms a missing maximum looks for the word again after its last read of the share.  What it formed counts only
// if the word is not there then: then nothing of the share was written yet.  (With words that another launch may write over
// this does not hold: the word may be missing because of that.)
//
// A graph launches the same ticket every time, so calls under capture take the launches without an exchange.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

namespace ssg {

constexpr int kMeetRows = 64;                               // launches enqueued in a row before two share a row of words
constexpr int kMeetBlocks = 256;                            // workgroups that exchange a maximum, each maybe two
// Looks before a workgroup forms what is missing, about a fifth of a microsecond each.  Alone no launch needs 20; where others hold the chip a
// waiting workgroup holds a compute unit that the missing ones may need, but of two such launches at once one is done in less than
// this wait.  Q of 4096 x 11008 with the transposed copy, on one stream, two and four at once, with 32 looks, 200 and 600: 35.6 us a call,
// 47.4 and 56.9; 35.5, 33.9 and 62.9; 35.5, 33.9 and 84.6 (the separate launches 49.9, 43.0 and 47.6).
constexpr int kMeetPolls = 200;
// how often a caller may have them look (< 0: the usual number)
inline int meet_polls(int asked) { return asked >= 0 && asked < kMeetPolls ? asked : kMeetPolls; }

// the words of a translation unit's launches
static __device__ uint64_t g_meet[kMeetRows][2 * kMeetBlocks][2];

// (64-bit accesses are whole; a word is a pair of them, each with half of the ticket and the maximum, which have to agree)
struct MeetRing {
    static constexpr bool kOverwritten = false;
    uint64_t ticket;
    int polls;
    __device__ __forceinline__ void leave(int word, uint32_t v) const {
        uint64_t *w = g_meet[ticket % kMeetRows][word];
        __hip_atomic_store(w, (ticket << 32) | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(w + 1, (ticket & ~(uint64_t)0xffffffffu) | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __device__ __forceinline__ bool look(int word, uint32_t &v) const {
        uint64_t *w = g_meet[ticket % kMeetRows][word];
        const uint64_t a = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint64_t b = __hip_atomic_load(w + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        v = (uint32_t)a;
        return a == ((ticket << 32) | v) && b == ((ticket & ~(uint64_t)0xffffffffu) | v);
    }
};

// 15 words in the upper 120 bytes of each 128-byte line from `base` on, 2 * kMeetBlocks of them in two runs `second` lines apart.
struct MeetOwned {
    static constexpr bool kOverwritten = true;
    uint32_t *base;
    int second;
    uint32_t tag;                                            // not zero
    int polls;
    __device__ __forceinline__ uint64_t *at(int word) const {
        const int run = word / kMeetBlocks, i = word % kMeetBlocks;
        return reinterpret_cast<uint64_t *>(base + (run * second + i / 15) * 32) + 1 + i % 15;
    }
    __device__ __forceinline__ void leave(int word, uint32_t v) const {
        // (with the old value returned: the word is in its place before anything after it is stored)
        const uint64_t old = __hip_atomic_exchange(at(word), (uint64_t)tag << 32 | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("; %0" :: "v"(old) : "memory");
    }
    __device__ __forceinline__ bool look(int word, uint32_t &v) const {
        const uint64_t a = __hip_atomic_load(at(word), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        v = (uint32_t)a;
        return (uint32_t)(a >> 32) == tag;
    }
};
constexpr int kMeetOwnedLines = (kMeetBlocks + 14) / 15;    // of a run

// The maximum over words first .. first + count - 1 (count <= kMeetBlocks <= the workgroup's threads), for all threads.
// share_max(k): this thread's part of the k-th one's maximum, formed from the tensor.  `salt`: a number that differs between
// the workgroups that wait: each forms another one of what is missing, leaves it and looks at all again, so that they share the work.
// lds: kMeetBlocks + 8 words.  Called by all threads of the workgroup.
template <int THREADS, class Place, class ShareMax>
__device__ __forceinline__ uint32_t meet_max(const Place &m, int first, int count, unsigned salt, uint32_t *lds, ShareMax &&share_max) {
    static_assert(THREADS >= kMeetBlocks && THREADS <= 512, "a thread looks at one word; a word of lds for each wave's maximum");
    const int t = threadIdx.x;
    constexpr uint32_t kMissing = 0xffffffffu;               // no maximum of magnitudes: above every number and infinity
    uint32_t v = 0u;
    bool have = t >= count;
    for (int n = 0; n < m.polls && !have; ++n) {
        have = m.look(first + t, v);
        if (!have) __builtin_amdgcn_s_sleep(2);
    }
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
    for (;;) {                                               // (at most `count` times: each adds one)
        const uint32_t all = over_workgroup(have ? v : kMissing);
        if (all != kMissing) return all;
        // the (salt % missing)-th of those that are missing
        const unsigned long long gone = __ballot(!have);
        if ((t & 63) == 0 && t < kMeetBlocks) lds[t >> 6] = (uint32_t)__popcll(gone);
        __syncthreads();
        unsigned before = 0, missing = 0;
#pragma unroll
        for (int w = 0; w < kMeetBlocks / 64; ++w) {
            before += w < t >> 6 ? lds[w] : 0u;
            missing += lds[w];
        }
        if (!have && before + (unsigned)__popcll(gone & ((1ull << (t & 63)) - 1)) == salt % missing) lds[kMeetBlocks / 64] = (uint32_t)t;
        __syncthreads();
        const int k = (int)lds[kMeetBlocks / 64];
        uint32_t one = over_workgroup(share_max(k));
        if (Place::kOverwritten) {                           // by now it may have come, and its share with it
            uint32_t late = kMissing;
            if (t == 0 && !m.look(first + k, late)) late = kMissing;
            late = over_workgroup(t == 0 ? late : 0u);
            if (late != kMissing) one = late;
            else if (t == 0) m.leave(first + k, one);
        } else if (t == 0) {
            m.leave(first + k, one);
        }
        if (t == k) { v = one; have = true; }
        if (!have) have = m.look(first + t, v);
    }
}

// Host: whether a launch on `st` would be recorded and could be replayed.
inline bool launch_recorded(hipStream_t st) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &status) != hipSuccess) {
        (void)hipGetLastError();                             // (the null stream while another one is captured)
        return true;
    }
    return status != hipStreamCaptureStatusNone;
}
// A ticket for a launch on `st`, or false where the launch could be replayed.
inline bool meet_ticket(hipStream_t st, MeetRing *m) {
    static std::atomic<uint64_t> next{1};
    if (launch_recorded(st)) return false;
    m->ticket = next.fetch_add(1, std::memory_order_relaxed);
    m->polls = kMeetPolls;
    return true;
}

}  // namespace ssg
