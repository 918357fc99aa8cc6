// Values handed over between the workgroups of a launch: 64-bit words of 32 bits of payload and a stamp that tells this launch's
// from older ones, written by relaxed device-scope atomic stores and polled with relaxed device-scope atomic loads, so no fence
// (a device-scope release writes back the L2: 6 us) and no clearing is needed.
#pragma once

#include "lif_common.h"

namespace lif {

constexpr int kWordReps = 8;         // copies of every word: hundreds of workgroups polling the same lines would queue up
// words of one copy, padded so that the copies do not fall on the same memory channels
__host__ __device__ __forceinline__ int words_pitch(int n) { return (n + 31) / 32 * 32 + 32; }

__device__ __forceinline__ unsigned long long word_load(const unsigned long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void word_store(unsigned long long* p, unsigned stamp, unsigned payload) {
    __hip_atomic_store(p, ((unsigned long long)stamp << 32) | payload, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Reads N words p[i * step] (i < n) of this stamp by the whole wave: all are requested before the first is looked at, and
// again as a whole until every lane has its words or `polls` more reads have failed (read again one after the other, a
// lane's second word cost a round trip of its own).  Returns whether all words of this lane have arrived.
template <int N>
__device__ __forceinline__ bool poll_words(const unsigned long long* p, int step, int n, unsigned stamp, int polls,
                                           unsigned (&out)[N]) {
    bool all;
    for (int tries = 0;; ++tries) {
        unsigned long long w[N];
#pragma unroll
        for (int i = 0; i < N; ++i) w[i] = (i < n) ? word_load(p + (size_t)i * step) : 0ull;
        all = true;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            all = all && (i >= n || (unsigned)(w[i] >> 32) == stamp);
            out[i] = (unsigned)w[i];
        }
        if (!__any(!all) || tries >= polls) break;
    }
    return all;
}

}  // namespace lif
