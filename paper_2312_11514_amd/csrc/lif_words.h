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
// Reads N words p[i * step] (i < n) of this stamp by the whole wave: all are requested before the first is looked at, the missing
// ones again until they have come or `polls` more reads have failed.  Returns whether all words of this lane have arrived.
// TOGETHER: again as a whole until every lane has its words (one after the other, a lane's second word cost a round trip of its
// own).  Else each word for itself: where words come over many microseconds, as those of the gate predictor do, reading all of
// them again and again stands in the way of the reads they are waiting for (one token, d = 2376, gate resident, 542 rows, 41
// added, 19 steps of a sequence 541.6 -> 537.5 us; Llama-2 shape, no rows added, 39.6 -> 39.2).
template <int N, bool TOGETHER = true>
__device__ __forceinline__ bool poll_words(const unsigned long long* p, int step, int n, unsigned stamp, int polls,
                                           unsigned (&out)[N]) {
    unsigned long long w[N];
    bool all;
    for (int tries = 0;; ++tries) {
#pragma unroll
        for (int i = 0; i < N; ++i) w[i] = (i < n) ? word_load(p + (size_t)i * step) : 0ull;
        if (!TOGETHER) break;
        all = true;
#pragma unroll
        for (int i = 0; i < N; ++i) all = all && (i >= n || (unsigned)(w[i] >> 32) == stamp);
        if (!__any(!all) || tries >= polls) break;
    }
    if (!TOGETHER) {
        all = true;
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (i < n) {
                for (int tries = 0; (unsigned)(w[i] >> 32) != stamp && tries < polls; ++tries) w[i] = word_load(p + (size_t)i * step);
                all = all && (unsigned)(w[i] >> 32) == stamp;
            }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) out[i] = (unsigned)w[i];
    return all;
}

}  // namespace lif
