// Step 4 for one token in one launch: the first workgroups are the activation stage (a wave per row) and publish every activation
// as a stamped word, the last ones are the down projection (a column slice each) and wait for the words of their slots.
//
// The sums are those of k_ffn_up and k_ffn_down1. What it saves is a launch: from the host a call was as slow as two launches
// could be submitted, and behind one another they have a gap and a round trip for the counts.  us a call, two launches -> one,
// every call from the host / in a graph: fp16 d = 256, 321 rows 7.60 -> 5.14 / 5.72 -> 5.27; d = 1024, 117 rows 7.61 -> 5.24 /
// 5.56 -> 5.43; d = 2048, gated, 85 rows 7.52 -> 5.29 / 5.83 -> 5.46; fp32 d = 256, 79 rows 7.61 -> 4.86 / 5.97 -> 5.04; d =
// 1024, 117 rows 7.72 -> 5.33 / 6.36 -> 5.47.
// Workgroups of the activation stage leave four of their eight waves idle: with a row for each wave, half as many workgroups, it
// was mostly slower (graph, fp16 d = 512, 312 rows 5.56 -> 5.91, d = 2048, 85 rows gated 5.55 -> 5.86; fp32 d = 256, 79 rows 5.19
// -> 4.85). Eight copies of a word instead of four are no faster.
// A word waits for workgroups with smaller numbers only, and at most `polls` reads: then the wave computes the activation itself.
// The stamp is a number of the layer that is counted on by the launch itself once nobody reads it any more: the down workgroups
// count themselves in behind their read of it, the last one to do so sets the next number when it has seen all activations.
#pragma once

#include "lif_ffn.h"
#include "lif_ffn_down1.h"
#include "lif_words.h"

namespace lif {

constexpr int kOneWaves = 8, kOneUpWaves = 4;        // waves of a workgroup; those of the activation stage that have rows
constexpr int kOneReps = 4;                          // copies of every word
constexpr int kOneSlices = 64, kOneWords = 65536;    // column slices, and words read by all of them, up to which this form is taken
constexpr int kOneRows = kDown1FewRows;              // ... and rows: one pass of 8 waves
constexpr int kOneCapacity = 16384;                  // (there is a word for every slot)
constexpr int kOneWaits = 1 << 20;                   // failed reads of a thread before a launch whose waits ran out is given up:
                                                     // about a second
__host__ __device__ __forceinline__ size_t one_pitch(int capacity) { return (size_t)words_pitch(capacity); }
// Looks at the slots first, first + stride, ... below n until each is there, or for `waits` failed looks in all; returns whether
// all are.
template <typename There>
__host__ __device__ __forceinline__ bool await_slots(int first, int n, int stride, int waits, There there) {
    for (int s = first; s < n; s += stride)
        while (!there(s))
            if (--waits <= 0) return false;
    return true;
}
struct OneState {
    unsigned number, counted;                        // of the last launch; down workgroups of this one so far
};

// n_up workgroups of the activation role, then `slices` of the down projection; block = 512.
template <typename T, int NI, bool GLU, bool SKIP>
__global__ __launch_bounds__(kOneWaves * 64, 2) void k_ffn_one(const T* __restrict__ matrix, const float* __restrict__ bias,
                                                               const T* __restrict__ x, T* __restrict__ y, int d, int capacity,
                                                               size_t row_elems, int spec, int n_up, int slices,
                                                               unsigned long long* __restrict__ words, OneState* __restrict__ one,
                                                               int polls, const int32_t* __restrict__ pointers,
                                                               const float* __restrict__ gact, int gact_n, DevState* __restrict__ st) {
    using V = typename Vec<T>::type;
    __shared__ int last, lost;
    const int tid = threadIdx.x, lane = tid & 63, block = blockIdx.x;
    const size_t pitch = one_pitch(capacity);
    const unsigned before = one->number, now = before == ~0u ? 1u : before + 1u;
    if (block < n_up) {
        if (tid >= kOneUpWaves * 64) return;
        ffn_up_role<T, NI, GLU, true, kOneUpWaves>(matrix, bias, x, (float*)nullptr, d, 1, capacity, row_elems, spec, block, n_up, pointers,
                                                 gact, gact_n, st, [&](int s, float act) {
            if (lane < kOneReps) word_store(words + lane * pitch + s, now, __builtin_bit_cast(unsigned, act));
        });
        return;
    }
    const int slice = block - n_up, down_off = (GLU ? 2 : 1) * d;
    asm volatile("" ::"s"(now) : "memory");
    if (tid == 0) lost = 0;
    __syncthreads();                                 // (every wave has read the number)
    if (tid == 0)
        last = st->cur.error == 0 && (int)atomicInc(&one->counted, (unsigned)slices - 1u) == slices - 1;
    const unsigned long long* mine = words + (slice & (kOneReps - 1)) * pitch;
    ffn_down1_role<T, SKIP, kOneWaves, false, false>(matrix, (const float*)nullptr, FusedRows{}, y, (float*)nullptr, (unsigned*)nullptr,
                                              d, capacity, row_elems, down_off, 0, slices, pointers, gact, gact_n, st, slice, 0, 1,
                                              [&](int s0, int stride, int count, float (&v)[kDown1Per]) {
        unsigned p[kDown1Per];
        const bool ok = poll_words<kDown1Per>(mine + s0, stride, count, now, polls, p);
#pragma unroll
        for (int q = 0; q < kDown1Per; ++q) v[q] = __builtin_bit_cast(float, p[q]);
        if (__builtin_expect(__any(!ok), 0)) {       // a wait ran out: in the order of the activation role
            lost = 1;
            const int nvec = d / Vec<T>::N;
#pragma unroll 1
            for (int q = 0; q < kDown1Per; ++q)
                for (unsigned long long rows = __ballot(q < count); rows; rows &= rows - 1) {
                    const int at = __ffsll((long long)rows) - 1, s = __builtin_amdgcn_readlane(s0, at) + q * stride;
                    const V* row = reinterpret_cast<const V*>(matrix + (size_t)s * row_elems);
                    const V* xv = reinterpret_cast<const V*>(x);
                    float du = 0.f, dg = 0.f;
#pragma unroll 1
                    for (int idx = lane; idx < nvec; idx += 64) {
                        du = dot_acc(row[(GLU ? nvec : 0) + idx], xv[idx], du);
                        if (GLU) dg = dot_acc(row[idx], xv[idx], dg);
                    }
                    du = wave_sum(du);
                    float act;
                    if (GLU) act = fmaxf(wave_sum(dg) + bias[s], 0.f) * du;
                    else if (gact) act = du;
                    else act = fmaxf(du + bias[s], 0.f);
#pragma unroll
                    for (int k = 0; k < kDown1Per; ++k) v[k] = (k == q && lane == at) ? act : v[k];
                }
        }
    });
    __syncthreads();
    if (!last) return;                               // uniform
    // (the activation role must have read the number before it changes; every wave of it that has rows has published a word)
    if (__builtin_expect(lost, 0)) {
        const bool there = await_slots(tid, st->cur.num_used, kOneWaves * 64, kOneWaits, [&](int s) {
            const bool ok = (unsigned)(word_load(mine + s) >> 32) == now;
            if (!ok) __builtin_amdgcn_s_sleep(8);
            return ok;
        });
        if (!there) st->cur.error = 4;               // LIF_HIP_ERROR
        __syncthreads();
    }
    if (tid == 0) one->number = now;
}

}  // namespace lif
