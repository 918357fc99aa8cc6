// Pieces of the window update (Section 3.1) shared by k_window_plan and the fused step.
#pragma once

#include "lif_common.h"

namespace lif {

constexpr int kScanThreads = 1024;   // single-workgroup kernels: 16 waves; one 64-neuron word or one 64-slot block per lane
constexpr int kMaxSpan = 64;         // d_ffn <= 1024 * 64; capacity <= 1024 * 64
constexpr int kHoleLds = 4096;       // holes kept in LDS; longer lists spill to the global scratch list
constexpr int kRingRegs = 8;         // window masks a lane keeps in registers (larger k takes a second pass)

// Age of ring entry j when the next mask goes to entry `slot`: 1 = written by the previous step, k = the entry that is
// overwritten next.
__device__ __forceinline__ int ring_age(int j, int slot, int k) {
    const int a = slot - j;
    return a > 0 ? a : a + k;
}

// 64 mask bits starting at neuron 64 * w; the mask has nbytes bytes (a multiple of 8 bits, maybe not of 64)
__device__ __forceinline__ unsigned long long load_mask_word(const uint8_t* __restrict__ m, int w, int nbytes) {
    const int b0 = w * 8;
    if (b0 + 8 <= nbytes) return *reinterpret_cast<const unsigned long long*>(m + b0);
    unsigned long long v = 0;
    for (int i = 0; i < 8; ++i)
        if (b0 + i < nbytes) v |= (unsigned long long)m[b0 + i] << (8 * i);
    return v;
}

// Exclusive prefix sums of two counts per thread (each at most 64) in one pass over a workgroup of NW waves.
// Inside a wave both counts travel in one 32-bit value (a wave sums to at most 4096 per count); the totals of
// the waves are kept as two 32-bit halves of a 64-bit LDS word.  One barrier, two with GUARD (needed when
// wave_tot may still be read from an earlier scan that no barrier separates from this one).
template <int NW, bool GUARD>
__device__ __forceinline__ void block_exclusive_scan2(int va, int vb, unsigned long long* wave_tot, int* off_a,
                                                      int* off_b, int* tot_a, int* tot_b) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid >> 6;
    const int v = (vb << 16) | va;
    const int inc = wave_inclusive_scan(v, lane);
    if (GUARD) lds_barrier();
    if (lane == kWave - 1) wave_tot[w] = ((unsigned long long)(unsigned)(inc >> 16) << 32) | (unsigned)(inc & 0xffff);
    lds_barrier();
    unsigned long long before = 0, all = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const unsigned long long t = wave_tot[i];
        if (i < w) before += t;
        all += t;
    }
    const int ex = inc - v;                                  // exclusive inside the wave, both halves at once
    *off_a = (int)(unsigned)(before & 0xffffffffull) + (ex & 0xffff);
    *off_b = (int)(unsigned)(before >> 32) + (ex >> 16);
    *tot_a = (int)(unsigned)(all & 0xffffffffull);
    *tot_b = (int)(unsigned)(all >> 32);
}

}  // namespace lif
