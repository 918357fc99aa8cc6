// One step up to the down projection: of a single token in one launch (k_step1: lif_step and lif_step_tokens, batch 1), of a
// batch or a pass of several tokens in one launch behind the two of the predictor (k_step_batch).
//
// A step is a chain of small dependent stages in front of one long one, the host-link gather of the new bundles
// (Section 3.3 item 2).  As separate launches every short stage costs 4 to 6 us on gfx950: 1.6 us of launch, a memory
// round trip for the state, another one for what the previous kernel wrote.  Here the workgroups of one launch take
// different roles and hand over inside it:
//   workgroups [0, n_pred)        predictor: the first ceil(rank / 4) of them compute t = x A (one column per wave) and
//                                 publish it; each of the first ceil(F / 64) waits for t and decides the 64 mask bits of
//                                 its neurons (their weights are requested before the wait).  Gate predictor: 32 neurons
//                                 per workgroup, nothing to wait for.
//   workgroup n_pred              bookkeeping: waits for the masks, writes the window state, id lists and counts
//   the next n_load workgroups    loaders: wait for the masks, work out the added ids and the deletion plan (every
//                                 workgroup for itself: cheaper than waiting for one that does), move rows, gather
//                                 bundles from pinned host memory and compute the activations of the rows they write
//                                 (h_new, stamped with the step)
//   the rest                      activations of the rows that were already in use; waits for nothing
// A value handed over is a 64-bit word: 32 bits of payload and the number of the step as a stamp, written by a relaxed
// device-scope atomic store and polled with relaxed device-scope atomic loads, so no fence (a device-scope release
// writes back the L2: 6 us) and no clearing is needed.  Stamps are unique between two resets, which clear the words.
// A workgroup waits only for workgroups with smaller numbers, and never without bound: after `polls` failed polls it
// computes what it is missing itself, with the same arithmetic (polls = 0: never waits at all).
// What other workgroups may still read is not overwritten: the new counts are left in st->next and the slot owners and
// biases of the rows a loader writes in ptr_new / bias_new; the down projection, which runs after all of them, commits
// them.  A matrix row that the activation role reads while a loader overwrites it gives a value that is never used: the
// loader's stamped activation takes precedence for that slot.
// Every sum is formed in the order of the separate kernels, so the step is bit-identical to the four calls.
//
// What bounds it: the host link, at 56 GB/s (a copy of 256 MiB by the runtime reaches 57), behind a chain of about 8 us
// (x A 3, masks 3, window and first ids 2) and in front of the down projection.  Measured on gfx950, one decode token,
// with five launches -> with this kernel and the down projection, side by side in one run (runs on other machines differ by up
// to 4 %): fp32 d = 256, F = 1024: 23.4 -> 14.4 us; OPT-6.7B shape 65.3 -> 59.1; Falcon-7B shape 149.5 -> 139.4; Llama-2 shape
// gated, from a graph, 148.7 -> 136.6, with the gate resident 112.8 -> 109.1.  Eight tokens, Llama-2 shape gated: 276.8 -> 253.6.
#pragma once

#include "lif_ffn.h"
#include "lif_ffn_mfma.h"
#include "lif_predict.h"
#include "lif_window_bits.h"

namespace lif {

constexpr int kWordReps = 8;         // copies of every word: hundreds of workgroups polling the same lines would queue up
// words of one copy, padded so that the copies do not fall on the same memory channels
__host__ __device__ __forceinline__ int words_pitch(int n) { return (n + 31) / 32 * 32 + 32; }
constexpr int kListItems = 2048;     // work items listed at a time

struct StepArgs {
    // predictor
    const void* A;                   // [rank x d], or the gate projection [F x d]
    const void* B;
    const float* c;
    int rank;
    float theta;
    unsigned long long* t_words;     // [kWordReps][t_pitch] stamped halves of t (doubles)
    unsigned long long* m_words;     // [kWordReps][m_pitch] stamped 32-bit halves of the mask words
    int t_pitch, m_pitch;
    uint8_t* masks;
    uint8_t* step_mask;
    float* gact;                     // gate predictor: relu(gate_i . x + b_i) per neuron
    // window
    unsigned long long* ring;
    unsigned long long* cur_set;     // [2][ring_words]
    int ring_words, k, shrink;
    int32_t *added, *n_added, *removed, *n_removed;
    int32_t* hole_list;
    // cache
    void* matrix;
    const int32_t* pointers;
    const float* bias;
    HostStore host;
    const float* b;
    size_t row_elems;
    int F, d, capacity;
    const void* x;
    float* h;
    float* h_new;
    int32_t* stamp;                  // step in which h_new, ptr_new and bias_new of a slot were written
    int32_t* ptr_new;
    float* bias_new;
    int batch;                       // tokens of the step; with several of them:
    int keep, multi;                 // ring entries the step fills; 1: a pass of tokens, whose masks the commit writes there
    int x_pitch;                     // bytes between the tokens' x in LDS
    int stage_rows;                  // rows of activation vectors a loader workgroup has room for in LDS (1, 2)
    int spec;                        // the activation role requests its first rows ahead of the row count
    int n_pred, n_load;
    int polls;
    DevState* st;
};

__device__ __forceinline__ unsigned long long word_load(const unsigned long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void word_store(unsigned long long* p, unsigned stamp, unsigned payload) {
    __hip_atomic_store(p, ((unsigned long long)stamp << 32) | payload, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Reads N words p[i * step] (i < n) of this stamp: all are requested before the first is looked at, the missing ones
// again until they arrive or `polls` more reads have failed.  Returns whether all have arrived.
template <int N>
__device__ __forceinline__ bool poll_words(const unsigned long long* p, int step, int n, unsigned stamp, int polls,
                                           unsigned (&out)[N]) {
    unsigned long long w[N];
#pragma unroll
    for (int i = 0; i < N; ++i) w[i] = (i < n) ? word_load(p + (size_t)i * step) : 0ull;
    bool all = true;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if (i < n) {
            for (int tries = 0; (unsigned)(w[i] >> 32) != stamp && tries < polls; ++tries) w[i] = word_load(p + (size_t)i * step);
            all = all && (unsigned)(w[i] >> 32) == stamp;
        }
        out[i] = (unsigned)w[i];
    }
    return all;
}

// ---- predictor -------------------------------------------------------------------------------------------------

struct PredictLds {
    double t[2048];                  // t = x A
    double red[4][kMaskCols][8];
};

// x . row j of A (the whole wave; every lane returns the sum), in the order of k_predict_xa
template <typename T, int NI>
__device__ __forceinline__ double column_dot(const typename Vec<T>::type (&a)[NI], const typename Vec<T>::type (&xr)[NI]) {
    double acc = 0.0;
#pragma unroll
    for (int it = 0; it < NI; ++it) acc = dot_f64(a[it], xr[it], acc);
    return wave_sum(acc);
}
template <typename T, int NI>
__device__ __forceinline__ void load_vec(typename Vec<T>::type (&v)[NI], const T* p, int nvec, int lane) {
    using V = typename Vec<T>::type;
#pragma unroll
    for (int it = 0; it < NI; ++it) {
        const int idx = it * 64 + lane;
        v[it] = (idx < nvec) ? reinterpret_cast<const V*>(p)[idx] : V(0);
    }
}

// The same sum straight from memory, for the rare case that a wait ran out: few registers instead of loads in flight
template <typename T>
__device__ __forceinline__ double column_dot_slow(const T* col, const T* x, int nvec, int lane) {
    using V = typename Vec<T>::type;
    double acc = 0.0;
#pragma unroll 1
    for (int idx = lane; idx < nvec; idx += 64)
        acc = dot_f64(reinterpret_cast<const V*>(col)[idx], reinterpret_cast<const V*>(x)[idx], acc);
    return wave_sum(acc);
}
// t computed by this workgroup alone (a wait that ran out)
template <typename T>
__device__ __forceinline__ void own_t(const StepArgs& a, PredictLds& L) {
    const int lane = threadIdx.x & 63;
#pragma unroll 1
    for (int j = threadIdx.x >> 6; j < a.rank; j += 4) {
        const double v = column_dot_slow((const T*)a.A + (size_t)j * a.d, (const T*)a.x, a.d / Vec<T>::N, lane);
        if (lane == 0) L.t[j] = v;
    }
    __syncthreads();
}

// The 64 mask bits of a tile of neurons: as k_predict_mask for one token.  The weights and offsets are requested by
// the constructor, before t is there.
template <typename T>
struct MaskTile {
    using V = typename Vec<T>::type;
    static constexpr int VE = Vec<T>::N, LPB = 8 / VE;
    V bv[kMaskRows][LPB];
    double bd[kMaskRows][8];
    float cv[8];
    int n0;
    __device__ __forceinline__ void request(const StepArgs& a, int tile) {
        const int tid = threadIdx.x, cl = tid & (kMaskCols - 1), jg = tid >> 3;
        n0 = (tile * kMaskCols + cl) * 8;
        const T* B = (const T*)a.B;
#pragma unroll
        for (int u = 0; u < kMaskRows; ++u) {
            const int j = jg + u * kMaskJg;
#pragma unroll
            for (int q = 0; q < LPB; ++q)
                bv[u][q] = (n0 < a.F && j < a.rank) ? reinterpret_cast<const V*>(B + (size_t)j * a.F + n0)[q] : V(0);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) cv[e] = (a.c && tid < kMaskCols && n0 < a.F) ? a.c[n0 + e] : 0.f;
    }
    // widening takes longer than the multiply-adds (64 values per thread, quarter-rate conversions: 0.6 us), so it is done
    // while t is still on its way
    __device__ __forceinline__ void widen() {
#pragma unroll
        for (int u = 0; u < kMaskRows; ++u)
#pragma unroll
            for (int q = 0; q < LPB; ++q)
#pragma unroll
                for (int e = 0; e < VE; ++e) bd[u][q * VE + e] = (double)bv[u][q][e];
    }
    // mask byte of neurons n0 .. n0 + 7 in the threads tid < kMaskCols (0 past the last neuron); one barrier
    template <bool WIDE>
    __device__ __forceinline__ unsigned finish(const StepArgs& a, PredictLds& L) {
        const int tid = threadIdx.x, wave = tid >> 6, cl = tid & (kMaskCols - 1), jg = tid >> 3;
        const T* B = (const T*)a.B;
        double v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = 0.0;
#pragma unroll
        for (int u = 0; u < kMaskRows; ++u) {
            const double tj = L.t[min(jg + u * kMaskJg, a.rank - 1)];            // bd[u] is 0 past the end
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = __builtin_fma(tj, WIDE ? bd[u][e] : (double)bv[u][e / VE][e % VE], v[e]);
        }
        if (n0 < a.F) {
            for (int j = jg + kMaskRows * kMaskJg; j < a.rank; j += kMaskJg) {   // only when rank > 256
                const double tj = L.t[j];
                const V* bp = reinterpret_cast<const V*>(B + (size_t)j * a.F + n0);
#pragma unroll
                for (int q = 0; q < LPB; ++q) {
                    const V bw = bp[q];
#pragma unroll
                    for (int e = 0; e < VE; ++e) v[q * VE + e] = __builtin_fma(tj, (double)bw[e], v[q * VE + e]);
                }
            }
        }
        // rank groups of a wave sit 8 lanes apart: halving folds, lanes 8 apart first (a DPP rotation)
        int owner = 0;
        auto halve = [&](auto half_c, int m) {
            constexpr int half = decltype(half_c)::value;
            const bool up = (tid & m) != 0;
#pragma unroll
            for (int i = 0; i < half; ++i) {
                const double send = up ? v[i] : v[i + half], keep = up ? v[i + half] : v[i];
                v[i] = keep + (m == 8 ? dpp_from<0x128, 0xf>(send) : __shfl_xor(send, m, kWave));
            }
            owner = owner * 2 + (up ? 1 : 0);
        };
        halve(std::integral_constant<int, 4>{}, 8);
        halve(std::integral_constant<int, 2>{}, 16);
        halve(std::integral_constant<int, 1>{}, 32);
        L.red[wave][cl][owner] = v[0];
        __syncthreads();
        unsigned byte = 0;
        if (tid < kMaskCols && n0 < a.F) {
            const double th = (double)a.theta;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                double z = ((L.red[0][cl][e] + L.red[1][cl][e]) + L.red[2][cl][e]) + L.red[3][cl][e];
                z += (double)cv[e];
                if (z > th) byte |= 1u << e;
            }
        }
        return byte;
    }
};

template <typename T, int NI>
__device__ __forceinline__ void lowrank_role(const StepArgs& a, int block, PredictLds& L) {
    using V = typename Vec<T>::type;
    const int tid = threadIdx.x, lane = tid & 63, nvec = a.d / Vec<T>::N;
    const int j = block * 4 + __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool producer = j < a.rank;                // uniform over the wave
    const bool has_tile = block * kMaskCols * 8 < a.F;
    V col[NI], xr[NI];
    if (producer) {
        load_vec<T, NI>(xr, (const T*)a.x, nvec, lane);
        load_vec<T, NI>(col, (const T*)a.A + (size_t)j * a.d, nvec, lane);
    }
    MaskTile<T> tile;
    if (has_tile) tile.request(a, block);
    const int err = a.st->cur.error;
    const unsigned now = (unsigned)a.st->cur.step + 1u;
    if (err) return;
    if (producer) {
        const double v = column_dot<T, NI>(col, xr);
        const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
        if (lane < 2 * kWordReps)
            word_store(a.t_words + (size_t)(lane >> 1) * a.t_pitch + 2 * j + (lane & 1), now,
                       (lane & 1) ? (unsigned)(u >> 32) : (unsigned)u);
    }
    if (!has_tile) return;
    tile.widen();
    unsigned* t32 = reinterpret_cast<unsigned*>(L.t);
    const unsigned long long* src = a.t_words + (size_t)(block & (kWordReps - 1)) * a.t_pitch;
    bool ok = true;
    for (int i0 = tid; i0 < 2 * a.rank; i0 += 4 * 256) {
        unsigned p[4];
        const int n = min(4, (2 * a.rank - i0 + 255) >> 8);
        ok = poll_words<4>(src + i0, 256, n, now, a.polls, p) && ok;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i < n) t32[i0 + i * 256] = p[i];
    }
    if (__syncthreads_or(!ok)) own_t<T>(a, L);
    const unsigned byte = tile.template finish<true>(a, L);
    if (tid < 64) {
        unsigned w = byte << (8 * (tid & 3));        // lanes 0..3 and 4..7: the halves of the 64-bit mask word
        w |= __shfl_xor(w, 1, kWave);
        w |= __shfl_xor(w, 2, kWave);
        w = __shfl(w, (tid & 1) * 4, kWave);
        if (tid < 2 * kWordReps) word_store(a.m_words + (size_t)(tid >> 1) * a.m_pitch + 2 * block + (tid & 1), now, w);
        if (tid < kMaskCols && tile.n0 < a.F) {
            a.masks[tile.n0 >> 3] = (uint8_t)byte;
            a.step_mask[tile.n0 >> 3] = (uint8_t)byte;
        }
    }
}

// Gate predictor: relu(gate_i . x + b_i) and the mask bit of 8 neurons per wave, as k_predict_gate for one token.
template <typename T, int NI>
__device__ __forceinline__ unsigned gate_byte(const StepArgs& a, int grp, const typename Vec<T>::type (&xr)[NI]) {
    using V = typename Vec<T>::type;
    const int lane = threadIdx.x & 63, nvec = a.d / Vec<T>::N;
    const double th = (double)a.theta;
    unsigned bits = 0;
#pragma unroll 2
    for (int e = 0; e < 8; ++e) {
        const int i = grp * 8 + e;
        V g[NI];
        load_vec<T, NI>(g, (const T*)a.A + (size_t)i * a.d, nvec, lane);
        const double v = column_dot<T, NI>(g, xr) + (double)a.b[i];
        if (v > th) bits |= 1u << e;
        if (lane == 0) a.gact[i] = (float)(v > 0.0 ? v : 0.0);
    }
    return bits;
}
template <typename T, int NI>
__device__ __forceinline__ void gate_role(const StepArgs& a, int block, unsigned* lds) {
    using V = typename Vec<T>::type;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    V xr[NI];
    load_vec<T, NI>(xr, (const T*)a.x, a.d / Vec<T>::N, lane);
    const int err = a.st->cur.error;
    const unsigned now = (unsigned)a.st->cur.step + 1u;
    if (err) return;
    const int grp = block * 4 + wave;
    unsigned byte = 0;
    if (grp * 8 < a.F) {
        byte = gate_byte<T, NI>(a, grp, xr);
        if (lane == 0) {
            a.masks[grp] = (uint8_t)byte;
            a.step_mask[grp] = (uint8_t)byte;
        }
    }
    if (lane == 0) lds[wave] = byte << (8 * wave);
    __syncthreads();
    if (tid < kWordReps) word_store(a.m_words + (size_t)tid * a.m_pitch + block, now, lds[0] | lds[1] | lds[2] | lds[3]);
}

// pieces of 1 KiB that every vector served by this NI has in full (launch_step1_as)
constexpr int full_pieces(int ni) { return ni <= 1 ? 0 : ni <= 2 ? 1 : ni <= 4 ? 2 : ni <= 6 ? 4 : ni <= 8 ? 6 : ni <= 9 ? 8 : ni <= 12 ? 9 : 12; }

// ---- window, deletion plan, loaders ----------------------------------------------------------------------------

constexpr int kPtrLds = 4096;        // slot owners staged in LDS
constexpr int kNoDst = 0xffff;       // dead tail slot (a hole lies below n' <= 65535, so it is never slot 65535)
constexpr int kHoleFew = 2048;       // holes kept in LDS; longer lists go to the global scratch list
struct PlanLds {
    unsigned long long rem[1024], add[1024]; // removed and added neurons, one bit each
    union {
        PredictLds predict;                  // only when a wait ran out
        struct {
            uint16_t ids[kListItems], dst[kListItems];       // work items: new neuron, destination of the tail row (kNoDst)
            uint16_t hole[kHoleFew];
            uint16_t blk_h[1024], blk_f[1024];       // per 64-slot block: counts, then exclusive prefixes
        };
    };
    uint16_t ptr[kPtrLds];                   // (of the slots in use: neurons are numbers below 65536)
    unsigned long long wave_tot[4];
    int cnt_age[264];
    unsigned byte[4];
    unsigned long long flag_h[64], flag_f[64];       // per block: which slots are holes, fillers (plan_alone)
    int classified;                          // waves that have written their share of those
    int planned;                             // wave 1 has written dst
};

// All mask words computed by this workgroup alone (a wait that ran out): m[i] of the words this thread owns
template <typename T, bool GATE>
__device__ __forceinline__ void own_masks(const StepArgs& a, PlanLds& L, int wpt, unsigned long long (&m)[4]) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nwords = (a.F + 63) >> 6;
    if constexpr (!GATE) own_t<T>(a, L.predict);
#pragma unroll
    for (int i = 0; i < 4; ++i) m[i] = 0ull;
#pragma unroll 1
    for (int w = 0; w < nwords; ++w) {
        unsigned half[2];
        if constexpr (GATE) {
            for (int hf = 0; hf < 2; ++hf) {
                const int grp = w * 8 + hf * 4 + wave;
                unsigned byte = 0;
#pragma unroll 1
                for (int e = 0; e < 8 && grp * 8 < a.F; ++e) {
                    const int i = grp * 8 + e;
                    const double v = column_dot_slow((const T*)a.A + (size_t)i * a.d, (const T*)a.x, a.d / Vec<T>::N, lane);
                    if (v + (double)a.b[i] > (double)a.theta) byte |= 1u << e;
                }
                __syncthreads();
                if (lane == 0) L.byte[wave] = byte << (8 * wave);
                __syncthreads();
                half[hf] = L.byte[0] | L.byte[1] | L.byte[2] | L.byte[3];
            }
        } else {
            MaskTile<T> tile;
            tile.request(a, w);
            __syncthreads();
            const unsigned byte = tile.template finish<false>(a, L.predict);
            unsigned v = byte << (8 * (tid & 3));
            v |= __shfl_xor(v, 1, kWave);
            v |= __shfl_xor(v, 2, kWave);
            if (tid < kMaskCols && (tid & 3) == 0) L.byte[tid >> 2] = v;
            __syncthreads();
            half[0] = L.byte[0];
            half[1] = L.byte[1];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i < wpt && w == tid * wpt + i) m[i] = ((unsigned long long)half[1] << 32) | half[0];
    }
    __syncthreads();
}

// wg = 0: bookkeeping; wg >= 1: loader workgroup wg - 1.
// Work item q covers tail slot s = n' + q (see k_load).  Rows of more than 2 KiB per vector are handled in two units,
// the vectors the activation needs (gate | up) with the bookkeeping of the slot, and the down vector; shorter rows
// are one unit.  Within a loader workgroup
//   wave 0      loads: requests its part of the host bundle, moves its part of the live tail row in slot s to its hole,
//               writes the bundle part to slot s, and requests the next unit before it finishes the current one.  The L1
//               of a compute unit returns loads in order over all its waves, so a load of device memory behind host
//               reads takes as long as they do (2 to 5 us): the tail row is requested just behind the bundle (ahead of
//               it, it would hold back the host read), and the loaders are spread over compute units (four
//               loading waves per workgroup moved 35 GB/s where one moves 50).  The units of a round are dealt to the workgroups one place further each round, so that all
//               get as many activation parts as down parts (a counter drawn from by atomics balanced no better, and the
//               wait for its answer cost 1.5 us per unit; with all activation parts first, rows of 16 KiB loaded a
//               quarter slower, all reads falling on the same half of every row);
//   waves 1..3  make the deletion plan meanwhile (LDS only), then move the tail rows that nothing overwrites (more
//               neurons removed than added; with several tokens one wave does).
// Lane l holds the same 16-byte pieces of every vector as in the activation role and sums in the same order.
//
// Several tokens (MODE kDots, kMfma): the masks were written by the launch before this one and x lies in LDS.  Wave 0 puts the
// activation vectors of the rows it writes (new, moved) into LDS and posts them there; waves 1..3 compute the activations
// while its next bundle is on its way, kDots as in ffn_up_role with the tokens dealt to the waves, kMfma with the matrix
// instruction and the order of ffn_up_mfma_tile_staged (the vectors of both rows are rows of one operand; the parts of the k
// range are dealt to the waves).  One wave alone took 6 us per bundle of 24 KiB and 8 tokens, as long as the link.
enum StepMode { kOneToken = 0, kDots = 1, kMfma = 2 };

// LDS behind PlanLds: PostLds, x of the tokens, the activation vectors of `stage_rows` rows
struct Slot {                                                // a row that was written
    int s, id;
    float bias;
};
struct PostLds {
    int seq, done, arrived;                                  // posts so far; waves that have finished, delivered their sums
    int rows;                                                // of this post (0: the last one)
    Slot slot[2];
    float gate[2][8];                                        // resident gate activations, per token
    alignas(16) float sums[8][16][4];                        // kMfma: sums of parts 2 g and 2 g + 1, per token and vector
};
constexpr int kStepXOff = (int)((sizeof(PlanLds) + 15) / 16 * 16 + (sizeof(PostLds) + 15) / 16 * 16);
__host__ __device__ __forceinline__ int step_x_pitch(int d, int elem) { return d * elem + 16; }     // (16: the reads of 16 tokens
                                                                                                     //  fall on different banks)
template <typename T, int NI, bool GLU, bool GATE, int MODE>
__device__ __forceinline__ void cache_role(const StepArgs& a, int wg, PlanLds& L, PostLds* post, unsigned char* lds_x) {
    using V = typename Vec<T>::type;
    constexpr int VE = Vec<T>::N;
    constexpr bool PAIRED = NI > 2;
    constexpr int GA = PAIRED ? (GLU ? 2 : 1) : (GLU ? 3 : 2);   // vectors of a unit at most
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned long long lt = (1ull << lane) - 1ull;
    const int F = a.F, d = a.d, capacity = a.capacity, k = a.k;
    const int nwords = (F + 63) >> 6, wpt = (nwords + 255) >> 8;   // mask words per thread (1..4)
    DevState* st = a.st;

    // ---- everything that does not depend on this step's masks: slot owners, window, x ----
    auto stage_owners = [&]() {
        int id[kPtrLds / 256];
#pragma unroll
        for (int q = 0; q < kPtrLds / 256; ++q) id[q] = (q * 256 + tid < capacity) ? a.pointers[q * 256 + tid] : -1;
#pragma unroll
        for (int q = 0; q < kPtrLds / 256; ++q) L.ptr[q * 256 + tid] = (uint16_t)id[q];
    };
    stage_owners();
    const StepCounts cur = st->cur;
    if (cur.error) {
        if (wg == 0 && tid == 0) {
            *a.n_added = 0;
            *a.n_removed = 0;
            StepCounts nx = cur;
            nx.n_added = nx.n_removed = 0;
            st->next = nx;
        }
        return;
    }
    const unsigned stamp_now = (unsigned)cur.step + 1u;
    const int n = cur.num_used, slot_now = cur.ring_pos % k, oldest = min(cur.window_len, k - a.keep);      // largest age that stays in the window
    unsigned long long prev[4], keep[4], m[4], now[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) prev[i] = keep[i] = m[i] = 0ull;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int w = tid * wpt + i;
        if (i < wpt && w < nwords) {
            prev[i] = a.cur_set[(size_t)cur.set_par * a.ring_words + w];
            for (int j0 = 0; j0 < k; j0 += kRingRegs) {
                unsigned long long v[kRingRegs];
#pragma unroll
                for (int j = 0; j < kRingRegs; ++j)
                    v[j] = (j0 + j < k && ring_age(j0 + j, slot_now, k) <= oldest) ? a.ring[(size_t)(j0 + j) * a.ring_words + w] : 0ull;
#pragma unroll
                for (int j = 0; j < kRingRegs; ++j) keep[i] |= v[j];
            }
        }
    }
    const int lw = wg - 1;                                        // loader wave
    const bool loads = wg > 0 && wave == 0;
    const int nvec = d / VE;
    const size_t row_bytes = a.row_elems * sizeof(T);
    T* matrix = (T*)a.matrix;
    V hv[GA][NI], mv[GA][NI];                                    // the vectors of a unit: host bundle, tail row
    int k_eff = k, off_a = 0, off_r = 0, tot_a = 0, tot_r = 0, n2 = 0, items = 0;
    auto diff = [&]() {
        int pa = 0, pr = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            pa += __popcll(now[i] & ~prev[i]);
            pr += __popcll(prev[i] & ~now[i]);
        }
        block_exclusive_scan2<4, true>(pa, pr, L.wave_tot, &off_a, &off_r, &tot_a, &tot_r);
    };
    // the added neurons q of [c0, c0 + kListItems) (the words come back from LDS: in registers they would be live through
    // the load loop)
    auto fill_ids = [&](int c0) {
        int q = off_a - c0;
#pragma unroll 1
        for (int i = 0; i < wpt; ++i) {
            unsigned long long bits = L.add[tid * wpt + i];
            while (bits) {
                if ((unsigned)q < (unsigned)kListItems) L.ids[q] = (uint16_t)((tid * wpt + i) * 64 + __ffsll((long long)bits) - 1);
                bits &= bits - 1;
                ++q;
            }
        }
    };
    // Addresses are kept uniform over the wave (one base per vector, the lane's 16 bytes as offset): a 64-bit address per
    // lane and piece cost more registers than the data, and spilled registers queue up behind the host reads.
    const size_t vec_bytes = (size_t)d * sizeof(T);
    auto host_vec = [&](int nid, int v) -> const char* {          // vector v (gate | up | down) of the bundle of neuron nid
        const size_t off = (size_t)v * vec_bytes;
        if (a.host.down && off >= a.host.act_bytes) return a.host.down + (size_t)nid * vec_bytes + (off - a.host.act_bytes);
        return a.host.rows + (size_t)nid * (a.host.down ? a.host.act_bytes : row_bytes) + off;
    };
    auto row_vec = [&](int s, int v) -> char* { return reinterpret_cast<char*>(matrix) + (size_t)s * row_bytes + (size_t)v * vec_bytes; };
    auto lane_bytes = [&]() {                                    // (opaque: keeps address arithmetic where it is used)
        unsigned off = (unsigned)lane * 16u;
        asm volatile("" : "+v"(off));
        return off;
    };
    // (no branch around a load: a conditional load makes the compiler keep a second copy of its registers.  Lanes past the
    // end of the vector read its last 16 bytes and keep 0.)
    auto load_pieces = [&](V (&dst)[NI], const char* p) {
        const unsigned off = lane_bytes(), end = (unsigned)vec_bytes;
#pragma unroll
        for (int it = 0; it < NI; ++it) {
            if (it < full_pieces(NI)) {
                dst[it] = *reinterpret_cast<const V*>(p + (off + it * 1024u));
            } else {
                const V v = *reinterpret_cast<const V*>(p + min(off + it * 1024u, end - 16u));
                dst[it] = (off + it * 1024u < end) ? v : V(0);
            }
        }
    };
    auto store_pieces = [&](char* p, const V (&v)[NI]) {
        const unsigned off = lane_bytes();
#pragma unroll
        for (int it = 0; it < NI; ++it)
            if (it < full_pieces(NI) || off + it * 1024u < (unsigned)vec_bytes) *reinterpret_cast<V*>(p + (off + it * 1024u)) = v[it];
    };
    // (the second vector of a unit exists only in its activation part, a third one only in unsplit gated bundles)
    auto in_part = [&](int g, int part) { return part ? g == 0 : true; };
    auto request_host = [&](int nid, int part) {
#pragma unroll
        for (int g = 0; g < GA; ++g)
            if (in_part(g, part)) load_pieces(hv[g], host_vec(nid, part * GA + g));
    };
    auto request_row = [&](int s, int part) {
#pragma unroll
        for (int g = 0; g < GA; ++g)
            if (in_part(g, part)) load_pieces(mv[g], row_vec(s, part * GA + g));
    };
    auto store_row = [&](int s, int part, const V (&v)[GA][NI]) {
#pragma unroll
        for (int g = 0; g < GA; ++g)
            if (in_part(g, part)) store_pieces(row_vec(s, part * GA + g), v[g]);
    };
    const int nblk = (n + kWave - 1) >> 6;
    // slot owner of this lane in block b; blocks past the staged ones are read again
    auto owner = [&](int b) {
        const int s = b * kWave + lane;
        int id = L.ptr[min(s, kPtrLds - 1)];
        if (b >= kPtrLds / kWave) id = s < n ? a.pointers[s] : -1;
        return id;
    };
    auto flags_of = [&](int b, int id, bool& hole, bool& fill) {
        const int s = b * kWave + lane;
        const bool dead = (unsigned)id >= (unsigned)F || ((L.rem[id >> 6] >> (id & 63)) & 1ull);
        hole = s < n2 && dead;
        fill = s >= n2 && s < n && !dead;
    };

    // ---- masks -> window -> id list -> first host read ----
    const int x_pieces = nvec * a.batch;
    V xs[MODE == kOneToken ? 1 : 16];
    if constexpr (MODE != kOneToken) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int w = tid * wpt + i;
            if (i < wpt && w < nwords) m[i] = load_mask_word(a.step_mask, w, F >> 3);
        }
        // x of the tokens (at most 64 KiB) is requested here and stored behind the first host read
        if (wg > 0) {
#pragma unroll
            for (int g = 0; g < 16; g += 4)
                if (g * 256 < x_pieces) {
#pragma unroll
                    for (int i = g; i < g + 4; ++i) xs[i] = reinterpret_cast<const V*>(a.x)[min(i * 256 + tid, x_pieces - 1)];
                }
        }
    } else {
        unsigned p[8];
        const int w0 = tid * wpt, nw = max(0, min(wpt, nwords - w0));
        const bool ok = poll_words<8>(a.m_words + (size_t)(wg & (kWordReps - 1)) * a.m_pitch + 2 * w0, 1, 2 * nw, stamp_now,
                                      a.polls, p);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i < nw) m[i] = ((unsigned long long)p[2 * i + 1] << 32) | p[2 * i];
        if (__syncthreads_or(!ok)) own_masks<T, GATE>(a, L, wpt, m);        // (does not touch the staged owners)
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) now[i] = keep[i] | m[i];
    diff();
    bool over = n - tot_r < 0 || n - tot_r + tot_a > capacity;
    if (over && a.shrink) {
        // Dynamic window (see k_window_plan): what this step needs in any case (m) and the ring entries of ages 1 .. j, for the
        // largest j for which they fit.
        auto age_word = [&](int age, int w) -> unsigned long long {
            return a.ring[(size_t)((slot_now - age + k) % k) * a.ring_words + w];
        };
        const int ages = max(k - a.keep, 0);                      // L.cnt_age[j], j = 0 .. ages
        for (int i = tid; i <= ages; i += 256) L.cnt_age[i] = 0;
        lds_barrier();
        unsigned long long u[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) u[i] = m[i];
        for (int a0 = 0; a0 <= ages; a0 += kRingRegs) {           // counts for j = a0 .. a0 + 7
            int pc[kRingRegs];
#pragma unroll
            for (int j = 0; j < kRingRegs; ++j) pc[j] = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int w = tid * wpt + i;
                if (i < wpt) {                                // uniform: one word after the other, few registers
                    unsigned long long e[kRingRegs];
#pragma unroll
                    for (int j = 0; j < kRingRegs; ++j) {
                        const int age = a0 + j;
                        e[j] = (w < nwords && age >= 1 && age <= oldest) ? age_word(age, w) : 0ull;
                    }
#pragma unroll
                    for (int j = 0; j < kRingRegs; ++j) {
                        u[i] |= e[j];
                        pc[j] += __popcll(u[i]);
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < kRingRegs; ++j) {
                const int tot = __builtin_amdgcn_readlane(wave_inclusive_scan(pc[j], lane), kWave - 1);
                if (lane == 0 && tot && a0 + j <= ages) atomicAdd(&L.cnt_age[a0 + j], tot);
            }
        }
        lds_barrier();
        int fit = -1;
        for (int j = 0; j <= ages; ++j)
            if (L.cnt_age[j] <= capacity) fit = j;                // (the counts grow with j)
        k_eff = a.keep + fit;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            now[i] = m[i];
            const int w = tid * wpt + i;
            if (i < wpt && w < nwords)
                for (int age = 1; age <= min(fit, oldest); ++age) now[i] |= age_word(age, w);
        }
        diff();
        over = fit < 0 || n - tot_r < 0 || n - tot_r + tot_a > capacity;
    }
    if (over) {                                      // uniform: leave everything untouched
        if (wg == 0 && tid == 0) {
            *a.n_added = 0;
            *a.n_removed = 0;
            StepCounts nx = cur;
            nx.error = 3;                                    // LIF_CAPACITY
            nx.n_added = nx.n_removed = 0;
            st->next = nx;
        }
        return;
    }
    n2 = n - tot_r;
    items = max(tot_a, tot_r);
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (i < wpt) {
            L.rem[tid * wpt + i] = prev[i] & ~now[i];
            L.add[tid * wpt + i] = now[i] & ~prev[i];
        }
    fill_ids(0);                                                 // (reads only what this thread has just written)
    if (tid == 0) L.planned = L.classified = 0;
    if constexpr (MODE != kOneToken)
        if (tid == 0) post->seq = post->done = post->arrived = 0;
    lds_barrier();

    // ---- deletion plan (see k_window_plan): holes = dead slots below n', fillers = live slots at or above it ----
    // Up to 4096 rows waves 1..3 make it while the first host read of wave 0 is on its way (plan_alone).  More rows, and
    // the bookkeeping workgroup (which needs the number of moves): all waves together, ahead of the host reads.
    const bool alone = wg > 0 && nblk <= kWave;
    int H = 0;
    // destination of the tail slot of this lane in block b (kNoDst: dead) for the items [c0, ...)
    auto put_dst = [&](int b, bool fill, int c0) {
        const unsigned long long bf = __ballot(fill);
        const int q = b * kWave + lane - n2;
        if (q >= 0 && q < tot_r && (unsigned)(q - c0) < (unsigned)kListItems) {
            const int r = H - 1 - (L.blk_f[b] + __popcll(bf & lt));
            int dst = kNoDst;
            if (fill && r >= 0 && r < H) {
                if (H <= kHoleFew) dst = L.hole[r];
                else dst = a.hole_list[r];
            }
            L.dst[q - c0] = (uint16_t)dst;
        }
    };
    if (tot_r > 0 && !alone) {                                   // uniform
        // The dead slots of block b are kept by the wave that classifies it (number i = b / 4 of its blocks) in lane i mod 64 of
        // dead[i / 64]: looked up again in every pass, the owners past the staged ones cost a memory round trip per block (OPT shape, 4
        // tokens: 140 -> 125 us a step at 15700 rows, 124 -> 111 at 14300; one token 91 -> 88 at 6600; up to 4096 rows the same).
        unsigned long long dead[4] = {0ull, 0ull, 0ull, 0ull};
        auto classify = [&](int b, int id, unsigned long long removed) {         // removed: word id / 64 of L.rem
            const int i = b >> 2, s = b * kWave + lane;
            const unsigned long long m = __ballot((unsigned)id >= (unsigned)F || ((removed >> (id & 63)) & 1ull));
#pragma unroll
            for (int r = 0; r < 4; ++r) dead[r] = (i == r * kWave + lane) ? m : dead[r];
            const int ch = __popcll(__ballot(s < n2) & m), cf = __popcll(__ballot(s >= n2 && s < n) & ~m);
            if (lane == 0 && b < nblk) {
                L.blk_h[b] = (uint16_t)ch;
                L.blk_f[b] = (uint16_t)cf;
            }
        };
        auto dead_of = [&](int b) -> unsigned long long {            // uniform; never under a condition that differs between lanes
            const int i = b >> 2;
            const unsigned long long v = i < 64 ? dead[0] : i < 128 ? dead[1] : i < 192 ? dead[2] : dead[3];
            return ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), i & 63) << 32) |
                   (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, i & 63);
        };
        static_assert(kPtrLds / kWave % 32 == 0, "a round is staged as a whole or not at all");
#pragma unroll 1
        for (int b0 = wave; b0 < nblk; b0 += 4 * 8) {
            int id[8];
            if (b0 < kPtrLds / kWave) {                          // uniform
#pragma unroll
                for (int q = 0; q < 8; ++q) id[q] = L.ptr[(b0 + q * 4) * kWave + lane];
            } else {
#pragma unroll
                for (int q = 0; q < 8; ++q) id[q] = a.pointers[min((b0 + q * 4) * kWave + lane, capacity - 1)];
            }
#pragma unroll
            for (int g = 0; g < 8; g += 4) {
                unsigned long long w[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) w[q] = L.rem[min((unsigned)id[g + q] >> 6, 1023u)];
#pragma unroll
                for (int q = 0; q < 4; ++q)                      // (one token: 0.7 us faster with the branch, a batch 0.6 without)
                    if (MODE != kOneToken || b0 + (g + q) * 4 < nblk) classify(b0 + (g + q) * 4, id[g + q], w[q]);
            }
        }
        lds_barrier();
        {                                                        // prefix over the blocks, bpt consecutive ones per thread
            const int bpt = (nblk + 255) >> 8;
            int vh = 0, vf = 0, fillers;
#pragma unroll 1
            for (int b = tid * bpt; b < min(nblk, tid * bpt + bpt); ++b) {
                vh += L.blk_h[b];
                vf += L.blk_f[b];
            }
            int ph, pf;
            block_exclusive_scan2<4, true>(vh, vf, L.wave_tot, &ph, &pf, &H, &fillers);
#pragma unroll 1
            for (int b = tid * bpt; b < min(nblk, tid * bpt + bpt); ++b) {
                const int ch = L.blk_h[b], cf = L.blk_f[b];
                L.blk_h[b] = (uint16_t)ph;
                L.blk_f[b] = (uint16_t)pf;
                ph += ch;
                pf += cf;
            }
        }
        lds_barrier();
        if (wg > 0) {
            const bool in_lds = H <= kHoleFew;                   // longer lists: every workgroup writes the same values to global
            const int hblk = (n2 + kWave - 1) >> 6;              // blocks with slots below the tail
#pragma unroll 1
            for (int b = wave; b < hblk; b += 4) {
                const int s = b * kWave + lane;
                const unsigned long long bh = dead_of(b) & __ballot(s < n2);
                if ((bh >> lane) & 1ull) {
                    const int pos = L.blk_h[b] + __popcll(bh & lt);
                    if (in_lds) L.hole[pos] = (uint16_t)s;
                    else a.hole_list[pos] = s;
                }
            }
            if (in_lds) lds_barrier();
            else __syncthreads();
            const int tail = n2 >> 6;                            // first block with slots of the first items
#pragma unroll 1
            for (int b = tail + ((wave - tail) & 3); b < nblk; b += 4) {
                const int s = b * kWave + lane;
                const unsigned long long m = dead_of(b);         // (by the whole wave)
                put_dst(b, s >= n2 && s < n && !((m >> lane) & 1ull), 0);
            }
        }
    }
    auto fill_dst = [&](int c0) {                                // later pieces of the list (`dead` is not kept through the load loop)
        const int tail = (n2 + c0) >> 6;
#pragma unroll 1
        for (int b = tail + ((wave - tail) & 3); b < nblk; b += 4) {
            bool hole, fill;
            flags_of(b, owner(b), hole, fill);
            put_dst(b, fill, c0);
        }
    };
    // The plan for at most 64 blocks, all of them staged, by waves 1..3: they share the classification, wave 1 does the rest.
    auto plan_alone = [&](int c0) {
        for (int b0 = (wave - 1) * 4; b0 < nblk; b0 += 12) {
            int id[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) id[q] = L.ptr[min(b0 + q, kPtrLds / kWave - 1) * kWave + lane];
#pragma unroll
            for (int q = 0; q < 4; ++q) {                        // (blocks past the last one have no slots in use)
                bool hole, fill;
                flags_of(b0 + q, id[q], hole, fill);
                const unsigned long long bh = __ballot(hole), bf = __ballot(fill);
                if (lane == 0 && b0 + q < kWave) {
                    L.flag_h[b0 + q] = bh;
                    L.flag_f[b0 + q] = bf;
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        if (lane == 0) __hip_atomic_fetch_add(&L.classified, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (wave != 1) return;
        while (__hip_atomic_load(&L.classified, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < 3) __builtin_amdgcn_s_sleep(1);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        // lane b keeps the flags of block b, and lists its holes
        unsigned long long mh = lane < nblk ? L.flag_h[lane] : 0ull;
        const unsigned long long mf = lane < nblk ? L.flag_f[lane] : 0ull;
        const int v = __popcll(mh) | (__popcll(mf) << 16), inc = wave_inclusive_scan(v, lane), ex = inc - v;
        const int holes = __builtin_amdgcn_readlane(inc, kWave - 1) & 0xffff;
        for (int pos = ex & 0xffff; __any(mh != 0ull); ++pos) {
            if (mh) L.hole[min(pos, kHoleFew - 1)] = (uint16_t)(lane * kWave + __ffsll((long long)mh) - 1);
            mh &= mh - 1;
        }
        // (at most half of 4096 rows can be holes: kHoleFew)
        __builtin_amdgcn_wave_barrier();
        for (int b = (n2 + c0) >> 6; b < nblk; ++b) {
            const unsigned long long bf = ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(mf >> 32), b) << 32) |
                                          (unsigned)__builtin_amdgcn_readlane((int)(unsigned)mf, b);
            const int q = b * kWave + lane - n2;
            if (q >= 0 && q < tot_r && (unsigned)(q - c0) < (unsigned)kListItems) {
                const int r = holes - 1 - ((int)((unsigned)__builtin_amdgcn_readlane(ex, b) >> 16) + __popcll(bf & lt));
                L.dst[q - c0] = (((bf >> lane) & 1ull) && r >= 0) ? L.hole[r] : (uint16_t)kNoDst;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        if (lane == 0) __hip_atomic_store(&L.planned, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    if (wg > 0 && !alone) lds_barrier();
    if (loads && lw < (PAIRED ? 2 * tot_a : tot_a))              // unit lw (below kListItems)
        request_host(__builtin_amdgcn_readfirstlane((int)L.ids[PAIRED ? lw >> 1 : lw]), PAIRED ? lw & 1 : 0);

    if constexpr (MODE != kOneToken) {
        if (wg > 0) {
            int t = tid / nvec, p = tid - t * nvec;
            const int dt = 256 / nvec, dp = 256 - dt * nvec;
#pragma unroll
            for (int g = 0; g < 16; g += 4)
                if (g * 256 < x_pieces) {
#pragma unroll
                    for (int i = g; i < g + 4; ++i) {
                        if (i * 256 + tid < x_pieces) reinterpret_cast<V*>(lds_x + t * a.x_pitch)[p] = xs[i];
                        t += dt;
                        p += dp;
                        if (p >= nvec) {
                            p -= nvec;
                            ++t;
                        }
                    }
                }
            lds_barrier();
        }
    }

    if (wg == 0) {
        // ---- bookkeeping: window state, id lists, counts ----
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int w = tid * wpt + i;
            if (i < wpt && w < nwords) {
                a.cur_set[(size_t)(cur.set_par ^ 1) * a.ring_words + w] = now[i];
                if (!a.multi) a.ring[(size_t)slot_now * a.ring_words + w] = m[i];
            }
        }
        for (int i = 0; i < wpt; ++i) {
            unsigned long long ab = L.add[tid * wpt + i], rb = L.rem[tid * wpt + i];
            while (ab) {
                a.added[off_a++] = (tid * wpt + i) * 64 + __ffsll((long long)ab) - 1;
                ab &= ab - 1;
            }
            while (rb) {
                a.removed[off_r++] = (tid * wpt + i) * 64 + __ffsll((long long)rb) - 1;
                rb &= rb - 1;
            }
        }
        if (tid == 0) {
            *a.n_added = tot_a;
            *a.n_removed = tot_r;
            StepCounts nx;
            nx.num_used = n2 + tot_a;
            nx.n_base = n2;
            nx.step = cur.step + 1;
            nx.error = 0;
            nx.n_added = tot_a;
            nx.n_removed = tot_r;
            nx.n_moved = H;
            nx.window_len = min(min(cur.window_len + a.keep, k), k_eff);
            nx.ring_pos = (cur.ring_pos + a.keep) % k;
            nx.set_par = cur.set_par ^ 1;
            st->next = nx;
            atomicAdd(&st->c_steps, 1ull);
            atomicAdd(&st->c_added, (unsigned long long)tot_a);
            atomicAdd(&st->c_removed, (unsigned long long)tot_r);
            atomicAdd(&st->c_rows_moved, (unsigned long long)H);
            atomicAdd(&st->c_h2d_bytes, (unsigned long long)tot_a * row_bytes);
        }
        return;
    }

    // ---- load and move ----
    const int new_step = cur.step + 1, nw = a.n_load;
    V xr[MODE == kOneToken ? NI : 1];                            // (behind the first host read: needed once that has arrived)
    auto load_x = [&]() {
        if constexpr (MODE == kOneToken) load_pieces(xr, (const char*)a.x);
    };
    if (wave == 0 || !alone) load_x();                           // (the others have a plan to make first)
    // What a slot becomes: the activation of a row, in the order of operations of the activation role
    constexpr int GV = GLU ? 2 : 1;                              // vectors it needs
    auto partial_dots = [&](const V (&v)[GA][NI], float& pu, float& pg) {
        pu = pg = 0.f;
        if constexpr (MODE == kOneToken) {
#pragma unroll
            for (int it = 0; it < NI; ++it) {
                pu = dot_acc(v[GLU ? 1 : 0][it], xr[it], pu);
                if (GLU) pg = dot_acc(v[0][it], xr[it], pg);
            }
        }
    };
    auto finish_slot = [&](int s, int id, float bs, float pu, float pg) {
        const float du = wave_sum(pu);
        float act;
        if (GLU) act = fmaxf(wave_sum(pg) + bs, 0.f) * du;
        else if (GATE) act = du;                                 // the down projection multiplies with the gate activation
        else act = fmaxf(du + bs, 0.f);
        if (lane == 0) {
            a.ptr_new[s] = id;
            a.bias_new[s] = bs;
            a.h_new[s] = act;
            a.stamp[s] = new_step;
        }
    };
    // several tokens: wave 0 stages the rows of a unit and posts them, waves 1..3 compute
    const int row_pitch = step_x_pitch(d, (int)sizeof(T));
    const int in_lds = a.stage_rows;                             // rows there is room for: 2, or one after the other
    unsigned char* lds_row = lds_x + a.batch * a.x_pitch;
    int seq = 0;                                                 // posts so far
    auto stage_row = [&](const V (&v)[GA][NI], int place) {
        if constexpr (MODE != kOneToken) {
            const unsigned off = lane_bytes();
#pragma unroll
            for (int g = 0; g < GV; ++g)
#pragma unroll
                for (int it = 0; it < NI; ++it)
                    if (it < full_pieces(NI) || off + it * 1024u < (unsigned)vec_bytes)
                        *reinterpret_cast<V*>(lds_row + (place * GV + g) * row_pitch + (off + it * 1024u)) = v[g][it];
        }
    };
    auto await_done = [&]() {                                    // the rows of the post before have been used
        if constexpr (MODE != kOneToken) {
            while (__hip_atomic_load(&post->done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < 3 * seq) __builtin_amdgcn_s_sleep(1);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        }
    };
    auto post_rows = [&](int rows, const Slot& r0, float g0, const Slot& r1, float g1) {        // g: lane t: of token t
        if constexpr (MODE != kOneToken) {
            if (lane == 0) {
                post->rows = rows;
                post->slot[0] = r0;
                post->slot[1] = r1;
            }
            if (GATE && lane < 8) {
                post->gate[0][lane] = g0;
                post->gate[1][lane] = g1;
            }
            ++seq;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
            if (lane == 0) __hip_atomic_store(&post->seq, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    };
    auto put = [&](int row, int t, float sg, float su) {         // activation of one row for token t
        if constexpr (MODE != kOneToken) {
            const Slot r = post->slot[row];
            float act;
            if (GLU) act = fmaxf(sg + r.bias, 0.f) * su;
            else if (GATE) act = post->gate[row][t] * su;
            else act = fmaxf(su + r.bias, 0.f);
            a.h_new[(size_t)t * capacity + r.s] = act;
            if (t == 0) {
                a.ptr_new[r.s] = r.id;
                a.bias_new[r.s] = r.bias;
                a.stamp[r.s] = new_step;
            }
        }
    };
    // kMfma: parts 2 g and 2 g + 1 for the NG groups g = first, first + 3, ..., independent chains side by side
    auto group_sums = [&](auto ng_c, int first, int rows) {
        if constexpr (MODE == kMfma) {
            constexpr int NP = 2 * decltype(ng_c)::value;
            const int i16 = lane & 15, q = lane >> 4, nks = d >> 5, per = (nks + kMfmaParts - 1) / kMfmaParts;
            const unsigned char* xl = lds_x + min(i16, a.batch - 1) * a.x_pitch + q * 16;       // (columns past the batch are not used)
            const unsigned char* rl = lds_row + (i16 & (GV * rows - 1)) * row_pitch + q * 16;   // (nor rows past the vectors)
            f32x4 acc[NP];
            int k0[NP], cnt[NP];
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const int part = 2 * (first + 3 * (p >> 1)) + (p & 1);
                acc[p] = f32x4{0.f, 0.f, 0.f, 0.f};
                k0[p] = part * per;
                cnt[p] = min(max(nks - part * per, 0), per);     // (does not grow with p)
            }
            auto step = [&](int ks, f32x4 v) {
                return __builtin_amdgcn_mfma_f32_16x16x32_f16(*reinterpret_cast<const f16x8*>(rl + ks * 64),
                                                              *reinterpret_cast<const f16x8*>(xl + ks * 64), v, 0, 0, 0);
            };
#pragma unroll 1
            for (int j = 0; j < cnt[NP - 1]; ++j)
#pragma unroll
                for (int p = 0; p < NP; ++p) acc[p] = step(k0[p] + j, acc[p]);
#pragma unroll
            for (int p = 0; p < NP - 1; ++p)
#pragma unroll 1
                for (int j = cnt[NP - 1]; j < cnt[p]; ++j) acc[p] = step(k0[p] + j, acc[p]);
#pragma unroll
            for (int p = 0; p < NP; p += 2)
                if (lane < 16) *reinterpret_cast<f32x4*>(post->sums[first + 3 * (p >> 1)][lane]) = acc[p] + acc[p + 1];   // D[v][t], v = 0..3
        }
    };
    auto work = [&]() {                                          // waves 1..3, until wave 0 has posted its last rows
        if constexpr (MODE != kOneToken) {
            for (;;) {
                ++seq;
                while (__hip_atomic_load(&post->seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < seq) __builtin_amdgcn_s_sleep(1);
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
                const int rows = __builtin_amdgcn_readfirstlane(post->rows);
                if constexpr (MODE == kMfma) {
                    if (rows > 0) {
                        if (wave < 3) group_sums(std::integral_constant<int, 3>{}, wave - 1, rows);
                        else group_sums(std::integral_constant<int, 2>{}, 2, rows);
                        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
                        int before = 0;
                        if (lane == 0) before = __hip_atomic_fetch_add(&post->arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        if (__builtin_amdgcn_readfirstlane(before) % 3 == 2) {   // the last of the three
                            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
                            // lane = 8 * vector + token; the tree over the groups as tree_push and tree_sum
                            const int t = lane & 7, v = (lane >> 3) & (2 * GV - 1);
                            float g8[8];
#pragma unroll
                            for (int g = 0; g < 8; ++g) g8[g] = post->sums[g][t][v];
                            const float su = tree_sum<8>(g8), sg = GLU ? __shfl(su, lane - 8, kWave) : 0.f;
                            if (lane < 16 * GV && t < a.batch && v % GV == GV - 1 && v / GV < rows) put(v / GV, t, sg, su);
                        }
                    }
                } else if (rows > 0) {
                    constexpr int TT = 3;                        // tokens of a wave, at most 8 in all
                    float acc[TT][2 * GV];
#pragma unroll
                    for (int t = 0; t < TT; ++t)
#pragma unroll
                        for (int v = 0; v < 2 * GV; ++v) acc[t][v] = 0.f;
#pragma unroll 1
                    for (int idx = lane; idx < nvec; idx += 64) {
                        V row[2 * GV];
#pragma unroll
                        for (int v = 0; v < 2 * GV; ++v)
                            row[v] = reinterpret_cast<const V*>(lds_row + min(v, GV * rows - 1) * row_pitch)[idx];
#pragma unroll
                        for (int t = 0; t < TT; ++t) {
                            const V xv = reinterpret_cast<const V*>(lds_x + min(wave - 1 + 3 * t, a.batch - 1) * a.x_pitch)[idx];
#pragma unroll
                            for (int v = 0; v < 2 * GV; ++v) acc[t][v] = dot_acc(row[v], xv, acc[t][v]);
                        }
                    }
#pragma unroll
                    for (int t = 0; t < TT; ++t)
#pragma unroll
                        for (int v = 0; v < 2 * GV; ++v) acc[t][v] = wave_sum(acc[t][v]);
#pragma unroll
                    for (int t = 0; t < TT; ++t)
                        if (wave - 1 + 3 * t < a.batch && lane < rows)
                            put(lane, wave - 1 + 3 * t, lane ? acc[t][GV] : acc[t][0], lane ? acc[t][2 * GV - 1] : acc[t][GV - 1]);
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
                if (lane == 0) __hip_atomic_fetch_add(&post->done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (rows == 0) break;
            }
        }
    };
    auto gate_of = [&](int id) -> float {                        // lane t: resident gate activation of neuron id for token t
        if constexpr (MODE != kOneToken && GATE) return a.gact[(size_t)min(lane, a.batch - 1) * F + min(max(id, 0), F - 1)];
        return 0.f;
    };
    auto old_owner = [&](int s) -> int {
        int id = L.ptr[min(s, kPtrLds - 1)];
        if (s >= kPtrLds) id = a.pointers[s];
        return id;
    };
    auto await_plan = [&]() {
        while (!__hip_atomic_load(&L.planned, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) __builtin_amdgcn_s_sleep(1);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    // Lists longer than kListItems are gone through piece by piece.
    for (int c0 = 0; c0 < items; c0 += kListItems) {
        if (c0 > 0) {
            lds_barrier();
            fill_ids(c0);
            if (tid == 0) L.planned = L.classified = 0;
            if (tot_r > 0 && !alone) fill_dst(c0);
            lds_barrier();
        }
        const int n_a = min(max(tot_a - c0, 0), kListItems), n_r = min(max(tot_r - c0, 0), kListItems);     // of this piece
        const int units = PAIRED ? 2 * n_a : n_a;
        if (alone && wave > 0) {
            if (tot_r > c0) plan_alone(c0);
            load_x();
        }
        const int only = max(n_r - n_a, 0);                      // rows that nothing overwrites
        if (MODE != kOneToken && wave > 0) work();
        if (wave == 0) {
            struct Unit {
                int i, part, nid, dst, old_id;                   // item c0 + i
                float old_bias, new_bias, old_gate, new_gate;
            };
            auto make_unit = [&](int u, bool ask) {              // its numbers, and the requests for its bundle
                Unit r;
                r.part = PAIRED ? u & 1 : 0;
                r.i = PAIRED ? u >> 1 : u;
                const int s = n2 + c0 + r.i;
                r.nid = __builtin_amdgcn_readfirstlane((int)L.ids[r.i]);
                r.dst = r.i < n_r ? __builtin_amdgcn_readfirstlane((int)L.dst[r.i]) : kNoDst;
                if constexpr (MODE == kOneToken) r.old_id = a.pointers[s];
                else r.old_id = old_owner(s);
                r.old_bias = a.bias[s];
                r.new_bias = a.b[r.nid];
                r.old_gate = gate_of(r.old_id);
                r.new_gate = gate_of(r.nid);
                if (ask) request_host(r.nid, r.part);
                return r;
            };
            int place = lw, round = 0;
            if (lw < units) {
                if (alone && n_r > 0) await_plan();
                Unit cu = make_unit(lw, c0 > 0);                 // (the bundle of the first piece was requested above)
                request_row(n2 + c0 + cu.i, cu.part);            // (also where nothing is moved: no branch around loads)
                for (;;) {
                    const int s = n2 + c0 + cu.i;
                    const bool act = cu.part == 0, moves = cu.dst != kNoDst;      // uniform over the wave
                    float mdu = 0.f, mdg = 0.f, hdu = 0.f, hdg = 0.f;
                    if (moves) {
                        store_row(cu.dst, cu.part, mv);
                        if (act) partial_dots(mv, mdu, mdg);
                    }
                    store_row(s, cu.part, hv);
                    const Slot fresh = {s, cu.nid, cu.new_bias}, moved = {cu.dst, cu.old_id, cu.old_bias};
                    if (act) {
                        partial_dots(hv, hdu, hdg);
                        if (MODE != kOneToken) {
                            await_done();
                            stage_row(hv, 0);
                            if (moves && in_lds > 1) stage_row(mv, 1);
                            post_rows(moves && in_lds > 1 ? 2 : 1, fresh, cu.new_gate, moved, cu.old_gate);
                            if (moves && in_lds < 2) {
                                await_done();
                                stage_row(mv, 0);
                                post_rows(1, moved, cu.old_gate, moved, cu.old_gate);
                            }
                        }
                    }
                    place = place + 1 < nw ? place + 1 : 0;
                    round += nw;
                    const bool more = round + place < units;
                    Unit nu = cu;
                    if (more) {
                        nu = make_unit(round + place, true);
                        request_row(n2 + c0 + nu.i, nu.part);
                    }
                    if (MODE == kOneToken && act) {
                        if (moves) finish_slot(cu.dst, cu.old_id, cu.old_bias, mdu, mdg);
                        finish_slot(s, cu.nid, cu.new_bias, hdu, hdg);
                    }
                    if (!more) break;
                    cu = nu;
                }
            }
        }
        // rows that nothing overwrites: by the waves that do not load, with several tokens by the one that does (whole rows)
        if constexpr (MODE == kOneToken) {
            if (wave > 0 && only > 0) {
                if (alone) await_plan();
                for (int v = lw * 3 + wave - 1; v < (PAIRED ? 2 * only : only); v += 3 * nw) {
                    const int part = (PAIRED && v >= only) ? 1 : 0, i = n_a + v - part * only;
                    const int dst = __builtin_amdgcn_readfirstlane((int)L.dst[i]), s = n2 + c0 + i;
                    if (dst == kNoDst) continue;
                    request_row(s, part);
                    const int id = a.pointers[s];
                    const float bs = a.bias[s];
                    store_row(dst, part, mv);
                    if (part == 0) {
                        float pu, pg;
                        partial_dots(mv, pu, pg);
                        finish_slot(dst, id, bs, pu, pg);
                    }
                }
            }
        } else if (wave == 0) {
            if (only > 0 && alone) await_plan();
            for (int i = n_a + (nw - 1 - lw); i < n_a + only; i += nw) {         // (the last ones have had the fewest units)
                const int dst = __builtin_amdgcn_readfirstlane((int)L.dst[i]), s = n2 + c0 + i;
                if (dst == kNoDst) continue;
                request_row(s, 0);
                if (PAIRED) load_pieces(hv[0], row_vec(s, GA));
                const int id = old_owner(s);
                const Slot r = {dst, id, a.bias[s]};
                const float gb = gate_of(id);
                store_row(dst, 0, mv);
                if (PAIRED) store_pieces(row_vec(dst, GA), hv[0]);
                await_done();
                stage_row(mv, 0);
                post_rows(1, r, gb, r, gb);
            }
            await_done();
            post_rows(0, Slot{}, 0.f, Slot{}, 0.f);
        }
    }
}

// Two workgroups per compute unit as long as a loader's bundle piece, row piece and x fit the registers of half a SIMD.
template <int NI, bool GLU>
constexpr int step1_wgs_per_cu() {
    constexpr int vectors = NI > 2 ? (GLU ? 2 : 1) : (GLU ? 3 : 2);
    return (2 * vectors + 1) * NI * 4 <= 120 ? 2 : 1;
}
template <typename T, int NI, bool GLU, bool GATE>
__global__ __launch_bounds__(256, (step1_wgs_per_cu<NI, GLU>())) void k_step1(const StepArgs a) {
    __shared__ __align__(16) unsigned char lds[sizeof(PlanLds) > sizeof(PredictLds) ? sizeof(PlanLds) : sizeof(PredictLds)];
    const int block = blockIdx.x;
    if (block < a.n_pred) {
        if constexpr (GATE) gate_role<T, NI>(a, block, reinterpret_cast<unsigned*>(lds));
        else lowrank_role<T, NI>(a, block, *reinterpret_cast<PredictLds*>(lds));
    } else if (block <= a.n_pred + a.n_load) {
        cache_role<T, NI, GLU, GATE, kOneToken>(a, block - a.n_pred, *reinterpret_cast<PlanLds*>(lds), nullptr, nullptr);
    } else {
        const int first = a.n_pred + a.n_load + 1;
        ffn_up_role<T, NI, GLU, true>((const T*)a.matrix, a.bias, (const T*)a.x, a.h, a.d, 1, a.capacity, a.row_elems, a.spec,
                                      block - first, gridDim.x - first, a.pointers, a.gact, a.F, a.st);
    }
}

// The same for a batch of tokens or a pass of several, behind the launches of the predictor: bookkeeping (workgroup 0),
// loaders, and the activation stage over the rows in use - on the matrix cores (MFMA: fp16, d a multiple of 32), else one
// wave per row.  Dynamic LDS: step_batch_lds bytes.
// Registers (gfx950, as the compiler reports them): the loader role has more uniform values than the 106 scalar registers hold,
// 97 to 148 of them live in lanes of vector registers (k_step1: 75 to 124).  None goes to memory, which would queue up behind the
// host reads.  The predictor is a template parameter for that reason: a kernel with both forms of the role spilled 169 to 246
// scalar registers and was 82 to 106 KB of code (41 to 60 KB each by itself), more than the 64 KB instruction cache of two compute units.
template <typename T, int NI, bool GLU, bool GATE, bool MFMA, int WAVES>
__global__ __launch_bounds__(WAVES * 64, 1) void k_step_batch(const StepArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_step[];
    const int block = blockIdx.x;
    if (block <= a.n_load) {
        if (WAVES > 4 && threadIdx.x >= 256) return;             // (a barrier waits for the waves that are left)
        PlanLds& plan = *reinterpret_cast<PlanLds*>(smem_step);
        PostLds* post = reinterpret_cast<PostLds*>(smem_step + (sizeof(PlanLds) + 15) / 16 * 16);
        cache_role<T, NI, GLU, GATE, MFMA ? kMfma : kDots>(a, block, plan, post, smem_step + kStepXOff);
    } else if constexpr (MFMA) {
        const int tile = block - a.n_load - 1;
        ffn_up_mfma_tile_staged<GLU, WAVES>(
            (const _Float16*)a.matrix, a.bias, (const _Float16*)a.x, a.h, a.d, a.batch, a.capacity, a.row_elems, tile,
            tile < a.spec, a.pointers, GATE ? a.gact : nullptr, a.F, a.st, smem_step);
    } else {
        const int first = a.n_load + 1;
        ffn_up_role<T, NI, GLU, false, WAVES>((const T*)a.matrix, a.bias, (const T*)a.x, a.h, a.d, a.batch, a.capacity, a.row_elems,
                                              a.spec, block - first, gridDim.x - first, a.pointers,
                                              GATE ? a.gact : nullptr, a.F, a.st);
    }
}
// LDS of a workgroup of k_step_batch
inline size_t step_batch_lds(int batch, int d, int elem, bool glu, bool mfma, int rows) {
    const size_t loader = kStepXOff + (size_t)batch * step_x_pitch(d, elem) + (size_t)rows * (glu ? 2 : 1) * step_x_pitch(d, elem);
    const size_t up = mfma ? (size_t)mfma_staged_lds(glu, kMfmaWaves) : (size_t)batch * d * elem;
    return loader > up ? loader : up;
}
constexpr size_t kStepLdsLimit = 160 * 1024;

// Launches for one element type and bundle form (NI by the row width).  Every combination is compiled in a source file of
// its own (step*.hip), side by side: together they are most of the library's compile time.
template <typename T, bool GLU, bool GATE>
inline void launch_step1_as(const StepArgs& a, int grid, hipStream_t s) {
    const int ni = (a.d / Vec<T>::N + 63) / 64;
#define LIF_S1(NI) hipLaunchKernelGGL((k_step1<T, NI, GLU, GATE>), dim3(grid), dim3(256), 0, s, a)
    if (ni <= 1) LIF_S1(1);
    else if (ni <= 2) LIF_S1(2);
    else if (ni <= 4) LIF_S1(4);
    else if (ni <= 6) LIF_S1(6);
    else if (ni <= 8) LIF_S1(8);
    else if (ni <= 9) LIF_S1(9);
    else if (ni <= 12) LIF_S1(12);
    else LIF_S1(16);
#undef LIF_S1
}
// Waves of a workgroup of k_step_batch: 4, or 8 where the LDS of a loader (x of the tokens and staged rows) leaves room for one
// workgroup per compute unit.  The activation workgroups of the launch carry the same LDS, and four waves that read a row each
// reach a fraction of the bandwidth, which shows where few rows are added and the load does not cover them.  fp32 rows, us a
// step with 4 -> 8 waves (rows in use, rows added): d = 1288, 8 tokens: (9277, 0) 77.7 -> 57.0, (9578, 47) 88.3 -> 71.2, (13408,
// 477) 157.8 -> 156.9; d = 2048, gated, 8 tokens: (4699, 0) 71.8 -> 55.1, (6444, 304) 187.8 -> 187.1; d = 2048, 4 tokens: (6221,
// 0) 51.9 -> 43.2.  With room for two workgroups four waves are better (d = 1288, 3 tokens, (929, 0): 25.7 against 26.6).
// The matrix-core stage keeps 4: it is at least as fast as in a launch of its own.  Gated rows of more than 12 KiB a vector
// would spill registers at 8 waves.
constexpr int step_batch_most_waves(int ni, bool glu, bool mfma) { return mfma || ni <= 2 || (glu && ni > 12) ? 4 : 8; }
inline int step_batch_waves(int ni, bool glu, bool mfma, size_t lds) { return lds > kStepLdsLimit / 2 ? step_batch_most_waves(ni, glu, mfma) : 4; }

// (more than 64 KiB of LDS has to be allowed once per kernel and device: `allow` does only that, for the kernels of a.d)
template <typename T, bool GLU, bool GATE, bool MFMA>
inline hipError_t launch_step_batch_as(const StepArgs& a, int grid, size_t lds, bool allow, hipStream_t s) {
    const int ni = (a.d / Vec<T>::N + 63) / 64;
#define LIF_SB(NI)                                                                                                      \
    do {                                                                                                                 \
        constexpr int kMost = step_batch_most_waves(NI, GLU, MFMA);                                                      \
        const auto few = &k_step_batch<T, NI, GLU, GATE, MFMA, 4>, many = &k_step_batch<T, NI, GLU, GATE, MFMA, kMost>;  \
        if (allow) {                                                                                                     \
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(few),                                 \
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)kStepLdsLimit);    \
            return e != hipSuccess ? e : hipFuncSetAttribute(reinterpret_cast<const void*>(many),                        \
                                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)kStepLdsLimit); \
        }                                                                                                                \
        const int waves = step_batch_waves(NI, GLU, MFMA, lds);                                                          \
        hipLaunchKernelGGL(waves == 4 ? few : many, dim3(grid), dim3(waves * 64), lds, s, a);                            \
        return hipSuccess;                                                                                               \
    } while (0)
    if (ni <= 1) LIF_SB(1);
    else if (ni <= 2) LIF_SB(2);
    else if (ni <= 4) LIF_SB(4);
    else if (ni <= 6) LIF_SB(6);
    else if (ni <= 8) LIF_SB(8);
    else if (ni <= 9) LIF_SB(9);
    else if (ni <= 12) LIF_SB(12);
    else LIF_SB(16);
#undef LIF_SB
}
void launch_step1_f16_plain(const StepArgs& a, int grid, hipStream_t s);
void launch_step1_f16_glu(const StepArgs& a, int grid, hipStream_t s);
void launch_step1_f16_gate(const StepArgs& a, int grid, hipStream_t s);
void launch_step1_f32_plain(const StepArgs& a, int grid, hipStream_t s);
void launch_step1_f32_glu(const StepArgs& a, int grid, hipStream_t s);
void launch_step1_f32_gate(const StepArgs& a, int grid, hipStream_t s);
hipError_t launch_step_batch_f16_plain(const StepArgs& a, int grid, size_t lds, bool allow, hipStream_t s);
hipError_t launch_step_batch_f16_glu(const StepArgs& a, int grid, size_t lds, bool allow, hipStream_t s);
hipError_t launch_step_batch_f16_gate(const StepArgs& a, int grid, size_t lds, bool allow, hipStream_t s);
hipError_t launch_step_batch_f16_mfma_plain(const StepArgs& a, int grid, size_t lds, bool allow, hipStream_t s);
hipError_t launch_step_batch_f16_mfma_glu(const StepArgs& a, int grid, size_t lds, bool allow, hipStream_t s);
hipError_t launch_step_batch_f16_mfma_gate(const StepArgs& a, int grid, size_t lds, bool allow, hipStream_t s);
hipError_t launch_step_batch_f32_plain(const StepArgs& a, int grid, size_t lds, bool allow, hipStream_t s);
hipError_t launch_step_batch_f32_glu(const StepArgs& a, int grid, size_t lds, bool allow, hipStream_t s);
hipError_t launch_step_batch_f32_gate(const StepArgs& a, int grid, size_t lds, bool allow, hipStream_t s);

}  // namespace lif
