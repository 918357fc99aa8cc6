// One step up to the down projection: of a single token in one launch (k_step1: lif_step and lif_step_tokens, batch 1), of a
// batch or a pass of several tokens in one launch behind the two of the predictor (k_step_batch).
//
// A step is a chain of small dependent stages in front of one long one, the host-link gather of the new bundles
// (Section 3.3 item 2).  As separate launches every short stage costs 4 to 6 us on gfx950: 1.6 us of launch, a memory
// round trip for the state, another one for what the previous kernel wrote.  Here the workgroups of one launch take
// different roles and hand over inside it:
//   workgroups [0, n_pred)        predictor: the first ones compute t = x A (a column each, 256 at a time) and publish it; each of
//                                 the first ceil(F / 64) waits for t and decides the 64 mask bits of its neurons (their weights
//                                 are requested before the wait).  Gate predictor: 32 neurons per workgroup, nothing to wait for.
//   workgroup n_pred              bookkeeping: waits for the masks, makes the deletion plan and publishes it, writes the window
//                                 state, id lists and counts
//   the next n_load workgroups    loaders: after a step that kept them all busy, wait for t, decide a tile of neurons each (each
//                                 pair) and ask for the first bundle it adds; wait for the masks, work out the added ids (every
//                                 workgroup for itself: cheaper than waiting for one that does), gather bundles from pinned host
//                                 memory, move the rows they overwrite where the plan says and compute the activations of the
//                                 rows they write (h_new, stamped with the step)
//   the rest                      activations of the rows that were already in use; behind the predictor where a load is
//                                 likely to hide them (await_predictor), else at once
// A value handed over is a 64-bit word: 32 bits of payload and the number of the step as a stamp, written by a relaxed
// device-scope atomic store and polled with relaxed device-scope atomic loads, so no fence (a device-scope release
// writes back the L2: 6 us) and no clearing is needed.  Stamps are unique between two resets, which clear the words.
// A workgroup waits for workgroups with smaller numbers or, a tile of neurons for the columns of x A, for workgroups that
// fit the chip at the same time (kStepColumns); and never without bound: after `polls` failed polls it computes what it is
// missing itself, with the same arithmetic (polls = 0: never waits at all).
// What other workgroups may still read is not overwritten: the new counts are left in st->next and the slot owners and
// biases of the rows a loader writes in ptr_new / bias_new; the down projection, which runs after all of them, commits
// them.  A matrix row that the activation role reads while a loader overwrites it gives a value that is never used: the
// loader's stamped activation takes precedence for that slot.
// Every sum is formed in the order of the separate kernels, so the step is bit-identical to the four calls.
//
// What bounds it: the host link.  From the first request to the last bundle it moves 55 to 57 GB/s (a copy of 256 MiB by the
// runtime: 57.5).  In front of the first request are a launch and two hand-overs, OPT-6.7B shape (Falcon-7B shape), us from the
// start of the first workgroup: x A published 2.4 (2.5), masks published 4.7 (5.0), known to the loaders 6.2 (6.6), first request 7
// (7.5), of an early bundle 5; behind the last bundle is the down projection.  A compute unit has about 5 KiB of host reads under way, whatever its
// waves ask for, so some 30 loaders fill the link.
// Measured on gfx950, one decode token, with five launches -> with this kernel and the down projection: fp32 d = 256, F = 1024:
// 23.4 -> 14.1 us; OPT-6.7B shape 65.3 -> 57; Falcon-7B shape 149.5 -> 136; Llama-2 shape gated, from a graph, 148.7 -> 132, with
// the gate resident 112.8 -> 105.
#pragma once

#include <cstddef>

#include "lif_ffn.h"
#include "lif_ffn_mfma.h"
#include "lif_predict.h"
#include "lif_window_bits.h"
#include "lif_words.h"

namespace lif {

constexpr int kListItems = 2048;     // work items listed at a time
// Two workgroups per compute unit as long as a loader's bundle piece, row piece and x fit the registers of half a SIMD.
template <int NI, bool GLU>
constexpr int step1_wgs_per_cu() {
    constexpr int vectors = NI > 2 ? (GLU ? 2 : 1) : (GLU ? 3 : 2);
    return (2 * vectors + 1) * NI * 4 <= 120 ? 2 : 1;
}
// Columns of x A are dealt to the first kStepColumns x step1_wgs_per_cu predictor workgroups: every tile of neurons waits for all
// columns, so these have to run at the same time, and that many fit the chip.  Dealt over all of them, one token at d = 5120,
// gated, F = 17000, rank 512 (266 predictor workgroups, one to a compute unit) took 1484 us, every wait running out; so 81.
constexpr int kStepColumns = 256;

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
    unsigned long long* plan_words;  // [capacity] stamped destinations of the tail slots (kNoDst: dead), in the order of the slots
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

// ---- predictor -------------------------------------------------------------------------------------------------

struct PredictLds {
    double t[2048 + 1];              // t = x A, then a 0
    double red[4][64];               // per wave and neuron of the tile
    double part[4];                  // parts of a column
    int missing[4];                  // per wave: a word did not arrive
};

template <typename T, int NI>
__device__ __forceinline__ void load_vec(typename Vec<T>::type (&v)[NI], const T* p, int nvec, int lane) {
    using V = typename Vec<T>::type;
#pragma unroll
    for (int it = 0; it < NI; ++it) {
        const int idx = it * 64 + lane;
        v[it] = (idx < nvec) ? reinterpret_cast<const V*>(p)[idx] : V(0);
    }
}

// x . column straight from memory, for the rare case that a wait ran out: few registers instead of loads in flight
template <typename T>
__device__ __forceinline__ double column_dot_slow(const T* col, const T* x, int first, int end, int lane) {
    using V = typename Vec<T>::type;
    double acc = 0.0;
#pragma unroll 1
    for (int idx = first + lane; idx < end; idx += 64)
        acc = dot_f64(reinterpret_cast<const V*>(col)[idx], reinterpret_cast<const V*>(x)[idx], acc);
    return wave_sum(acc);
}
// t computed by this workgroup alone (a wait that ran out), the parts of a column as in ColumnPart
template <typename T, int NI>
__device__ __forceinline__ void own_t(const StepArgs& a, PredictLds& L) {
    const int lane = threadIdx.x & 63, nvec = a.d / Vec<T>::N, per = ColumnPart<T, NI>::P * 64;
    if (threadIdx.x == 0) L.t[a.rank] = 0.0;
#pragma unroll 1
    for (int j = threadIdx.x >> 6; j < a.rank; j += 4) {
        double part[4];
#pragma unroll
        for (int w = 0; w < 4; ++w)
            part[w] = column_dot_slow((const T*)a.A + (size_t)j * a.d, (const T*)a.x, min(w * per, nvec), min((w + 1) * per, nvec), lane);
        if (lane == 0) L.t[j] = column_total(part);
    }
    __syncthreads();
}

// The 64 mask bits of a tile of neurons: as k_predict_mask for one token.  The weights and offsets are requested by
// the constructor, before t is there.
// WIDE: the weights are widened (`widen`) ahead of t.
template <typename T, bool WIDE = true>
struct MaskTile {
    using V = typename Vec<T>::type;
    static constexpr int VE = Vec<T>::N, LPB = 8 / VE;
    V bv[kMaskRows][LPB];
    double bd[WIDE ? kMaskRows : 1][8];
    float cv;                        // offset of neuron 64 * tile + lane
    int n0;
    bool own_ok;                     // ... which exists
    __device__ __forceinline__ void request(const StepArgs& a, int tile) {
        const int tid = threadIdx.x, cl = tid & (kMaskCols - 1), jg = tid >> 3, own = tile * 64 + (tid & 63);
        n0 = (tile * kMaskCols + cl) * 8;
        own_ok = own < a.F;
        const T* B = (const T*)a.B;
#pragma unroll
        for (int u = 0; u < kMaskRows; ++u) {
            const int j = jg + u * kMaskJg;
#pragma unroll
            for (int q = 0; q < LPB; ++q)
                bv[u][q] = (n0 < a.F && j < a.rank) ? reinterpret_cast<const V*>(B + (size_t)j * a.F + n0)[q] : V(0);
        }
        cv = (a.c && own_ok) ? a.c[own] : 0.f;
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
    // the 64 mask bits of the tile (0 past the last neuron), in every wave; one barrier
    __device__ __forceinline__ unsigned long long finish(const StepArgs& a, PredictLds& L) {
        const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, cl = tid & (kMaskCols - 1), jg = tid >> 3;
        const T* B = (const T*)a.B;
        double v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = 0.0;
#pragma unroll
        for (int u = 0; u < kMaskRows; ++u) {
            if (u * kMaskJg < a.rank) {              // (uniform; bd[u] is 0 past the end)
                const double tj = L.t[min(jg + u * kMaskJg, a.rank)];
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = __builtin_fma(tj, WIDE ? bd[WIDE ? u : 0][e] : (double)bv[u][e / VE][e % VE], v[e]);
            }
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
        // (In registers throughout, and the 64 decisions become the mask word by one ballot: 1.3 -> 0.7 us from t to the published
        // word against exchanges through LDS and a byte per lane.)
        L.red[wave][cl * 8 + fold_owner(lane)] = fold_groups(v, lane);
        __syncthreads();
        double z = ((L.red[0][lane] + L.red[1][lane]) + L.red[2][lane]) + L.red[3][lane];
        z += (double)cv;
        return __ballot(own_ok && z > (double)a.theta);
    }
};

// t of this step into LDS (with the 0 behind it), from copy `rep` of its words; one barrier.  Returns whether all of it has come.
__device__ __forceinline__ bool await_t(const StepArgs& a, PredictLds& L, int rep, unsigned now) {
    const int tid = threadIdx.x;
    unsigned* t32 = reinterpret_cast<unsigned*>(L.t);
    const unsigned long long* src = a.t_words + (size_t)(rep & (kWordReps - 1)) * a.t_pitch;
    bool ok = true;
    for (int i0 = tid; i0 < 2 * a.rank + 2; i0 += 4 * 256) {
        unsigned p[4];
        const int n = min(4, (2 * a.rank - i0 + 255) >> 8);
        ok = poll_words<4>(src + i0, 256, n, now, a.polls, p) && ok;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i0 + i * 256 < 2 * a.rank + 2) t32[i0 + i * 256] = p[i];         // (0 from n on)
    }
    const bool missing = __any(!ok);
    if ((tid & 63) == 0) L.missing[tid >> 6] = missing;
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(L.missing[0] | L.missing[1] | L.missing[2] | L.missing[3]) == 0;
}

template <typename T, int NI, int WGS>
__device__ __forceinline__ void lowrank_role(const StepArgs& a, int block, PredictLds& L) {
    const int tid = threadIdx.x, nvec = a.d / Vec<T>::N;
    const int dealt = min(a.n_pred, kStepColumns * WGS);
    const bool producer = block < min(a.rank, dealt);
    const bool has_tile = block * kMaskCols * 8 < a.F;
    ColumnPart<T, NI> col;
    if (producer) {
        col.load(col.x, (const T*)a.x, nvec);
        col.load(col.a, (const T*)a.A + (size_t)block * a.d, nvec);
    }
    MaskTile<T> tile;
    if (has_tile) tile.request(a, block);
    const int err = a.st->cur.error;
    const unsigned now = (unsigned)a.st->cur.step + 1u;
    if (err) return;
    for (int j = block; producer && j < a.rank; j += dealt) {
        if (j != block) __syncthreads();             // (the parts of the column before are still read)
        const double v = col.sum();
        if (j + dealt < a.rank) col.load(col.a, (const T*)a.A + (size_t)(j + dealt) * a.d, nvec);
        if ((tid & 63) == 0) L.part[tid >> 6] = v;
        __syncthreads();
        if (tid < 2 * kWordReps) {
            const unsigned long long u = __builtin_bit_cast(unsigned long long, column_total(L.part));
            word_store(a.t_words + (size_t)(tid >> 1) * a.t_pitch + 2 * j + (tid & 1), now, (tid & 1) ? (unsigned)(u >> 32) : (unsigned)u);
        }
    }
    if (!has_tile) return;
    tile.widen();
    if (__builtin_expect(!await_t(a, L, block, now), 0)) {
        __syncthreads();
        own_t<T, NI>(a, L);
    }
    const unsigned long long word = tile.finish(a, L);
    if (tid < 64) {
        if (tid < 2 * kWordReps)
            word_store(a.m_words + (size_t)(tid >> 1) * a.m_pitch + 2 * block + (tid & 1), now,
                       (tid & 1) ? (unsigned)(word >> 32) : (unsigned)word);
        const int at = block * kMaskCols + tid;              // mask byte
        if (tid < kMaskCols && at * 8 < a.F) {
            a.masks[at] = (uint8_t)(word >> (8 * tid));
            a.step_mask[at] = (uint8_t)(word >> (8 * tid));
        }
    }
}

// Gate predictor: relu(gate_i . x + b_i) and the mask bit of 8 neurons per wave, as k_predict_gate for one token.
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
        byte = gate_byte<T, NI>((const T*)a.A, a.b, a.gact, grp, a.d / Vec<T>::N, xr, (double)a.theta);
        if (lane == 0) {
            a.masks[grp] = (uint8_t)byte;
            a.step_mask[grp] = (uint8_t)byte;
        }
    }
    if (lane == 0) lds[wave] = byte << (8 * wave);
    __syncthreads();
    if (tid < kWordReps) word_store(a.m_words + (size_t)tid * a.m_pitch + block, now, lds[0] | lds[1] | lds[2] | lds[3]);
}

// ---- window, deletion plan, loaders ----------------------------------------------------------------------------

constexpr int kPtrLds = 8192;        // slot owners staged in LDS
constexpr int kNoDst = 0xffff;       // dead tail slot (a hole lies below n' <= 65535, so it is never slot 65535)
constexpr int kHoleFew = 2048;       // holes kept in LDS; longer lists go to the global scratch list
struct PlanLds {
    unsigned long long rem[1024], add[1024]; // removed and added neurons, one bit each
    unsigned long long wave_tot[4];
    int cnt_age[264];
    unsigned byte[4];
    int off[64];                             // list positions of the first wave's added neurons
    unsigned long long first_bits;           // the neuron of the loader's first unit: bit number first_at.y of these that is
    int2 first_at;                           //  set, from neuron first_at.x on
    int listed;                              // waves that have written their part of ids
    unsigned long long early;                // early tiles with added neurons, one bit each
    union {
        PredictLds predict;                  // an early tile; when a wait ran out
        uint16_t ids[kListItems];            // loaders: the new neurons of the work items
        struct {                             // bookkeeping: the deletion plan
            uint16_t hole[kHoleFew];
            uint16_t fill_before[1024];      // fillers below the granule
            uint16_t ptr[kPtrLds];           // owners (neurons are numbers below 65536)
            unsigned long long dead[1024];   // dead slots of the block
        };
    };
};
// What a loader uses of it in a batched step.  The rest of a loader's LDS (PostLds, x, rows) lies where the deletion plan of the
// bookkeeping workgroup does: all workgroups of the launch carry the same LDS, and behind the whole plan x left room for one of
// them per compute unit instead of two.
constexpr size_t kLoaderPlanLds = (offsetof(PlanLds, ids) + sizeof(uint16_t) * kListItems + 15) / 16 * 16;

// All mask words computed by this workgroup alone (a wait that ran out): m[i] of the words this thread owns
template <typename T, int NI, bool GATE>
__device__ __forceinline__ void own_masks(const StepArgs& a, PlanLds& L, int wpt, unsigned long long (&m)[4]) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nwords = (a.F + 63) >> 6;
    if constexpr (!GATE) own_t<T, NI>(a, L.predict);
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
                    const double v = column_dot_slow((const T*)a.A + (size_t)i * a.d, (const T*)a.x, 0, a.d / Vec<T>::N, lane);
                    if (v + (double)a.b[i] > (double)a.theta) byte |= 1u << e;
                }
                __syncthreads();
                if (lane == 0) L.byte[wave] = byte << (8 * wave);
                __syncthreads();
                half[hf] = L.byte[0] | L.byte[1] | L.byte[2] | L.byte[3];
            }
        } else {
            MaskTile<T, false> tile;
            tile.request(a, w);
            __syncthreads();
            const unsigned long long word = tile.finish(a, L.predict);
            half[0] = (unsigned)word;
            half[1] = (unsigned)(word >> 32);
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
//               loading waves per workgroup moved 35 GB/s where one moves 50).  The units of a round are dealt to the
//               workgroups one place further each round, so that all get as many activation parts as down parts (a counter
//               drawn from by atomics balanced no better, and the wait for its answer cost 1.5 us per unit; with all
//               activation parts first, rows of 16 KiB loaded a quarter slower, all reads falling on the same half of every
//               row);
//   waves 1..3  list the added neurons meanwhile, then move the tail rows that nothing overwrites (more neurons removed than
//               added; with several tokens wave 0 does).
// Lane l holds the same 16-byte pieces of every vector as in the activation role and sums in the same order.
//
// Several tokens (MODE kDots, kMfma): the masks were written by the launch before this one and x lies in LDS.  Wave 0 puts the
// activation vectors of the rows it writes (new, moved) into LDS and posts them there; waves 1..3 compute the activations
// while its next bundle is on its way, kDots as in ffn_up_role with the tokens dealt to the waves, kMfma with the matrix
// instruction and the order of ffn_up_mfma_tile_staged (the vectors of both rows are rows of one operand; the parts of the k
// range are dealt to the waves).  One wave alone took 6 us per bundle of 24 KiB and 8 tokens, as long as the link.
enum StepMode { kOneToken = 0, kDots = 1, kMfma = 2 };

// LDS of a loader behind its part of PlanLds: PostLds, x of the tokens, the activation vectors of `stage_rows` rows
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
constexpr int kStepXOff = (int)(kLoaderPlanLds + (sizeof(PostLds) + 15) / 16 * 16);
__host__ __device__ __forceinline__ int step_x_pitch(int d, int elem) { return d * elem + 16; }     // (16: the reads of 16 tokens
                                                                                                     //  fall on different banks)
// Early bundles (see cache_role): the forms that have them, the tiles of neurons whose first added one is asked for early (the first
// words of `firsts` threads, one tile per pair of loaders), and the first of the units dealt in turn that loader lw takes if it has
// none of the `early` tiles: a whole number of bundles before lw, so its part is lw % parts.
constexpr bool early_form(int ni, bool gate) { return ni > 2 && !gate; }
__host__ __device__ __forceinline__ int early_tiles(int added, int loaders, int firsts) {
    const int pairs = loaders / 2 < kWave ? loaders / 2 : kWave;
    return added * 2 >= loaders ? (pairs < firsts ? pairs : firsts) : 0;
}
__host__ __device__ __forceinline__ int first_unit(int lw, int parts, int tiles, unsigned long long early) {
    const int pair = lw / parts;
    return lw - parts * __builtin_popcountll(pair < tiles ? early & ((1ull << (pair & 63)) - 1ull) : early);
}
template <typename T, int NI, bool GLU, bool GATE, int MODE>
__device__ __forceinline__ void cache_role(const StepArgs& a, int wg, PlanLds& L, PostLds* post, unsigned char* lds_x) {
    using V = typename Vec<T>::type;
    constexpr int VE = Vec<T>::N;
    constexpr bool PAIRED = NI > 2;
    constexpr int GA = PAIRED ? (GLU ? 2 : 1) : (GLU ? 3 : 2);   // vectors of a unit at most
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
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
    if (wg == 0) stage_owners();
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
    // Early bundles (one token, low-rank predictor).  A loader decides the mask word of an early tile for itself, as soon as t is
    // there, and asks for the first neuron it adds: that is 2 us before all masks are known and its place in the list with them,
    // time in which the link did nothing.  The early tiles are the first words of the first threads' runs, one per loader (per pair
    // of them, who take a part each); which neurons they add follows from the masks, so every loader knows what the others have
    // taken.  What is read early holds up what the loader reads next, the masks, until it has arrived, so it is done where the
    // last step kept every loader busy.  us a step, without -> with, two timings in turn: OPT shape 55.9 -> 53.7 and 54.3 -> 52.5, eight
    // stacked layers from a graph 463 -> 448, Llama-2 shape from a graph 131.4 -> 130.8, 24 steps with the dynamic window 2816 -> 2781;
    // gated d = 4544 110.9 -> 109.1; fp32 gated d = 2048, F = 8192 74.7 -> 72.8, d = 4096 112.8 -> 110.4.  Rows of up to 2 KiB have 64
    // to 128 loaders and seldom as much to load, and there the code alone costs more than it gives: d = 736, 18 added 13.7 -> 14.9
    // (d = 1024, F = 8192, many added 21.1 -> 20.4).
    // Where a wait for the masks runs out the early bundle is given up.  Kept in registers through own_masks it cost most fp32 forms
    // and some gated ones a workgroup per compute unit, which shows where the predictor fills the chip or little is loaded: fp32,
    // without early bundles / kept / given up: gated d = 2048, F = 16384 96.2 / 98.4 / 94.2, with 3 added 39.0 / 42.1 / 38.4; plain
    // F = 32768 d = 640 44.6 / 46.8 / 44.3, d = 1288 59.1 / 59.4 / 55.9, d = 2304 79.4 / 80.7 / 77.0.
    // The gated forms are 67 to 86 KB of code, more than the 64 KB instruction cache of two compute units.  With the tile decided by
    // the predictor's own code (53 to 75 KB), which leaves the window's words to be read behind the bundle, most were slower all the
    // same: OPT shape 52.6 -> 53.0, Llama-2 shape 130.0 -> 131.2, fp32 d = 4096 80.3 -> 81.1.
    constexpr bool EARLY = MODE == kOneToken && early_form(NI, GATE);
    constexpr int PARTS = PAIRED ? 2 : 1;                         // loaders of a bundle
    const int tiles = EARLY ? early_tiles(cur.n_added, a.n_load, (nwords + wpt - 1) / wpt) : 0;
    const int mine = (wg - 1) / PARTS;                            // (wg >= 1)
    const bool has_early = wg > 0 && mine < tiles;
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
    unsigned long long adding = 0ull;                             // early tiles with added neurons
    // counts and list positions of the added and removed neurons; returns whether any thread is `missing` its words
    auto diff = [&](bool missing) -> bool {
        int pa = 0, pr = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            pa += __popcll(now[i] & ~prev[i]);
            pr += __popcll(prev[i] & ~now[i]);
        }
        const int v = (pr << 16) | pa, inc = wave_inclusive_scan(v, lane), ex = inc - v;         // (a wave counts at most 16384)
        const unsigned long long none = __any(missing) ? 1ull << 63 : 0ull;
        if constexpr (EARLY) {
            const unsigned long long adds = __ballot(lane < tiles && (now[0] & ~prev[0]) != 0ull);
            if (tid == 0) L.early = adds;
        }
        if (lane == kWave - 1) L.wave_tot[wave] = none | ((unsigned long long)(unsigned)(inc >> 16) << 32) | (unsigned)(inc & 0xffff);
        lds_barrier();
        if constexpr (EARLY) adding = L.early;
        unsigned long long before = 0, all = 0, flags = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const unsigned long long t = L.wave_tot[i];
            flags |= t;
            if (i < wave) before += t & ~(1ull << 63);
            all += t & ~(1ull << 63);
        }
        off_a = (int)(unsigned)before + (ex & 0xffff);
        off_r = (int)(unsigned)(before >> 32) + (ex >> 16);
        tot_a = (int)(unsigned)all;
        tot_r = (int)(unsigned)(all >> 32);
        return (flags >> 63) != 0;
    };
    // the added neurons q of [c0, c0 + kListItems) (the words come back from LDS: in registers they would be live through
    // the load loop)
    auto fill_ids = [&](int c0, int of, int at) {                // the words of thread `of`, whose first one has list position `at`
        int q = at - c0;
#pragma unroll 1
        for (int i = 0; i < wpt; ++i) {
            unsigned long long bits = L.add[of * wpt + i];
            while (bits) {
                if ((unsigned)q < (unsigned)kListItems) L.ids[q] = (uint16_t)((of * wpt + i) * 64 + __ffsll((long long)bits) - 1);
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
            if (it < full_pieces(NI) || off + it * 1024u < (unsigned)vec_bytes) store_through(p, off + it * 1024u, (unsigned)vec_bytes, v[it]);
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
    // ---- masks -> window -> id list -> first host read ----
    const int x_pieces = nvec * a.batch;
    V xs[MODE == kOneToken ? 1 : 16];
    bool missing = false;
    int asked = -1;                                              // neuron whose part is on its way already
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
        if constexpr (EARLY) {
            if (has_early) {                                     // uniform
                MaskTile<T> tile;
                tile.request(a, mine * wpt);
                const unsigned long long held = a.cur_set[(size_t)cur.set_par * a.ring_words + mine * wpt];
                tile.widen();
                if (await_t(a, L.predict, wg, stamp_now)) {
                    const unsigned long long bits = tile.finish(a, L.predict) & ~uniform(held);
                    if (bits) {
                        asked = __builtin_amdgcn_readfirstlane(mine * wpt * 64 + __ffsll((long long)bits) - 1);
                        if (wave == 0) request_host(asked, lw & 1);
                    }
                }
            }
        }
        unsigned p[8];
        const int w0 = tid * wpt, nw = max(0, min(wpt, nwords - w0));
        missing = !poll_words<8, !GATE>(a.m_words + (size_t)(wg & (kWordReps - 1)) * a.m_pitch + 2 * w0, 1, 2 * nw, stamp_now,
                                      a.polls, p);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i < nw) m[i] = ((unsigned long long)p[2 * i + 1] << 32) | p[2 * i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) now[i] = keep[i] | m[i];
    const bool none = diff(missing);
    if constexpr (MODE == kOneToken) {
        if (__builtin_expect(none, 0)) {                         // a wait ran out
            lds_barrier();
            if constexpr (EARLY) {                               // what was asked for early is given up: no register is held through this
                asked = -1;
#pragma unroll
                for (int g = 0; g < GA; ++g)
#pragma unroll
                    for (int it = 0; it < NI; ++it) hv[g][it] = V(0);
            }
            own_masks<T, NI, GATE>(a, L, wpt, m);
            if (wg == 0) stage_owners();                         // (their place has been used)
#pragma unroll
            for (int i = 0; i < 4; ++i) now[i] = keep[i] | m[i];
            diff(false);
        }
    }
    bool over = n - tot_r < 0 || n - tot_r + tot_a > capacity;
    if (__builtin_expect(over && a.shrink, 0)) {
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
        diff(false);
        over = fit < 0 || n - tot_r < 0 || n - tot_r + tot_a > capacity;
    }
    if (__builtin_expect(over, 0)) {                 // uniform: leave everything untouched
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
    // Early tiles with added neurons; the first neuron of each is taken, the others are dealt to the loaders in turn, in the first
    // round to those that have no early one.  (Nothing is taken early where the list does not go in one piece.)
    const unsigned long long early = EARLY && __builtin_amdgcn_readfirstlane(tot_a) <= kListItems ? uniform(adding) : 0ull;
    const int n_early = __popcll(early);
    const bool is_early = has_early && ((early >> mine) & 1ull);
    const int unit_first = first_unit(lw, PARTS, tiles, early);
    auto early_before = [&]() {                                   // ... of the threads below this one
        return wave == 0 ? (int)__builtin_amdgcn_mbcnt_hi((unsigned)(early >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)early, 0u)) : n_early;
    };
    // The word with the neuron of this loader's first unit is looked up by the thread that holds it (the neuron is its r-th bit);
    // the list is written while the first host read is on its way.
    {
        int r = unit_first / PARTS - (off_a - early_before());
        bool open = wg > 0 && r >= 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i < wpt) {
                const unsigned long long bits = now[i] & ~prev[i];
                L.rem[tid * wpt + i] = prev[i] & ~now[i];
                L.add[tid * wpt + i] = bits;
                const unsigned long long dealt = i == 0 && wave == 0 && ((early >> lane) & 1ull) ? bits & (bits - 1ull) : bits;
                const int c = __popcll(dealt);
                if (open && r < c) {
                    L.first_bits = dealt;
                    L.first_at = make_int2((tid * wpt + i) * 64, r);
                    open = false;
                }
                r -= c;
            }
        }
    }
    if (wave == 0) L.off[lane] = off_a;
    if (tid == 0) L.listed = 0;
    if constexpr (MODE != kOneToken)
        if (wg > 0 && tid == 0) post->seq = post->done = post->arrived = 0;
    lds_barrier();

    if (wg == 0) {
        // ---- deletion plan (see k_window_plan): holes = dead slots below n', fillers = live slots at or above it ----
        // Made here once and handed to the loaders as stamped words, which arrive before their first bundle does.  (Made by every
        // loader for itself, by the waves that do not load, it was known 1 us later with few rows; with more than 4096 rows,
        // ahead of the host reads, it kept them waiting for 14 us: a loader cannot look owners up behind a host read.)
        // (All of it by a wave and 64 slots at a time took 0.4 us each: 8700 rows 14 us, now 6.)
        int H = 0;
        if (tot_r > 0) {                                         // uniform
            // (Compact on purpose: one workgroup runs this once, so most of its time are instructions on their way to the cache.)
            constexpr int kRound = 8, kStaged = kPtrLds / kWave; // blocks of a wave at a time; blocks whose owners are staged
            static_assert(kStaged % (4 * kRound) == 0, "a round is staged as a whole or not at all");
            int far[kRound];                                     // owners past the staged ones, requested a round ahead
            auto request = [&](int b0) {
#pragma unroll
                for (int q = 0; q < kRound; ++q) far[q] = a.pointers[min((b0 + q * 4) * kWave + lane, capacity - 1)];
            };
            if (nblk > kStaged) request(kStaged + wave);
#pragma unroll 1
            for (int b0 = wave; b0 < nblk; b0 += 4 * kRound) {
                int id[kRound];
                if (b0 < kStaged) {                              // uniform
#pragma unroll
                    for (int q = 0; q < kRound; ++q) id[q] = L.ptr[(b0 + q * 4) * kWave + lane];
                } else {
#pragma unroll
                    for (int q = 0; q < kRound; ++q) id[q] = far[q];
                    request(b0 + 4 * kRound);
                }
                unsigned long long w[kRound];
#pragma unroll
                for (int q = 0; q < kRound; ++q) w[q] = L.rem[min((unsigned)id[q] >> 6, 1023u)];
                unsigned long long dead = 0ull;                  // of block b0 + 4 * lane
#pragma unroll
                for (int q = 0; q < kRound; ++q) {
                    const unsigned long long m = __ballot((unsigned)id[q] >= (unsigned)F || ((w[q] >> (id[q] & 63)) & 1ull));
                    dead = lane == q ? m : dead;
                }
                if (lane < kRound && b0 + lane * 4 < nblk) L.dead[b0 + lane * 4] = dead;
            }
            lds_barrier();
            // A thread counts the holes and fillers of consecutive granules (one, or up to four with more than 16384 rows) and,
            // behind a prefix sum, lists the holes.  Granules of 16 slots where that many threads are there: a thread takes 0.1
            // us a hole.
            const int gl = nblk <= 64 ? 4 : nblk <= 128 ? 5 : 6, g = 1 << gl;            // slots of a granule
            auto slots_below = [](int k) -> unsigned long long { return k <= 0 ? 0ull : k < 64 ? ~(~0ull << k) : ~0ull; };
            auto dead_in = [&](int i) -> unsigned long long { return L.dead[(i << gl) >> 6] >> ((i << gl) & 63); };
            auto holes_in = [&](int i) -> unsigned long long { return dead_in(i) & slots_below(min(n2 - (i << gl), g)); };
            auto fill_in = [&](int i) -> unsigned long long {
                return ~dead_in(i) & slots_below(min(n - (i << gl), g)) & ~slots_below(n2 - (i << gl));
            };
            const int per = (((n + g - 1) >> gl) + 255) >> 8, i_first = tid * per, i_end = min((n + g - 1) >> gl, i_first + per);
            int vh = 0, vf = 0, ph, pf, fillers;
#pragma unroll 1
            for (int i = i_first; i < i_end; ++i) {
                vh += __popcll(holes_in(i));
                vf += __popcll(fill_in(i));
            }
            block_exclusive_scan2<4, false>(vh, vf, L.wave_tot, &ph, &pf, &H, &fillers);
            const bool in_lds = H <= kHoleFew;                   // (longer lists go through memory)
#pragma unroll 1
            for (int i = i_first; i < i_end; ++i) {
                L.fill_before[i] = (uint16_t)pf;
                pf += __popcll(fill_in(i));
#pragma unroll 1
                for (unsigned long long bits = holes_in(i); bits; bits &= bits - 1) {
                    const int hole = (i << gl) + __ffsll((long long)bits) - 1;
                    if (__builtin_expect(in_lds, 1)) L.hole[ph] = (uint16_t)hole;
                    else a.hole_list[ph] = hole;
                    ++ph;
                }
            }
            if (in_lds) lds_barrier();
            else __syncthreads();
#pragma unroll 1
            for (int q = tid; q < tot_r; q += 256) {
                const int s = n2 + q;
                const unsigned long long fill = fill_in(s >> gl), self = 1ull << (s & (g - 1));
                int dst = kNoDst;
                if (fill & self) {
                    const int r = H - 1 - (L.fill_before[s >> gl] + __popcll(fill & (self - 1ull)));
                    if (r >= 0) dst = in_lds ? (int)L.hole[r] : a.hole_list[r];
                }
                word_store(a.plan_words + q, stamp_now, (unsigned)dst);
            }
        }

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

    if (loads && is_early) {
        const int w = mine * wpt, id = w * 64 + __ffsll((long long)uniform(L.add[w])) - 1;
        if (__builtin_expect(id != asked, 0)) request_host(id, lw & 1);              // (t did not come in time)
    } else if (loads && unit_first < PARTS * (tot_a - n_early)) {        // (below kListItems)
        const unsigned long long bits = L.first_bits;
        const int2 at = L.first_at;
        const int before = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(bits >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bits, 0u));
        const unsigned long long it = __ballot(((bits >> lane) & 1ull) && before == at.y);
        request_host(__builtin_amdgcn_readfirstlane(at.x) + __ffsll((long long)it) - 1, lw & (PARTS - 1));
    }
    if (wave > 0) {
        if (wave == 1) fill_ids(0, lane, L.off[lane]);           // (for the wave that loads)
        fill_ids(0, tid, off_a);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        if (lane == 0) __hip_atomic_fetch_add(&L.listed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }

    if constexpr (MODE != kOneToken) {
        {
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

    // ---- load and move ----
    const int new_step = cur.step + 1, nw = a.n_load;
    V xr[MODE == kOneToken ? NI : 1];                            // (behind the first host read: needed once that has arrived)
    auto load_x = [&]() {
        if constexpr (MODE == kOneToken) load_pieces(xr, (const char*)a.x);
    };
    if (wave == 0) load_x();
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
    // What was in the cache before this step does not change during the launch and is read through the scalar cache: a vector
    // load behind host reads takes as long as they do.  (s and id are uniform.)
    auto owner_of = [&](int s) -> int { return uniform_load(a.pointers + s); };
    // destination of the tail slot n' + q: its word is asked for behind the host read and arrives with it
    auto plan_word = [&](int q) -> unsigned long long { return q < tot_r ? word_load(a.plan_words + q) : 0ull; };
    // ... worked out by this wave alone (a wait that ran out): the place of the slot among the fillers, then the hole
    auto own_dst = [&](int q) -> int {
        auto dead_slots = [&](int b) -> unsigned long long {     // of block b
            const int id = a.pointers[min(b * kWave + lane, capacity - 1)];
            return __ballot((unsigned)id >= (unsigned)F || ((L.rem[min((unsigned)id >> 6, 1023u)] >> (id & 63)) & 1ull));
        };
        auto slots = [&](int b, int from, int to) -> unsigned long long {        // those of block b in [from, to)
            const int s = b * kWave + lane;
            return __ballot(s >= from && s < to);
        };
        const int s = n2 + q;
        if ((dead_slots(s >> 6) >> (s & 63)) & 1ull) return kNoDst;
        int above = 0;                                           // fillers above s: the lowest hole takes the last one
#pragma unroll 4
        for (int b = s >> 6; b <= (n - 1) >> 6; ++b) above += __popcll(~dead_slots(b) & slots(b, s + 1, n));
        for (int b = 0; b * kWave < n2; ++b) {
            unsigned long long h = dead_slots(b) & slots(b, 0, n2);
            const int c = __popcll(h);
            if (above < c) {
                for (; above > 0; --above) h &= h - 1;
                return b * kWave + __ffsll((long long)h) - 1;
            }
            above -= c;
        }
        return kNoDst;
    };
    auto dst_of = [&](int q, unsigned long long word) -> int {
        if (q >= tot_r) return kNoDst;
        for (int tries = 0; (unsigned)(word >> 32) != stamp_now && tries < a.polls; ++tries) word = word_load(a.plan_words + q);
        if (__builtin_expect((unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(word >> 32)) != stamp_now, 0)) return own_dst(q);
        return __builtin_amdgcn_readfirstlane((int)(unsigned)word);
    };
    if (wave == 0) {                                             // the list of the first piece
        while (__hip_atomic_load(&L.listed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < 3) __builtin_amdgcn_s_sleep(1);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    }
    // Lists longer than kListItems are gone through piece by piece.
    for (int c0 = 0; c0 < items; c0 += kListItems) {
        if (c0 > 0) {
            lds_barrier();
            fill_ids(c0, tid, off_a);
            lds_barrier();
        }
        const int n_a = min(max(tot_a - c0, 0), kListItems), n_r = min(max(tot_r - c0, 0), kListItems);     // of this piece
        const bool early_first = c0 == 0 && is_early;
        const int taken = c0 == 0 ? PARTS * n_early : 0, units = PARTS * n_a - taken;        // units dealt in turn
        const int only = max(n_r - n_a, 0);                      // rows that nothing overwrites
        if (MODE != kOneToken && wave > 0) work();
        if (wave == 0) {
            struct Unit {
                int i, part, nid, old_id;                        // item c0 + i
                float old_bias, new_bias, old_gate, new_gate;
                unsigned long long plan;
            };
            // (item of the dealt bundle j: behind it in the list are the early ones below)
            const int early_at = EARLY && ((early >> lane) & 1ull) ? L.off[lane] - early_before() : 0x7fffffff;
            auto make_item = [&](int i, int part, bool ask) {    // its numbers, and the requests for its bundle
                Unit r;
                r.part = part;
                r.i = i;
                const int s = n2 + c0 + r.i;
                r.nid = __builtin_amdgcn_readfirstlane((int)L.ids[r.i]);
                r.old_id = owner_of(s);
                r.old_bias = uniform_load(a.bias + s);
                r.new_bias = uniform_load(a.b + r.nid);
                if (ask) request_host(r.nid, r.part);
                request_row(s, r.part);                          // (also where nothing is moved: no branch around loads)
                r.plan = plan_word(c0 + r.i);
                r.old_gate = gate_of(r.old_id);
                r.new_gate = gate_of(r.nid);
                return r;
            };
            auto item_of = [&](int u) { return EARLY ? u / PARTS + __popcll(__ballot(early_at <= u / PARTS)) : u / PARTS; };
            int place = lw, round = -taken;
            if (early_first || unit_first < units) {             // (the bundle of the first piece was requested above)
                Unit cu = make_item(early_first ? __builtin_amdgcn_readfirstlane(L.off[mine]) : item_of(unit_first),
                                    lw & (PARTS - 1), c0 > 0);
                for (;;) {
                    const int s = n2 + c0 + cu.i;
                    const int dst = dst_of(c0 + cu.i, cu.plan);
                    const bool act = cu.part == 0, moves = dst != kNoDst;         // uniform over the wave
                    float mdu = 0.f, mdg = 0.f, hdu = 0.f, hdg = 0.f;
                    if (moves) {
                        store_row(dst, cu.part, mv);
                        if (act) partial_dots(mv, mdu, mdg);
                    }
                    store_row(s, cu.part, hv);
                    const Slot fresh = {s, cu.nid, cu.new_bias}, moved = {dst, cu.old_id, cu.old_bias};
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
                    if (more) nu = make_item(item_of(round + place), (round + place) & (PARTS - 1), true);
                    if (MODE == kOneToken && act) {
                        if (moves) finish_slot(dst, cu.old_id, cu.old_bias, mdu, mdg);
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
                load_x();
                for (int v = lw * 3 + wave - 1; v < (PAIRED ? 2 * only : only); v += 3 * nw) {
                    const int part = (PAIRED && v >= only) ? 1 : 0, i = n_a + v - part * only;
                    const int dst = dst_of(c0 + i, plan_word(c0 + i)), s = n2 + c0 + i;
                    if (dst == kNoDst) continue;
                    request_row(s, part);
                    const int id = owner_of(s);
                    const float bs = uniform_load(a.bias + s);
                    store_row(dst, part, mv);
                    if (part == 0) {
                        float pu, pg;
                        partial_dots(mv, pu, pg);
                        finish_slot(dst, id, bs, pu, pg);
                    }
                }
            }
        } else if (wave == 0) {
            for (int i = n_a + (nw - 1 - lw); i < n_a + only; i += nw) {         // (the last ones have had the fewest units)
                const int dst = dst_of(c0 + i, plan_word(c0 + i)), s = n2 + c0 + i;
                if (dst == kNoDst) continue;
                request_row(s, 0);
                if (PAIRED) load_pieces(hv[0], row_vec(s, GA));
                const int id = owner_of(s);
                const Slot r = {dst, id, uniform_load(a.bias + s)};
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

// The activation role reads megabytes that nothing needs before the down projection; read at once they hold up the predictor,
// whose few reads the host link waits for (x A published 3.9 to 6.2 us after the launch began instead of 2.2, Falcon and Llama-2
// shapes). So its waves begin when a mask word has been published, or after kActWaits reads of it at the latest.
constexpr int kActWaits = 64;
// ... but only where the load that follows is likely to take longer than they do, which the last step tells: bundles of `vectors`
// vectors at the rate of the link against all but the down vector of the rows in use at kLinkSlower times that rate.  (Else a
// step that adds nothing waits for nothing and reads then.) d = 4096, us a step at once / behind the predictor, (rows in use,
// added): (3414, 0) 31.2 / 37.0, (3504, 13) 36.1 / 37.7, (3617, 16) 41.1 / 39.4, (3812, 40) 48.3 / 44.1; gated (3217, 0) 33.9 /
// 41.0, (3343, 8) 39.3 / 42.8.
constexpr int kLinkSlower = 128;
__host__ __device__ __forceinline__ bool load_hides_activations(int added, int in_use, int vectors) {
    return added * vectors * kLinkSlower >= in_use * (vectors - 1);
}
template <int VECTORS>
__device__ __forceinline__ void await_predictor(const StepArgs& a, int block) {
    const int words = 2 * ((a.F + 63) >> 6);
    const unsigned long long* p = a.m_words + (size_t)(block & (kWordReps - 1)) * a.m_pitch + (unsigned)block % (unsigned)words;
    const StepCounts& cur = a.st->cur;
    if (cur.error || a.polls == 0 || !load_hides_activations(cur.n_added, cur.num_used, VECTORS)) return;
    const unsigned now = (unsigned)cur.step + 1u;
    __builtin_amdgcn_s_sleep(127);
    for (int tries = min(kActWaits, a.polls); tries > 0 && (unsigned)(word_load(p) >> 32) != now; --tries) __builtin_amdgcn_s_sleep(32);
    __builtin_amdgcn_s_sleep(40);
}

// The gate form stays at two workgroups per compute unit (LDS): rows of more than 4 KiB would leave room for three, whose
// predictors, all at once, hold up the loaders.  us a step from a graph, three / two: fp32 d = 1400, F = 18000 60.7 / 59.5, d = 2048,
// F = 18000 78.7 / 78.0; d = 4544, F = 18000 84.9 / 84.1; d = 4096, F = 11008 58.2 / 57.8; but fp32 d = 2304, F = 16000, where two have
// one round of predictors just full, 74.6 / 75.8.
constexpr int kGatePairNi = 6;
constexpr size_t kGatePairLds = 56 * 1024;           // more than a third of the 160 KiB of a compute unit
template <typename T, int NI, bool GLU, bool GATE>
__global__ __launch_bounds__(256, (step1_wgs_per_cu<NI, GLU>())) void k_step1(const StepArgs a) {
    constexpr size_t kRoles = sizeof(PlanLds) > sizeof(PredictLds) ? sizeof(PlanLds) : sizeof(PredictLds);
    __shared__ __align__(16) unsigned char lds[GATE && NI >= kGatePairNi && kRoles < kGatePairLds ? kGatePairLds : kRoles];
    const int block = blockIdx.x;
    if (block < a.n_pred) {
        if constexpr (GATE) gate_role<T, NI>(a, block, reinterpret_cast<unsigned*>(lds));
        else lowrank_role<T, NI, step1_wgs_per_cu<NI, GLU>()>(a, block, *reinterpret_cast<PredictLds*>(lds));
    } else if (block <= a.n_pred + a.n_load) {
        cache_role<T, NI, GLU, GATE, kOneToken>(a, block - a.n_pred, *reinterpret_cast<PlanLds*>(lds), nullptr, nullptr);
    } else {
        const int first = a.n_pred + a.n_load + 1;
        await_predictor<GLU ? 3 : 2>(a, block);
        ffn_up_role<T, NI, GLU, true>((const T*)a.matrix, a.bias, (const T*)a.x, a.h, a.d, 1, a.capacity, a.row_elems, a.spec,
                                      block - first, gridDim.x - first, a.pointers, a.gact, a.F, a.st);
    }
}

// The same for a batch of tokens or a pass of several, behind the launches of the predictor: bookkeeping (workgroup 0),
// loaders, and the activation stage over the rows in use - on the matrix cores (MFMA: fp16, d a multiple of 32), else one
// wave per row.  Dynamic LDS: step_batch_lds bytes.
// Registers (gfx950, as the compiler reports them): the loader role has more uniform values than the 106 scalar registers hold,
// 85 to 146 of them live in lanes of vector registers (k_step1: 76 to 171).  No vector register goes to memory, which would queue
// up behind the host reads; 17 of the 106 forms, all with the gate predictor, keep 36 bytes a lane there (k_step1: none).  The
// predictor is a template parameter for that reason: a kernel with both forms of the role spilled 169 to 246 scalar registers and
// was 82 to 106 KB of code (43 to 61 KB each by itself), more than the 64 KB instruction cache of two compute units.
template <typename T, int NI, bool GLU, bool GATE, bool MFMA, int WAVES>
__global__ __launch_bounds__(WAVES * 64, 1) void k_step_batch(const StepArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_step[];
    const int block = blockIdx.x;
    if (block <= a.n_load) {
        if (WAVES > 4 && threadIdx.x >= 256) return;             // (a barrier waits for the waves that are left)
        PlanLds& plan = *reinterpret_cast<PlanLds*>(smem_step);
        PostLds* post = reinterpret_cast<PostLds*>(smem_step + kLoaderPlanLds);
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
    const size_t most = loader > up ? loader : up;
    return most > sizeof(PlanLds) ? most : sizeof(PlanLds);          // (the bookkeeping workgroup)
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
// Waves of a workgroup of k_step_batch: 4, or 8 where the LDS of a loader (x of the tokens and staged rows) leaves room for fewer
// than three of them per compute unit.  The activation workgroups of the launch carry the same LDS, and four waves that read a
// row each reach a fraction of the bandwidth, which shows where few rows are added and the load does not cover them.  fp32 rows,
// us a step with 4 -> 8 waves (rows in use, rows added): d = 1288, 8 tokens: (9277, 0) 77.7 -> 57.0, (9578, 47) 88.3 -> 71.2,
// (13408, 477) 157.8 -> 156.9; d = 2048, gated, 8 tokens: (4699, 0) 71.8 -> 55.1, (6444, 304) 187.8 -> 187.1; d = 2048, 4 tokens:
// (6221, 0) 51.9 -> 43.2. With room for three workgroups four waves are better (d = 1288, 3 tokens, (929, 0): 25.7 against 26.6),
// with room for two eight in one (d = 1288, 8 tokens, (8614, 0): 60.9 against 62.5; d = 2048, 4 tokens, (7235, 0): 49.8 against
// 50.7).
// The matrix-core stage keeps 4: it is at least as fast as in a launch of its own.  Gated rows of more than 12 KiB a vector
// would spill registers at 8 waves.
constexpr int step_batch_most_waves(int ni, bool glu, bool mfma) { return mfma || ni <= 2 || (glu && ni > 12) ? 4 : 8; }
inline int step_batch_waves(int ni, bool glu, bool mfma, size_t lds) { return lds > kStepLdsLimit / 3 ? step_batch_most_waves(ni, glu, mfma) : 4; }

// A workgroup of eight waves keeps its compute unit to itself: beside another one of its activation workgroups a loader, and the
// bookkeeping workgroup that makes the deletion plan, are slower.  fp32, us a step with the LDS for one / for two per compute
// unit (rows in use, rows added): d = 836, gated, 6 tokens, (21805, 291) 115.9 / 121.1; fp16 d = 2664, 6 tokens, (4398, 61) 46.0
// / 46.8; but d = 1288, 8 tokens, (9585, 48) 70.7 / 67.6.
inline size_t step_batch_lds_launched(int waves, size_t lds) {
    return waves == 8 && lds <= kStepLdsLimit / 2 ? kStepLdsLimit / 2 + 1024 : lds;
}

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
        hipLaunchKernelGGL(waves == 4 ? few : many, dim3(grid), dim3(waves * 64), step_batch_lds_launched(waves, lds), s, a);                            \
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
