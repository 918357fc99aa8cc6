// Step 4: FFN over the cached rows (Section 3.3 item 3):
//   y = sum_{s < num_used} relu(up_s . x + bias_s) * down_s        (gated: relu(gate_s . x + bias_s) * (up_s . x))
//
// Two kernels, both pure streaming of bundle bytes (1 flop per byte at fp16).  At the sizes of
// one decode token (10-60 MB) they run a few microseconds, so what counts is the number of
// dependent memory round trips; each kernel has two (state + first loads, then the rest).
//   ffn_up    one wave per cached row: all 16-byte loads of the row's up (and gate) vector are
//             issued before the first use; the wave reduces the dot product and writes the
//             activation h[s].
//   ffn_down  workgroups per slice of output columns (and per chunk of rows once the cache is large): no
//             atomics, fixed summation order.  It compacts the rows with a non-zero activation and
//             streams only their down columns: k_ffn_down1 (lif_ffn_down1.h) for one token,
//             k_ffn_down below for several tokens in fp32.
#pragma once

#include <type_traits>

#include "lif_common.h"
#include "lif_window_bits.h"

namespace lif {

// grid-stride over rows, one row per wave at a time; block = 256 by itself, 256 or 512 in k_step_batch.
// NI = 16-byte loads per lane and vector (ceil(d / (64 * VE))).
// XREG (batch 1): every lane keeps its fragments of x in registers, loaded straight from
// global memory.  Otherwise x is staged once per workgroup in LDS (dynamic LDS: batch * d
// elements) and re-read per token.
// spec != 0: the first row of every wave is requested before the row count is known (slot <
// capacity is always valid memory; the result is dropped if the slot is not in use), so the
// state, x and the first rows travel in one round trip.  The host only asks for this when it
// was told how many rows to expect and has sized the grid to that many waves.
// `block` / `nblocks`: index and count of the workgroups (of WAVES waves) that share this role.
// `gact` (may be null, plain bundles only): per-neuron gate activations relu(gate_i . x + b_i) written by the
// gate predictor (Appendix, Llama 2, "Alternative approaches": the resident gate projection is the predictor);
// the activation of slot s for token t is then gact[t][pointers[s]] * (up_s . x_t), gact [batch x gact_n];
// gact_n = d_ffn bounds the lookup.  A single token (XREG) leaves up_s . x and k_ffn_down1 multiplies: a fused step
// computes both in the same launch.
// `put(slot, activation)`, by the whole wave, takes the activations of a single token; without it they go to h.
template <typename T, int NI, bool GLU, bool XREG, int WAVES = 4, typename Put = int>
__device__ __forceinline__ void ffn_up_role(const T* __restrict__ matrix, const float* __restrict__ bias,
                                            const T* __restrict__ x, float* __restrict__ h, int d, int batch,
                                            int capacity, size_t row_elems, int spec, int block, int nblocks,
                                            const int32_t* __restrict__ pointers,
                                            const float* __restrict__ gact, int gact_n,
                                            const DevState* __restrict__ st, Put put = Put()) {
    using V = typename Vec<T>::type;
    constexpr int VE = Vec<T>::N;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    V* xs = reinterpret_cast<V*>(smem_raw);
    const int tid = threadIdx.x, lane = tid & 63;
    const int nvec = d / VE;
    const int gw = block * WAVES + (tid >> 6), nw = nblocks * WAVES;
    const V* xv = reinterpret_cast<const V*>(x);

    V xr[XREG ? NI : 1];
    if (XREG) {
#pragma unroll
        for (int it = 0; it < NI; ++it) {
            const int idx = it * 64 + lane;
            xr[it] = (idx < nvec) ? xv[idx] : V(0);
        }
    }
    // speculative first row
    V u[NI], g[GLU ? NI : 1];
    float bs = 0.f;
    if (spec) {
        const bool ok = gw < capacity;
        const V* row = reinterpret_cast<const V*>(matrix + (size_t)(ok ? gw : 0) * row_elems);
#pragma unroll
        for (int it = 0; it < NI; ++it) {
            const int idx = it * 64 + lane;
            const bool in = ok && idx < nvec;
            if (GLU) {
                g[it] = in ? row[idx] : V(0);
                u[it] = in ? row[nvec + idx] : V(0);
            } else {
                u[it] = in ? row[idx] : V(0);
            }
        }
        if (ok) bs = !gact ? bias[gw] : XREG ? 0.f : gact[min(max(pointers[gw], 0), gact_n - 1)];      // of token 0
    }
    const int err = st->cur.error;
    const int n = st->cur.num_used;
    if (err || block * WAVES >= n) return;           // whole workgroup has no row (uniform)

    if (!XREG) {
        for (int i = tid; i < batch * nvec; i += WAVES * 64) xs[i] = xv[i];
        __syncthreads();
    }

    if (!spec && gw < n) {                            // not requested yet: load now that the count is known
        const V* row = reinterpret_cast<const V*>(matrix + (size_t)gw * row_elems);
#pragma unroll
        for (int it = 0; it < NI; ++it) {
            const int idx = it * 64 + lane;
            const bool in = idx < nvec;
            if (GLU) {
                g[it] = in ? row[idx] : V(0);
                u[it] = in ? row[nvec + idx] : V(0);
            } else {
                u[it] = in ? row[idx] : V(0);
            }
        }
        bs = !gact ? bias[gw] : XREG ? 0.f : gact[min(max(pointers[gw], 0), gact_n - 1)];
    }
    for (int s = gw; s < n; s += nw) {
        // the next row of this wave is requested before the current one is reduced (when the grid is
        // smaller than the row count, every wave keeps two rows in flight)
        const int sn = s + nw;
        V un[NI], gn[GLU ? NI : 1];
        float bsn = 0.f;
        if (sn < n) {
            const V* row = reinterpret_cast<const V*>(matrix + (size_t)sn * row_elems);
#pragma unroll
            for (int it = 0; it < NI; ++it) {
                const int idx = it * 64 + lane;
                const bool in = idx < nvec;
                if (GLU) {
                    gn[it] = in ? row[idx] : V(0);
                    un[it] = in ? row[nvec + idx] : V(0);
                } else {
                    un[it] = in ? row[idx] : V(0);
                }
            }
            bsn = !gact ? bias[sn] : XREG ? 0.f : gact[min(max(pointers[sn], 0), gact_n - 1)];
        }
        for (int b = 0; b < (XREG ? 1 : batch); ++b) {
            float du = 0.f, dg = 0.f;
#pragma unroll
            for (int it = 0; it < NI; ++it) {
                const int idx = it * 64 + lane;
                if (XREG) {
                    du = dot_acc(u[it], xr[it], du);              // both are 0 past the end of the vector
                    if (GLU) dg = dot_acc(g[it], xr[it], dg);
                } else if (idx < nvec) {
                    const V xb = xs[b * nvec + idx];
                    du = dot_acc(u[it], xb, du);
                    if (GLU) dg = dot_acc(g[it], xb, dg);
                }
            }
            du = wave_sum(du);
            float act;
            if (GLU) {
                dg = wave_sum(dg);
                act = fmaxf(dg + bs, 0.f) * du;
            } else if (gact) {
                // resident gate: relu(gate . x_b + bias) from the predictor (bs holds token 0's)
                const float gb = b == 0 ? bs : gact[(size_t)b * gact_n + min(max(pointers[s], 0), gact_n - 1)];
                act = XREG ? du : gb * du;
            } else {
                act = fmaxf(du + bs, 0.f);
            }
            if constexpr (!std::is_same<Put, int>::value) put(s, act);
            else if (lane == 0) h[(size_t)b * capacity + s] = act;
        }
        if (sn < n) {
#pragma unroll
            for (int it = 0; it < NI; ++it) {
                u[it] = un[it];
                if (GLU) g[it] = gn[it];
            }
            bs = bsn;
        }
    }
}

template <typename T, int NI, bool GLU, bool XREG>
__global__ __launch_bounds__(256) void k_ffn_up(const T* __restrict__ matrix, const float* __restrict__ bias,
                                                const T* __restrict__ x, float* __restrict__ h, int d, int batch,
                                                int capacity, size_t row_elems, int spec,
                                                const int32_t* __restrict__ pointers, const float* __restrict__ gact,
                                                int gact_n, const DevState* __restrict__ st) {
    ffn_up_role<T, NI, GLU, XREG>(matrix, bias, x, h, d, batch, capacity, row_elems, spec, blockIdx.x, gridDim.x,
                                  pointers, gact, gact_n, st);
}

// After a fused step (k_step1, k_step_batch): the activations, slot owners and biases of the rows that it wrote, valid for the
// slots whose stamp is the number of that step.  All null otherwise.
struct FusedRows {
    const float* h_new;
    const int32_t* stamp;
    const int32_t* ptr_new;
    const float* bias_new;
    int32_t* pointers;               // where they are committed to
    float* bias;
    // a pass of several tokens: the masks of the first `keep` go into the ring
    const uint8_t* masks;            // [tokens x F / 8], null: the ring is up to date
    unsigned long long* ring;
    int ring_words, nbytes, k, keep;
};

// The end of a fused step, by one workgroup: counts, slot owners and biases.  The other workgroups of the launch read
// st->next and not what is written here.
template <int THREADS>
__device__ __forceinline__ void commit_step(const FusedRows& f, int capacity, DevState* st) {
    constexpr int PER = 4;
    const StepCounts nx = st->next;
    if (threadIdx.x == 0) st->cur = nx;
    if (nx.error) return;
    if (f.masks) {
        const int pos = nx.ring_pos - f.keep;                    // entry of the first kept token, modulo k
        for (int i = max(0, f.keep - f.k); i < f.keep; ++i) {
            unsigned long long* to = f.ring + (size_t)((((pos + i) % f.k) + f.k) % f.k) * f.ring_words;
            for (int w = threadIdx.x; w * 8 < f.nbytes; w += THREADS) to[w] = load_mask_word(f.masks + (size_t)i * f.nbytes, w, f.nbytes);
        }
    }
    for (int s0 = threadIdx.x; s0 < nx.num_used; s0 += PER * THREADS) {
        int stamp[PER], p[PER];
        float b[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int s = min(s0 + q * THREADS, capacity - 1);
            stamp[q] = f.stamp[s];
            p[q] = f.ptr_new[s];
            b[q] = f.bias_new[s];
        }
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int s = s0 + q * THREADS;
            if (s < nx.num_used && stamp[q] == nx.step) {
                f.pointers[s] = p[q];
                f.bias[s] = b[q];
            }
        }
    }
}

constexpr int kUpMaxWgs = 1024;   // workgroups of the activation stage: beyond this, waves loop over rows (x stays in registers)

constexpr int kXcds = 8;            // accelerator complex dies of an MI355X, each with a private L2
constexpr int kDownTile = 2048;     // activations (rows x tokens) compacted per pass (at least 512 rows)
constexpr int kDownChunksMax = 32;  // row chunks of the down projection (partial outputs per chunk)
constexpr int kDownLanesB = 16;       // lanes per column slice for several tokens
constexpr int kDownRowsMost = 512, kDownRowsLeast = 128;      // rows per chunk for several tokens
constexpr int kDownWgs = 512;         // workgroups that chunks of fewer than kDownRowsMost rows are made for

// Row chunks in use for n cached rows, several tokens and `slices` column slices: their active sets add up, most rows are read, and
// a chunk is at most kDownRowsMost rows: one chunk (no partial sums) up to there, beyond it chunks of down to
// kDownRowsLeast until kDownWgs workgroups stream at once.  With chunks of 512 rows throughout, half of the compute units had
// nothing to do and a thread went through 32 rows, four at a time.  One FFN call, us, 512 -> now: d = 1288, 3 tokens, 988 rows
// 14.5 -> 12.3, 2044 rows 16.1 -> 13.4, 4081 rows 18.9 -> 16.4; 8 tokens, 1634 rows 20.6 -> 17.4, 6859 rows 35.1 -> 33.9; d =
// 4096, 3 tokens, 949 rows 19.5 -> 17.3, 3874 rows the same.  Up to 512 rows one chunk is better
// (3 tokens, d = 1288, 208 rows 8.9 against 11.3).
// The host sizes the grid with the same rule.
__host__ __device__ __forceinline__ int down_chunks(int n, int slices) {
    const int least = (n + kDownRowsMost - 1) / kDownRowsMost, most = (n + kDownRowsLeast - 1) / kDownRowsLeast, fill = kDownWgs / slices;
    const int c = most < fill ? most : least > fill ? least : fill;
    return n <= kDownRowsMost ? 1 : (c > kDownChunksMax ? kDownChunksMax : c);
}

// Whether the sums of so many chunks are added by a launch of its own: the last workgroup of a slice goes through more than 24 of
// them in four round trips, the longer the more tokens there are, and many workgroups that wait keep others out.  us a call in a
// graph, skipping, the last workgroup -> a launch, means over 2048 to 16384 rows and, if not said, d = 256 to 2048: 32 chunks 5, 6, 8 tokens
// 0.95, 0.86, 0.80 better (d = 512, 8 tokens, 4096 rows 16.2 -> 15.3; submitted by the host 0.5 better), 3 and 4 tokens 0.2 worse, d = 4096 1.4
// better; 21 to 24 chunks 5 to 8 tokens the same, 2 to 4 tokens 0.5 to 0.9 worse; 16 chunks 0.6 to 1.5 worse.
// In a fused step the last workgroup adds them always: us a step, against a launch, 5 tokens, d = 1288, 27 chunks 151.4 / 153.65, 6 tokens, d =
// 1536, 31 chunks 162.1 / 164.8, 8 tokens, d = 1024, 32 chunks of 419 rows 93.8 / 94.4, of 219 rows 64.9 / 64.4, d = 256 45.3 / 44.8, 4 tokens, d =
// 4096 270.7 / 270.1.
__host__ __device__ __forceinline__ bool down_finish(int chunks, int slices, int batch) {
    return chunks > 24 && (batch > 4 || slices * chunks > 1024);
}

// Where several workgroup rows of a down projection share the row chunks, their sums meet in the launch that forms them: each
// writes the sums of its chunks to ypart[chunk][token][d] and counts itself in at its column slice, and the last one to do so adds the
// slice's sums in chunk order.  Nobody waits.  The sums are written and read past the caches, so that an acknowledged store is
// where every XCD reads it and no fence is needed (the last workgroup behind __threadfence(), which writes back and invalidates
// the L2, was twice as slow as a launch that adds them).  The count wraps to 0 by itself, whatever launches have been before.
// us a pass, a launch of its own for these sums -> here, two timings in turn: 8 tokens of the Llama-2 shape 229.7 -> 226.8 (the launch
// took 4.6, the down projection now 0.5 more), 12 passes of 5 tokens 2300 -> 2286, fp32 d = 1288, 3 tokens, four calls 68.6 -> 67.4;
// 10989 rows all read, 8 tokens, d = 4096, 22 chunks, both stages 56.8 -> 56.5; one FFN call of few chunks 0.5 to 0.9 (2 tokens, d =
// 2048, 8 chunks 11.7 -> 10.8; fp32, 3 tokens, d = 1024, 16 chunks 12.8 -> 11.8).  16 chunks asked for at a time are better from 25
// on (8 at a time -> 16, fp16: 26 chunks, 2 tokens, d = 1024 14.4 -> 13.6, d = 2048 17.8 -> 17.05, d = 3072 22.4 -> 21.6; 27 chunks, 2
// tokens, d = 1024 19.9 -> 19.1; 32 chunks, 8 tokens, d = 1024 21.7 -> 21.1, d = 3072 39.6 -> 39.0; 4 tokens, d = 2560 40.1 -> 39.4), 8
// below (18 and 24 chunks, d = 1024, 8 tokens 13.65 -> 13.9 and 14.4 -> 14.65, 5 tokens 13.2 -> 13.1 and 13.8 -> 14.05, 2 tokens 0.1 to
// 0.3 better with 16; the 22 chunks above 56.6 -> 56.9).  In fp32 16 at a time cost a resident wave: 8 always.
// SHARED: the kernel form that does so.  A grid of one workgroup row has nothing to add, and where a launch of its own is better
// (down1_finish, down_finish, down_mfma_finish) k_ffn_down_finish adds: there the form without the code and its registers is taken.
// These rules go by the rows that a hint tells.  Without one the grid is made for the capacity, of which few rows may be in use, and
// then a third launch costs more than it gives: us a call, the last workgroup / a launch, 8 tokens, d = 1024, 1203 of 8192 rows 10.6 /
// 12.7, in a graph 9.6 / 10.8, fp32 14.1 / 15.8; one token, d = 4096, 283 of 20000 rows, every row read, 8.9 / 12.3.
constexpr int kArrivedPitch = 32;     // counters of two slices are this many words apart: a cache line
// (Also where a later launch reads them: with plain stores there 8 tokens, d = 1024, 16384 rows took 22.3 us instead of 21.4.)
__device__ __forceinline__ void store_part(float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// Whether this workgroup is the last of `parts` whose sums of a slice are written (uniform; `flag` is in LDS)
__device__ __forceinline__ bool last_part(unsigned* arrived, int parts, int* flag) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // this wave's stores are acknowledged,
    __syncthreads();                                             // and those of the others
    if (threadIdx.x == 0) *flag = (int)atomicInc(arrived, (unsigned)parts - 1u) == parts - 1;
    __syncthreads();
    return *flag != 0;
}
// sum[e] = the four floats from ypart[at + c * stride + e] on (at and stride multiples of 4), added over the chunks c in order; PER of
// them are asked for at a time, the next ones ahead of the adds
template <int PER, typename A>
__device__ __forceinline__ void sum_parts(const float* ypart, unsigned at, unsigned stride, int chunks, A (&sum)[4]) {
    const unsigned bytes = stride * (unsigned)chunks * 4u;
    auto request = [&](f32x4 (&v)[PER], int c0) {
#pragma unroll
        for (int i = 0; i < PER; ++i) v[i] = load_through(ypart, (at + (unsigned)min(c0 + i, chunks - 1) * stride) * 4u, bytes);
    };
#pragma unroll
    for (int e = 0; e < 4; ++e) sum[e] = 0;
    f32x4 now[PER], next[PER];
    request(now, 0);
#pragma unroll 1
    for (int c0 = 0; c0 < chunks; c0 += PER) {
        if (c0 + PER < chunks) request(next, c0 + PER);
#pragma unroll
        for (int i = 0; i < PER; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] = c0 + i < chunks ? sum[e] + (A)now[i][e] : sum[e];
#pragma unroll
        for (int i = 0; i < PER; ++i) now[i] = next[i];
    }
}

// Down projection  y[t][j] = sum_s H[t][s] * D[s][j]  over the rows in use, for 2..BT tokens (fp32 layers; fp16
// batches run on the matrix cores, single tokens in k_ffn_down1).
// grid = (column slices, row-chunk workgroups), block = 256 = (256 / LANES) row groups x LANES lanes; a
// lane owns 16 bytes of every down column it reads, a workgroup LANES * 16 contiguous bytes.
// SKIP: rows whose activation is zero for every token of the batch are not read (they are compacted
// away with a prefix sum in LDS, in a fixed order).
// FUSED: the launch after k_step_batch.  One more workgroup commits the step and the activations of fresh rows are picked
// up; a form of its own because the run-time test cost the plain call 0.2 to 0.6 us of 17 (2 to 5 tokens, d 400 to 2800).
// The rows are cut into down_chunks chunks - a function of n and the width alone, so the arithmetic does not
// depend on the launch geometry - and workgroup row y takes the chunks y, y + gridDim.y, ...  Every
// chunk is summed from zero.  With one chunk in use the workgroup writes its columns of y.  With more,
// a grid of one workgroup row adds its chunk sums in chunk order and writes y; of a taller grid the last workgroup of a slice
// (SHARED, last_part) or k_ffn_down_finish adds them in the same order, in fp64: every chunk would be another rounding of the whole
// (3 tokens in fp32, d = 320: 1.43e-7 from the sum in fp64 against 1.60e-7).
template <typename T, int BT, bool SKIP, int LANES, bool FUSED, bool SHARED>
__global__ __launch_bounds__(256) void k_ffn_down(const T* __restrict__ matrix, const float* __restrict__ h,
                                                  const FusedRows fused, T* __restrict__ y,
                                                  float* ypart, unsigned* __restrict__ arrived, int d, int batch,
                                                  int capacity, size_t row_elems, int down_off, int slices,
                                                  DevState* __restrict__ st) {
    static_assert(BT > 1, "single tokens: k_ffn_down1");
    using V = typename Vec<T>::type;
    constexpr int VE = Vec<T>::N;
    constexpr int RG = 256 / LANES;                  // row groups per workgroup
    constexpr int TS = (kDownTile / BT < 512) ? 512 : kDownTile / BT;      // rows per compaction pass
    constexpr int PER = TS / 256;                    // slots per thread in the compaction
    static_assert(LANES * 16 >= 128, "a slice covers whole L2 lines");
    __shared__ int list[TS];
    __shared__ float hv[BT][TS];
    __shared__ int wave_tot[4];
    __shared__ float red[4][LANES][BT * VE];
    __shared__ int n_active, last;

    if (FUSED && (int)blockIdx.x == slices) {
        if (blockIdx.y == 0) commit_step<256>(fused, capacity, st);
        return;
    }
    const float* __restrict__ h_new = fused.h_new;
    const int32_t* __restrict__ stamp = FUSED ? fused.stamp : nullptr;
    const int tid = threadIdx.x, l = tid & (LANES - 1), rg = tid / LANES;
    const int slice = blockIdx.x;
    const int col = slice * (LANES * VE) + l * VE;
    const bool col_ok = col < d;
    const T* base = matrix + down_off + (col_ok ? col : 0);

    if (tid == 0) n_active = 0;
    // the first workgroup row requests the activations of its first pass before the row count is known
    // (the activation array spans the whole capacity, so the addresses are valid; values past
    // num_used are masked below): one memory round trip less on the critical path
    const bool first_row = blockIdx.y == 0;
    float hfirst[PER][BT], hnfirst[PER][BT];
    int sfirst[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        sfirst[q] = -1;
#pragma unroll
        for (int b = 0; b < BT; ++b) hfirst[q][b] = hnfirst[q][b] = 0.f;
    }
    if (first_row) {
#pragma unroll
        for (int q = 0; q < PER; ++q)
            if (stamp) sfirst[q] = stamp[min(q * 256 + tid, capacity - 1)];
#pragma unroll
        for (int b = 0; b < BT; ++b) {
            if (b < batch) {
#pragma unroll
                for (int q = 0; q < PER; ++q) {
                    hfirst[q][b] = h[(size_t)b * capacity + min(q * 256 + tid, capacity - 1)];
                    if (stamp) hnfirst[q][b] = h_new[(size_t)b * capacity + min(q * 256 + tid, capacity - 1)];
                }
            }
        }
    }
    const StepCounts* counts = stamp ? &st->next : &st->cur;
    const int err = counts->error, n = counts->num_used, cur_step = counts->step;
    if (err) return;
    const int chunks = down_chunks(n, slices);
    if ((int)blockIdx.y >= chunks) return;           // uniform
    const int per_chunk = (n + chunks - 1) / chunks;
    const int ob = tid / LANES, ol = tid - ob * LANES;            // (token, lane) whose 16-byte piece this thread writes
    const int ocol = slice * (LANES * VE) + ol * VE;
    const bool writer = tid < LANES * BT && ocol < d && ob < batch;
    double total[VE];
#pragma unroll
    for (int e = 0; e < VE; ++e) total[e] = 0.0;

    for (int chunk = blockIdx.y; chunk < chunks; chunk += gridDim.y) {
        const int r0 = chunk * per_chunk, r1 = min(n, r0 + per_chunk);
        float acc[BT * VE];                          // acc[b * VE + e]: token b, element e of this lane's 16 bytes
#pragma unroll
        for (int i = 0; i < BT * VE; ++i) acc[i] = 0.f;
        __syncthreads();
        for (int s_base = r0; s_base < r1; s_base += TS) {
            // compaction of the rows that contribute, in a fixed order (thread-major over slots q * 256 + tid)
            float hloc[PER][BT];
            unsigned flags = 0, nonzero = 0;
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const int s = s_base + q * 256 + tid;
                bool any = false;
                const bool ahead = s_base == 0;              // only chunk 0 (first workgroup row) starts at row 0
                const bool fresh = stamp && (ahead ? sfirst[q] : s < r1 ? stamp[s] : -1) == cur_step;
                const float* from = fresh ? h_new : h;
#pragma unroll
                for (int b = 0; b < BT; ++b) {
                    float v = 0.f;
                    if (s < r1 && b < batch) {
                        if (ahead) v = fresh ? hnfirst[q][b] : hfirst[q][b];
                        else v = from[(size_t)b * capacity + s];
                    }
                    hloc[q][b] = v;
                    any |= (v != 0.f);
                }
                if (any) nonzero |= 1u << q;
                if (!SKIP) any = s < r1;
                if (any) flags |= 1u << q;
            }
            if (slice == 0 && nonzero) atomicAdd(&n_active, __popc(nonzero));   // statistics only
            int cnt;
            int off = block_exclusive_scan<4>(__popc(flags), wave_tot, &cnt);
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                if (flags & (1u << q)) {
                    list[off] = s_base + q * 256 + tid;
#pragma unroll
                    for (int b = 0; b < BT; ++b) hv[b][off] = hloc[q][b];
                    ++off;
                }
            }
            __syncthreads();
            if (col_ok) {
                // all row loads of a pass over kInFlight rows per thread are issued before the first use (a loop with a
                // run-time trip count would wait for every load in turn); the adds stay in ascending row order
                constexpr int kInFlight = 4;
                for (int i0 = rg; i0 < cnt; i0 += RG * kInFlight) {
                    V v[kInFlight];
#pragma unroll
                    for (int u = 0; u < kInFlight; ++u) {
                        const int i = i0 + u * RG;
                        const int s = list[i < cnt ? i : i0];
                        v[u] = (i < cnt) ? *reinterpret_cast<const V*>(base + (size_t)s * row_elems) : V(0);
                    }
#pragma unroll
                    for (int u = 0; u < kInFlight; ++u) {
                        const int i = i0 + u * RG;
                        if (i < cnt) {
#pragma unroll
                            for (int b = 0; b < BT; ++b) {
                                const float hb = hv[b][i];
#pragma unroll
                                for (int e = 0; e < VE; ++e)
                                    acc[b * VE + e] = __builtin_fmaf(hb, (float)v[u][e], acc[b * VE + e]);
                            }
                        }
                    }
                }
            }
            __syncthreads();
        }
        // the row groups of one wave sit LANES lanes apart: halving butterfly over the upper lane bits (a lane
        // ends with a few finished sums), then LDS over waves
        {
            constexpr int held = wave_fold_held<BT * VE, LANES>();
            constexpr int dup = wave_fold_dup_mask<BT * VE, LANES>();
            const int first = wave_fold<BT * VE, LANES>(acc, tid & 63);
            if (((tid & 63) & dup) == 0) {
#pragma unroll
                for (int i = 0; i < held; ++i) red[tid >> 6][l][first + i] = acc[i];
            }
        }
        __syncthreads();
        if (writer) {
            float sum[VE];
#pragma unroll
            for (int e = 0; e < VE; ++e)
                sum[e] = ((red[0][ol][ob * VE + e] + red[1][ol][ob * VE + e]) + red[2][ol][ob * VE + e]) +
                         red[3][ol][ob * VE + e];
            if (chunks > 1 && gridDim.y > 1) {
                const unsigned at = ((unsigned)chunk * batch + ob) * d + ocol;
#pragma unroll
                for (int e = 0; e < VE; ++e) store_part(ypart + at + e, sum[e]);
            } else {
#pragma unroll
                for (int e = 0; e < VE; ++e) total[e] += (double)sum[e];
            }
        }
    }
    if (slice == 0 && tid == 0) {
        if (first_row) {
            atomicAdd(&st->c_ffn_calls, 1ull);
            atomicAdd(&st->c_ffn_rows, (unsigned long long)n);
        }
        if (n_active) atomicAdd(&st->c_ffn_active, (unsigned long long)n_active);
    }
    if (chunks > 1 && gridDim.y > 1) {
        if (!SHARED || !last_part(arrived + slice * kArrivedPitch, min(chunks, (int)gridDim.y), &last)) return;
        if (writer) sum_parts<8>(ypart, (unsigned)(ob * d + ocol), (unsigned)(batch * d), chunks, total);
    }
    if (writer) {
        V out;
#pragma unroll
        for (int e = 0; e < VE; ++e) out[e] = (T)total[e];
        *reinterpret_cast<V*>(y + (size_t)ob * d + ocol) = out;
    }
}

// y = sum of the chunk partials in chunk order, rounded once to the element type: the launch behind a down projection whose
// workgroups do not add them themselves.  Does nothing when a single chunk was in use (y is written already).  CHUNKS(n, by) is the
// chunk rule of that kernel; A: the type it adds in.  The partials of the first `ahead` chunks, which its grid had workgroup rows for,
// are requested before the row count is known; behind it they cost another round trip.  (Straight code: branches for each of them
// were 0.5 us of instructions that run once.)  grid = ceil(batch * d / 256), block = 256.
template <typename T, typename A, int (*CHUNKS)(int, int)>
__global__ __launch_bounds__(256) void k_ffn_down_finish(const float* ypart, T* __restrict__ y, int d, int batch, int by, int ahead,
                                                         const DevState* st) {
    const int i = blockIdx.x * 256 + threadIdx.x, stride = batch * d;
    const float* p = ypart + min(i, stride - 1);
    const int err = st->cur.error, n = st->cur.num_used;
    float v[kDownChunksMax];
#pragma unroll
    for (int c = 0; c < kDownChunksMax; ++c) v[c] = p[min(c, ahead - 1) * stride];         // (beyond: lines that are on their way already)
    asm volatile("" ::: "memory");                   // (the compiler would ask for them, and for the count, where they are used)
    if (err) return;
    const int chunks = CHUNKS(n, by), here = min(ahead, chunks);
    if (chunks == 1) return;
    A sum = 0;
#pragma unroll
    for (int c = 0; c < kDownChunksMax; ++c) sum = c < here ? sum + (A)v[c] : sum;
#pragma unroll 1
    for (int c = ahead; c < chunks; ++c) sum += (A)p[c * stride];                          // more rows in use than the hint let expect
    if (i < stride) y[i] = (T)sum;
}

}  // namespace lif
