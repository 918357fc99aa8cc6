// Step 4, down projection of a single token (Section 3.3 item 3):  y[j] = sum_s h[s] * D[s][j]  over the rows in use.
//
// What bounds it: a few hundred to a few thousand 64-byte pieces per workgroup behind three dependent memory round
// trips (activations and row count -> down columns -> y), so latency first and the loads in flight per compute unit
// second.  A workgroup owns 64 bytes of every down column (d / 32 workgroups in fp16: about half the compute units) and
// has many waves, so that each wave compacts few slots and each thread has few rows, all of them in flight at once.
// Measured in a HIP graph on gfx950 (rows in use / rows with an activation, fp16, d = 4096; before = 4 waves per
// workgroup, partial sums and a second launch above 4096 rows or when every row is read):
//     1060 / 337    4.0 -> 3.6 us      1927 / 864    6.0 -> 4.2      4096 / 1366   9.0 -> 5.0
//     8000 / 2500  11.5 -> 8.6         1060, all rows read  7.2 -> 4.6         2977, all rows read  7.8 -> 6.3
// Slices of 32 or 128 bytes were slower at most sizes (half a line wasted per piece; too few workgroups).
#pragma once

#include <type_traits>

#include "lif_common.h"
#include "lif_ffn.h"

namespace lif {

constexpr int kDown1Lanes = 4;           // lanes per row: 64 bytes of its down column
constexpr int kDown1Per = 4;             // slots a thread compacts per pass
constexpr int kDown1FewRows = 2048;      // up to here one pass of 8 waves covers all rows
constexpr int kDown1OneSkip = 8192;      // one chunk up to here when rows without activation are skipped
constexpr int kDown1OneFull = 3584;      // ... when every row is read
constexpr int kDown1RowsSkip = 4096;     // rows per chunk beyond, for workgroups of 8 waves
constexpr int kDown1RowsFull = 1024;

// Row chunks in use for n cached rows and `slices` column slices.  One chunk (no partial sums) as long as
// d / 32 workgroups of 16 waves keep up with the rows: skipping rows, 8000 rows take 8.6 us in one chunk against 11.5 us in two
// chunks and the launch that added their sums then; reading every row (one whole call, OPT shape) 3072 rows 15.7 against 16.8, 3584 rows 17.3 either
// way, 4096 rows 18.7 in four chunks.
// Beyond, workgroups of 8 waves, several to a compute unit (with 16 waves one workgroup fills it, and what is left of the
// workgroups after 256 of them runs almost alone): us a call, 16 waves -> 8 waves, every row read: OPT shape 5120 rows 23.1 ->
// 21.7, 10240 rows 36.0 -> 32.7; Falcon shape 16384 rows 64.8 -> 56.7; skipping rows, Falcon shape, 10240 rows 27.5 -> 24.1.
// Skipping rows in two chunks, where workgroups of 16 waves just fill the compute units (down1_rows16), they are better: OPT
// shape, half of 10240 rows active, 27.5 against 28.7.
// rows up to which workgroups have 16 waves (from kDown1FewRows on): known before the row count is
template <bool SKIP>
__host__ __device__ __forceinline__ int down1_rows16(int slices) {
    return !SKIP ? kDown1OneFull : slices > 96 && slices <= 128 ? 2 * kDown1OneSkip : kDown1OneSkip;
}
template <bool SKIP>
__host__ __device__ __forceinline__ int down1_chunks(int n, int slices) {
    if (n <= (SKIP ? kDown1OneSkip : kDown1OneFull)) return 1;
    if (n <= down1_rows16<SKIP>(slices)) return 2;
    constexpr int per = SKIP ? kDown1RowsSkip : kDown1RowsFull;
    const int c = (n + per - 1) / per;
    return c < kDownChunksMax ? c : kDownChunksMax;
}

// Whether the sums of so many chunks are added by a launch of its own (see last_part): a workgroup that waits for its stores and its
// count keeps the next one out where there are many rounds of them, and beyond 16 sums the last workgroup of a slice goes through a third
// round trip.  us a call in a graph, the last workgroup of a slice -> a launch, every row read, fp16 unless it says fp32: d = 1024, 16 x 32
// workgroups 18.9 -> 19.2, 18 x 32 22.0 -> 21.55, 20 x 32 22.9 -> 22.5; d = 2048, 18 x 64 30.3 -> 30.2; d = 3072, 16 x 96 36.95 -> 37.05,
// 18 x 96 41.2 -> 40.5; fp32 d = 1288, 18 x 80 40.4 -> 39.7; d = 4096, 14 x 128 41.3 either way, 16 x 128 46.7 -> 46.5 (fp32 d = 2048 45.75
// -> 46.2), 18 x 128 59.4 -> 57.9; d = 5120, 10 x 160 39.9 -> 39.6, 12 x 160 45.4 either way, 14 x 160 61.4 -> 60.0, 20 x 160 93.1 -> 90.1;
// d = 8192, 8 x 256 46.8 -> 47.5, 10 x 256 68.7 -> 67.7, 20 x 256 127.9 -> 124.4.  Up to 8 chunks the last workgroup is 0.6 to 1.5 better at
// every width, every row read or not.
__host__ __device__ __forceinline__ bool down1_finish(int chunks, int slices) { return chunks > 16 || slices * chunks > 2048; }

// Waves of the summation order for n rows: a function of n and the width alone.  The slots are dealt to that many (virtual) waves,
// 64 consecutive slots at a time; every wave compacts its own slots with ballots into its own list, takes the list
// positions i with i mod 16 = row group in ascending order, folds its row groups, and the waves are added in order.  A
// workgroup launched with other than that many waves goes through the virtual waves in turn (or leaves some idle), so
// the result does not depend on the launch geometry.
template <bool SKIP>
__host__ __device__ __forceinline__ int down1_waves(int n, int slices) {
    return n > kDown1FewRows && n <= down1_rows16<SKIP>(slices) ? 16 : 8;
}

// grid = (column slices of 64 bytes, rounded up to a multiple of 8, + 1 after a fused step (FUSED): the workgroup that commits
// it; row-chunk workgroups), block = WAVES * 64.
// gact (may be null): the activations in h and h_new are up . x alone and are multiplied with the gate activation of the
// slot's neuron here (gate predictor; gact_n = number of neurons).
// spec: groups of WAVES * 64 slots whose activations are requested before the row count is known (the arrays span the
// capacity, so the addresses are valid; values past the count are masked).
// Workgroup row y takes the chunks y, y + gridDim.y, ...; with several chunks and several workgroup rows the sums go to
// ypart[chunk][d] (fp32) and the last workgroup of a slice (SHARED, last_part) or k_ffn_down_finish adds them, else every workgroup its
// own, in the same order.
// The same as a role of a larger launch (k_ffn_one): bx, by, rows_by take the place of blockIdx.x, blockIdx.y, gridDim.y, and
// WORDS is where the activations come from: `activations(s0, stride, count, v)` fills v[q] with those of the slots s0 + q *
// stride (q < count, different for every lane).
struct NoWords {};
template <typename T, bool SKIP, int WAVES, bool FUSED, bool SHARED, typename Words>
__device__ __forceinline__ void ffn_down1_role(const T* __restrict__ matrix, const float* __restrict__ h, const FusedRows& fused,
                                               T* __restrict__ y, float* ypart, unsigned* __restrict__ arrived, int d,
                                               int capacity, size_t row_elems, int down_off, int spec, int slices,
                                               const int32_t* __restrict__ pointers, const float* __restrict__ gact, int gact_n,
                                               DevState* __restrict__ st, int bx, int by, int rows_by, Words activations) {
    constexpr bool WORDS = !std::is_same<Words, NoWords>::value;
    using V = typename Vec<T>::type;
    constexpr int VE = Vec<T>::N, LANES = kDown1Lanes, PER = kDown1Per, THREADS = WAVES * 64;
    constexpr int WL = PER * 64;                     // list entries per wave and pass
    constexpr int RG = 64 / LANES;                   // row groups per wave
    constexpr int VWMAX = 16;
    __shared__ int list[WAVES][WL];
    __shared__ float hv[WAVES][WL];
    __shared__ float red[VWMAX][LANES][VE + 1];
    __shared__ int last;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, l = lane & (LANES - 1), rg = lane / LANES;
    // XCD-aware slice order: workgroups are dealt round-robin to the 8 XCDs, each with its own L2; giving every XCD a
    // contiguous run of slices makes the two halves of a 128-byte line meet in one L2 instead of being fetched twice
    if (FUSED && bx == slices) {
        if (by == 0) commit_step<THREADS>(fused, capacity, st);
        return;
    }
    const float* __restrict__ h_new = fused.h_new;
    const int32_t* __restrict__ stamp = FUSED ? fused.stamp : nullptr;
    const int per_xcd = slices / kXcds;
    const int slice = (bx % kXcds) * per_xcd + bx / kXcds;
    const int col = slice * (LANES * VE) + l * VE;
    const bool col_ok = col < d;
    const T* base = matrix + down_off + (col_ok ? col : 0);

    float hfirst[PER], hnfirst[PER];
    int sfirst[PER], ofirst[PER], onfirst[PER];      // o..: slot owners, only with gact
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        hfirst[q] = hnfirst[q] = 0.f;
        sfirst[q] = -1;
        ofirst[q] = onfirst[q] = 0;
    }
    const bool first_row = by == 0;
    if (!WORDS && first_row) {                               // (uniform branches around loads from clamped slots)
#pragma unroll
        for (int q = 0; q < PER; ++q)
            if (q < spec) hfirst[q] = h[min(q * THREADS + tid, capacity - 1)];
        if (stamp) {
#pragma unroll
            for (int q = 0; q < PER; ++q)
                if (q < spec) {
                    sfirst[q] = stamp[min(q * THREADS + tid, capacity - 1)];
                    hnfirst[q] = h_new[min(q * THREADS + tid, capacity - 1)];
                }
        }
        if (gact) {
#pragma unroll
            for (int q = 0; q < PER; ++q)
                if (q < spec) {
                    ofirst[q] = pointers[min(q * THREADS + tid, capacity - 1)];
                    if (stamp) onfirst[q] = fused.ptr_new[min(q * THREADS + tid, capacity - 1)];
                }
        }
    }
    const StepCounts* counts = stamp ? &st->next : &st->cur;
    const int err = counts->error, n = counts->num_used, cur_step = counts->step;
    if (err) return;
    const int chunks = down1_chunks<SKIP>(n, slices);
    if (by >= chunks) return;                        // uniform
    const int per_chunk = chunks == 1 ? n : (n + chunks - 1) / chunks;      // (no division on the shortest path)
    const int vwaves = down1_waves<SKIP>(n, slices);
    const int stride = vwaves * 64;                  // slots between the groups of a (virtual) wave
    int asked = vwaves == WAVES ? spec : 0;          // groups of these waves that the requests above were for
    if constexpr (WAVES == 16 && !WORDS) {
        // Few rows, which 8 of the waves take (one chunk): the others hold every second group of theirs, and hand it over in LDS.  Asked for
        // again it was another round trip behind the row count.  us, 16 waves launched, asked again -> handed over / 8 waves launched: a step
        // with the gate resident, d = 4096, 1992 rows 99.5 -> 99.15 / 98.9; low-rank, OPT shape, 1994 rows 80.9 -> 80.6 / 80.8; an FFN call
        // in a graph fp32 d = 2048, 1600 rows 7.2 -> 7.0 / 7.1, fp16 d = 4096 the same.
        if (n <= kDown1FewRows && spec > 0) {        // uniform
            constexpr int HALF = PER / 2;            // (groups of 1024 slots that hold 2048)
            float hq[HALF];
            int oq[HALF];
#pragma unroll
            for (int q = 0; q < HALF; ++q) {
                const bool fresh = stamp && sfirst[q] == cur_step;
                hq[q] = fresh ? hnfirst[q] : hfirst[q];
                oq[q] = fresh ? onfirst[q] : ofirst[q];
                if (wv >= 8) {
                    hv[wv][q * 64 + lane] = hq[q];
                    if (gact) list[wv][q * 64 + lane] = oq[q];
                }
            }
            lds_barrier();
#pragma unroll
            for (int q = 0; q < HALF; ++q) {
                hfirst[2 * q] = hq[q];
                hfirst[2 * q + 1] = hv[8 + (wv & 7)][q * 64 + lane];
                ofirst[2 * q] = oq[q];
                if (gact) ofirst[2 * q + 1] = list[8 + (wv & 7)][q * 64 + lane];
                sfirst[2 * q] = sfirst[2 * q + 1] = -1;
            }
            asked = min(PER, 2 * spec);
        }
    }
    double total = 0.0;
    for (int chunk = by; chunk < chunks; chunk += rows_by) {
        const int r0 = chunk * per_chunk, r1 = min(n, r0 + per_chunk);
        for (int vw = wv; vw < vwaves; vw += WAVES) {
            float acc[VE];
#pragma unroll
            for (int i = 0; i < VE; ++i) acc[i] = 0.f;
            int cnt = 0;                             // entries of this wave's list so far (uniform over the wave)
            int nz = 0;
            for (int s_base = r0; s_base < r1; s_base += PER * stride) {
                const int s0 = s_base + vw * 64 + lane;
                const int start = cnt;               // list position of the first entry of this pass
                const int need = min(PER, (r1 - s_base - vw * 64 + stride - 1) / stride);       // groups with rows in them
                const int have = first_row && s_base == 0 ? asked : 0;                          // ... requested at the start
                float hval[PER];
                int owner[PER];
#pragma unroll
                for (int q = 0; q < PER; ++q) {
                    const bool fresh = stamp && sfirst[q] == cur_step;
                    hval[q] = fresh ? hnfirst[q] : hfirst[q];
                    owner[q] = fresh ? onfirst[q] : ofirst[q];
                }
                if constexpr (WORDS) {
                    if (gact) {
#pragma unroll
                        for (int q = 0; q < PER; ++q) owner[q] = pointers[min(s0 + q * stride, capacity - 1)];
                    }
                    int count = 0;
#pragma unroll
                    for (int q = 0; q < PER; ++q) count += s0 + q * stride < r1;
                    activations(s0, stride, count, hval);
                } else if (need > have) {
#pragma unroll
                    for (int q = 0; q < PER; ++q)
                        if (q >= have && q < need) {
                            const int sc = min(s0 + q * stride, capacity - 1);
                            hval[q] = h[sc];
                            if (gact) owner[q] = pointers[sc];
                        }
                    if (stamp) {
#pragma unroll
                        for (int q = 0; q < PER; ++q) {
                            if (q >= have && q < need) {
                                const int sc = min(s0 + q * stride, capacity - 1);
                                const float hn = h_new[sc];
                                const int on = gact ? fused.ptr_new[sc] : 0;
                                if (stamp[sc] == cur_step) {
                                    hval[q] = hn;
                                    owner[q] = on;
                                }
                            }
                        }
                    }
                }
                if (gact) {
                    float g[PER];
#pragma unroll
                    for (int q = 0; q < PER; ++q) g[q] = (q < need) ? gact[min(max(owner[q], 0), gact_n - 1)] : 0.f;
#pragma unroll
                    for (int q = 0; q < PER; ++q) hval[q] = g[q] * hval[q];
                }
#pragma unroll
                for (int q = 0; q < PER; ++q) {
                    if (q < need) {                  // uniform over the wave
                        const int s = s0 + q * stride;
                        const float v = (s < r1) ? hval[q] : 0.f;
                        const bool nonzero = v != 0.f;
                        const bool take = SKIP ? nonzero : s < r1;
                        const unsigned long long m = __ballot(take);
                        if (take) {
                            const int pos = cnt + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                                                  __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
                            list[wv][pos - start] = s;
                            hv[wv][pos - start] = v;
                        }
                        cnt += __popcll(m);
                        nz += SKIP ? __popcll(m) : __popcll(__ballot(nonzero));
                    }
                }
                // (the list is this wave's alone and a wave's LDS operations complete in order: no barrier instruction)
                __builtin_amdgcn_wave_barrier();
                if (col_ok) {
                    // all row loads of a pass over kInFlight rows per thread are issued before the first use; a thread
                    // takes the list positions i with i mod RG = its row group, counted over the whole chunk
                    constexpr int kInFlight = 8;
                    const int first = start + ((rg - start) & (RG - 1));
                    for (int i0 = first; i0 < cnt; i0 += RG * kInFlight) {
                        V v[kInFlight];
#pragma unroll
                        for (int u = 0; u < kInFlight; ++u) {
                            const int i = i0 + u * RG;
                            const int sr = list[wv][(i < cnt ? i : i0) - start];
                            v[u] = (i < cnt) ? *reinterpret_cast<const V*>(base + (size_t)sr * row_elems) : V(0);
                        }
#pragma unroll
                        for (int u = 0; u < kInFlight; ++u) {
                            const int i = i0 + u * RG;
                            if (i < cnt) {
                                const float hb = hv[wv][i - start];
#pragma unroll
                                for (int e = 0; e < VE; ++e) acc[e] = __builtin_fmaf(hb, (float)v[u][e], acc[e]);
                            }
                        }
                    }
                }
                __builtin_amdgcn_wave_barrier();
            }
            if (slice == 0 && lane == 0 && nz) atomicAdd(&st->c_ffn_active, (unsigned long long)nz);     // statistics only
            constexpr int held = wave_fold_held<VE, LANES>();
            constexpr int dup = wave_fold_dup_mask<VE, LANES>();
            const int first = wave_fold<VE, LANES>(acc, lane);
            if ((lane & dup) == 0) {
#pragma unroll
                for (int i = 0; i < held; ++i) red[vw][l][first + i] = acc[i];
            }
        }
        __syncthreads();
        if (tid < LANES * VE) {                      // one column per thread, waves in order
            float part[VWMAX], sum = 0.f;            // (all of them asked for at once: a wait for each took 0.03 us)
#pragma unroll
            for (int w = 0; w < VWMAX; ++w) part[w] = red[w][tid / VE][tid % VE];
#pragma unroll
            for (int w = 0; w < VWMAX; ++w) sum = w < vwaves ? sum + part[w] : sum;
            const int oc = slice * (LANES * VE) + tid;
            if (chunks > 1 && rows_by > 1) {
                if (oc < d) store_part(ypart + (size_t)chunk * d + oc, sum);
            } else {
                total += (double)sum;                // 0 + first sum is exact
                if (chunk + rows_by >= chunks && oc < d) y[oc] = (T)total;
            }
        }
        if (chunk + rows_by < chunks) __syncthreads();       // (red is written again)
    }
    if (slice == 0 && tid == 0 && first_row) {
        atomicAdd(&st->c_ffn_calls, 1ull);
        atomicAdd(&st->c_ffn_rows, (unsigned long long)n);
    }
    if (chunks > 1 && rows_by > 1) {
        if (!SHARED || !last_part(arrived + slice * kArrivedPitch, min(chunks, rows_by), &last)) return;
        const int oc = slice * (LANES * VE) + tid * 4;
        if (tid < LANES * VE / 4 && oc < d) {        // four columns per thread
            double sum[4];
            sum_parts<8>(ypart, (unsigned)oc, (unsigned)d, chunks, sum);
#pragma unroll
            for (int e = 0; e < 4; ++e) y[oc + e] = (T)sum[e];
        }
    }
}

template <typename T, bool SKIP, int WAVES, bool FUSED, bool SHARED>
__global__ __launch_bounds__(WAVES * 64) void k_ffn_down1(const T* __restrict__ matrix, const float* __restrict__ h,
                                                          const FusedRows fused, T* __restrict__ y,
                                                          float* ypart, unsigned* __restrict__ arrived, int d, int capacity,
                                                          size_t row_elems, int down_off, int spec, int slices,
                                                          const int32_t* __restrict__ pointers,
                                                          const float* __restrict__ gact, int gact_n,
                                                          DevState* __restrict__ st) {
    ffn_down1_role<T, SKIP, WAVES, FUSED, SHARED>(matrix, h, fused, y, ypart, arrived, d, capacity, row_elems, down_off, spec, slices, pointers, gact,
                                          gact_n, st, blockIdx.x, blockIdx.y, gridDim.y, NoWords());
}

}  // namespace lif
