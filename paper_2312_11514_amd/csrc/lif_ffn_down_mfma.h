// Step 4, down projection for a batch of 2..8 tokens (fp16) on the matrix cores:
//   Y[t][j] = sum_s H[t][s] * D[s][j]      over the cached rows s that contribute (Section 3.3 item 3).
// With several tokens the vector units are the limit of the streaming form (k_ffn_down: 64 multiply-adds and 8 LDS
// reads per 16 bytes of a down column; measured at the Llama-2 shape, 8 tokens, 8700 rows: 9 us in the row loop,
// 5.6 us with the arithmetic taken out).  Here one v_mfma_f32_16x16x32_f16 covers K = 32 rows x N = 16 groups of
// columns x M = 16 token slots.  Memory is contiguous along the columns and the matrix instruction wants K (rows)
// packed per lane, so a lane loads 16 bytes (its 8 columns) of 8 rows and transposes the 8 x 8 block in its own
// registers (32 v_perm_b32); column j of the block feeds the j-th of eight accumulator tiles.
// The activations are fp32.  They enter as fp16 pairs: scaled by a power of two so that the largest of a pass is
// below 2^15 (exact), then split into a high and a low part (h * scale = hi + lo up to 2^-22 relative); token
// slots 0..7 of M carry the high parts of tokens 0..7, slots 8..15 their low parts, and the two halves of the
// result are added at the end of a pass.  Products are exact, accumulation is fp32.
#pragma once

#include "lif_ffn.h"

namespace lif {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int kDmRows = 512;             // rows compacted per pass
constexpr int kDmRowsFew = 256;          // ... where the whole cache in such pieces fits the chip at once
constexpr int kDmWgsAtOnce = 3 * 256;    // workgroups that do: three to a compute unit
constexpr int kDmSmall = 1280;           // capacity up to which passes are 512 rows all the same
constexpr int kDmCols = 128;             // columns per workgroup: 16 lanes x 16 bytes
constexpr int kDmWaves = 4;              // waves per workgroup: 8 are a little faster below 5000 rows (196 against 197 us for a
                                         // step of 4 tokens at 1250 rows) but leave two workgroups per compute unit and so a
                                         // second, nearly empty round of them above (24 against 19 us at 8600 rows)

// Rows per pass and per chunk (one partial output per chunk): functions of the capacity and the width alone, so a workgroup row
// knows where its first chunk starts before the row count arrives; a chunk is whole passes, and at most kDownChunksMax chunks are
// ever in use.  Passes of 256 rows have half the activations to wait for and twice the workgroups: one FFN call, us, 512 -> 256
// rows: d = 512, 3 tokens, 1835 rows 15.6 -> 13.3; d = 1024, 8 tokens, 6948 rows 19.8 -> 17.7; d = 4096, 8 tokens, 1674 rows 19.8
// -> 17.2. But where 256-row workgroups would need a second round on the chip 512 are better: d = 4096, 8 tokens, 8177 of 8192
// rows 33.9 against 37.2. (Chunks of 256 rows in passes made for 512 gain a third of it.) And small caches are likely to hold the
// 257 to 450 rows that one chunk of 512 takes without partial sums: d = 512, 2 tokens, 299 rows 12.1 against 12.9.
__host__ __device__ __forceinline__ int down_mfma_pass_rows(int capacity, int slices) {
    const int few = (capacity + kDmRowsFew - 1) / kDmRowsFew;
    return capacity > kDmSmall && few <= kDownChunksMax && few * slices <= kDmWgsAtOnce ? kDmRowsFew : kDmRows;
}
__host__ __device__ __forceinline__ int down_mfma_chunk_rows(int capacity, int slices) {
    const int rows = down_mfma_pass_rows(capacity, slices), per = rows * kDownChunksMax;
    const int passes = (capacity + per - 1) / per;
    return rows * (passes < 1 ? 1 : passes);
}
__host__ __device__ __forceinline__ int down_mfma_chunks(int n, int chunk_rows) {
    const int c = (n + chunk_rows - 1) / chunk_rows;
    return c < 1 ? 1 : c;
}

// Whether the chunk sums of that grid are added by a launch of its own (see last_part); told: chunks of the row-count hint, 0 without one
// and in a fused step.
// Of more workgroups than the chip holds at once one that waits for its stores and its count keeps the next one out: d = 5120, gated, 6
// tokens, 27 chunks, both stages 79.1 us with the launch, 80.1 to 80.4 with the last workgroup of a slice.  Else all workgroups end at about
// the same time, and what the last one of a slice then reads by itself, a sum per chunk and token, nothing hides: us a call, skipping, a launch
// against the last workgroup, means over d = 512 to 3072 and chunks of 256 and 512 rows, in a graph / submitted by the host: 8 tokens 32 chunks 0.7
// / 0.4 better (d = 1024, 16384 rows 22.4 -> 21.4), 17 to 24 chunks 0.45 / 0.15 better, 16 chunks 0.2 / 0.5 worse; 5 tokens 0.3 to 0.4 / 0.05 better
// from 17 on, 0.3 / 0.7 worse with 16; 4 tokens 0.15 to 0.3 better / 0.05 worse; 2 tokens the same / 0.35 worse.  d = 3584, 17 to 32 chunks
// 0.4 better in a graph; d = 4096 0.2 better skipping, the same with every row read, gated 0.3 worse (56.2 -> 56.5).  In a fused step the last
// workgroup is better: 8 tokens d = 1024, 22 chunks 74.75 against 75.8 us, d = 2048 74.45 against 75.5, the Llama-2 shape 226.1 against 228.7.
__host__ __device__ __forceinline__ bool down_mfma_finish(int wg_rows, int told, int slices, int batch) {
    return slices * wg_rows > kDmWgsAtOnce || (told > 16 && batch > 4 && slices < 32);
}

// Two fp16 values (one from each source register) packed into one: the low halves or the high halves.
// v_perm_b32 picks bytes out of {s0 = bytes 7..4, s1 = bytes 3..0}.
__device__ __forceinline__ unsigned pack_halves(unsigned second, unsigned first, bool high) {
    return high ? __builtin_amdgcn_perm(second, first, 0x07060302u) : __builtin_amdgcn_perm(second, first, 0x05040100u);
}

// What bounds it: HBM, about 5.5 TB/s for this access pattern, between a prologue of 5 us (activations, compaction) and the
// reductions.  All workgroups are resident at once (three per compute unit need at most 168 registers, which the launch
// bound asks for), so the prologue is not hidden by other workgroups; where every row is read it overlaps with the first
// quarter of the rows: 10976 rows, 8 tokens, d = 4096, gated, activations and down projection 63.3 -> 60.2 us.
// The sums of the waves and the two halves of the token slots meet in LDS as 16-byte pieces: by 32 lane exchanges and as many
// read-add-writes of 4 bytes per lane it took 2.0 us from the last row to the last sum, twelve waves sharing the LDS of a unit; now
// 0.7.  us, two timings in turn: d = 4096, gated, 8 tokens, 10989 rows, all read, both stages 58.0 -> 56.7 and 58.0 -> 56.8; 12 passes of
// 5 tokens, OPT shape, 2435 -> 2409 and 2349 -> 2327.
// grid = (ceil(d / 128) column slices, row-chunk workgroups), block = WAVES waves; lane l of a wave: column
// group n16 = l mod 16 (8 columns) and token slot n16, row block q = l div 16 (8 of the 32 rows of an instruction).
// A pass compacts the contributing rows of ROWS slots (SKIP: rows with some activation; else all rows in use) in a
// fixed order (thread-major over slots p * threads + tid); the waves take groups of 32 compacted rows in turn.
// The waves of a pass are added in wave order, a chunk's passes in order, the chunks in chunk order (by this kernel when
// one workgroup row is launched, else by the last workgroup of a slice from ypart[chunk][token][d] (SHARED, last_part), or by
// k_ffn_down_finish).  No sum depends on the launch geometry.
template <bool SKIP, int WAVES, int ROWS, bool FUSED, bool SHARED>
__global__ __launch_bounds__(WAVES * 64, 3) void k_ffn_down_mfma(const _Float16* __restrict__ matrix,
                                                              const float* __restrict__ h, const FusedRows fused,
                                                              _Float16* __restrict__ y, float* ypart,
                                                              unsigned* __restrict__ arrived, int d, int batch, int capacity,
                                                              size_t row_elems, int down_off, int chunk_rows, int slices,
                                                              DevState* __restrict__ st) {
    constexpr int BT = 8, T = WAVES * 64;
    constexpr int PER = ROWS / T;                    // slots per thread in the compaction
    constexpr int kPitch = ROWS + 8;                 // fp16 values per token slot in LDS (16 bytes of padding: lanes of one
                                                     // row block read 16 different slots at the same offset)
    static_assert(ROWS % T == 0 && BT * kDmCols == 4 * T, "whole slots and one column of four tokens per thread");
    __shared__ int list[ROWS];
    __shared__ __attribute__((aligned(16))) _Float16 hv[16][kPitch];
    __shared__ int wave_tot[WAVES];
    __shared__ float wave_max[WAVES];
    __shared__ f32x4 red[WAVES][8][64];              // per wave, column of a lane's 8, and lane: sums of four token slots
    __shared__ int n_active, last;

    if (FUSED && (int)blockIdx.x == slices) {
        if (blockIdx.y == 0) commit_step<WAVES * 64>(fused, capacity, st);
        return;
    }
    const float* __restrict__ h_new = fused.h_new;
    const int32_t* __restrict__ stamp = FUSED ? fused.stamp : nullptr;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int n16 = lane & 15, q = lane >> 4;
    const int col = blockIdx.x * kDmCols + n16 * 8;
    const bool col_ok = col < d;
    // (offsets in bytes from the uniform base: 65536 rows of 48 KiB stay below 4 GiB)
    const unsigned row_bytes = (unsigned)row_elems * 2u, col_bytes = (unsigned)(down_off + (col_ok ? col : 0)) * 2u;

    if (tid == 0) n_active = 0;
    // What a pass begins with is requested at the end of the one before, for the first one before the row count is known (the
    // arrays span the capacity; values past the rows in use are masked): its activations and, where every row is read, the
    // rows of the first group of each wave.
    float ha[PER][BT], hb[PER][BT];
    int fresh_at[PER];
    f16x8 v[8];
    // the rows of a group: 8 loads of 16 bytes per lane
    auto load = [&](int g, int cnt, auto slot) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int i = g * 32 + q * 8 + r;
            v[r] = *reinterpret_cast<const f16x8*>(reinterpret_cast<const char*>(matrix) + ((unsigned)slot(i < cnt ? i : 0) * row_bytes + col_bytes));
        }
    };
    auto request = [&](int s_base) {
#pragma unroll
        for (int p = 0; p < PER; ++p) {
            const unsigned s = min(s_base + p * T + tid, capacity - 1);
            fresh_at[p] = stamp ? stamp[s] : -1;
#pragma unroll
            for (int b = 0; b < BT; ++b) {
                ha[p][b] = b < batch ? (h + (size_t)b * capacity)[s] : 0.f;
                hb[p][b] = stamp && b < batch ? (h_new + (size_t)b * capacity)[s] : 0.f;
            }
        }
        asm volatile("" ::: "memory");       // (behind the activations: loads return in order)
        if constexpr (!SKIP) load(w, ROWS, [&](int i) { return min(s_base + i, capacity - 1); });
    };
    request(blockIdx.y * chunk_rows);
    const StepCounts* counts = stamp ? &st->next : &st->cur;
    const int err = counts->error, n = counts->num_used, cur_step = counts->step;
    if (err) return;
    const int chunks = down_mfma_chunks(n, chunk_rows);
    if ((int)blockIdx.y >= chunks) return;           // uniform

    const int oc = tid & (kDmCols - 1), og = tid / kDmCols, ocol = blockIdx.x * kDmCols + oc;     // this thread finishes column oc
    f32x4 total = {0.f, 0.f, 0.f, 0.f};                                                           //  of tokens 4 og .. 4 og + 3

    for (int chunk = blockIdx.y; chunk < chunks; chunk += gridDim.y) {
        const int r0 = chunk * chunk_rows, r1 = min(n, r0 + chunk_rows);
        f32x4 part = {0.f, 0.f, 0.f, 0.f};
        for (int s_base = r0; s_base < r1; s_base += ROWS) {
            // compaction of the rows that contribute and the largest |activation| of the pass
            unsigned flags = 0, nonzero = 0;
            float amax = 0.f;
#pragma unroll
            for (int p = 0; p < PER; ++p) {
                const int s = s_base + p * T + tid;
                bool any = false;
                const bool fresh = stamp && fresh_at[p] == cur_step;
#pragma unroll
                for (int b = 0; b < BT; ++b) {
                    const float a = s >= r1 ? 0.f : fresh ? hb[p][b] : ha[p][b];
                    ha[p][b] = a;
                    any |= (a != 0.f);
                    amax = fmaxf(amax, fabsf(a));
                }
                if (any) nonzero |= 1u << p;
                if (SKIP ? any : s < r1) flags |= 1u << p;
            }
            if (blockIdx.x == 0 && nonzero) atomicAdd(&n_active, __popc(nonzero));   // statistics only
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) amax = fmaxf(amax, __shfl_xor(amax, m, kWave));
            if (lane == 0) wave_max[w] = amax;       // (the barriers of the scan order this write and the reads below,
                                                     //  and keep the previous pass's readers of list / hv ahead of the writes)
            int cnt = min(r1 - s_base, ROWS), off = 0;
            if constexpr (SKIP) off = block_exclusive_scan<WAVES>(__popc(flags), wave_tot, &cnt);
            else __syncthreads();
            float smax = wave_max[0];
#pragma unroll
            for (int i = 1; i < WAVES; ++i) smax = fmaxf(smax, wave_max[i]);
            // power-of-two scale: the largest scaled activation lies in [2^14, 2^15)
            const bool scalable = smax > 0.f && smax < 3.0e38f;
            const int ex = scalable ? ilogbf(smax) : 14;
            const float scale = ldexpf(1.f, 14 - ex), inv_scale = ldexpf(1.f, ex - 14);
#pragma unroll
            for (int p = 0; p < PER; ++p) {
                if (!SKIP) off = p * T + tid;
                if (flags & (1u << p)) {
                    if (SKIP) list[off] = s_base + p * T + tid;
#pragma unroll
                    for (int b = 0; b < BT; ++b) {
                        const float hs = ha[p][b] * scale;
                        const _Float16 hi = (_Float16)hs;
                        hv[b][off] = hi;
                        hv[BT + b][off] = (_Float16)(hs - (float)hi);
                    }
                    ++off;
                }
            }
            // the matrix instruction reads whole groups of 32 rows: zero activations behind the last row
            if (tid < 32 && cnt + tid < ((cnt + 31) & ~31)) {
#pragma unroll
                for (int m = 0; m < 16; ++m) hv[m][cnt + tid] = (_Float16)0.f;
            }
            __syncthreads();
            if (smax > 0.f) {                        // uniform over the workgroup
                f32x4 acc[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
                auto compute = [&](int g) {
                    // this lane's token slot: activations of rows i0 .. i0 + 7
                    const f16x8 a = *reinterpret_cast<const f16x8*>(&hv[n16][g * 32 + q * 8]);
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        // column j of the 8 x 8 block: rows 2 r2 and 2 r2 + 1 packed into dword r2
                        u32x4 bj;
#pragma unroll
                        for (int r2 = 0; r2 < 4; ++r2) {
                            const u32x4 lo = __builtin_bit_cast(u32x4, v[2 * r2]), hi = __builtin_bit_cast(u32x4, v[2 * r2 + 1]);
                            bj[r2] = pack_halves(hi[j >> 1], lo[j >> 1], (j & 1) != 0);
                        }
                        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, __builtin_bit_cast(f16x8, bj), acc[j], 0, 0, 0);
                    }
                };
                // (rows past the last one are read as the first one, against activations of 0; a second register set that
                // requests the wave's next group ahead of the arithmetic was no faster at 1400 rows)
                auto row = [&](int i) { return SKIP ? list[i] : s_base + i; };
                if constexpr (SKIP) {
                    if (w * 32 < cnt) load(w, cnt, row);
                } else {
#pragma unroll
                    for (int r = 0; r < 8; ++r)
                        if (w * 32 + q * 8 + r >= cnt) v[r] = f16x8(0);      // (slots not in use hold anything)
                }
                for (int g = w; g * 32 < cnt;) {
                    compute(g);
                    g += WAVES;
                    if (g * 32 < cnt) load(g, cnt, row);
                }
                // The waves took different rows, and token slots 8..15 (lanes with q >= 2) hold the low-part products of tokens 0..7:
                // all of them are added through LDS, the waves in wave order.  (The 16-byte places of odd columns are swapped by
                // eight, so that the columns that a wave reads side by side fall on different banks.)
                auto place = [](int j, int l) { return l ^ ((j & 1) << 3); };
#pragma unroll
                for (int j = 0; j < 8; ++j) red[w][j][place(j, lane)] = acc[j];
                lds_barrier();
                f32x4 sum;
#pragma unroll
                for (int ww = 0; ww < WAVES; ++ww) {
                    const f32x4* from = red[ww][oc & 7];
                    const int l = og * 16 + (oc >> 3);
                    const f32x4 v = (from[place(oc, l)] + from[place(oc, l + 32)]) * inv_scale;
                    sum = ww ? sum + v : v;
                }
                part += sum;                         // (0 + first pass is exact)
            }
            const int next = s_base + ROWS < r1 ? s_base + ROWS
                                                   : chunk + (int)gridDim.y < chunks ? (chunk + (int)gridDim.y) * chunk_rows : -1;
            if (next >= 0) request(next);
        }
        if (chunks > 1 && gridDim.y > 1) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (og * 4 + r < batch && ocol < d) store_part(ypart + ((size_t)chunk * batch + og * 4 + r) * d + ocol, part[r]);
        } else {
            total += part;                           // chunk order; 0 + first sum is exact
        }
    }
    if (blockIdx.x == 0 && tid == 0) {
        if (blockIdx.y == 0) {
            atomicAdd(&st->c_ffn_calls, 1ull);
            atomicAdd(&st->c_ffn_rows, (unsigned long long)n);
        }
        if (n_active) atomicAdd(&st->c_ffn_active, (unsigned long long)n_active);
    }
    if (chunks == 1 || gridDim.y == 1) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (og * 4 + r < batch && ocol < d) y[(size_t)(og * 4 + r) * d + ocol] = (_Float16)total[r];
        return;
    }
    if (!SHARED || !last_part(arrived + blockIdx.x * kArrivedPitch, min(chunks, (int)gridDim.y), &last)) return;
    // four columns of a token per thread
    static_assert(BT * kDmCols == 4 * T, "one piece of every token and four columns");
    const int pt = tid / (kDmCols / 4), pc = blockIdx.x * kDmCols + tid % (kDmCols / 4) * 4;
    if (pt < batch && pc < d) {
        float sum[4];
        if (chunks > 24) sum_parts<16>(ypart, (unsigned)(pt * d + pc), (unsigned)(batch * d), chunks, sum);
        else sum_parts<8>(ypart, (unsigned)(pt * d + pc), (unsigned)(batch * d), chunks, sum);
        typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
        *reinterpret_cast<f16x4*>(y + (size_t)pt * d + pc) = f16x4{(_Float16)sum[0], (_Float16)sum[1], (_Float16)sum[2], (_Float16)sum[3]};
    }
}

}  // namespace lif
