// Step 1: low-rank predictor  mask_i = [ ((x A) B)_i + c_i > theta ]
// (Section 3.1 "Anticipating ReLU Sparsity", Fig. 3b; active = strictly positive output).
//
// Both contractions accumulate in fp64: every product of two fp16 or two fp32 values is
// exact in fp64, so the result depends on the summation order only at the 1e-16 level
// and the thresholded bits can be compared bit for bit with a CPU evaluation.  The path
// stays bandwidth bound (one fp64 FMA per 2 or 4 bytes read).
//
// Both kernels are a few microseconds long, i.e. latency bound: each issues all of its
// global loads (weights, offsets, state) before the first dependent use.
#pragma once

#include <type_traits>

#include "lif_common.h"

namespace lif {

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// acc[r] + sum_q a[r][q] * b[q] with every product and sum in fp64, for R rows at a time.  A product of two fp16 values is exact in
// fp32 (22 significant bits, exponents far inside the fp32 range), so for fp16 it is formed there and widened once: the same bits
// as widening both factors, at half the conversions.  One instruction forms it, which the compiler does not use by itself (a
// product of -0 becomes +0, which changes no sum that begins with +0).
// The compiler is held to the order products, conversions, sums: left to itself it has every sum wait for its own conversion.
__device__ __forceinline__ void in_order() { __builtin_amdgcn_sched_barrier(0x94); }      // (scalar, memory and LDS operations may pass)
template <int R>
__device__ __forceinline__ void dot_f64(const f16x8 (&a)[R], f16x8 b, double (&acc)[R]) {
    float p[R][8];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int q = 0; q < 8; q += 2) {
            const f16x2 ap = {a[r][q], a[r][q + 1]}, bp = {b[q], b[q + 1]};
            asm("v_fma_mix_f32 %0, %1, %2, 0 op_sel_hi:[1,1,0]" : "=v"(p[r][q]) : "v"(ap), "v"(bp));
            asm("v_fma_mix_f32 %0, %1, %2, 0 op_sel:[1,1,0] op_sel_hi:[1,1,0]" : "=v"(p[r][q + 1]) : "v"(ap), "v"(bp));
        }
    in_order();
    double w[R][8];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int q = 0; q < 8; ++q) w[r][q] = (double)p[r][q];
    in_order();
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r] += w[r][q];
    in_order();
}
template <int R>
__device__ __forceinline__ void dot_f64(const f32x4 (&a)[R], f32x4 b, double (&acc)[R]) {
    double w[R][4], x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        x[q] = (double)b[q];
#pragma unroll
        for (int r = 0; r < R; ++r) w[r][q] = (double)a[r][q];
    }
    in_order();
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r] = __builtin_fma(w[r][q], x[q], acc[r]);
    in_order();
}
template <typename V>
__device__ __forceinline__ double dot_f64(V a, V b, double acc) {
    const V row[1] = {a};
    double sum[1] = {acc};
    dot_f64<1>(row, b, sum);
    return sum[0];
}

constexpr int kMaskCols = 8;       // mask bytes (groups of 8 neurons) per workgroup of predict_mask
constexpr int kMaskJg = 32;        // rank groups per workgroup of predict_mask
constexpr int kMaskRows = 8;       // rows of B a thread keeps in flight

// t[j] = x . row j of At (the first predictor matrix with the contraction dimension contiguous, [r x d]) by a workgroup of four
// waves: wave w takes the 1 KiB pieces [w * P, w * P + P), P = ceil(NI / 4) of NI = ceil(d / (64 * VE)), in fp64, and the four
// sums are added in wave order.  A whole row per wave took 1.8 us from the last load to the sum at d = 4096 in fp16: a conversion
// and a dependent fp64 add for each of 64 products, one wave to a SIMD (k_step1, x A known after 3.1 us instead of 2.3).
template <typename T, int NI>
struct ColumnPart {
    using V = typename Vec<T>::type;
    static constexpr int P = (NI + 3) / 4;
    V a[P], x[P];
    static __device__ __forceinline__ int piece(int it) { return (threadIdx.x >> 6) * P + it; }
    static __device__ __forceinline__ void load(V (&v)[P], const T* p, int nvec) {
#pragma unroll
        for (int it = 0; it < P; ++it) {
            const int idx = piece(it) * 64 + (threadIdx.x & 63);
            v[it] = (piece(it) < NI && idx < nvec) ? reinterpret_cast<const V*>(p)[idx] : V(0);
        }
    }
    // this wave's part of the sum, in every lane
    __device__ __forceinline__ double sum() const {
        double acc = 0.0;
#pragma unroll
        for (int it = 0; it < P; ++it) acc = dot_f64(a[it], x[it], acc);
        return wave_sum(acc);
    }
};
// the parts of the four waves
__device__ __forceinline__ double column_total(const double (&part)[4]) { return ((part[0] + part[1]) + part[2]) + part[3]; }

// t[b][j] for every token and column: complete after this kernel, so the mask kernel needs no partial sums.
// grid = (r, batch), block = 256.
template <typename T, int NI>
__global__ __launch_bounds__(256) void k_predict_xa(const T* __restrict__ x, const T* __restrict__ At,
                                                    double* __restrict__ t, int d, int r,
                                                    const DevState* __restrict__ st) {
    __shared__ double part[4];
    const int j = blockIdx.x, b = blockIdx.y, nvec = d / Vec<T>::N;
    ColumnPart<T, NI> c;
    c.load(c.a, At + (size_t)j * d, nvec);
    c.load(c.x, x + (size_t)b * d, nvec);
    const int err = st->cur.error;
    const double v = c.sum();
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0 && !err) t[(size_t)b * r + j] = column_total(part);
}

// The sums v[e] of neurons 8 cl + e over a thread's ranks -> the sum over the eight rank groups of the wave, which sit 8 lanes
// apart: every exchange leaves a lane with half of its neurons, in the end with neuron 8 cl + fold_owner(lane).
__device__ __forceinline__ double fold_groups(double (&v)[8], int lane) {
    const bool up = (lane & 8) != 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const double send = up ? v[e] : v[e + 4], keep = up ? v[e + 4] : v[e];
        v[e] = keep + dpp_from<0x128, 0xf>(send);    // lanes 8 apart: a rotation in a row of 16
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) v[e] = swap_add<16>(v[e], v[e + 2]);
    return swap_add<32>(v[0], v[1]);
}
__device__ __forceinline__ int fold_owner(int lane) { return ((lane >> 3) & 1) * 4 + ((lane >> 4) & 1) * 2 + (lane >> 5); }

// logits = t B + c, threshold, 64 mask bits at a time; step mask = OR over the batch.
// grid = ceil(F / 64), block = 256 = 32 rank groups x 8 column lanes; a column lane owns 8 consecutive neurons.  A thread adds
// its ranks jg, jg + 32, ... in that order, then come the rank groups of a wave (fold_groups), then the waves: the one order of a
// logit, which MaskTile in k_step1 keeps too.  Past the last rank both t and B are 0 (t may be infinite, and 0 x infinity is no
// number).
// MANY: several tokens at a rank of one chunk; their t and the sums of the waves lie in LDS (dynamic, mask_lds_bytes). Else one
// token, and t comes straight from memory with the rows of B. (Several tokens and more chunks: k_predict_mask_long.)
// What bounds it: the chain from the launch over one round trip for B and t, 64 fp64 multiply-adds per thread and token, and the
// sums across the rank groups; a few hundred KB to a few MB are read.  A token at a time, with B widened once: the code is 2 KB
// instead of 10, and instructions that run once wait for their way into the cache (8 tokens at once, rank 256: 8.1 us).  The sums
// across a wave go through register exchanges that leave a lane with one neuron, so that a ballot is the mask word.  8 tokens,
// rank 256: 10.4 -> 7.5 us; 5 tokens, rank 128, 9.5 -> 6.1 us; 3 tokens in fp32, rank 68, 6.6 -> 5.2 us (all tokens at once,
// exchanges through LDS, sums and bits by 64 threads).
constexpr int kMaskChunk = kMaskRows * kMaskJg;      // ranks at a time
inline size_t mask_lds_bytes(int r, int tokens) { return sizeof(double) * (tokens * ((size_t)r + 4 * 64) + 1); }
template <typename T, bool MANY>
__global__ __launch_bounds__(256, 1) void k_predict_mask(const T* __restrict__ B, const float* __restrict__ c,
                                                      const double* __restrict__ t, int r, int F, int batch, float theta,
                                                      uint8_t* __restrict__ masks, uint8_t* __restrict__ step_mask,
                                                      const DevState* __restrict__ st) {
    using V = typename Vec<T>::type;
    constexpr int VE = Vec<T>::N;
    constexpr int LPB = 8 / VE;             // 16-byte loads per group of 8 neurons
    extern __shared__ __attribute__((aligned(16))) double lds_mask[];
    __shared__ double red_one[MANY ? 1 : 4 * 64];
    __shared__ unsigned long long ors[4];
    double* const red = MANY ? lds_mask : red_one;   // [token][wave][neuron of the tile]
    double* const tl = lds_mask + batch * (4 * 64);  // [token][r], then a 0

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int cl = tid & (kMaskCols - 1), jg = tid >> 3;
    const int n0 = (blockIdx.x * kMaskCols + cl) * 8, own = blockIdx.x * 64 + lane;
    const bool col_ok = n0 < F;
    const int mask_stride = F >> 3, byte = blockIdx.x * kMaskCols + lane;                // lanes 0..7: a mask byte each
    const int nb = MANY ? batch : 1;
    V bv[kMaskRows][LPB];
    double tr[MANY ? 1 : kMaskRows];
    auto request = [&](int j0) {                     // the rows j0 + jg + u * kMaskJg of B (0 past the end)
#pragma unroll
        for (int u = 0; u < kMaskRows; ++u) {
            const int j = j0 + jg + u * kMaskJg;
#pragma unroll
            for (int q = 0; q < LPB; ++q)
                bv[u][q] = (col_ok && j < r) ? reinterpret_cast<const V*>(B + (size_t)j * F + n0)[q] : V(0);
            if constexpr (!MANY) tr[u] = j < r ? t[j] : 0.0;
        }
    };
    request(0);
    const float cv = (c && own < F) ? c[own] : 0.f;      // (widened where it is used: here that would wait for it)
    const int err = st->cur.error;

    if constexpr (MANY) {
        // t of the tokens is one contiguous run: 16-byte pieces, several of them in flight per thread
        constexpr int kAhead = 4;
        typedef double f64x2 __attribute__((ext_vector_type(2)));
        const int pieces = nb * r / 2;               // (r is even)
        const f64x2* src = reinterpret_cast<const f64x2*>(t);
        for (int i0 = tid; i0 < pieces; i0 += 256 * kAhead) {
            f64x2 p[kAhead];
#pragma unroll
            for (int i = 0; i < kAhead; ++i) p[i] = src[min(i0 + i * 256, pieces - 1)];
#pragma unroll
            for (int i = 0; i < kAhead; ++i)
                if (i0 + i * 256 < pieces) reinterpret_cast<f64x2*>(tl)[i0 + i * 256] = p[i];
        }
        if (tid == 0) tl[nb * r] = 0.0;
        __syncthreads();
    }
    double bd[kMaskRows][8];
    auto widen = [&]() {
#pragma unroll
        for (int u = 0; u < kMaskRows; ++u)
#pragma unroll
            for (int e = 0; e < 8; ++e) bd[u][e] = (double)bv[u][e / VE][e % VE];
    };
    double v[8];                                     // logit sums of the 8 neurons of this lane's byte
    auto multiply = [&](const double (&tn)[kMaskRows]) {
#pragma unroll
        for (int u = 0; u < kMaskRows; ++u)
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = __builtin_fma(tn[u], bd[u][e], v[e]);         // (0 past the last rank)
    };
    const int at = wave * 64 + cl * 8 + fold_owner(lane);
    if constexpr (MANY) {
        widen();
        double ahead[kMaskRows];                     // of the next token
        int from[kMaskRows];                         // where they lie (past the last rank: at the 0 behind all tokens)
#pragma unroll
        for (int u = 0; u < kMaskRows; ++u) from[u] = jg + u * kMaskJg < r ? jg + u * kMaskJg : nb * r;
        auto read_t = [&]() {
#pragma unroll
            for (int u = 0; u < kMaskRows; ++u) {
                ahead[u] = tl[from[u]];
                from[u] += jg + u * kMaskJg < r ? r : 0;
            }
        };
        read_t();
#pragma unroll 1
        for (int bt = 0; bt < nb; ++bt) {
            double tn[kMaskRows];
#pragma unroll
            for (int u = 0; u < kMaskRows; ++u) tn[u] = ahead[u];
            if (bt + 1 < nb) read_t();
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = 0.0;
            multiply(tn);
            red[bt * 256 + at] = fold_groups(v, lane);
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = 0.0;
        for (int j0 = 0; j0 < r; j0 += kMaskChunk) {
            double tn[kMaskRows];
            widen();
#pragma unroll
            for (int u = 0; u < kMaskRows; ++u) tn[u] = tr[u];
            if (j0 + kMaskChunk < r) request(j0 + kMaskChunk);
            multiply(tn);
        }
        red[at] = fold_groups(v, lane);
    }
    __syncthreads();
    unsigned long long or_word = 0ull;               // of this wave's tokens
    for (int bt = wave; bt < nb; bt += 4) {
        const double* p = red + bt * 256 + lane;
        double z = ((p[0] + p[64]) + p[128]) + p[192];
        z += (double)cv;
        const unsigned long long word = __ballot(own < F && z > (double)theta);
        or_word |= word;
        if (lane < kMaskCols && byte < mask_stride && !err) masks[(size_t)bt * mask_stride + byte] = (uint8_t)(word >> (8 * lane));
    }
    if (lane == 0) ors[wave] = or_word;
    __syncthreads();
    if (tid < kMaskCols && byte < mask_stride && !err)
        step_mask[byte] = (uint8_t)(((ors[0] | ors[1]) | (ors[2] | ors[3])) >> (8 * lane));
}

// The same for several tokens at more than kMaskChunk ranks.  A thread's sums have to stay apart from the other rank groups'
// until its last rank, so they stay in registers for NT tokens at a time (the batch at most; tokens past it are worked for and
// left out). A row of B is widened once for all of them and asked for again, a chunk on, as soon as it is used; t goes through
// LDS a chunk ahead.
// lif_predict, us, d = 4096, F = 16384, against folding every chunk and adding the folded sums (another order): fp16, 8 tokens,
// rank 512 16.5 -> 13.8, 768 25.3 -> 18.3, 2048 64.8 -> 41.5; 2 tokens, rank 2048 22.8 -> 23.1; fp32, 3 tokens, rank 512 14.8 ->
// 14.6.
template <typename T, int NT>
__global__ __launch_bounds__(256, 1) void k_predict_mask_long(const T* __restrict__ B, const float* __restrict__ c,
                                                              const double* __restrict__ t, int r, int F, int batch, float theta,
                                                              uint8_t* __restrict__ masks, uint8_t* __restrict__ step_mask,
                                                              const DevState* __restrict__ st) {
    using V = typename Vec<T>::type;
    constexpr int VE = Vec<T>::N, LPB = 8 / VE;
    __shared__ double tl[2][NT][kMaskChunk];
    __shared__ double red[NT][4][64];
    __shared__ unsigned long long ors[4];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int cl = tid & (kMaskCols - 1), jg = tid >> 3;
    const int n0 = (blockIdx.x * kMaskCols + cl) * 8, own = blockIdx.x * 64 + lane;
    const bool col_ok = n0 < F;
    const int mask_stride = F >> 3, byte = blockIdx.x * kMaskCols + lane;
    V bv[kMaskRows][LPB];
    double td[NT];
    auto request_row = [&](int u, int j0) {
        const int j = j0 + jg + u * kMaskJg;
#pragma unroll
        for (int q = 0; q < LPB; ++q)
            bv[u][q] = (col_ok && j < r) ? reinterpret_cast<const V*>(B + (size_t)j * F + n0)[q] : V(0);
    };
    auto request_t = [&](int j0) {                   // (0 past the end, and for the tokens past the last one)
#pragma unroll
        for (int bt = 0; bt < NT; ++bt) td[bt] = (bt < batch && j0 + tid < r) ? t[(size_t)bt * r + j0 + tid] : 0.0;
    };
    auto stage_t = [&](int buf) {
#pragma unroll
        for (int bt = 0; bt < NT; ++bt) tl[buf][bt][tid] = td[bt];
    };
    request_t(0);
#pragma unroll
    for (int u = 0; u < kMaskRows; ++u) request_row(u, 0);
    const float cv = (c && own < F) ? c[own] : 0.f;      // (widened where it is used: here that would wait for it)
    const int err = st->cur.error;
    double v[NT][8];
#pragma unroll
    for (int bt = 0; bt < NT; ++bt)
#pragma unroll
        for (int e = 0; e < 8; ++e) v[bt][e] = 0.0;
    stage_t(0);
    for (int j0 = 0, buf = 0; j0 < r; j0 += kMaskChunk, buf ^= 1) {
        __syncthreads();                             // (also: nobody reads the other half of tl any more)
        const bool more = j0 + kMaskChunk < r;       // uniform
        if (more) request_t(j0 + kMaskChunk);
#pragma unroll
        for (int u = 0; u < kMaskRows; ++u) {
            double bd[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) bd[e] = (double)bv[u][e / VE][e % VE];
            if (more) request_row(u, j0 + kMaskChunk);
#pragma unroll
            for (int bt = 0; bt < NT; ++bt) {
                const double tj = tl[buf][bt][jg + u * kMaskJg];
#pragma unroll
                for (int e = 0; e < 8; ++e) v[bt][e] = __builtin_fma(tj, bd[e], v[bt][e]);
            }
        }
        if (more) stage_t(buf ^ 1);
    }
#pragma unroll
    for (int bt = 0; bt < NT; ++bt) red[bt][wave][cl * 8 + fold_owner(lane)] = fold_groups(v[bt], lane);
    __syncthreads();
    unsigned long long or_word = 0ull;
    for (int bt = wave; bt < batch; bt += 4) {
        double z = ((red[bt][0][lane] + red[bt][1][lane]) + red[bt][2][lane]) + red[bt][3][lane];
        z += (double)cv;
        const unsigned long long word = __ballot(own < F && z > (double)theta);
        or_word |= word;
        if (lane < kMaskCols && byte < mask_stride && !err) masks[(size_t)bt * mask_stride + byte] = (uint8_t)(word >> (8 * lane));
    }
    if (lane == 0) ors[wave] = or_word;
    __syncthreads();
    if (tid < kMaskCols && byte < mask_stride && !err)
        step_mask[byte] = (uint8_t)(((ors[0] | ors[1]) | (ors[2] | ors[3])) >> (8 * lane));
}

// pieces of 1 KiB that every vector served by this NI has in full (NI in 1, 2, 4, 6, 8, 9, 12, 16: the least that covers a vector)
constexpr int full_pieces(int ni) { return ni <= 1 ? 0 : ni <= 2 ? 1 : ni <= 4 ? 2 : ni <= 6 ? 4 : ni <= 8 ? 6 : ni <= 9 ? 8 : ni <= 12 ? 9 : 12; }

// relu(gate_i . x + b_i) and the mask bits of the 8 neurons of a mask byte by one wave, x in registers (0 past the end).
// Two rows are worked on side by side, piece by piece; the registers of a piece are asked for again, for the piece kGateAhead further
// (of these rows or the next two), as soon as its products are formed.  The sums of four rows cross the wave together, in the tree of
// wave_sum: lanes 1, 2, 4 apart, then 8, 16, 32; at 8 and 16 the rows of a lane are halved.
// What bounds it: HBM, and next to it 64 conversions to fp64 a lane and row, each as long as four multiply-adds.
// A wave that holds whole rows takes the registers of others: four of them, asked for again two at a time, were 200 to 500 registers a
// lane at rows of 8 KiB and more, one workgroup per compute unit from 9 KiB on (and registers in memory in the fp32 step of 9 KiB), so
// that layers of many neurons went over the chip twice.  us a step from a graph (2 % of the neurons fire), two rows interleaved by
// the compiler and none on its way meanwhile / four whole rows / now: d = 5120, F = 4096 44.5 / 40.8 / 38.4, F = 8192 57.6 / 54.5 /
// 53.0, F = 13824 75.7 / 78.6 / 74.5, F = 17000 98.6 / 98.7 / 92.4; d = 8192, F = 12288 103.8 / 108.0 / 104.4; d = 4096, F = 11008
// 60.5 / 59.8 / 58.9; fp32 d = 2304, F = 6000 43.9 / 44.5 / 41.1, F = 20000 90.1 / 95.9 / 88.6.
// The same piece of four rows side by side falls on too few channels of the memory where a row is a power of two: lif_predict, two
// / four rows, d = 4096, F = 20000 27.1 / 30.6, fp32 d = 4096, F = 12000 31.1 / 36.2 (d = 5120, F = 8192 14.6 / 14.8).  Pieces ahead,
// 6 / 8 / 10 / 16: d = 5120, F = 13824 21.8 / 21.8 / 22.2 / 23.3, fp32 d = 4096, F = 8000 22.0 / 21.2 / 21.8 / 23.1.
// Tokens of a batch (one row at a time from LDS, the same order), four calls with sums that wait for their own conversion / that do
// not: d = 1496, F = 19864, 8 tokens 182.7 / 174.4; d = 1232, F = 11728, 6 tokens 107.3 / 101.3.
constexpr int kGateAhead = 8;
template <typename T, int NI>
__device__ __forceinline__ unsigned gate_byte(const T* __restrict__ Wg, const float* __restrict__ b, float* __restrict__ gact, int grp,
                                              int nvec, typename Vec<T>::type (&xr)[NI], double th) {
    using V = typename Vec<T>::type;
    constexpr int R = 4, W = NI < kGateAhead / 2 ? 2 * NI : kGateAhead;
    const int lane = threadIdx.x & 63, owner = ((lane >> 3) & 1) * 2 + ((lane >> 4) & 1);
    const V* rows = reinterpret_cast<const V*>(Wg) + (size_t)grp * 8 * nvec;
    const float bias0 = b[grp * 8 + owner], bias1 = b[grp * 8 + R + owner];
    V g[W][2];
    auto request = [&](int k) {                      // piece k mod NI of row 2 (k / NI) and of the row behind it
        const int e = k / NI * 2, it = k % NI;
#pragma unroll
        for (int u = 0; u < 2; ++u)
            g[k % W][u] = rows[(size_t)(e + u) * nvec + (it < full_pieces(NI) ? it * 64 + lane : min(it * 64 + lane, nvec - 1))];
    };
#pragma unroll
    for (int k = 0; k < W; ++k) request(k);
    unsigned byte = 0;
#pragma unroll
    for (int e0 = 0; e0 < 8; e0 += R) {
        double v[R];
#pragma unroll
        for (int u = 0; u < R; u += 2) {
#pragma unroll
            for (int it = 0; it < NI; ++it) asm volatile("" : "+v"(xr[it]));  // (else x is widened once, and twice as many registers kept)
            double sum[2] = {0.0, 0.0};
#pragma unroll
            for (int it = 0; it < NI; ++it) {
                const int k = (e0 + u) / 2 * NI + it;
                const bool in = it < full_pieces(NI) || it * 64 + lane < nvec;
                const V pair[2] = {in ? g[k % W][0] : V(0), in ? g[k % W][1] : V(0)};
                dot_f64<2>(pair, xr[it], sum);
                if (k + W < 4 * NI) request(k + W);
                __builtin_amdgcn_sched_barrier(0);   // (the requests go out in turn, each as soon as its registers are free)
            }
            v[u] = sum[0];
            v[u + 1] = sum[1];
        }
#pragma unroll
        for (int u = 0; u < R; ++u) v[u] += dpp_from<0xB1, 0xf>(v[u]);       // quad_perm 1 0 3 2
#pragma unroll
        for (int u = 0; u < R; ++u) v[u] += dpp_from<0x4E, 0xf>(v[u]);       // quad_perm 2 3 0 1
#pragma unroll
        for (int u = 0; u < R; ++u) v[u] += dpp_from<0x141, 0xf>(v[u]);      // half row mirrored: the other quad, all of whose lanes are alike
        const bool up = (lane & 8) != 0;
#pragma unroll
        for (int u = 0; u < R / 2; ++u) {
            const double send = up ? v[u] : v[u + R / 2], keep = up ? v[u + R / 2] : v[u];
            v[u] = keep + dpp_from<0x128, 0xf>(send);
        }
        double a = swap_add<16>(v[0], v[1]);
        a = swap_add<32>(a, a) + (double)(e0 ? bias1 : bias0);
        const unsigned long long fires = __ballot(a > th);
#pragma unroll
        for (int u = 0; u < R; ++u) byte |= (unsigned)(fires >> ((u >> 1) * 8 + (u & 1) * 16) & 1u) << (e0 + u);
        if ((lane & 0x27) == 0) gact[grp * 8 + e0 + owner] = (float)(a > 0.0 ? a : 0.0);
    }
    return byte;
}

// Gate projection as the predictor (Appendix, Llama 2, "Alternative approaches"): the gate matrix stays
// resident and  a_i = gate_i . x + b_i  decides exactly which neurons fire (mask bit = a_i > theta); the same
// pass leaves relu(a_i) per token and neuron for the FFN, so bundles hold only up row | down column.
// One wave per group of 8 neurons (one mask byte per token): 16-byte loads along the row, fp64 accumulation
// (bit-exact decision), wave reduction.  grid-stride over F / 8 groups, block = 256.  NI as in the FFN kernels.
// XREG (one token): x stays in registers.  Otherwise the tokens' x are staged in LDS (dynamic LDS: batch * d
// elements) and every gate row, loaded once, is applied to each token in turn; masks [batch x F/8], step mask = OR
// over the tokens, gact [batch x F].
template <typename T, int NI, bool XREG>
__global__ __launch_bounds__(256) void k_predict_gate(const T* __restrict__ Wg, const float* __restrict__ b,
                                                      const T* __restrict__ x, int d, int F, int batch, float theta,
                                                      uint8_t* __restrict__ mask, uint8_t* __restrict__ step_mask,
                                                      float* __restrict__ gact, const DevState* __restrict__ st) {
    using V = typename Vec<T>::type;
    constexpr int VE = Vec<T>::N;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_gate[];
    V* xs = reinterpret_cast<V*>(smem_gate);
    const int tid = threadIdx.x, lane = tid & 63;
    const int nvec = d / VE;
    const int gw = blockIdx.x * 4 + (tid >> 6), nw = gridDim.x * 4;
    const V* xv = reinterpret_cast<const V*>(x);
    V xr[XREG ? NI : 1];
    if (XREG) {
#pragma unroll
        for (int it = 0; it < NI; ++it) {
            const int idx = it * 64 + lane;
            xr[it] = (idx < nvec) ? xv[idx] : V(0);
        }
    } else {
        for (int i = tid; i < batch * nvec; i += 256) xs[i] = xv[i];
        __syncthreads();
    }
    if (st->cur.error) return;
    const double th = (double)theta;
    const int mask_stride = F >> 3;
    for (int grp = gw; grp * 8 < F; grp += nw) {
        if constexpr (XREG) {
            const unsigned byte = gate_byte<T, NI>(Wg, b, gact, __builtin_amdgcn_readfirstlane(grp), nvec, xr, th);
            if (lane == 0) {
                mask[grp] = (uint8_t)byte;
                if (step_mask != mask) step_mask[grp] = (uint8_t)byte;   // one token: the step mask is the mask
            }
            continue;
        }
        unsigned long long bits = 0;                 // bit 8 * token + e: neuron grp * 8 + e fires for that token
#pragma unroll 2
        for (int e = 0; e < 8; ++e) {
            const int i = grp * 8 + e;
            const V* row = reinterpret_cast<const V*>(Wg + (size_t)i * d);
            V g[NI];
#pragma unroll
            for (int it = 0; it < NI; ++it) {
                const int idx = it * 64 + lane;
                g[it] = (idx < nvec) ? row[idx] : V(0);
            }
            const double bi = (double)b[i];
            for (int t = 0; t < batch; ++t) {
                double acc = 0.0;
#pragma unroll
                for (int it = 0; it < NI; ++it) {
                    const int idx = it * 64 + lane;
                    if (idx < nvec) acc = dot_f64(g[it], xs[t * nvec + idx], acc);
                }
                acc = wave_sum(acc);
                const double a = acc + bi;
                if (a > th) bits |= 1ull << (8 * t + e);
                if (lane == 0) gact[(size_t)t * F + i] = (float)(a > 0.0 ? a : 0.0);
            }
        }
        if (lane < batch) mask[(size_t)lane * mask_stride + grp] = (uint8_t)(bits >> (8 * lane));
        if (lane == 0) {
            unsigned long long o = bits | (bits >> 32);
            o |= o >> 16;
            o |= o >> 8;
            step_mask[grp] = (uint8_t)o;
        }
    }
}

}  // namespace lif
