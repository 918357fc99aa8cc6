// Shared device-side definitions of the sparse-FFN hot path (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lif {

constexpr int kWave = 64;

// Counts of one layer.
struct StepCounts {
    int32_t num_used;     // rows of the cache in use (Section 3.3 "num_used")
    int32_t n_base;       // rows kept after the pending deletion (n' = num_used - c)
    int32_t step;         // completed window updates
    int32_t error;        // sticky lif_status (0, LIF_CAPACITY, or LIF_HIP_ERROR: k_ffn_one)
    int32_t n_added;      // |added| of the pending / last update
    int32_t n_removed;    // |removed| of the pending / last update
    int32_t n_moved;      // rows moved by the last deletion
    int32_t window_len;   // step masks currently in the window (<= k; smaller after a dynamic shrink)
    int32_t ring_pos;     // ring entry the next mask goes to
    int32_t set_par;      // which of the two bitmaps of the cached set is current
};

// Device-resident state of one layer.  Lives at the start of the caller's workspace so
// that the hot calls chain on a stream without the host ever knowing a count.
// `next`: a fused step (k_step1) decides the new counts while all its workgroups still read the old ones, so it leaves
// them here and the down projection of the same step, whose workgroups read only `next`, copies them into `cur`.
struct DevState {
    StepCounts cur;
    StepCounts next;
    // counters: only ever updated with atomic adds whose result is not used (a load-add-store at the end of a kernel
    // would keep its last wave waiting for a memory round trip)
    unsigned long long c_steps, c_added, c_removed, c_rows_moved, c_h2d_bytes;
    unsigned long long c_ffn_calls, c_ffn_rows, c_ffn_active;   // FFN calls, rows in use, rows with a non-zero activation
};

// Where the bundle of neuron i lives in pinned host memory (Section 3.2, Fig. 5).  Bundled (down == null): one
// contiguous chunk of row_bytes at rows + i * row_bytes.  Not bundled: the activation vectors ((gate |) up row,
// act_bytes) at rows + i * act_bytes and the down column at down + i * (row_bytes - act_bytes): two reads per
// neuron, the layout that bundling replaces.  All sizes are multiples of 16 bytes.
struct HostStore {
    const char* rows;
    const char* down;
    size_t act_bytes;
};
// address of byte `off` (a multiple of 16, < row_bytes) of the bundle of neuron i
__device__ __forceinline__ const char* host_piece(const HostStore& hs, int i, size_t off, size_t row_bytes) {
    if (hs.down && off >= hs.act_bytes) return hs.down + (size_t)i * (row_bytes - hs.act_bytes) + (off - hs.act_bytes);
    return hs.rows + (size_t)i * (hs.down ? hs.act_bytes : row_bytes) + off;
}

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// 16-byte vector view of the element type.
template <typename T> struct Vec;
template <> struct Vec<_Float16> {
    using type = f16x8;
    static constexpr int N = 8;
};
template <> struct Vec<float> {
    using type = f32x4;
    static constexpr int N = 4;
};

// acc + sum_e a[e] * b[e], products of E-typed values, fp32 accumulation.
#if defined(__HIP_DEVICE_COMPILE__)     // (the host pass only parses device functions)
static_assert(__has_builtin(__builtin_amdgcn_fdot2), "built for gfx950: the packed fp16 dot product is required");
#endif
__device__ __forceinline__ float dot_acc(f16x8 a, f16x8 b, float acc) {
    acc = __builtin_amdgcn_fdot2(__builtin_shufflevector(a, a, 0, 1), __builtin_shufflevector(b, b, 0, 1), acc, false);
    acc = __builtin_amdgcn_fdot2(__builtin_shufflevector(a, a, 2, 3), __builtin_shufflevector(b, b, 2, 3), acc, false);
    acc = __builtin_amdgcn_fdot2(__builtin_shufflevector(a, a, 4, 5), __builtin_shufflevector(b, b, 4, 5), acc, false);
    acc = __builtin_amdgcn_fdot2(__builtin_shufflevector(a, a, 6, 7), __builtin_shufflevector(b, b, 6, 7), acc, false);
    return acc;
}
__device__ __forceinline__ float dot_acc(f32x4 a, f32x4 b, float acc) {
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_fmaf(a[e], b[e], acc);
    return acc;
}

// Sum over the 64 lanes of a wave; every lane receives the result.  Data-parallel-primitive moves instead of
// shuffles through the LDS crossbar: an inclusive prefix sum (shifts by 1, 2, 4, 8 inside the rows of 16 lanes,
// lane 15 of a row into the next row, lane 31 into the upper half) leaves the total in lane 63, which is then
// broadcast.  Lanes without a source add 0.
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_from(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROWS, 0xf, false));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_from(double v) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, ROWS, 0xf, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, ROWS, 0xf, false);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// a + b where lanes M apart (16 or 32) trade first: the lane whose bit M is clear gets its own and its partner's a, the other one
// both b.
template <int M>
__device__ __forceinline__ double swap_add(double a, double b) {
    static_assert(M == 16 || M == 32, "rows or halves of the wave");
    const unsigned long long ua = __builtin_bit_cast(unsigned long long, a), ub = __builtin_bit_cast(unsigned long long, b);
    auto trade = [](unsigned x, unsigned y) {
        if constexpr (M == 16) return __builtin_amdgcn_permlane16_swap(x, y, false, false);
        else return __builtin_amdgcn_permlane32_swap(x, y, false, false);
    };
    const auto lo = trade((unsigned)ua, (unsigned)ub), hi = trade((unsigned)(ua >> 32), (unsigned)(ub >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi[0] << 32) | lo[0]) +
           __builtin_bit_cast(double, ((unsigned long long)hi[1] << 32) | lo[1]);
}
__device__ __forceinline__ float wave_sum(float v) {
    v += dpp_from<0x111, 0xf>(v);   // row_shr:1
    v += dpp_from<0x112, 0xf>(v);   // row_shr:2
    v += dpp_from<0x114, 0xf>(v);   // row_shr:4
    v += dpp_from<0x118, 0xf>(v);   // row_shr:8
    v += dpp_from<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
    v += dpp_from<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
__device__ __forceinline__ double wave_sum(double v) {
    v += dpp_from<0x111, 0xf>(v);
    v += dpp_from<0x112, 0xf>(v);
    v += dpp_from<0x114, 0xf>(v);
    v += dpp_from<0x118, 0xf>(v);
    v += dpp_from<0x142, 0xa>(v);
    v += dpp_from<0x143, 0xc>(v);
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, 63);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), 63);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// a value that is the same in all lanes, as one of the whole wave
__device__ __forceinline__ unsigned long long uniform(unsigned long long v) {
    return ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(v >> 32)) << 32) |
           (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)v);
}

// *p at an address that is the same for the whole wave, through the scalar cache: of memory that nothing writes during the launch
template <typename U>
__device__ __forceinline__ U uniform_load(const U* p) {
    static_assert(sizeof(U) == 4, "one dword");
    const unsigned long long u = reinterpret_cast<unsigned long long>(p);
    const unsigned long long q = ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(u >> 32)) << 32) |
                                 (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)u);
    return *reinterpret_cast<const __attribute__((address_space(4))) U*>(q);
}

// v to the 16 bytes at base + off, written through the L2 to memory; base is the same for the whole wave and off + 16 <= bytes.
// A launch ends when every L2 has written back what it holds changed: the rows that a fused step has loaded and moved, a few MB, stood
// in front of the down projection.  us a step, plain stores -> these, two timings in turn: OPT shape 57.9 -> 57.3 and 58.2 -> 57.7, eight
// stacked layers of it from a graph 467.5 -> 465.2 and 476.4 -> 471.3, Falcon shape 134.6 -> 133.3 and 135.9 -> 134.8, Llama-2 shape from
// a graph 132.1 -> 130.5 and 132.0 -> 130.8, gate resident 105.1 -> 104.1 and 105.8 -> 104.8, 8 tokens 230.6 -> 229.5 and 231.0 -> 230.4
// (two runs of one build differ by up to 0.4 %).  lif_load_bundles keeps plain stores: the
// activation stage behind it finds the rows in the L2 (fp32 d = 1288, 3 tokens, four calls 68.6 against 69.2).  Activations
// were no faster written through; partial outputs are (store_part), and have to be where the same launch reads them.
template <typename V>
__device__ __forceinline__ void store_through(char* base, unsigned off, unsigned bytes, V v) {
    static_assert(sizeof(V) == 16, "four dwords");
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
    constexpr int kFlags = 0x00027000, kWriteThrough = 1 << 4;    // a raw buffer of dwords; the cache policy bit sc1
    const unsigned long long u = reinterpret_cast<unsigned long long>(base);
    const unsigned long long q = ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(u >> 32)) << 32) |
                                 (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)u);
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v),
                                           __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(q), 0, (int)bytes, kFlags), (int)off, 0,
                                           kWriteThrough);
}

// 16 bytes at base + off past the caches, so what another workgroup of the launch has written past them (store_part); base is the same
// for the whole wave and off + 16 <= bytes
__device__ __forceinline__ f32x4 load_through(const float* base, unsigned off, unsigned bytes) {
    constexpr int kFlags = 0x00027000, kPast = 1 << 4;           // a raw buffer of dwords; the cache policy bit sc1
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                         __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, (int)bytes, kFlags), (int)off, 0, kPast));
}

// Workgroup barrier that orders LDS accesses only: unlike __syncthreads() it does not wait for the global
// stores a wave has in flight (their acknowledgement from the L2 costs several hundred nanoseconds).  Use it
// where the data handed over lives in LDS and no thread reads global memory that another one has just written.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Inclusive prefix sum over the lanes of a wave.
__device__ __forceinline__ int wave_inclusive_scan(int v, int /*lane*/) {
    // data-parallel-primitive moves instead of six shuffles through the LDS crossbar: shifts by 1, 2, 4, 8 inside
    // the rows of 16 lanes (lanes without a source add 0), then lane 15 of a row into the next row (rows 1 and 3)
    // and lane 31 into rows 2 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31
    return v;
}

// Exclusive prefix sum of one int per thread over a workgroup of NW waves (thread order).
// `wave_tot` is LDS scratch of at least NW ints.  Returns the exclusive prefix; *total receives the
// workgroup sum.  Contains two barriers (the first keeps a previous scan's readers of wave_tot ahead of the writes).
template <int NW>
__device__ __forceinline__ int block_exclusive_scan(int v, int* wave_tot, int* total) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid >> 6;
    const int inc = wave_inclusive_scan(v, lane);
    __syncthreads();
    if (lane == kWave - 1) wave_tot[w] = inc;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const int t = wave_tot[i];
        if (i < w) before += t;
        all += t;
    }
    *total = all;
    return before + inc - v;
}


// Sum of v[0..N) over the lanes that differ in the lane bits M, 2M, ..., 32 (groups of lanes M apart).
// While a lane holds more than one value, a step halves them: the lane keeps the half selected by its own
// bit and hands the other half to its partner, so N - N / 2^steps (+ the remaining full steps) exchanges
// replace steps * N.  Returns through `first` the index of the first value this lane ends up with; it then
// holds wave_fold_held<N, M>() finished sums in v[0..held).  Lanes whose bits of the steps taken after a
// single value was left are not all zero hold a duplicate (wave_fold_dup_mask gives those bits).
template <int N, int M>
constexpr int wave_fold_held() {
    int held = N;
    for (int m = M; m < kWave; m <<= 1)
        if (held > 1) held >>= 1;
    return held;
}
template <int N, int M>
constexpr int wave_fold_dup_mask() {
    int held = N, mask = 0;
    for (int m = M; m < kWave; m <<= 1) {
        if (held > 1) held >>= 1;
        else mask |= m;
    }
    return mask;
}
// The exchanges are register moves (lanes 4 and 8 apart: permutations in a row of 16; 16 and 32 apart: swaps of rows and halves):
// through the LDS crossbar each of them is a round trip that the next one waits for.
template <int M>
__device__ __forceinline__ float from_xor(float v) {                 // v of the lane whose number differs in bit M
    static_assert(M == 4 || M == 8, "inside a row of 16 lanes");
    if constexpr (M == 4) return dpp_from<0x1b, 0xf>(dpp_from<0x141, 0xf>(v));      // mirrored in 8 lanes (^7), then in 4 (^3)
    else return dpp_from<0x128, 0xf>(v);                             // a rotation by 8
}
// a + b where lanes M apart trade first, as the fp64 form above
template <int M>
__device__ __forceinline__ float swap_add(float a, float b) {
    static_assert(M == 16 || M == 32, "rows or halves of the wave");
    const unsigned ua = __builtin_bit_cast(unsigned, a), ub = __builtin_bit_cast(unsigned, b);
    if constexpr (M == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(ua, ub, false, false);
        return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(ua, ub, false, false);
        return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
    }
}
template <int HELD, int M, int N>
__device__ __forceinline__ void wave_fold_step(float (&v)[N], int& first, int lane) {
    if constexpr (M < kWave) {
        if constexpr (HELD > 1) {
            constexpr int half = HELD / 2;
            const bool up = (lane & M) != 0;
#pragma unroll
            for (int i = 0; i < half; ++i) {
                if constexpr (M >= 16) {
                    v[i] = swap_add<M>(v[i], v[i + half]);
                } else {
                    const float send = up ? v[i] : v[i + half], keep = up ? v[i + half] : v[i];
                    v[i] = keep + from_xor<M>(send);
                }
            }
            first += up ? half : 0;
            wave_fold_step<half, M * 2, N>(v, first, lane);
        } else {
            if constexpr (M >= 16) v[0] = swap_add<M>(v[0], v[0]);
            else v[0] += from_xor<M>(v[0]);
            wave_fold_step<1, M * 2, N>(v, first, lane);
        }
    }
}
template <int N, int M>
__device__ __forceinline__ int wave_fold(float (&v)[N], int lane) {
    static_assert((N & (N - 1)) == 0, "power of two");
    int first = 0;
    wave_fold_step<N, M, N>(v, first, lane);
    return first;
}

}  // namespace lif
