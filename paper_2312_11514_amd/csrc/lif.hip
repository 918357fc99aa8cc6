// C ABI of the sparse-FFN hot path (see include/lif.h for the contract of every call).
// Host side only: argument checks, launch geometry, call-order bookkeeping, event timing.
#include "../../include/lif.h"

#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstring>
#include <new>
#include <type_traits>
#include <vector>

#include "lif_common.h"
#include "lif_ffn.h"
#include "lif_ffn_down1.h"
#include "lif_ffn_one.h"
#include "lif_ffn_mfma.h"
#include "lif_ffn_down_mfma.h"
#include "lif_predict.h"
#include "lif_step1.h"
#include "lif_window.h"

using namespace lif;

// Scratch of lif_sparse_ffn_static: activations and partial outputs of one FFN call.  One copy per GPU, at its own
// address on each; host code reaches it only through the pointer hipGetSymbolAddress returns for the current device.
constexpr size_t kStaticScratchBytes = 5u << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

thread_local char g_err[512] = "";

int fail(int code, const char* fmt, const char* detail = "") {
    snprintf(g_err, sizeof(g_err), fmt, detail);
    return code;
}

#define LIF_HIP(call)                                                             \
    do {                                                                          \
        hipError_t e_ = (call);                                                   \
        if (e_ != hipSuccess) return fail(LIF_HIP_ERROR, #call ": %s", hipGetErrorString(e_)); \
    } while (0)

// Bytes of host reads that lif_step keeps outstanding: pairs of loader workgroups (one bundle in flight per pair) =
// kStepInflightBytes / bundle bytes, within 5..kStepPairs.  The link needs about 128 KiB (56 GB/s at 1.5 to 2.4 us); the rest
// covers the time in which a loader writes a bundle out and asks for the next.  One token with 144 / 192 / 256 / 320 / 384 KiB:
// OPT shape 60.4 / 59.4 / 58.2 / 58.4 / 60.0 us, Falcon shape 188 / 159 / 143 / 141 / 140 us, gated Llama-2 shape 147 / 138 / 137
// / 138 / 143 us.
// For rows of at most 10 KiB the number of loaders is what limits (kStepPairs).
// Where a vector is at most 2 KiB a loader takes whole bundles, a pair has two in flight, and 256 KiB of them are asked for by
// at most kStepPairsWhole pairs: bundles of 1 KiB, 1278 and 395 added, with 32 / 48 / 64 pairs 77.1 / 65.1 / 62.1 and 43.8 / 40.5 /
// 39.5 us (five separate launches: 70.2 and 43.6); of 2 KiB, 783 and 198 added, 57.0 / 55.7 / 55.3 and 28.9 / 27.6 / 26.8; of
// 4 KiB, 455 and 136 added, with 32 / 40 / 64 54.0 / 53.5 / 54.3 and 29.3 / 29.4 / 30.1.
// Vectors of more than 12 KiB: a loader takes so long with each (16 pieces a lane) that kStepPairsWide pairs are needed; d = 8192,
// with 10 / 14 / 20 / 32 pairs: plain 75.0 / 63.3 / 60.2 / 61.6 us (five separate launches: 67.1), gated 92.1 / 87.5 / 83.9 /
// 84.7, with the gate resident 91.1 / 79.6 / 76.0 / 78.0; d = 7168 59.4 / 53.8 / 53.0 / 55.1; but d = 6144 44.0 / 44.6 / 45.9 /
// 46.2.
// Several tokens: more loaders, a bundle takes longer to deal with; 20 / 32 / 48 / 64 pairs of 16 KiB rows: 205 / 207 / 200 / 200
// us a pass, of 24 KiB: 262 / 252 / 249 / 250; but every loader workgroup costs a compute unit of the activation stage (11 KiB
// rows, 60 loaded: 52 / 52 / 53 / 56).
constexpr size_t kStepInflightBytes = 320 * 1024, kStepInflightBytesWhole = 256 * 1024, kStepInflightBytesB = 768 * 1024;
constexpr int kStepPairs = 32, kStepPairsWhole = 64, kStepPairsWide = 20, kStepPairsB = 48;
// lif_load_bundles by itself: with 320 / 640 KiB rows of 25 and 30 KiB took 121 / 117 and 110 / 105 us (all four calls).
constexpr size_t kLoadInflightBytes = 640 * 1024;
constexpr int kDefaultPolls = 4096;      // a failed poll takes about 0.7 us: 3 ms before a workgroup helps itself

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

struct Layout {
    size_t state, words, one, arrived, ring, tpart, move_dst, hole_list, h, ypart, h_new, stamp, ptr_new, bias_new, gact, total;
    int reset_words;                   // 64-bit words from `words` on that a reset clears
};

int elem_bytes(const lif_config& c) { return c.dtype == LIF_F32 ? 4 : 2; }
int vec_elems(const lif_config& c) { return 16 / elem_bytes(c); }
int ring_words(const lif_config& c) { return (c.d_ffn + 63) / 64; }

bool config_ok(const lif_config* c, const char** why) {
    *why = "";
    if (!c) return (*why = "null config", false);
    if (c->dtype != LIF_F32 && c->dtype != LIF_F16) return (*why = "dtype", false);
    const int ve = vec_elems(*c);
    if (c->d_model <= 0 || c->d_model % ve) return (*why = "d_model must be a positive multiple of 16 bytes", false);
    if ((c->d_model / ve + 63) / 64 > 16) return (*why = "d_model too large (at most 1024 16-byte vectors)", false);
    if (c->d_ffn <= 0 || c->d_ffn % 8 || c->d_ffn > kScanThreads * kMaxSpan) return (*why = "d_ffn must be a multiple of 8, at most 65536", false);
    if (c->predictor != LIF_PRED_GATE &&
        (c->rank <= 0 || c->rank % ve || c->rank > 2048)) return (*why = "rank", false);
    if (c->window_k < 1 || c->window_k > 256) return (*why = "window_k must be in 1..256", false);
    if (c->capacity_rows < 1 || c->capacity_rows > kScanThreads * kMaxSpan) return (*why = "capacity_rows must be in 1..65536", false);
    if (c->max_batch < 1 || c->max_batch > 8) return (*why = "max_batch must be in 1..8", false);
    if (c->glu != 0 && c->glu != 1) return (*why = "glu", false);
    if (c->shrink_window != 0 && c->shrink_window != 1) return (*why = "shrink_window", false);
    if (c->predictor != LIF_PRED_LOWRANK && c->predictor != LIF_PRED_GATE) return (*why = "predictor", false);
    if (c->predictor == LIF_PRED_GATE && c->glu)
        return (*why = "the gate predictor takes plain (up | down) bundles", false);
    if (c->ffn_mode != LIF_FFN_SKIP_DEAD && c->ffn_mode != LIF_FFN_FULL_BUNDLE) return (*why = "ffn_mode", false);
    if ((size_t)c->max_batch * c->d_model * elem_bytes(*c) > 64 * 1024) return (*why = "max_batch * d_model exceeds the 64 KiB LDS staging area", false);
    return true;
}

// column slices of the down projection of one token: whole runs of them per XCD
int down1_slices(const lif_config& c) {
    const int cols = kDown1Lanes * vec_elems(c);
    return ((c.d_model + cols - 1) / cols + kXcds - 1) / kXcds * kXcds;
}

// whether calls on the layer can take the single-launch FFN (ffn_one), so that it has words to hand over
bool ffn_one_possible(const lif_config& c) { return c.capacity_rows <= kOneCapacity && down1_slices(c) <= kOneSlices; }

Layout make_layout(const lif_config& c) {
    Layout L;
    size_t off = 0;
    L.state = off;
    off = align_up(off + sizeof(DevState), 256);
    L.words = off;                     // words handed over inside a fused step: t = x A, the mask words
    off = off + sizeof(uint64_t) * kWordReps * ((size_t)words_pitch(2 * std::max(c.rank, 0)) + words_pitch(2 * ring_words(c)));
    off = off + sizeof(uint64_t) * c.capacity_rows;               // ... and the deletion plan;
    L.one = off;                       // inside a single-launch FFN, and its launch number
    if (ffn_one_possible(c)) off = off + sizeof(uint64_t) * kOneReps * one_pitch(c.capacity_rows) + sizeof(OneState);
    L.arrived = off;                   // per column slice: workgroups whose partial outputs are written
    off = off + sizeof(unsigned) * kArrivedPitch * down1_slices(c);      // (no down projection has more slices)
    L.ring = off;                      // window_k step masks, each padded to whole 64-bit words
    off = off + (size_t)(c.window_k + 2) * ring_words(c) * 8;     // ... directly followed by the two bitmaps of the cached set
    L.reset_words = (int)((off - L.words) / 8);
    off = align_up(off, 256);
    L.tpart = off;
    off = align_up(off + sizeof(double) * c.max_batch * std::max(c.rank, 0), 256);
    L.move_dst = off;
    off = align_up(off + sizeof(int32_t) * c.capacity_rows, 256);
    L.hole_list = off;
    off = align_up(off + sizeof(int32_t) * c.capacity_rows, 256);
    L.h = off;
    off = align_up(off + sizeof(float) * c.max_batch * c.capacity_rows, 256);
    L.ypart = off;                     // per-chunk partial outputs of the down projection
    off = align_up(off + sizeof(float) * kDownChunksMax * c.max_batch * c.d_model, 256);
    L.h_new = off;                     // activations written by the loaders of a fused step
    off = align_up(off + sizeof(float) * c.max_batch * c.capacity_rows, 256);
    L.stamp = off;                     // step number at which h_new[slot] was written
    off = align_up(off + sizeof(int32_t) * c.capacity_rows, 256);
    L.ptr_new = off;                   // slot owners and biases written by the fused step
    off = align_up(off + sizeof(int32_t) * c.capacity_rows, 256);
    L.bias_new = off;
    off = align_up(off + sizeof(float) * c.capacity_rows, 256);
    L.gact = off;                      // gate predictor: relu(gate_i . x_t + b_i) per token and original neuron
    off = align_up(off + (c.predictor == LIF_PRED_GATE ? sizeof(float) * c.max_batch * c.d_ffn : 0), 256);
    L.total = off;
    return L;
}

}  // namespace

struct lif_layer {
    lif_config cfg;
    lif_buffers buf;
    Layout lay;
    HostStore host;             // device-visible addresses of the pinned bundle store (bundled or in two parts)
    int loader_pairs;           // loader wave pairs of the fused step, 0 = chosen from the bundle size
    DevState* st;
    unsigned long long* ring;
    double* tpart;
    int32_t* move_dst;
    int32_t* hole_list;
    float* h;
    float* ypart;
    float* h_new;
    int32_t* stamp;
    int32_t* ptr_new;
    float* bias_new;
    unsigned long long* words;
    unsigned long long* one_words;  // of k_ffn_one, null where it is never launched
    OneState* one;
    unsigned* arrived;
    int polls;                  // failed polls of a hand-over word before a workgroup computes the value itself
    float* gact;                // null unless the gate projection is the predictor
    size_t row_elems, row_bytes;
    bool window_pending;
    int expected_rows;          // hint, at most the capacity; 0 = none
    unsigned char* static_scratch;  // this device's copy of the library's static scratch array (null: lookup failed)
    // event timing
    bool prof_on;
    int prof_max;
    std::vector<hipEvent_t> ev;     // 2 per timed launch
    std::vector<int> ev_kernel;
};

namespace {

struct Timed {
    lif_layer* L;
    hipStream_t s;
    int slot;
    Timed(lif_layer* layer, int kid, hipStream_t stream) : L(layer), s(stream), slot(-1) {
        if (L->prof_on && (int)L->ev_kernel.size() < L->prof_max) {
            slot = (int)L->ev_kernel.size();
            L->ev_kernel.push_back(kid);
            (void)hipEventRecord(L->ev[2 * slot], s);
        }
    }
    ~Timed() {
        if (slot >= 0) (void)hipEventRecord(L->ev[2 * slot + 1], s);
    }
};

template <typename T>
int launch_predict(lif_layer* L, const void* x, int batch, uint8_t* masks, uint8_t* step_mask, hipStream_t s) {
    const lif_config& c = L->cfg;
    {
        Timed t(L, LIF_K_PREDICT_XA, s);
        const int ni = (c.d_model / Vec<T>::N + 63) / 64;
#define LIF_XA(NI)                                                                                          \
    hipLaunchKernelGGL((k_predict_xa<T, NI>), dim3(c.rank, batch), dim3(256), 0, s, (const T*)x,       \
                       (const T*)L->buf.A, L->tpart, c.d_model, c.rank, L->st)
        if (ni <= 1) LIF_XA(1);
        else if (ni <= 2) LIF_XA(2);
        else if (ni <= 4) LIF_XA(4);
        else if (ni <= 8) LIF_XA(8);
        else if (ni <= 9) LIF_XA(9);
        else if (ni <= 12) LIF_XA(12);
        else LIF_XA(16);
#undef LIF_XA
    }
    const int grid = (c.d_ffn + kMaskCols * 8 - 1) / (kMaskCols * 8);
    Timed t(L, LIF_K_PREDICT_MASK, s);
#define LIF_MASK(KERNEL, LDS)                                                                               \
    hipLaunchKernelGGL((KERNEL), dim3(grid), dim3(256), LDS, s, (const T*)L->buf.B, L->buf.c, L->tpart, c.rank, c.d_ffn,   \
                       batch, c.threshold, masks, step_mask, L->st)
    if (batch == 1) LIF_MASK((k_predict_mask<T, false>), 0);
    else if (c.rank <= kMaskChunk) LIF_MASK((k_predict_mask<T, true>), mask_lds_bytes(c.rank, batch));
    else if (batch <= 2) LIF_MASK((k_predict_mask_long<T, 2>), 0);
    else if (batch <= 4) LIF_MASK((k_predict_mask_long<T, 4>), 0);
    else LIF_MASK((k_predict_mask_long<T, 8>), 0);
#undef LIF_MASK
    return LIF_OK;
}

template <typename T>
void launch_predict_gate(lif_layer* L, const void* x, int batch, uint8_t* masks, uint8_t* step_mask, hipStream_t s) {
    const lif_config& c = L->cfg;
    const int nvec = c.d_model / Vec<T>::N;
    const int ni = (nvec + 63) / 64;
    const int grid = std::min((c.d_ffn / 8 + 3) / 4, 2048);
    const size_t shm = batch == 1 ? 0 : (size_t)batch * c.d_model * sizeof(T);
    Timed t(L, LIF_K_PREDICT_MASK, s);
#define LIF_PG_X(NI, XREG)                                                                                   \
    hipLaunchKernelGGL((k_predict_gate<T, NI, XREG>), dim3(grid), dim3(256), shm, s, (const T*)L->buf.A,         \
                       L->buf.b, (const T*)x, c.d_model, c.d_ffn, batch, c.threshold, masks, step_mask, L->gact, \
                       L->st)
#define LIF_PG(NI) do { if (batch == 1) LIF_PG_X(NI, true); else LIF_PG_X(NI, false); } while (0)
    if (ni <= 1) LIF_PG(1);
    else if (ni <= 2) LIF_PG(2);
    else if (ni <= 4) LIF_PG(4);
    else if (ni <= 6) LIF_PG(6);           // (full_pieces)
    else if (ni <= 8) LIF_PG(8);
    else if (ni <= 9) LIF_PG(9);
    else if (ni <= 12) LIF_PG(12);
    else LIF_PG(16);
#undef LIF_PG
#undef LIF_PG_X
}

// `h` (activations) and `ypart` (partial outputs) of the FFN launches: the workspace arrays of the layer, or the
// library's static scratch (lif_sparse_ffn_static)
template <typename T, bool GLU>
void launch_ffn_up(lif_layer* L, const void* x, int batch, float* h, hipStream_t s) {
    const lif_config& c = L->cfg;
    const int nvec = c.d_model / Vec<T>::N;
    const int ni = (nvec + 63) / 64;
    // one wave per row; with a row-count hint the grid is sized to it and the first pass is speculative
    const int spec = L->expected_rows > 0 ? 1 : 0;
    const int grid = spec ? std::min(kUpMaxWgs, std::max(1, L->expected_rows / 4))
                          : std::min((c.capacity_rows + 3) / 4, 512);
    const size_t shm = batch == 1 ? 0 : (size_t)batch * c.d_model * sizeof(T);
#define LIF_UP_X(NI, XREG)                                                                                   \
    hipLaunchKernelGGL((k_ffn_up<T, NI, GLU, XREG>), dim3(grid), dim3(256), shm, s, (const T*)L->buf.matrix,    \
                       L->buf.bias, (const T*)x, h, c.d_model, batch, c.capacity_rows, L->row_elems, spec,        \
                       L->buf.pointers, L->gact, c.d_ffn, L->st)
#define LIF_UP(NI) do { if (batch == 1) LIF_UP_X(NI, true); else LIF_UP_X(NI, false); } while (0)
    if (ni <= 1) LIF_UP(1);
    else if (ni <= 2) LIF_UP(2);
    else if (ni <= 4) LIF_UP(4);
    else if (ni <= 6) LIF_UP(6);
    else if (ni <= 8) LIF_UP(8);
    else if (ni <= 9) LIF_UP(9);
    else if (ni <= 12) LIF_UP(12);
    else LIF_UP(16);
#undef LIF_UP
#undef LIF_UP_X
}

// rows the launch geometry is made for: the row-count hint with some slack, else the capacity
int geometry_rows(const lif_layer* L) {
    return L->expected_rows > 0 ? std::min(L->cfg.capacity_rows, L->expected_rows + L->expected_rows / 8)
                                : L->cfg.capacity_rows;
}

// what the down projection of a fused step commits (`pass`: token-granular window update; the masks enter the ring here)
struct FusedCall {
    bool on = false;
    const uint8_t* masks = nullptr;
    int keep = 1;
    bool pass = false;
};
FusedRows fused_rows(const lif_layer* L, const FusedCall& f) {
    FusedRows r = {};
    if (!f.on) return r;
    r.h_new = L->h_new; r.stamp = L->stamp; r.ptr_new = L->ptr_new; r.bias_new = L->bias_new;
    r.pointers = L->buf.pointers; r.bias = L->buf.bias;
    if (f.pass) {
        r.masks = f.masks; r.ring = L->ring; r.ring_words = ring_words(L->cfg); r.nbytes = L->cfg.d_ffn / 8;
        r.k = L->cfg.window_k; r.keep = f.keep;
    }
    return r;
}

// one token
template <typename T, bool SKIP>
void launch_ffn_down1(lif_layer* L, void* y, float* h, float* ypart, hipStream_t s, const FusedCall& fc) {
    const lif_config& c = L->cfg;
    const int slices = down1_slices(c);
    const int rows = geometry_rows(L);
    // fewer workgroup rows than chunks are still correct; one, and no partial sums, where the hint itself needs one chunk
    const bool one = L->expected_rows > 0 && down1_chunks<SKIP>(L->expected_rows, slices) == 1;
    const int wg_rows = one ? 1 : down1_chunks<SKIP>(rows, slices);
    const int down_off = (c.glu ? 2 : 1) * c.d_model;
    // Waves of a workgroup: what the rows likely in use need, a little less than the hint says.  Any choice is correct, but a
    // workgroup of 8 goes twice through the work of 16 (Falcon shape, 5120 rows, skipping: 16.9 -> 19.3 us), while one of 16 leaves
    // half of its waves idle where 8 are in use, so without a hint 8 are taken only where every row is read and most layers of
    // this capacity hold more than one chunk (OPT shape, 8192 rows: 29.9 -> 28.3 us).
    // Few rows: 8 waves as long as a sixteenth more than the hint says are still few.  One FFN call in a graph, us, launched with 8 / 16
    // waves: d = 4096 2000 rows 6.8 / 7.0, 2060 rows 8.6 / 7.2; fp32 d = 2048 2000 rows 7.05 / 7.0, 2060 rows 8.75 / 7.3; a step with the
    // gate resident, d = 4096, rows around 1992 98.9 / 99.15, around 2255 107.5 / 104.7: to be wrong with 8 costs several times as much as
    // with 16, and the hint is a mean that the rows in use are around.
    const int told = L->expected_rows;
    const int likely = told > 0 ? (std::min(c.capacity_rows, told + told / 16) <= kDown1FewRows ? told : std::max(kDown1FewRows + 1, told - told / 8))
                       : rows <= kDown1FewRows ? rows : std::max(kDown1FewRows + 1, SKIP ? kDown1OneSkip : c.capacity_rows / 2);
    const int waves = down1_waves<SKIP>(likely, slices);
    // groups of slots whose activations are asked for ahead of the row count: those the hint covers; without a hint 2048
    // slots if that many rows make one pass (else the order of the slots is not known yet)
    const int spec = L->expected_rows > 0 || waves == 8 ? std::min(kDown1Per, (rows + waves * 64 - 1) / (waves * 64)) : 0;
    const FusedRows f = fused_rows(L, fc);
    const bool finish = told > 0 && wg_rows > 1 && down1_finish(down1_chunks<SKIP>(told, slices), slices);
#define LIF_D1(W, FUSED, SHARED)                                                                             \
    hipLaunchKernelGGL((k_ffn_down1<T, SKIP, W, FUSED, SHARED>), dim3(slices + (FUSED ? 1 : 0), wg_rows), dim3(W * 64), 0, s, \
                       (const T*)L->buf.matrix, h, f, (T*)y, ypart, L->arrived, c.d_model, c.capacity_rows, L->row_elems,        \
                       down_off, spec, slices, L->buf.pointers, L->gact, c.d_ffn, L->st)
#define LIF_D1W(W)                                                                                           \
    do {                                                                                                     \
        if (wg_rows == 1 || finish) { if (fc.on) LIF_D1(W, true, false); else LIF_D1(W, false, false); }     \
        else { if (fc.on) LIF_D1(W, true, true); else LIF_D1(W, false, true); }                              \
    } while (0)
    if (waves == 8) LIF_D1W(8);
    else LIF_D1W(16);
#undef LIF_D1W
#undef LIF_D1
    if (finish)
        hipLaunchKernelGGL((k_ffn_down_finish<T, double, down1_chunks<SKIP>>), dim3((c.d_model + 255) / 256), dim3(256), 0, s, ypart, (T*)y,
                           c.d_model, 1, slices, wg_rows, L->st);
}

// several tokens, fp32
template <typename T, int BT, bool SKIP>
void launch_ffn_down_batch(lif_layer* L, int batch, void* y, float* h, float* ypart, hipStream_t s, const FusedCall& fc) {
    const lif_config& c = L->cfg;
    constexpr int cols = kDownLanesB * Vec<T>::N;
    // workgroup rows: enough for the chunks of the expected number of rows; fewer than the chunks in use is still
    // correct (a workgroup row then takes several chunks)
    const int slices = (c.d_model + cols - 1) / cols;
    const int wg_rows = down_chunks(geometry_rows(L), slices);
    const int down_off = (c.glu ? 2 : 1) * c.d_model;
    const bool finish = !fc.on && L->expected_rows > 0 && wg_rows > 1 && down_finish(down_chunks(L->expected_rows, slices), slices, batch);
#define LIF_DB(FUSED, SHARED)                                                                                \
    hipLaunchKernelGGL((k_ffn_down<T, BT, SKIP, kDownLanesB, FUSED, SHARED>), dim3(slices + (FUSED ? 1 : 0), wg_rows), dim3(256),  \
                       0, s, (const T*)L->buf.matrix, h, fused_rows(L, fc), (T*)y, ypart, L->arrived, c.d_model, batch,          \
                       c.capacity_rows, L->row_elems, down_off, slices, L->st)
    if (wg_rows == 1 || finish) { if (fc.on) LIF_DB(true, false); else LIF_DB(false, false); }
    else { if (fc.on) LIF_DB(true, true); else LIF_DB(false, true); }
#undef LIF_DB
    if (finish)
        hipLaunchKernelGGL((k_ffn_down_finish<T, double, down_chunks>), dim3((batch * c.d_model + 255) / 256), dim3(256), 0, s, ypart, (T*)y,
                           c.d_model, batch, slices, wg_rows, L->st);
}

// several tokens, fp16: the down projection on the matrix cores
template <bool SKIP, int ROWS>
void launch_ffn_down_mfma_rows(lif_layer* L, int batch, void* y, float* h, float* ypart, hipStream_t s, const FusedCall& fc) {
    const lif_config& c = L->cfg;
    const int slices = (c.d_model + kDmCols - 1) / kDmCols;
    const int chunk_rows = down_mfma_chunk_rows(c.capacity_rows, slices);
    // workgroup rows: enough for the chunks of the expected number of rows (with some slack), else of the
    // capacity; fewer than the chunks in use is still correct (a workgroup row then takes several chunks)
    const int wg_rows = down_mfma_chunks(geometry_rows(L), chunk_rows);
    const int down_off = (c.glu ? 2 : 1) * c.d_model;
    const int told = L->expected_rows > 0 ? down_mfma_chunks(L->expected_rows, chunk_rows) : 0;       // chunks of the hint
    const bool finish = wg_rows > 1 && down_mfma_finish(wg_rows, fc.on ? 0 : told, slices, batch);
#define LIF_DM(FUSED, SHARED)                                                                                \
    hipLaunchKernelGGL((k_ffn_down_mfma<SKIP, kDmWaves, ROWS, FUSED, SHARED>), dim3(slices + (FUSED ? 1 : 0), wg_rows),       \
                       dim3(kDmWaves * 64), 0, s, (const _Float16*)L->buf.matrix, h, fused_rows(L, fc), (_Float16*)y,  \
                       ypart, L->arrived, c.d_model, batch, c.capacity_rows, L->row_elems, down_off, chunk_rows, slices, L->st)
    if (wg_rows == 1 || finish) { if (fc.on) LIF_DM(true, false); else LIF_DM(false, false); }
    else { if (fc.on) LIF_DM(true, true); else LIF_DM(false, true); }
#undef LIF_DM
    if (finish)
        hipLaunchKernelGGL((k_ffn_down_finish<_Float16, float, down_mfma_chunks>), dim3((batch * c.d_model + 255) / 256), dim3(256), 0, s,
                           ypart, (_Float16*)y, c.d_model, batch, chunk_rows, wg_rows, L->st);
}

template <bool SKIP>
void launch_ffn_down_mfma(lif_layer* L, int batch, void* y, float* h, float* ypart, hipStream_t s, const FusedCall& fc) {
    const int slices = (L->cfg.d_model + kDmCols - 1) / kDmCols;
    if (down_mfma_pass_rows(L->cfg.capacity_rows, slices) == kDmRowsFew) launch_ffn_down_mfma_rows<SKIP, kDmRowsFew>(L, batch, y, h, ypart, s, fc);
    else launch_ffn_down_mfma_rows<SKIP, kDmRows>(L, batch, y, h, ypart, s, fc);
}

template <typename T>
void launch_ffn_down(lif_layer* L, int batch, void* y, float* h, float* ypart, hipStream_t s, const FusedCall& fc = FusedCall()) {
    const bool skip = L->cfg.ffn_mode == LIF_FFN_SKIP_DEAD;
    if (batch == 1) {
        if (skip) launch_ffn_down1<T, true>(L, y, h, ypart, s, fc);
        else launch_ffn_down1<T, false>(L, y, h, ypart, s, fc);
        return;
    }
    if constexpr (std::is_same<T, _Float16>::value) {
        if (skip) launch_ffn_down_mfma<true>(L, batch, y, h, ypart, s, fc);
        else launch_ffn_down_mfma<false>(L, batch, y, h, ypart, s, fc);
    } else if (batch <= 4) {
        if (skip) launch_ffn_down_batch<T, 4, true>(L, batch, y, h, ypart, s, fc);
        else launch_ffn_down_batch<T, 4, false>(L, batch, y, h, ypart, s, fc);
    } else {
        if (skip) launch_ffn_down_batch<T, 8, true>(L, batch, y, h, ypart, s, fc);
        else launch_ffn_down_batch<T, 8, false>(L, batch, y, h, ypart, s, fc);
    }
}

// One token in one launch, where few workgroups wait for few words.  What the waiting costs grows with slices x rows (every word
// is read by every slice), what the second launch costs does not.  us a call, two launches -> one, twenty calls in a graph / from the
// host (rows in use, the hint 1.15 times as many): 64 slices, d = 2048 341: 5.9 -> 5.4 / 6.8 -> 5.5, 685: 6.0 -> 5.8 / 6.8 -> 5.8 (8.8 -> 6.4 where
// the host is slow), 1111: 6.1 -> 6.1 / 6.7 -> 6.3; 48 slices 685: 6.0 -> 5.9 / 6.8 -> 5.7, 1111: 6.1 -> 6.0 / 6.8 -> 6.0; 32 slices 1111:
// 6.0 -> 5.8 / 6.8 -> 5.7; fp32, 64 slices, d = 1024 685: 6.4 -> 5.6 / 6.9 -> 5.6.  Rows gated or read in full are longer on their way:
// 64 slices 685: gated 6.15 -> 6.27 / 6.8 -> 6.3, in full 6.45 -> 6.55 / 6.8 -> 6.4, so half as many words there.  128 slices (OPT shape),
// 927: 6.5 -> 7.2 / 8.8 -> 7.7, 7.4 -> 7.9 where the host is fast: two launches.
// Without a hint the capacity counts, and every slot of it has a wave in the launch (rows in use of capacity): 64 slices 174 of 500: 5.8 ->
// 5.45 / 8.6 -> 5.6, gated 194 of 500 5.9 -> 5.55 / 8.8 -> 5.8, in full 174 of 500 5.9 -> 5.6 / 8.7 -> 5.7, 174 of 1000 5.7 -> 6.0 / 8.7 ->
// 6.2, 552 of 1000 6.0 -> 6.5 / 8.7 -> 6.6; 32 slices 164 of 2000 5.5 -> 5.1 / 8.7 -> 5.3, 970 of 2000 5.9 -> 5.4 / 8.5 -> 5.8; fp32, 64
// slices 369 of 1000 6.0 -> 6.0 / 8.7 -> 6.3: what a graph loses at the end of the range is a fifth of what the host gains.
bool ffn_one(const lif_layer* L, int batch) {
    const int rows = geometry_rows(L), slices = down1_slices(L->cfg);
    const int most = L->cfg.glu || L->cfg.ffn_mode == LIF_FFN_FULL_BUNDLE ? kOneWords / 2 : kOneWords;
    return batch == 1 && L->one_words && rows <= kOneRows && slices * rows <= most;
}
template <typename T, bool GLU, bool SKIP>
void launch_ffn_one(lif_layer* L, const void* x, void* y, hipStream_t s) {
    const lif_config& c = L->cfg;
    const int ni = (c.d_model / Vec<T>::N + 63) / 64, slices = down1_slices(c), spec = L->expected_rows > 0 ? 1 : 0;
    const int rows = spec ? L->expected_rows : c.capacity_rows;
    const int n_up = std::max(1, (rows + kOneUpWaves - 1) / kOneUpWaves);
#define LIF_ONE(NI)                                                                                          \
    hipLaunchKernelGGL((k_ffn_one<T, NI, GLU, SKIP>), dim3(n_up + slices), dim3(kOneWaves * 64), 0, s,              \
                       (const T*)L->buf.matrix, L->buf.bias, (const T*)x, (T*)y, c.d_model, c.capacity_rows, L->row_elems, \
                       spec, n_up, slices, L->one_words, L->one, L->polls, L->buf.pointers, L->gact, c.d_ffn, L->st)
    if (ni <= 1) LIF_ONE(1);
    else if (ni <= 2) LIF_ONE(2);
    else LIF_ONE(4);                   // d <= kOneSlices slices
#undef LIF_ONE
}
template <typename T>
void launch_ffn_one(lif_layer* L, const void* x, void* y, hipStream_t s) {
    const bool skip = L->cfg.ffn_mode == LIF_FFN_SKIP_DEAD;
    if (L->cfg.glu) skip ? launch_ffn_one<T, true, true>(L, x, y, s) : launch_ffn_one<T, true, false>(L, x, y, s);
    else skip ? launch_ffn_one<T, false, true>(L, x, y, s) : launch_ffn_one<T, false, false>(L, x, y, s);
}

// bundles of host reads kept in flight
int loader_pairs(const lif_layer* L, size_t inflight, int most) {
    if (L->loader_pairs > 0) return L->loader_pairs;
    return std::min(most, std::max(5, (int)std::min<size_t>(inflight / L->row_bytes, most)));
}

// arguments that both forms of a fused step take
StepArgs step_args(lif_layer* L, const void* x, uint8_t* masks, uint8_t* step_mask, int32_t* added, int32_t* n_added,
                   int32_t* removed, int32_t* n_removed, int batch) {
    const lif_config& c = L->cfg;
    const int words = ring_words(c);
    StepArgs a = {};
    a.A = L->buf.A; a.B = L->buf.B; a.c = L->buf.c; a.rank = c.rank; a.theta = c.threshold;
    a.t_pitch = words_pitch(2 * std::max(c.rank, 0)); a.m_pitch = words_pitch(2 * words);
    a.t_words = L->words; a.m_words = L->words + (size_t)kWordReps * a.t_pitch;
    a.plan_words = a.m_words + (size_t)kWordReps * a.m_pitch;
    a.masks = masks; a.step_mask = step_mask; a.gact = L->gact;
    a.ring = L->ring; a.cur_set = L->ring + (size_t)c.window_k * words; a.ring_words = words;
    a.k = c.window_k; a.shrink = c.shrink_window;
    a.added = added; a.n_added = n_added; a.removed = removed; a.n_removed = n_removed; a.hole_list = L->hole_list;
    a.matrix = L->buf.matrix; a.pointers = L->buf.pointers; a.bias = L->buf.bias; a.host = L->host; a.b = L->buf.b;
    a.row_elems = L->row_elems; a.F = c.d_ffn; a.d = c.d_model; a.capacity = c.capacity_rows;
    a.x = x; a.h = L->h; a.h_new = L->h_new; a.stamp = L->stamp; a.ptr_new = L->ptr_new; a.bias_new = L->bias_new;
    a.batch = batch; a.keep = 1; a.polls = L->polls; a.st = L->st;
    // loader waves: two per bundle in flight
    const size_t vector = (size_t)c.d_model * elem_bytes(c);
    a.n_load = 2 * (batch > 1              ? loader_pairs(L, kStepInflightBytesB, kStepPairsB)
                    : vector <= 2 * 1024   ? loader_pairs(L, kStepInflightBytesWhole / 2, kStepPairsWhole)
                    : vector <= 12 * 1024  ? loader_pairs(L, kStepInflightBytes, kStepPairs)
                                           : loader_pairs(L, kStepPairsWide * L->row_bytes, kStepPairsWide));
    return a;
}
// workgroups of the activation role with one wave per row; with a row-count hint the grid is sized to it
int up_blocks(const lif_layer* L) {
    return L->expected_rows > 0 ? std::min(kUpMaxWgs, std::max(1, L->expected_rows / 4))
                                : std::min((L->cfg.capacity_rows + 3) / 4, 512);
}

// one token: everything up to the down projection
void launch_step1(lif_layer* L, StepArgs a, hipStream_t s) {
    const lif_config& c = L->cfg;
    const bool gate = c.predictor == LIF_PRED_GATE;
    // predictor workgroups: one per 64 neurons (32 with the gate predictor), and one per column of A as far as kStepColumns
    a.n_pred = gate ? 2 * a.ring_words : std::max(a.ring_words, std::min(c.rank, kStepColumns));
    a.spec = L->expected_rows > 0 ? 1 : 0;
    const int grid = a.n_pred + 1 + a.n_load + up_blocks(L);
    if (c.dtype == LIF_F32) (gate ? launch_step1_f32_gate : c.glu ? launch_step1_f32_glu : launch_step1_f32_plain)(a, grid, s);
    else (gate ? launch_step1_f16_gate : c.glu ? launch_step1_f16_glu : launch_step1_f16_plain)(a, grid, s);
}

bool mfma_path(const lif_config& c, int batch) {
    return c.dtype == LIF_F16 && batch > 1 && c.d_model % 32 == 0;
}

// 16-row tiles a row-count hint covers (at least one)
int mfma_hint_tiles(const lif_layer* L) { return std::max(1, (L->expected_rows + 15) / 16); }

// several tokens, the predictor's launches done: window, load and activations (allow: see launch_step_batch_as)
hipError_t launch_step_batch(lif_layer* L, StepArgs a, bool allow, hipStream_t s) {
    const lif_config& c = L->cfg;
    const bool mfma = mfma_path(c, 2);
    a.x_pitch = step_x_pitch(c.d_model, elem_bytes(c));
    // (one row always fits)
    a.stage_rows = 2;
    size_t lds = step_batch_lds(a.batch, c.d_model, elem_bytes(c), c.glu, mfma, 2);
    if (lds > kStepLdsLimit) {
        a.stage_rows = 1;
        lds = step_batch_lds(a.batch, c.d_model, elem_bytes(c), c.glu, mfma, 1);
    }
    int up;
    if (mfma) {
        up = (c.capacity_rows + 15) / 16;
        a.spec = L->expected_rows > 0 ? mfma_hint_tiles(L) : 0;
    } else {
        const int waves = step_batch_waves((c.d_model / vec_elems(c) + 63) / 64, c.glu, mfma, lds);
        up = (4 * up_blocks(L) + waves - 1) / waves;
        a.spec = L->expected_rows > 0 ? 1 : 0;
    }
    const int grid = 1 + a.n_load + up;
    const bool gate = c.predictor == LIF_PRED_GATE;
#define LIF_FORM(NAME) (gate ? launch_step_batch_##NAME##_gate : c.glu ? launch_step_batch_##NAME##_glu : launch_step_batch_##NAME##_plain)
    if (c.dtype == LIF_F32) return LIF_FORM(f32)(a, grid, lds, allow, s);
    if (mfma) return LIF_FORM(f16_mfma)(a, grid, lds, allow, s);
    return LIF_FORM(f16)(a, grid, lds, allow, s);
#undef LIF_FORM
}

void launch_ffn_up_mfma(lif_layer* L, const void* x, int batch, float* h, hipStream_t s) {
    const lif_config& c = L->cfg;
    // with a row-count hint the grid is sized to it (a workgroup strides on if more rows are in use) and every
    // workgroup asks for its first rows before the count arrives
    const int spec = L->expected_rows > 0 ? 1 : 0;
    const int grid = spec ? mfma_hint_tiles(L) : (c.capacity_rows + 15) / 16;
    const bool few = spec && up_mfma_waves(grid, c.d_model, c.glu != 0) == kMfmaWavesFew;      // (without a hint most tiles are likely not in use)
#define LIF_UM(GLU, W)                                                                                       \
    hipLaunchKernelGGL((k_ffn_up_mfma<GLU, W>), dim3(grid), dim3(W * 64), 0, s, (const _Float16*)L->buf.matrix,  \
                       L->buf.bias, (const _Float16*)x, h, c.d_model, batch, c.capacity_rows, L->row_elems,        \
                       L->buf.pointers, L->gact, c.d_ffn, spec, L->st)
    if (c.glu && few) LIF_UM(true, kMfmaWavesFew);
    else if (c.glu) LIF_UM(true, kMfmaWavesAll);
    else if (few) LIF_UM(false, kMfmaWavesFew);
    else LIF_UM(false, kMfmaWavesAll);
#undef LIF_UM
}

// Bandwidth reference: every 16-byte piece of [src, src + bytes) is read once; the pieces are folded into one word
// per workgroup so that the loads cannot be dropped.  bytes = 0: an empty launch.  grid-stride, eight loads per
// thread in flight.
constexpr int kProbePer = 8;
__global__ __launch_bounds__(256) void k_probe_read(const uint4* __restrict__ src, size_t pieces,
                                                    unsigned* __restrict__ sink) {
    unsigned acc = 0;
    const size_t stride = (size_t)gridDim.x * 256 * kProbePer;
    for (size_t base = (size_t)blockIdx.x * 256 * kProbePer; base < pieces; base += stride) {
        uint4 v[kProbePer];
#pragma unroll
        for (int p = 0; p < kProbePer; ++p) {
            const size_t i = base + (size_t)p * 256 + threadIdx.x;
            v[p] = i < pieces ? src[i] : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int p = 0; p < kProbePer; ++p) acc ^= v[p].x ^ v[p].y ^ v[p].z ^ v[p].w;
    }
    if (pieces == 0) return;
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) acc ^= __shfl_xor(acc, m, kWave);
    if ((threadIdx.x & 63) == 0 && acc == 0x9e3779b9u) sink[0] = acc;      // practically never: keeps the loads alive
}

// Cost reference for merging two dependent kernels without a second launch: 256 workgroups read 16 KiB each and
// produce 8 bytes (the shape of the mask kernel), then hand them to one workgroup of the same launch.
//   mode 0  no hand-off: every workgroup writes its 8 bytes and ends
//   mode 1  fence + ticket: every workgroup passes a device-scope fence and takes a ticket; the last to arrive reads
//           the 2 KiB the others wrote.  No workgroup waits.
//   mode 2  no fences: the 8 bytes go out as two 64-bit words (32 bits of payload + the launch's 32-bit stamp) by
//           relaxed device-scope atomic stores; workgroup 0 polls all 512 words with relaxed device-scope atomic loads
//           until they carry this launch's stamp.  The wait is bounded (kHandoffPolls per word, then it gives up and
//           counts the give-up) and the grid of 256 workgroups is resident as a whole on the 256 compute units.
constexpr int kHandoffWgs = 256;
constexpr int kHandoffPolls = 20000;
__global__ __launch_bounds__(256) void k_probe_handoff(const uint4* __restrict__ src, unsigned long long* __restrict__ words,
                                                       unsigned* __restrict__ counter, unsigned long long* __restrict__ out,
                                                       int mode, unsigned stamp) {
    __shared__ unsigned ticket;
    __shared__ unsigned long long part[4];
    const int tid = threadIdx.x;
    uint4 v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = src[(size_t)blockIdx.x * 1024 + i * 256 + tid];
    unsigned long long bits = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) bits ^= ((unsigned long long)(v[i].x ^ v[i].z) << 32) | (v[i].y ^ v[i].w);
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) bits ^= __shfl_xor(bits, m, kWave);
    if ((tid & 63) == 0) part[tid >> 6] = bits;
    __syncthreads();
    const unsigned long long mine = part[0] ^ part[1] ^ part[2] ^ part[3];
    if (mode == 2) {
        if (tid < 2) {
            const unsigned long long w = ((unsigned long long)stamp << 32) | (unsigned)(tid ? (mine >> 32) : mine);
            __hip_atomic_store(&words[blockIdx.x * 2 + tid], w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (blockIdx.x != 0) return;
        unsigned long long acc = 0;
        bool ok = true;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            unsigned long long w = 0;
            int polls = 0;
            do {
                w = __hip_atomic_load(&words[tid * 2 + j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } while ((unsigned)(w >> 32) != stamp && ++polls < kHandoffPolls);
            ok = ok && (unsigned)(w >> 32) == stamp;
            acc ^= w & 0xffffffffull;
        }
        if (!ok) atomicAdd(counter + 1, 1u);           // give-ups, reported by the caller
#pragma unroll
        for (int sft = 32; sft >= 1; sft >>= 1) acc ^= __shfl_xor(acc, sft, kWave);
        __syncthreads();
        if ((tid & 63) == 0) part[tid >> 6] = acc;
        __syncthreads();
        if (tid == 0) out[0] = part[0] ^ part[1] ^ part[2] ^ part[3];
        return;
    }
    if (tid == 0) words[blockIdx.x] = mine;
    if (mode == 0) return;
    if (tid == 0) {
        __threadfence();
        ticket = atomicAdd(counter, 1u);
    }
    __syncthreads();
    if (ticket != gridDim.x - 1) return;
    __threadfence();
    unsigned long long m = words[tid];                // gridDim.x == 256 == blockDim.x
#pragma unroll
    for (int sft = 32; sft >= 1; sft >>= 1) m ^= __shfl_xor(m, sft, kWave);
    if ((tid & 63) == 0) part[tid >> 6] = m;
    __syncthreads();
    if (tid == 0) {
        out[0] = part[0] ^ part[1] ^ part[2] ^ part[3];
        *counter = 0;                                 // ready for the next launch on this stream
    }
}

int check_launch() {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(LIF_HIP_ERROR, "kernel launch: %s", hipGetErrorString(e));
    return LIF_OK;
}

}  // namespace

extern "C" {

int lif_version(void) { return 2; }

const char* lif_last_error_string(void) { return g_err; }

size_t lif_workspace_bytes(const lif_config* cfg) {
    const char* why;
    if (!config_ok(cfg, &why)) return 0;
    return make_layout(*cfg).total;
}

int lif_create(const lif_config* cfg, const lif_buffers* buf, lif_layer** out) {
    const char* why;
    if (!out) return fail(LIF_INVALID_ARG, "out is null");
    *out = nullptr;
    if (!config_ok(cfg, &why)) return fail(LIF_INVALID_ARG, "invalid config: %s", why);
    if (!buf) return fail(LIF_INVALID_ARG, "buffers are null");
    if (!buf->A || (!buf->B && cfg->predictor != LIF_PRED_GATE) || !buf->b || !buf->host_bundles || !buf->matrix || !buf->pointers || !buf->bias ||
        !buf->workspace)
        return fail(LIF_INVALID_ARG, "a required buffer is null");
    const void* ptrs[] = {buf->A, buf->B ? buf->B : buf->A, buf->host_bundles, buf->matrix};
    for (const void* p : ptrs)
        if ((uintptr_t)p % 16) return fail(LIF_INVALID_ARG, "A, B, host_bundles and matrix must be 16-byte aligned");
    if ((uintptr_t)buf->workspace % 256) return fail(LIF_INVALID_ARG, "workspace must be 256-byte aligned");
    Layout lay = make_layout(*cfg);
    if (buf->workspace_bytes < lay.total) return fail(LIF_INVALID_ARG, "workspace smaller than lif_workspace_bytes");

    void* alias = nullptr;
    LIF_HIP(hipHostGetDevicePointer(&alias, const_cast<void*>(buf->host_bundles), 0));
    if (!alias) return fail(LIF_HIP_ERROR, "bundle store has no device alias");
    void* alias_down = nullptr;
    if (buf->host_down) {
        if ((uintptr_t)buf->host_down % 16) return fail(LIF_INVALID_ARG, "host_down must be 16-byte aligned");
        LIF_HIP(hipHostGetDevicePointer(&alias_down, const_cast<void*>(buf->host_down), 0));
        if (!alias_down) return fail(LIF_HIP_ERROR, "down-column store has no device alias");
    }

    lif_layer* L = new (std::nothrow) lif_layer();
    if (!L) return fail(LIF_INVALID_ARG, "out of host memory");
    L->cfg = *cfg;
    L->buf = *buf;
    L->lay = lay;
    L->host.rows = (const char*)alias;
    L->host.down = (const char*)alias_down;
    L->host.act_bytes = (size_t)(cfg->glu ? 2 : 1) * cfg->d_model * elem_bytes(*cfg);
    L->loader_pairs = 0;
    char* ws = (char*)buf->workspace;
    L->st = (DevState*)(ws + lay.state);
    L->ring = (unsigned long long*)(ws + lay.ring);
    L->tpart = (double*)(ws + lay.tpart);
    L->move_dst = (int32_t*)(ws + lay.move_dst);
    L->hole_list = (int32_t*)(ws + lay.hole_list);
    L->h = (float*)(ws + lay.h);
    L->ypart = (float*)(ws + lay.ypart);
    L->h_new = (float*)(ws + lay.h_new);
    L->stamp = (int32_t*)(ws + lay.stamp);
    L->ptr_new = (int32_t*)(ws + lay.ptr_new);
    L->bias_new = (float*)(ws + lay.bias_new);
    L->words = (unsigned long long*)(ws + lay.words);
    L->one_words = ffn_one_possible(*cfg) ? (unsigned long long*)(ws + lay.one) : nullptr;
    L->one = L->one_words ? (OneState*)(L->one_words + kOneReps * one_pitch(cfg->capacity_rows)) : nullptr;
    L->arrived = (unsigned*)(ws + lay.arrived);
    L->polls = kDefaultPolls;
    L->gact = cfg->predictor == LIF_PRED_GATE ? (float*)(ws + lay.gact) : nullptr;
    L->row_elems = (size_t)(cfg->glu ? 3 : 2) * cfg->d_model;
    L->row_bytes = L->row_elems * elem_bytes(*cfg);
    L->window_pending = false;
    L->expected_rows = 0;
    L->prof_on = false;
    L->prof_max = 0;
    {
        // address of the static scratch array on the device that is current now (the layer's device)
        void* p = nullptr;
        hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        L->static_scratch = (e == hipSuccess) ? (unsigned char*)p : nullptr;
        if (e != hipSuccess) (void)hipGetLastError();      // reported by lif_sparse_ffn_static, not by a later launch
    }
    if (cfg->max_batch > 1) {
        StepArgs a = {};                                     // (the row width names the kernel form)
        a.d = cfg->d_model;
        a.batch = cfg->max_batch;
        hipError_t e = launch_step_batch(L, a, true, nullptr);
        if (e != hipSuccess) {
            delete L;
            return fail(LIF_HIP_ERROR, "LDS of the batched step: %s", hipGetErrorString(e));
        }
    }
    *out = L;
    return LIF_OK;
}

int lif_destroy(lif_layer* layer) {
    if (!layer) return LIF_OK;
    for (hipEvent_t e : layer->ev) (void)hipEventDestroy(e);
    delete layer;
    return LIF_OK;
}

int lif_reset(lif_layer* L, void* stream) {
    if (!L) return fail(LIF_INVALID_ARG, "layer is null");
    hipStream_t s = (hipStream_t)stream;
    const int grid = std::min((L->lay.reset_words + 255) / 256, 256);
    hipLaunchKernelGGL(k_reset, dim3(grid), dim3(256), 0, s, L->words, L->lay.reset_words, L->stamp, L->cfg.capacity_rows,
                       L->st);
    L->window_pending = false;
    return check_launch();
}

static int check_predict(lif_layer* L, const void* x_dev, int32_t batch, uint8_t* masks_dev, uint8_t* step_mask_dev) {
    if (!L || !x_dev || !masks_dev || !step_mask_dev) return fail(LIF_INVALID_ARG, "null argument");
    if (batch < 1 || batch > L->cfg.max_batch) return fail(LIF_INVALID_ARG, "batch out of range");
    if ((uintptr_t)x_dev % 16) return fail(LIF_INVALID_ARG, "x must be 16-byte aligned");
    if (batch > 1 && masks_dev == step_mask_dev) return fail(LIF_INVALID_ARG, "step mask must not alias the masks when batch > 1");
    return LIF_OK;
}

int lif_predict(lif_layer* L, const void* x_dev, int32_t batch, uint8_t* masks_dev, uint8_t* step_mask_dev,
                void* stream) {
    int rc = check_predict(L, x_dev, batch, masks_dev, step_mask_dev);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    if (L->cfg.predictor == LIF_PRED_GATE) {
        if (L->cfg.dtype == LIF_F32) launch_predict_gate<float>(L, x_dev, batch, masks_dev, step_mask_dev, s);
        else launch_predict_gate<_Float16>(L, x_dev, batch, masks_dev, step_mask_dev, s);
    } else if (L->cfg.dtype == LIF_F32) {
        launch_predict<float>(L, x_dev, batch, masks_dev, step_mask_dev, s);
    } else {
        launch_predict<_Float16>(L, x_dev, batch, masks_dev, step_mask_dev, s);
    }
    return check_launch();
}

static int check_update_window(lif_layer* L, const uint8_t* masks_dev, const int32_t* added_dev,
                               const int32_t* n_added_dev, const int32_t* removed_dev, const int32_t* n_removed_dev) {
    if (!L || !masks_dev || !added_dev || !n_added_dev || !removed_dev || !n_removed_dev)
        return fail(LIF_INVALID_ARG, "null argument");
    if ((uintptr_t)masks_dev % 8) return fail(LIF_INVALID_ARG, "step mask must be 8-byte aligned");
    if (L->window_pending) return fail(LIF_BAD_STATE, "lif_update_window called twice without lif_load_bundles");
    return LIF_OK;
}

static int check_window_tokens(lif_layer* L, int32_t n_tokens, int32_t keep) {
    if (!L) return fail(LIF_INVALID_ARG, "layer is null");
    if (n_tokens < 1 || n_tokens > L->cfg.max_batch) return fail(LIF_INVALID_ARG, "n_tokens out of range");
    if (keep < 0 || keep > n_tokens) return fail(LIF_INVALID_ARG, "keep must be in 0..n_tokens");
    if (L->cfg.d_ffn % 64) return fail(LIF_INVALID_ARG, "token-granular window updates need d_ffn % 64 == 0");
    return LIF_OK;
}

static int update_window_impl(lif_layer* L, const uint8_t* masks_dev, int ntok, int keep, int32_t* added_dev,
                              int32_t* n_added_dev, int32_t* removed_dev, int32_t* n_removed_dev, void* stream) {
    int rc = check_update_window(L, masks_dev, added_dev, n_added_dev, removed_dev, n_removed_dev);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    const lif_config& c = L->cfg;
    {
        Timed t(L, LIF_K_WINDOW, s);
        hipLaunchKernelGGL(k_window_plan, dim3(1), dim3(kScanThreads), 0, s, masks_dev, ntok, keep, L->ring,
                           L->ring + (size_t)c.window_k * ring_words(c), ring_words(c), L->buf.pointers, c.d_ffn,
                           c.window_k, c.capacity_rows, c.shrink_window, added_dev, n_added_dev, removed_dev,
                           n_removed_dev, L->move_dst, L->hole_list, L->st);
    }
    L->window_pending = true;
    return check_launch();
}

int lif_update_window(lif_layer* L, const uint8_t* step_mask_dev, int32_t* added_dev, int32_t* n_added_dev,
                      int32_t* removed_dev, int32_t* n_removed_dev, void* stream) {
    return update_window_impl(L, step_mask_dev, 1, 1, added_dev, n_added_dev, removed_dev, n_removed_dev, stream);
}

int lif_update_window_tokens(lif_layer* L, const uint8_t* masks_dev, int32_t n_tokens, int32_t keep,
                             int32_t* added_dev, int32_t* n_added_dev, int32_t* removed_dev, int32_t* n_removed_dev,
                             void* stream) {
    int rc = check_window_tokens(L, n_tokens, keep);
    if (rc) return rc;
    if (n_tokens == 1 && keep == 1)
        return update_window_impl(L, masks_dev, 1, 1, added_dev, n_added_dev, removed_dev, n_removed_dev, stream);
    return update_window_impl(L, masks_dev, n_tokens, keep, added_dev, n_added_dev, removed_dev, n_removed_dev, stream);
}

int lif_load_bundles(lif_layer* L, const int32_t* added_dev, const int32_t* n_added_dev, const int32_t* removed_dev,
                     const int32_t* n_removed_dev, void* stream) {
    if (!L || !added_dev || !n_added_dev || !removed_dev || !n_removed_dev)
        return fail(LIF_INVALID_ARG, "null argument");
    if (!L->window_pending) return fail(LIF_BAD_STATE, "lif_load_bundles needs a preceding lif_update_window");
    hipStream_t s = (hipStream_t)stream;
    const lif_config& c = L->cfg;
    {
        const int chunks = load_chunks(L->row_bytes);
        const int chunk_bytes = (int)align_up((L->row_bytes + chunks - 1) / chunks, 16);
        const int grid = (int)std::min<long long>((long long)c.capacity_rows * chunks, 2 * loader_pairs(L, kLoadInflightBytes, kStepPairs));
        Timed t(L, LIF_K_LOAD, s);
#define LIF_LD(NP)                                                                                                       \
    case NP:                                                                                                             \
        hipLaunchKernelGGL(k_load<NP>, dim3(grid), dim3(64), 0, s, (char*)L->buf.matrix, L->buf.pointers, L->buf.bias,     \
                           L->host, L->buf.b, added_dev, L->move_dst, L->row_bytes, chunks, chunk_bytes, c.d_ffn,          \
                           c.capacity_rows, L->st);                                                                        \
        break
        switch ((chunk_bytes + 1023) / 1024) {
            LIF_LD(1); LIF_LD(2); LIF_LD(3); LIF_LD(4); LIF_LD(5); LIF_LD(6); LIF_LD(7); LIF_LD(8);
        }
#undef LIF_LD
    }
    L->window_pending = false;
    return check_launch();
}

static int check_ffn(lif_layer* L, const void* x_dev, int32_t batch, void* y_dev) {
    if (!L || !x_dev || !y_dev) return fail(LIF_INVALID_ARG, "null argument");
    if (batch < 1 || batch > L->cfg.max_batch) return fail(LIF_INVALID_ARG, "batch out of range");
    if ((uintptr_t)x_dev % 16 || (uintptr_t)y_dev % 16) return fail(LIF_INVALID_ARG, "x and y must be 16-byte aligned");
    return LIF_OK;
}

// the two FFN stages with their scratch: activations h, partial outputs ypart
static int ffn_launches(lif_layer* L, const void* x_dev, int32_t batch, void* y_dev, float* h, float* ypart,
                        hipStream_t s) {
    const lif_config& c = L->cfg;
    if (ffn_one(L, batch)) {
        Timed t(L, LIF_K_FFN_DOWN, s);
        if (c.dtype == LIF_F32) launch_ffn_one<float>(L, x_dev, y_dev, s);
        else launch_ffn_one<_Float16>(L, x_dev, y_dev, s);
        return check_launch();
    }
    if (mfma_path(c, batch)) {
        // batched tokens: the activation stage is a dense contraction -> matrix cores
        Timed t(L, LIF_K_FFN_UP, s);
        launch_ffn_up_mfma(L, x_dev, batch, h, s);
    } else {
        Timed t(L, LIF_K_FFN_UP, s);
        if (c.dtype == LIF_F32) {
            if (c.glu) launch_ffn_up<float, true>(L, x_dev, batch, h, s);
            else launch_ffn_up<float, false>(L, x_dev, batch, h, s);
        } else {
            if (c.glu) launch_ffn_up<_Float16, true>(L, x_dev, batch, h, s);
            else launch_ffn_up<_Float16, false>(L, x_dev, batch, h, s);
        }
    }
    {
        Timed t(L, LIF_K_FFN_DOWN, s);
        if (c.dtype == LIF_F32) launch_ffn_down<float>(L, batch, y_dev, h, ypart, s);
        else launch_ffn_down<_Float16>(L, batch, y_dev, h, ypart, s);
    }
    return check_launch();
}

int lif_sparse_ffn(lif_layer* L, const void* x_dev, int32_t batch, void* y_dev, void* stream) {
    int rc = check_ffn(L, x_dev, batch, y_dev);
    if (rc) return rc;
    return ffn_launches(L, x_dev, batch, y_dev, L->h, L->ypart, (hipStream_t)stream);
}

size_t lif_static_scratch_bytes(void) { return kStaticScratchBytes; }

int lif_sparse_ffn_static(lif_layer* L, const void* x_dev, int32_t batch, void* y_dev, void* stream) {
    int rc = check_ffn(L, x_dev, batch, y_dev);
    if (rc) return rc;
    if (!L->static_scratch) return fail(LIF_HIP_ERROR, "the static scratch array has no address on this device");
    // activations [batch x capacity_rows] fp32, then the partial outputs [row chunks x batch x d_model] fp32
    const lif_config& c = L->cfg;
    const size_t h_bytes = align_up(sizeof(float) * (size_t)batch * c.capacity_rows, 256);
    const size_t ypart_bytes = sizeof(float) * (size_t)kDownChunksMax * batch * c.d_model;
    if (h_bytes + ypart_bytes > kStaticScratchBytes)
        return fail(LIF_INVALID_ARG, "batch x capacity_rows and batch x d_model exceed the static scratch (5 MiB); use lif_sparse_ffn");
    // the kernels take the scratch as arguments, exactly as they take the workspace arrays in lif_sparse_ffn;
    // nothing in it has to start at zero: every activation and every partial that is read was written by this call
    return ffn_launches(L, x_dev, batch, y_dev, reinterpret_cast<float*>(L->static_scratch),
                        reinterpret_cast<float*>(L->static_scratch + h_bytes), (hipStream_t)stream);
}

// keep < 0: the window advances by one step whose mask is the OR over the batch (lif_update_window);
// keep >= 0: token-granular update of a speculative pass (lif_update_window_tokens)
static int step_impl(lif_layer* L, const void* x_dev, int32_t batch, int32_t keep, void* y_dev, uint8_t* masks_dev,
                     uint8_t* step_mask_dev, int32_t* added_dev, int32_t* n_added_dev, int32_t* removed_dev,
                     int32_t* n_removed_dev, void* stream) {
    // every argument and call-order check of the four calls comes before the first launch: a rejected step
    // leaves the device buffers untouched
    int rc = check_predict(L, x_dev, batch, masks_dev, step_mask_dev);
    if (rc) return rc;
    if (!y_dev || (uintptr_t)y_dev % 16) return fail(LIF_INVALID_ARG, "y must be a 16-byte aligned device pointer");
    if (keep >= 0 && (rc = check_window_tokens(L, batch, keep))) return rc;
    rc = check_update_window(L, keep < 0 ? step_mask_dev : masks_dev, added_dev, n_added_dev, removed_dev, n_removed_dev);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    const lif_config& c = L->cfg;
    // Passes of tokens that go through the separate kernels: one token that is not kept, and a step mask that k_step_batch
    // cannot read by 64-bit words.
    if (keep >= 0 && ((batch == 1 && keep == 0) || (batch > 1 && (uintptr_t)step_mask_dev % 8))) {
        rc = lif_predict(L, x_dev, batch, masks_dev, step_mask_dev, stream);
        if (!rc) rc = lif_update_window_tokens(L, masks_dev, batch, keep, added_dev, n_added_dev, removed_dev, n_removed_dev, stream);
        if (!rc) rc = lif_load_bundles(L, added_dev, n_added_dev, removed_dev, n_removed_dev, stream);
        return rc ? rc : lif_sparse_ffn(L, x_dev, batch, y_dev, stream);
    }
    StepArgs a = step_args(L, x_dev, masks_dev, step_mask_dev, added_dev, n_added_dev, removed_dev, n_removed_dev, batch);
    FusedCall fc;
    fc.on = true;
    if (batch > 1) {
        if (keep >= 0) {
            a.multi = fc.pass = true;
            a.keep = fc.keep = keep;
            fc.masks = masks_dev;
        }
        rc = lif_predict(L, x_dev, batch, masks_dev, step_mask_dev, stream);
        if (rc) return rc;
    }
    {
        Timed t(L, LIF_K_LOAD, s);
        if (batch == 1) launch_step1(L, a, s);
        else LIF_HIP(launch_step_batch(L, a, false, s));
    }
    Timed t(L, LIF_K_FFN_DOWN, s);
    if (c.dtype == LIF_F32) launch_ffn_down<float>(L, batch, y_dev, L->h, L->ypart, s, fc);
    else launch_ffn_down<_Float16>(L, batch, y_dev, L->h, L->ypart, s, fc);
    return check_launch();
}

int lif_step(lif_layer* L, const void* x_dev, int32_t batch, void* y_dev, uint8_t* masks_dev,
             uint8_t* step_mask_dev, int32_t* added_dev, int32_t* n_added_dev, int32_t* removed_dev,
             int32_t* n_removed_dev, void* stream) {
    return step_impl(L, x_dev, batch, -1, y_dev, masks_dev, step_mask_dev, added_dev, n_added_dev, removed_dev,
                     n_removed_dev, stream);
}

int lif_step_tokens(lif_layer* L, const void* x_dev, int32_t n_tokens, int32_t keep_tokens, void* y_dev,
                    uint8_t* masks_dev, uint8_t* step_mask_dev, int32_t* added_dev, int32_t* n_added_dev,
                    int32_t* removed_dev, int32_t* n_removed_dev, void* stream) {
    if (keep_tokens < 0) return fail(LIF_INVALID_ARG, "keep must be in 0..n_tokens");
    return step_impl(L, x_dev, n_tokens, keep_tokens, y_dev, masks_dev, step_mask_dev, added_dev, n_added_dev,
                     removed_dev, n_removed_dev, stream);
}

int lif_set_loader_pairs(lif_layer* L, int32_t pairs) {
    if (!L || pairs < 0 || pairs > 64) return fail(LIF_INVALID_ARG, "loader pairs must be in 0..64");
    L->loader_pairs = pairs;
    return LIF_OK;
}

int lif_set_handoff_polls(lif_layer* L, int32_t polls) {
    if (!L || polls < 0) return fail(LIF_INVALID_ARG, "polls must be at least 0");
    L->polls = polls;
    return LIF_OK;
}

int lif_set_expected_rows(lif_layer* L, int32_t rows) {
    if (!L || rows < 0) return fail(LIF_INVALID_ARG, "bad row hint");
    L->expected_rows = std::min(rows, L->cfg.capacity_rows);       // (more are never in use)
    return LIF_OK;
}

static int read_state(lif_layer* L, DevState* host, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    LIF_HIP(hipStreamSynchronize(s));
    LIF_HIP(hipMemcpy(host, L->st, sizeof(DevState), hipMemcpyDeviceToHost));
    return LIF_OK;
}

int lif_get_state(lif_layer* L, lif_state* out, void* stream) {
    if (!L || !out) return fail(LIF_INVALID_ARG, "null argument");
    DevState h;
    int rc = read_state(L, &h, stream);
    if (rc) return rc;
    out->num_used = h.cur.num_used;
    out->step = h.cur.step;
    out->error = h.cur.error;
    out->last_added = h.cur.n_added;
    out->last_removed = h.cur.n_removed;
    out->last_moved = h.cur.n_moved;
    out->window_len = h.cur.window_len;
    return LIF_OK;
}

int lif_get_counters(lif_layer* L, lif_counters* out, void* stream) {
    if (!L || !out) return fail(LIF_INVALID_ARG, "null argument");
    DevState h;
    int rc = read_state(L, &h, stream);
    if (rc) return rc;
    out->steps = h.c_steps;
    out->added = h.c_added;
    out->removed = h.c_removed;
    out->rows_moved = h.c_rows_moved;
    out->h2d_bytes = h.c_h2d_bytes;
    out->ffn_calls = h.c_ffn_calls;
    out->ffn_rows = h.c_ffn_rows;
    out->ffn_active = h.c_ffn_active;
    return LIF_OK;
}

int lif_profile_read(const void* src_dev, size_t bytes, void* sink_dev, void* stream) {
    if (!sink_dev || (bytes && !src_dev)) return fail(LIF_INVALID_ARG, "null argument");
    if ((uintptr_t)src_dev % 16 || bytes % 16 || (uintptr_t)sink_dev % 4)
        return fail(LIF_INVALID_ARG, "src must be 16-byte aligned and bytes a multiple of 16");
    const size_t pieces = bytes / 16;
    const size_t wgs = (pieces + 256 * kProbePer - 1) / (256 * kProbePer);
    const int grid = (int)std::min<size_t>(std::max<size_t>(wgs, 1), 4096);
    hipLaunchKernelGGL(k_probe_read, dim3(grid), dim3(256), 0, (hipStream_t)stream, (const uint4*)src_dev, pieces,
                       (unsigned*)sink_dev);
    return check_launch();
}

size_t lif_profile_handoff_bytes(void) { return (size_t)kHandoffWgs * 16384 + 8192; }

int lif_profile_handoff(void* scratch_dev, int32_t mode, uint32_t stamp, void* stream) {
    if (!scratch_dev || (uintptr_t)scratch_dev % 256) return fail(LIF_INVALID_ARG, "scratch must be a 256-byte aligned device pointer");
    if (mode < 0 || mode > 2) return fail(LIF_INVALID_ARG, "mode must be 0, 1 or 2");
    char* p = (char*)scratch_dev;
    char* tail = p + (size_t)kHandoffWgs * 16384;      // 4 KiB of words, then the ticket counter, the give-up count, the result
    hipLaunchKernelGGL(k_probe_handoff, dim3(kHandoffWgs), dim3(256), 0, (hipStream_t)stream, (const uint4*)p,
                       (unsigned long long*)tail, (unsigned*)(tail + 4096), (unsigned long long*)(tail + 4096 + 64), mode,
                       stamp);
    return check_launch();
}

int lif_profile_begin(lif_layer* L, int32_t max_launches) {
    if (!L || max_launches < 1 || max_launches > (1 << 20)) return fail(LIF_INVALID_ARG, "bad profile request");
    for (hipEvent_t e : L->ev) (void)hipEventDestroy(e);
    L->ev.clear();
    L->ev_kernel.clear();
    L->ev.resize(2 * (size_t)max_launches);
    for (size_t i = 0; i < L->ev.size(); ++i) {
        hipError_t e = hipEventCreate(&L->ev[i]);
        if (e != hipSuccess) {
            L->ev.resize(i);
            return fail(LIF_HIP_ERROR, "hipEventCreate: %s", hipGetErrorString(e));
        }
    }
    L->prof_max = max_launches;
    L->prof_on = true;
    return LIF_OK;
}

int lif_profile_collect(lif_layer* L, double* ms, int64_t* launches, void* stream) {
    if (!L || !ms || !launches) return fail(LIF_INVALID_ARG, "null argument");
    L->prof_on = false;
    LIF_HIP(hipStreamSynchronize((hipStream_t)stream));
    for (int k = 0; k < LIF_K_COUNT; ++k) {
        ms[k] = 0.0;
        launches[k] = 0;
    }
    for (size_t i = 0; i < L->ev_kernel.size(); ++i) {
        float t = 0.f;
        LIF_HIP(hipEventElapsedTime(&t, L->ev[2 * i], L->ev[2 * i + 1]));
        ms[L->ev_kernel[i]] += t;
        launches[L->ev_kernel[i]] += 1;
    }
    for (hipEvent_t e : L->ev) (void)hipEventDestroy(e);
    L->ev.clear();
    L->ev_kernel.clear();
    return LIF_OK;
}

}  // extern "C"
