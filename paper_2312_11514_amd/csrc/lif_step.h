// Fused cache update + activation stage of batches (lif_step, lif_step_tokens); single tokens: lif_step1.h.
//
// The host-to-device gather of new bundles is bound by the host link and keeps only ~32
// workgroups busy for tens of microseconds (Section 3.3 item 2), while the activation stage of
// the FFN (Section 3.3 item 3) streams the rows that are already resident.  Both only need the
// token's x and the deletion plan, so one launch runs them side by side:
//   workgroups [0, load_wgs)       loaders: row moves + pinned-host appends with the layout of k_load;
//   workgroups [load_wgs, ...)     activation role over the rows kept by the deletion (slots < n').
#pragma once

#include "lif_ffn.h"
#include "lif_ffn_mfma.h"
#include "lif_window.h"

namespace lif {

// fp16: loader workgroups (layout of k_load) next to the MFMA activation
// stage over the rows that survive the deletion.  The slots the loaders write (filled holes, appended rows) get
// their activations from a second, short launch of k_ffn_up_mfma<GLU, kRowsChanged> once the load is complete.
// grid = load_wgs + ceil(capacity / 16), block = 256.
template <bool GLU>
__global__ __launch_bounds__(256) void k_load_up_mfma(_Float16* __restrict__ matrix, int32_t* __restrict__ pointers,
                                                      float* __restrict__ bias, const HostStore host,
                                                      const float* __restrict__ b, const int32_t* __restrict__ added,
                                                      const int32_t* __restrict__ move_dst, size_t row_bytes, int F,
                                                      const _Float16* __restrict__ x, float* __restrict__ h, int d,
                                                      int batch, int capacity, int load_wgs, int spec_tiles,
                                                      const float* __restrict__ gact, DevState* st) {
    if ((int)blockIdx.x < load_wgs)
        load_rows_role(reinterpret_cast<char*>(matrix), pointers, bias, host, b, added, move_dst, row_bytes, F,
                       blockIdx.x, load_wgs, st);
    else
        // (with the gate predictor a hole's pointer may change under this role: the lookup is clamped and the
        // slot's activation is recomputed by the pass over the written slots)
        // (tiles below spec_tiles - those a row-count hint covers - ask for their first rows ahead of the state)
        ffn_up_mfma_tile_staged<GLU, kRowsKept, kMfmaWaves>(matrix, bias, x, h, d, batch, capacity, row_bytes / sizeof(_Float16),
                                                blockIdx.x - load_wgs, (int)blockIdx.x - load_wgs < spec_tiles, pointers,
                                                gact, F, st);
}

}  // namespace lif
