"""Row chunks of the down projection, whose sums the last workgroup of a column slice adds: the bits do not depend on how many
workgroup rows share the chunks (a row-count hint that is far too small leaves one, which adds its own), nor on the call, and are
those of the oracle's FFN over the cached rows within the tolerance of one FFN call.  2 to more than 24 chunks (asked for 8 at a
time, then 16), ragged last slices, every kernel, and more workgroups than the chip holds, where a launch of its own adds them."""
import numpy as np
import pytest
import torch

import paper_2312_11514_amd as lif
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,batch,full,d,F", [
    ("f16", 1, False, 136, 16384), ("f16", 1, True, 72, 8000), ("f32", 1, True, 68, 16384),
    ("f16", 5, False, 160, 4800), ("f16", 8, True, 264, 15000), ("f16", 3, False, 4104, 1480), ("f16", 2, False, 4104, 12304),
    ("f32", 3, False, 132, 1400), ("f32", 8, True, 68, 9000)])
def test_chunks_shared_or_not(dtype, batch, full, d, F):
    from oracle import lif_oracle as O
    from tests.harness import MAX_ABS_TOL, REL_L2_TOL, GpuLayer, max_abs_excess, rel_l2
    w = wl.scaled(wl.WORKLOADS["C1"], name="down-chunks", d_model=d, d_ffn=F, rank=8, window_k=2, p_active=0.6, dtype=dtype,
                  capacity_rows=F, batch=batch, tokens=2)
    L, X = wl.make_layer(w), (wl.make_batch_inputs(w) if batch > 1 else wl.make_inputs(w))
    g = GpuLayer(w, L, ffn_mode=lif.FFN_FULL_BUNDLE if full else lif.FFN_SKIP_DEAD)
    for t in range(len(X)):
        x = g.upload_x(X[t])
        g.layer.step(x, g.y, batch)
        n = g.layer.state()["num_used"]
        assert n > F // 2 and g.layer.state()["error"] == 0
        step, got = g.y[:batch].clone(), []
        for hint in (0, 1, n // 2, n, F, 0):
            print(f"{dtype} d {d}, {batch} tokens, {n} rows, hint {hint}", flush=True)
            g.layer.set_expected_rows(hint)
            for _ in range(3):
                g.y.fill_(float("nan"))
                g.layer.sparse_ffn(x, g.y, batch)
                got.append(g.y[:batch].clone())
        g.layer.set_expected_rows(0)
        assert all(torch.equal(v, step) for v in got)
        cache = O.NeuronCache(n, g.layer.matrix.shape[1], g.layer.matrix.cpu().numpy().dtype)
        cache.matrix[:], cache.pointers[:], cache.bias[:] = (a[:n].cpu().numpy() for a in (g.layer.matrix, g.layer.pointers, g.layer.bias))
        cache.num_used = n
        ref = np.asarray(O.sparse_ffn(cache, np.asarray(X[t]), d, False)).reshape(batch, d)
        y = step.double().cpu().numpy().reshape(batch, d)
        assert rel_l2(y, ref) <= REL_L2_TOL and max_abs_excess(y, ref)[0] <= MAX_ABS_TOL
