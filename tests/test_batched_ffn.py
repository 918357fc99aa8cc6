"""The activation stage of a batch (fp16, matrix cores) with the waves per tile that a row-count hint of more than 512 tiles selects,
against those of a call without a hint, bit for bit, and both against the oracle's FFN over the cached rows: rows whose parts are no
whole stages, a last tile with few rows, more rows in use than the hint and fewer; gated rows on both sides of their second line."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,glu,gate,batch", [(96, False, False, 8), (1056, True, False, 2), (544, False, True, 5), (2080, True, False, 3)])
def test_many_tiles_equal_no_hint(d, glu, gate, batch):
    from oracle import lif_oracle as O
    from tests.harness import MAX_ABS_TOL, REL_L2_TOL, GpuLayer, max_abs_excess, rel_l2
    w = wl.scaled(wl.WORKLOADS["C1"], name="many-tiles", d_model=d, d_ffn=16384, rank=8, window_k=2, p_active=0.5, dtype="f16",
                  glu=glu or gate, gate_resident=gate, capacity_rows=16384, batch=batch, tokens=2)
    L, X = wl.make_layer(w), wl.make_batch_inputs(w)
    g = GpuLayer(w, L)
    for t in range(len(X)):
        x = g.upload_x(X[t])
        g.layer.step(x, g.y, batch)
        n, got = g.layer.state()["num_used"], []
        assert n > 8192 and g.layer.state()["error"] == 0
        for hint in (0, 8193, max(8193, n - 5), 16384):
            print(f"d {d}, {batch} tokens, {n} rows, hint {hint}", flush=True)
            g.layer.set_expected_rows(hint)
            g.y.fill_(float("nan"))
            g.layer.sparse_ffn(x, g.y, batch)
            got.append(g.y[:batch].clone())
        g.layer.set_expected_rows(0)
        cache = O.NeuronCache(n, g.layer.matrix.shape[1], np.float16)
        cache.matrix[:], cache.pointers[:], cache.bias[:] = (a[:n].cpu().numpy() for a in (g.layer.matrix, g.layer.pointers, g.layer.bias))
        cache.num_used = n
        x = np.asarray(X[t])
        ref = O.sparse_ffn_resident_gate(cache, O.gate_predict_mask(x, L.w_gate, L.b, L.theta)[2], x, d) if gate else \
            O.sparse_ffn(cache, x, d, glu)
        y = got[0].double().cpu().numpy()
        assert rel_l2(y, ref) <= REL_L2_TOL and max_abs_excess(y, ref)[0] <= MAX_ABS_TOL
        assert all(torch.equal(v, got[0]) for v in got[1:])
