"""The activation stage of a batch (fp16, matrix cores) with the waves per tile that a row-count hint of more than 512 tiles selects,
against those of a call without a hint, bit for bit: rows whose parts are no whole stages, a last tile with few rows, more rows in
use than the hint and fewer."""
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,glu,gate,batch", [(96, False, False, 8), (1056, True, False, 2), (544, False, True, 5)])
def test_many_tiles_equal_no_hint(d, glu, gate, batch):
    from tests.harness import GpuLayer
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
            g.y.fill_(7)
            g.layer.sparse_ffn(x, g.y, batch)
            got.append(g.y[:batch].clone())
        g.layer.set_expected_rows(0)
        assert got[0].any() and all(torch.equal(y, got[0]) for y in got[1:])
