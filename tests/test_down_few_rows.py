"""One-token down projection launched with 16 waves where few rows are in use: eight of the waves take them, and the others hand over what they
asked for ahead of the row count.  Bit for bit what eight waves give (a hint of one row), in a fused step, where rows just loaded have
their activations elsewhere, and in an FFN call; at the edges of a group (64 rows), of a round of the eight waves (512) and of what
they take in one go (2048); the low-rank predictor and the gate, whose rows have their owners handed over too."""
import numpy as np
import pytest
import torch

import paper_2312_11514_amd as lif
from tests.test_step1 import _make

pytestmark = pytest.mark.gpu

ROWS = (1, 64, 511, 513, 1024, 1025, 1600, 2047, 2048, 2049, 2500)


@pytest.mark.parametrize("dtype,glu,gate,full", [("f16", False, False, False), ("f32", True, False, True), ("f16", False, True, False),
                                                 ("f32", False, True, False)])
def test_sixteen_waves_with_few_rows(dtype, glu, gate, full):
    from tests.harness import GpuLayer
    F = 2600
    for n in ROWS:
        w, L, X, _ = _make("few-rows", (dtype, glu, gate, 264, F, 8, 2, 0.3, F, False, 0))
        # `n` neurons that are on for every token; beside more than 300 of them, 200 that come and go
        held = np.random.default_rng(n).permutation(F)[:n]
        offset = L.b if gate else L.c
        offset[:] = -60.0
        offset[held] = 60.0
        come_and_go = held[:200] if 300 < n < 1900 else held[:0]
        offset[come_and_go] = 0.0
        got = {}
        for hint in (1, 1929, 2400, 0):
            print(f"{dtype} gate {gate}, {n} rows, hint {hint}", flush=True)
            g = GpuLayer(w, L, ffn_mode=lif.FFN_FULL_BUNDLE if full else lif.FFN_SKIP_DEAD)
            g.layer.set_expected_rows(hint)
            ys = []
            for x in X[:3]:
                xd = g.upload_x(x)
                for call in (g.layer.step, g.layer.sparse_ffn):
                    g.y.fill_(float("nan"))
                    call(xd, g.y, 1)
                    ys.append(g.y.clone())
                ys.append(g.layer.state()["num_used"])
            assert g.layer.state()["error"] == 0
            got[hint] = ys
        assert all(n - len(come_and_go) <= rows <= n for rows in got[1][2::3])
        for hint, ys in got.items():
            for i, (a, b) in enumerate(zip(ys, got[1])):
                assert (a == b) if isinstance(a, int) else (torch.equal(a, b) and bool(torch.isfinite(a).all())), (n, hint, i)
