"""lif_sparse_ffn of one token in a single launch (few column slices, few rows likely in use) against the two launches that a larger
row-count hint selects, bit for bit: more rows in use than the hint, several row chunks, an empty cache, widths at the ends of what a
lane holds, a word for the last slot - waiting for the activations of other workgroups and (polls = 0) computing them - eagerly
and in a graph, whose replays go on with the launch numbers of eager calls and start again with a reset."""
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

CASES = {
    # name: (dtype, glu, gate, full, d, F, p, capacity, hints of the single launch)
    "narrow": ("f16", False, False, False, 256, 1024, 0.1, 16384, (1, 600, 1820)),
    "every-slot": ("f16", False, False, True, 8, 16384, 0.7, 16384, (64, 1820)),
    "more-chunks": ("f32", False, False, False, 12, 16384, 0.7, 16384, (64, 1820)),
    "widest": ("f16", False, False, False, 2048, 2048, 0.05, 2048, (1, 227)),
    "widest-f32": ("f32", True, False, True, 1024, 2048, 0.05, 2048, (1, 227)),
    "two-vectors": ("f16", True, False, False, 520, 3000, 0.06, 3000, (300, 606)),
    "three-vectors": ("f32", False, False, False, 516, 2000, 0.05, 2000, (1, 364)),
    "gate": ("f16", False, True, False, 1032, 4096, 0.08, 4096, (1, 364)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_single_launch_ffn_equals_two_launches(name):
    from tests.harness import GpuLayer
    dtype, glu, gate, full, d, F, p, cap, hints = CASES[name]
    w = wl.scaled(wl.WORKLOADS["C1"], name="one-" + name, d_model=d, d_ffn=F, rank=8, window_k=2, p_active=p, dtype=dtype, glu=glu or gate,
                  gate_resident=gate, capacity_rows=cap, tokens=4)
    L, X = wl.make_layer(w), wl.make_inputs(w)
    ref = GpuLayer(w, L, ffn_mode=int(full))
    xd = ref.upload_x(X)
    want, y = torch.zeros_like(ref.y), torch.zeros_like(ref.y)
    for hint in hints:
        for polls in (None, 0, 3):
            g = GpuLayer(w, L, ffn_mode=int(full), share=ref)
            if polls is not None:
                g.layer.set_handoff_polls(polls)
            g.layer.set_expected_rows(hint)
            ref.layer.set_expected_rows(0)          # (the capacity: two launches)
            for lay in (ref.layer, g.layer):
                lay.reset()
            graph = torch.cuda.CUDAGraph()
            for t in range(len(X)):
                print(f"{name}: hint {hint} polls {polls} token {t}", flush=True)
                for lay in (ref.layer, g.layer):    # (a gate predictor's FFN reads this token's gate activations)
                    lay.predict(xd[t])
                    lay.update_window()
                    lay.load_bundles()
                for again in range(2):
                    ref.layer.sparse_ffn(xd[t], want)
                    g.layer.sparse_ffn(xd[t], y)
                    assert torch.equal(y, want)
                y.fill_(7)
                g.layer.sparse_ffn_static(xd[t], y)
                assert torch.equal(y, want)
                if t == 0:
                    torch.cuda.synchronize()
                    with torch.cuda.graph(graph):
                        g.layer.sparse_ffn(xd[0], y)
                y.fill_(7)
                ref.layer.sparse_ffn(xd[0], want)
                graph.replay()
                assert torch.equal(y, want)
                assert g.layer.state()["error"] == 0
            n = g.layer.state()["num_used"]
            g.layer.reset()                         # an empty cache, and launch numbers from the start
            graph.replay()
            assert not y.any()
            g.layer.sparse_ffn(xd[0], y)
            assert not y.any() and g.layer.state()["error"] == 0
    if name in ("every-slot", "more-chunks"):
        assert n > 8192
