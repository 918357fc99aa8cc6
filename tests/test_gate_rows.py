"""The gate predictor's decisions where its row loop can go wrong: widths just behind those that take more pieces per lane, and the
widest; the fewest neurons; rows of subnormal fp16 values, whose products are exact all the same; one token and several, lif_predict
and lif_step, waiting for the mask words and (polls = 0) computing them again."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

WIDTHS = [("f16", d) for d in (8, 512, 520, 1032, 2056, 2568, 3080, 3592, 4104, 4616, 6152, 8192)] + \
         [("f32", d) for d in (4, 260, 516, 1028, 1284, 1796, 2052, 2308, 3076, 4096)]


@pytest.mark.parametrize("dtype,d", WIDTHS)
@pytest.mark.parametrize("F", [8, 104])
def test_gate_decisions(dtype, d, F):
    import paper_2312_11514_amd as lif
    from tests.harness import require_gpu
    require_gpu()
    dt = torch.float16 if dtype == "f16" else torch.float32
    rng = np.random.default_rng(d + F)
    batch = 2 if d * dt.itemsize <= 16384 // 2 else 1
    gate = rng.standard_normal((F, d)) / np.sqrt(d)
    gate[1::4] *= 2.0 ** -14                        # fp16: subnormal
    gate, x = torch.from_numpy(gate).to(dt), torch.from_numpy(rng.standard_normal((batch, d))).to(dt)
    b = torch.from_numpy(np.where(np.arange(F) % 4 == 1, 0.0, rng.standard_normal(F) * 0.1)).to(torch.float32)
    z = x.double().numpy() @ gate.double().numpy().T + b.double().numpy()
    # the largest error of a sum of d products in fp64, in any order
    bound = d * 2.0 ** -52 * (np.abs(x.double().numpy()) @ np.abs(gate.double().numpy()).T + np.abs(b.double().numpy()))
    assert (np.abs(z) > bound).all()
    want = np.packbits(z > 0, axis=1, bitorder="little")
    lay = lif.Layer(d_model=d, d_ffn=F, rank=8, window_k=2, capacity_rows=F, max_batch=batch, dtype=dtype, predictor=lif.PRED_GATE,
                    A=gate.cuda(), B=None, c=None, b=b.cuda(), host_bundles=torch.zeros((F, 2 * d), dtype=dt).pin_memory())
    xg, y = x.cuda(), torch.zeros((batch, d), dtype=dt, device="cuda")
    for polls in (None, 0):
        if polls is not None:
            lay.set_handoff_polls(polls)
        for t in range(batch):
            for call in (lambda: lay.predict(xg[t:t + 1], 1), lambda: lay.step(xg[t:t + 1], y, 1)):
                print(f"{dtype} d {d} F {F}, token {t}, polls {polls}", flush=True)
                lay.reset()
                lay.masks.zero_()
                call()
                assert (lay.masks[0].cpu().numpy() == want[t]).all(), (t, polls)
                assert (lay.step_mask.cpu().numpy() == want[t]).all(), (t, polls)
    if batch > 1:
        lay.predict(xg, batch)
        assert (lay.masks.cpu().numpy() == want).all()
        assert (lay.step_mask.cpu().numpy() == np.bitwise_or.reduce(want, axis=0)).all()
    lay.reset()                                     # and the caches hold what was decided
    lay.step(xg[:1], y, 1)
    assert sorted(lay.pointers[:int(lay.n_added.item())].tolist()) == np.flatnonzero(z[0] > 0).tolist()
