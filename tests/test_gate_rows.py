"""The gate predictor's decisions and activations where its row loop can go wrong: widths just behind those that take more pieces per
lane, and the widest; the fewest neurons, and more than the workgroups that a chip holds at once decide; rows of subnormal fp16 values,
whose products are exact all the same; one token and several, lif_predict and lif_step, waiting for the mask words and (polls = 0)
computing them again.  One element decides the sign of every row, in the last piece of 64 vectors for every other row, else in each
piece in turn."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

WIDTHS = [("f16", d) for d in (8, 512, 520, 1032, 2056, 2568, 3080, 3592, 4104, 4616, 6152, 8192)] + \
         [("f32", d) for d in (4, 260, 516, 1028, 1284, 1796, 2052, 2308, 3076, 4096)]
# 514 and 769 workgroups of the predictor, of which two and three fit a compute unit
MANY = [("f16", 4616, 16424), ("f32", 1028, 24584)]


def _layer(dtype, d, F, batch):
    """x, gate, b and the bundles' up and down rows, on the GPU, and the logits in fp64"""
    dt, e = (torch.float16, 8) if dtype == "f16" else (torch.float32, 4)
    rng = np.random.default_rng(d + F)
    pieces = -(-d // (64 * e))
    x = ((0.5 + rng.random((batch, d))) * rng.choice([-1.0, 1.0], (batch, d))).astype(np.float32)
    x = torch.from_numpy(x).to(dt).cuda()
    g = torch.Generator(device="cuda")
    g.manual_seed(d + F)
    gate, up, down = (torch.randn((F, d), generator=g, device="cuda") / d ** 0.5 for _ in range(3))
    gate = gate.double() * 0.125                                    # (the two elements of a row outweigh the rest of it)
    b = np.where(np.arange(F) % 4 == 1, 0.0, rng.standard_normal(F) * 0.1).astype(np.float32)
    i = np.arange(F)
    of = np.where(i % 2 == 0, pieces - 1, i // 2 % pieces)          # the piece whose element decides
    lo, hi = of * 64 * e, np.minimum((of + 1) * 64 * e, d)
    at = np.where(i % 4 == 0, d - 1, lo + rng.integers(0, 1 << 30, F) % (hi - lo))
    other = (at + 1 + rng.integers(0, 1 << 30, F) % (d - 1)) % d
    token, rows, sign = i % batch, torch.arange(F, device="cuda"), np.where(rng.random(F) < 0.5, -1.0, 1.0)
    at, other, token, sign = (torch.from_numpy(a).cuda() for a in (at, other, token, sign))
    bg = torch.from_numpy(b).cuda()
    xt = x.double()[token]
    gate[rows, at] = gate[rows, other] = 0
    for col, want in ((other, sign), (at, -sign)):                  # the sum is `sign` without the one element, `-sign` with it
        gate[rows, col] = (want - (gate * xt).sum(1) - bg.double()) / xt[rows, col]
    small = rows % 4 == 1                                           # fp16: subnormal
    gate[small] *= 2.0 ** -14
    up[small] *= 2.0 ** 13
    gate, up, down = gate.to(dt), up.to(dt), down.to(dt)
    z = x.double() @ gate.double().T + bg.double()
    # the largest error of a sum of d products in fp64, in any order
    bound = d * 2.0 ** -52 * (x.double().abs() @ gate.double().abs().T + bg.double().abs())
    assert bool((z.abs() > bound).all())
    for p in range(pieces):                                         # a piece left out changes the decisions that lie in it
        cols = slice(p * 64 * e, min((p + 1) * 64 * e, d))
        left = z - x[:, cols].double() @ gate[:, cols].double().T
        mine = torch.from_numpy(of == p).cuda()
        if pieces > 1:
            changed = (left > 0)[token, rows] != (z > 0)[token, rows]
            # (where the other element lies in the same piece, what is left need not have its sign)
            assert bool(changed[mine & ((other < cols.start) | (other >= cols.stop))].all())
    return x, gate, bg, up, down, z


@pytest.mark.parametrize("dtype,d,F", [(t, d, F) for t, d in WIDTHS for F in (8, 104)] + MANY)
def test_gate_decisions(dtype, d, F):
    import paper_2312_11514_amd as lif
    from tests.harness import MAX_ABS_TOL, REL_L2_TOL, max_abs_excess, rel_l2, require_gpu
    require_gpu()
    batch = 2
    x, gate, b, up, down, z = _layer(dtype, d, F, batch)
    want = np.packbits(z.cpu().numpy() > 0, axis=1, bitorder="little")
    # every neuron that fires for a token of the step is in the cache, and the others add nothing
    yref = ((z.clamp(min=0) * (x.double() @ up.double().T)) @ down.double()).cpu().numpy()
    host = torch.empty((F, 2 * d), dtype=gate.dtype, pin_memory=True)
    host.copy_(torch.cat([up, down], dim=1))
    lay = lif.Layer(d_model=d, d_ffn=F, rank=8, window_k=2, capacity_rows=F, max_batch=batch, dtype=dtype, predictor=lif.PRED_GATE,
                    A=gate, B=None, c=None, b=b, host_bundles=host)
    y = torch.empty((batch, d), dtype=gate.dtype, device="cuda")

    def check(what, t, n, call, outputs=True):
        print(f"{dtype} d {d} F {F}, {what}, token {t} of {n}", flush=True)
        lay.reset()
        lay.masks.zero_()
        y.fill_(float("nan"))
        call(x[t:t + n], n)
        assert (lay.masks[:n].cpu().numpy() == want[t:t + n]).all(), (what, t)
        assert (lay.step_mask.cpu().numpy() == np.bitwise_or.reduce(want[t:t + n], axis=0)).all(), (what, t)
        if outputs:
            assert sorted(lay.pointers[:int(lay.n_added.item())].tolist()) == (z[t:t + n] > 0).any(0).nonzero()[:, 0].tolist(), (what, t)
            got = y[:n].double().cpu().numpy()
            assert rel_l2(got, yref[t:t + n]) <= REL_L2_TOL and max_abs_excess(got, yref[t:t + n])[0] <= MAX_ABS_TOL, (what, t)

    for polls in (None, 0):
        if polls is not None:
            lay.set_handoff_polls(polls)
        for t in range(batch):
            check(f"predict, polls {polls}", t, 1, lambda v, n: lay.predict(v, n), outputs=False)
            check(f"calls, polls {polls}", t, 1, lambda v, n: lay.step_calls(v, y, n))
            check(f"step, polls {polls}", t, 1, lambda v, n: lay.step(v, y, n))
    check("predict", 0, batch, lambda v, n: lay.predict(v, n), outputs=False)
    check("calls", 0, batch, lambda v, n: lay.step_calls(v, y, n))
    check("step", 0, batch, lambda v, n: lay.step(v, y, n))
