"""The order in which a logit of the low-rank predictor is summed: one for every kernel that decides mask bits (lif_predict of one and
of several tokens, the single-launch step, a workgroup of it that helps itself), at every rank.  Logits whose large terms cancel and whose
small ones are as large as the rounding of the large ones, so that the sum in fp64 has the sign that its order gives it; against that
order, followed in numpy."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [("f16", 8, 1), ("f16", 40, 2), ("f32", 100, 3), ("f16", 256, 1), ("f16", 256, 8), ("f32", 260, 1), ("f16", 264, 2),
         ("f16", 320, 1), ("f16", 320, 4), ("f32", 512, 3), ("f16", 512, 8), ("f32", 516, 5), ("f16", 768, 1), ("f16", 1152, 8),
         ("f16", 2048, 1), ("f32", 2048, 2), ("f16", 2048, 7)]


def _cancelling(rng, rank, F, batch, dt):
    """t [batch, rank] and B [rank, F], exact in dt: for neuron i and token i mod batch large terms in pairs of opposite sign"""
    big = rng.random((batch, rank)) < 0.5
    sign = rng.choice([-1.0, 1.0], (batch, rank))
    t = np.where(big, 2.0 ** 15, 2.0 ** -10 * (1 + rng.integers(0, 512, (batch, rank)) / 512)) * sign
    B = (rng.standard_normal((rank, F)) * 2.0 ** -12).astype(dt).astype(np.float64)
    for i in range(F):
        of = i % batch
        at = rng.permutation(np.flatnonzero(big[of]))
        B[at, i] = 0.0
        at = at[:len(at) // 2 * 2].reshape(-1, 2)[:6]
        B[at[:, 0], i] = 2.0 ** 15 * sign[of, at[:, 0]]
        B[at[:, 1], i] = -2.0 ** 15 * sign[of, at[:, 1]]
    assert (B.astype(dt) == B).all() and (t.astype(dt) == t).all()
    return t, B


def _logits(t, B):
    """32 rank groups, each over its ranks in turn (products are exact in fp64); the groups of a wave by neighbours, then the waves"""
    rank, F = B.shape
    v = np.zeros((32, F))
    for j in range(rank):
        v[j % 32] += t[j] * B[j]
    w = v.reshape(4, 2, 2, 2, F)
    w = w[:, :, :, 0] + w[:, :, :, 1]
    w = w[:, :, 0] + w[:, :, 1]
    w = w[:, 0] + w[:, 1]
    return ((w[0] + w[1]) + w[2]) + w[3]


@pytest.mark.parametrize("dtype,rank,batch", CASES)
def test_one_order_of_summation(dtype, rank, batch):
    import paper_2312_11514_amd as lif
    from tests.harness import require_gpu
    require_gpu()
    d, F = 16, 1096
    dt, nt = (torch.float16, np.float16) if dtype == "f16" else (torch.float32, np.float32)
    t, B = _cancelling(np.random.default_rng(rank * 10 + batch), rank, F, batch, nt)
    z = np.stack([_logits(t[b], B) for b in range(batch)])
    want = np.packbits(z > 0.0, axis=1, bitorder="little")
    if rank > 256:                                  # (the data tell orders apart)
        other = np.stack([sum(_logits(t[b, j:j + 256], B[j:j + 256]) for j in range(0, rank, 256)) for b in range(batch)])
        assert ((z > 0) != (other > 0)).sum() > 10
    A = np.zeros((rank, d))
    A[:, :batch] = t.T                              # token b is the unit vector b, so x A = t
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a.astype(nt))).cuda()
    lay = lif.Layer(d_model=d, d_ffn=F, rank=rank, window_k=2, capacity_rows=F, max_batch=batch, dtype=dtype, A=up(A), B=up(B), c=None,
                    b=torch.zeros(F, device="cuda"), host_bundles=torch.zeros((F, 2 * d), dtype=dt).pin_memory())
    x, y = torch.eye(batch, d, dtype=dt, device="cuda"), torch.zeros((batch, d), dtype=dt, device="cuda")
    masks, step_mask = lay.predict(x, batch)
    assert (masks.cpu().numpy() == want).all()
    assert (step_mask.cpu().numpy() == np.bitwise_or.reduce(want, axis=0)).all()
    for polls in (None, 0):
        if polls is not None:
            lay.set_handoff_polls(polls)
        lay.reset()
        lay.masks.zero_()
        print(f"{dtype} rank {rank}, {batch} tokens, polls {polls}", flush=True)
        lay.step(x, y, batch)
        assert (lay.masks.cpu().numpy() == want).all(), polls
    for b in range(batch):                          # each token by itself: the same decisions
        lay.predict(x[b:b + 1], 1)
        assert (lay.masks[0].cpu().numpy() == want[b]).all(), b


@pytest.mark.parametrize("dtype,rank", [("f32", 4), ("f16", 8), ("f16", 32), ("f16", 40), ("f32", 128), ("f16", 264), ("f32", 320)])
def test_infinite_activations(dtype, rank):
    """An x that has overflowed: every x A is infinite, of one sign with positive weights, and so is every logit - in all kernels, whatever
    lies past the last rank."""
    import paper_2312_11514_amd as lif
    from tests.harness import require_gpu
    require_gpu()
    d, F, dt = 16, 200, torch.float16 if dtype == "f16" else torch.float32
    rng = np.random.default_rng(rank)
    up = lambda *s: torch.from_numpy(rng.uniform(0.1, 1.0, s)).to(dt).cuda()
    lay = lif.Layer(d_model=d, d_ffn=F, rank=rank, window_k=2, capacity_rows=F, max_batch=3, dtype=dtype, A=up(rank, d), B=up(rank, F), c=None,
                    b=torch.zeros(F, device="cuda"), host_bundles=torch.zeros((F, 2 * d), dtype=dt).pin_memory())
    x, y = up(3, d), torch.zeros((3, d), dtype=dt, device="cuda")
    x[0, 3], x[2, 5] = float("inf"), float("-inf")
    want = [255, 255, 0]
    for batch in (1, 2, 3):
        for polls in (None, 0):
            if polls is not None:
                lay.set_handoff_polls(polls)
            for call in (lambda: lay.predict(x, batch), lambda: lay.step(x, y, batch)):
                print(f"{dtype} rank {rank}, {batch} tokens, polls {polls}", flush=True)
                lay.reset()
                lay.masks.zero_()
                call()
                for b in range(batch):
                    assert (lay.masks[b] == want[b]).all(), (batch, b, polls)
    for b in range(3):
        lay.predict(x[b:b + 1], 1)
        assert (lay.masks[0] == want[b]).all(), b
