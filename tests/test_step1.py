"""The single-launch step of one token (lif_step, batch 1) against the four separate calls, bit for bit, where its
hand-overs, lists and loops can go wrong: edges of the 64-neuron tiles, slots of more than 512 work items, more than
4096 holes, more than 256 blocks of slots, long windows, the dynamic window, overflow - each waiting for the values that
other workgroups publish, and (polls = 0) never waiting, so that every workgroup computes them itself."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

CASES = {
    # name: (dtype, glu, gate, d, F, rank, k, p, capacity, shrink, pairs)
    "one-tile": ("f32", False, False, 8, 8, 4, 2, 0.4, 8, False, 0),
    "partial-tile": ("f16", False, False, 264, 1096, 40, 3, 0.08, 700, False, 0),
    "more-columns-than-tiles": ("f16", False, False, 128, 192, 320, 4, 0.1, 192, False, 0),
    "glu": ("f16", True, False, 1544, 712, 24, 5, 0.1, 500, False, 3),
    "gate": ("f16", False, True, 1032, 1096, 8, 3, 0.1, 900, False, 0),
    "gate-f32": ("f32", False, True, 260, 136, 8, 2, 0.2, 136, False, 1),
    "long-window": ("f32", False, False, 64, 4104, 16, 11, 0.02, 3000, False, 0),
    "dynamic-window": ("f16", False, False, 64, 4160, 16, 9, 0.1, 900, True, 0),
    "dynamic-window-two-words": ("f16", False, False, 64, 17000, 64, 4, 0.1, 4500, True, 0),
    "slot-of-many-items": ("f16", False, False, 520, 6000, 32, 2, 0.35, 6000, False, 1),
    "most-rows": ("f16", False, False, 16, 65536, 16, 1, 0.85, 65536, False, 0),
    # the deletion plan where its granules and staged owners change: about 4096, 8192 and 16384 rows in use
    "plan-64-blocks": ("f16", False, False, 16, 4352, 16, 1, 0.94, 4352, False, 0),
    "plan-128-blocks": ("f16", False, False, 16, 8704, 16, 1, 0.94, 8704, False, 0),
    "plan-256-blocks": ("f16", False, False, 16, 17408, 16, 1, 0.94, 17408, False, 0),
    "many-holes": ("f16", False, False, 16, 40000, 64, 1, 0.5, 40000, False, 0),
}


def _make(name, case=None, seed=5):
    dtype, glu, gate, d, F, rank, k, p, cap, shrink, pairs = case or CASES[name]
    w = wl.scaled(wl.WORKLOADS["C1"], name=name, d_model=d, d_ffn=F, rank=rank, window_k=k, p_active=p, dtype=dtype,
                  glu=glu or gate, gate_resident=gate, capacity_rows=cap, shrink=shrink)
    rng = np.random.default_rng(seed)
    dt = w.np_dtype
    g = lambda *s: rng.standard_normal(s, dtype=np.float32)
    mats = [(g(F, d) / np.sqrt(d)).astype(dt) for _ in range(3 if w.glu else 2)]
    act = mats[0]
    z = float(wl.norm.ppf(1 - p))
    b = (-z * np.linalg.norm(act.astype(np.float64), axis=1)).astype(np.float32)
    A, B = (g(d, rank) / np.sqrt(d)).astype(dt), (g(rank, F) / np.sqrt(rank)).astype(dt)
    c = (-z * np.linalg.norm(B.astype(np.float64), axis=0)).astype(np.float32)
    w_gate, w_up, w_down = (mats if w.glu else [None] + mats)
    parts = ([w_gate] if (w.glu and not gate) else []) + [w_up, w_down]
    L = wl.LayerData(w_up, w_down, w_gate, b, A, B, c, 0.0, np.ascontiguousarray(np.concatenate(parts, axis=1)))
    return w, L, wl.make_inputs(w, tokens=16), pairs


def _snapshot(gpu):
    lay = gpu.layer
    st = lay.state()
    n, na, nr = st["num_used"], int(lay.n_added.item()), int(lay.n_removed.item())
    return (st, gpu.y.cpu().numpy().tobytes(), lay.masks.cpu().numpy().tobytes(), lay.step_mask.cpu().numpy().tobytes(),
            lay.added[:na].cpu().numpy().tobytes(), lay.removed[:nr].cpu().numpy().tobytes(),
            lay.pointers[:n].cpu().numpy().tobytes(), lay.bias[:n].cpu().numpy().tobytes(),
            lay.matrix[:n].cpu().numpy().tobytes(), lay.counters())


@pytest.mark.parametrize("name", list(CASES))
def test_single_launch_step_equals_four_calls(name):
    from tests.harness import GpuLayer
    w, L, X, pairs = _make(name)
    ref = GpuLayer(w, L)
    runs = []
    for polls, hint in ((None, 0), (0, 0), (None, 1), (None, w.capacity_rows)):     # (a hint: rows requested ahead of the count)
        g = GpuLayer(w, L, share=ref)
        if polls is not None:
            g.layer.set_handoff_polls(polls)
        if pairs:
            g.layer.set_loader_pairs(pairs)
        g.layer.set_expected_rows(hint)
        runs.append(((polls, hint), g))
    xd = ref.upload_x(X)
    for again in range(2):                          # the second time after a reset: the stamps start again
        for g in [ref] + [g for _, g in runs]:
            g.layer.reset()
        for t in range(len(X)):
            ref.layer.step_calls(xd[t], ref.y)
            want = _snapshot(ref)
            assert want[0]["error"] == 0
            for polls, g in runs:
                print(f"{name}: token {t} polls {polls}", flush=True)
                g.layer.step(xd[t], g.y)
                got = _snapshot(g)
                for i, (a, b) in enumerate(zip(got, want)):
                    assert a == b, f"{name}: token {t}, polls and hint {polls}, item {i}"
    moved = ref.layer.counters()["rows_moved"]
    assert moved > 0 or name in ("one-tile", "more-columns-than-tiles")


@pytest.mark.parametrize("shrink", [False, True])
def test_single_launch_step_overflow(shrink):
    """A step whose mask does not fit: the sticky error, nothing loaded, and mixed use with the four calls before it."""
    from tests.harness import GpuLayer
    w, L, X, _ = _make("partial-tile")
    ref = GpuLayer(w, L, capacity=150, shrink=shrink)
    g = GpuLayer(w, L, capacity=150, shrink=shrink, share=ref)
    L_all = np.full(w.d_ffn, 10.0, np.float32)
    xd = ref.upload_x(X)
    for t in range(3):
        ref.layer.step_calls(xd[t], ref.y)
        (g.layer.step if t % 2 == 0 else g.layer.step_calls)(xd[t], g.y)
        assert _snapshot(g) == _snapshot(ref)
    for lay in (ref.layer, g.layer):                # every neuron is predicted from here on
        lay.c.copy_(torch.from_numpy(L_all))
    ref.layer.step_calls(xd[3], ref.y)
    g.layer.step(xd[3], g.y)
    want, got = _snapshot(ref), _snapshot(g)
    assert got[0]["error"] != 0 and got == want
    g.layer.step(xd[4], g.y)
    ref.layer.step_calls(xd[4], ref.y)
    want, got = _snapshot(ref), _snapshot(g)
    assert got[0] == want[0] and got[4:] == want[4:]


BATCH_CASES = {
    # name: (dtype, glu, gate, d, F, rank, k, p, capacity, shrink, pairs), then the batch
    "mfma": (("f16", False, False, 1056, 1096, 40, 3, 0.06, 900, False, 0), 3),
    "mfma-glu": (("f16", True, False, 544, 2048, 24, 5, 0.04, 1700, False, 3), 8),
    "mfma-gate": (("f16", False, True, 96, 1088, 8, 3, 0.05, 900, False, 0), 5),
    "mfma-dynamic": (("f16", False, False, 64, 4160, 16, 9, 0.03, 1100, True, 0), 4),
    "mfma-many-rows": (("f16", True, False, 32, 20032, 64, 2, 0.1, 18000, False, 0), 6),
    "mfma-widest-glu": (("f16", True, False, 8192, 384, 16, 2, 0.1, 300, False, 2), 4),
    "mfma-most-rows": (("f16", False, False, 32, 65536, 16, 2, 0.35, 65536, False, 0), 4),
    "dots-many-rows": (("f16", False, False, 24, 20032, 16, 2, 0.2, 20032, False, 0), 3),
    "dots-eight-waves": (("f32", False, False, 1288, 704, 16, 2, 0.05, 600, False, 0), 8),
    "dots-eight-waves-gate": (("f32", False, True, 2564, 192, 8, 2, 0.1, 192, False, 0), 6),
    "dots-eight-waves-glu": (("f16", True, False, 6152, 256, 16, 2, 0.1, 256, False, 0), 4),
    "dots-widest-glu": (("f32", True, False, 4096, 256, 16, 2, 0.1, 256, False, 0), 4),
    "dots": (("f16", False, False, 1032, 1088, 40, 3, 0.06, 900, False, 0), 3),
    "dots-glu": (("f16", True, False, 264, 704, 24, 2, 0.05, 600, False, 1), 8),
    "dots-gate": (("f32", False, True, 260, 192, 8, 2, 0.05, 192, False, 0), 2),
    "dots-f32-dynamic": (("f32", True, False, 516, 4160, 16, 4, 0.05, 900, True, 0), 2),
}


@pytest.mark.parametrize("name", list(BATCH_CASES))
def test_single_launch_batch_equals_calls(name):
    """Batches (lif_step) and passes of several tokens (lif_step_tokens, every number of kept tokens) the same way."""
    from tests.harness import GpuLayer
    case, batch = BATCH_CASES[name]
    w, L, _, pairs = _make(name, case)
    X = wl.make_inputs(w, tokens=12 * batch)
    ref = GpuLayer(w, L, max_batch=batch)
    runs = []
    for hint in (0, 1, w.capacity_rows):            # (a hint: rows requested ahead of the count)
        g = GpuLayer(w, L, max_batch=batch, share=ref)
        if pairs:
            g.layer.set_loader_pairs(pairs)
        g.layer.set_expected_rows(hint)
        runs.append((hint, g))
    for lay in [ref.layer] + [g.layer for _, g in runs]:        # (fewer tokens than max_batch leave the rest of these alone)
        lay.masks.zero_()
    xd = ref.upload_x(X)
    for t in range(12):
        x = xd[t * batch:(t + 1) * batch]
        tokens = batch if t % 4 else 1 + t % batch
        keep = t % (tokens + 1)
        print(f"{name}: step {t} tokens {tokens}", flush=True)
        whole = t % 3 == 0 or w.d_ffn % 64
        if whole:
            ref.layer.step_calls(x, ref.y, batch=tokens)
        else:
            ref.layer.predict(x, batch=tokens)
            ref.layer.update_window_tokens(tokens, keep)
            ref.layer.load_bundles()
            ref.layer.sparse_ffn(x, ref.y, batch=tokens)
        want = _snapshot(ref)
        assert want[0]["error"] == 0
        for hint, g in runs:
            if whole:
                g.layer.step(x, g.y, batch=tokens)
            else:
                g.layer.step_tokens(x, g.y, tokens, keep)
            for i, (a, b) in enumerate(zip(_snapshot(g), want)):
                assert a == b, f"{name}: step {t}, tokens {tokens}, keep {keep}, hint {hint}, item {i}"
    assert ref.layer.counters()["rows_moved"] > 0


@pytest.mark.parametrize("batch", [1, 3])
def test_two_layers_step_on_two_streams(batch):
    """Layers share nothing: steps of two of them in flight at once leave what each leaves by itself."""
    from tests.harness import GpuLayer
    w, L, X, _ = _make("dots", BATCH_CASES["dots"][0])
    X = wl.make_inputs(w, tokens=20 * batch)
    alone = GpuLayer(w, L, max_batch=batch)
    pair = [GpuLayer(w, L, max_batch=batch, share=alone) for _ in range(2)]
    xd = alone.upload_x(X)
    ys = [[torch.zeros_like(alone.y) for _ in range(20)] for _ in range(3)]
    streams = [torch.cuda.Stream() for _ in pair]
    torch.cuda.synchronize()
    print(f"two streams, batch {batch}", flush=True)
    for t in range(20):                             # the second layer goes through the tokens the other way round
        for i, (g, s) in enumerate(zip(pair, streams)):
            at = t if i == 0 else 19 - t
            with torch.cuda.stream(s):
                g.layer.step(xd[at * batch:(at + 1) * batch], ys[i][t], batch=batch)
    torch.cuda.synchronize()
    got = [_snapshot(g) for g in pair]
    for i in range(2):
        alone.layer.reset()
        for t in range(20):
            at = t if i == 0 else 19 - t
            alone.layer.step_calls(xd[at * batch:(at + 1) * batch], ys[2][t], batch=batch)
        want = _snapshot(alone)
        assert got[i][0] == want[0] and got[i][2:] == want[2:]
        assert all(torch.equal(a, b) for a, b in zip(ys[i], ys[2]))


@pytest.mark.parametrize("batch", [1, 3])
def test_graph_replay_across_resets(batch):
    """A captured step replayed with eager steps and resets in between: the stamps of what workgroups hand over come from
    device state, not from what was captured."""
    from tests.harness import GpuLayer
    w, L, X, _ = _make("dots", BATCH_CASES["dots"][0])
    X = wl.make_inputs(w, tokens=8 * batch)
    ref = GpuLayer(w, L, max_batch=batch)
    g = GpuLayer(w, L, max_batch=batch, share=ref)
    xd = ref.upload_x(X).view(8, batch, -1)
    stage = xd[0].clone()
    g.layer.step(stage, g.y, batch=batch)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        g.layer.step(stage, g.y, batch=batch)
    for again in range(3):
        for lay in (ref.layer, g.layer):
            lay.reset()
        for t in range(8):
            print(f"graph, batch {batch}: sequence {again} token {t}", flush=True)
            ref.layer.step_calls(xd[t], ref.y, batch=batch)
            if (t + again) % 3 == 2:
                g.layer.step(xd[t], g.y, batch=batch)
            else:
                stage.copy_(xd[t])
                graph.replay()
            assert _snapshot(g) == _snapshot(ref), f"sequence {again} token {t}"


def test_pass_of_tokens_with_a_step_mask_at_an_odd_address():
    """lif_step_tokens takes a step mask of any alignment (it then runs the separate kernels)."""
    from tests.harness import GpuLayer
    w, L, X, _ = _make("dynamic-window")
    ref = GpuLayer(w, L, max_batch=4)
    g = GpuLayer(w, L, max_batch=4, share=ref)
    room = torch.zeros(w.d_ffn // 8 + 8, dtype=torch.uint8, device=g.dev)
    g.layer.step_mask = room[3:3 + w.d_ffn // 8]
    for lay in (ref.layer, g.layer):
        lay.masks.zero_()
    xd = ref.upload_x(X)
    for t in range(5):
        x = xd[2 * t:2 * t + 4]
        ref.layer.step_tokens(x, ref.y, 4, 2)
        g.layer.step_tokens(x, g.y, 4, 2)
        assert _snapshot(g) == _snapshot(ref), f"pass {t}"
    assert int(room[:3].sum()) == 0 and int(room[3 + w.d_ffn // 8:].sum()) == 0


LOAD_CASES = {
    # name: ((dtype, glu, gate, d, F, rank, k, p, capacity, shrink, pairs), bundles in two parts)
    "32-byte-rows": (("f32", False, False, 4, 264, 4, 2, 0.2, 264, False, 0), False),
    "one-chunk": (("f16", False, False, 1288, 800, 16, 2, 0.1, 800, False, 0), False),
    "short-last-chunk": (("f32", True, False, 2052, 320, 16, 3, 0.1, 320, False, 0), False),
    "six-chunks": (("f16", True, False, 8192, 200, 16, 2, 0.1, 200, False, 0), False),
    "two-parts": (("f16", True, False, 2072, 640, 16, 2, 0.1, 640, False, 0), True),
    "many-units-a-wave": (("f16", False, False, 264, 4096, 16, 1, 0.3, 4096, False, 1), False),
}


@pytest.mark.parametrize("name", list(LOAD_CASES))
def test_load_bundles_chunks_and_lists(name):
    """lif_load_bundles where its units can go wrong: the cache rows, owners and biases against the oracle."""
    from oracle import lif_oracle as O
    from tests.harness import GpuLayer, compare_step
    case, unbundled = LOAD_CASES[name]
    w, L, X, pairs = _make(name, case)
    gpu = GpuLayer(w, L, unbundled=unbundled)
    if pairs:
        gpu.layer.set_loader_pairs(pairs)
    ora = O.OracleLayer(w.d_model, w.d_ffn, w.window_k, w.capacity_rows, w.glu, L.A, L.B, L.c, L.theta, L.b, L.bundles)
    moved = 0
    for t in range(5):
        print(f"{name}: token {t}", flush=True)
        moved += compare_step(gpu, ora, X[t], w, t)["moved"]
    assert moved > 0


@pytest.mark.parametrize("n", [1, 31, 33, 128, 511, 513, 1030])
def test_batched_down_projection_reading_every_row(n):
    """fp16 batch, every row read: rows are requested ahead of the row count, so slots not in use may hold anything."""
    import paper_2312_11514_amd as lif
    from tests.harness import REL_L2_TOL, GpuLayer, rel_l2
    w = wl.scaled(wl.WORKLOADS["C1"], name="full", d_model=136, d_ffn=1096, rank=16, capacity_rows=1030, dtype="f16", p_active=0.4)
    L = wl.make_layer(w)
    gpu = GpuLayer(w, L, ffn_mode=lif.FFN_FULL_BUNDLE, max_batch=3)
    ids = np.random.default_rng(n).permutation(w.d_ffn)[:n]
    gpu.layer.matrix.fill_(float("nan"))
    gpu.fill_cache(ids, L)
    x = wl.make_inputs(w, tokens=3)
    gpu.layer.sparse_ffn(gpu.upload_x(x), gpu.y, batch=3)
    bun = L.bundles[ids].astype(np.float64)
    d = w.d_model
    h = np.maximum(x.astype(np.float64) @ bun[:, :d].T + L.b[ids], 0.0)
    assert rel_l2(gpu.y.cpu().numpy().astype(np.float64), h @ bun[:, d:]) <= REL_L2_TOL


@pytest.mark.parametrize("d,F,rows", [(96, 33000, (2048, 2049, 3584, 3585, 4097, 8192, 8193, 16385, 33000)),
                                      (4096, 16384, (3585, 8193, 16384)), (4544, 10240, (3584, 8193, 10240))])
@pytest.mark.parametrize("full", [False, True])
def test_down_projection_of_one_token_by_row_chunks(d, F, rows, full):
    """The chunks and waves of the down projection follow from the rows in use, whatever launch the hint leads to: the same
    bytes with every hint, and the sum itself, around the row counts where the rule changes."""
    import paper_2312_11514_amd as lif
    from tests.harness import REL_L2_TOL, rel_l2, require_gpu
    require_gpu()
    g = torch.Generator(device="cuda")
    g.manual_seed(d + full)
    zeros = lambda *s, dt=torch.float16: torch.zeros(s, dtype=dt, device="cuda")
    lay = lif.Layer(d_model=d, d_ffn=F, rank=8, window_k=2, capacity_rows=F, dtype="f16",
                    ffn_mode=lif.FFN_FULL_BUNDLE if full else lif.FFN_SKIP_DEAD, A=zeros(8, d), B=zeros(8, F), c=None,
                    b=zeros(F, dt=torch.float32), host_bundles=torch.zeros((F, 2 * d), dtype=torch.float16).pin_memory())
    lay.matrix.copy_(torch.randn((F, 2 * d), generator=g, device="cuda").div_(d ** 0.5))
    lay.bias.fill_(-0.7)
    x = torch.randn((1, d), generator=g, device="cuda").half()
    h = torch.relu(lay.matrix[:, :d].double() @ x[0].double() - 0.7)
    for n in rows:
        lay.workspace[:4] = torch.tensor([n], dtype=torch.int32).view(torch.uint8).cuda()
        got = []
        for hint in (0, 1, n // 2, n, n + n // 7, F):
            print(f"one token, d {d}, full {full}: {n} rows, hint {hint}", flush=True)
            lay.set_expected_rows(hint)
            y = torch.full_like(x, 9.0)
            lay.sparse_ffn(x, y)
            got.append(y)
        assert all(torch.equal(y, got[0]) for y in got[1:]), n
        want = h[:n] @ lay.matrix[:n, d:].double()
        assert rel_l2(got[0].double().cpu().numpy(), want.cpu().numpy()) <= REL_L2_TOL, n


@pytest.mark.parametrize("dtype,d,F,rows", [("f32", 1288, 13000, (512, 513, 3073, 4097, 12300, 13000)), ("f32", 4096, 1100, (512, 513, 1100)),
                                            ("f16", 136, 1280, (256, 512, 513, 1280)), ("f16", 136, 1281, (256, 257, 513, 1281)),
                                            ("f16", 512, 8193, (512, 8193)), ("f16", 4096, 6145, (513, 6145)), ("f16", 4096, 6144, (257, 6144))])
@pytest.mark.parametrize("full", [False, True])
def test_down_projection_of_a_batch_by_row_chunks(dtype, d, F, rows, full):
    """The same for three tokens: fp32 chunks by rows and width, fp16 chunks and passes by capacity and width."""
    import paper_2312_11514_amd as lif
    from tests.harness import REL_L2_TOL, rel_l2, require_gpu
    require_gpu()
    g = torch.Generator(device="cuda")
    g.manual_seed(d + full)
    dt = torch.float32 if dtype == "f32" else torch.float16
    zeros = lambda *s, dt=dt: torch.zeros(s, dtype=dt, device="cuda")
    lay = lif.Layer(d_model=d, d_ffn=(F + 7) // 8 * 8, rank=8, window_k=2, capacity_rows=F, max_batch=3, dtype=dtype,
                    ffn_mode=lif.FFN_FULL_BUNDLE if full else lif.FFN_SKIP_DEAD, A=zeros(8, d), B=zeros(8, (F + 7) // 8 * 8), c=None,
                    b=zeros((F + 7) // 8 * 8, dt=torch.float32),
                    host_bundles=torch.zeros(((F + 7) // 8 * 8, 2 * d), dtype=dt).pin_memory())
    lay.matrix.copy_(torch.randn((F, 2 * d), generator=g, device="cuda").div_(d ** 0.5))
    lay.bias.fill_(-0.7)
    x = torch.randn((3, d), generator=g, device="cuda").to(dt)
    h = torch.relu(x.double() @ lay.matrix[:, :d].double().t().contiguous() - 0.7)
    for n in rows:
        lay.workspace[:4] = torch.tensor([n], dtype=torch.int32).view(torch.uint8).cuda()
        got = []
        for hint in (0, 1, n // 2, n, F):
            print(f"three tokens, {dtype}, d {d}, full {full}: {n} rows, hint {hint}", flush=True)
            lay.set_expected_rows(hint)
            y = torch.full_like(x, 9.0)
            lay.sparse_ffn(x, y, batch=3)
            got.append(y)
        assert all(torch.equal(y, got[0]) for y in got[1:]), n
        want = h[:, :n].contiguous() @ lay.matrix[:n, d:].double()
        assert rel_l2(got[0].cpu().numpy().astype(np.float64), want.cpu().numpy()) <= (1e-5 if dtype == "f32" else REL_L2_TOL), n


def test_columns_of_x_a_come_from_workgroups_that_run_together():
    """More predictor workgroups (266) than fit the chip with the widest gated rows: none of those that run first may wait for columns
    of those that start when they end.  At rank 512 a step then took 1484 us, each wait until it runs out; now 81.  At rank 256 the columns
    were never dealt that far, so a step of that rank is the measure."""
    import paper_2312_11514_amd as lif
    from tests.harness import require_gpu
    require_gpu()
    d, F, cap = 5120, 17000, 512
    zeros = lambda *s, dt=torch.float16: torch.zeros(s, dtype=dt, device="cuda")
    host = torch.empty((F, 3 * d), dtype=torch.float16, pin_memory=True)     # (zeros predict no neuron: nothing is loaded)
    x, y = zeros(1, d), zeros(1, d)
    us = {}
    for rank in (256, 512):
        lay = lif.Layer(d_model=d, d_ffn=F, rank=rank, window_k=2, capacity_rows=cap, glu=True, dtype="f16", A=zeros(rank, d),
                        B=zeros(rank, F), c=None, b=zeros(F, dt=torch.float32), host_bundles=host)
        lay.step(x, y)
        us[rank] = []
        for _ in range(7):
            print(f"rank {rank}", flush=True)
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            begin.record()
            for _ in range(4):
                lay.step(x, y)
            end.record()
            end.synchronize()
            us[rank].append(250.0 * begin.elapsed_time(end))
        assert lay.state()["error"] == 0 and not y.any()
    assert sorted(us[512])[3] < 5 * sorted(us[256])[3], us
