"""Bundles that the loaders of a one-token step ask for ahead of the list of all added neurons (many were added the step before): the
step against the four calls, bit for bit, with few loaders and with more than 64, whole bundles and bundles in two parts, several mask
words per thread, lists of more than one piece on either side, the dynamic window, passes of tokens in between (whose rejected
tokens leave neurons in the cache that are in no mask of the window), and polls = 0, where no loader knows its own tile in time."""
import numpy as np
import pytest
import torch

import workloads as wl
from tests.test_step1 import _make, _snapshot

pytestmark = pytest.mark.gpu

CASES = {
    # name: (dtype, glu, gate, d, F, rank, k, p, capacity, shrink, pairs), "whole": on the other side of the rule (rows of up to 2 KiB have none)
    "whole": ("f16", False, False, 1024, 1960, 32, 3, 0.15, 1960, False, 1),
    "whole-most-loaders": ("f16", True, False, 768, 6000, 24, 2, 0.1, 6000, False, 64),
    "parts": ("f16", False, False, 2064, 3000, 40, 3, 0.1, 3000, False, 5),
    "parts-f32-gated": ("f32", True, False, 772, 1600, 20, 2, 0.2, 1600, False, 2),
    "two-words-a-thread": ("f16", False, False, 1032, 17000, 16, 2, 0.02, 4000, False, 40),
    "four-words-a-thread": ("f16", False, False, 1032, 50000, 16, 2, 0.01, 5000, False, 64),
    "many-ranks": ("f16", False, False, 1096, 2000, 320, 3, 0.1, 2000, False, 3),
    "pieces": ("f16", False, False, 1040, 12000, 16, 1, 0.35, 12000, False, 3),
    "dynamic-window": ("f16", False, False, 1040, 4160, 16, 9, 0.1, 900, True, 4),
}


@pytest.mark.parametrize("polls", [4096, 0])
@pytest.mark.parametrize("name", CASES)
def test_early_bundles_equal_four_calls(name, polls):
    from tests.harness import GpuLayer
    w, L, X, pairs = _make(name, CASES[name])
    fused, calls = GpuLayer(w, L, shrink=w.shrink, max_batch=3), GpuLayer(w, L, shrink=w.shrink, max_batch=3)
    parts = 1 if w.d_model * w.elem_bytes <= 2048 else 2
    for g in (fused, calls):
        g.layer.masks.zero_()                        # (rows of tokens that a call does not have)
    early = 0
    t = 0
    for at, tokens in enumerate([1, 1, 1, 3, 1, 1, 3, 1, 1]):
        if w.d_ffn % 64 and tokens > 1:              # (passes of tokens need whole words)
            continue
        print(f"{name}, polls {polls}, call {at}, {tokens} tokens", flush=True)
        x = X[t:t + tokens]
        xf, xc = fused.upload_x(x if tokens > 1 else x[0]), calls.upload_x(x if tokens > 1 else x[0])
        t += tokens
        fused.layer.set_loader_pairs(pairs)
        fused.layer.set_handoff_polls(polls)
        if tokens == 1:
            early += fused.layer.state()["last_added"] * parts >= 2 * pairs
            fused.layer.step(xf, fused.y, 1)
            calls.layer.step_calls(xc, calls.y, 1)
        else:
            for g, v in ((fused, xf), (calls, xc)):
                g.layer.step_tokens(v, g.y, tokens, 1)
        fused_y, calls_y = fused.y[:tokens], calls.y[:tokens]
        assert torch.equal(fused_y, calls_y), (name, at)
        a, b = _snapshot(fused), _snapshot(calls)
        assert a[0]["error"] == 0 and a[0] == b[0], (name, at, a[0], b[0])
        for i, (u, v) in enumerate(zip(a[2:], b[2:])):
            assert u == v, (name, at, i)
    assert early >= 2


@pytest.mark.parametrize("name", CASES)
def test_cases_have_early_bundles_where_the_form_has_them(name):
    """By the rule that tests/test_step_rules.py looks at: rows of more than 2 KiB, and a last step that added as many neurons as there are pairs
    of loaders.  (Results cannot tell which request a bundle came with.)"""
    from tests.harness import GpuLayer
    w, L, X, pairs = _make(name, CASES[name])
    g = GpuLayer(w, L, shrink=w.shrink, max_batch=3)
    g.layer.set_loader_pairs(pairs)
    early, t = 0, 0
    for tokens in [1, 1, 1, 3, 1, 1, 3, 1, 1]:               # (the calls of the test above)
        if w.d_ffn % 64 and tokens > 1:
            continue
        x, t = X[t:t + tokens], t + tokens
        if tokens == 1:
            early += w.d_model * w.elem_bytes > 2048 and g.layer.state()["last_added"] >= pairs
            g.layer.step(g.upload_x(x[0]), g.y, 1)
        else:
            g.layer.step_tokens(g.upload_x(x), g.y, tokens, 1)
    print(f"{name}: {early} steps with early bundles", flush=True)
    assert g.layer.state()["error"] == 0 and (early == 0 if name.startswith("whole") else early >= 2)
