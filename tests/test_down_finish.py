"""Who adds the chunk sums of the down projection, the last workgroup of a column slice or a launch of its own: both on either side of their
lines (looked at without a GPU), and that the cases of tests/test_down_chunks.py and the three more of this file, which are checked the
same way, have the chunks that are meant: a few, and more than 24, which are asked for 16 at a time."""
import pytest

import paper_2312_11514_amd as lif
import workloads as wl
from tests.test_launches import _run

# dtype, tokens, every row read, d, F = capacity, chunks that the rows in use make, whether a hint of all rows has the sums added by a
# launch of its own
MANY_WORKGROUPS = ("f16", 2, False, 4104, 12304, (19, 24), True)
CASES = [("f16", 1, False, 136, 16384, (2, 4), False), ("f16", 1, True, 72, 8000, (5, 6), False), ("f32", 1, True, 68, 16384, (9, 13), False),
         ("f16", 1, True, 8192, 9304, (5, 7), True), ("f16", 1, True, 136, 30000, (17, 24), True),
         ("f16", 5, False, 160, 4800, (18, 19), True), ("f16", 8, False, 136, 7000, (27, 28), True), ("f16", 8, True, 264, 15000, (29, 30), True),
         ("f16", 3, False, 4104, 1480, (5, 6), False), MANY_WORKGROUPS,
         ("f32", 3, False, 132, 1400, (10, 11), False), ("f32", 8, True, 68, 9000, (32, 32), True), ("f32", 5, False, 1020, 4200, (30, 32), True)]
# (those of tests/test_down_chunks.py)
BESIDE = [("f16", 1, False, 136, 16384), ("f16", 1, True, 72, 8000), ("f32", 1, True, 68, 16384), ("f16", 5, False, 160, 4800),
          ("f16", 8, True, 264, 15000), ("f16", 3, False, 4104, 1480), MANY_WORKGROUPS[:5], ("f32", 3, False, 132, 1400),
          ("f32", 8, True, 68, 9000)]


def test_launch_that_adds_the_chunk_sums(tmp_path_factory):
    """A launch of its own where a hint makes more than 16 chunks of one token, or many workgroups; more than 16 chunks of fp16 rows of five tokens
    and more, below 4096 columns; more than 24 chunks of fp32 rows of as many tokens, or of wide rows: on either side of each line.  A hint of one chunk:
    none.  No hint, and so a grid for the capacity: only behind more workgroups of fp16 rows than the chip holds."""
    lines = {
        # hints on either side of the line, then one of a single chunk
        "one": ("f16", 1, True, 8192, 20480, (8190 * 8 // 9, 9300 * 8 // 9, 900)), "one-skip": ("f32", 1, False, 4096, 50000, (29000, 36000, 900)),
        "one-many-sums": ("f16", 1, True, 1024, 20480, (16384, 16385, 900)), "one-many-sums-f32": ("f32", 1, True, 512, 65536, (16384, 16385, 900)),
        "many-workgroups": ("f16", 2, False, 4104, 16384, (10400, 11000, 200)),
        "many-sums": ("f16", 8, False, 1024, 8192, (4096, 4097, 200)), "many-sums-512": ("f16", 5, True, 3968, 16384, (8192, 8193, 200)),
        "4096-columns": ("f16", 8, True, 4096, 11008, (8192, 10000, 200)), "few-tokens": ("f16", 4, False, 1024, 8192, (4000, 8192, 200)),
        "f32": ("f32", 5, False, 1024, 20000, (3072, 3073, 200)), "f32-narrow": ("f32", 8, True, 256, 9000, (3072, 3073, 200)),
        "f32-few-tokens": ("f32", 4, False, 2048, 20000, (4096, 16384, 200)),
        "f32-wide": ("f32", 4, False, 4096, 20000, (9000, 16384, 200)),
    }
    last = ("4096-columns", "few-tokens", "f32-few-tokens")            # never a launch
    got = _run(tmp_path_factory, "ffn_down", lines)
    for name, case in lines.items():
        few, many, none = (got["%s %d" % (name, h)] for h in case[-1])
        assert [len(v) for v in (few, many, none)] == [1, 1 if name in last else 2, 1], (name, few, many, none)
        assert len(many) == 1 or "k_ffn_down_finish" in many[1][0]
    cases = {str(i): (dtype, batch, full, d, F, (0, F)) for i, (dtype, batch, full, d, F, _, _) in enumerate(CASES)}
    got = _run(tmp_path_factory, "ffn_down", cases)
    for i, case in enumerate(CASES):
        assert (len(got["%d %d" % (i, case[4])]) == 2) == case[-1], case
        assert (len(got["%d 0" % i]) == 2) == (case == MANY_WORKGROUPS), case


def _chunks(dtype, batch, full, d, F, n):
    """Chunks that n rows make, as the kernels have it"""
    if batch == 1:
        if n <= (3584 if full else 8192):
            return 1
        return 2 if not full and 96 * 32 < d <= 128 * 32 and n <= 16384 else -(-n // (1024 if full else 4096))
    if dtype == "f16":
        few = -(-F // 256)
        rows = 256 if F > 1280 and few <= 32 and few * -(-d // 128) <= 768 else 512
        return -(-n // (rows * -(-F // (32 * rows))))
    return 1 if n <= 512 else min(32, max(-(-n // 512), min(-(-n // 128), 512 // -(-d // 64))))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,batch,full,d,F,chunks,launch", CASES)
def test_chunks_of_the_rows_in_use(dtype, batch, full, d, F, chunks, launch):
    from tests.harness import GpuLayer
    w = wl.scaled(wl.WORKLOADS["C1"], name="down-chunks", d_model=d, d_ffn=F, rank=8, window_k=2, p_active=0.6, dtype=dtype,
                  capacity_rows=F, batch=batch, tokens=2)
    X = wl.make_batch_inputs(w) if batch > 1 else wl.make_inputs(w)
    g = GpuLayer(w, wl.make_layer(w), ffn_mode=lif.FFN_FULL_BUNDLE if full else lif.FFN_SKIP_DEAD)
    for x in X:
        print(f"{dtype} d {d}, {batch} tokens", flush=True)
        g.layer.step(g.upload_x(x), g.y, batch)
        assert chunks[0] <= _chunks(dtype, batch, full, d, F, g.layer.state()["num_used"]) <= chunks[1]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,batch,full,d,F", [c[:5] for c in CASES if c[:5] not in BESIDE])
def test_more_chunks_shared_or_not(dtype, batch, full, d, F):
    from tests.test_down_chunks import test_chunks_shared_or_not as check
    check(dtype, batch, full, d, F)
