"""The single-launch FFN at the most rows it is taken for: which hints take it (looked at without a GPU), and its bits against two
launches, as tests/test_ffn_one.py does for fewer rows."""
import pytest

from tests import test_ffn_one as one
from tests.test_launches import _run

CASES = {
    # as there; the hint and an eighth more, times 64 column slices, at most 65536; rows read in full, or gated, half as many
    "widest-rows": ("f16", False, False, False, 2048, 4096, 0.12, 4096, (910,)),
    "widest-rows-gated": ("f32", True, False, False, 1024, 3000, 0.08, 3000, (455,)),
    "widest-rows-full": ("f16", False, False, True, 2048, 3000, 0.08, 3000, (455,)),
    "narrow-rows": ("f32", False, False, False, 512, 8192, 0.1, 8192, (1820,)),
}


def test_line_between_one_launch_and_two(tmp_path_factory):
    got = _run(tmp_path_factory, "ffn_one", {n: c[:-1] + ([c[-1][0], c[-1][0] + 2],) for n, c in CASES.items()})
    for n, c in CASES.items():
        for call in ("lif_sparse_ffn", "lif_sparse_ffn_static"):
            assert len(got["%s %d %s" % (n, c[-1][0], call)]) == 1, n
            assert len(got["%s %d %s" % (n, c[-1][0] + 2, call)]) == 2, n


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_single_launch_of_many_rows_equals_two_launches(name, monkeypatch):
    monkeypatch.setitem(one.CASES, name, CASES[name])
    one.test_single_launch_ffn_equals_two_launches(name)
