"""Rules of the single-launch step that decide how fast it is and nothing else, as the header has them: compiled for the host."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2312_11514_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("no hipcc")
    at = tmp_path_factory.mktemp("rules")
    (at / "rules.hip").write_text("""#include "lif_step1.h"
#include <cstdio>
int main() {
    int a, n, v;
    while (scanf("%d %d %d", &a, &n, &v) == 3) printf("%d\\n", (int)lif::load_hides_activations(a, n, v));
}
""")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-std=c++17", "-I", CSRC, "-o", str(at / "rules"), str(at / "rules.hip")], check=True,
                   capture_output=True)

    def run(*cases):
        text = "\n".join("%d %d %d" % c for c in cases)
        return [int(l) for l in subprocess.run([str(at / "rules")], input=text, capture_output=True, text=True, check=True).stdout.split()]
    return run


def test_activations_wait_for_the_predictor_only_behind_a_load(rule):
    """(rows added by the last step, rows in use, vectors of a bundle)"""
    assert rule((0, 3414, 2), (0, 3217, 3), (0, 1, 2), (13, 3504, 2), (8, 3343, 3), (1, 65536, 2)) == [0] * 6      # begin at once
    assert rule((0, 0, 2), (143, 975, 2), (489, 3246, 2), (210, 1961, 3), (40, 3812, 2), (19, 3524, 3), (65536, 65536, 3)) == [1] * 7
