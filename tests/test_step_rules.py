"""Rules and bounds of the single launches that run on the device, as the headers have them: compiled for the host."""
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
#include "lif_ffn_one.h"
#include <cstdio>
#include <cstring>
int main() {
    char what[16];
    int a, b, c;
    while (scanf("%15s %d %d %d", what, &a, &b, &c) == 4) {
        if (!strcmp(what, "hides")) printf("%d\\n", (int)lif::load_hides_activations(a, b, c));
        if (!strcmp(what, "form")) printf("%d\\n", (int)lif::early_form(a, b != 0));
        if (!strcmp(what, "tiles")) printf("%d\\n", lif::early_tiles(a, b, c));
        if (!strcmp(what, "unit")) printf("%d\\n", lif::first_unit(a, 2, b, (unsigned long long)c << (b > 31 ? b - 31 : 0)));
        if (!strcmp(what, "waves")) printf("%d\\n", lif::up_mfma_waves(a, b, c != 0));
        if (!strcmp(what, "await")) {           // b slots, the first c of them there, by thread a of 512: looks, and the answer
            int looks = 0;
            const bool all = lif::await_slots(a, b, 512, 1000, [&](int s) { ++looks; return s < c; });
            printf("%d\\n", all ? looks : -looks);
        }
    }
}
""")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-std=c++17", "-I", CSRC, "-o", str(at / "rules"), str(at / "rules.hip")], check=True,
                   capture_output=True)

    def run(what, *cases):
        text = "\n".join("%s %d %d %d" % ((what,) + c) for c in cases)
        return [int(l) for l in subprocess.run([str(at / "rules")], input=text, capture_output=True, text=True, check=True).stdout.split()]
    return run


def test_activations_wait_for_the_predictor_only_behind_a_load(rule):
    """(rows added by the last step, rows in use, vectors of a bundle)"""
    assert rule("hides", (0, 3414, 2), (0, 3217, 3), (0, 1, 2), (13, 3504, 2), (8, 3343, 3), (1, 65536, 2)) == [0] * 6      # begin at once
    assert rule("hides", (0, 0, 2), (143, 975, 2), (489, 3246, 2), (210, 1961, 3), (40, 3812, 2), (19, 3524, 3), (65536, 65536, 3)) == [1] * 7


def test_a_lost_wait_is_bounded_over_all_slots_of_a_thread(rule):
    """The last workgroup of a single-launch FFN looks for the words of all slots, up to 32 of them a thread, before it gives the launch up:
    the bound is one for the thread, not one a slot."""
    assert rule("await", (0, 16384, 16384), (5, 0, 0), (511, 513, 0)) == [32, 0, -1000]      # all there; none to look for; the first is missing
    assert rule("await", (0, 16384, 8192), (3, 16384, 15000), (3, 16384, 0)) == [-1016, -1030, -1000]


def test_waves_per_tile_by_rounds_on_the_chip(rule):
    """(16-row tiles that a hint covers, columns, gated).  Plain rows: one line.  Gated rows of 2048 columns and more: 8 waves again where
    4 take two rounds as well.  Rows of more than 4096 columns and few tiles: always 8."""
    assert rule("waves", (512, 4096, 0), (513, 4096, 0), (513, 4128, 0), (897, 4096, 0), (4096, 32, 0)) == [8, 4, 8, 4, 4]
    assert rule("waves", (512, 2048, 1), (513, 2048, 1), (896, 4096, 1), (897, 4096, 1), (897, 2016, 1), (1194, 2048, 1), (1195, 2048, 1),
                (600, 4128, 1)) == [8, 4, 4, 8, 4, 8, 4, 8]


def test_early_bundles_where_the_last_step_kept_every_loader_busy(rule):
    """Rows of more than 2 KiB and the low-rank predictor; (neurons added by the last step, loaders, threads with a first word) -> tiles decided
    early: one per pair of loaders, at most as many as there are."""
    assert rule("form", (1, 0, 0), (2, 0, 0), (4, 0, 0), (16, 0, 0), (4, 1, 0), (16, 1, 0)) == [0, 0, 1, 1, 0, 0]
    assert rule("tiles", (0, 40, 256), (19, 40, 256), (20, 40, 256), (65536, 40, 256), (500, 128, 256), (500, 128, 31), (500, 10, 3),
                (1, 2, 256)) == [0, 0, 20, 20, 64, 31, 3, 1]


def test_first_units_of_the_loaders_without_an_early_bundle(rule):
    """Every unit that is dealt in turn has one loader in the first round, and is the part of a bundle that its number says; some of `tiles` pairs
    have an early bundle (a mask of 31 bits, those of the last tiles)."""
    for loaders, tiles in ((40, 20), (128, 64), (128, 31), (10, 3), (2, 1), (26, 13)):
        for mask in (0, 1, 2, 0x155, 0x7fffffff, 0x40080001):
            mask &= (1 << min(tiles, 31)) - 1
            early = mask << max(tiles - 31, 0)
            others = [lw for lw in range(loaders) if lw // 2 >= tiles or not early >> (lw // 2) & 1]
            units = rule("unit", *[(lw, tiles, mask) for lw in others]) if others else []
            assert units == list(range(len(others))), (loaders, tiles, mask)
            assert all(u % 2 == lw % 2 for u, lw in zip(units, others))
