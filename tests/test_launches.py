"""What the host side of liblif.so launches, looked at without a GPU: the library is loaded behind a stand-in for the HIP
runtime (hip_host_stub.cpp) that runs nothing and writes every launch down.  In a process of its own, because the stand-in
takes the place of the runtime."""
import ctypes as C
import json
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LDS_DEFAULT, LDS_MOST = 64 * 1024, 160 * 1024      # of a workgroup: without asking, and in all


class Library:
    """liblif.so over the stand-in (in the child process)."""

    def __init__(self, stub):
        self.stub = C.CDLL(stub, mode=C.RTLD_GLOBAL)
        self.stub.stub_kernel.restype = C.c_char_p
        sys.path.insert(0, ROOT)
        from paper_2312_11514_amd import binding
        self.b = binding
        self.lib = C.CDLL(binding.LIB_PATH)
        for name, (res, args) in binding.EXPORTS.items():
            getattr(self.lib, name).restype, getattr(self.lib, name).argtypes = res, args
        self.p = 1 << 32                           # a device address: 256-byte aligned, never read

    def layer(self, d, F=1024, rank=16, k=3, capacity=512, max_batch=1, glu=0, f16=True, gate=False, full=False):
        b, p = self.b, self.p
        cfg = b.LifConfig(d, F, rank, k, capacity, max_batch, int(glu), b.LIF_F16 if f16 else b.LIF_F32, int(full), 0, int(gate), 0.0)
        buf = b.LifBuffers(p, None if gate else p, None, p, p, p, p, p, p, self.lib.lif_workspace_bytes(C.byref(cfg)), None)
        assert buf.workspace_bytes, (d, F, rank, max_batch, glu, f16)
        h = C.c_void_p()
        assert self.lib.lif_create(C.byref(cfg), C.byref(buf), C.byref(h)) == 0, self.lib.lif_last_error_string()
        return h

    def launches(self, call):
        """[kernel, grid, block, dynamic LDS, LDS allowed] of every launch of a call, and what it returned"""
        self.stub.stub_clear()
        rc = call()
        got = []
        for i in range(self.stub.stub_launches()):
            grid, block, lds, allowed = C.c_uint32(), C.c_uint32(), C.c_size_t(), C.c_int()
            self.stub.stub_geometry(i, C.byref(grid), C.byref(block), C.byref(lds), C.byref(allowed))
            got.append([self.stub.stub_kernel(i).decode(), grid.value, block.value, lds.value, allowed.value])
        return rc, got

    def step(self, h, batch, step_mask=None):
        p = self.p
        return self.launches(lambda: self.lib.lif_step(h, p, batch, p, p, step_mask or p + 4096, p, p, p, p, None))


def _every_width():
    """One row width for every kernel form: 64-lane loads per vector 1, 2, 4, 6, 8, 9, 12, 16, whole and ragged"""
    for f16 in (True, False):
        ve = 8 if f16 else 4
        for ni in (1, 2, 3, 5, 7, 9, 11, 16):
            for d in (64 * ni * ve, 64 * ni * ve - 3 * ve):
                yield f16, d


def child_lds(lib):
    seen = 0
    for f16, d in _every_width():
        for glu, gate in ((0, False), (1, False), (0, True)):
            most = min(8, 64 * 1024 // (d * (2 if f16 else 4)))
            h = lib.layer(d, max_batch=most, glu=glu, f16=f16, gate=gate)
            for batch in range(1, most + 1):
                rc, got = lib.step(h, batch)
                assert rc == 0 and got, (f16, d, glu, gate, batch)
                for kernel, grid, block, lds, allowed in got:
                    assert lds <= max(LDS_DEFAULT, allowed) and lds <= LDS_MOST, (f16, d, glu, gate, batch, kernel, lds, allowed)
                    assert grid > 0 and block % 64 == 0
                    seen += lds > LDS_DEFAULT
            lib.lib.lif_destroy(h)
    return seen


def child_step_mask(lib):
    """Kernels launched for a pass of tokens, by the address of the step mask"""
    p, got = lib.p, {}
    for gate in (False, True):
        h = lib.layer(512, max_batch=4, gate=gate)
        for offset in (0, 8, 1, 2, 4, 7):
            rc, seen = lib.launches(lambda: lib.lib.lif_step_tokens(h, p, 3, 2, p, p, p + 4096 + offset, p, p, p, p, None))
            assert rc == 0, offset
            got["%d%s" % (offset, " gate" if gate else "")] = [k[0] for k in seen]
        assert lib.step(h, 3, p + 4096 + 4)[0] == lib.b.LIF_INVALID_ARG
        lib.lib.lif_destroy(h)
    return got


def child_step_lds(lib):
    """Dynamic LDS of the batched step, by shape"""
    got = {}
    for d, batch, glu, f16 in ((4096, 2, 0, True), (2048, 5, 0, True), (2048, 6, 0, True), (2560, 4, 0, True), (1536, 7, 0, True),
                               (1536, 8, 0, True), (4096, 1, 1, True), (1024, 2, 0, False)):
        h = lib.layer(d, max_batch=max(batch, 2), glu=glu, f16=f16)
        rc, seen = lib.step(h, max(batch, 2))
        assert rc == 0
        got["d %d, %d tokens%s" % (d, max(batch, 2), ", gated" if glu else "")] = max(k[3] for k in seen if "k_step_batch" in k[0])
        lib.lib.lif_destroy(h)
    return got


def child_one_words(lib):
    """Bytes of workspace and workgroups of a reset, by width and capacity"""
    got = {}
    for d in (2048, 2056, 4096):
        for capacity in (8192, 16384, 24576):
            h = lib.layer(d, capacity=capacity)
            cfg = lib.b.LifConfig(d, 1024, 16, 3, capacity, 1, 0, lib.b.LIF_F16, 0, 0, 0, 0.0)
            rc, seen = lib.launches(lambda: lib.lib.lif_reset(h, None))
            assert rc == 0 and len(seen) == 1
            got["%d %d" % (d, capacity)] = [lib.lib.lif_workspace_bytes(C.byref(cfg)), seen[0][1]]
            lib.lib.lif_destroy(h)
    return got


def child_ffn_one(lib, cases):
    """Kernels of one lif_sparse_ffn call of one token, by row-count hint"""
    got = {}
    for name, (dtype, glu, gate, full, d, F, _, capacity, hints) in cases.items():
        h = lib.layer(d, F=F, rank=8, k=2, capacity=capacity, glu=glu, f16=dtype == "f16", gate=gate, full=full)
        for hint in [0] + hints:
            assert lib.lib.lif_set_expected_rows(h, hint) == 0
            for call in (lib.lib.lif_sparse_ffn, lib.lib.lif_sparse_ffn_static):
                rc, seen = lib.launches(lambda: call(h, lib.p, 1, lib.p, None))
                assert rc == 0
                got["%s %d %s" % (name, hint, call.__name__)] = [k[0] for k in seen]
        lib.lib.lif_destroy(h)
    return got


def child_ffn_down(lib, cases):
    """[kernel, workgroups, threads] of the launches of one lif_sparse_ffn call behind the activations, by case and row-count hint"""
    got = {}
    for name, (dtype, batch, full, d, capacity, hints) in cases.items():
        h = lib.layer(d, F=65536, rank=8, k=2, capacity=capacity, max_batch=batch, f16=dtype == "f16", full=full)
        for hint in hints:
            assert lib.lib.lif_set_expected_rows(h, hint) == 0
            rc, seen = lib.launches(lambda: lib.lib.lif_sparse_ffn(h, lib.p, batch, lib.p, None))
            assert rc == 0
            got["%s %d" % (name, hint)] = [k[:3] for k in seen[1:]]
        lib.lib.lif_destroy(h)
    return got


def _run(tmp_path_factory, what, *args):
    stub = str(tmp_path_factory.getbasetemp() / "hip_host_stub.so")
    if not os.path.exists(stub):
        subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", stub, os.path.join(HERE, "hip_host_stub.cpp")], check=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), stub, what] + [json.dumps(a) for a in args], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return json.loads(r.stdout.splitlines()[-1])


@pytest.fixture
def child(tmp_path_factory):
    from paper_2312_11514_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2312_11514_amd.build import build_library
        build_library()
    return lambda what, *args: _run(tmp_path_factory, what, *args)


def test_lds_of_every_launch_is_allowed(child):
    """A launch with more than 64 KiB of LDS needs the limit of its own kernel form raised (lif_create)."""
    assert child("lds") > 0


def test_two_workgroups_of_a_batched_step_per_compute_unit(child):
    """Every workgroup of the launch carries the same LDS: what the bookkeeping workgroup needs for the deletion plan must not come on
    top of the x and rows of a loader."""
    for shape, lds in child("step_lds").items():
        assert 0 < lds <= LDS_MOST // 2, (shape, lds)


def test_step_mask_of_a_pass_may_have_any_address(child):
    """The batched step reads the step mask by 64-bit words; a pass of tokens whose step mask is not aligned to them goes
    through the separate kernels, which write it byte by byte and read the tokens' masks (lif_step refuses such a mask)."""
    for case, kernels in child("step_mask").items():
        by_words = any("k_step_batch" in k for k in kernels)
        assert by_words == (int(case.split()[0]) % 8 == 0), (case, kernels)
        assert by_words or [n for n in ("window_plan", "k_load", "ffn_up", "ffn_down") if not any(n in k for k in kernels)] == []


def test_words_of_the_single_launch_ffn_only_where_it_is_launched(child):
    """Four copies of a word for every slot, cleared by every reset: for at most 64 column slices (d = 2048 in fp16) and 16384 slots."""
    got = child("one_words")
    for d in (2048, 2056, 4096):
        (less, _), (most, reset), (more, _) = (got["%d %d" % (d, c)] for c in (8192, 16384, 24576))
        extra = (most - less) - (more - most)       # over what grows with every slot
        if d <= 2048:
            assert extra >= 4 * 8 * 16384
        else:
            assert abs(extra) < 4096 and reset <= (16384 + 8192) // 256, (d, extra, reset)


def test_single_launch_ffn_is_compared_with_two_launches(child):
    """tests/test_ffn_one.py compares what it says: its hints take the single launch, and no hint (the capacity) two."""
    from tests.test_ffn_one import CASES
    got = child("ffn_one", CASES)
    assert len(got) == sum(2 + 2 * len(c[-1]) for c in CASES.values())
    for case, kernels in got.items():
        if case.split()[1] == "0":
            assert "k_ffn_up" in kernels[0] and "k_ffn_down" in kernels[1], (case, kernels)
        else:
            assert len(kernels) == 1 and "k_ffn_one" in kernels[0], (case, kernels)


def test_waves_of_a_layer_whose_capacity_the_hint_exceeds(child):
    """Rows past the capacity are never in use: a hint beyond it counts as the capacity.  Eight waves (512 threads) for at most 2048 rows of
    one token, whatever the hint says."""
    cases = {"%s%d %d" % (dtype, full, capacity): (dtype, 1, bool(full), 4096, capacity, [0, capacity, capacity + 1, 2400, 5000, 2**31 - 1])
             for dtype in ("f16", "f32") for full in (0, 1) for capacity in (900, 2048)}
    got = child("ffn_down", cases)
    assert len(got) == 8 * 6
    for case, kernels in got.items():
        assert len(kernels) == 1 and "k_ffn_down1" in kernels[0][0] and kernels[0][2] == 512, (case, kernels)


def test_waves_of_a_hint_around_the_rows_of_eight(child):
    """The hint is the mean number of rows in use: 16 waves (1024 threads) where a sixteenth more than that is beyond what eight waves take in
    one go (2048), eight up to there, and again where every row is read and the rows make several chunks."""
    hints = {"f16": (1, 1900, 1928, 1929, 2048, 2100, 2340, 3000, 9000), "f32": (1928, 1929, 2100)}
    got = child("ffn_down", {dtype: (dtype, 1, False, 4096, 9000, h) for dtype, h in hints.items()})
    for case, kernels in got.items():
        assert len(kernels) == 1 and kernels[0][2] == (512 if int(case.split()[1]) <= 1928 else 1024), (case, kernels)
    got = child("ffn_down", {"full": ("f16", 1, True, 4096, 9000, (1928, 1929, 4000, 4200))})
    assert [k[0][2] for k in got.values()] == [512, 1024, 1024, 512]


if __name__ == "__main__":
    print(json.dumps(globals()["child_" + sys.argv[2]](Library(sys.argv[1]), *map(json.loads, sys.argv[3:]))))
