"""bench.py's command-line contract that can be checked without a GPU."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert r.returncode != 0
    assert "one GPU" in r.stderr and r.stdout.strip() == ""


def test_bench_never_reaches_the_oracle_outside_its_cpu_baseline_leg():
    src = open(os.path.join(ROOT, "bench.py")).read()
    body = src.split("def cpu_baseline", 1)[1].split("\ndef ", 1)[0]
    assert "from oracle import" in body
    assert src.count("oracle import") == 1, "the oracle may only be imported inside cpu_baseline"
    pkg = os.path.join(ROOT, "paper_2312_11514_amd")
    for name in os.listdir(pkg):
        if name.endswith(".py"):
            assert "oracle" not in open(os.path.join(pkg, name)).read(), name
    for name in os.listdir(os.path.join(ROOT, "workloads")):
        if name.endswith(".py"):
            text = open(os.path.join(ROOT, "workloads", name)).read()
            assert "import oracle" not in text and "from oracle" not in text, name


def test_traffic_counts_every_form_of_an_ffn_call(tmp_path):
    """The counter files of a run that has FFN calls of two stages, with and without the finish kernel, and of a single launch, between
    steps: the copy of 256 MiB is reported as half, so everything counts double."""
    sys.path.insert(0, ROOT)
    import bench
    kernels = ["__amd_rocclr_copyBuffer", "k_step1", "k_ffn_down1", "k_ffn_up", "k_ffn_down1", "k_ffn_one", "k_ffn_up", "k_ffn_down",
               "k_ffn_down_finish", "k_ffn_one", "k_ffn_one", "k_predict_xa", "k_ffn_down1"]
    kib = [131072, 1000, 1000, 8, 2, 5, 16, 3, 1, 6, 9, 1000, 1000]
    for counter in ("FETCH_SIZE", "WRITE_SIZE"):
        d = tmp_path / ("pmc_" + counter)
        d.mkdir()
        lines = ["Dispatch_Id,Kernel_Name,Counter_Name,Counter_Value"]
        lines += ["%d,void lif::%s(args),%s,%d" % (i, k, counter, v) for i, (k, v) in enumerate(zip(kernels, kib))]
        (d / "run_counter_collection.csv").write_text("\n".join(lines) + "\n")
    got = bench.pmc_traffic(str(tmp_path))
    for counter in ("FETCH_SIZE", "WRITE_SIZE"):
        assert got[counter]["calls"] == 5
        assert got[counter]["bytes_per_call"] == 2 * 1024 * (8 + 2 + 5 + 16 + 3 + 1 + 6 + 9) / 5
