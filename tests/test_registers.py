"""Registers of the single-launch step with the gate predictor, as the compiler reports them: two workgroups fit a compute unit at every
width, and no register goes to memory, which would queue up behind the host reads."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2312_11514_amd import build


def _report(source):
    """Per kernel, by its mangled name: what -Rpass-analysis=kernel-resource-usage prints"""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("no hipcc")
    text = subprocess.run([hipcc, *build.HIPCC_FLAGS, "--offload-device-only", "-Rpass-analysis=kernel-resource-usage", "-c", "-o",
                           os.devnull, os.path.join(build.HERE, "csrc", source)], capture_output=True, text=True, check=True).stderr
    kernels = {}
    for key, value in re.findall(r"remark: .*?([A-Za-z][A-Za-z ]*?)(?: \[[^\]]*\])?: (\S+)", text):
        if key == "Function Name":
            kernels[value] = {}
        elif kernels:
            list(kernels.values())[-1][key] = value
    return kernels


@pytest.mark.parametrize("source,element", [("step1_f16_gate.hip", "DF16_"), ("step1_f32_gate.hip", "f")])
def test_two_workgroups_per_compute_unit(source, element):
    kernels = _report(source)
    for ni in (1, 2, 4, 6, 8, 9, 12, 16):
        name = f"_ZN3lif7k_step1I{element}Li{ni}ELb0ELb1EEEvNS_8StepArgsE"
        got = kernels[name]
        assert got["VGPRs Spill"] == "0", (name, got)
        assert int(got["Occupancy"]) >= 2, (name, got)


# Low-rank predictor: three workgroups as long as a loader's bundle piece, row piece and x leave room, two for rows of more than 9 KiB
# and gated rows of more than 6 KiB, one for gated rows of more than 9 KiB.  An early bundle must not cost one.
@pytest.mark.parametrize("form,workgroups", [("plain", (3, 3, 3, 3, 3, 3, 2, 2)), ("glu", (3, 3, 3, 3, 2, 2, 1, 1))])
@pytest.mark.parametrize("dtype,element", [("f16", "DF16_"), ("f32", "f")])
def test_workgroups_of_the_lowrank_forms(dtype, element, form, workgroups):
    kernels = _report(f"step1_{dtype}_{form}.hip")
    for ni, least in zip((1, 2, 4, 6, 8, 9, 12, 16), workgroups):
        name = f"_ZN3lif7k_step1I{element}Li{ni}ELb{int(form == 'glu')}ELb0EEEvNS_8StepArgsE"
        got = kernels[name]
        assert got["VGPRs Spill"] == "0" and got["ScratchSize"] == "0", (name, got)
        assert int(got["Occupancy"]) >= least, (name, got)
