"""What the compiler reports of kernels whose speed rests on their registers."""
from __future__ import annotations

import os
import re
import subprocess

import pytest

from paper_2604_08971_amd import build


# The staged active pass: two workgroups of eight waves share a compute unit up to 128 registers a lane, without scratch
@pytest.mark.parametrize("half", ["bf16", "f16"])
def test_two_workgroups_of_the_staged_active_pass(half, tmp_path):
    cmd = ["hipcc"] + build.FLAGS + (["-DSF_HALF_F16"] if half == "f16" else []) + ["--cuda-device-only", "-Rpass-analysis=kernel-resource-usage",
           "-c", os.path.join(build.CSRC, "attention_bf16.hip"), "-o", str(tmp_path / "a.o")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    found = 0
    for part in r.stderr.split("Function Name: ")[1:]:
        if re.match(r"\S*attend_bf16_kernelILi(32|64)ELi8E", part):
            total = sum(int(re.search(rf" {n}: (\d+)", part).group(1)) for n in ("VGPRs", "AGPRs"))
            assert total <= 128 and re.search(r"ScratchSize \[bytes/lane\]: 0 ", part), part.split("\n")[0]
            found += 1
    assert found == 2


# The whole-row kernels: 64-row tiles share a compute unit (sixteen waves, 128 registers), and only the widest FFN spills, ten registers
# a lane and chunk of channels
@pytest.mark.parametrize("half", ["bf16", "f16"])
def test_whole_row_kernels(half, tmp_path):
    cmd = ["hipcc"] + build.FLAGS + (["-DSF_HALF_F16"] if half == "f16" else []) + ["--cuda-device-only", "-Rpass-analysis=kernel-resource-usage",
           "-c", os.path.join(build.CSRC, "gemm_bf16_rows.hip"), "-o", str(tmp_path / "a.o")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    found = 0
    for part in r.stderr.split("Function Name: ")[1:]:
        m = re.match(r"\S*(gemm|ffn)_rows_kernelILi(\d)ELi(\d)E", part)
        if m:
            total = sum(int(re.search(rf" {n}: (\d+)", part).group(1)) for n in ("VGPRs", "AGPRs"))
            scratch = int(re.search(r"ScratchSize \[bytes/lane\]: (\d+)", part).group(1))
            assert total <= (128 if m.group(2) == "1" else 256), part.split("\n")[0]
            assert scratch <= (40 if m.groups() == ("ffn", "2", "4") else 0), part.split("\n")[0]
            found += 1
    assert found == 12


# Those that keep a sum per K slice: no scratch, and two workgroups per compute unit but for the FFN of 256 columns
@pytest.mark.parametrize("half", ["bf16", "f16"])
def test_whole_row_kernels_with_k_slices(half, tmp_path):
    cmd = ["hipcc"] + build.FLAGS + (["-DSF_HALF_F16"] if half == "f16" else []) + ["--cuda-device-only", "-Rpass-analysis=kernel-resource-usage",
           "-c", os.path.join(build.CSRC, "gemm_bf16_rows.hip"), "-o", str(tmp_path / "a.o")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    found = 0
    for part in r.stderr.split("Function Name: ")[1:]:
        m = re.match(r"\S*(gemm|ffn)_rows_sliced_kernelILi1ELi(\d)E", part)
        if m:
            total = sum(int(re.search(rf" {n}: (\d+)", part).group(1)) for n in ("VGPRs", "AGPRs"))
            assert total <= (256 if m.groups() == ("ffn", "2") else 128), part.split("\n")[0]
            assert re.search(r"ScratchSize \[bytes/lane\]: 0 ", part), part.split("\n")[0]
            found += 1
    assert found == 6


# The router's partial sums (up to 64 a lane) stay in registers
@pytest.mark.parametrize("half", ["bf16", "f16"])
def test_router_without_scratch(half, tmp_path):
    cmd = ["hipcc"] + build.FLAGS + (["-DSF_HALF_F16"] if half == "f16" else []) + ["--cuda-device-only", "-Rpass-analysis=kernel-resource-usage",
           "-c", os.path.join(build.CSRC, "moe.hip"), "-o", str(tmp_path / "a.o")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    found = 0
    for part in r.stderr.split("Function Name: ")[1:]:
        if "moe_router_kernel" in part.split("\n")[0]:
            assert re.search(r"ScratchSize \[bytes/lane\]: 0 ", part), part.split("\n")[0]
            found += 1
    assert found == 16
