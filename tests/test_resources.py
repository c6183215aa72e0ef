"""What the compiler says about the registers of kernels that are written for a number of them (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2506_14158_amd import build


def resources(source):
    """{kernel: {"VGPRs": .., "SGPRs Spill": .., "ScratchSize": .., "VGPRs Spill": .., "Occupancy": waves per SIMD}}"""
    r = subprocess.run([build.HIPCC] + build.FLAGS + ["-Rpass-analysis=kernel-resource-usage", "--offload-device-only", "-c",
                        os.path.join(build.CSRC, source), "-o", os.devnull], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    out, name = {}, None
    for line in r.stderr.splitlines():
        m = re.search(r"remark: (?:.*: )?\s*Function Name: (\S+)", line)
        if m:
            name = m.group(1)
            out[name] = {}
            continue
        m = re.search(r"(SGPRs Spill|VGPRs Spill|VGPRs|ScratchSize|Occupancy)(?: \[[^\]]*\])?: (\d+)", line)
        if m and name:
            out[name][m.group(1)] = int(m.group(2))
    return out


@pytest.fixture(scope="module")
def resample():
    return resources("accept_resample.hip")


@pytest.mark.parametrize("kernel, blocks", [("accept_resample_kernel", 1), ("accept_resample_kernel", 2), ("accept_resample_kernel", 4),
                                            ("accept_resample_kernel", 8), ("resample_rows_kernel", 1), ("resample_rows_kernel", 2),
                                            ("resample_rows_kernel", 4)])
def test_sequential_acceptance_keeps_its_rows_in_registers(resample, kernel, blocks):
    """`blocks` of 512 tokens a wave: no kernel spills, and as many workgroups (of eight waves on four SIMDs) fit on a CU as the
    launches count on."""
    got = {k: v for k, v in resample.items() if kernel in k and "Li%dE" % blocks in k}
    assert len(got) == 3, sorted(resample)                   # a kernel per type
    for name, r in got.items():
        assert r["VGPRs Spill"] == 0 and r["ScratchSize"] == 0, (name, r)
        assert r["Occupancy"] >= (4 if blocks <= 2 else 2), (name, r)


def test_attention_that_merges_nothing_keeps_nothing_for_it():
    """Many-row kernels: no scratch memory in any of them; those without the rest of a step (kNoStep, 0) spill no scalar registers where
    they walk one unit (parts::kWhole, 0), next to none where they walk shares (kShares, 1; a few paged, for the page table)."""
    got = {k: v for k, v in resources("tree_attn_mfma_f16.hip").items() if "tree_attn_mfma_kernel" in k}
    for name, r in got.items():
        assert r["VGPRs Spill"] == 0 and r["ScratchSize"] == 0, (name, r)
        # as many waves on a SIMD as the launches count on: two of four-wave workgroups of head size 64, or of eight waves
        assert r["Occupancy"] >= (1 if "kernelILi4E" in name and "ELi128E" in name else 2), (name, r)
    for merge, paged, most in ((0, False, 0), (0, True, 0), (1, False, 2), (1, True, 8)):
        lean = {k: v for k, v in got.items() if "StepKindE0ELNS_5parts5MergeE%dE" % merge in k and ("Lb1ELb1E" in k) == paged}
        assert len(lean) == 4, sorted(got)                   # rows, head sizes
        for name, r in lean.items():
            assert r["SGPRs Spill"] <= most, (name, r)
