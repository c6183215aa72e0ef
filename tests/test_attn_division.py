"""The division of attention work between workgroups (csrc/attn_division.h), played on the host: no GPU."""
import os
import subprocess

import pytest

from tests.test_gpu_division import CASES, plan_inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def player(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("division") / "attn_division")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2506_14158_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "attn_division.cpp"), "-o", exe], check=True)
    return exe


# 20000 random launches of a kind: tiles walked once, the merge reads what this call wrote and all of it
KINDS = ["split", "balanced"]


@pytest.mark.parametrize("kind", KINDS)
def test_merge_reads_what_the_call_wrote(player, kind):
    r = subprocess.run([player, kind, "20000"], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


@pytest.mark.parametrize("case", CASES, ids=lambda c: c.name)
def test_gpu_cases_are_divided_as_they_say(player, case):
    r = subprocess.run([player, "plan"] + [str(x) for x in plan_inputs(case)], capture_output=True, text=True, check=True)
    teams, split = (int(x) for x in r.stdout.split())
    units = case.B * case.Hkv
    assert split > 1 if case.kind == "split" else split == 0 and teams > units // 2, r.stdout
