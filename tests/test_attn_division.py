"""The division of attention work between workgroups (csrc/attn_division.h), played on the host: no GPU."""
import os
import subprocess

import pytest

from paper_2506_14158_amd import binding as B
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
    teams, split, parts = (int(x) for x in r.stdout.split())
    units = case.B * case.Hkv
    assert split > 1 if case.kind == "split" else split == 0 and teams > units // 2, r.stdout
    # and the library's own plan is this one (rows, keys and workgroups per CU are the kernel's)
    shape = B.AttnShape(case.B, case.Hkv * case.G, case.Hkv, case.D, case.N, case.max_len + case.N, {"f32": B.S4C_F32, "bf16": B.S4C_BF16, "f16": B.S4C_F16}[case.dtype])
    assert B.s4c_tree_attn_num_splits(shape, case.max_len) == parts


# (B, Hkv, N, query rows, max_cache_len), the tile of 16-bit data of head size 128 (rows, keys, workgroups per CU): sequences so
# short that parts of them, or several in a row on one team, cost more than a workgroup for each
WHOLE = [
    ((16, 32, 20, 20, 64), (64, 32, 2)),
    ((5, 32, 60, 60, 500), (64, 32, 2)),
    ((20, 32, 20, 20, 300), (64, 32, 2)),
    ((40, 32, 60, 60, 1200), (64, 32, 2)),
    ((15, 32, 60, 60, 8000), (64, 32, 2)),
    ((17, 8, 20, 80, 500), (128, 64, 1)),
    ((25, 8, 60, 240, 1200), (256, 64, 1)),
    ((3, 8, 128, 1024, 500), (256, 64, 1)),
    ((40, 8, 60, 240, 150), (256, 64, 1)),
]


@pytest.mark.parametrize("sizes, tile", WHOLE, ids=lambda x: "-".join(map(str, x)))
def test_short_sequences_are_not_divided(player, sizes, tile):
    r = subprocess.run([player, "plan"] + [str(x) for x in sizes + tile + (1, 256)], capture_output=True, text=True, check=True)
    teams, split, _ = (int(x) for x in r.stdout.split())
    assert split == 1 and teams == sizes[0] * sizes[1], r.stdout


# a full round of the chip and more, exactly: no team walks fewer units than another, and no unit is divided
@pytest.mark.parametrize("B, teams", [(16, 512), (32, 512), (64, 512)])
def test_short_sequences_fill_the_chip(player, B, teams):
    r = subprocess.run([player, "plan"] + [str(x) for x in (B, 32, 20, 20, 64, 64, 32, 2, 1, 256)], capture_output=True, text=True, check=True)
    assert int(r.stdout.split()[0]) == teams, r.stdout
