"""Workgroups of a one-launch step that wait for others of it (csrc/attn_division.h, heads_of_copier), played on the host: no GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# sequences, KV heads, attention workgroups, scanning workgroups
CALLS = [(4, 40, 320, 188), (1, 32, 128, 380), (8, 8, 256, 100), (16, 8, 256, 64), (16, 1, 16, 480), (1, 4, 8, 64), (3, 7, 56, 300), (15, 40, 300, 60),
         (32, 8, 256, 32), (32, 1, 32, 448), (31, 64, 248, 31), (17, 2, 40, 100), (32, 40, 1280, 32)]


@pytest.mark.parametrize("overlap", [2, 3, 4])
def test_of_overlapping_launches_all_end(tmp_path, overlap):
    """Whichever stream each XCD serves first, what waits leaves room for what it waits for."""
    exe = str(tmp_path / "attn_waiting")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2506_14158_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "attn_waiting.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe, "60", str(overlap)] + [str(x) for c in CALLS for x in c], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
