"""Workgroups of a one-launch step that wait for others of it (csrc/attn_division.h, heads_of_copier), played on the host: no GPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# sequences, KV heads, attention workgroups, scanning workgroups
CALLS = [(4, 40, 320, 188), (1, 32, 128, 380), (32, 8, 256, 32), (32, 1, 32, 448), (31, 64, 248, 31), (16, 8, 256, 64), (1, 4, 8, 64),
         (3, 7, 56, 300), (32, 40, 1280, 32)]


def test_of_overlapping_launches_all_end(tmp_path):
    """Whichever stream each XCD serves first, what waits leaves room for what it waits for."""
    exe = str(tmp_path / "attn_waiting")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2506_14158_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "attn_waiting.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe, "40", "2"] + [str(x) for c in CALLS for x in c], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
