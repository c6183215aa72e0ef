"""Waiting workgroups of attention launches (csrc/attn_division.h, plan_waiting), played on the host: no GPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# sequences, KV heads, workgroups that would merge in one turn, attention workgroups, scanning workgroups (0: no step)
CALLS = [(4, 40, 320, 320, 188), (1, 32, 64, 128, 380), (32, 8, 512, 256, 32), (32, 1, 64, 32, 448), (31, 64, 1984, 248, 31), (16, 8, 128, 256, 64),
         (1, 4, 8, 8, 64), (3, 7, 10, 56, 300), (8, 8, 256, 256, 0), (64, 32, 4096, 512, 0), (13, 8, 416, 512, 0), (1, 1, 1, 8, 0), (32, 40, 0, 1280, 32)]


def test_of_two_overlapping_launches_both_end(tmp_path):
    """Whichever stream each XCD serves first, what waits leaves room for what it waits for."""
    exe = str(tmp_path / "attn_waiting")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2506_14158_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "attn_waiting.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe, "20"] + [str(x) for c in CALLS for x in c], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
