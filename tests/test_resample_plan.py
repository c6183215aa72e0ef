"""How sequential acceptance is divided between workgroups (csrc/resample_plan.h), played on the host: no GPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# (sequences, nodes, vocabulary): teams of every size and kernel, one launch and several, with sequences that fill no round
TEAMS = [(4, 64, 32000), (16, 64, 32000), (100, 8, 32000), (8, 64, 128256), (16, 64, 128256), (17, 64, 128256), (32, 64, 128256),
         (64, 64, 128256), (130, 8, 128256), (9, 64, 256000), (16, 64, 256000), (33, 64, 151936), (51, 64, 151936), (1, 64, 1000000),
         (8, 64, 524288), (7, 64, 600000), (2, 64, 2097152), (5, 64, 2097152)]
# a workgroup a node, or short rows of so many sequences that they are not decided that way
ROWS = [(1, 20, 1000), (16, 128, 4096), (4, 128, 16384), (128, 8, 8000), (128, 4, 16000), (250, 8, 4000), (256, 8, 4096), (257, 7, 4096),
        (500, 2, 16384), (1000, 2, 1000), (2048, 1, 1000)]
CALLS = TEAMS + ROWS


def test_of_two_overlapping_calls_one_goes_on(tmp_path):
    """Workgroups of a team wait for each other: whichever stream each XCD serves first, no two calls hold each other up."""
    exe = str(tmp_path / "resample_plan")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2506_14158_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "resample_plan.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe, "10"] + [str(x) for c in CALLS for x in c], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
