"""How sequential acceptance is divided between workgroups (csrc/resample_plan.h), played on the host: no GPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# (sequences, vocabulary): teams of every size and kernel, one launch and several, with sequences that fill no round
CALLS = [(4, 32000), (16, 32000), (100, 32000), (8, 128256), (16, 128256), (17, 128256), (32, 128256), (64, 128256), (130, 128256),
         (9, 256000), (16, 256000), (33, 151936), (51, 151936), (1, 1000000), (8, 524288), (7, 600000), (2, 2097152), (5, 2097152)]


def test_of_two_overlapping_calls_one_goes_on(tmp_path):
    """Workgroups of a team wait for each other: whichever stream each XCD serves first, no two calls hold each other up."""
    exe = str(tmp_path / "resample_plan")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2506_14158_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "resample_plan.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe, "20"] + [str(x) for c in CALLS for x in c], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
