"""Which steps go in one launch (csrc/step_plan.h), against measured times of both ways: no GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# chunks of a scanning workgroup, chunks of a row, key tiles, bytes of logits, fp32, greedy, many rows, workgroups on a CU; us in one launch, in two
TWO = [
    (55, 1, 54, 4627260, 0, 1, 0, 2, 189.5, 87.2), (8, 1, 5, 3417276, 0, 1, 1, 1, 30.5, 25.2), (9, 1, 6, 5499900, 0, 1, 1, 1, 33.0, 29.9),
    (175, 16, 14, 150829056, 0, 0, 1, 1, 58.8, 50.2), (114, 4, 12, 38080000, 0, 1, 1, 1, 99.6, 37.2), (31, 4, 4, 47808000, 0, 1, 1, 1, 35.6, 31.5),
    (137, 10, 8, 46516386, 0, 0, 1, 1, 56.5, 36.4), (71, 16, 12, 67719168, 1, 1, 0, 2, 73.6, 52.9), (87, 4, 7, 37440000, 0, 1, 1, 1, 80.0, 31.0),
    (1328, 16, 14, 383228928, 0, 0, 1, 1, 365.1, 59.7), (32, 3, 5, 5992132, 0, 1, 1, 1, 54.0, 33.7), (44, 4, 4, 122496000, 0, 1, 1, 1, 45.6, 39.6),
    (45, 7, 5, 156995496, 0, 1, 1, 2, 63.2, 47.0), (39, 16, 5, 219317760, 0, 1, 1, 2, 59.3, 54.1), (30, 6, 25, 23911680, 0, 1, 0, 2, 43.6, 41.7),
]
ONE = [
    (1, 1, 5, 60000, 1, 1, 0, 1, 13.1, 20.9), (1, 4, 9, 3840000, 0, 1, 0, 2, 15.4, 22.3), (37, 4, 45, 16384000, 0, 0, 0, 2, 75.0, 84.3),
    (24, 16, 6, 59254272, 0, 0, 1, 1, 21.4, 29.1), (10, 16, 4, 27703296, 0, 0, 1, 1, 16.3, 26.2), (26, 16, 5, 44633088, 0, 0, 1, 1, 22.4, 30.8),
    (44, 16, 23, 62845440, 0, 1, 1, 1, 45.7, 61.0), (9, 4, 8, 29184000, 0, 1, 0, 2, 20.6, 25.8), (13, 3, 5, 6870144, 0, 0, 1, 1, 19.4, 24.8),
    (9, 7, 4, 28658880, 0, 1, 1, 1, 18.2, 25.3), (5, 8, 8, 24226400, 1, 1, 0, 1, 29.4, 40.0), (2, 3, 9, 6302800, 0, 0, 0, 2, 12.8, 19.4),
    (3, 16, 5, 20520960, 0, 0, 0, 2, 13.0, 19.8), (6, 4, 4, 20992000, 0, 0, 1, 1, 14.3, 22.3), (3, 4, 5, 7424000, 0, 1, 1, 1, 18.9, 26.1),
    (16, 16, 5, 48224256, 0, 1, 1, 1, 19.9, 32.9),
]


@pytest.fixture(scope="module")
def says(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("step") / "step_plan")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2506_14158_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "step_plan.cpp"), "-o", exe], check=True)
    return lambda steps: subprocess.run([exe] + [str(x) for s in steps for x in s[:8]], capture_output=True, text=True, check=True).stdout.split()


@pytest.mark.parametrize("steps, one", [(TWO, "0"), (ONE, "1")], ids=["two", "one"])
def test_the_faster_way_is_taken(says, steps, one):
    assert all((s[8] < s[9]) == (one == "1") for s in steps)
    assert [(s, x) for s, x in zip(steps, says(steps)) if x != one] == []
