"""How workgroups of a launch hand things to each other, played on the host: those of a divided unit (csrc/attn_meet.h; where their parts lie:
csrc/attn_division.h), and writers and readers that may give up (csrc/told.h).  No GPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run(tmp_path, source, *args):
    exe = str(tmp_path / source)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2506_14158_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", source + ".cpp"), "-o", exe], check=True)
    return subprocess.run([exe, *args], capture_output=True, text=True)


def test_every_launch_ends_and_merges_its_own_parts_once(tmp_path):
    """Late starters, workgroups that are gone before others start, replays under one tag, one workspace for several launches."""
    r = run(tmp_path, "attn_meet", "6000")
    assert r.returncode == 0, r.stdout


def test_parts_do_not_overlap(tmp_path):
    """Slabs, words and statistics of a team: inside its region, no byte in two of them; every column of every row once."""
    r = run(tmp_path, "attn_region")
    assert r.returncode == 0, r.stdout


def test_what_was_told_is_heard_or_taken_back(tmp_path):
    """Readers that are gone before the writer begins, and the other way round, replays under one tag."""
    r = run(tmp_path, "told", "60000")
    assert r.returncode == 0, r.stdout
