"""How the candidate-tree scan cuts its rows (csrc/build_plan.h), on the host: no GPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_lists_fit_the_row_kernels_registers(tmp_path):
    """Up to 64 lists a row are merged from registers; more only where a row is longer than 64 of the longest lists cover."""
    exe = str(tmp_path / "build_plan")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2506_14158_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "build_plan.cpp"), "-o", exe], check=True)
    sizes = [(rows, chunks) for rows in (1, 20, 64, 127, 128, 256, 1000, 2048, 16384)
             for chunks in (1, 2, 7, 15, 16, 17, 19, 31, 32, 33, 63, 64, 65, 127, 128, 129, 256)]
    r = subprocess.run([exe] + [str(x) for s in sizes for x in s], capture_output=True, text=True, check=True)
    for (rows, chunks), line in zip(sizes, r.stdout.splitlines()):
        seg, lists = (int(x) for x in line.split())
        assert 1 <= seg <= min(8, chunks), (rows, chunks, seg)
        assert lists <= 64 or seg == 8, (rows, chunks, seg, lists)
    assert len(r.stdout.splitlines()) == len(sizes)
