"""Host check of the kernels' launch shapes: tests/c/grid_check.cpp includes
the same grid header as the kernels (paper_2102_02888_amd/csrc/onebit_grid.h)
and enumerates whole launches, up to sizes that no GPU test reaches."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_every_tile_and_item_is_taken_once(tmp_path):
    exe = str(tmp_path / "grid_check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-Werror",
                    "-I" + os.path.join(ROOT, "paper_2102_02888_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "grid_check.cpp"), "-o", exe],
                   check=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:]
    assert "grid_check: ok" in r.stdout


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_every_row_and_block_of_the_worker_pass_is_taken_once(tmp_path):
    exe = str(tmp_path / "items_check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-Werror",
                    "-I" + os.path.join(ROOT, "paper_2102_02888_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "items_check.cpp"), "-o", exe],
                   check=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:]
    assert "items_check: ok" in r.stdout


def test_parity_cases_reach_every_partial_tile_shape():
    """A wave of the passes over blocks takes one 256-element sub-block of a
    block, or two of them, so a segment's last tile can end inside the first
    sub-block, inside the second (the second wave or half of a wave's part) or
    in the block's second half (the wave pairs' other wave).  The GPU parity
    cases must hold all three."""
    import oracle
    from test_gpu_parity import CASES
    kinds = set()
    for numel, n in CASES:
        L = oracle.Layout(numel, n)
        for b, e in zip(L.seg_begin, L.seg_end):
            tail = (int(e) - int(b)) % 1024
            if tail:
                kinds.add(0 if tail <= 256 else 1 if tail <= 512 else 2)
    assert kinds == {0, 1, 2}
