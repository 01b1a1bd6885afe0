"""CPU test of the margin with which the adjoint marks the bricks its sums go
to (dock_internal.h, corner_range and fk_spread): tests/cpp/corner_range_check.cpp
places atoms by two roundings of the same kinematics and requires the marked
nodes of one to hold the cell of the other, which a fixed margin of a hundredth
of a cell does not far from the origin or on fine grids."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_marked_nodes_hold_either_rounding(tmp_path):
    hipcc = next((c for c in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc") if c and os.path.exists(c)), None)
    if hipcc is None:
        pytest.skip("hipcc not found")
    exe = str(tmp_path / "corner_range_check")
    csrc = os.path.join(ROOT, "paper_2510_24186_amd", "csrc")
    r = subprocess.run([hipcc, "-O2", "-std=c++17", "-ffp-contract=off", "-I", os.path.join(ROOT, "include"), "-I", csrc,
                        os.path.join(ROOT, "tests", "cpp", "corner_range_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(r.stdout)
    missed, far, fixed = [int(t) for t in r.stdout.split()[1::2]]
    assert missed == 0 and r.returncode == 0
    assert far > 1000 and fixed > 100   # the cases do tell the two margins apart
