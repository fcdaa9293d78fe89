"""The plane passes' transposes (planes.hip) keep every lane, those without a plane among them, inside
its wave's LDS buffer: the index functions of plane_lds.hpp over all lanes and plane shapes, built
for the host."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1507_05156_amd", "csrc")


def test_every_lane_stays_in_its_buffer(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path / "plane_lds_check")
    subprocess.run([gxx, "-O1", "-std=c++17", "-I", CSRC, os.path.join(HERE, "host", "plane_lds_check.cpp"), "-o", exe],
                   check=True)
    rows = [tuple(map(int, l.split())) for l in
            subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()]
    assert len(rows) == 16
    assert [r for r in rows if r[3] != 0] == []
