"""Tile shapes of the NUFFT stages on both sides of each line of the rule: few
tiles are halved, up to 1024 of them only where the points are dense (sparse
points on a wide grid pay for the halos of small tiles: 1.5 times the time of
spreading and interpolation at 16 x 32)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
INC = os.path.join(os.path.dirname(HERE), "paper_2603_17166_amd", "csrc")


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("shape") / "tile_shape_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", INC, os.path.join(HERE, "tile_shape_check.cpp"), "-o", exe],
                   check=True)
    return exe


@pytest.mark.parametrize("rows,cols,w,n,shape", [
    (50, 350, 11, 20000, "8x8"), (33, 256, 6, 45000, "8x8"), (50, 350, 11, 0, "8x8"),  # under 256 tiles
    (97, 700, 6, 100000, "8x8"), (111, 840, 11, 300000, "8x16"),                        # dense points
    (165, 540, 11, 20000, "16x16"), (165, 540, 11, 200000, "16x16"), (165, 540, 11, 300000, "8x16"),
    (111, 840, 11, 30000, "16x16"),
    (237, 810, 11, 20000, "16x32"), (348, 1250, 11, 30000, "16x32"), (238, 810, 11, 300000, "16x16"),
    (297, 2016, 6, 1100000, "16x32"), (1, 4, 2, 1, "8x8"), (6000, 13440, 11, 20000000, "16x32"),
])
def test_shapes(harness, rows, cols, w, n, shape):
    out = subprocess.run([harness, str(rows), str(cols), str(w), str(n)], check=True, capture_output=True, text=True)
    assert out.stdout.strip() == shape
