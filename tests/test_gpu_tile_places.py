"""Tiles in unusual places: planes anywhere along z, boxes far from the
origin, particles on or beyond a periodic edge, other units.  FP64 against the
oracle bit for bit, FP32 pair by pair."""
import numpy as np
import pytest

from paper_1210_8084_amd import workloads as W
from test_gpu_tiles import T, check  # noqa: F401  (T: fixture)

pytestmark = pytest.mark.gpu

R, P = W.REFLECT, W.PERIODIC


@pytest.mark.parametrize("n", [700, 6001])  # c-bins whole, c-bins in sort cells
@pytest.mark.parametrize("z", [-0.5, 0.0, 0.499, -0.7])
def test_plane_anywhere_along_z(T, oracle, n, z):  # noqa: F811
    w = W.random_plane(n=n, seed=3, ncell=(9, 8), bc=(R, P), nobin=(2, 2))
    w.state["z"][:] = z
    assert check(T, oracle, w.state, w.grid, w.params) > 100
