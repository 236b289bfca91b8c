"""The FP32 tile search where its code is its own (records read again from LDS,
the nearest image by rounding, the rounding of shifted origins): periodic axes
of one to five c-bins, whole and in sort cells, tiles that are not full,
particles outside the box and fast ones.  Pair by pair against the oracle."""
import numpy as np
import pytest

from paper_1210_8084_amd import workloads as W
from test_gpu_fp32_parity import check_against_oracle
from test_gpu_tiles import T  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

R, P = W.REFLECT, W.PERIODIC


@pytest.mark.parametrize("ncell", [(1, 1, 1), (2, 3, 4), (4, 4, 4), (5, 1, 2), (3, 5, 1), (9, 2, 5)], ids=str)
@pytest.mark.parametrize("d_over_w,dt_over", [(0.05, 0.05), (0.6, 0.4), (0.3, 1.5)])
def test_few_periodic_cbins(T, oracle, ncell, d_over_w, dt_over):  # noqa: F811
    w = W.random_box(n=6001, seed=17, ncell=ncell, bc=(P, P, P), d_over_w=d_over_w, dt_over=dt_over, nobin=(2, 2, 1))
    check_against_oracle(T, oracle, w, min_pairs=20)


@pytest.mark.parametrize("n", [1025, 1983, 4097])
@pytest.mark.parametrize("bc", [(R, P, P), (P, P, P)], ids=["rpp", "ppp"])
def test_tile_edges(T, oracle, n, bc):  # noqa: F811
    w = W.random_box(n=n, seed=n, ncell=(5, 4, 3), bc=bc, d_over_w=0.7, dt_over=0.6, nobin=(2, 2, 1))
    check_against_oracle(T, oracle, w, min_pairs=20)


def test_particles_outside_and_fast(T, oracle):  # noqa: F811
    """Positions up to a fifth of the box outside it, a tenth of the particles
    ten times faster."""
    w = W.random_box(n=4001, seed=5, ncell=(3, 2, 6), bc=(P, P, R), d_over_w=0.4, dt_over=0.5, nobin=(2, 2, 1))
    for k, L in zip(("x", "y", "z"), (1.0, 0.8, 0.6)):
        w.state[k] = w.state[k] * 1.4 - 0.2 * L
        w.state["v" + k][::10] *= 10.0
    check_against_oracle(T, oracle, w)


@pytest.mark.parametrize("ncell", [(40, 1, 1), (3, 1, 1)], ids=str)
def test_thin_tube_in_sort_cells(T, oracle, ncell):  # noqa: F811
    w = W.sod(n=30_001, ncell=ncell[0], nobin=ncell[0])
    check_against_oracle(T, oracle, w, min_pairs=1000)
