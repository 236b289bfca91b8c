"""The range of the tile search's filter: the constants of the kernels are
those test_tile_filter.py builds its forms with, and records up to the limits
that the kernel takes as tame (the largest coordinate of a tile beside the
largest speed that goes with it) lose no candidate and keep their own terms
between those of the wild and the absent records."""
import os
import re

import numpy as np
import pytest

import test_tile_filter as tf

SRC = os.path.join(os.path.dirname(__file__), "..", "paper_1210_8084_amd", "csrc", "tpkmc_kernels.h")


def constants():
    out = {}
    for name, text in re.findall(r"constexpr float (kTile\w+) = ([^;]+);", open(SRC).read()):
        out[name] = eval(re.sub(r"(\d)f\b", r"\1", text), {}, dict(out))
    return out


K = constants()


def test_constants_are_the_kernels():
    for name, value in (("Kappa", tf.KAPPA), ("HalfUlp", tf.E), ("E2", tf.E2), ("E3", tf.E3), ("E6", tf.E6),
                        ("E18", tf.E18), ("Abs", tf.ABS)):
        assert K["kTile" + name] == pytest.approx(value, rel=1e-12), name


def vlim(x):
    return min(K["kTileVMax"], K["kTileOwn"] / (x + K["kTileVMax"] / K["kTileKappa"]))


@pytest.mark.parametrize("x", [0.6, 2.5, 6.0, 11.0, 20.0, 40.0, 64.0])
@pytest.mark.parametrize("D", [0.05, 0.6, 300.0])
def test_no_candidate_is_lost_up_to_the_limits(x, D):
    rng = np.random.default_rng(int(10 * x))
    v, ni, nj = vlim(x), 64, 6000
    hd2 = min(0.5001 * D * D, 30000.0)

    def draw(n):
        X = rng.uniform(-x, x, size=(n, 3))
        V = rng.normal(size=(n, 3))
        V *= (v * rng.uniform(0.2, 1.0, size=(n, 1))) / np.abs(V).sum(1, keepdims=True)
        return X, V

    Xi, Vi = draw(ni)
    Xj, Vj = draw(nj)
    # Two partners in three meet a record of the tile close to the edge of
    # one of the criteria, and stay within the limits.
    k = rng.integers(0, ni, nj)
    u = Vi[k] - Vj
    e = np.cross(u, rng.normal(size=u.shape))
    e /= np.linalg.norm(e, axis=1, keepdims=True)
    t = rng.choice([0.0, 0.5, 1.0], size=(nj, 1)) + 10.0 ** rng.uniform(-5, -1, (nj, 1)) * rng.choice([-1, 1], (nj, 1))
    near = Xi[k] + u * t / tf.KAPPA - e * np.minimum(D * (1.0 + rng.normal(size=(nj, 1)) * 1e-3), 0.5 * x)
    ok = (np.abs(near).max(1) <= x) & (np.arange(nj) % 3 > 0)
    Xj[ok] = near[ok]
    Xi, Xj, Vi, Vj = (a.astype(tf.F).astype(float) for a in (Xi, Xj, Vi, Vj))
    I, J = tf.record(Xi, Vi, hd2), tf.record(Xj, Vj, hd2)
    for rec in (I, J):
        for form in "pqr":
            assert (rec[form] > -K["kTileNever"] + 1000).all() and (rec[form] < -K["kTileWild"] - 1000).all()
    P, Q, R = tf.forms(I, J)
    assert all(np.isfinite(f).all() for f in (P, Q, R))
    passed = (P < 0) & (Q < 0) & (R < 0)
    r, w = Xi[:, None] - Xj[None], Vi[:, None] - Vj[None]
    s0, ww = (r * w).sum(2), (w * w).sum(2)
    d2 = ((r - w * (s0 / ww)[..., None]) ** 2).sum(2)
    cand = (s0 < 0) & (s0 + ww / tf.KAPPA > 0) & (d2 <= D * D)
    assert cand.sum() > 100
    lost = cand & ~passed
    assert not lost.any(), f"{lost.sum()} of {cand.sum()} candidates lost"
