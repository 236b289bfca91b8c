"""bench.py quotes a committed HBM traffic figure only for the search it was counted on."""
import pytest

import bench

TAKEN = dict(shape=(2, 64), order=16, cbins=(4, 5, 6))


@pytest.mark.parametrize("other", [{}, {"shape": (1, 64)}, {"order": 0}, {"cbins": (4, 5, 7)}])
def test_traffic_belongs_to_the_search_run(tmp_path, monkeypatch, other):
    (tmp_path / "profiles").mkdir()
    (tmp_path / "profiles" / "search_w_fp32_traffic.txt").write_text(
        "hbm_bytes_per_launch: 2.5e+09\nsearch_order: 16\nsearch_shape: 2,64\nsearch_cbins: 4,5,6\n"
        "kernel_code_sha256: abc\n")
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    monkeypatch.setattr(bench, "kernel_code_sha256", lambda path: "abc")
    got = bench.read_traffic("w", "fp32", **{**TAKEN, **other})
    assert got == (None if other else 2.5e9)
