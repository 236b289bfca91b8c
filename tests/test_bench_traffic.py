"""bench.py quotes a committed HBM traffic figure only for the search it was counted on."""
import pytest

import bench

TAKEN = dict(shape=(2, 64), order=16, cbins=(4, 5, 6))


@pytest.mark.parametrize("other", [{}, {"order": 0}, {"shape": (1, 64)}, {"order": 1}, {"cbins": (4, 5, 7)}])
def test_traffic_belongs_to_the_search_run(tmp_path, monkeypatch, other):
    (tmp_path / "profiles").mkdir()
    (tmp_path / "profiles" / "search_w_fp32_traffic.txt").write_text(
        "hbm_bytes_per_launch: 2.5e+09\nhbm_bytes_per_launch_order_0: 7e+08\nsearch_order: 16\n"
        "search_shape: 2,64\nsearch_cbins: 4,5,6\nkernel_code_sha256: abc\n")
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    monkeypatch.setattr(bench, "kernel_code_sha256", lambda path: "abc")
    got = bench.read_traffic("w", "fp32", **{**TAKEN, **other})
    assert got == (2.5e9 if not other else 7e8 if other == {"order": 0} else None)
