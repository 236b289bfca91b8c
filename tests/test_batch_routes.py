"""Which search the instances of a batch take together, from the costs of each:
the rule is taken from the host source and built alone."""
import os
import shutil
import subprocess

import pytest

HOST = os.path.join(os.path.dirname(__file__), "..", "paper_1210_8084_amd", "csrc", "tpkmc_host.hip")
CXX = shutil.which("g++") or shutil.which("clang++")

SHELL = """
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
%s
int main() {
    Routes r;
    double tile, tile_wave, lane, lane_wave;
    int open, tiles;
    long count, all;
    while (std::scanf("%%lf %%lf %%lf %%lf %%d %%d %%ld %%ld", &tile, &tile_wave, &lane, &lane_wave, &open, &tiles, &count,
                      &all) == 8)
        r.add(SearchCost{tile, tile_wave, lane, lane_wave, open != 0, tiles != 0}, count, all);
    std::printf("%%d %%g", (int)r.any, r.any ? r.cap() : HUGE_VAL);
}
"""
TUBE = (9000.0, 580.0, 6600.0, 3300.0, 1, 0)   # dense and thin: lanes, were all the records of its kind
DENSE = (1070.0, 80.0, 694.0, 347.0, 1, 0)     # 404 per c-bin
THIN = (1000.0, 80.0, 300.0, 150.0, 1, 0)      # the same, far less dense
BOX = (400.0, 50.0, 600.0, 300.0, 0, 1)        # sort cells: tiles
SPARSE = (0.0, 0.0, 0.0, 0.0, 0, 0)            # FP32 below the density of tiles: staged


def route(tmp_path, batch):
    text = open(HOST).read()
    a, b = text.index("struct SearchCost {"), text.index("template <typename real>\nSearchCost search_cost")
    c, d = text.index("constexpr double kBatchGain"), text.index("struct Routes {")
    rule = text[a:b] + text[c:text.index("\n};\n", d) + 4]
    src = tmp_path / "routes.cpp"
    src.write_text(SHELL % rule)
    exe = str(tmp_path / "routes")
    subprocess.run([CXX, "-O1", "-std=c++17", str(src), "-o", exe], check=True)
    total = sum(n for _, n in batch)
    lines = "\n".join(" ".join(map(str, cost + (n, total))) for cost, n in batch)
    out = subprocess.run([exe], input=lines, capture_output=True, text=True, check=True).stdout.split()
    return bool(int(out[0])), float(out[1])


@pytest.mark.skipif(CXX is None, reason="no host compiler")
@pytest.mark.parametrize("batch,any_lane,lanes", [
    ([(BOX, 1_000_000), (SPARSE, 50_000)], False, []),
    ([(TUBE, 10_000)] * 100, True, [TUBE]),                          # all alike: a full launch of lanes
    ([(THIN, 10_000)] * 100 + [(SPARSE, 10_000)], True, [THIN]),
    # Its slowest wave by lanes 1980 us after the 360 of the box, by tiles 2700 beside them: within a quarter.
    ([(BOX, 900_000), (TUBE, 70_000)], True, []),
    ([(BOX, 900_000), (THIN, 600_000), (TUBE, 70_000)], True, []),
    # 208 us after the 360, by tiles 321 beside them; beside THIN's 180 us of lanes it makes them 208.
    ([(BOX, 900_000), (DENSE, 17_000)], True, []),
    ([(BOX, 900_000), (THIN, 600_000), (DENSE, 17_000)], True, [THIN]),
])
def test_few_lanes_beside_tiles_go_to_the_tiles(tmp_path, batch, any_lane, lanes):
    found, cap = route(tmp_path, batch)
    assert found == any_lane
    if found:
        assert [c for c in (TUBE, DENSE, THIN) if c[2] < cap and any(b[0] is c for b in batch)] == lanes
