"""Rules of csrc/plan.h at 256 compute units, compiled for the CPU: products on tiles with copying waves, products that take the LayerNorm
behind them along, and which tiles go to which XCD."""
import pytest

from host_cpp import compile_cpp, run

MAIN = r"""
#include <cstdio>
#include "plan.h"
using namespace ppll;
int main(int n, char**) {
  int M, N, K, units;
  if (n > 1) {   // the map of 64 x 64 tiles: per_xcd, and XCD and place of every tile in order
    if (std::scanf("%d %d", &M, &N) != 2) return 1;
    const TileMap t = tile_map(M, N, 64, 64, 256);
    std::printf("%d %d %d %d %d %d\n", t.tiles_m, t.tiles_n, t.per_xcd, t.rows, t.cols, t.across);
    return 0;
  }
  while (std::scanf("%d %d %d %d", &M, &N, &K, &units) == 4) {
    const int tiles = (M + 127) / 128 * ((N + 127) / 128);
    std::printf("%d %d %d\n", copy_wave_tiles(M, N, K, units), helper_workgroups((tiles + 7) / 8, units), norm_tiles(M, N, K, units));
  }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    exe = compile_cpp(str(tmp_path_factory.mktemp("plan")), MAIN)
    return lambda *a: tuple(int(v) for v in run(exe, " ".join(map(str, a))).split())


@pytest.mark.parametrize("M,N,K,copying,helpers,norm", [
    (8320, 384, 1536, 1, 7, 0), (8320, 384, 384, 1, 7, 1), (5200, 384, 384, 0, 8, 0), (5400, 384, 384, 1, 8, 0), (640, 3072, 768, 0, 8, 0), (9850, 384, 1536, 0, 0, 0), (10500, 384, 1536, 1, 0, 0),
    (10880, 384, 384, 1, 0, 1), (10881, 384, 384, 0, 0, 1), (4160, 384, 384, 0, 8, 0), (4160, 384, 1152, 1, 8, 0), (8320, 384, 120, 0, 7, 1),
    (8320, 192, 768, 1, 8, 1), (4160, 192, 768, 0, 8, 0), (25216, 192, 576, 0, 0, 1), (16640, 384, 384, 0, 0, 0), (1300, 384, 384, 0, 8, 0),
])
def test_products_on_tiles_with_copying_waves(plan, M, N, K, copying, helpers, norm):
    assert plan(M, N, K, 256) == (copying, helpers, norm)
    assert plan(M, N, K, 4)[0] == plan(M, N, K, 4)[2] == 0          # too few units for any of it


@pytest.fixture(scope="module")
def tile_map(tmp_path_factory):
    exe = compile_cpp(str(tmp_path_factory.mktemp("map")), MAIN.replace("if (n > 1)", "if (n >= 1)"))
    return lambda *a: tuple(int(v) for v in run(exe, " ".join(map(str, a))).split())


@pytest.mark.parametrize("M,N", [(640, 768), (300, 768), (2688, 384), (5440, 192), (64, 64), (1105, 768), (1, 2304), (1000, 1000), (1024, 1024), (65, 15 * 64)])
def test_every_tile_of_a_launch_of_one_round_has_one_place(tile_map, M, N):
    tiles_m, tiles_n, per_xcd, rows, cols, across = tile_map(M, N)
    assert per_xcd <= 32
    seen = set()
    for xcd in range(8):
        for slot in range(per_xcd):
            if rows:
                tm, tn = xcd // across * rows + slot // cols, xcd % across * cols + slot % cols
            else:
                i = xcd * per_xcd + slot
                tm, tn = (i % tiles_m, i // tiles_m) if tiles_m < tiles_n else (i // tiles_n, i % tiles_n)
            if tm < tiles_m and tn < tiles_n:
                assert (tm, tn) not in seen
                seen.add((tm, tn))
    assert len(seen) == tiles_m * tiles_n


def test_blocks_of_tiles_where_they_share_more(tile_map):
    assert tile_map(640, 768)[2:] == (15, 5, 3, 4)
    assert tile_map(2688, 384)[3] == 0 and tile_map(64, 64)[3] == 0
