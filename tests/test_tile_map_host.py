"""tile_at() and tiles_of() of csrc/plan.h, the functions that the product kernels call themselves: every tile has one place, and what the helpers
of an XCD bring holds all of its tiles and no row or column of tiles that it has none in."""
import pytest

from host_cpp import compile_cpp, run

MAIN = r"""
#include <cstdio>
#include "plan.h"
using namespace ppll;
int main() {
  int M, N, edge, units;
  while (std::scanf("%d %d %d %d", &M, &N, &edge, &units) == 4) {
    const TileMap t = tile_map(M, N, edge, edge, units);
    for (int xcd = 0; xcd < 8; ++xcd) {
      const TileRange r = tiles_of(t, xcd);
      std::printf("range %d %d %d %d %d\n", xcd, r.m0, r.m1, r.n0, r.n1);
      for (int slot = 0; slot < t.per_xcd + 8; ++slot) {
        int tm = -1, tn = -1;
        if (tile_at(t, xcd, slot, tm, tn)) std::printf("tile %d %d %d\n", xcd, tm, tn);
      }
    }
  }
}
"""


@pytest.fixture(scope="module")
def tiles(tmp_path_factory):
    exe = compile_cpp(str(tmp_path_factory.mktemp("tiles")), MAIN)
    return lambda *a: [l.split() for l in run(exe, " ".join(map(str, a))).splitlines()]


# few rows and many columns of tiles, the other way round, a remainder on either side, fewer tiles than XCDs, one, blocks and stretches
@pytest.mark.parametrize("units", [256, 64])
@pytest.mark.parametrize("M,N,edge", [(640, 768, 64), (2688, 384, 64), (5440, 192, 64), (64, 64, 64), (1105, 768, 64), (1, 2304, 64), (65, 960, 64),
                                      (256, 3072, 64), (20, 768, 32), (200, 2304, 32), (256, 768, 32), (8320, 384, 128), (10500, 384, 128),
                                      (4160, 768, 128), (129, 5000, 128), (321, 64, 64)])
def test_tiles_and_helpers_of_an_xcd(tiles, M, N, edge, units):
    made = tiles(M, N, edge, units)
    placed = [tuple(map(int, l[1:])) for l in made if l[0] == "tile"]
    rows, columns = -(-M // edge), -(-N // edge)
    assert sorted(p[1:] for p in placed) == [(m, n) for m in range(rows) for n in range(columns)]
    for xcd, m0, m1, n0, n1 in (map(int, l[1:]) for l in made if l[0] == "range"):
        here = [p[1:] for p in placed if p[0] == xcd]
        if here:
            assert (m0, m1) == (min(m for m, _ in here), max(m for m, _ in here) + 1) or (m0, m1) == (0, rows)
            assert (n0, n1) == (min(n for _, n in here), max(n for _, n in here) + 1) or (n0, n1) == (0, columns)
            assert 0 <= m0 and m1 <= rows and 0 <= n0 and n1 <= columns
            assert all(m0 <= m < m1 and n0 <= n < n1 for m, n in here)
        else:
            assert m0 >= m1 or n0 >= n1
