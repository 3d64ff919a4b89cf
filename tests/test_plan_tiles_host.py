"""Rules of csrc/plan.h at 256 compute units, compiled for the CPU: products on tiles with copying waves, and products that take the
LayerNorm behind them along."""
import pytest

from host_cpp import compile_cpp, run

MAIN = r"""
#include <cstdio>
#include "plan.h"
using namespace ppll;
int main() {
  int M, N, K, units;
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
    (8320, 384, 1536, 1, 7, 0), (8320, 384, 384, 1, 7, 1), (5200, 384, 384, 1, 8, 0), (9850, 384, 1536, 0, 0, 0), (10500, 384, 1536, 1, 0, 0),
    (10880, 384, 384, 1, 0, 1), (10881, 384, 384, 0, 0, 1), (4160, 384, 384, 0, 8, 0), (4160, 384, 1152, 1, 8, 0), (8320, 384, 120, 0, 7, 1),
    (8320, 192, 768, 1, 8, 1), (4160, 192, 768, 0, 8, 0), (25216, 192, 576, 0, 0, 1), (16640, 384, 384, 0, 0, 0), (1300, 384, 384, 0, 8, 0),
])
def test_products_on_tiles_with_copying_waves(plan, M, N, K, copying, helpers, norm):
    assert plan(M, N, K, 256) == (copying, helpers, norm)
    assert plan(M, N, K, 4)[0] == plan(M, N, K, 4)[2] == 0          # too few units for any of it
