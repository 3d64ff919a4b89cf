"""The rules of the dispatch (csrc/plan.h) at 256 compute units, compiled for the CPU: which kernel a shape goes to and how its
work is cut."""
import pytest

from host_cpp import compile_cpp, run

UNITS = 256

MAIN = r"""
#include <cstdio>
#include <cstring>
#include <vector>
#include "plan.h"
using namespace ppll;
int main() {
  char what[32];
  while (std::scanf("%31s", what) == 1) {
    if (!std::strcmp(what, "wgrad")) {
      int units, workspace, n;
      if (std::scanf("%d %d %d", &units, &workspace, &n) != 3) return 1;
      std::vector<ProductShape> p(n);
      for (ProductShape& q : p) if (std::scanf("%d %d %d", &q.M, &q.N, &q.K) != 3) return 1;
      const WeightGradPlan w = plan_weight_grads(p.data(), n, workspace, true, units);
      std::printf("%d %d %d %d %d %d\n", w.wide, w.cuts, w.long_tiles, w.whole_tiles, w.tiles, w.long_steps);
    } else if (!std::strcmp(what, "big")) {
      int units, n;
      if (std::scanf("%d %d", &units, &n) != 2) return 1;
      std::vector<ProductShape> p(n);
      for (ProductShape& q : p) if (std::scanf("%d %d %d", &q.M, &q.N, &q.K) != 3) return 1;
      const BigGradPlan b = big_grad_tiles(p.data(), n, units);
      std::printf("%d %d %d %d %d %d\n", b.take, b.cuts, b.long_tiles, b.whole_tiles, b.tiles, b.long_steps);
    } else if (!std::strcmp(what, "product")) {
      int M, N, K, end, units;
      if (std::scanf("%d %d %d %d %d", &M, &N, &K, &end, &units) != 5) return 1;
      std::printf("%d\n", 32 * wide_tile_rows(M, N, K, (ProductEnd)end, units));
    } else if (!std::strcmp(what, "unit")) {
      int M, N, K, end, units;
      if (std::scanf("%d %d %d %d %d", &M, &N, &K, &end, &units) != 5) return 1;
      std::printf("%d\n", 32 * unit_tile_rows(M, N, K, (ProductEnd)end, wide_tile_rows(M, N, K, (ProductEnd)end, units), units));
    } else if (!std::strcmp(what, "few")) {
      int M, N, K, units;
      if (std::scanf("%d %d %d %d", &M, &N, &K, &units) != 4) return 1;
      std::printf("%d\n", few_tiles(M, N, K, units) ? few_tiles_wide(M, N, units) ? 64 : 32 : 0);
    } else if (!std::strcmp(what, "split")) {
      int M, N, K, units;
      if (std::scanf("%d %d %d %d", &M, &N, &K, &units) != 4) return 1;
      std::printf("%d\n", split_tiles(M, N, K, units));
    } else if (!std::strcmp(what, "attention")) {
      int T, H, dh, bwd, units;
      long heads;
      if (std::scanf("%d %d %d %d %ld %d", &T, &H, &dh, &bwd, &heads, &units) != 6) return 1;
      std::printf("%d\n", att_by_rows(T, H, dh, bwd, heads, units));
    } else if (!std::strcmp(what, "offsets")) {
      int T, H;
      if (std::scanf("%d %d", &T, &H) != 2) return 1;
      std::printf("%d\n", att_offsets_fit(T, H));
    } else {
      return 2;
    }
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    exe = compile_cpp(str(tmp_path_factory.mktemp("plan")), MAIN)
    return lambda *words: [int(v) for v in run(exe, " ".join(map(str, words))).split()]


def block_products(batch, tokens, dim, layers, pruned, mlp=None):
    """(M, N, K) of the weight gradients of a ViT block: `layers` whole encoder layers and, if `pruned`, the class-token one."""
    F, rows, out = mlp or 4 * dim, batch * tokens, []
    for _ in range(layers):
        out += [(F, dim, rows), (dim, F, rows), (dim, dim, rows), (dim, 3 * dim, rows)]
    if pruned:
        out += [(F, dim, batch), (dim, F, batch), (dim, dim, batch), (dim, 2 * dim, rows), (dim, dim, batch)]
    return out


def weight_grad_plan(plan, products, workspace=1, units=UNITS):
    names = ("wide", "cuts", "long_tiles", "whole_tiles", "tiles", "long_steps")
    return dict(zip(names, plan("wgrad", units, workspace, len(products), *(v for p in products for v in p))))


@pytest.mark.parametrize("batch", [128, 448, 449, 512, 1024, 4096])
def test_reductions_over_images_are_short_beside_those_over_all_tokens(plan, batch):
    # width 384, one whole and one class-token layer: 126 tiles over batch x 65 rows; the class-token layer's others, over the
    # images alone, are whole at the end and leave the long ones their parts
    w = weight_grad_plan(plan, block_products(batch, 65, 384, 1, True))
    assert (w["wide"], w["tiles"], w["long_tiles"], w["whole_tiles"]) == (0, 126 + 90, 126, 0)
    assert w["cuts"] == 2


def test_every_tile_is_planned_once_and_the_parts_fit_the_workspace(plan):
    for batch in (1, 3, 24, 128, 700):
        for tokens in (2, 5, 65, 197):
            for dim in (64, 192, 384, 768):
                for layers, pruned in ((1, False), (3, True), (8, True)):
                    products = block_products(batch, tokens, dim, layers, pruned)
                    tiles = sum(-(-m // 128) * -(-n // 128) for m, n, _ in products)
                    w = weight_grad_plan(plan, products)
                    steps = [-(-k // 64) for _, _, k in products]
                    assert w["tiles"] == tiles and 0 <= w["whole_tiles"] <= w["long_tiles"] <= tiles
                    assert w["cuts"] >= 1
                    if w["cuts"] > 1:
                        assert not w["wide"]
                        assert (w["long_tiles"] - w["whole_tiles"]) * w["cuts"] <= 2 * UNITS
                        assert min(s for s in steps if s >= w["long_steps"]) // w["cuts"] >= (8 if w["cuts"] > 8 else 4)


def big_grad_plan(plan, products, units=UNITS):
    names = ("take", "cuts", "long_tiles", "whole_tiles", "tiles", "long_steps")
    return dict(zip(names, plan("big", units, len(products), *(v for p in products for v in p))))


@pytest.mark.parametrize("rows,dim,layers,pruned,take", [
    # where they were measured to be ahead, and where not
    (8320, 384, 3, True, 1), (9280, 384, 3, True, 1), (16640, 384, 3, True, 1), (5200, 384, 4, True, 1), (4160, 384, 3, True, 0),
    (2080, 384, 3, True, 0), (1040, 768, 2, True, 1), (6304, 768, 1, True, 1), (640, 768, 3, True, 0), (25216, 192, 3, True, 1),
])
def test_weight_gradients_go_to_big_tiles_where_those_are_ahead(plan, rows, dim, layers, pruned, take):
    assert big_grad_plan(plan, block_products(rows // 5, 5, dim, layers, pruned))["take"] == take


def test_products_of_the_step_cases_go_where_they_say(plan):
    # tests/test_gpu_parity.py, test_weight_gradients_on_*: 21 x 197 rows of width 768 on big tiles; 64 x 65 rows of width 576 not, with
    # enough 128 x 128 tiles a layer for the side stream
    assert big_grad_plan(plan, block_products(21, 197, 768, 1, True))["take"] == 1
    narrow = block_products(64, 65, 576, 1, True)
    assert big_grad_plan(plan, narrow)["take"] == 0
    assert sum(-(-m // 128) * -(-n // 128) for m, n, _ in narrow[4:]) >= 256


def test_every_big_tile_is_planned_once_and_the_parts_fill_a_round_at_most(plan):
    for rows in (5, 325, 1040, 8320, 25216, 130000):
        for dim in (64, 192, 200, 384, 768, 1024):
            for layers, pruned in ((1, False), (3, True), (7, True)):
                products = block_products(rows // 5, 5, dim, layers, pruned)
                b = big_grad_plan(plan, products)
                assert b["tiles"] == sum(-(-m // 384) * -(-n // 192) for m, n, _ in products)
                assert 0 <= b["whole_tiles"] <= b["long_tiles"] <= b["tiles"] and b["cuts"] >= 1
                rest = b["long_tiles"] - b["whole_tiles"]
                assert rest * b["cuts"] <= UNITS and (rest > 0) == (b["cuts"] > 1)
                if b["cuts"] > 1:      # none of the divided reductions is left with less than two steps of 64 a part
                    assert min(-(-k // 64) for m, n, k in products if -(-k // 64) >= b["long_steps"]) // b["cuts"] >= 2
    assert big_grad_plan(plan, block_products(100, 65, 384, 10, True))["take"] == 0       # more products than a launch takes


@pytest.mark.parametrize("rows,cuts", [(8320, 16), (131072, 36), (262144, 36), (1048576, 36)])
def test_few_tiles_over_many_rows_are_cut_into_a_part_per_unit(plan, rows, cuts):
    # one layer of width 64 has 7 tiles: 36 parts each fill 256 units; fewer where a part would have less than 8 steps
    w = weight_grad_plan(plan, block_products(rows, 1, 64, 1, False))
    assert (w["tiles"], w["whole_tiles"], w["cuts"]) == (7, 0, cuts)


@pytest.mark.parametrize("tokens,head,bwd,few,many", [
    # at 128 heads and at 512 (batch x heads) the kernel that was measured to be the faster one: 1 rows, 0 heads
    (17, 16, 0, 1, 1), (65, 32, 1, 1, 1), (65, 96, 1, 1, 1), (65, 128, 0, 1, 1), (65, 128, 1, 1, 0), (130, 32, 1, 1, 1),
    (130, 96, 0, 1, 1), (130, 96, 1, 1, 1), (197, 16, 1, 1, 1), (197, 32, 0, 1, 1), (197, 32, 1, 1, 0), (256, 16, 0, 1, 1),
    (256, 32, 0, 1, 0), (256, 32, 1, 1, 0),
    # no room for the rows kernel
    (130, 128, 1, 0, 0), (197, 96, 0, 0, 0),
])
def test_attention_goes_to_the_kernel_that_is_ahead(plan, tokens, head, bwd, few, many):
    assert plan("attention", tokens, 4, head, bwd, 128, UNITS) == [few]
    assert plan("attention", tokens, 4, head, bwd, 512, UNITS) == [many]


PLAIN, BIAS, RESIDUAL, GELU, DGELU = range(5)


@pytest.mark.parametrize("M,N,K,end,rows", [
    # rows of the 256-wide tiles (0: the tiled kernel).  Last rounds well filled, long reductions:
    (25216, 768, 3072, RESIDUAL, 160), (25216, 2304, 768, BIAS, 160), (25216, 3072, 768, GELU, 160), (25216, 768, 768, RESIDUAL, 160),
    (8320, 1536, 384, GELU, 128), (12608, 1536, 384, GELU, 160), (10400, 1536, 512, BIAS, 128),
    # the gain does not make up for the change of kernels
    (8320, 384, 1536, RESIDUAL, 0), (8320, 1152, 384, BIAS, 0), (8320, 1536, 384, DGELU, 0), (18560, 1536, 384, GELU, 0), (25216, 1152, 384, BIAS, 0),
    # short reductions behind the derivative or a bias: measured 27 -> 38, 31 -> 40, 24 -> 32, 19 -> 25 us on the wide tiles
    (50432, 512, 128, DGELU, 0), (33280, 768, 192, DGELU, 0), (33280, 576, 192, BIAS, 0), (24960, 576, 192, BIAS, 0),
    # one column of wide tiles and a long reduction
    (33280, 256, 768, PLAIN, 0), (33280, 256, 1024, RESIDUAL, 0),
    # below the shortest loop of the wide tiles
    (25216, 768, 120, PLAIN, 0),
])
def test_products_go_to_the_tiles_that_are_ahead(plan, M, N, K, end, rows):
    assert plan("product", M, N, K, end, UNITS) == [rows]


@pytest.mark.parametrize("M,N,K,end,rows", [
    # rows of the tiles that have a unit to themselves (0: others are ahead), as measured on 256 units
    (25216, 768, 3072, BIAS, 320), (25216, 2304, 768, BIAS, 320), (25216, 3072, 768, GELU, 320), (8320, 1152, 384, BIAS, 256),
    (8320, 1536, 384, DGELU, 256), (8320, 384, 1536, BIAS, 0), (8320, 384, 384, BIAS, 0), (12608, 768, 3072, BIAS, 0),
    (6304, 768, 768, BIAS, 0), (25216, 3072, 120, BIAS, 0),
])
def test_products_go_to_tiles_of_a_unit_where_those_are_ahead(plan, M, N, K, end, rows):
    assert plan("unit", M, N, K, end, UNITS) == [rows]


def test_products_of_the_parity_cases_reach_the_kernels_they_name(plan):
    # tests/test_gpu_parity.py, test_vit_bf16_products_with_many_tiles: (batch, tokens, dim, mlp) and the products that have to
    # run on tiles of 128 and of 160 rows
    def kinds(batch, tokens, dim, mlp):
        rows = batch * tokens
        products = {"qkv": (3 * dim, dim, BIAS), "proj": (dim, dim, RESIDUAL), "fc1": (mlp, dim, GELU), "fc2": (dim, mlp, RESIDUAL),
                    "d fc2": (mlp, dim, DGELU), "d fc1": (dim, mlp, PLAIN), "d proj": (dim, dim, PLAIN), "d qkv": (dim, 3 * dim, PLAIN)}
        return {k: plan("product", rows, n, kk, e, UNITS)[0] for k, (n, kk, e) in products.items()}

    def on(rows, *case):
        return {k for k, v in kinds(*case).items() if v == rows}

    for case in ((129, 65, 128, 1528), (71, 131, 136, 3064)):
        assert not on(128, *case) and not on(160, *case)
    assert on(128, 129, 65, 328, 1528) == {"fc1"}
    assert on(160, 97, 129, 520, 1528) == {"fc1", "d fc2"}
    assert on(160, 97, 129, 768, 64) == {"qkv", "proj", "d proj", "d qkv"}
    assert on(128, 143, 130, 768, 64) == {"proj", "d proj", "d qkv"}


@pytest.mark.parametrize("M,N,K,columns", [
    # columns of a tile of the few-tile kernel (0: not its product)
    (1, 768, 3072, 32), (256, 3072, 768, 32), (257, 384, 1536, 32), (585, 384, 384, 32), (640, 384, 1536, 32), (683, 384, 384, 64),
    (585, 1152, 384, 0), (257, 1536, 384, 64), (640, 768, 3072, 0), (257, 768, 768, 0), (640, 768, 48, 64), (8320, 384, 384, 0),
])
def test_products_with_few_tiles(plan, M, N, K, columns):
    assert plan("few", M, N, K, UNITS) == [columns]


@pytest.mark.parametrize("M,N,K,taken", [
    # 64 x 64 tiles, one a unit at most, from K = 128
    (640, 768, 3072, 1), (640, 1600, 384, 1), (640, 1608, 384, 0), (2688, 384, 1536, 1), (2689, 384, 1536, 0), (1, 16384, 128, 1),
    (16384, 64, 128, 1), (16385, 64, 128, 0), (640, 768, 120, 0), (8320, 384, 1536, 0),
])
def test_products_with_a_tile_a_unit(plan, M, N, K, taken):
    assert plan("split", M, N, K, UNITS) == [taken]
    assert plan("split", M, N, K, 4) == [0]


@pytest.mark.parametrize("T,H,fit", [(1, 1, 1), (256, 1, 1), (197, 12, 1), (256, 21845, 1), (256, 21846, 0), (1, 5592405, 1), (1, 5592406, 0), (255, 2147483647, 0)])
def test_matrix_core_attention_within_its_32_bit_offsets(plan, T, H, fit):
    # T rows of 3 x 64 H bf16 values: 2^31 - 1 bytes at most
    assert plan("offsets", T, H) == [fit]
