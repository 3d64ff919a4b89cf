"""What a call asks of the HIP runtime, and in which order: on the CPU, against a stand-in for the runtime (host_hip.py)."""
import pytest

from host_hip import calls, compile_runtime
from paper_2411_12780_amd import synth


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    exe = compile_runtime(str(tmp_path_factory.mktemp("runtime")))
    return lambda workloads, *what: calls(exe, workloads, *what)


def vit(dim, batch, tokens, precision=synth.BF16, **more):
    return synth.workload("vit_stage_act_bf16", tokens=tokens, dim=dim, heads=dim // 64, mlp_dim=4 * dim, batch=batch, precision=precision, **more)


@pytest.mark.parametrize("wl", [vit(768, 8, 65, depth=2, aux_depth=2), vit(768, 4, 5, depth=1, aux_depth=1), vit(384, 128, 65, depth=2, aux_depth=1),
                                vit(192, 128, 65, depth=2, aux_depth=2), vit(64, 4, 5, precision=synth.FP32, depth=2, aux_depth=1),
                                vit(384, 16, 65, depth=1, aux_depth=0)])
def test_a_block_publishes_its_output_behind_the_launch_that_stores_it(runtime, wl):
    # the next block of a pipeline waits for this record: no launch of the auxiliary layers may come before it
    (batch,) = runtime([wl, wl], "batch")
    (wait,) = [c for c in batch if c[0] == "wait"]
    at = batch.index(("record", 1, wait[2]))
    last = [c[5] for c in batch[:at] if c[0] == "launch"][-1]
    assert "gemm" in last, last


@pytest.mark.parametrize("wl,call", [(vit(192, 4, 5, depth=3, aux_depth=3), "batch"), (vit(384, 48, 5, depth=3, aux_depth=1), "batch"),
                                     (vit(768, 12, 17, depth=2, aux_depth=1), "batch"), (vit(384, 4, 5, depth=1, aux_depth=1), "step"),
                                     (vit(384, 4, 5, depth=1, aux_depth=1), "eval")])
def test_a_launch_asks_for_the_device_less_than_once(runtime, wl, call):
    # each query is host time that a batch of small blocks waits for
    (made,) = runtime([wl] * (3 if call == "batch" else 1), call)
    asked, launches = (sum(c[0] == kind for c in made) for kind in ("device", "launch"))
    assert asked < launches, (asked, launches)


@pytest.mark.parametrize("batch,workgroups", [
    # maps of 8 x 8 x 64 and, behind the auxiliary convolution, 4 x 4 x 64: of 256 threads with a piece of 8 channels each up to 160
    # workgroups of four pieces, with four beyond
    (24, [12, 48]), (320, [160, 640]), (322, [161, 161]), (1024, [512, 512]),
])
def test_an_evaluation_of_small_maps_keeps_the_units_busy(runtime, batch, workgroups):
    (made,) = runtime([synth.workload("resnet32_stage3_bf16", batch=batch)], "eval")
    grids = [c[2][0] for c in made if c[0] == "launch" and "bn_apply_bf16" in c[5]]
    assert [grids[-1], grids[0]] == workgroups


@pytest.mark.parametrize("evaluate", ["eval", "eval_noalloc"])
@pytest.mark.parametrize("wl", [vit(384, 70, 65, depth=1, aux_depth=1), vit(768, 8, 65, depth=2, aux_depth=1), vit(384, 40, 5, depth=1, aux_depth=2)])
def test_an_evaluation_is_the_same_whatever_trained_the_block(runtime, wl, evaluate):
    # a pipeline's blocks share the chip while it runs; a block that is evaluated has it to itself
    launches = lambda made: [c[2:] for c in made if c[0] == "launch"]
    _, behind_a_batch = runtime([wl, wl], "batch", evaluate)
    fresh, _, behind_a_step = runtime([wl], evaluate, "step", evaluate)
    assert launches(behind_a_batch) == launches(fresh) == launches(behind_a_step)


@pytest.mark.parametrize("dim,batch,alone,shared", [
    # rows of 65 tokens: at width 384 a LayerNorm is behind in the product's launch where that product alone has 128 x 128 tiles with copying
    # waves, up to 10880 rows, and those are for launches that share the device with none
    (384, 128, False, True), (384, 151, True, True), (384, 166, False, True), (384, 170, True, True), (384, 100, False, False),
    (192, 128, True, True), (192, 32, False, False),
])
def test_which_products_take_the_layernorm_behind_them(runtime, dim, batch, alone, shared):
    wl = vit(dim, batch, 65, depth=2, aux_depth=1)
    takes = lambda made: any(c[0] == "launch" and "gemm_norm" in c[5] for c in made)
    assert [takes(made) for made in runtime([wl], "step", "eval")] == [alone, alone]
    batch_made, eval_made = runtime([wl, wl], "batch", "eval")
    assert (takes(batch_made), takes(eval_made)) == (shared, alone)


@pytest.mark.parametrize("stage,batch,blocks", [(1, 64, 4), (1, 200, 8), (3, 64, 1), (1, 200, 1), (2, 48, 1)])
def test_a_resnet_call_asks_for_the_device_less_than_once_a_launch(runtime, stage, batch, blocks):
    wls = synth.resnet32_modules(blocks, batch=batch) if blocks > 1 else [synth.workload("resnet32_stage%d_bf16" % stage, batch=batch)]
    for made in runtime(wls, "batch" if blocks > 1 else "step", "eval"):
        asked, launches = (sum(c[0] == kind for c in made) for kind in ("device", "launch"))
        assert asked < launches, (asked, launches)
