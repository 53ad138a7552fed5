"""Epilogues of the persistent kernel and of those with asynchronous copies whose arguments make them an instance of their own, as stages pass them (bias alone, ReLU, GELU and its derivative, a
residual source; masks of both activations), on tiles that the output's last rows and columns leave partly empty, in both tile sizes, over
as few k-tiles as the kernel takes; beside them combinations that keep the general epilogue.  Against the oracle.  (Every combination of arguments, over
several units of a workgroup: tests/test_gpu_epilogue_arguments.py.)"""
import pytest

from tests import routes
from tests.test_gpu_stage import run_stage_case
from workloads.configs import layernorm, linear, softmax_ce

WIDE = 12400   # rows of 49 tiles of 256, the last one with 112; 1000 columns are 4 tiles, the last one with 232
CASES = [
    # (layers, rows)
    ([linear(128, 1000, False), linear(1000, 128, False)], WIDE),
    ([linear(128, 1000, True), linear(1000, 128, False)], WIDE),
    ([linear(192, 1000, False, act="gelu"), linear(1000, 192, False)], WIDE),
    ([layernorm(1000, 1), linear(1000, 128, False), linear(128, 1000, False, skip=2), linear(1000, 128, False)], WIDE),   # a residual source; its gradient is added to
    ([linear(128, 1000, True)], WIDE),                                                               # the result twice: general
    ([linear(128, 1000, False), softmax_ce(1000)], WIDE),                                            # fp32 results
    ([linear(1024, 1024, True), linear(1024, 1024, False)], 4200),                                   # 256 x 128 tiles
    ([layernorm(1024, 1), linear(1024, 1024, False, act="gelu"), linear(1024, 1024, False, skip=2), linear(1024, 1024, False)], 4200),
    ([linear(776, 2952, True), linear(2952, 776, False)], 1000),                                     # 128 x 128 tiles; 64 x 64 shared by k
    ([layernorm(776, 1), linear(776, 2952, False, act="gelu"), linear(2952, 776, False, skip=2), linear(776, 64, False)], 1000),
    ([linear(2056, 712, True), linear(712, 64, False)], 760),
]


KERNELS = {WIDE: "persistent", 4200: "persistent narrow", 1000: "async", 760: "by_k"}


MASKS = [   # the kernel of the input gradient of each dense layer that reads another's result
    ["persistent"], ["persistent"], ["persistent"], ["persistent", "tiled", "persistent"], [], [], ["persistent narrow"], ["persistent narrow"] * 3,
    ["async"], ["by_k", "async", "joint small"], ["joint small"]]


def test_cases_reach_their_kernels():
    for (layers, rows), masks in zip(CASES, MASKS):
        dense = [l for l in layers if l["kind"] == "linear"]
        assert routes.dense_routes(max(dense, key=lambda l: l["dout"]), "bf16", rows, 1)[0] == KERNELS[rows]
        assert [routes.dense_routes(l, "bf16", rows, 1)[1] for l in dense if l is not layers[0]] == masks


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(CASES)))
def test_forms(case):
    layers, rows = CASES[case]
    run_stage_case(layers, "bf16", rows, 1, seed=case)
