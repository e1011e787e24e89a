"""Heads of 16 columns in the attention kernels, whose tile rows have room for 32: one key tile, ragged ones, tiles of queries singly and
in pairs, the query heads of a group in one workgroup and split, with and without rotation (undone in the backward kernels' outputs)."""
import pytest

pytestmark = pytest.mark.gpu

import stage_inputs as si
from gpu_util import assert_close
from test_gpu_stage import TOL, run_stage

SHAPES = {                                     # heads, kv heads, causal, rope, B, S
    "one_tile": (4, 4, True, True, 1, 64),
    "shorter_than_a_tile": (8, 2, True, True, 3, 17),
    "ragged": (8, 8, True, True, 2, 331),
    "ragged_no_rope": (4, 4, True, False, 2, 129),
    "bidir": (8, 4, False, True, 2, 200),
    "group_split": (16, 4, True, True, 1, 500),
    "group_together": (32, 16, True, True, 33, 130),
    "paired": (32, 8, True, True, 5, 390),
}


@pytest.mark.parametrize("case", list(SHAPES))
def test_heads_of_16(case):
    H, Hkv, causal, rope, B, S = SHAPES[case]
    desc = si.StageDesc(1, H * 16, H, Hkv, 128, causal=causal, rope=rope)
    (gh, gg), (wh, wg), _ = run_stage(desc, B, S, seed=41, backward=True, weight_scale=2.0)
    assert_close(gh, wh, TOL["bf16"], "h")
    assert_close(gg, wg, TOL["bf16"], "g")
