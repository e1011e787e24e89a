"""Attention over its launch shapes: numbers of (sequence, kv head) pairs on either side of a multiple of eight, tiles taken singly
and in pairs, the group of query heads in one workgroup and split, sequences of one key tile up to several, with a ragged last one."""
import pytest

pytestmark = pytest.mark.gpu

import stage_inputs as si
from gpu_util import assert_close
from test_gpu_stage import TOL, run_stage

SHAPES = {                                     # heads, kv heads, head_dim, causal, B, S
    "one_pair_one_tile": (1, 1, 64, True, 1, 64),
    "one_pair_ragged": (2, 1, 64, True, 1, 65),
    "three_pairs": (6, 3, 64, True, 1, 257),
    "nine_pairs": (6, 3, 64, True, 3, 321),
    "ten_pairs_bidir": (4, 2, 64, False, 5, 200),
    "seven_heads_128": (7, 1, 128, True, 2, 449),
    "four_kv_128_long": (4, 2, 128, True, 1, 1100),
    "bidir_128": (2, 2, 128, False, 3, 700),
    "hd32": (8, 4, 32, True, 3, 390),
    "hd32_bidir": (4, 2, 32, False, 1, 513),
    "many_heads_paired": (8, 8, 32, True, 16, 300),
    "many_heads_paired_128": (4, 4, 128, True, 33, 260),
}


@pytest.mark.parametrize("case", list(SHAPES))
def test_attention_launch_shapes(case):
    H, Hkv, hd, causal, B, S = SHAPES[case]
    desc = si.StageDesc(1, H * hd, H, Hkv, 128, causal=causal)
    (gh, gg), (wh, wg), _ = run_stage(desc, B, S, seed=31, backward=True, weight_scale=2.0)
    assert_close(gh, wh, TOL["bf16"], "h")
    assert_close(gg, wg, TOL["bf16"], "g")
