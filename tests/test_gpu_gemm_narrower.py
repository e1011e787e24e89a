"""Products with an activation in the epilogue whose 256x256 tiles are less than one round of the compute units and whose 192x256 tiles are
one: 1537 rows are seven tiles of 256 or eight of 192 and one row, times 24 columns of tiles.  Forward with and without the stashes that the
backward needs, and the backward products' own epilogues, against the oracle."""
import pytest

pytestmark = pytest.mark.gpu

import stage_inputs as si
from gpu_util import assert_close
from test_gpu_stage import TOL, run_stage


@pytest.mark.parametrize("mlp,norm,ffn,backward", [("gelu", "ln", 6144, False), ("gelu", "rms", 6144, True), ("swiglu", "rms", 3072, False),
                                                  ("swiglu", "ln", 3072, True), ("swiglu", "rms", 6144, True)])
def test_activation_products_on_narrower_tiles(mlp, norm, ffn, backward):
    desc = si.StageDesc(1, 512, 8, 4, ffn, mlp=mlp, norm=norm)
    out = run_stage(desc, 29, 53, seed=43, backward=backward)
    (gh, gg), (wh, wg), _ = out
    assert_close(gh, wh, TOL["bf16"], "h")
    if backward:
        assert_close(gg, wg, TOL["bf16"], "g")
