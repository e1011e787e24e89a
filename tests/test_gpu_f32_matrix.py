"""fp32 stages on the matrix cores at the edges of their tiles: rows, columns, keys and k that end inside a 16-wide block, both
tile sizes, and an infinite value behind the causal mask."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import stage_inputs as si
from gpu_util import assert_close, dev, dev_weights, host
from test_gpu_stage import run_stage

CASES = {
    "one_token": (si.StageDesc(1, 32, 2, 1, 40, dtype="f32"), 1, 1),
    "hd16_gqa_tails": (si.StageDesc(2, 64, 4, 2, 104, dtype="f32"), 1, 17),
    "hd32_bidir": (si.StageDesc(1, 96, 3, 1, 136, causal=False, dtype="f32"), 3, 33),
    "hd64_gelu_ln": (si.StageDesc(1, 128, 2, 2, 264, mlp="gelu", norm="ln", rope=False, dtype="f32"), 2, 65),
    "hd128": (si.StageDesc(1, 256, 2, 1, 200, dtype="f32"), 1, 79),
    "wide_tiles": (si.StageDesc(1, 512, 8, 4, 1048, dtype="f32"), 2, 257),
}


@pytest.mark.parametrize("case", list(CASES))
def test_fp32_stage_at_the_edges_of_the_tiles(case):
    desc, B, S = CASES[case]
    (gh, gg), (wh, wg), _ = run_stage(desc, B, S, seed=31, backward=True, weight_scale=2.0, grad_std=1.0)
    # fp32 sums of up to 1048 products, three deep: a few 2^-24 sqrt(1048) of the row, well inside 1e-5
    assert_close(gh, wh, 1e-5, "h")
    assert_close(gg, wg, 1e-5, "g")


def test_what_a_causal_mask_hides_stays_hidden():
    """A value that is infinite or NaN at one token must not reach earlier tokens, also not through a product with a probability of
    zero."""
    import paper_2603_03592_amd as sv
    desc, S, at = si.StageDesc(1, 64, 2, 1, 96, dtype="f32"), 45, 21
    w = dev_weights(si.make_weights(desc, 5), "f32")
    h = si.make_activations(desc, 1, S, 5)
    ver = sv.Verifier(desc, S, S)
    wc = ver.pack_weights(w)
    clean = host(ver.verify_forward(wc, dev(h, "f32"), want_h_hat=True)["h_hat"])
    for bad in (np.inf, -np.inf, np.nan):
        hb = h.copy()
        hb[0, at, 3] = bad
        got = host(ver.verify_forward(wc, dev(hb, "f32"), want_h_hat=True)["h_hat"])
        np.testing.assert_allclose(got[0, :at], clean[0, :at], rtol=1e-5, atol=1e-6)     # the block is added in another order
        assert np.isnan(got[0, at:]).all()
    ver.close()
