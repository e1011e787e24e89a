"""Backward products over several weight matrices whose parts of k are as short as one slice of 64 each: the slices at which a part ends stand
apart from the others in the k loop, here most or all of them, on tiles of 64x64 up to 256x256.  And activations on 192x256 tiles with fewer
slices than the tile has buffers."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import stage_inputs as si
from gpu_util import assert_close, dev, dev_weights, host
from oracle import stage_oracle as so


@pytest.mark.parametrize("D,heads,kv,F,B,S", [(64, 1, 1, 64, 3, 77), (128, 2, 1, 64, 3, 77), (192, 3, 1, 320, 5, 100), (128, 2, 2, 128, 40, 100), (256, 4, 1, 64, 40, 200),
                                              (512, 8, 1, 192, 16, 256), (1024, 16, 1, 64, 17, 256)])
@pytest.mark.parametrize("mlp", ["swiglu", "gelu"])
def test_gradients_through_short_segments(D, heads, kv, F, B, S, mlp):
    _against_the_oracle(D, heads, kv, F, B, S, mlp)


@pytest.mark.parametrize("D", [64, 128, 192, 256])
@pytest.mark.parametrize("mlp,F,B,S,tiles", [("gelu", 3072, 30, 100, (6, 6)), ("swiglu", 1024, 60, 100, (6, None)), ("swiglu", 1024, 120, 100, (None, 6))])
def test_activations_on_192x256_tiles_with_few_slices(D, mlp, F, B, S, tiles):
    import torch

    import paper_2603_03592_amd as sv
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are chosen for 256 compute units")
    for epilogue, tile in zip((mlp, mlp + "_bwd"), tiles):
        assert tile is None or sv.sv_gemm_tiles(B * S, F, D, epilogue, 0, 8 * 160 * 128 * 128)[0] == tile
    _against_the_oracle(D, D // 64, 1, F, B, S, mlp)


def _against_the_oracle(D, heads, kv, F, B, S, mlp):
    import paper_2603_03592_amd as sv
    desc = si.StageDesc(1, D, heads, kv, F, mlp=mlp)
    w = si.make_weights(desc, 4)
    h, g = si.make_activations(desc, B, S, 4), si.make_output_grad(desc, B, S, 4)
    ver = sv.Verifier(desc, B * S, S, backward=True)
    wc = ver.pack_weights(wd := dev_weights(w, "bf16"))
    o = ver.verify_backward(wc, dev(h, "bf16"), dev(g, "bf16"), want_g_hat=True, want_h_hat=True)
    got_h, got_g = host(o["h_hat"]), host(o["g_hat"])
    ver.close()
    for b in sorted({0, B // 2, B - 1}):                   # the stage acts on every sequence on its own
        want_h, want_g = so.stage_backward(h[b:b + 1], g[b:b + 1], w, desc)
        assert_close(got_h[b], want_h[0], 2e-2, (D, F, b, "h"))
        assert_close(got_g[b], want_g[0], 2e-2, (D, F, b, "g"))
    assert np.isfinite(got_g).all()
