"""Norms inside the products where the product that leaves the row sums would be cheaper over runs of k: two blocks, so that the
second block's first norm takes its sums from the first block's down-projection."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import stage_inputs as si
from gpu_util import assert_close, dev, dev_weights, host
from oracle import stage_oracle as so


@pytest.mark.parametrize("D,heads,kv,F,B,S", [(2048, 16, 16, 10240, 18, 256), (4096, 32, 8, 14336, 9, 256)], ids=["2048x10240", "4096x14336"])
def test_second_block_scales_its_rows_by_their_own_sums(D, heads, kv, F, B, S):
    import paper_2603_03592_amd as sv
    desc = si.StageDesc(2, D, heads, kv, F)
    w = si.make_weights(desc, 9)
    h = si.make_activations(desc, B, S, seed=9)
    ver = sv.Verifier(desc, B * S, S, fuse_norm=True)
    wc = ver.pack_weights(wd := dev_weights(w, "bf16"))
    ver.prepare_weights(wc)
    got = host(ver.verify_forward(wc, dev(h, "bf16"), want_h_hat=True)["h_hat"])
    ver.close()
    for b in (0, B - 1):                                   # the stage acts on every sequence on its own
        assert_close(got[b], so.stage_forward(h[b:b + 1], w, desc)[0], 2e-2, (D, F, b))
    plain = sv.Verifier(desc, B * S, S)
    all_rows = host(plain.verify_forward(plain.pack_weights(wd), dev(h, "bf16"), want_h_hat=True)["h_hat"])
    plain.close()
    assert_close(got, all_rows, 2e-2, (D, F, "norm as a pass of its own"))
