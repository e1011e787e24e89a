"""The order in which a residual product adds up a row's squares for the norm behind it, which every bit of a check with norms inside the
products follows: 128 values are 32 chunks of 4, and chunk c's sum meets that of c ^ 16 first, then c ^ 8, 4, 2, 1.  Exchanging the
two sides of any of these additions changes no bit, so a stage whose columns are permuted that way, weights and all, has to give the
permuted output, bit for bit: its products have one term each, so nothing else depends on the order of the columns.  (Any other
order of the sums gives about half of the rows another last bit, and of the 17 million outputs behind them some dozens.)"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import stage_inputs as si


def _exchanged(rng, order=(1, 2, 4, 8, 16)):
    """The chunks 0 .. 31 with the sides of the additions exchanged at random; order: the bit at the root first."""
    if not order:
        return [0]
    bit, sides = order[0], [_exchanged(rng, order[1:]) for _ in range(2)]
    flip = rng.integers(2) * bit
    # the positions of either side hold the chunks of one of them
    at = lambda i, o: sum(b for j, b in enumerate(o) if i >> (len(o) - 1 - j) & 1)
    pos = [at(i, order[1:]) for i in range(len(sides[0]))]
    out = {}
    for s in range(2):
        for i, p in enumerate(pos):
            out[p | (bit * s)] = dict(zip(pos, sides[s]))[p] | (flip ^ (bit * s))
    return [out[at(i, order)] for i in range(2 * len(pos))]


def _column_order(D, rng):
    at = [sum(b for j, b in enumerate((1, 2, 4, 8, 16)) if i >> (4 - j) & 1) for i in range(32)]
    cols = np.empty(D, np.int64)
    for p in range(D // 128):
        for place, chunk in zip(at, _exchanged(rng)):
            cols[p * 128 + place * 4:][:4] = p * 128 + chunk * 4 + np.arange(4)
    return cols


def test_exchanging_the_sides_of_the_sums_changes_no_bit():
    import torch

    import paper_2603_03592_amd as sv
    D, M = 2048, 8192
    desc = si.StageDesc(2, D, 16, 16, 2048, rope=False)
    if not sv.sv_gemm_plan(M, D, D, row_sums=True)[0]:
        pytest.skip("the sizes are chosen for 256 compute units")
    cols = torch.from_numpy(_column_order(D, np.random.default_rng(0))).cuda()
    assert sorted(cols.tolist()) == list(range(D)) and (cols != torch.arange(D, device="cuda")).sum() > D // 2
    h = torch.randn((M, 1, D), generator=torch.Generator(device="cuda").manual_seed(0), device="cuda").bfloat16()
    ver = sv.Verifier(desc, M, 1, fuse_norm=True)

    def run(cols):
        zero = torch.zeros((D, D), device="cuda", dtype=torch.bfloat16)
        one = torch.ones(D, device="cuda", dtype=torch.bfloat16)
        eye = torch.eye(D, device="cuda", dtype=torch.bfloat16)
        nothing = dict(wq=zero, wk=zero, wv=zero, wo=zero, w_gate=zero, w_up=zero, w_down=zero, norm1_g=one, norm2_g=one)
        # the second block's values are its rows times their factors; attention over one token returns them, the out-projection brings
        # them back, over the residual's bits
        blocks = [nothing, dict(nothing, wv=eye[:, cols].contiguous(), wo=(64 * eye)[cols].contiguous())]
        wc = ver.pack_weights(blocks)
        ver.prepare_weights(wc)
        x = h[..., cols].contiguous()
        out = ver.verify_forward(wc, x, x, want_h_hat=True)["h_hat"].reshape(M, D).clone()
        torch.cuda.synchronize()
        return out

    same = torch.arange(D, device="cuda")
    assert torch.equal(run(cols), run(same)[:, cols])
    ver.close()
