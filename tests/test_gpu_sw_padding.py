"""The projections sv_sw_against_projection hands out: the first T entries of a row are the projections, the rest infinities, for
tokens that end in every part of a tile and rows with and without padding."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import stage_inputs as si
from gpu_util import dev


@pytest.mark.parametrize("T,L", [(1, 32), (127, 64), (128, 64), (129, 32), (300, 64), (300, 128), (1025, 96), (2100, 64)])
def test_rows_end_in_infinities(T, L):
    import paper_2603_03592_amd as sv
    n, D = 3, 192
    ver = sv.Verifier(si.TINY.desc, T, 64, sliced_w=True)
    g = torch.Generator(device="cuda").manual_seed(T + L)
    x = torch.randn((n, T, D), generator=g, device="cuda").to(torch.bfloat16)
    u = dev(si.make_directions(D, L, 0), "bf16")
    Tpad = int(sv.binding.lib.sv_sw_row_len(T))
    ref = torch.zeros((L, Tpad), device="cuda")
    _, proj = ver.sw_against_projection(x, ref, u, 1.0)
    want = torch.matmul(u.double(), x.double().transpose(1, 2).contiguous())
    assert proj.shape[-1] == Tpad
    # exact products of bf16, at most 192 of them added in fp32
    assert (proj[..., :T].double() - want).abs().max() <= 1e-5 * want.abs().max()
    assert torch.isinf(proj[..., T:]).all() and (proj[..., T:] > 0).all()
    ver.close()
