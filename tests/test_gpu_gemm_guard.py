"""What a product leaves alone: the rows behind its last and the columns between its rows, on every tile.  Row counts that end inside a
tile, inside its first rows (all later row blocks of the tile lie past the end of C) and on its edge; row strides that are an odd multiple
of 8 bytes, so that 16-byte accesses stand on 8-byte boundaries."""
import ctypes

import pytest

import paper_2603_03592_amd as sv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [0, 1, 2, 3, 4], ids=["auto", "256x256", "128x128", "256x128", "64x128"])
@pytest.mark.parametrize("M,gap", [(1, 0), (5, 4), (130, 4), (256, 4), (300, 0), (511, 4), (4097, 0), (4160, 4)])
def test_rows_behind_the_last_and_columns_between_rows_stay(M, gap, tile):
    import torch
    N, K = 512, 192
    gen = torch.Generator(device="cuda").manual_seed(M)
    A, B = (torch.randn((r, K), generator=gen, device="cuda").bfloat16() for r in (M, N))
    C = torch.full((M + 256, N + gap), 7.0, device="cuda", dtype=torch.bfloat16)
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    assert sv.lib.sv_gemm_bf16(p(A), K, p(B), K, 0, p(C), N + gap, M, N, K, tile, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    assert (C[M:] == 7.0).all() and (C[:, N:] == 7.0).all()
    ref = A.float() @ B.float().t()
    bound = 2.0 ** -8 * ref.abs() + K * 2.0 ** -24 * (A.float().abs() @ B.float().abs().t())       # one rounding to bf16, K steps of fp32
    assert ((C[:M, :N].float() - ref).abs() <= bound).all()


@pytest.mark.parametrize("mlp,B,S", [("swiglu", 11, 1500), ("gelu", 11, 1500), ("gelu", 3, 777)])
def test_rows_behind_a_stage_output_stay(mlp, B, S):
    """The residual products of the last block write the recomputed output, the backward pass' last norm the gradient."""
    import torch

    import stage_inputs as si
    from gpu_util import dev_weights
    desc = si.StageDesc(1, 1024, 16, 16, 1024, mlp=mlp)
    ver = sv.Verifier(desc, B * S, S, backward=True)
    wc = ver.pack_weights(wd := dev_weights(si.make_weights(desc, 3), "bf16"))
    gen = torch.Generator(device="cuda").manual_seed(S)
    h, g = (torch.randn((B, S, 1024), generator=gen, device="cuda").bfloat16() for _ in range(2))
    outs = [torch.full((B * S + 256, 1024), 7.0, device="cuda", dtype=torch.bfloat16) for _ in range(2)]
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    assert sv.lib.sv_verify_backward(ver._ctx, wc, p(h), p(g), B, S, None, 1, (ctypes.c_float * 4)(), 0, p(outs[0]), p(outs[1]), None, None,
                                     ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    for o in outs:
        assert (o[B * S:] == 7.0).all() and not (o[:B * S] == 7.0).all()
    ver.close()
