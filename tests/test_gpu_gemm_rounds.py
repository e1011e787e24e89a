"""Products of more tiles than a round of the compute units takes: their last round in a second launch or in the persistent kernel, whose
stream of slices then runs on from tile to tile (as short as one slice a tile), two workgroups of 128x128 tiles on a compute unit, and activations
on 192x256 tiles in two rounds.  Every tile adds up an element in the same order, so all give the same bits; against fp32 the bound
is the rounding to bf16 and K steps of fp32."""
import ctypes

import pytest

import paper_2603_03592_amd as sv
from test_gpu_gemm_same_bits import Case, _whole_and_pieces, stage_plan

pytestmark = pytest.mark.gpu


def _product(A, B, tile, runs=1, ws=None, as_runs=False):
    import torch
    M, K, N = A.shape[0], A.shape[1], B.shape[0]
    C = torch.full((M + 1, N), 7.0, device="cuda", dtype=torch.bfloat16)          # the row behind the last stays as it is
    p, st = (lambda t: ctypes.c_void_p(t.data_ptr() if t is not None else 0)), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    if as_runs:
        r = sv.lib.sv_gemm_bf16_runs(p(A), K, p(B), K, p(C), N, M, N, K, tile, runs, p(ws), ws.numel() if ws is not None else 0, st)
    else:
        r = sv.lib.sv_gemm_bf16(p(A), K, p(B), K, 0, p(C), N, M, N, K, tile, st)
    assert r == 0
    assert (C[M] == 7.0).all()
    return C[:M]


def _operands(M, N, K):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    return tuple(torch.randn((r, K), generator=gen, device="cuda").bfloat16() for r in (M, N))


# 17 x 18 tiles of 256x256 (the last of them with 1, 64 or all rows), the second round in a launch of its own; 33 and more x 36 of 128x128
@pytest.mark.parametrize("M", [4097, 4160, 4352])
@pytest.mark.parametrize("K", [64, 128, 192, 320])
def test_tiles_agree_beyond_a_round(M, K):
    import torch
    A, B = _operands(M, 4608, K)
    want = _product(A, B, 5, as_runs=True)
    ref = A.float() @ B.float().t()
    bound = 2.0 ** -8 * ref.abs() + K * 2.0 ** -24 * (A.float().abs() @ B.float().abs().t())
    assert ((want.float() - ref).abs() <= bound).all()
    for tile in (1, 2, 3, 4):
        assert torch.equal(_product(A, B, tile), want), tile


# 24 x 18 tiles, 54 per XCD: 22 of its 32 workgroups run a second one (the last row of tiles with 1, 64 or all rows); 39 x 18: 24 a third
@pytest.mark.parametrize("M", [5889, 5952, 6144, 9984])
@pytest.mark.parametrize("K", [64, 128, 192, 320])
def test_a_workgroup_runs_on_to_its_next_tile(M, K):
    import torch
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are chosen for 256 compute units")
    assert sv.sv_gemm_tiles(M, 4608, K, "store")[2] == 0 and (M + 255) // 256 * 18 > 256
    A, B = _operands(M, 4608, K)
    want = _product(A, B, 2)
    for _ in range(3):
        assert torch.equal(_product(A, B, 1), want)


@pytest.mark.parametrize("mlp", ["swiglu", "gelu"])
def test_forward_without_stashes_runs_on_to_the_next_tile(mlp):
    """Without gate, up or the input of the activation to keep, a tile's epilogue makes the fewest stores."""
    import torch

    import stage_inputs as si
    from gpu_util import dev_weights
    from test_gpu_gemm_same_bits import STAGES
    c = STAGES[mlp + "_rounds"]
    gen = torch.Generator(device="cuda").manual_seed(5)
    h = torch.randn((c.batch, c.seq, c.d), generator=gen, device="cuda").bfloat16()
    ver = sv.Verifier(c.desc, c.batch * c.seq, c.seq)
    wc = ver.pack_weights(wd := dev_weights(si.make_weights(c.desc, 7), "bf16"))
    run = lambda x: ver.verify_forward(wc, x, x, want_h_hat=True)["h_hat"].clone()
    whole = run(h)
    assert torch.isfinite(whole).all() and torch.equal(whole, torch.cat([run(x[None].contiguous()) for x in h]))
    ver.close()


@pytest.mark.parametrize("M,N,K,runs", [(4099, 1152, 512, 3), (4099, 1152, 576, 8), (4099, 896, 512, 3)])
def test_settled_sums_with_two_workgroups_on_a_cu(M, N, K, runs):
    """297 tiles (two on a compute unit) and 231 (one each)."""
    import torch
    A, B = _operands(M, N, K)
    ws = torch.empty(runs * M * N, device="cuda")
    assert torch.equal(_product(A, B, 2, runs, ws, as_runs=True), _product(A, B, 2, runs, None, as_runs=True))


@pytest.mark.parametrize("mlp,batch,piece", [("swiglu", 8, 2), ("gelu", 16, 3)])
def test_activations_on_192x256_tiles_in_two_rounds(mlp, batch, piece):
    import torch

    import stage_inputs as si
    from gpu_util import dev_weights
    c = Case(mlp, 1024, 2816, batch, 512, piece, {})
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are chosen for 256 compute units")
    whole, part = stage_plan(c, batch), stage_plan(c, piece)
    assert whole["up"][0] == whole["dact"][0] == 6 and part["up"][0] != 6 and part["dact"][0] != 6
    assert all(runs == 1 for _, runs, _ in [*whole.values(), *part.values()])
    gen = torch.Generator(device="cuda").manual_seed(batch)
    h, g = (torch.randn((batch, c.seq, c.d), generator=gen, device="cuda").bfloat16() for _ in range(2))
    ver = sv.Verifier(c.desc, batch * c.seq, c.seq, backward=True)
    wc = ver.pack_weights(wd := dev_weights(si.make_weights(c.desc, 7), "bf16"))
    _whole_and_pieces(ver, wc, h, g, piece)
    ver.close()
