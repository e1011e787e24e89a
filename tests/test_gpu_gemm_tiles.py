"""The direct-to-LDS products on smaller tiles: each tile alone at its edges (one row, one slice fewer and more than the stages it
keeps in flight, ragged rows), and through stages whose widths are multiples of 8 only or sit on either side of a choice of tile."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import stage_inputs as si
from gpu_util import assert_close, dev, host, rel_l2
from test_gpu_moe import run_constructed
from test_gpu_stage import run_stage


def assert_one_rounding(got, a, b):
    """bf16 keeps 8 significant bits (7 of them stored), so rounding moves a result by at most half of 2^-7 of itself; before it stands
    the fp32 sum, whose K additions are each off by at most 2^-24 of a partial sum <= sum |a b|, with 1 + 2^-8 for the rounding of that
    error."""
    a, b = a.astype(np.float64), b.astype(np.float64)
    want, K = a @ b.T, a.shape[1]
    bound = 2.0 ** -8 * np.abs(want) + (1 + 2.0 ** -8) * K * 2.0 ** -24 * (np.abs(a) @ np.abs(b).T)
    worst = np.abs(got - want) / bound
    assert worst.max() <= 1.0, (worst.max(), np.unravel_index(worst.argmax(), worst.shape))


@pytest.mark.parametrize("tile", [0, 2, 3, 4], ids=["auto", "128x128", "256x128", "64x128"])
@pytest.mark.parametrize("M,N,K", [(1, 128, 64), (63, 256, 128), (64, 256, 192), (129, 512, 256), (255, 256, 320), (257, 768, 576), (520, 256, 2304)])
def test_product_at_the_edges_of_the_tiles(tile, M, N, K):
    import paper_2603_03592_amd as sv
    if tile == 3 and N % 256:
        z = dev(np.zeros((128, 128), np.float32), "bf16")
        with pytest.raises(sv.SVError):
            sv.sv_gemm_bf16(z, z, tile=3)
        return
    g = np.random.default_rng(M * 7 + K)
    a = si.round_to_bf16(g.standard_normal((M, K)).astype(np.float32))
    b = si.round_to_bf16(g.standard_normal((N, K)).astype(np.float32))
    got = host(sv.sv_gemm_bf16(dev(a, "bf16"), dev(b, "bf16"), tile=tile))
    want = a.astype(np.float64) @ b.astype(np.float64).T
    assert_one_rounding(got, a, b)
    assert rel_l2(got, want) < 3e-3


RUN_SHAPES = [(1, 8, 64 * 5), (77, 136, 64 * 7), (128, 128, 64 * 8), (200, 72, 64 * 13), (257, 264, 64 * 17), (300, 520, 64 * 40)]


@pytest.mark.parametrize("M,N,K", RUN_SHAPES)
def test_runs_of_k_give_the_same_bits_on_every_tile(M, N, K):
    """Whole and over runs that do not divide the slices, rows and columns that end inside a tile: the partial products of every tile,
    added by the second launch, against the sums one workgroup makes of the same runs, and those against 64 bits."""
    import paper_2603_03592_amd as sv
    g = np.random.default_rng(M + N + K)
    a = si.round_to_bf16(g.standard_normal((M, K)).astype(np.float32))
    b = si.round_to_bf16(g.standard_normal((N, K)).astype(np.float32))
    ad, bd = dev(a, "bf16"), dev(b, "bf16")
    for runs in (1, 2, 3, 5, 8):
        if runs > K // 64:
            continue
        want = host(sv.sv_gemm_bf16_runs(ad, bd, 2, runs, apart=False))
        assert_one_rounding(want, a, b)
        for tile in (2, 3, 4, 5):
            assert np.array_equal(host(sv.sv_gemm_bf16_runs(ad, bd, tile, runs, apart=True)), want), (tile, runs)
            if runs == 1:
                assert np.array_equal(host(sv.sv_gemm_bf16_runs(ad, bd, tile, 1, apart=False)), want), tile
            else:
                assert tile == 2 or refused(sv, ad, bd, tile, runs)
    assert refused(sv, ad, bd, 2, K // 64 + 1) and refused(sv, ad, bd, 1, 1) and refused(sv, ad, bd, 6, 1)


def refused(sv, a, b, tile, runs):
    try:
        sv.sv_gemm_bf16_runs(a, b, tile, runs, apart=False)
    except sv.SVError:
        return True
    return False


def test_product_refuses_what_it_refused():
    import paper_2603_03592_amd as sv
    for n, k in ((64, 128), (192, 128), (128, 96), (128, 32)):
        with pytest.raises(sv.SVError):
            sv.sv_gemm_bf16(dev(np.zeros((130, k), np.float32), "bf16"), dev(np.zeros((n, k), np.float32), "bf16"))


@pytest.mark.parametrize("tile", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("far,ld", [("a", 1 << 23), ("b", 1 << 23), ("c", 1 << 22), ("c", 1 << 23)], ids=["a", "b", "c22", "c23"])
def test_rows_too_far_apart_for_32_bit_offsets(far, ld, tile):
    """Operands and results that are narrow views of very wide matrices."""
    import torch
    import paper_2603_03592_amd as sv
    M, N, K = 70, 256, 128
    g = np.random.default_rng(5)
    a = si.round_to_bf16(g.standard_normal((M, K)).astype(np.float32))
    b = si.round_to_bf16(g.standard_normal((N, K)).astype(np.float32))

    def view(x, rows, cols, is_far):
        base = torch.zeros((rows - 1) * (ld if is_far else cols) + cols, dtype=torch.bfloat16, device="cuda")
        v = base.as_strided((rows, cols), (ld if is_far else cols, 1))
        if x is not None:
            v.copy_(dev(x, "bf16"))
        return v

    got = host(sv.sv_gemm_bf16(view(a, M, K, far == "a"), view(b, N, K, far == "b"), tile=tile, out=view(None, M, N, far == "c")))
    assert_one_rounding(got, a, b)


# widths that are multiples of 64 (or 8, for the MLP) but not of 128; one kv head of 64 columns; fewer rows than a tile and ragged
# row tiles; a sequence shorter than a tile (RoPE positions wrap several times inside it)
EDGES = {
    "swiglu_192_kv64": (si.StageDesc(2, 192, 3, 1, 320), 3, 43),
    "gelu_ln_320": (si.StageDesc(1, 320, 5, 5, 832, mlp="gelu", norm="ln", rope=False), 2, 77),
    "odd_mlp_width": (si.StageDesc(1, 192, 3, 3, 200), 2, 65),
    "one_token": (si.StageDesc(1, 192, 3, 1, 320), 1, 1),
    "mqa_128_bidir": (si.StageDesc(1, 384, 3, 1, 960, causal=False), 5, 61),
    "ragged_960": (si.StageDesc(1, 960, 15, 5, 1088), 1, 301),
    "gelu_rms_runs": (si.StageDesc(1, 448, 7, 1, 3200, mlp="gelu"), 1, 130),
}


@pytest.mark.parametrize("case", list(EDGES))
@pytest.mark.parametrize("fuse", [False, True], ids=["norm_pass", "norm_inside"])
def test_stage_at_widths_that_are_no_multiple_of_a_tile(case, fuse):
    desc, B, S = EDGES[case]
    (gh, gg), (wh, wg), _ = run_stage(desc, B, S, seed=21, backward=True, weight_scale=2.0, fuse=fuse)
    assert_close(gh, wh, 2e-2, "h")
    assert_close(gg, wg, 2e-2, "g")


@pytest.mark.parametrize("desc,B,S", [(si.StageDesc(1, 192, 3, 1, 192, n_experts=4, top_k=1, n_shared=1), 8, 25),
                                      (si.StageDesc(1, 320, 5, 5, 448, n_experts=8, top_k=2, router_norm=True), 16, 16)])
def test_grouped_products_on_small_tiles(desc, B, S):
    """Rows of one expert start on multiples of 256 and the row count comes from device memory; expert widths are multiples of 64."""
    run_constructed(desc, B, S, 5, backward=True)
