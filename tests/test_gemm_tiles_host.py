"""Which tiles a block's products run on is decided on the host: what the device tests of those tiles count on, and what the kernels do."""
import numpy as np
import pytest

import paper_2603_03592_amd as sv
from test_gpu_gemm_same_bits import MIXTURES, STAGES, mixture_plan, stage_plan, stage_products

SCRATCH = 8 * 160 * 128 * 128


@pytest.mark.parametrize("case", list(STAGES))
def test_stages_run_on_what_their_device_test_names(case):
    """In one run each, the whole stage and its pieces: else the sums would be cut in other places."""
    c = STAGES[case]
    whole, piece = stage_plan(c, c.batch), stage_plan(c, c.piece)
    assert all(runs == 1 for _, runs, _ in [*whole.values(), *piece.values()]), (whole, piece)
    for name, (tile, tail) in c.aims.items():
        assert whole[name][0] == tile and tail(whole[name][2]), (name, whole[name])
        assert piece[name][0] != tile or (whole[name][2] > 0 and piece[name][2] == 0), (name, whole[name], piece[name])


@pytest.mark.parametrize("case", [c for c in STAGES if "_rounds" in c])
def test_stages_of_several_rounds_take_them(case):
    for name, (N, K, e) in stage_products(STAGES[case]).items():
        M = STAGES[case].batch * STAGES[case].seq
        assert (M + 255) // 256 * (N // (128 if e == "swiglu" else 256)) > 256, name


@pytest.mark.parametrize("case", list(MIXTURES))
def test_mixtures_leave_tails(case):
    c = MIXTURES[case]
    for name, (tile, runs, tail) in mixture_plan(c, c.batch).items():
        assert (tile, runs) == (1, 1) and tail > 0, (name, tile, tail)


@pytest.mark.parametrize("M,mlp,ffn", [(1537, "gelu", 6144), (1537, "swiglu", 3072)])
def test_the_stages_of_the_narrower_tile_take_it(M, mlp, ffn):
    """test_gpu_gemm_narrower.py: 512 columns."""
    assert sv.sv_gemm_tiles(M, ffn, 512, mlp, 0, SCRATCH)[0] == 6
    assert sv.sv_gemm_tiles(M, 6144, 512, mlp + "_bwd", 0, SCRATCH)[0] == 6


def test_the_narrower_tile_is_never_planned_over_runs_of_k():
    """It has no form that leaves partial products."""
    rng, six = np.random.default_rng(0), 0
    for _ in range(20000):
        M, N, K = int(2 ** rng.uniform(5, 16)), 256 * int(2 ** rng.uniform(0, 7)), 64 * int(rng.integers(1, 49))
        for epilogue in ("gelu", "gelu_bwd", "swiglu", "swiglu_bwd"):
            tile, runs, _ = sv.sv_gemm_tiles(M, N, K, epilogue, 0, 1 << 40)
            six += tile == 6
            assert tile != 6 or runs == 1, (M, N, K, epilogue)
    assert six > 1000


@pytest.mark.parametrize("epilogue", ["store", "swiglu", "swiglu_bwd"])
@pytest.mark.parametrize("E,K", [(1, 1), (2, 1), (4, 1), (8, 1), (8, 2), (8, 6), (16, 4)])
def test_the_second_launch_in_groups_covers_whatever_the_router_does(epilogue, E, K):
    """How many rows are in use is known on the device only, between the tokens' and a part of a tile more for every group, and with
    them how many tiles the first launch leaves.  The second is made for as many as there can be, or not at all."""
    made = 0
    for N in (256, 512, 1024, 2048, 4096):
        for k in (64, 512, 2048, 4096):
            for T in (1, 255, 257, 1000, 2048, 4099, 5120, 8192, 11264, 16385, 20000, 32768, 33793, 40961):
                least = (T * K + 255) // 256
                tail = sv.sv_gemm_tiles((least + E) * 256, N, k, epilogue, E)[2]
                if tail == 0:
                    continue
                made += 1
                for tiles in range(least, least + E + 1):
                    assert sv.sv_gemm_tiles(tiles * 256, N, k, epilogue)[2] <= tail, (N, k, T, tiles)
    assert made > 20


def test_arguments_are_checked():
    for bad in [(0, 256, 64, 0, 0, 0), (256, 256, 64, 7, 0, 0), (256, 256, 64, -1, 0, 0), (256, 256, 64, 0, -1, 0), (256, 256, 64, 0, 0, -1)]:
        M, N, K, e, groups, ws = bad
        import ctypes
        i = [ctypes.c_int32() for _ in range(3)]
        assert sv.lib.sv_gemm_tiles(M, N, K, e, groups, ws, *(ctypes.byref(x) for x in i)) == 1
    assert sv.sv_gemm_tiles(256, 200, 100, "store") == (0, 1, 0)               # the vector kernel
