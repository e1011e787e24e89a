"""Which kernel a product of the stage takes is decided on the host, so its promises to the rest of the stage are checked without
a device."""
import pytest

import paper_2603_03592_amd as sv

WIDTHS = [(1024, 2816), (1024, 16384), (2048, 5632), (2048, 10240), (2048, 12288), (2048, 16384), (3584, 18944), (4096, 4096), (4096, 11008),
          (4096, 14336), (5120, 13824), (960, 3840), (2048, 2048), (2560, 64)]
ROWS = sorted({1, 64, 129, 512, *range(256, 10497, 256), *range(257, 10497, 512), *range(255, 10496, 768), 2304, 4779, 16384})
SCRATCH = 8 * 160 * 128 * 128                              # the most a context holds


@pytest.mark.parametrize("N,K", WIDTHS)
def test_row_sums_are_promised_only_by_products_that_write_them(N, K):
    """A norm that runs inside the next product takes its rows' sums of squares from the product that writes the stream.  Only the
    whole 256x256 kernel leaves them, with scratch for partial products at hand or without."""
    promised = 0
    for M in ROWS:
        for ws in (0, 8 * M * max(N, K), SCRATCH, 4 * SCRATCH):
            leaves, tile, runs = sv.sv_gemm_plan(M, N, K, ws, row_sums=True)
            assert tile != 0 and runs >= 1
            assert not leaves or (tile, runs) == (1, 1), (M, N, K, ws, tile, runs)
            promised += leaves
        assert not sv.sv_gemm_plan(M, N, K, SCRATCH)[0]
    assert promised > 0 or N % 256 or N < 2048


def test_the_stage_tests_reach_products_whole_and_over_runs():
    """The stages of test_gpu_gemm_tiles.py are there for the epilogues behind both kinds of launch: if another price moves them, this
    fails and they need other sizes."""
    def ws(T, D, F):
        return min(SCRATCH, 8 * T * max(D, F))
    assert sv.sv_gemm_plan(130, 448, 3200, ws(130, 448, 3200))[2] > 1              # gelu_rms_runs, down-projection
    assert sv.sv_gemm_plan(301, 960, 1088, ws(301, 960, 1088))[2] == 1             # ragged_960
    assert sv.sv_gemm_plan(130, 192, 200, ws(130, 192, 200)) == (False, 0, 1)      # odd_mlp_width: k is no multiple of 64


def test_every_tile_serves_some_size():
    seen = {sv.sv_gemm_plan(M, N, K, SCRATCH)[1] for M in (64, 512, 2331, 4096, 8192) for N in (960, 1024, 2048, 4096) for K in (512, 2048, 14336)}
    assert seen == {1, 2, 3, 4, 5}
