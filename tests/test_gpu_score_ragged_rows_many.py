"""Rows that are no multiple of 2 KB against one shared reference, at numbers of workgroups for which the kernel that keeps the reference in
registers is taken on any number of compute units: about three per unit with all sums or narrow rows, more than six with the relative L2
alone and rows of 3 KB and more.  Rows in one and several parts of two to four units, and signals of more than 256 MB, whose loads leave
nothing in the caches."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from test_gpu_score_ragged_rows import METRICS, _inputs, _verifier, _want


def _tokens(n, per_cu):
    """Tokens, ending inside a tile of 16, that make per_cu workgroups per compute unit of groups of at most four submissions."""
    groups = (n + 3) // 4
    return 16 * int(round(per_cu * torch.cuda.get_device_properties(0).multi_processor_count / groups)) - 7


@pytest.mark.parametrize("n,per_cu,D", [(4, 2.9, 8), (5, 2.9, 504), (17, 3.6, 520), (4, 2.9, 1160), (17, 3.6, 1664), (5, 2.9, 2056), (4, 3.8, 3080),
                                        (8, 6.7, 904), (8, 6.7, 1160), (7, 6.7, 1664), (8, 6.7, 2056)])
@pytest.mark.parametrize("cd,rd", [("bf16", "bf16"), ("bf16", "f32"), ("f32", "bf16"), ("f32", "f32")])
@pytest.mark.parametrize("full", [True, False])
def test_ragged_rows_of_many_workgroups(n, per_cu, D, cd, rd, full):
    T = _tokens(n, per_cu)
    ver = _verifier(T)
    claims, ref = _inputs(n, T, D, cd, rd)
    o = ver.score_and_flag(claims, ref, metrics=METRICS if full else METRICS[:1], tau=(0, 0, 0, 0), reduce="global", want_token_scores=True)
    res, tok = ver.read_results(o["result"]), o["token_scores"]
    for i in range(n):
        t, s = _want(claims[i], ref)
        # a token's sums: at most 3080 terms in fp32, some 2^-24 each, in chains of at most 64
        assert (tok[i].double() - t).abs().max() <= 1e-5 * t.max()
        got = torch.tensor(res[i]["score"][:4 if full else 1].copy()).double()
        want = s.cpu()[:4 if full else 1]
        assert ((got - want).abs() <= 2e-5 * want + 1e-7).all(), (i, got, want)
        if full:                                           # a count: the quotient's rounding only
            assert abs(got[3] * T * D - want[3] * T * D) <= 0.5 + T * D * 2.0 ** -24
    ver.close()
