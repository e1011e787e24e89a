"""Submissions against one shared reference, rows that are no multiple of 2 KB, enough of them for the kernel that keeps the
reference in registers: parts of two, three and four units with the row's end in every place of them, one and several parts, groups
of submissions that do not divide their number, every pair of types; against 64 bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import stage_inputs as si

METRICS = ("rel_l2", "l1", "zl2", "sfr")
DT = {"bf16": torch.bfloat16, "f32": torch.float32}


def _verifier(T):
    import paper_2603_03592_amd as sv
    return sv.Verifier(si.TINY.desc, T, 64)


def _inputs(n, T, D, cd, rd):
    g = torch.Generator(device="cuda").manual_seed(n * T + D)
    ref = torch.randn((T, D), generator=g, device="cuda")
    ref[:, ::5] = 0.0
    ref[:, 3::11] = -0.0
    claims = torch.stack([ref * (1.0 + 0.25 * i) + 0.1 * (i + 1) * torch.randn((T, D), generator=g, device="cuda") for i in range(n)])
    claims[:, :, ::7] = 0.0
    return claims.to(DT[cd]).contiguous(), ref.to(DT[rd])


def _want(a, r):
    a, r = a.double(), r.double()
    d = a - r
    tok = d.norm(dim=1) / r.norm(dim=1)
    z = ((a - a.mean()) / a.std(unbiased=False) - (r - r.mean()) / r.std(unbiased=False)).square().mean()
    return tok, torch.stack((d.norm() / r.norm(), d.abs().mean(), z, (torch.sign(a) != torch.sign(r)).double().mean()))


@pytest.mark.parametrize("n,T,D", [(2, 8200, 8), (2, 8177, 504), (3, 8192, 520), (2, 8200, 1160), (5, 4100, 1664), (9, 2750, 2056), (2, 8200, 3080), (17, 2750, 904)])
@pytest.mark.parametrize("cd,rd", [("bf16", "bf16"), ("bf16", "f32"), ("f32", "bf16"), ("f32", "f32")])
@pytest.mark.parametrize("full", [True, False])
def test_ragged_rows(n, T, D, cd, rd, full):
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


def test_non_finite_values_stay_with_their_token():
    n, T, D = 3, 8192, 1160
    ver = _verifier(T)
    claims, ref = _inputs(n, T, D, "bf16", "f32")
    claims[1, 4000, D - 1] = float("nan")
    claims[2, 17, D - 8] = float("inf")
    o = ver.score_and_flag(claims, ref, metrics=METRICS, tau=(9, 9, 9, 9), reduce="global", want_token_scores=True)
    res, tok = ver.read_results(o["result"]), o["token_scores"]
    assert [int(r["flag"]) for r in res] == [0, 1, 1]
    ok = torch.isfinite(tok)
    assert not ok[1, 4000] and not ok[2, 17] and int((~ok).sum()) == 2
    ver.close()
