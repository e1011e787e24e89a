"""Scores formed by the workgroup that comes last with a record of its submission: equal, bit for bit, to those of a launch of their own
over the same records (the entry point without a context always makes one), call after call, on either side of the record count up to which
the pass does it and of the number of records at which the reduction takes more threads."""
import pytest

pytestmark = pytest.mark.gpu

import paper_2603_03592_amd as sv
import stage_inputs as si

SHAPES = [  # submissions, tokens, columns, with a reference each
    (1, 1, 64, False), (1, 128, 128, False), (1, 129, 64, False), (1, 256, 1024, False), (1, 257, 72, False), (1, 1000, 128, False),
    (3, 77, 960, True), (16, 16, 64, True), (64, 4, 64, True), (65, 3, 64, True), (9, 5000, 64, True),
]


@pytest.mark.parametrize("n,T,D,own", SHAPES)
def test_scores_do_not_depend_on_who_forms_them(n, T, D, own):
    import torch

    torch.manual_seed(n * 1000 + T)
    ver = sv.Verifier(si.StageDesc(1, 128, 4, 4, 512, mlp="gelu", norm="ln", rope=False, dtype="f32"), 64, 64)
    for call in range(3):
        ref = torch.randn(n, T, D, device="cuda") if own else torch.randn(T, D, device="cuda")
        claims = (ref + (0.01 + call) * torch.randn(n, T, D, device="cuda")).bfloat16()
        args = dict(metrics=("rel_l2", "l1", "zl2", "sfr"), tau={"rel_l2": 0.5, "l1": 0.5, "zl2": 0.5, "sfr": 0.2})
        got = ver.score_and_flag(claims, ref, **args)["result"].view(torch.uint8).reshape(-1)
        want = sv.score_and_flag_noalloc(claims, ref, torch.zeros(n, 32, dtype=torch.uint8, device="cuda"), **args).reshape(-1)
        assert torch.equal(got, want), (n, T, D, call)
    ver.close()
