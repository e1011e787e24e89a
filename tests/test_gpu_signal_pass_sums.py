"""The sums of the verifier loop's one pass over long rows whose mean is many times their spread, where the z-scored statistic is a small
difference of large moments: against 64 bits.  And a submission of one value only, which has no spread."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import stage_inputs as si
from gpu_util import dev
from test_gpu_signal_pass import _loops

MEAN = 30.0


def _statistics(a, m):
    d = a - m
    z = ((a - a.mean()) / a.std(unbiased=False) - (m - m.mean()) / m.std(unbiased=False)).square().mean()
    return torch.stack((d.norm() / m.norm(), d.abs().mean(), z)).cpu().numpy()


@pytest.mark.parametrize("n,L", [(3, 32), (4, 64), (8, 32), (8, 64), (11, 64), (12, 32), (16, 32), (16, 64)])
def test_moments_of_signals_far_from_zero(n, L):
    T, D = 64, 4096
    ver, (one, sep) = _loops(n, T, D, L)
    g = torch.Generator(device="cuda").manual_seed(n + L)
    base = MEAN + torch.randn((T, D), generator=g, device="cuda")
    x = torch.stack([base + 0.5 * torch.randn((T, D), generator=g, device="cuda") for _ in range(n)]).bfloat16()
    for t in range(4):
        m = torch.from_numpy(one.ema(0, "h")).cuda().double().view(T, D)
        one.begin_iteration(True)
        _, gamma = one.forward(0, x)
        if t == 0:
            continue                                       # against zeros
        for i in range(n):
            want = _statistics(x[i].double(), m)
            # float results; a token's sums of squares within some eight roundings of 2^-25, which the subtraction of the squared mean
            # makes (mean / spread)^2 times as large in the variances; other tokens' errors are others
            assert (np.abs(gamma[i][:2] - want[:2]) <= 2.0 ** -22 * want[:2]).all(), (t, i)
            assert abs(gamma[i][2] - want[2]) <= 8 * 2.0 ** -25 * MEAN ** 2 * 2 * want[2], (t, i, gamma[i][2] / want[2] - 1)
    assert one.counters()["ema_from_sum"] == 4             # all by the one pass or the summing one, whose rows are whole
    one.close(); sep.close(); ver.close()


def test_a_constant_submission_has_no_spread():
    n, T, D = 8, 48, 4096
    ver, (one, sep) = _loops(n, T, D, 64)
    g = np.random.default_rng(3)
    x = si.round_to_bf16((MEAN + g.standard_normal((n, T, D))).astype(np.float32))
    for i, c in enumerate((1.2890625, 255.0, -0.0419921875)):
        x[2 * i] = c
    for t in range(2):
        for loop in (one, sep):
            loop.begin_iteration(True)
        (_, a), (_, b) = one.forward(0, dev(x, "bf16")), sep.forward(0, dev(x, "f32"))
    for i in (0, 2, 4):
        assert a[i, 2] == b[i, 2] == 2.0
    assert (a[[1, 3, 5, 6, 7], 2] < 2.1).all()
    one.close(); sep.close(); ver.close()
