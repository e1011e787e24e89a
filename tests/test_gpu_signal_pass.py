"""The verifier loop's one pass over bf16 signals (statistics, sum, projections) against the separate passes: the same signals as
float32 take those, so both loops must report the same statistics and keep the same averages.  Numbers of workers on every
side of a wave's four, token counts that end inside a tile of 16, one and several chunks of features, both direction counts."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import stage_inputs as si
from gpu_util import dev

METRICS = ("rel_l2", "l1", "zl2", "sfr", "sw")
POLICY = dict(c=5, t_forgive=100, k0=1.5, alpha=0.01, grow=1.1, shrink=0.9, n_max=10, window=64, min_dist_mult=0.35, eps=1e-4)


def _loops(n, T, D, L):
    import paper_2603_03592_amd as sv
    ver = sv.Verifier(si.TINY.desc, T, 64, sliced_w=True)
    u = dev(si.make_directions(D, L, 0), "bf16")
    return ver, [sv.Sentinel(ver, 1, n, T, D, METRICS, u, 0.9, 0.8, POLICY, POLICY) for _ in range(2)]


def _signals(n, T, D, t):
    g = np.random.default_rng(1000 * n + t)
    x = (1.0 + 0.1 * np.arange(n))[:, None, None] * g.standard_normal((n, T, D))
    x[:, :, ::7] = 0.0                                     # zeros on both sides of the sign test
    return si.round_to_bf16(x.astype(np.float32))


@pytest.mark.parametrize("n,T,D,L", [(1, 1, 64, 32), (2, 15, 64, 64), (4, 16, 128, 64), (5, 17, 192, 32), (8, 100, 64, 64), (9, 33, 1024, 64),
                                     (12, 47, 320, 32), (13, 64, 192, 64), (16, 130, 1024, 64), (3, 4099, 64, 32), (6, 4100, 128, 64), (8, 4097, 64, 32),
                                     (11, 4111, 64, 64), (12, 4098, 192, 32), (15, 4100, 64, 64)])
def test_one_pass_equals_the_separate_passes(n, T, D, L):
    ver, (one, sep) = _loops(n, T, D, L)
    for t in range(4):
        x = _signals(n, T, D, t)
        for loop, dtype in ((one, "bf16"), (sep, "f32")):
            loop.begin_iteration(t < 3)
        (ta, ga), (tb, gb) = one.forward(0, dev(x, "bf16")), sep.forward(0, dev(x, "f32"))
        assert ta == tb
        # fp32 sums of at most D terms per token in another order, double beyond
        np.testing.assert_allclose(ga, gb, rtol=2e-5, atol=1e-7)
        a, b = one.ema(0, "h"), sep.ema(0, "h")
        assert np.linalg.norm(a - b) <= 1e-6 * np.linalg.norm(b)
    c = one.counters()
    assert c["sw_carried"] == c["calls"] and c["ema_from_sum"] >= 3
    one.close(); sep.close(); ver.close()


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_non_finite_signals_stay_with_their_worker(bad):
    """One worker's non-finite value reaches its own statistics only; once that worker is excluded, the average stays finite."""
    n, T, D = 6, 40, 128
    ver, (one, sep) = _loops(n, T, D, 64)
    for t in range(6):
        x = _signals(n, T, D, t % 2)
        if t >= 4:
            x[3, 21, 50] = bad
        for loop in (one, sep):
            loop.begin_iteration(t < 4)
        (ta, ga), (tb, gb) = one.forward(0, dev(x, "bf16")), sep.forward(0, dev(x, "f32"))
        assert ta == tb
        ok = [r for r in range(n) if t < 4 or r != 3]
        np.testing.assert_allclose(ga[ok], gb[ok], rtol=2e-5, atol=1e-7)
        if t == 4:                                         # later it may be banned and no longer examined
            assert 3 in ta and not np.isfinite(ga[3, 0]) and not np.isfinite(ga[3, 4])
        assert np.isfinite(one.ema(0, "h")).all()
    one.close(); sep.close(); ver.close()


@pytest.mark.parametrize("n,T,D,one", [(9, 128, 1728, False), (16, 64, 448, False), (5, 700, 1088, False), (2, 33, 1088, False), (16, 1535, 384, False),
                                       (4, 64, 960, True), (16, 64, 320, True), (16, 1536, 384, True), (6, 4096, 448, True)])
def test_few_tokens_take_the_separate_passes(n, T, D, one):
    """Rows that the score pass cannot sum, so that the average's update tells which way a call went: from the sum that the one pass
    leaves, or from the signals."""
    ver, (a, b) = _loops(n, T, D, 32)
    x = _signals(n, T, D, 0)
    for loop, dtype in ((a, "bf16"), (b, "f32")):
        loop.begin_iteration(True)
    (_, ga), (_, gb) = a.forward(0, dev(x, "bf16")), b.forward(0, dev(x, "f32"))
    np.testing.assert_allclose(ga, gb, rtol=2e-5, atol=1e-7)
    c = a.counters()
    assert (c["ema_from_sum"], c["calls"]) == (int(one), 1)
    assert np.linalg.norm(a.ema(0, "h") - b.ema(0, "h")) <= 1e-6 * np.linalg.norm(b.ema(0, "h"))
    a.close(); b.close(); ver.close()
