"""The verifier loop's one pass updates the EMA over the submissions nobody expected to exclude, and a verdict that excludes one all
the same goes back to what the EMA was: against the separate passes (the same signals as float32), which decide first.  Every
number of places for submissions with both direction counts, with and without a free place, one and several turns of chunks."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_util import dev
from test_gpu_signal_pass import _loops, _signals


@pytest.mark.parametrize("n,T,D,L", [(4, 33, 64, 32), (4, 16, 448, 64), (7, 40, 320, 32), (8, 17, 256, 32), (8, 50, 1024, 64), (12, 21, 192, 64),
                                     (11, 16, 320, 32), (16, 35, 256, 32), (16, 16, 1024, 64), (15, 64, 320, 32)])
@pytest.mark.parametrize("bad", [5.0, np.nan])
def test_unexpected_exclusion_goes_back(n, T, D, L, bad):
    ver, (one, sep) = _loops(n, T, D, L)
    for t in range(6):
        x = _signals(n, T, D, 0)
        if t >= 4:                                         # one worker leaves the fences
            x[2] *= bad
        for loop in (one, sep):
            loop.begin_iteration(t < 4)
        back = {}
        for name, loop, dtype in (("one", one, "bf16"), ("sep", sep, "f32")):
            tf, gf = loop.forward(0, dev(x, dtype))
            g = dev(0.5 * x, dtype)
            tb, gb = loop.backward(0, g)
            back[name] = (tf, tb, g.float().cpu().numpy())
        (tf, tb, g1), (sf, sb, g2) = back["one"], back["sep"]
        assert (tf, tb) == (sf, sb)
        if t == 4:
            assert 2 in tf
        for kind in "hg":
            a, b = one.ema(0, kind), sep.ema(0, kind)
            assert np.isfinite(a).all() and np.linalg.norm(a - b) <= 1e-6 * np.linalg.norm(b)
        # what replaced a gradient: the average, in bf16 here (half an ulp is 2^-9 of the value's power of two, the averages differ by 1e-6)
        np.testing.assert_allclose(g1, g2, rtol=2.0 ** -8, atol=1e-6)
    c1, c2 = one.counters(), sep.counters()
    assert c1["ema_from_signals"] >= 1 and c1["calls"] == c2["calls"] == 12
    assert c1["ema_from_sum"] >= 8                         # the warm-up's calls at least: the one pass, or the test has missed its aim
    one.close(); sep.close(); ver.close()
