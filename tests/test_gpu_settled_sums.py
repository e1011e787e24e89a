"""The sums that lead to a router keep their cut into runs of k whatever tile is cheapest, in every block that another one follows."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import stage_inputs as si
from gpu_util import dev, dev_weights, host


def settled_runs(M, N, K):
    """The cut as 256x256 tiles over runs of k slices, or 128x64 tiles over runs, once brought it about."""
    slices = K // 64
    if N % 256 == 0:
        tiles = -(-M // 256) * (N // 256)
        if tiles >= 192:
            return 1
        n = min(8, 256 // tiles, slices // 4)
        if n >= 2:
            return n
    rows = -(-M // 128)
    if N % 128 == 0 and rows * (N // 128) < 160:
        n = min(8, slices // 8, -(-768 // (rows * (N // 64))))
        if n >= 2:
            return n
    return 1


# the free choice for these: 64x64 tiles whole, 64x64 or 128x128 tiles over fewer or more runs
@pytest.mark.parametrize("T,D,F,shared", [(1024, 1024, 1024, 1), (200, 256, 512, 2), (512, 512, 1024, 1), (2048, 1024, 704, 1), (640, 384, 1024, 2)])
def test_the_shared_experts_sum_is_cut_alike_wherever_a_router_follows(T, D, F, shared):
    """The first block adds sum_f a_f to every element, over k = the shared experts' width: a_0 = 2^24, two ones in every slice of 64,
    2^24 taken off at the very end.  In 32 bits the ones of the first run are lost beside 2^24, those of the others are not, so the
    result counts the slices outside the first run.  The second block adds nothing and shows the first one's output."""
    import paper_2603_03592_amd as sv
    Fs, H = shared * F, D // 64
    desc = si.StageDesc(2, D, H, H, F, n_experts=2, top_k=1, n_shared=shared)
    g = np.random.default_rng(T)
    h = np.where(g.random((1, T, D)) < 0.5, -1.0, 1.0).astype(np.float32)
    h[..., :2] = 1.0                                       # the norm leaves +-1: 1 / sqrt(1 + eps) is 1 in bf16
    w = si.make_weights(desc, 3)
    for b in w:
        for k in ("wo", "w_down", "ws_down"):
            b[k] = np.zeros_like(b[k])
        b["norm2_g"] = np.ones_like(b["norm2_g"])
    a = np.zeros(Fs, np.float32)
    a[16::64] = a[32::64] = 1.0
    a[0], a[-1] = 2.0 ** 24, -2.0 ** 24
    w[0]["ws_gate"], w[0]["ws_up"] = np.zeros_like(w[0]["ws_gate"]), np.zeros_like(w[0]["ws_up"])
    w[0]["ws_gate"][:, 0] = 32.0                           # silu(32) is 32 in 32 bits
    w[0]["ws_up"][:, 1] = a / 32.0
    w[0]["ws_down"] = np.ones_like(w[0]["ws_down"])
    for backward in (False, True):
        ver = sv.Verifier(desc, T, T, backward=backward)
        got = host(ver.verify_forward(ver.pack_weights(wd := dev_weights(w, "bf16")), dev(h, "bf16"), want_h_hat=True)["h_hat"])
        ver.close()
        slices, runs = Fs // 64, settled_runs(T, D, Fs)
        assert np.array_equal(got, h + 2.0 * (slices - slices // runs)), (runs, np.unique(got - h))


def test_routing_does_not_depend_on_the_room_for_more_tokens():
    """Two blocks, two contexts of different capacity (the scratch holds the cut in both): the same experts and the same gates."""
    import paper_2603_03592_amd as sv
    desc = si.StageDesc(2, 512, 8, 2, 1024, n_experts=8, top_k=2, n_shared=1, router_norm=True)
    B, S = 3, 230
    wd, h = dev_weights(si.make_weights(desc, 6), "bf16"), dev(si.make_activations(desc, B, S, 6), "bf16")
    seen = []
    for room in (B * S, 8192):
        ver = sv.Verifier(desc, room, 1024, backward=True)
        ver.verify_forward(ver.pack_weights(wd), h, want_h_hat=True)
        seen.append([t.cpu().numpy() for l in range(2) for t in ver.last_routing(l, B * S)])
        ver.close()
    assert all(np.array_equal(a, b) for a, b in zip(*seen))
