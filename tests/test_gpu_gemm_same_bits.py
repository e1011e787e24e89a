"""Products with every epilogue on 192x256 tiles, and on 256x256 tiles whose last round is left to a second launch on smaller ones: bit for bit
what the same products give on the tiles that a check of fewer sequences takes.  A sequence's results do not depend on the others, and
every tile adds up an element in the same order, so a whole check has to equal the checks of its pieces.  test_gemm_tiles_host.py says
which tiles they are."""
import dataclasses

import pytest

import paper_2603_03592_amd as sv
import stage_inputs as si


@dataclasses.dataclass(frozen=True)
class Case:
    mlp: str
    d: int
    ffn: int
    batch: int
    seq: int
    piece: int
    aims: dict                                             # product: (tile, what its tail is)
    rope: bool = True
    fuse: bool = False

    @property
    def desc(self):
        return si.StageDesc(1, self.d, self.d // 64, self.d // 64, self.ffn, mlp=self.mlp, norm="rms", rope=self.rope)


# the kinds of products that take more rounds of 256x256 tiles than one without leaving any to a second launch, so that a workgroup goes on from a
# tile to the next with its stores on their way
_rounds = {n: (1, lambda t: t == 0) for n in ("qkv", "o", "up", "down", "dact", "dn2", "do", "dn1")}
_some, _half, _any = (lambda t: 0 < t <= 8), (lambda t: t > 8), (lambda t: True)
_quarter = {n: (1, _some) for n in ("qkv", "o", "up", "down", "dact", "dn2", "do", "dn1")}
STAGES = {
    "gelu": Case("gelu", 1024, 1024, 11, 1500, 1, _quarter),
    "swiglu": Case("swiglu", 1024, 1024, 11, 1500, 1, _quarter),
    "swiglu_no_rope": Case("swiglu", 1024, 1024, 11, 1500, 1, _quarter, rope=False),
    "gelu_half": Case("gelu", 2048, 2048, 8, 1500, 1, {n: (1, _half) for n in _quarter}),
    "swiglu_half": Case("swiglu", 2048, 2048, 4, 1500, 1, {"up": (1, _half)}),
    "swiglu_bwd_half": Case("swiglu", 2048, 2048, 7, 1500, 1, {n: (1, _half) for n in ("dact", "o", "down")}),
    "row_factors": Case("swiglu", 1024, 1536, 11, 1500, 1, {"qkv": (1, _some), "up": (1, _some)}, fuse=True),
    "row_factors_gelu": Case("gelu", 1280, 1024, 12, 1500, 1, {"qkv": (1, _some), "up": (1, _some)}, fuse=True),
    "gelu_rounds": Case("gelu", 1024, 1024, 18, 1500, 1, _rounds),
    "swiglu_rounds": Case("swiglu", 1024, 1024, 18, 1500, 1, _rounds),
    "swiglu_rounds_no_rope": Case("swiglu", 1024, 1024, 18, 1500, 1, _rounds, rope=False),
    "narrower_gelu": Case("gelu", 1536, 1024, 9, 1229, 1, {"up": (6, _any), "dact": (6, _any)}),
    "narrower_gelu_ragged": Case("gelu", 768, 3840, 3, 777, 1, {"up": (6, _any), "dact": (6, _any)}),
    "narrower_swiglu": Case("swiglu", 512, 1536, 5, 777, 1, {"up": (6, _any)}),
    "narrower_row_factors": Case("swiglu", 512, 1536, 5, 777, 1, {"up": (6, _any)}, fuse=True),
    "narrower_row_factors_gelu": Case("gelu", 768, 3840, 3, 777, 1, {"up": (6, _any)}, fuse=True),
    "narrower_swiglu_bwd": Case("swiglu", 768, 1024, 11, 777, 1, {"dact": (6, _any), "up": (1, _some)}),
}


@dataclasses.dataclass(frozen=True)
class Mixture:
    d: int
    ffn: int
    experts: int
    top_k: int
    batch: int
    seq: int
    piece: int

    @property
    def desc(self):
        # without rotation, which before a router rounds its input by the number of tokens
        return si.StageDesc(1, self.d, 4, 4, self.ffn, rope=False, n_experts=self.experts, top_k=self.top_k)


MIXTURES = {"top2": Mixture(256, 256, 8, 2, 35, 1024, 6), "top1": Mixture(256, 256, 4, 1, 66, 1024, 12)}


def stage_products(c):
    D, F, two = c.d, c.ffn, 2 if c.mlp == "swiglu" else 1
    return {"qkv": (3 * D, D, "rope" if c.rope else "store"), "o": (D, D, "residual"), "up": (F, D, c.mlp), "down": (D, F, "residual"),
            "dact": (F, D, c.mlp + "_bwd"), "dn2": (D, two * F, "store"), "do": (D, D, "store"), "dn1": (D, 3 * D, "store")}


def stage_plan(c, batch):
    M, ws = batch * c.seq, min(8 * 160 * 128 * 128, 8 * c.batch * c.seq * max(c.d, c.ffn))
    return {n: sv.sv_gemm_tiles(M, N, K, e, 0, ws) for n, (N, K, e) in stage_products(c).items()}


def mixture_plan(c, batch):
    M, D, F = ((batch * c.seq * c.top_k + 255) // 256 + c.experts) * 256, c.d, c.ffn
    products = {"up": (F, D, "swiglu"), "down": (D, F, "store"), "dact": (F, D, "swiglu_bwd"), "dx": (D, 2 * F, "store")}
    return {n: sv.sv_gemm_tiles(M, N, K, e, c.experts) for n, (N, K, e) in products.items()}


def _whole_and_pieces(ver, wc, h, g, piece):
    import torch
    def run(a, b):
        o = ver.verify_backward(wc, h[a:b].contiguous(), g[a:b].contiguous(), want_g_hat=True, want_h_hat=True)
        return o["h_hat"].clone(), o["g_hat"].clone()
    B = h.shape[0]
    whole = run(0, B)
    parts = [run(a, min(a + piece, B)) for a in range(0, B, piece)]
    for name, w, p in zip("hg", whole, zip(*parts)):
        p = torch.cat(p)
        assert torch.isfinite(w).all() and w.float().abs().mean() > 0
        assert torch.equal(w, p), (name, (w != p).nonzero()[:4].tolist(), int((w != p).sum()))


@pytest.mark.gpu
@pytest.mark.parametrize("case", list(STAGES))
def test_stage_equals_its_pieces(case):
    import torch
    from gpu_util import dev_weights
    c = STAGES[case]
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are chosen for 256 compute units")
    if c.fuse:                                             # the norms' row sums come from the same place in both
        ws = min(8 * 160 * 128 * 128, 8 * c.batch * c.seq * max(c.d, c.ffn))
        assert len({sv.sv_gemm_plan(b * c.seq, c.d, K, ws, row_sums=True)[0] for b in (c.batch, c.piece) for K in (c.d, c.ffn)}) == 1
    gen = torch.Generator(device="cuda").manual_seed(len(case))
    h, g = (torch.randn((c.batch, c.seq, c.d), generator=gen, device="cuda").bfloat16() for _ in range(2))
    ver = sv.Verifier(c.desc, c.batch * c.seq, c.seq, backward=True, fuse_norm=c.fuse)
    wc = ver.pack_weights(wd := dev_weights(si.make_weights(c.desc, 7), "bf16"))
    _whole_and_pieces(ver, wc, h, g, c.piece)
    ver.close()


@pytest.mark.gpu
@pytest.mark.parametrize("case", list(MIXTURES))
@pytest.mark.parametrize("routing", ["as_it_comes", "all_to_the_first", "all_to_the_last"])
def test_mixture_equals_its_pieces(case, routing):
    """Also with every token's experts the same: the least rows that there can be, in as few groups."""
    import torch
    from gpu_util import dev_weights
    c = MIXTURES[case]
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are chosen for 256 compute units")
    gen = torch.Generator(device="cuda").manual_seed(len(case + routing))
    h, g = (torch.randn((c.batch, c.seq, c.d), generator=gen, device="cuda").bfloat16() for _ in range(2))
    w = si.make_weights(c.desc, 7)
    wd = dev_weights(w, "bf16")
    if routing != "as_it_comes":                           # one feature, large in every token, decides for top_k experts
        h[:, :, 5] = 40.0
        chosen = list(range(c.top_k)) if routing == "all_to_the_first" else list(range(c.experts - c.top_k, c.experts))
        r = torch.zeros_like(wd[0]["w_router"])
        r[:, 5] = -0.5
        for i, e in enumerate(chosen):
            r[e, 5] = 0.5 + 0.125 * i
        wd[0]["w_router"] = r
    ver = sv.Verifier(c.desc, c.batch * c.seq, c.seq, backward=True)
    wc = ver.pack_weights(wd)
    _whole_and_pieces(ver, wc, h, g, c.piece)
    ver.verify_backward(wc, h, g, want_g_hat=True, want_h_hat=True)
    if routing != "as_it_comes":
        assert set(ver.last_routing(0, c.batch * c.seq)[0].flatten().tolist()) == set(chosen)
    ver.close()
