"""Products on 256 x 256 tiles whose last round is left to a second launch on smaller ones: against the same product on smaller tiles
alone, which adds up every element in the same order, so bit for bit.  Last rounds of one tile per XCD and of a quarter and a half
of the chip, tile counts that leave an XCD short, a ragged row end inside the last round, a k loop too short for the half."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(256 * 66, 1024, 256), (256 * 72, 1024, 128), (256 * 96, 1024, 2048), (256 * 96, 1024, 256), (256 * 90, 768, 192),
                                   (256 * 66 - 100, 1024, 64), (256 * 93 - 1, 768, 2112), (256 * 263, 256, 128)])
def test_last_round_on_smaller_tiles(M, N, K):
    import paper_2603_03592_amd as sv
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are chosen for 256 compute units")
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    a = torch.randn((M, K), generator=g, device="cuda").to(torch.bfloat16)
    b = torch.randn((N, K), generator=g, device="cuda").to(torch.bfloat16)
    whole, small = sv.sv_gemm_bf16(a, b, tile=1), sv.sv_gemm_bf16(a, b, tile=2)
    assert torch.equal(whole, small)
    rows = torch.cat((torch.arange(0, M, 977), torch.arange(M - 300, M))).cuda()
    want = a[rows].double() @ b.double().t()
    # a bf16 result: half an ulp is 2^-8 of the value's power of two at most; K products in fp32 behind it
    assert ((whole[rows].double() - want).abs() <= 2.0 ** -8 * want.abs() + K * 2.0 ** -22).all()
