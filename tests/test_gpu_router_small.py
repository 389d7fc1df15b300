"""Router logits of few tokens (one launch, weights split in registers) at the
edges of its 16-token and 16-expert blocks, of its 32-wide steps and 256-wide
stages, and of its three token counts per workgroup; against 64 bits, within the
logits' 1e-5 * max(|ref|, 1), and bit for bit against the same tokens in a call
that is too large for it.
"""
import pytest
import torch

from paper_2608_28511_amd import layer

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("S,E", [(1, 1), (15, 16), (16, 17), (17, 40), (65, 511), (1024, 64),   # 16 tokens a workgroup
                                 (1041, 64), (2064, 40),                                        # 32
                                 (2049, 64), (4100, 40), (4096, 64),                            # 64
                                 (4097, 64)])                                                   # split and tiles
@pytest.mark.parametrize("D", [8, 248, 256, 264, 1032, 2048])
def test_few_tokens(S, E, D):
    g = torch.Generator(device=DEV).manual_seed(S * 7 + E + D)
    x = torch.randn((S, D), generator=g, device=DEV).to(torch.bfloat16)
    Wr = torch.randn((D, E), generator=g, device=DEV) * D ** -0.5
    for bias in (None, torch.randn((E,), generator=g, device=DEV)):
        ref = x.double() @ Wr.double()
        if bias is not None:
            ref = ref + bias.double()
        got = layer.router_logits(x, Wr, bias).double()
        assert ((got - ref).abs() <= 1e-5 * ref.abs().clamp(min=1)).all()


@pytest.mark.parametrize("S,E", [(1, 1), (17, 40), (130, 511), (1024, 64), (1041, 64), (4100, 40), (4096, 64)])
@pytest.mark.parametrize("D", [8, 248, 264, 520, 1032, 2688])
def test_independent_of_the_call(S, E, D):
    """A token's logits are the same whether few or many others share its call."""
    g = torch.Generator(device=DEV).manual_seed(S * 5 + E + D)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    many = 64 * (cus // -(-E // 16)) + 65      # past the last workgroup of one round
    x = torch.randn((many, D), generator=g, device=DEV).to(torch.bfloat16)
    Wr = torch.randn((D, E), generator=g, device=DEV) * D ** -0.5
    bias = torch.randn((E,), generator=g, device=DEV)
    at = many - S - 3
    assert torch.equal(layer.router_logits(x[at:at + S].clone(), Wr, bias), layer.router_logits(x, Wr, bias)[at:at + S])
