"""The grouped GEMM's 128-column tile, which the smallest launches take, and the
256-column one just past it: widths that end inside a wave's 64 columns and at
and beside a tile's edge, contractions of one stage to more than its ring holds
(whole and cut), segments at the edges of its 32-row waves, gathered rows, every
epilogue.  Small integers: every product and sum is exact, so the results are
compared bit for bit.
"""
import pytest
import torch

from paper_2608_28511_amd import _lib as L
from paper_2608_28511_amd import layer

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
COUNTS = [0, 1, 31, 32, 33, 64, 127, 128, 129, 3]   # R = 548


def _ints(g, shape, hi):
    return torch.randint(-hi, hi + 1, shape, generator=g, device=DEV).to(torch.bfloat16)


def _product(A, off, W):
    o = off.tolist()
    return torch.cat([A[a:b].float() @ W[e].float() for e, (a, b) in enumerate(zip(o, o[1:]))])


# 13 m-tiles at most, two an XCD: N <= 2,048 is narrow on 256 compute units
@pytest.mark.parametrize("N", [8, 120, 128, 136, 264, 2048, 2056])
@pytest.mark.parametrize("Kd", [8, 64, 72, 328])
def test_grouped(Kd, N):
    g = torch.Generator(device=DEV).manual_seed(Kd * 1000 + N)
    off = torch.zeros(len(COUNTS) + 1, dtype=torch.int32)
    off[1:] = torch.tensor(COUNTS).cumsum(0)
    off = off.to(DEV)
    R, E, K = sum(COUNTS), len(COUNTS), 4
    S = R // K
    x = _ints(g, (S, Kd), 1)
    perm = torch.randperm(R, generator=g, device=DEV).to(torch.int32)
    A = x[(perm // K).long()].contiguous()
    W = _ints(g, (E, Kd, N), 1)
    sched = layer.grouped_schedule(off, E, R)
    ref = _product(A, off, W)
    for epi, want in ((0, ref), (1, ref.clamp(min=0) ** 2)):
        out = torch.full((R, N), 7.0, dtype=torch.bfloat16, device=DEV)
        u = torch.full((R, N), 7.0, dtype=torch.bfloat16, device=DEV) if epi else None
        L.moe_grouped_gemm(A, sched, E, R, Kd, N, W, epi, out, u)
        assert torch.equal(out, want.to(torch.bfloat16))
        if u is not None:
            assert torch.equal(u, ref.to(torch.bfloat16))
        got = torch.full_like(out, 7.0)
        L.moe_grouped_gemm_gather(x, perm, S, K, sched, E, R, Kd, N, W, epi, got, None)
        assert torch.equal(got, out)
    dy = _ints(g, (R, N), 1) * (torch.rand((R, N), generator=g, device=DEV) < 0.05)
    uu, W2 = _ints(g, (R, Kd), 2), _ints(g, (E, Kd, N), 1)   # an FFN of width Kd over N-wide rows
    W1 = _ints(g, (E, N, Kd), 1)
    dx, _, _ = layer.grouped_ffn_bwd(dy, uu, uu, dy, off, W1, W2)
    du = (_product(dy, off, W2.transpose(1, 2)) * 2 * uu.float().clamp(min=0)).to(torch.bfloat16)
    assert torch.equal(dx, _product(du, off, W1.transpose(1, 2)).to(torch.bfloat16))


@pytest.mark.parametrize("S,D,F", [(1, 8, 8), (33, 136, 264), (129, 72, 120), (1000, 264, 2680)])
@pytest.mark.parametrize("accumulate", [False, True])
def test_dense_fp32(S, D, F, accumulate):
    g = torch.Generator(device=DEV).manual_seed(S)
    x = _ints(g, (S, D), 1) * (torch.rand((S, D), generator=g, device=DEV) < 0.1)
    W1, W2 = _ints(g, (D, F), 1), _ints(g, (F, D), 1)
    h, u, y = layer.shared_expert_fwd(x, W1, W2)
    uf = x.float() @ W1.float()
    assert torch.equal(h, (uf.clamp(min=0) ** 2).to(torch.bfloat16)) and torch.equal(y, h.float() @ W2.float())
    dy = _ints(g, (S, D), 1) * (torch.rand((S, D), generator=g, device=DEV) < 0.05)
    dx = _ints(g, (S, D), 3).float()
    want = dx.clone() if accumulate else torch.zeros_like(dx)
    du = ((dy.float() @ W2.float().T) * 2 * u.float().clamp(min=0)).to(torch.bfloat16)
    got, _, _ = layer.shared_expert_bwd(x, u, h, dy, W1, W2, dx=dx, accumulate_dx=accumulate)
    assert torch.equal(got, want + du.float() @ W1.float().T)
