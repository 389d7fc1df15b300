"""The grouped GEMM's phased 256-row tile at the sizes where it can go wrong:
segments that end at and beside the edges of its 64-row wave blocks and its
128-row halves, contractions of two k tiles to several (whole and cut), widths
that end inside a wave's columns, gathered rows, every epilogue, and a
workgroup's tile list longer than its LDS table.

Inputs are small integers, so every product and sum is an exact integer in
fp32 (all below 2^24) and the bf16 rounding of the results is the only one:
the outputs are compared bit for bit.
"""
import pytest
import torch

from paper_2608_28511_amd import _lib as L
from paper_2608_28511_amd import layer

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# eight segments of 16 to 17 128-row tiles, ending at and beside the block edges
COUNTS = [2048 + r for r in (1, 63, 64, 65, 127, 128, 129, 191)]
MORE = [2048 + r for r in (0, 192, 193, 255, 16, 17, 240, 33)]


def _cdiv(a, b):
    return -(-a // b)


def phased(counts, N):
    """The launch's rule, restated: rounds of the phased tile x 1.35 < rounds of the 128-row tile."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    gx = cus // 8
    nt = _cdiv(N, 256)
    r = [_cdiv(_cdiv(sum(_cdiv(c, h) for c in counts), 8) * nt, gx) for h in (128, 256)]
    return r[1] * 135 < r[0] * 100


def _ints(g, shape, hi):
    return torch.randint(-hi, hi + 1, shape, generator=g, device=DEV).to(torch.bfloat16)


def _segments(counts):
    off = torch.zeros(len(counts) + 1, dtype=torch.int32)
    off[1:] = torch.tensor(counts).cumsum(0)
    return off.to(DEV)


def _product(A, off, W):
    o = off.tolist()
    return torch.cat([A[a:b].float() @ W[e].float() for e, (a, b) in enumerate(zip(o, o[1:]))])


@pytest.mark.parametrize("counts", [COUNTS, MORE], ids=["low_edges", "high_edges"])
@pytest.mark.parametrize("Kd,N", [(72, 264), (128, 512), (136, 264), (192, 520), (320, 328)])
def test_forward_epilogues_and_gather(counts, Kd, N):
    if not phased(counts, N):
        pytest.skip("this device keeps 128-row tiles for the shape")
    g = torch.Generator(device=DEV).manual_seed(Kd * 1000 + N)
    R, E, K = sum(counts), len(counts), 4
    R -= R % K
    counts = counts[:-1] + [counts[-1] - sum(counts) % K]
    off = _segments(counts)
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


@pytest.mark.parametrize("D,F", [(264, 328), (320, 264), (392, 520)])
def test_backward_products(D, F):
    """Both dgrads (k-major weights; the activation derivative fused) on the phased tile."""
    counts = COUNTS
    if not (phased(counts, D) and phased(counts, F)):
        pytest.skip("this device keeps 128-row tiles for the shape")
    g = torch.Generator(device=DEV).manual_seed(D * 1000 + F)
    R, E = sum(counts), len(counts)
    off = _segments(counts)
    W1, W2 = _ints(g, (E, D, F), 1), _ints(g, (E, F, D), 1)
    # sparse rows keep du and its products below 2^8 and 2^24
    dy = _ints(g, (R, D), 1) * (torch.rand((R, D), generator=g, device=DEV) < 0.05)
    u = _ints(g, (R, F), 2)
    x = _ints(g, (R, D), 1) * (torch.rand((R, D), generator=g, device=DEV) < 0.05)
    h = _ints(g, (R, F), 1)
    dx, dW1, dW2 = layer.grouped_ffn_bwd(x, u, h, dy, off, W1, W2)
    du = (_product(dy, off, W2.transpose(1, 2)) * 2 * u.float().clamp(min=0)).to(torch.bfloat16)
    assert torch.equal(dx, _product(du, off, W1.transpose(1, 2)).to(torch.bfloat16))
    o = off.tolist()
    for e, (a, b) in enumerate(zip(o, o[1:])):
        assert torch.equal(dW1[e], x[a:b].float().T @ du[a:b].float())
        assert torch.equal(dW2[e], h[a:b].float().T @ dy[a:b].float())


# rows per expert at and beside the edges of the 64-row k tiles, empty experts
# among them, twice over for a device's worth of items (and, in the last, one
# expert so busy that its items are cut across the XCDs)
WGRAD = [0, 1, 2, 63, 64, 65, 100, 127, 128, 129, 191, 192, 193, 0, 320, 7]


def wgrad_kernel(counts, D, F):
    """The pair launch's rule, restated."""
    cus, E = torch.cuda.get_device_properties(0).multi_processor_count, len(counts)
    items = [E * sum(_cdiv(m, h) * _cdiv(n, 256) for m, n in ((F, D), (D, F))) for h in (128, 256)]
    r = [_cdiv(i, cus) for i in items]
    if sum(counts) < 64 * E:
        if D % 16 or F % 16:
            return "phased" if items[1] > cus and E * D * F * 8 <= 220 << 20 else "small"
        return "tall" if items[1] >= cus else "small"
    if items[1] >= 2 * cus and r[1] * 152 < r[0] * 100:
        return "phased"
    return "tall" if items[1] >= 4 * cus else "small"


def _check_wgrads(counts, D, F):
    g = torch.Generator(device=DEV).manual_seed(D * 1000 + F)
    R, E = sum(counts), len(counts)
    off = _segments(counts)
    W1, W2 = _ints(g, (E, D, F), 1), _ints(g, (E, F, D), 1)
    dy = _ints(g, (R, D), 1) * (torch.rand((R, D), generator=g, device=DEV) < 0.05)
    u, x, h = _ints(g, (R, F), 2), _ints(g, (R, D), 1), _ints(g, (R, F), 1)
    for _ in range(2):   # a second call finds the first one's counters used up
        _, dW1, dW2 = layer.grouped_ffn_bwd(x, u, h, dy, off, W1, W2)
        du = (_product(dy, off, W2.transpose(1, 2)) * 2 * u.float().clamp(min=0)).to(torch.bfloat16)
        o = off.tolist()
        for e, (a, b) in enumerate(zip(o, o[1:])):
            assert torch.equal(dW1[e], x[a:b].float().T @ du[a:b].float()), e
            assert torch.equal(dW2[e], h[a:b].float().T @ dy[a:b].float()), e


@pytest.mark.parametrize("D,F", [(504, 512), (1000, 264), (760, 504)])
@pytest.mark.parametrize("heavy", [0, 4000])
def test_weight_gradients(D, F, heavy):
    """Both weight gradients on the phased tile: short, empty and busy contractions, cut widths."""
    counts = WGRAD * 4 + [heavy or 100]
    if wgrad_kernel(counts, D, F) != "phased":
        pytest.skip("this device keeps 128-row tiles for the shape")
    _check_wgrads(counts, D, F)


# the pair launch's item lists: heavy experts only, some heavy ones among light ones
# (whole items, and half-height ones where the busiest outlasts the rest), the
# kernel's largest expert table
@pytest.mark.parametrize("counts,D,F", [([250] * 8, 1032, 1800), ([700, 30, 600, 20, 650, 0, 500] + [40] * 9, 776, 1000),
                                        ([3000, 64, 2000, 1500, 0, 900] + [65] * 10, 776, 1000),
                                        ([0, 2500] + [70] * 30, 1000, 520), (WGRAD * 64, 520, 520)],
                         ids=["all_heavy", "four_heavy", "half_height", "one_half_height", "1024_experts"])
def test_weight_gradient_items(counts, D, F):
    if wgrad_kernel(counts, D, F) != "phased":
        pytest.skip("the shape is for 256 compute units")
    _check_wgrads(counts, D, F)


# fewer than 64 rows an expert: by the rows' alignment, the items and the gradients' size
@pytest.mark.parametrize("E,D,F,kernel", [(43, 528, 1040, "tall"), (90, 1008, 272, "tall"), (5, 528, 1040, "small"),
                                          (43, 520, 1032, "phased"), (5, 520, 1032, "small"), (40, 1000, 904, "small")])
def test_weight_gradients_of_few_rows(E, D, F, kernel):
    counts = ([0, 1, 2, 31, 32, 33, 63, 64, 65, 96, 97, 130] * 8)[:E]
    if wgrad_kernel(counts, D, F) != kernel:
        pytest.skip("the shape is for 256 compute units")
    _check_wgrads(counts, D, F)


# how the gradients leave: rows on cache lines, on 64-byte pieces, off them (held by
# the last-level cache, and larger), and rows on lines that start beside one
@pytest.mark.parametrize("E,D,F,shift", [(66, 768, 544, 0), (66, 528, 560, 0), (66, 520, 568, 0), (66, 712, 664, 0),
                                         (66, 768, 544, 4), (66, 768, 544, 16)])
def test_weight_gradient_stores(E, D, F, shift):
    counts = ([0, 64, 65, 130, 191, 64] * 11)[:E]
    if wgrad_kernel(counts, D, F) != "phased":
        pytest.skip("the shape is for 256 compute units")
    g = torch.Generator(device=DEV).manual_seed(D + F)
    R = sum(counts)
    off = _segments(counts)
    W1, W2 = _ints(g, (E, D, F), 1), _ints(g, (E, F, D), 1)
    dy = _ints(g, (R, D), 1) * (torch.rand((R, D), generator=g, device=DEV) < 0.05)
    u, x, h = _ints(g, (R, F), 2), _ints(g, (R, D), 1), _ints(g, (R, F), 1)
    ws = torch.empty(L.moe_grouped_ffn_bwd_workspace_bytes(E, R, D, F), dtype=torch.uint8, device=DEV)
    bufs = [torch.full((E * D * F + 32,), 7.0, device=DEV) for _ in range(2)]
    dW1, dW2 = (b[shift:shift + E * D * F].view(E, *s) for b, s in zip(bufs, ((D, F), (F, D))))
    dx = torch.empty((R, D), dtype=torch.bfloat16, device=DEV)
    L.moe_grouped_ffn_bwd(x, u, h, dy, off, E, R, D, F, W1, W2, dx, dW1, dW2, ws)
    du = (_product(dy, off, W2.transpose(1, 2)) * 2 * u.float().clamp(min=0)).to(torch.bfloat16)
    o = off.tolist()
    for e, (a, b) in enumerate(zip(o, o[1:])):
        assert torch.equal(dW1[e], x[a:b].float().T @ du[a:b].float()), e
        assert torch.equal(dW2[e], h[a:b].float().T @ dy[a:b].float()), e
    for b in bufs:
        assert (b[:shift] == 7).all() and (b[shift + E * D * F:] == 7).all()


@pytest.mark.parametrize("R", [0, 1, 64, 65, 130, 1000, 5000, 16384])
@pytest.mark.parametrize("M,N", [(8, 8), (72, 40), (264, 248), (1024, 776)])
def test_dense_weight_gradient(R, M, N):
    """Pieces of the contraction and their sum: none to 64 of them, the last ones short."""
    g = torch.Generator(device=DEV).manual_seed(R + M)
    x, dout, W = _ints(g, (R, M), 1), _ints(g, (R, N), 1), _ints(g, (M, N), 1)
    _, dW = layer.latent_proj_bwd(x, W, dout, want_dx=False)
    assert torch.equal(dW, x.float().T @ dout.float())


@pytest.mark.parametrize("shift", [0, 1])
def test_dense_weight_gradient_whole_tiles(shift):
    """More tiles than a device's round: whole ones, then pieces; dW aligned to 16 and to 4 bytes."""
    R, M, N = 520, 4112, 4104
    g = torch.Generator(device=DEV).manual_seed(3)
    x, dout, W = _ints(g, (R, M), 1), _ints(g, (R, N), 1), _ints(g, (M, N), 1)
    ws = torch.empty(L.moe_latent_proj_bwd_workspace_bytes(R, M, N), dtype=torch.uint8, device=DEV)
    buf = torch.full((M * N + 8,), 7.0, device=DEV)
    dW = buf[shift:shift + M * N].view(M, N)
    L.moe_latent_proj_bwd(x, W, dout, R, M, N, None, dW, ws)
    assert torch.equal(dW, x.float().T @ dout.float())
    assert (buf[:shift] == 7).all() and (buf[shift + M * N:] == 7).all()


@pytest.mark.parametrize("S,D,F", [(700, 264, 520), (3000, 2056, 4360)])
def test_dense_weight_gradient_pair(S, D, F):
    """The shared expert's two gradients in one launch, their tiles in one list."""
    g = torch.Generator(device=DEV).manual_seed(S)
    x, h, u = _ints(g, (S, D), 1), _ints(g, (S, F), 1), _ints(g, (S, F), 2)
    dy = _ints(g, (S, D), 1) * (torch.rand((S, D), generator=g, device=DEV) < 0.02)
    W1, W2 = _ints(g, (D, F), 1), _ints(g, (F, D), 1)
    _, dW1, dW2 = layer.shared_expert_bwd(x, u, h, dy, W1, W2, want_dx=False)
    du = ((dy.float() @ W2.float().T) * 2 * u.float().clamp(min=0)).to(torch.bfloat16)
    assert torch.equal(dW1, x.float().T @ du.float()) and torch.equal(dW2, h.float().T @ dy.float())


@pytest.mark.parametrize("accumulate", [False, True])
def test_fp32_outputs(accumulate):
    """The shared expert's fp32 products, forward and (with an addend) backward."""
    S, D, F = 16500, 264, 520
    if not phased([S], D) or not phased([S], F):
        pytest.skip("this device keeps 128-row tiles for the shape")
    g = torch.Generator(device=DEV).manual_seed(5)
    x = _ints(g, (S, D), 1) * (torch.rand((S, D), generator=g, device=DEV) < 0.05)
    W1, W2 = _ints(g, (D, F), 1), _ints(g, (F, D), 1)
    h, u, y = layer.shared_expert_fwd(x, W1, W2)
    uf = x.float() @ W1.float()
    assert torch.equal(u, uf.to(torch.bfloat16)) and torch.equal(h, (uf.clamp(min=0) ** 2).to(torch.bfloat16))
    assert torch.equal(y, h.float() @ W2.float())
    dy = _ints(g, (S, D), 1) * (torch.rand((S, D), generator=g, device=DEV) < 0.05)
    dx = _ints(g, (S, D), 3).float()
    want = dx.clone() if accumulate else torch.zeros_like(dx)
    du = ((dy.float() @ W2.float().T) * 2 * u.float().clamp(min=0)).to(torch.bfloat16)
    got, _, _ = layer.shared_expert_bwd(x, u, h, dy, W1, W2, dx=dx, accumulate_dx=accumulate)
    assert torch.equal(got, want + du.float() @ W1.float().T)


def test_long_tile_list():
    """More output tiles per workgroup than its LDS list holds (896): the list is refilled."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    Kd, N, M = 72, 8, 256 * (cus * 897 + 3) + 70
    g = torch.Generator(device=DEV).manual_seed(9)
    A = torch.empty((M, Kd), dtype=torch.bfloat16, device=DEV)
    step = 1 << 22
    for i in range(0, M, step):
        A[i:i + step] = _ints(g, (min(step, M - i), Kd), 1)
    W = _ints(g, (Kd, N), 1)
    out = layer.latent_proj(A, W)
    for i in range(0, M, step):
        assert torch.equal(out[i:i + step], (A[i:i + step].float() @ W.float()).to(torch.bfloat16)), i
