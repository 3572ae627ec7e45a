"""The 256 x 256-tile kernels of the bf16 and packed MXFP4 products at ragged edges and at every remainder of their
three-step loops, and the launch rule's lines. Each case first asks the library's plan for its tile, so that a change of
the rule cannot take the case to another kernel unnoticed.

Forward: operands are FP4 grid values with unit scales, so every product and partial sum is a multiple of 1/4 below 2^22 and
exact in fp32 in any order: the plain product rounds once to bf16, D = Y_hat - Y_ref is exact, dY one product and one
rounding; the column sums of D^2 take 16 terms in fp32 (2^-20), the rest in fp64.

Backward: operands are small integers, so G = dY^T X is exact in fp32; the gradients are compared with the streaming
backward on that G, each within 33 roundings of 2^-24 of the sum of its terms' magnitudes, a last division or product adds
two and up to 8 token ranges (terms bounded through |dY|^T |X|) as many additions: 2 * 43 * 2^-24 times that sum. MXFP4's
gradients from packed operands have the bits of those from bf16 operands. Layers of fewer than about 600 tokens take the
small tiles, so a workgroup runs 21 steps of 32 tokens or more here.
"""
import pytest
import torch

from gpu_common import announce, require_gpu, to_k_slabs
from host_plans import fwd_tile_rows, plan_bwd
from test_gpu_gemm_small import operand

pytestmark = pytest.mark.gpu

MX, NV = 0, 1


@pytest.fixture(scope="module")
def F():
    return require_gpu()


# K: 3 to 7 bf16 steps of 32 (fewer than, as many as and more than the Y_ref steps), then 12, 16, 20 and 36; packed operands
# (K % 128 == 0) run 1 to 9 of 128. The last two shapes lie on either side of the MXFP4 rule's line of 512 small tiles.
@pytest.mark.parametrize("M,N,K", [(3004, 3080, k) for k in (96, 128, 160, 192, 224, 256, 384, 512, 640, 1152)] +
                         [(2820, 3208, 144), (2048, 4096, 128), (2048, 4104, 128)])
def test_forward_is_exact(F, M, N, K):
    small_tiles = -(-M // 128) * -(-N // 128)
    assert fwd_tile_rows(M, N, False) == 256 and fwd_tile_rows(M, N, True) == (128 if small_tiles <= 512 else 256)
    announce(f"large-tile forward {M}x{N}x{K}")
    g = torch.Generator().manual_seed(M + N + K)
    xc, X = operand(g, M, K)
    wc, W = operand(g, N, K)
    ref = X.cuda().double() @ W.cuda().double().t()
    Y = (torch.randint(-64, 65, (M, N), generator=g) * 0.25).cuda()
    D = ref - Y.double()
    scale = torch.tensor(2.0 / (M * N), dtype=torch.float64).float().cuda()
    calls = [("bf16", F.recon_gemm_fwd, (X.to(torch.bfloat16).cuda(), W.to(torch.bfloat16).cuda()))]
    if K % 128 == 0:
        ones = lambda r: torch.full((K // 32, r), 127, dtype=torch.uint8, device="cuda")
        calls.append(("mx", F.recon_gemm_fwd_mxfp4, (xc.cuda(), ones(M), to_k_slabs(wc).cuda(), ones(N))))
    for name, call, ops in calls:
        plain, _, _ = call(*ops)
        assert torch.equal(plain, ref.float().to(torch.bfloat16)), name
        dY, loss, col = call(*ops, Y.to(torch.bfloat16), want_col_sq=True)
        assert torch.equal(dY, (D.float() * scale).to(torch.bfloat16)), name
        want = (D * D).sum(0)
        assert bool(((col - want).abs() <= 2.0 ** -20 * want).all()), name
        assert abs(loss.item() - float(col.sum()) / (M * N)) <= 4e-15 * loss.item(), name


# One token range (the gradients written by the kernel): 21, 22, 23 whole steps of 32 tokens and 22 and 23 whole ones and a ragged
# one; then three ranges. N and K end inside a tile, N with fewer than 128 columns in it or more.
@pytest.mark.parametrize("M,N,K,splits", [(672, 4072, 4064, 1), (704, 4072, 4064, 1), (736, 3848, 4064, 1), (708, 4072, 3872, 1),
                                          (740, 4072, 4064, 1), (2460, 3680, 1056, 3), (2416, 1296, 2976, 3),
                                          (5076, 3000, 1664, 3)])
@pytest.mark.parametrize("fmt,sb,wdt", [(MX, 8, torch.bfloat16), (MX, None, torch.float32), (NV, 16, torch.bfloat16),
                                        (NV, 8, torch.float32)])
def test_backward_matches_streaming_backward(F, M, N, K, splits, fmt, sb, wdt):
    sub = sb or 8
    p = plan_bwd(F.BF16, fmt, sub, M, N, K)
    assert (p.path, p.tile, p.splits) == (1, 256, splits)
    announce(f"large-tile backward {M}x{N}x{K} fmt={fmt} sb={sb} {wdt}")
    g = torch.Generator(device="cuda").manual_seed(M * 7 + N + K)
    ints = lambda *shape: torch.randint(-3, 4, shape, generator=g, device="cuda").to(torch.bfloat16)
    dY, X = ints(M, N), ints(M, K)
    W = (torch.randn(N, K, generator=g, device="cuda") * 0.02).to(wdt)
    s, c, alpha = F.scales_init(W, fmt, sub)
    s = (s * torch.exp2(torch.rand(s.shape, generator=g, device="cuda") - 0.5)).contiguous()
    c = 0.75 + 0.5 * torch.rand(c.shape, generator=g, device="cuda")
    cc = c if sb else None
    G = torch.mm(dY.float().t().contiguous(), X.float())
    Ga = torch.mm(dY.float().abs().t().contiguous(), X.float().abs()).double()
    assert float(Ga.max()) < 2 ** 24
    gs, gc, _ = F.recon_gemm_bwd(dY, X, W, fmt, sub, s, cc, alpha)
    rs, rc = F.fakequant_bwd(G, W, fmt, sub, s, cc, alpha)
    block = 32 if fmt == MX else 16
    # |q - m u| <= 12 within the clip
    mag = Ga.view(N, -1, block).sum(2) * 12.0 * (float(alpha) if fmt == NV else 1.0)
    assert bool(((gs.double() - rs.double()).abs() <= 86 * 2.0 ** -24 * mag).all())
    mag = (Ga * W.double().abs()).view(N, -1, sub).sum(2) / (c.double() ** 2 if sb else 1.0)
    assert bool(((gc.double() - rc.double()).abs() <= 86 * 2.0 ** -24 * mag).all())
    if fmt == MX:
        x_hat, xc, xs, _ = F.fakequant_fwd(X, MX, 8, want_codes=True, want_scale_bytes=True, scale_layout=F.SCALES_BLOCK_MAJOR)
        ps, pc = F.recon_gemm_bwd_mxfp4(dY, xc, xs, W, sub, s, cc)
        bs, bc, _ = F.recon_gemm_bwd(dY, x_hat, W, MX, sub, s, cc, alpha)
        assert torch.equal(ps, bs) and torch.equal(pc, bc)
