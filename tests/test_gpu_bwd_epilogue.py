"""The fused straight-through epilogue of the MFMA backward against the streaming backward
(focus_fakequant_bwd) on the same G: both read W, S_fp and c themselves, so only the sums differ.

The operands are small integers, so G = dY^T X is exact in fp32 whatever the order of its sums, and the
two calls differ by the order (and fused multiply-adds) of at most 32 products: each is within 33 roundings
of 2^-24 of the sum of its terms' magnitudes, and the last division or product adds two. Where the
tokens are split (up to 8 ranges here), the terms are those of each range's own G, whose magnitudes
|dY|^T |X| bounds, and the ranges' sums add up to 8 roundings, so the difference is below 2 * 43 * 2^-24
times the sum formed with |dY|^T |X|. Sizes lie at the edges of the 128 x 128 and 256 x 256 tiles (the last size takes the large ones), with one
token range (the gradients written by the kernel itself) and with several, at a ragged number of 32-token steps; scales inside the fast
division's range, outside it, and zero.
"""
import pytest
import torch

from gpu_common import announce, require_gpu

pytestmark = pytest.mark.gpu

MX, NV = 0, 1


@pytest.fixture(scope="module")
def F():
    return require_gpu()


@pytest.mark.parametrize("fmt,sb,wdt,clip,scale", [
    (MX, 8, torch.bfloat16, 1, "normal"), (MX, 2, torch.float32, 1, "normal"), (MX, 4, torch.bfloat16, 0, "normal"),
    (MX, 16, torch.float32, 1, "tiny"), (MX, 32, torch.bfloat16, 1, "huge"), (MX, None, torch.bfloat16, 1, "normal"),
    (NV, 8, torch.bfloat16, 1, "normal"), (NV, 16, torch.bfloat16, 0, "zero"), (NV, 4, torch.float32, 1, "zero"),
    (NV, 2, torch.bfloat16, 1, "normal"),
])
@pytest.mark.parametrize("M,N,K", [(20, 8, 32), (70, 256, 256), (36, 264, 544), (1040, 520, 288), (100, 136, 112 * 16),
                                   (5076, 3000, 1664)])
def test_epilogue_matches_streaming_backward(F, fmt, sb, wdt, clip, scale, M, N, K):
    announce(f"bwd epilogue fmt={fmt} sb={sb} {wdt} clip={clip} {scale} {M}x{N}x{K}")
    g = torch.Generator().manual_seed(M * 7 + N + K)
    dY = torch.randint(-3, 4, (M, N), generator=g).to(torch.bfloat16).cuda()
    X = torch.randint(-3, 4, (M, K), generator=g).to(torch.bfloat16).cuda()
    W = (torch.randn(N, K, generator=g) * 0.02).to(wdt).cuda()
    sub = sb or 8
    s, c, alpha = F.scales_init(W, fmt, sub)
    s = s * torch.exp2(torch.rand(s.shape, generator=g).cuda() - 0.5)
    c = (0.75 + 0.5 * torch.rand(c.shape, generator=g)).cuda()
    odd = (torch.rand(s.shape, generator=g) < 0.2).cuda()
    s = torch.where(odd, {"normal": s, "tiny": s * 2.0 ** -60, "huge": s * 2.0 ** 60, "zero": s * 0}[scale], s).contiguous()
    cc = c if sb else None
    gs, gc, _ = F.recon_gemm_bwd(dY, X, W, fmt, sub, s, cc, alpha, ste_clip=clip)
    G = torch.mm(dY.float().t().contiguous(), X.float())
    Ga = torch.mm(dY.float().abs().t().contiguous(), X.float().abs()).double()
    assert float(Ga.max()) < 2 ** 24
    rs, rc = F.fakequant_bwd(G, W, fmt, sub, s, cc, alpha, ste_clip=clip)
    torch.cuda.synchronize()
    block = 32 if fmt == MX else 16
    # |q - m u| <= 6 + |u|, |u| = |w| / S_q; the smallest S_q of a block bounds its elements' u
    if fmt == MX:
        sdq = torch.exp2(torch.ceil(torch.log2(s.double())))
    else:
        sdq = alpha.double() * s.clamp(0, 448).to(torch.float8_e4m3fn).double()
    low = sdq * 0.5 if sb else sdq
    u = (W.double().abs().view(N, -1, block) / low.clamp(min=1e-300)[..., None]).clamp(max=6.0 if clip else 1e300)
    u = torch.where(low[..., None] > 0, u, torch.zeros_like(u))
    mag = (Ga.view(N, -1, block) * (6.0 + u)).sum(2) * (float(alpha) if fmt == NV else 1.0)
    assert bool(((gs.double() - rs.double()).abs() <= 86 * 2.0 ** -24 * mag).all())
    mag = (Ga * W.double().abs()).view(N, -1, sub).sum(2) / (c.double() ** 2 if sb else 1.0)
    assert bool(((gc.double() - rc.double()).abs() <= 86 * 2.0 ** -24 * mag).all())
