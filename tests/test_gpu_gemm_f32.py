"""The fp32 MFMA reconstruction GEMMs at the edges of their tiles, steps and launch rules.

Operands are small integers, so every product and every partial sum is an integer below 2^24 and exact in
fp32 in any order: the plain product, D = Y_hat - Y_ref and dY = fl(D * fl(2 / (M N))) must come out bit for
bit, the column sums of D^2 (fp64 integers below 2^53) too, and the loss up to its final division. The
backward's G is exact likewise; its straight-through sums are compared with the streaming backward's on that
G: each is within 33 roundings of 2^-24 of the sum of its terms' magnitudes, a last division or product adds
two and the split token ranges (at most 33 here, each with terms bounded through |dY|^T |X|) as many
additions, so the difference is below 2 * 68 * 2^-24 times that sum.
"""
import pytest
import torch

from gpu_common import announce, require_gpu

pytestmark = pytest.mark.gpu

MX, NV = 0, 1


@pytest.fixture(scope="module")
def F():
    return require_gpu()


def ints(g, *shape, lim=3):
    return torch.randint(-lim, lim + 1, shape, generator=g).float()


# the last two take 64 x 64 tiles (at least 256 of them), the others 32 x 32 with K split over the waves
@pytest.mark.parametrize("M,N,K", [(1, 1, 16), (31, 33, 48), (32, 32, 64), (33, 65, 80), (128, 256, 256), (100, 7, 1040),
                                   (1030, 1001, 16), (961, 1088, 528)])
def test_forward_is_exact_on_integers(F, M, N, K):
    announce(f"f32 forward {M}x{N}x{K}")
    g = torch.Generator().manual_seed(M + 3 * N + 5 * K)
    X, W = ints(g, M, K), ints(g, N, K)
    Y = ints(g, M, N, lim=40)
    ref = (X.double() @ W.double().t())
    plain, _, _ = F.recon_gemm_fwd(X.cuda(), W.cuda())
    assert torch.equal(plain.cpu().double(), ref)
    dY, loss, col = F.recon_gemm_fwd(X.cuda(), W.cuda(), Y.cuda(), want_col_sq=True)
    D = ref - Y.double()
    scale = torch.tensor(2.0 / (M * N), dtype=torch.float64).float()
    assert torch.equal(dY.cpu(), D.float() * scale)
    assert torch.equal(col.cpu(), (D * D).sum(0))
    assert abs(loss.item() - float((D * D).sum()) / (M * N)) <= 4e-16 * loss.item()


@pytest.mark.parametrize("M,N,K,fmt,sb,wdt,clip", [
    (1, 1, 32, MX, 8, torch.float32, 1), (31, 64, 64, MX, 4, torch.bfloat16, 1), (33, 65, 96, NV, 2, torch.float32, 1),
    (128, 256, 256, MX, 8, torch.float32, 1), (1037, 130, 208, NV, 16, torch.float32, 0), (70, 63, 160, MX, 32, torch.float32, 1),
    (64, 66, 64, MX, None, torch.float32, 0), (2050, 516, 528, NV, 8, torch.bfloat16, 1), (0, 5, 32, MX, 8, torch.float32, 1),
])
@pytest.mark.parametrize("want_G", [False, True])
def test_backward_matches_streaming_backward(F, M, N, K, fmt, sb, wdt, clip, want_G):
    announce(f"f32 backward {M}x{N}x{K} fmt={fmt} sb={sb} {wdt} clip={clip} G={want_G}")
    g = torch.Generator().manual_seed(M + 3 * N + 5 * K)
    dY, X = ints(g, M, N).cuda(), ints(g, M, K).cuda()
    W = (torch.randn(N, K, generator=g) * 0.02).to(wdt).cuda()
    sub = sb or 8
    s, c, alpha = F.scales_init(W, fmt, sub)
    s = (s * torch.exp2(torch.rand(s.shape, generator=g).cuda() - 0.5)).contiguous()
    c = (0.75 + 0.5 * torch.rand(c.shape, generator=g)).cuda()
    cc = c if sb else None
    gs, gc, G = F.recon_gemm_bwd(dY, X, W, fmt, sub, s, cc, alpha, ste_clip=clip, want_G=want_G)
    ref = torch.mm(dY.double().t().contiguous(), X.double())
    Ga = torch.mm(dY.double().abs().t().contiguous(), X.double().abs())
    if want_G:
        assert torch.equal(G.double(), ref)
    rs, rc = F.fakequant_bwd(ref.float().contiguous(), W, fmt, sub, s, cc, alpha, ste_clip=clip)
    torch.cuda.synchronize()
    block = 32 if fmt == MX else 16
    sdq = torch.exp2(torch.ceil(torch.log2(s.double()))) if fmt == MX else \
        alpha.double() * s.clamp(0, 448).to(torch.float8_e4m3fn).double()
    u = (W.double().abs().view(N, -1, block) / (sdq * (0.5 if sb else 1.0)).clamp(min=1e-300)[..., None])
    mag = (Ga.view(N, -1, block) * (6.0 + u)).sum(2) * (float(alpha) if fmt == NV else 1.0)
    assert bool(((gs.double() - rs.double()).abs() <= 136 * 2.0 ** -24 * mag).all())
    mag = (Ga * W.double().abs()).view(N, -1, sub).sum(2) / (c.double() ** 2 if sb else 1.0)
    assert bool(((gc.double() - rc.double()).abs() <= 136 * 2.0 ** -24 * mag).all())


# One token's products of 2^26 and ones from all others, in every element of G: the large term's chain of 64 tokens loses up to
# 63 of its ones, the others are integers below 2^24, and G is rounded once to multiples of 8. A single chain loses them all.
@pytest.mark.parametrize("M,N,K,first", [(4096, 64, 64, 0), (4096, 130, 80, 2000), (4129, 65, 96, 33), (190, 64, 64, 130),
                                         (224, 33, 64, 100)])
def test_backward_sums_tokens_in_short_chains(F, M, N, K, first):
    announce(f"f32 backward chains {M}x{N}x{K} large term at {first}")
    dY, X = torch.ones(M, N, device="cuda"), torch.ones(M, K, device="cuda")
    dY[first], X[first] = 2.0 ** 13, 2.0 ** 13
    W = torch.full((N, K), 0.5, device="cuda")
    s, c, alpha = F.scales_init(W, NV, 8)
    _, _, G = F.recon_gemm_bwd(dY, X, W, NV, 8, s, c, alpha, want_G=True)
    assert float((G.double() - (2.0 ** 26 + M - 1)).abs().max()) <= 63 + 4


# Rows whose tiles pass 2^31 bytes take the kernels without buffer offsets. Operands of -1, 0 and 1: the partial sums stay far
# below 2^24.
def test_rows_past_the_buffer_range(F):
    from host_plans import plan_bwd, plan_fwd
    M, N, K = 2, 3, (1 << 23) + 16
    assert plan_fwd(F.F32, M, N, K).path == 0 and plan_bwd(F.F32, NV, 16, M, 1, 2 * K).path == 0
    announce(f"f32 forward {M}x{N}x{K}, backward {M}x1x{2 * K}")
    g = torch.Generator(device="cuda").manual_seed(3)
    def unit(*shape):
        return torch.randint(-1, 2, shape, generator=g, device="cuda").float()
    X, W, Y = unit(M, K), unit(N, K), unit(M, N)
    dY, loss, _ = F.recon_gemm_fwd(X, W, Y)
    D = (X.double() @ W.double().t()) - Y.double()
    scale = torch.tensor(2.0 / (M * N), dtype=torch.float64).float().cuda()
    assert torch.equal(dY, D.float() * scale) and abs(loss.item() - float((D * D).sum()) / (M * N)) <= 4e-15 * loss.item()
    K *= 2
    dY, X, W = unit(M, 1), unit(M, K), torch.randn(1, K, generator=g, device="cuda") * 0.02
    s, c, alpha = F.scales_init(W, NV, 16)
    gs, gc, _ = F.recon_gemm_bwd(dY, X, W, NV, 16, s, c, alpha)
    G = (dY.t() @ X).contiguous()
    rs, rc = F.fakequant_bwd(G, W, NV, 16, s, c, alpha)
    mag = (G.abs().view(-1, 16) * 12.0).sum(1) * float(alpha)  # |q - m u| <= 12; 16 terms in either order and a product
    assert bool(((gs - rs).abs().view(-1) <= 34 * 2.0 ** -24 * mag).all())
    mag = (G.abs() * W.abs()).view(-1, 16).sum(1)
    assert bool(((gc - rc).abs().view(-1) <= 36 * 2.0 ** -24 * mag).all())
