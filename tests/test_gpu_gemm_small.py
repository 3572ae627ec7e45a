"""The 128 x 128-tile forward kernels (bf16 and packed MXFP4) at the edges of their tiles, steps and launch rule,
and the one-workgroup finishing sums at theirs (up to 4,096 partials, 1,024 columns and 16 tile rows).

Operands are FP4 grid values with unit scales, so every product and partial sum is a multiple of 1/4 below 2^22 and
exact in fp32 in any order: the plain product rounds once to bf16; D = Y_hat - Y_ref is exact, dY one product and one
rounding, and the column sums of D^2 are sums of multiples of 1/16 that stay below 2^24 of them per 16 terms, exact
in fp32 and fp64 here. The loss is compared with the fp64 mean to 4 roundings.
"""
import pytest
import torch

from gpu_common import announce, require_gpu, to_k_slabs

pytestmark = pytest.mark.gpu

GRID = torch.tensor([0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0])


@pytest.fixture(scope="module")
def F():
    return require_gpu()


def operand(g, rows, K):
    """Codes with a sign, and the values they stand for."""
    i = torch.randint(0, 8, (rows, K), generator=g)
    s = torch.randint(0, 2, (rows, K), generator=g)
    code = (i | (s << 3)).to(torch.uint8)
    return code[:, 0::2] | (code[:, 1::2] << 4), GRID[i] * (1.0 - 2.0 * s)


# M x N in 128 x 128 tiles: the sixth and seventh shapes lie on either side of bf16's line of 384 tiles, 16 x 24 = 384 and
# 16 x 25 = 400 (MXFP4's line of 512: test_gpu_large_tiles.py)
@pytest.mark.parametrize("M,N,K", [(4, 8, 128), (124, 136, 256), (128, 128, 384), (260, 120, 640), (1000, 264, 1152),
                                   (2048, 3072, 128), (2048, 3080, 128), (4, 1024, 128), (508, 1032, 128),
                                   # tile order: 5 rows of 9 and of 10 columns, 9 of 18 (groups of 5 and 4), 12 of 29
                                   (516, 1152, 128), (516, 1160, 128), (1036, 2184, 128), (1412, 3680, 256)])
def test_small_tiles_are_exact(F, M, N, K):
    announce(f"small-tile forward {M}x{N}x{K}")
    g = torch.Generator().manual_seed(M + N + K)
    xc, X = operand(g, M, K)
    wc, W = operand(g, N, K)
    ref = (X.cuda().double() @ W.cuda().double().t())
    Y = (torch.randint(-64, 65, (M, N), generator=g) * 0.25).cuda()
    D = ref - Y.double()
    ones = lambda r: torch.full((K // 32, r), 127, dtype=torch.uint8, device="cuda")
    packed = (xc.cuda(), ones(M), to_k_slabs(wc).cuda(), ones(N))
    full = (X.to(torch.bfloat16).cuda(), W.to(torch.bfloat16).cuda())
    scale = torch.tensor(2.0 / (M * N), dtype=torch.float64).float().cuda()
    for name, call, ops in (("mx", F.recon_gemm_fwd_mxfp4, packed), ("bf16", F.recon_gemm_fwd, full)):
        plain, _, _ = call(*ops)
        assert torch.equal(plain, ref.float().to(torch.bfloat16)), name
        dY, loss, col = call(*ops, Y.to(torch.bfloat16), want_col_sq=True)
        assert torch.equal(dY, (D.float() * scale).to(torch.bfloat16)), name
        want = (D * D).sum(0)
        assert bool(((col - want).abs() <= 2.0 ** -20 * want).all()), name  # 16-term fp32 sums
        assert abs(loss.item() - float(col.sum()) / (M * N)) <= 4e-15 * loss.item(), name
        dY2, loss2, _ = call(*ops, Y.to(torch.bfloat16))
        assert torch.equal(dY, dY2) and loss.item() == loss2.item(), name
