"""Column sums of D^2 and the loss where their loads run in several batches or end inside one: exact on integers (every
sum an integer below 2^53), the loss up to its final division."""
import pytest
import torch

from gpu_common import announce, require_gpu

pytestmark = pytest.mark.gpu


# rows of tiles (64 rows each) past one batch of 16 x 8 and inside it, columns past one batch of 256 x 8; 16 rows of tiles (32
# rows each), the most that one workgroup sums, and 17
@pytest.mark.parametrize("M,N", [(512, 24), (520, 24), (481, 256), (64 * 131 + 5, 24), (64 * 128, 1032), (64 * 17, 2309), (300, 4097), (1, 2048)])
def test_sums_are_exact_on_integers(M, N):
    F = require_gpu()
    announce(f"forward sums {M}x{N}")
    g = torch.Generator().manual_seed(M + N)
    X, W = torch.randint(-3, 4, (M, 16), generator=g).float(), torch.randint(-3, 4, (N, 16), generator=g).float()
    Y = torch.randint(-40, 41, (M, N), generator=g).float()
    D = X.double() @ W.double().t() - Y.double()
    _, loss, col = F.recon_gemm_fwd(X.cuda(), W.cuda(), Y.cuda(), want_col_sq=True)
    assert torch.equal(col.cpu(), (D * D).sum(0))
    assert abs(loss.item() - float((D * D).sum()) / (M * N)) <= 4e-16 * loss.item()
