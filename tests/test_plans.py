"""Launch plans and workspace sizes, on the host.

Backward splits: more token splits cost a finishing launch and their fp32 sums, so a near tie in rounds stays with the
fewer. The shapes below were timed with every tile and split count; each entry names the plan that was fastest (241 us
with one split for 263 with four at 11,004 x 8,096 x 1,408)."""
import pytest

from host_plans import plan_bwd
from paper_2608_01847_amd import focus as F

F32, BF16 = F.F32, F.BF16
MX, NV = F.MXFP4, F.NVFP4


@pytest.mark.parametrize("fmt,sb,M,N,K,tile,splits", [
    (MX, 8, 11004, 8096, 1408, 256, 1), (MX, 8, 11592, 5808, 1920, 256, 1), (NV, 4, 16290, 7776, 8832, 256, 1),
    (MX, 8, 1535, 1936, 2144, 128, 1), (MX, 8, 1724, 19944, 1152, 256, 1), (MX, 8, 8260, 832, 17536, 256, 2),
    (MX, 8, 2048, 1024, 2560, 128, 3), (MX, 8, 131072, 8192, 28672, 256, 1), (NV, 8, 65536, 2560, 4096, 256, 3),
])
def test_backward_splits_are_worth_their_sums(fmt, sb, M, N, K, tile, splits):
    p = plan_bwd(BF16, fmt, sb, M, N, K)
    assert (p.path, p.tile, p.splits) == (1, tile, splits)


def test_backward_splits_of_a_large_fp32_layer():
    assert plan_bwd(F32, MX, 8, 65536, 9728, 2560).splits == 1
    assert F.workspace_size(F.CALL_RECON_GEMM_BWD, F.qconfig(MX, 8), 65536, 9728, 2560) == 256 + 2 * 9728 * (80 + 320) * 4
