"""Launch plans and workspace sizes, on the host.

Backward splits: more token splits cost a finishing launch and their fp32 sums, so a near tie in rounds stays with the
fewer. The shapes below were timed with every tile and split count; each entry names the plan that was fastest (241 us
with one split for 263 with four at 11,004 x 8,096 x 1,408).

Workspace sizes: each covers the plan of every operand type, and those of the forward and of the input gradient do not
fall as the tokens grow, so that a workspace for the largest batch serves the others."""
import math
import random

import pytest

from host_plans import fwd_finish_in_one, plan_bwd, plan_dx, plan_fwd
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


def _log(rng, lo, hi, multiple=1):
    return max(multiple, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / multiple)) * multiple)


def test_workspace_sizes_cover_the_plans_and_smaller_batches():
    rng = random.Random(11)
    for _ in range(3000):
        M, N, K = _log(rng, 1, 200000), _log(rng, 8, 40000, 8), _log(rng, 16, 30000, 16)
        less = _log(rng, 1, M)
        fmt, sb = rng.choice([(MX, 2), (MX, 8), (MX, 32), (NV, 2), (NV, 8), (NV, 16)])
        q = F.qconfig(fmt, sb)
        fwd, dx = F.workspace_size(F.CALL_RECON_GEMM_FWD, q, M, N, K), F.workspace_size(F.CALL_RECON_GEMM_DX, q, M, N, K)
        for m in (M, less):
            for dt in (F32, BF16):
                assert plan_fwd(dt, m, N, K).ws_bytes <= fwd, (dt, m, M, N, K)
                assert plan_dx(dt, m, N, K).ws_bytes <= dx, (dt, m, M, N, K)
            assert F.workspace_size(F.CALL_RECON_GEMM_FWD, q, m, N, K) <= fwd
            assert F.workspace_size(F.CALL_RECON_GEMM_DX, q, m, N, K) <= dx
        # 128 x 128 tiles of the packed MXFP4 forward, up to 512 of them
        if -(-M // 128) * -(-N // 128) <= 512:
            assert 256 + (-(-M // 128) + 1) * N * 8 <= fwd
        if K % (32 if fmt == MX else 16) == 0:
            bwd = F.workspace_size(F.CALL_RECON_GEMM_BWD, q, M, N, K)
            assert all(plan_bwd(dt, fmt, sb, M, N, K, g).ws_bytes <= bwd for dt in (F32, BF16) for g in (False, True))


@pytest.mark.parametrize("call,N,K,more,less", [
    (F.CALL_RECON_GEMM_DX, 4096, 1024, 16384, 4096), (F.CALL_RECON_GEMM_DX, 4096, 1024, 16384, 8192),
    (F.CALL_RECON_GEMM_DX, 672, 2400, 8316, 562), (F.CALL_RECON_GEMM_FWD, 1000, 512, 1000, 960),
    (F.CALL_RECON_GEMM_FWD, 5296, 192, 230, 146),
])
def test_workspace_of_the_larger_batch_serves_the_smaller(call, N, K, more, less):
    q = F.qconfig(MX, 8)
    assert F.workspace_size(call, q, less, N, K) <= F.workspace_size(call, q, more, N, K)


def test_input_gradient_splits_that_few_tiles_need():
    assert plan_dx(BF16, 4096, 32000, 2560).splits == 3
    assert plan_dx(BF16, 640, 31808, 1184).splits > 8
    assert plan_dx(BF16, 65536, 9728, 2560).splits == 1


def test_fp32_outputs_past_one_grid_take_the_two_dimensional_one():
    """2^24 tiles of 256 threads are 2^32 work-items, more than one launch dimension holds."""
    assert plan_fwd(F32, 1 << 21, (1 << 15) - 64, 16).path == 2
    assert plan_fwd(F32, 1 << 21, 1 << 15, 16).path == 0
    assert plan_bwd(F32, MX, 8, 1, 1 << 20, (1 << 16) - 64).path == 2
    assert plan_bwd(F32, MX, 8, 1, 1 << 20, 1 << 16).path == 0


def test_many_tile_rows_are_not_summed_by_one_workgroup():
    """30 us for 102 tile rows of 24 columns, 6 by the two kernels."""
    assert fwd_finish_in_one(4, 256) and fwd_finish_in_one(16, 256) and fwd_finish_in_one(4, 1024)
    assert not fwd_finish_in_one(102, 24) and not fwd_finish_in_one(17, 24) and not fwd_finish_in_one(5, 1024)
