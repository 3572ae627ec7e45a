"""Fake quantisation of fp32 weights on the E2M1 decision points, and the NVFP4 activation pass on both sides of the
size from which its tensor scale is folded by a launch of its own; all bit-exact.

fp32 weights: each sub-block places one weight whose quotient W / S_q (Eq. 7, 8) lies within +-3 units in the last place
of a rounding midpoint of E2M1 or of 6. Other rows leave the range of the reciprocal: non-finite, huge and subnormal
weights, scales outside [2^-40, 2^40], zero scales. Codes, scale bytes and W_hat against the oracle.
"""
import numpy as np
import pytest
import torch

from gpu_common import announce, assert_bits_equal, host_bits16, host_bits32, require_gpu

pytestmark = pytest.mark.gpu

POINTS = np.array([0.25, 0.75, 1.25, 1.75, 2.5, 3.5, 5.0, 6.0], np.float32)


def fp32_case(fmt, sb, N, K, seed):
    from oracle import focus_oracle as O
    rng = np.random.default_rng(seed)
    B = 32 if fmt == 0 else 16
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    if fmt == 0:
        alpha, s = 1.0, np.exp2(rng.integers(-9, -4, size=(N, K // B))).astype(np.float32)
        sdq = s
    else:
        alpha = float(np.float32(0.02 * 1.7 / 2688.0))
        s = rng.uniform(20.0, 440.0, size=(N, K // B)).astype(np.float32)
        sdq = O.fq_weight(np.zeros((N, K), np.float32), fmt, sb, s, np.ones((N, K // sb), np.float32), alpha).s_dq
    n, k = np.meshgrid(np.arange(N), np.arange(K // sb), indexing="ij")
    w = np.abs(W[n, k * sb + (5 * k + n) % sb])
    sq = (w / POINTS[(k + 3 * n) % len(POINTS)]).view(np.int32) + ((k + n) % 7 - 3).astype(np.int32)
    c = (sq.view(np.float32) / sdq[n, k * sb // B]).astype(np.float32)
    c[w < 1e-4] = 1.0
    W[0, 3], W[0, 70], W[1, 5], W[2, 9], W[3, 17] = np.inf, -np.inf, np.nan, 2.0 ** 90, -(2.0 ** 100)
    W[7, :64] = np.float32(-1e-42)
    c[4, :], c[5, :] = np.float32(2.0 ** -60), np.float32(2.0 ** 60)
    s[6, 0] = 0.0 if fmt == 1 else np.float32(2.0 ** -120)
    return W, s, c, alpha


@pytest.mark.parametrize("fmt,sb", [(0, 32), (0, 8), (0, 4), (1, 16), (1, 8), (1, 2)])
def test_fp32_weights_on_decision_points(fmt, sb):
    F = require_gpu()
    from oracle import focus_oracle as O
    N, K = 37, 416 if fmt == 0 else 400  # 1,924 / 1,850 chunks: a partly filled last workgroup and wave
    W, s, c, alpha = fp32_case(fmt, sb, N, K, seed=7 + 10 * fmt + sb)
    announce(f"fp32 weights fmt={fmt} sb={sb} {N}x{K}")
    Wd, sd, cd = (torch.from_numpy(a).cuda() for a in (W, s, c))
    ad = torch.tensor([alpha], dtype=torch.float32, device="cuda") if fmt == 1 else None
    for coeff, cg in ((c, cd), (np.ones_like(c), None)):
        fq = O.fq_weight(W, fmt, sb, s, coeff, alpha)
        for layout in (0, 1):
            w32, codes, sbytes, _ = F.fakequant_fwd(Wd, fmt, sb, sd, cg, ad, want_codes=True, want_scale_bytes=True,
                                                    scale_layout=layout)
            w16 = F.fakequant_fwd(Wd, fmt, sb, sd, cg, ad, out_dtype=torch.bfloat16)[0]
            torch.cuda.synchronize()
            ref_bytes = fq.scale_bytes if layout == 0 else np.ascontiguousarray(fq.scale_bytes.T)
            assert_bits_equal(codes.cpu().numpy(), O.pack_codes(fq.codes), f"codes (layout {layout})")
            assert_bits_equal(sbytes.cpu().numpy(), ref_bytes, f"scale bytes (layout {layout})")
            assert_bits_equal(host_bits32(w32), fq.w_hat.view(np.uint32), "W_hat fp32")
            assert_bits_equal(host_bits16(w16), O.bf16_bits(O.bf16_round(fq.w_hat)), "W_hat bf16")


# 2,048 workgroups fold the partial maxima themselves; one row of workgroups more, and a launch does it once
@pytest.mark.parametrize("dtype,rows,more", [(torch.bfloat16, 16384, 1), (torch.float32, 2048, 1), (torch.float32, 3, 0)])
@pytest.mark.parametrize("fill", ["normal", "zeros"])
def test_tensor_scale_is_the_same_on_both_sides_of_the_fold(dtype, rows, more, fill):
    F = require_gpu()
    announce(f"nvfp4 activations {dtype} {rows} and {rows + more} x 2048, {fill}")
    g = torch.Generator(device="cuda").manual_seed(rows)
    X = torch.zeros(rows + more, 2048, device="cuda", dtype=dtype)
    if fill == "normal":
        X.copy_(torch.randn(X.shape, generator=g, device="cuda"))
        X[rows // 2, 77] = -9.5
        X[rows:] *= 0.5
    a = F.fakequant_fwd(X, 1, want_codes=True, want_scale_bytes=True, want_alpha=True)
    b = F.fakequant_fwd(X[:rows].contiguous(), 1, want_codes=True, want_scale_bytes=True, want_alpha=True)
    for p, q in zip(a[:3], b[:3]):
        assert torch.equal(p[:rows], q)
    want = np.float32(9.5) / np.float32(2688.0) if fill == "normal" else np.float32(1.0)
    assert a[3].item() == want and b[3].item() == want
