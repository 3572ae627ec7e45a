"""KL-Top's sample-select path on rows of every alignment: odd vocabularies (each row starts at another
remainder of 16 bytes), tensors whose first elements lie at different remainders, rows with fewer than a
16-byte piece at either end, the shortest row of the path and one below it, segments of dZ that end inside a
row, ties at the cut, and the domain flag for a value that is not finite anywhere in the row.

Against the oracle (fp64); tolerances: dZ is one rounding to its type of a double (2^-9 for bf16 and 2^-24
for fp32, relative), the loss a double sum of k terms whose logarithms agree to 1e-12.
"""
import numpy as np
import pytest
import torch

from gpu_common import announce, assert_close, host_f32, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    return require_gpu()


@pytest.fixture(scope="module")
def C():
    from oracle import chain_oracle
    return chain_oracle


def at_offset(x, off):
    """x on the GPU, contiguous, its first element `off` elements past a 16-byte boundary."""
    buf = torch.empty(x.numel() + 16, dtype=x.dtype, device="cuda")
    v = buf[off:off + x.numel()].view(x.shape)
    v.copy_(x)
    return v


@pytest.mark.parametrize("T,V,k,dt,offs,ties", [
    (9, 8001, 300, torch.bfloat16, (0, 0, 0), False), (9, 8191, 200, torch.float32, (0, 0, 0), True),
    (3, 32000, 1000, torch.bfloat16, (3, 3, 3), False), (3, 12289, 500, torch.bfloat16, (1, 4, 7), True),
    (3, 12290, 500, torch.float32, (1, 2, 3), False), (2, 4096, 100, torch.bfloat16, (0, 0, 0), True),
    (2, 4095, 100, torch.bfloat16, (5, 5, 5), False), (2, 4103, 50, torch.float32, (0, 0, 1), False),
    (2, 4110, 1, torch.bfloat16, (0, 7, 0), False), (2, 65537, 1400, torch.bfloat16, (0, 0, 0), False),
    # the largest k that the sample takes at this length, and the passes past it
    (2, 32000, 1583, torch.bfloat16, (0, 0, 0), False), (2, 32000, 1584, torch.float32, (1, 0, 0), True),
    (2, 32000, 4000, torch.bfloat16, (0, 0, 0), True),
])
def test_rows_of_any_alignment(F, C, T, V, k, dt, offs, ties):
    announce(f"kl_top rows T={T} V={V} k={k} {dt} offsets={offs} ties={ties}")
    rng = np.random.default_rng(V + k)
    z = rng.normal(size=(T, V)) * 3.0
    z = np.round(z * 4.0) / 4.0 if ties else z
    Zt = torch.from_numpy(z).to(dt)
    Zs = (Zt.double() + torch.from_numpy(rng.normal(size=(T, V)))).to(dt)
    zs, zt = at_offset(Zs, offs[0]), at_offset(Zt, offs[1])
    guard = torch.full((T * V + 16,), 7.0, dtype=dt, device="cuda")
    out = guard[offs[2]:offs[2] + T * V].view(T, V)
    dZ, loss = F.kl_top(zs, zt, k, out=out)
    torch.cuda.synchronize()
    assert bool((guard[:offs[2]] == 7).all()) and bool((guard[offs[2] + T * V:] == 7).all())
    lo, dZo = C.kl_top(host_f32(Zs), host_f32(Zt), k)
    assert abs(loss.item() - lo) <= 1e-9 * lo
    assert_close(host_f32(dZ), dZo, 2.0 ** -23 if dt == torch.float32 else 2.0 ** -8, "dZ")
    assert not np.any((host_f32(dZ) != 0) & (dZo == 0)), "dZ nonzero off the teacher's top-k set"


@pytest.mark.parametrize("V", [1000, 8001])
@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("which,at,value", [("s", 0, float("nan")), ("s", 777, float("inf")), ("t", 999, float("-inf"))])
def test_values_that_are_not_finite_raise_the_flag(F, V, dt, which, at, value):
    announce(f"kl_top flag V={V} {dt} {which} {at} {value}")
    g = torch.Generator().manual_seed(V)
    zs, zt = torch.randn(2, V, generator=g).to(dt), torch.randn(2, V, generator=g).to(dt)
    ws = F.workspace(F.workspace_size(F.CALL_KL_TOP, F.qconfig(0, 8), 2, V, 0))
    F.kl_top(zs.cuda(), zt.cuda(), 50, ws=ws)
    assert F.check_flags(ws) == F.OK
    (zs if which == "s" else zt)[1, at] = value
    F.kl_top(zs.cuda(), zt.cuda(), 50, ws=ws)
    assert F.check_flags(ws) == F.ERR_DOMAIN


# A teacher's NaN has the highest key and is selected (with its sign set, the lowest, and is not), whichever way its row takes;
# rows beside it keep their results.
@pytest.mark.parametrize("V", [1000, 8001, 32000])
@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("at", [0, 501, 999])
def test_a_teacher_nan_shows_in_the_loss(F, V, dt, at):
    announce(f"kl_top teacher NaN V={V} {dt} at {at}")
    g = torch.Generator().manual_seed(V + at)
    zs, zt = torch.randn(3, V, generator=g).to(dt).cuda(), torch.randn(3, V, generator=g).to(dt).cuda()
    clean, _ = F.kl_top(zs, zt, 50)
    zt[1, at] = float("nan")
    dZ, loss = F.kl_top(zs, zt, 50)
    assert bool(torch.isnan(loss)) and bool(torch.isnan(dZ[1, at]))
    assert torch.equal(dZ[0], clean[0]) and torch.equal(dZ[2], clean[2])
    bits = torch.int16 if dt == torch.bfloat16 else torch.int32
    zt.view(bits)[1, at] |= -(1 << 15) if dt == torch.bfloat16 else -(1 << 31)
    dZ, loss = F.kl_top(zs, zt, 50)
    assert not bool(torch.isnan(loss)) and dZ[1, at].item() == 0.0
