"""GELU and SwiGLU, forward and backward, over every bf16 value: the bf16 kernels, whether they call erff or read
it from a table, give the fp32 formula's value rounded once, no other formula; and that value is the
64-bit one to its rounding."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N = 65536


def same(got, want):
    """Equal bits, or NaN in both."""
    return bool(((got.view(torch.int16) == want.view(torch.int16)) | (got.isnan() & want.isnan())).all())


def test_every_bf16_value():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_18710_amd import binding as mb
    z = torch.arange(N, dtype=torch.int32).sub(32768).to(torch.int16).view(torch.bfloat16).cuda()
    g = torch.Generator(device="cuda").manual_seed(5)
    up, da = [(torch.rand(N, generator=g, device="cuda") * 1.5 + 0.5).to(torch.bfloat16) for _ in range(2)]
    gu = torch.cat([z.view(256, 256), up.view(256, 256)], dim=1).contiguous()
    got = {}
    for dtype, td in (("bf16", torch.bfloat16), ("f32", torch.float32)):
        z_, da_, gu_ = z.to(td), da.to(td), gu.to(td)
        a, dz, s, dgu = [torch.full_like(t, 7.0) for t in (z_, z_, da_, gu_)]
        mb.op_gelu_fwd(None, 256, dtype, N, z_, a)
        mb.op_gelu_bwd(None, 256, dtype, N, z_, da_, dz)
        mb.op_swiglu_fwd(None, 256, dtype, 256, 256, gu_, s)
        mb.op_swiglu_bwd(None, 256, dtype, 256, 256, gu_, da_, dgu)
        torch.cuda.synchronize()
        got[dtype] = dict(gelu=a, gelu_grad=dz, swiglu=s, d_gate=dgu[:, :256].reshape(-1), d_up=dgu[:, 256:].reshape(-1))
    for k in got["bf16"]:
        assert same(got["bf16"][k], got["f32"][k].to(torch.bfloat16)), k

    zd, ud, dd = [t.cpu().double() for t in (z, up, da)]
    cdf = 0.5 * torch.special.erfc(-zd / np.sqrt(2.0))
    pdf = torch.exp(-0.5 * zd * zd) / np.sqrt(2.0 * np.pi)
    sig = torch.sigmoid(zd)
    # half a unit of bf16's last place, 2^-8 of the value at most; what fp32 leaves of 1 + erf where it
    # cancels (two roundings of a number near 1, times the factor before it); results below bf16's normal range
    want = dict(gelu=(zd * cdf, zd.abs() * 2.0 ** -23), gelu_grad=(dd * (cdf + zd * pdf), dd * 2.0 ** -22),
                swiglu=(zd * sig * ud, 1e-36), d_gate=(dd * ud * sig * (1 + zd * (1 - sig)), dd * ud * 2.0 ** -20), d_up=(dd * zd * sig, 1e-36))
    for k, (ref, floor) in want.items():
        y = got["bf16"][k].cpu().double()
        sel = (zd.abs() < 1e30) & (zd.abs() >= 2.0 ** -100)
        assert bool(((y - ref).abs() <= ref.abs() * 2.0 ** -8 * 1.01 + floor)[sel].all()), k
    at = lambda v: int((zd == v).nonzero()[0])
    for k in ("gelu", "swiglu"):
        y = got["bf16"][k].cpu().double()
        assert y[at(float("inf"))] == float("inf") and y[at(0.0)] == 0.0 and bool(y[zd.isnan()].isnan().all()), k


@pytest.mark.parametrize("quota", [256, 1])
def test_every_finite_bf16_value_through_the_epilogue(quota):
    """The product of unit rows and a weight that holds every finite bf16 value, on one CU in 256-wide tiles, on
    the whole device in small ones that have a CU each: both epilogues read erf from a table."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_18710_amd import binding as mb
    T, k, n = 130, 128, 512
    w = torch.arange(N, dtype=torch.int32).sub(32768).to(torch.int16).view(torch.bfloat16).cuda().view(k, n)
    w = torch.where(w.isfinite(), w, torch.zeros_like(w)).contiguous()
    x = torch.zeros(T, k, dtype=torch.bfloat16, device="cuda")
    x[:k] = torch.eye(k, dtype=torch.bfloat16, device="cuda")
    z, a, want = [torch.full((T, n), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(3)]
    mb.op_linear_act_fwd(None, quota, "bf16", mb.GELU, T, k, n, x, w, None, z, a)
    mb.op_gelu_fwd(None, 256, "bf16", T * n, z, want)
    torch.cuda.synchronize()
    assert bool((z[:k] == w).all()) and bool((z[k:] == 0).all())
    assert same(a, want)
