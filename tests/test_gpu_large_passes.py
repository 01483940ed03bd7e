"""Byte-bound passes over tensors that are walked in order, one workgroup per block (from 64 MB on), or past the caches (from
256 MB on): the same bits as in pieces that take neither road."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_18710_amd import binding
    binding.lib()
    return binding


def normal(dtype, *shape):
    g = torch.Generator(device="cuda").manual_seed(sum(shape))
    return torch.randn(shape, generator=g, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32)


def nan_like(t):
    return torch.full_like(t, float("nan"))


# the last block is partly past the end
@pytest.mark.parametrize("dtype,T,f,q", [("bf16", 1229, 5632, 256), ("bf16", 4099, 6568, 256), ("f32", 2051, 6572, 64)])
def test_swiglu(mb, dtype, T, f, q):
    gu, da = normal(dtype, T, 2 * f), normal(dtype, T, f)
    a, dgu = nan_like(da), nan_like(gu)
    mb.op_swiglu_fwd(None, q, dtype, T, f, gu, a)
    mb.op_swiglu_bwd(None, q, dtype, T, f, gu, da, dgu)
    a2, dgu2 = nan_like(da), nan_like(gu)
    for r in range(0, T, 256):
        n = min(256, T - r)
        mb.op_swiglu_fwd(None, 256, dtype, n, f, gu[r:], a2[r:])
        mb.op_swiglu_bwd(None, 256, dtype, n, f, gu[r:], da[r:], dgu2[r:])
    torch.cuda.synchronize()
    assert torch.equal(a, a2) and torch.equal(dgu, dgu2)


@pytest.mark.parametrize("dtype,norm,T,h,q", [("bf16", "layernorm", 8201, 4104, 256), ("bf16", "rmsnorm", 8201, 4104, 64), ("f32", "rmsnorm", 17003, 1028, 256)])
def test_norm_forward(mb, dtype, norm, T, h, q):
    x, gain, bias = normal(dtype, T, h), normal(dtype, h), normal(dtype, h, 1).reshape(-1)
    y, y2 = nan_like(x), nan_like(x)
    st, st2 = [torch.full((T, 2), float("nan"), device="cuda") for _ in range(2)]
    mb.op_norm_fwd(None, q, dtype, norm, T, h, 1e-5, x, gain, bias, y, st)
    for r in range(0, T, 512):
        mb.op_norm_fwd(None, 256, dtype, norm, min(512, T - r), h, 1e-5, x[r:], gain, bias, y2[r:], st2[r:])
    torch.cuda.synchronize()
    assert torch.equal(y, y2) and torch.equal(st, st2)


def test_rotary(mb):
    B, N, H, d = 3, 1030, 48, 128
    x = normal("bf16", B * N, 3 * H * d)
    table = torch.empty(mb.rope_table_bytes(N, d), dtype=torch.uint8, device="cuda")
    mb.op_rope_table(None, 256, N, d, 10000.0, table)
    one = x.clone()
    mb.op_rope(None, 256, "bf16", B, N, H, d, 1, one, table)
    for b in range(B):
        mb.op_rope(None, 256, "bf16", 1, N, H, d, 1, x[b * N:], table)
    torch.cuda.synchronize()
    assert torch.equal(one, x)
