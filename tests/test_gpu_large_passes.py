"""Byte-bound passes over tensors that are walked in order, one workgroup per block (from 64 MB on), or past the caches (from
256 MB on), and norms, whose grid is what the CUs hold at once: the same bits as in pieces that take neither road."""
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


def native(mb, q):
    """A share of the CUs: the stream masked to it, which is where its passes are walked in order."""
    if q == 256:
        return None
    mb.pool_reserve(q, 0, mb.STRIPED)
    return mb.pool_get(q, 0, mb.STRIPED).native


# the last block is partly past the end
@pytest.mark.parametrize("dtype,T,f,q", [("bf16", 1229, 5632, 256), ("bf16", 4099, 6568, 256), ("f32", 2051, 6572, 64)])
def test_swiglu(mb, dtype, T, f, q):
    gu, da = normal(dtype, T, 2 * f), normal(dtype, T, f)
    a, dgu = nan_like(da), nan_like(gu)
    torch.cuda.synchronize()
    mb.op_swiglu_fwd(native(mb, q), q, dtype, T, f, gu, a)
    mb.op_swiglu_bwd(native(mb, q), q, dtype, T, f, gu, da, dgu)
    a2, dgu2 = nan_like(da), nan_like(gu)
    for r in range(0, T, 256):
        n = min(256, T - r)
        mb.op_swiglu_fwd(None, 256, dtype, n, f, gu[r:], a2[r:])
        mb.op_swiglu_bwd(None, 256, dtype, n, f, gu[r:], da[r:], dgu2[r:])
    torch.cuda.synchronize()
    assert torch.equal(a, a2) and torch.equal(dgu, dgu2)


@pytest.mark.parametrize("dtype,norm,T,h,q", [("bf16", "layernorm", 40001, 1536, 64), ("f32", "layernorm", 3001, 2048, 64), ("bf16", "rmsnorm", 9001, 5120, 64),
                                              ("bf16", "layernorm", 8201, 4104, 256), ("bf16", "rmsnorm", 8201, 4104, 64), ("f32", "rmsnorm", 17003, 1028, 256)])
def test_norm_forward(mb, dtype, norm, T, h, q):
    x, gain, bias = normal(dtype, T, h), normal(dtype, h), normal(dtype, h, 1).reshape(-1)
    y, y2 = nan_like(x), nan_like(x)
    st, st2 = [torch.full((T, 2), float("nan"), device="cuda") for _ in range(2)]
    torch.cuda.synchronize()
    mb.op_norm_fwd(native(mb, q), q, dtype, norm, T, h, 1e-5, x, gain, bias, y, st)
    for r in range(0, T, 512):
        mb.op_norm_fwd(None, 256, dtype, norm, min(512, T - r), h, 1e-5, x[r:], gain, bias, y2[r:], st2[r:])
    torch.cuda.synchronize()
    assert torch.equal(y, y2) and torch.equal(st, st2)


# the sizes between which GELU's grid is chosen: in order from 64 MB, fp32 striding up to 100 MB and from 256 to 320
@pytest.mark.parametrize("dtype,megabytes,q", [("bf16", 65, 256), ("bf16", 65, 64), ("f32", 70, 256), ("f32", 120, 256), ("f32", 280, 256), ("f32", 330, 256),
                                               ("f32", 120, 64), ("f32", 280, 64)])
def test_gelu_forward(mb, dtype, megabytes, q):
    n = (megabytes << 20) // (4 if dtype == "bf16" else 8) + 1032            # the last block is partly past the end
    z = normal(dtype, n)
    a, a2 = nan_like(z), nan_like(z)
    torch.cuda.synchronize()
    mb.op_gelu_fwd(native(mb, q), q, dtype, n, z, a)
    for at in range(0, n, 1 << 22):
        mb.op_gelu_fwd(None, 256, dtype, min(1 << 22, n - at), z[at:], a2[at:])
    torch.cuda.synchronize()
    assert torch.equal(a, a2)


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


@pytest.mark.parametrize("op", ["norm", "gelu", "swiglu_fwd", "swiglu_bwd", "rope", "adamw"])
def test_the_quota_holds_without_a_mask(mb, op):
    """A quota of two CUs on a stream without a mask: sixteen workgroups, several times slower than the device, and the same bits."""
    T, f = 6000, 4096
    x, gu, g = normal("bf16", T, 3 * f), normal("bf16", T, 2 * f), normal("bf16", f)
    out, st, table = nan_like(x), torch.empty(T, 2, device="cuda"), torch.empty(mb.rope_table_bytes(T // 4, 128), dtype=torch.uint8, device="cuda")
    mb.op_rope_table(None, 256, T // 4, 128, 1e4, table)
    n = T * f
    m, v = torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")

    def run(s, q):
        if op == "norm": mb.op_norm_fwd(s, q, "bf16", "rmsnorm", 3 * T, f, 1e-5, x, g, None, out, st.new_empty(3 * T, 2))
        elif op == "gelu": mb.op_gelu_fwd(s, q, "bf16", 3 * n, x, out)
        elif op == "swiglu_fwd": mb.op_swiglu_fwd(s, q, "bf16", T, f, gu, out)
        elif op == "swiglu_bwd": mb.op_swiglu_bwd(s, q, "bf16", T, f, gu, x, out)
        elif op == "rope": out.copy_(x); mb.op_rope(s, q, "bf16", 4, T // 4, f // 128, 128, 1, out, table)
        else: out.copy_(x); m.zero_(); v.zero_(); mb.op_adamw(s, q, "bf16", n, out, gu, m, v, None, 1e-3, 0.9, 0.999, 1e-8, 0.01, 1)

    def timed(q):
        side = torch.cuda.Stream()
        with torch.cuda.stream(side):
            run(side.cuda_stream, q)
            torch.cuda.synchronize()
            a, b = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            a.record(); run(side.cuda_stream, q); b.record()
            torch.cuda.synchronize()
        return a.elapsed_time(b), out.clone()

    (whole, want), (share, got) = timed(256), timed(2)
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    assert share > 6 * whole, (op, share, whole)
