"""Column sums of bias gradients: the order of their additions is a function of the shape, the same in the plain pass and in the
one that applies GELU's derivative, whatever the CUs and so the width of an access and the rows requested at once.
fp32, where the order shows in the bits: rows of a partition (8, or enough for 512 partitions) in ascending order, in four
quarters for long partitions of wide rows; then the partitions in eight slices."""
import pytest

from paper_2605_18710_amd import synth
from helpers import to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_18710_amd import binding
    return binding


def in_order(rows):                      # [..., rows, n] -> [..., n], one after the other
    acc = rows.new_zeros(rows.shape[:-2] + rows.shape[-1:])
    for i in range(rows.shape[-2]):
        acc = acc + rows[..., i, :]
    return acc


def partition_sum(x, quarters):
    if not quarters:
        return in_order(x)
    per = -(-x.shape[-2] // 4)
    return in_order(torch.stack([in_order(x[..., k * per:(k + 1) * per, :]) for k in range(4)], -2))


def column_sums(x):
    T, n = x.shape
    rp = max(8, -(-T // 512))
    whole, quarters = T // rp, rp >= 28 and n >= 2048
    parts = partition_sum(x[:whole * rp].view(whole, rp, n), quarters)
    if T % rp:
        parts = torch.cat([parts, partition_sum(x[whole * rp:], quarters)[None]])
    per = -(-parts.shape[0] // 8)
    return in_order(torch.stack([in_order(parts[s * per:(s + 1) * per]) for s in range(8)]))


# one row; partitions of 8 and a last one of 1 to 8; 9, 12 and 24 rows; one column tile partly past the width; both sides of the
# limits for quarters, with a last partition of 1, 2, 3 and 27 rows
SIZES = [(1, 8), (7, 72), (300, 260), (1568, 768), (4609, 1032), (6144, 256), (12000, 640), (13825, 2048), (13824, 2048), (14329, 2056), (14338, 2048), (14339, 2044),
         (14363, 2052)]
PLAIN = SIZES + [(16355, 4096)]           # quarters 128 KB apart: on many CUs by four waves


def same(a, b):
    return torch.equal(a.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("T,n", PLAIN)
def test_plain(mb, T, n):
    x, dy = to_dev(synth.normal(1200 + T, (T, 4)), "f32"), to_dev(synth.normal(1201 + T, (T, n)), "f32")
    dw, sc = torch.empty(4, n, device="cuda"), torch.empty(mb.linear_wgrad_scratch_bytes(T, 4, n), dtype=torch.uint8, device="cuda")
    ref = column_sums(dy)
    for q in (256, 24):
        db = torch.full((n,), float("nan"), device="cuda")
        mb.op_linear_wgrad(None, q, "f32", T, 4, n, x, dy, dw, db, sc)
        torch.cuda.synchronize()
        assert same(db, ref), q


@pytest.mark.parametrize("T,n", SIZES)
def test_with_gelu(mb, T, n):
    m = mb.Module(dict(kind="projector", batch=1, seq=T, in_dim=8, out_dim=n), "f32")
    m.params.copy_(torch.randn(m.params.numel(), generator=torch.Generator().manual_seed(T)).mul_(0.1))
    part = lambda buf, name: buf[m.tensors[name][0]:m.tensors[name][0] + m.tensors[name][1] * m.tensors[name][2]].view(m.tensors[name][1], -1).contiguous()
    e = lambda *sh: torch.full(sh, float("nan"), device="cuda")
    x, dy, y = to_dev(synth.normal(1300 + T, (T, 8)), "f32"), to_dev(synth.normal(1301 + T, (T, n)), "f32"), e(T, n)
    z, a, da, dz = e(T, n), e(T, n), e(T, n), e(T, n)
    mb.op_linear_act_fwd(None, 256, "f32", mb.GELU, T, 8, n, x, part(m.params, "w_1"), part(m.params, "b_1"), z, a)
    mb.op_linear_dgrad(None, 256, "f32", T, n, n, dy, part(m.params, "w_2"), None, da)
    mb.op_gelu_bwd(None, 256, "f32", T * n, z, da, dz)
    ref = column_sums(dz)
    for q in (256, 24):
        m.grads.fill_(float("nan"))
        m.step(q, None, x, y, dy=dy)
        torch.cuda.synchronize()
        assert same(part(m.grads, "b_1").reshape(-1), ref), q
        assert same(part(m.grads, "b_2").reshape(-1), column_sums(dy)), q
    m.destroy()


@pytest.mark.parametrize("B,lo,C,h", [(1, 1, 8, 8), (5, 1, 8, 64), (3, 37, 8, 264), (1, 600, 8, 128), (2, 3600, 8, 2048)])
def test_with_gelu_and_taps(mb, B, lo, C, h):
    """The gradient of a gathered input: row 2t takes tap 1 of output t, row 2t + 1 tap 2 of it and before that tap 0 of the next one."""
    m = mb.Module(dict(kind="conv_stem", batch=B, seq=lo, in_dim=C, hidden=h), "f32")
    m.params.copy_(torch.randn(m.params.numel(), generator=torch.Generator().manual_seed(lo)).mul_(0.1))
    part = lambda buf, name: buf[m.tensors[name][0]:m.tensors[name][0] + m.tensors[name][1] * m.tensors[name][2]].view(m.tensors[name][1], -1).contiguous()
    e = lambda *sh: torch.full(sh, float("nan"), device="cuda")
    T = B * lo
    x, dy, y = to_dev(synth.normal(1400 + lo, (2 * T, C)), "f32"), to_dev(synth.normal(1401 + lo, (T, h)), "f32"), e(T, h)

    def gathered(t, stride):             # [B, L, c] -> [B * (L / stride), 3 c]
        p = torch.nn.functional.pad(t, (0, 0, 1, 1))
        n = t.shape[1] // stride
        return torch.cat([p[:, i:i + stride * (n - 1) + 1:stride] for i in range(3)], dim=2).reshape(B * n, -1).contiguous()

    z1, a1, z2, a2 = e(2 * T, h), e(2 * T, h), e(T, h), e(T, h)
    mb.op_linear_act_fwd(None, 256, "f32", mb.GELU, 2 * T, 3 * C, h, gathered(x.view(B, 2 * lo, C), 1), part(m.params, "w_c1"), part(m.params, "b_c1"), z1, a1)
    mb.op_linear_act_fwd(None, 256, "f32", mb.GELU, T, 3 * h, h, gathered(a1.view(B, 2 * lo, h), 2), part(m.params, "w_c2"), part(m.params, "b_c2"), z2, a2)
    dz2, dp2, dz1 = e(T, h), e(T, 3 * h), e(2 * T, h)
    mb.op_gelu_bwd(None, 256, "f32", T * h, z2, dy, dz2)
    mb.op_linear_dgrad(None, 256, "f32", T, 3 * h, h, dz2, part(m.params, "w_c2"), None, dp2)
    taps = dp2.view(B, lo, 3, h)
    da1 = torch.stack([taps[:, :, 1], taps[:, :, 2]], dim=2)
    da1[:, :-1, 1] = taps[:, 1:, 0] + taps[:, :-1, 2]
    mb.op_gelu_bwd(None, 256, "f32", 2 * T * h, z1, da1.contiguous(), dz1)
    ref1, ref2 = column_sums(dz1), column_sums(dz2)
    for q in (256, 24):
        m.grads.fill_(float("nan"))
        m.step(q, None, x, y, dy=dy)
        torch.cuda.synchronize()
        assert same(part(m.grads, "b_c2").reshape(-1), ref2), q
        assert same(part(m.grads, "b_c1").reshape(-1), ref1), q
    m.destroy()


# sums that a later kernel takes along: encoders whose norms take them (one layer, and several: the top layer's and each layer's q|k|v bias), and
# rows too wide for the norms that do, where they get a launch of their own before dx is written, which may lie on the incoming gradient
@pytest.mark.parametrize("dtype,B,N,h,heads,f,L", [("f32", 1, 9, 64, 4, 96, 2), ("bf16", 2, 70, 256, 4, 512, 2), ("f32", 1, 6, 2052, 18, 64, 1)])
def test_sums_taken_along(mb, dtype, B, N, h, heads, f, L):
    m = mb.Module(dict(kind="encoder", batch=B, seq=N, hidden=h, heads=heads, mlp=f, layers=L, norm="layernorm", act="gelu", causal=0, bias=1, eps=1e-5), dtype)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    m.params.copy_(torch.randn(m.params.numel(), generator=torch.Generator().manual_seed(h)).mul_(0.05).to(td))
    x, dy = [to_dev(synth.normal(1500 + i + h, (B * N, h)), dtype) for i in range(2)]
    ref = column_sums(dy.float()).to(td)
    outs = []
    for q in (256, 24):
        y, grad = torch.empty_like(x), dy.clone()
        m.grads.fill_(float("nan"))
        m.step(q, None, x, y, dy=grad, dx=grad)            # dx over dy
        torch.cuda.synchronize()
        off, rows, cols = m.tensors["L%d.b_2" % (L - 1)]
        assert same(m.grads[off:off + rows * cols].float(), ref.float()), q
        grads = torch.cat([m.grads[o:o + r * c] for o, r, c in m.tensors.values()])
        assert not torch.isnan(grads.float()).any()
        outs.append((y, grad, grads))
    assert all(torch.equal(a, b) for a, b in zip(*outs))
    m.destroy()
