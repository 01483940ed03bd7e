"""fp32 contractions and attention at the sizes where their tiles can go wrong: one row, one past a
block of 16, a tile of 32 or 64 and a K-tile of 64, products on both sides of the tile rule (512 tiles of
64 x 64), widths that allow no 4-element access, every head-size class, grouped heads, bf16
shapes that the bf16 kernels do not take, tensors off a 16-byte boundary."""
import numpy as np
import pytest

from oracle import layers as O
from paper_2605_18710_amd import synth
from helpers import quantize, quantize_tree, to_dev, from_dev, assert_close, layer_params, load_layer_params

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_18710_amd import binding
    binding.lib()
    return binding


def off(a, dtype, offset):
    t = to_dev(a, dtype)
    out = torch.empty(t.numel() + offset, dtype=t.dtype, device="cuda")
    out[offset:] = t.reshape(-1)
    return out[offset:].view(t.shape)


def bits(t):
    return t.view(torch.uint8)


@pytest.mark.parametrize("dtype,T,k,n,offset", [
    ("f32", 1, 4, 4, 0), ("f32", 33, 64, 32, 0), ("f32", 32, 68, 36, 0), ("f32", 65, 128, 100, 0), ("f32", 7, 5, 3, 0),
    ("f32", 31, 63, 65, 0), ("f32", 40, 32, 32, 1), ("f32", 1408, 60, 1472, 0), ("f32", 1408, 60, 1476, 0), ("f32", 2, 1500, 8, 0),
    ("bf16", 33, 12, 20, 0), ("bf16", 65, 30, 7, 0), ("bf16", 64, 64, 64, 1), ("bf16", 100, 588, 36, 0)])
def test_linear(mb, dtype, T, k, n, offset):
    s = 6100 + T + k + n
    X, W, b, R, dY = [quantize(synth.normal(s + i, sh, 0, sd), dtype) for i, (sh, sd) in
                      enumerate([((T, k), 1), ((k, n), 0.05), ((n,), 0.1), ((T, n), 1), ((T, n), 1)])]
    X_, W_, b_, R_, dY_ = [off(a, dtype, offset) for a in (X, W, b, R, dY)]
    Rx = quantize(synth.normal(s + 9, (T, k)), dtype)
    Rx_ = off(Rx, dtype, offset)
    outs = []
    for q in (256, 24):
        Y, dX, dW, db = [off(np.full(sh, np.nan), dtype, offset) for sh in ((T, n), (T, k), (k, n), (n,))]
        sc = torch.empty(max(16, mb.linear_wgrad_scratch_bytes(T, k, n)), dtype=torch.uint8, device="cuda")
        mb.op_linear_fwd(None, q, dtype, T, k, n, X_, W_, b_, R_, Y)
        mb.op_linear_dgrad(None, q, dtype, T, k, n, dY_, W_, Rx_, dX)
        mb.op_linear_wgrad(None, q, dtype, T, k, n, X_, dY_, dW, None, sc)
        torch.cuda.synchronize()
        outs.append((Y, dX, dW))
    dx_ref, dw_ref, _ = O.linear_bwd(X, W, dY)
    assert_close(from_dev(Y), O.linear_fwd(X, W, b) + R, dtype, "Y")
    assert_close(from_dev(dX), dx_ref + Rx, dtype, "dX")
    assert_close(from_dev(dW), dw_ref, dtype, "dW")
    assert all(torch.equal(bits(a), bits(c)) for a, c in zip(*outs))


# the activation on an input of the product, or Z itself: several tile columns, k == n (GELU) and n == 2k (SwiGLU)
@pytest.mark.parametrize("act,T,h,on", [(a, *c) for a in ("gelu", "swiglu") for c in ((96, 160, "X"), (300, 128, "X"), (40, 64, "W"), (64, 64, "bias"))] +
                         [("gelu", 33, 96, "Z")])
def test_activation_on_an_input(mb, act, T, h, on):
    n, code = (h, mb.GELU) if act == "gelu" else (2 * h, mb.SWIGLU)
    rnd = lambda i, *sh: to_dev(synth.normal(6200 + T + i, sh, 0, 0.3), "f32")
    X, W, b, Z = rnd(0, T, h), rnd(1, h, n), rnd(2, max(n, T * h)), torch.full((T, n), float("nan"), device="cuda")
    want_z, want_a = torch.full_like(Z, float("nan")), torch.full((T, h), float("nan"), device="cuda")
    mb.op_linear_act_fwd(None, 256, "f32", code, T, h, n, X.clone(), W.clone(), b.clone(), want_z, want_a)
    A = {"X": X, "W": W, "Z": Z, "bias": b}[on]
    mb.op_linear_act_fwd(None, 256, "f32", code, T, h, n, X, W, b, Z, A)
    torch.cuda.synchronize()
    assert torch.equal(bits(A.reshape(-1)[:T * h]), bits(want_a.reshape(-1)))
    assert on == "Z" or torch.equal(bits(Z), bits(want_z))


@pytest.mark.parametrize("dtype,B,N,H,Hkv,d,causal,offset", [
    ("f32", 1, 1, 1, 1, 4, 1, 0), ("f32", 2, 16, 2, 1, 16, 1, 0), ("f32", 1, 17, 4, 2, 20, 0, 0), ("f32", 2, 33, 2, 2, 32, 1, 0),
    ("f32", 1, 100, 6, 2, 64, 0, 0), ("f32", 1, 65, 2, 2, 128, 1, 0), ("f32", 2, 31, 3, 1, 5, 0, 0), ("f32", 1, 48, 2, 2, 80, 1, 0),
    ("f32", 1, 40, 2, 1, 32, 1, 1), ("bf16", 2, 50, 4, 2, 32, 1, 0), ("bf16", 1, 37, 2, 2, 80, 0, 0), ("bf16", 1, 37, 2, 2, 13, 1, 0),
    ("bf16", 1, 64, 2, 2, 64, 1, 1)])
def test_attention(mb, dtype, B, N, H, Hkv, d, causal, offset):
    w, s = (H + 2 * Hkv) * d, 6300 + N + d
    qkv, dO = quantize(synth.normal(s, (B * N, w)), dtype), quantize(synth.normal(s + 1, (B * N, H * d)), dtype)
    qkv_, dO_ = off(qkv, dtype, offset), off(dO, dtype, offset)
    outs = []
    for q in (256, 24):
        Oo, dq = off(np.full((B * N, H * d), np.nan), dtype, offset), off(np.full((B * N, w), np.nan), dtype, offset)
        lse, delta = [torch.full((B, H, N), float("nan"), device="cuda") for _ in range(2)]
        mb.op_attention_gqa_fwd(None, q, dtype, B, N, H, Hkv, d, causal, qkv_, Oo, lse)
        mb.op_attention_gqa_bwd(None, q, dtype, B, N, H, Hkv, d, causal, qkv_, Oo, lse, dO_, dq, delta)
        torch.cuda.synchronize()
        outs.append((Oo, lse, dq))
    assert_close(from_dev(Oo), O.attention_fwd(qkv, B, N, H, causal, Hkv), dtype, "O", roundings=2)
    assert_close(from_dev(lse), O.attention_lse(qkv, B, N, H, causal, Hkv), "f32", "lse", roundings=4)
    if N > 1:          # over one key dS vanishes: only its rounding would be compared
        assert_close(from_dev(dq), O.attention_bwd(qkv, dO, B, N, H, causal, Hkv), dtype, "dqkv", roundings=8)
    assert all(torch.equal(bits(a), bits(c)) for a, c in zip(*outs))


@pytest.mark.parametrize("B,N,H,Hkv,d,causal", [(2, 128, 4, 4, 32, 1), (1, 33, 4, 2, 16, 0), (2, 17, 2, 1, 64, 1), (1, 1, 2, 2, 4, 0), (1, 100, 3, 3, 28, 1)])
def test_attention_backward_in_one_launch_has_the_bits_of_two(mb, B, N, H, Hkv, d, causal):
    """dQ and dK/dV share a launch where every tile of 16 rows has a wave slot (256 CUs) and dK/dV then forms the row
    sums of dO O itself; with one CU they are two launches.  The gradients and the row sums must not show which."""
    w = (H + 2 * Hkv) * d
    qkv, dO = [to_dev(synth.normal(900 + N + i, (B * N, n)), "f32") for i, n in enumerate((w, H * d))]
    outs = []
    for q in (256, 1):
        Oo, dqkv = [torch.full((B * N, n), float("nan"), device="cuda") for n in (H * d, w)]
        lse, delta = [torch.full((B, H, N), float("nan"), device="cuda") for _ in range(2)]
        mb.op_attention_gqa_fwd(None, q, "f32", B, N, H, Hkv, d, causal, qkv, Oo, lse)
        mb.op_attention_gqa_bwd(None, q, "f32", B, N, H, Hkv, d, causal, qkv, Oo, lse, dO, dqkv, delta)
        torch.cuda.synchronize()
        outs.append([bits(dqkv), bits(delta)])
    assert not torch.isnan(outs[0][0].view(torch.float32)).any()
    assert all(torch.equal(a, b) for a, b in zip(*outs))


# one step of keys more than one wave takes, waves without a key, the most items that four waves share and one tile more, grouped heads
@pytest.mark.parametrize("B,N,H,Hkv,d,causal", [(1, 33, 2, 1, 32, 1), (1, 33, 2, 2, 64, 0), (1, 49, 2, 1, 16, 1), (2, 128, 16, 4, 16, 1), (2, 129, 16, 4, 16, 1),
                                                (1, 250, 3, 1, 60, 0)])
def test_attention_items_of_four_waves(mb, B, N, H, Hkv, d, causal):
    test_attention(mb, "f32", B, N, H, Hkv, d, causal, 0)
    if d % 16 == 0:
        test_attention_backward_in_one_launch_has_the_bits_of_two(mb, B, N, H, Hkv, d, causal)


@pytest.mark.parametrize("B,N,H,Hkv,d,causal", [(1, 33, 2, 1, 32, 1), (1, 48, 4, 4, 64, 0), (2, 100, 4, 2, 60, 1), (1, 257, 3, 3, 16, 1), (1, 250, 3, 1, 28, 0),
                                                (2, 256, 8, 8, 32, 1), (1, 64, 64, 64, 16, 0)])
def test_attention_four_sums_by_four_waves_or_one(mb, B, N, H, Hkv, d, causal):
    """The share of the CUs decides whether four waves form an item's four sums or one: the bits must not show which."""
    w = (H + 2 * Hkv) * d
    qkv, dO = [to_dev(synth.normal(1000 + N + i, (B * N, n)), "f32") for i, n in enumerate((w, H * d))]
    first = None
    for q in (256, 128, 64, 32, 16, 8, 1):
        Oo, dqkv = [torch.full((B * N, n), float("nan"), device="cuda") for n in (H * d, w)]
        lse, delta = [torch.full((B, H, N), float("nan"), device="cuda") for _ in range(2)]
        mb.op_attention_gqa_fwd(None, q, "f32", B, N, H, Hkv, d, causal, qkv, Oo, lse)
        mb.op_attention_gqa_bwd(None, q, "f32", B, N, H, Hkv, d, causal, qkv, Oo, lse, dO, dqkv, delta)
        torch.cuda.synchronize()
        got = [bits(t) for t in (Oo, lse, dqkv, delta)]
        first = first or got
        assert all(torch.equal(a, b) for a, b in zip(got, first)), q


@pytest.mark.parametrize("q", [256, 2])
@pytest.mark.parametrize("d", [32, 64])
def test_attention_non_finite_scores(mb, d, q):
    """NaN in a query row, and in all keys of one of the four waves: O and the log-sum-exp of the rows that see them are NaN, the
    others untouched.  Scores of -inf in all keys of one wave: those keys have no weight."""
    B, N, H, step, cus = 1, 128, 2, 32 if d == 32 else 16, q          # 2 CUs: one wave forms the four sums
    def run(q, k, v, causal):
        qkv = to_dev(np.concatenate([q, k, v], 1), "f32")
        Oo, lse = torch.empty(N, H * d, device="cuda"), torch.empty(B, H, N, device="cuda")
        mb.op_attention_fwd(None, cus, "f32", B, N, H, d, causal, qkv, Oo, lse)
        torch.cuda.synchronize()
        return from_dev(Oo).reshape(N, H, d), from_dev(lse)[0]
    q, k, v = [synth.normal(6400 + d + i, (N, H * d)) for i in range(3)]
    base_o, base_l = run(q, k, v, 1)
    bad = q.copy()
    bad[37, :d] = np.nan                                   # head 0
    o, l = run(bad, k, v, 1)
    assert np.isnan(l[0, 37]) and np.isnan(o[37, 0]).all()
    o[37, 0], l[0, 37] = base_o[37, 0], base_l[0, 37]
    assert np.array_equal(o, base_o) and np.array_equal(l, base_l)
    bad = k.copy()
    for j in range(step, N, 4 * step):                     # the second wave's steps
        bad[j:j + step] = np.nan
    o, l = run(q, bad, v, 1)
    assert np.isnan(l[:, step:]).all() and np.isnan(o[step:]).all()
    assert np.array_equal(o[:step], base_o[:step]) and np.array_equal(l[:, :step], base_l[:, :step])
    q, k = 1e20 * (0.5 + np.abs(q)), 1e-20 * k
    for j in range(step, N, 4 * step):
        k[j:j + step] = -1e20
    o, l = run(q, k, v, 0)
    qkv = quantize(np.concatenate([q, k, v], 1), "f32")
    assert_close(o.reshape(N, -1), O.attention_fwd(qkv, B, N, H, 0, H), "f32", "O", roundings=2)
    assert_close(l, O.attention_lse(qkv, B, N, H, 0, H)[0], "f32", "lse", roundings=4)


@pytest.mark.parametrize("T,k,n", [(1, 4, 4), (33, 64, 36), (256, 128, 384), (31, 132, 68), (300, 36, 8)])
def test_backward_products_in_one_launch_have_the_bits_of_two(mb, T, k, n):
    """A module takes the input and the weight gradient of a linear layer in one launch, the entry points one each."""
    m = mb.Module(dict(kind="projector", batch=1, seq=T, in_dim=k, out_dim=n), "f32")
    m.params.copy_(torch.randn(m.params.numel(), generator=torch.Generator().manual_seed(T)).mul_(0.1))
    x, dy = to_dev(synth.normal(950 + T, (T, k)), "f32"), to_dev(synth.normal(951 + T, (T, n)), "f32")
    y, dx = torch.full_like(dy, float("nan")), torch.full_like(x, float("nan"))
    m.grads.fill_(float("nan"))
    m.step(256, None, x, y, dy=dy, dx=dx)
    part = lambda buf, name: buf[m.tensors[name][0]:m.tensors[name][0] + m.tensors[name][1] * m.tensors[name][2]].view(m.tensors[name][1], -1)
    e = lambda *sh: torch.full(sh, float("nan"), device="cuda")
    sc = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    z, a, da, dz, dx2, dw1, dw2 = e(T, n), e(T, n), e(T, n), e(T, n), e(T, k), e(k, n), e(n, n)
    mb.op_linear_act_fwd(None, 256, "f32", mb.GELU, T, k, n, x, part(m.params, "w_1").contiguous(), part(m.params, "b_1").contiguous(), z, a)
    mb.op_linear_dgrad(None, 256, "f32", T, n, n, dy, part(m.params, "w_2").contiguous(), None, da)
    mb.op_linear_wgrad(None, 256, "f32", T, n, n, a, dy, dw2, None, sc)
    mb.op_gelu_bwd(None, 256, "f32", T * n, z, da, dz)
    mb.op_linear_dgrad(None, 256, "f32", T, k, n, dz, part(m.params, "w_1").contiguous(), None, dx2)
    mb.op_linear_wgrad(None, 256, "f32", T, k, n, x, dz, dw1, None, sc)
    torch.cuda.synchronize()
    for name, got, want in (("dx", dx, dx2), ("w_1", part(m.grads, "w_1"), dw1), ("w_2", part(m.grads, "w_2"), dw2)):
        assert torch.equal(bits(got.contiguous()), bits(want)), name
    m.destroy()


@pytest.mark.parametrize("h", [32, 64])
def test_norm_of_large_constant_rows(mb, h):
    """Rows of one value have no variance and the normalised row is zero, though mean * rstd is beyond fp32.  Widths below and of
    a whole K-tile of the product that the norm shares a launch with."""
    m = mb.Module(dict(kind="encoder", batch=1, seq=40, hidden=h, heads=2, mlp=2 * h, layers=1, norm="layernorm", act="gelu", causal=0, bias=1, eps=1e-5), "f32")
    m.params.copy_(torch.randn(m.params.numel(), generator=torch.Generator().manual_seed(h)).mul_(0.1))
    x = torch.full((40, h), 2.0 ** 121, device="cuda")
    y = torch.full_like(x, float("nan"))
    m.forward(256, None, x, y)
    torch.cuda.synchronize()
    assert torch.equal(y, x)                # the layer adds values far below x's last bit
    m.destroy()


# 504 and 528 tiles of the q|k|v product: the norm in its launch and apart
@pytest.mark.parametrize("kind,batch", [("encoder", 42), ("encoder", 44), ("decoder", 42), ("decoder", 44)])
def test_norm_in_the_launch_of_the_product(mb, kind, batch):
    ln = kind == "encoder"
    cfg = dict(kind=kind, batch=batch, seq=32, hidden=128, heads=4, mlp=128, layers=1, norm="layernorm" if ln else "rmsnorm",
               act="gelu" if ln else "swiglu", causal=int(not ln), bias=int(ln), eps=1e-5)
    layers = quantize_tree([layer_params(cfg, 6600 + batch)], "f32")
    x = quantize(synth.normal(6700 + batch, (batch * 32, 128)), "f32")
    y_ref, _ = O.stack_fwd(x, layers, cfg)
    m = mb.Module(cfg, "f32")
    load_layer_params(m, layers)
    x_, outs = to_dev(x, "f32"), []
    for q in (256, 24):
        y = torch.full_like(x_, float("nan"))
        m.forward(q, None, x_, y)
        torch.cuda.synchronize()
        outs.append(y)
    m.destroy()
    assert_close(from_dev(outs[0]), y_ref, "f32", "y", roundings=8)
    assert torch.equal(bits(outs[0]), bits(outs[1]))
