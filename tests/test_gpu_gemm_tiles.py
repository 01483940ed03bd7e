"""Small products: 128 x 128 tiles take 64-deep K-tiles where every workgroup has a CU to itself and
32-deep ones otherwise, and where the CUs hold them all, tiles of 64 x 128 take their place (not in the weight gradient, nor
with SwiGLU); the bits must not show which.  Contractions around one and two K-tiles and around the
ring of stages, ragged in all dimensions, all three forms, bias, residual and activations."""
import numpy as np
import pytest

from oracle import layers as O
from paper_2605_18710_amd import synth
from helpers import quantize, to_dev, from_dev, assert_close

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_18710_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("T,k,n", [(130, 8, 128), (40, 56, 264), (257, 64, 136), (129, 72, 8), (300, 128, 520), (1, 320, 256),
                                   (190, 384, 200), (136, 1000, 392), (1568, 776, 768)])
def test_k_tile_depths_agree(mb, T, k, n):
    s = 7000 + T + k + n
    X, W, b, R, dY = [quantize(synth.normal(s + i, sh, 0, sd), "bf16") for i, (sh, sd) in
                      enumerate([((T, k), 1), ((k, n), 0.05), ((n,), 0.1), ((T, n), 1), ((T, n), 1)])]
    X_, W_, b_, R_, dY_ = [to_dev(a, "bf16") for a in (X, W, b, R, dY)]
    # CUs for tiles of 128 rows, one to a CU, but not for those of 64 (above 32, shares count in steps of 32)
    deep = set()
    for cols in (n, k):
        t128, t64 = -(-T // 128) * -(-cols // 128), -(-T // 64) * -(-cols // 128)
        q = t128 if t128 <= 32 else -(-t128 // 32) * 32
        deep |= {q} if q < t64 else set()
    outs = []
    for q in [256, 1] + sorted(deep):     # one workgroup per CU; more tiles than slots
        e = lambda *sh: torch.full(sh, float("nan"), dtype=torch.bfloat16, device="cuda")
        Y, Z, A, dX, dW = e(T, n), e(T, n), e(T, n), e(T, k), e(k, n)
        sc = torch.empty(max(16, mb.linear_wgrad_scratch_bytes(T, k, n)), dtype=torch.uint8, device="cuda")
        mb.op_linear_fwd(None, q, "bf16", T, k, n, X_, W_, b_, R_, Y)
        mb.op_linear_act_fwd(None, q, "bf16", mb.GELU, T, k, n, X_, W_, b_, Z, A)
        mb.op_linear_dgrad(None, q, "bf16", T, k, n, dY_, W_, None, dX)
        mb.op_linear_wgrad(None, q, "bf16", T, k, n, X_, dY_, dW, None, sc)
        got = [Y, Z, A, dX] + [dW]
        if n % 256 == 0:
            G, S = e(T, n), e(T, n // 2)
            mb.op_linear_act_fwd(None, q, "bf16", mb.SWIGLU, T, k, n, X_, W_, None, G, S)
            got += [G, S]
        torch.cuda.synchronize()
        outs.append(got)
    z_ref = O.linear_fwd(X, W, b)
    dx_ref, dw_ref, _ = O.linear_bwd(X, W, dY)
    assert_close(from_dev(Y), z_ref + R, "bf16", "Y")
    assert_close(from_dev(A), O.gelu(from_dev(Z)), "bf16", "A")
    assert_close(from_dev(dX), dx_ref, "bf16", "dX")
    assert_close(from_dev(dW), dw_ref, "bf16", "dW")
    if n % 256 == 0:
        g = from_dev(G)
        assert_close(g, O.linear_fwd(X, W), "bf16", "gate | up")
        assert_close(from_dev(S), O.swiglu_fwd(g[:, :n // 2], g[:, n // 2:]), "bf16", "swiglu")
    assert all(torch.equal(a.view(torch.int16), c.view(torch.int16)) for o in outs[1:] for a, c in zip(o, outs[0]))


@pytest.mark.parametrize("T,k,n", [(1, 8, 8), (63, 72, 136), (64, 128, 128), (65, 64, 264), (128, 1000, 120), (129, 136, 392), (200, 520, 1024)])
def test_tiles_of_64_rows(mb, T, k, n):
    """The share of the CUs decides between 64 and 128 rows to a tile: on both sides of that line, for the forward
    product (plain, with a residual, with GELU) and the input gradient."""
    s = 7600 + T + k + n
    X, W, b, R, dY = [quantize(synth.normal(s + i, sh, 0, sd), "bf16") for i, (sh, sd) in
                      enumerate([((T, k), 1), ((k, n), 0.05), ((n,), 0.1), ((T, n), 1), ((T, n), 1)])]
    X_, W_, b_, R_, dY_ = [to_dev(a, "bf16") for a in (X, W, b, R, dY)]
    tiles = lambda cols: -(-T // 64) * -(-cols // 128)
    quotas = sorted({q for t in (tiles(n), tiles(k)) for q in (t - 1, t, t + 1) if q > 0} | {1, 256})
    first = None
    for q in quotas:
        Y, Z, A, dX = [torch.full(sh, float("nan"), dtype=torch.bfloat16, device="cuda") for sh in ((T, n), (T, n), (T, n), (T, k))]
        mb.op_linear_fwd(None, q, "bf16", T, k, n, X_, W_, b_, R_, Y)
        mb.op_linear_act_fwd(None, q, "bf16", mb.GELU, T, k, n, X_, W_, b_, Z, A)
        mb.op_linear_dgrad(None, q, "bf16", T, k, n, dY_, W_, None, dX)
        torch.cuda.synchronize()
        got = [t.view(torch.int16) for t in (Y, Z, A, dX)]
        first = first or got
        assert all(torch.equal(a, c) for a, c in zip(got, first)), f"bits at {q} CUs differ from those at {quotas[0]}"
    z_ref = O.linear_fwd(X, W, b)
    assert_close(from_dev(Y), z_ref + R, "bf16", "Y")
    assert_close(from_dev(Z), z_ref, "bf16", "Z")
    assert_close(from_dev(A), O.gelu(from_dev(Z)), "bf16", "A")
    assert_close(from_dev(dX), O.linear_bwd(X, W, dY)[0], "bf16", "dX")


@pytest.mark.parametrize("T,k,n,note", [
    (2048, 264, 1032, "27 small tiles in pieces beside each other, ragged tile row and column"),
    (2056, 128, 128, "one tile in pieces that end in mid K-tile of 64"),
    (4096, 1024, 2048, "eight pieces: chained in small tiles, or large tiles"),
    (3000, 768, 3072, "pieces of an odd number of 32 k-values, chained one and two tiles to a CU"),
    (9216, 1024, 4096, "four pieces: chained, small tiles and large tiles by the quota"),
    (9216, 600, 1024, "patch embedding shape: 40 small tiles in 8 pieces"),
    (12000, 1280, 1280, "large tiles in 8 pieces, small ones on 192 and 160 CUs"),
])
def test_weight_gradient_of_few_tiles(mb, T, k, n, note):
    """Pieces follow the shape; tile size and whether the pieces stand beside each other or follow one
    another go by the quota: same bits at every quota, every column against the oracle."""
    X, dY = quantize(synth.normal(7300, (T, k)), "bf16"), quantize(synth.normal(7301, (T, n)), "bf16")
    X_, dY_ = to_dev(X, "bf16"), to_dev(dY, "bf16")
    nbytes = mb.linear_wgrad_scratch_bytes(T, k, n)
    assert nbytes > mb.colsum_scratch_bytes(n), "this shape has scratch for pieces"
    outs = []
    for q in (256, 224, 192, 64, 32, 8, 1):
        ws = torch.full((nbytes + 4096,), 255, dtype=torch.uint8, device="cuda")        # NaN: nothing may be read before it is written
        dW = torch.full((k, n), float("nan"), dtype=torch.bfloat16, device="cuda")
        mb.op_linear_wgrad(None, q, "bf16", T, k, n, X_, dY_, dW, None, ws)
        torch.cuda.synchronize()
        assert bool((ws[nbytes:] == 255).all()), "written past the scratch"
        outs.append(dW)
    assert_close(from_dev(outs[0]), X.T @ dY, "bf16", note)
    assert all(torch.equal(o.view(torch.int16), outs[0].view(torch.int16)) for o in outs[1:]), note


@pytest.mark.parametrize("T,k,n", [(510, 128, 504), (255, 192, 1016), (768, 320, 512), (1000, 1088, 768),      # forward: contraction k
                                   (510, 248, 128), (1000, 760, 192), (249, 1024, 1088),                       # input gradient: n
                                   (72, 504, 760), (136, 256, 1024), (1000, 512, 504),                         # weight gradient: T, any length
                                   (150, 192, 504), (330, 128, 1016), (181, 192, 512), (215, 320, 256), (430, 128, 768),
                                   (160, 504, 128), (192, 256, 320), (224, 248, 192), (670, 256, 256)])        # tiles of 160, 192 and 224 rows
def test_large_tiles_agree_with_small_ones(mb, T, k, n):
    """On the whole device these products take 128 x 128 tiles, on one CU 256 columns by 256, 224, 192 or 160
    rows (where a form fits them: otherwise both runs take small tiles), several to a workgroup: two and more K-tiles of 64, odd counts, a contraction that ends in
    mid K-tile, ragged rows and columns, every epilogue."""
    s = 7600 + T + k + n
    X, W, b, R, dY = [quantize(synth.normal(s + i, sh, 0, sd), "bf16") for i, (sh, sd) in
                      enumerate([((T, k), 1), ((k, n), 0.05), ((n,), 0.1), ((T, n), 1), ((T, n), 1)])]
    X_, W_, b_, R_, dY_ = [to_dev(a, "bf16") for a in (X, W, b, R, dY)]
    R2 = quantize(synth.normal(s + 9, (T, k)), "bf16")
    R2_ = to_dev(R2, "bf16")
    outs = []
    for q in (256, 1, 3):
        e = lambda *sh: torch.full(sh, float("nan"), dtype=torch.bfloat16, device="cuda")
        P, Y, Yr, Z, A, dX, dXr, dW = e(T, n), e(T, n), e(T, n), e(T, n), e(T, n), e(T, k), e(T, k), e(k, n)
        sc = torch.empty(max(16, mb.linear_wgrad_scratch_bytes(T, k, n)), dtype=torch.uint8, device="cuda")
        mb.op_linear_fwd(None, q, "bf16", T, k, n, X_, W_, None, None, P)
        mb.op_linear_fwd(None, q, "bf16", T, k, n, X_, W_, b_, None, Y)
        mb.op_linear_fwd(None, q, "bf16", T, k, n, X_, W_, b_, R_, Yr)
        mb.op_linear_act_fwd(None, q, "bf16", mb.GELU, T, k, n, X_, W_, b_, Z, A)
        mb.op_linear_dgrad(None, q, "bf16", T, k, n, dY_, W_, None, dX)
        mb.op_linear_dgrad(None, q, "bf16", T, k, n, dY_, W_, R2_, dXr)
        mb.op_linear_wgrad(None, q, "bf16", T, k, n, X_, dY_, dW, None, sc)
        got = [P, Y, Yr, Z, A, dX, dXr, dW]
        if n % 256 == 0:
            G, S = e(T, n), e(T, n // 2)
            mb.op_linear_act_fwd(None, q, "bf16", mb.SWIGLU, T, k, n, X_, W_, b_, G, S)
            got += [G, S]
        torch.cuda.synchronize()
        outs.append(got)
    z_ref = O.linear_fwd(X, W, b)
    dx_ref, dw_ref, _ = O.linear_bwd(X, W, dY)
    P, Y, Yr, Z, A, dX, dXr, dW = outs[1][:8]
    for got, want, what in ((P, O.linear_fwd(X, W), "P"), (Y, z_ref, "Y"), (Yr, z_ref + R, "Yr"), (Z, z_ref, "Z"), (A, O.gelu(from_dev(Z)), "A"),
                            (dX, dx_ref, "dX"), (dXr, dx_ref + R2, "dXr"), (dW, dw_ref, "dW")):
        assert_close(from_dev(got), want, "bf16", what)
    if n % 256 == 0:
        g = from_dev(outs[1][8])
        assert_close(g, z_ref, "bf16", "gate | up")
        assert_close(from_dev(outs[1][9]), O.swiglu_fwd(g[:, :n // 2], g[:, n // 2:]), "bf16", "swiglu")
    for o in outs[1:]:
        assert all(torch.equal(a.view(torch.int16), c.view(torch.int16)) for a, c in zip(o, outs[0]))


def _hard(torch, g, kind, shape):
    x = torch.randn(shape, generator=g, device="cuda")
    if kind == "spread":            # terms that differ by up to 2^60, and by all powers between
        x *= torch.exp2(torch.randint(-30, 31, shape, generator=g, device="cuda").float())
    elif kind == "denormal":        # bf16 numbers at and below the smallest normal one
        x *= torch.exp2(torch.randint(-133, -120, shape, generator=g, device="cuda").float())
    elif kind == "small":           # products at and below fp32's normal range
        x *= 2.0 ** -62
    return x.to(torch.bfloat16)


@pytest.mark.parametrize("a,b", [("spread", "spread"), ("spread", "normal"), ("cancel", "spread"), ("cancel", "normal"), ("denormal", "normal"),
                                 ("normal", "denormal"), ("small", "small")])
@pytest.mark.parametrize("T,k,n", [(510, 1024, 504), (256, 128, 256), (330, 320, 512), (200, 256, 264)])
def test_matrix_instructions_agree_on_hard_data(mb, T, k, n, a, b):
    """128 x 128 tiles multiply with the 32x32x16 instruction, the large ones of one CU with 16x16x32: the quota
    decides which one an element meets.  Sums that show how an instruction aligns and rounds its terms."""
    g = torch.Generator(device="cuda").manual_seed(T + k + n)
    X, W, dY = _hard(torch, g, "spread" if a == "cancel" else a, (T, k)), _hard(torch, g, b, (k, n)), _hard(torch, g, "spread" if a == "cancel" else a, (T, n))
    if a == "cancel":               # neighbouring terms of opposite sign, and a few that do not cancel
        X[:, 1::2] = -X[:, 0::2]
        W[1::2] = W[0::2]
        W[5::16] = _hard(torch, g, b, tuple(W[5::16].shape))
        dY[1::2] = -dY[0::2][:dY[1::2].shape[0]]
    outs = []
    for q in (256, 1, 3):
        Y, dX, dW = [torch.full(s, float("nan"), dtype=torch.bfloat16, device="cuda") for s in ((T, n), (T, k), (k, n))]
        sc = torch.empty(max(16, mb.linear_wgrad_scratch_bytes(T, k, n)), dtype=torch.uint8, device="cuda")
        mb.op_linear_fwd(None, q, "bf16", T, k, n, X, W, None, None, Y)
        mb.op_linear_dgrad(None, q, "bf16", T, k, n, dY, W, None, dX)
        mb.op_linear_wgrad(None, q, "bf16", T, k, n, X, dY, dW, None, sc)
        torch.cuda.synchronize()
        outs.append((Y, dX, dW))
    for o in outs[1:]:
        assert all(torch.equal(x.view(torch.int16), y.view(torch.int16)) for x, y in zip(o, outs[0]))
    # one rounding to bf16 (2^-9 of an element on average over the mantissas) of the 64-bit sum
    ref = X.double() @ W.double()
    assert float((outs[0][0].double() - ref).norm() / ref.norm()) < 2.5e-3


@pytest.mark.parametrize("T,k,n", [(130, 136, 520), (257, 264, 8), (40, 1000, 72), (1568, 776, 768), (2048, 128, 2048)])
def test_backward_products_in_one_launch(mb, T, k, n):
    """Input and weight gradient side by side in one launch (from 16 CUs on, small products; 2048 rows: the weight
    gradient's pieces chained) have the bits of two launches (8 CUs), and dx may lie on x."""
    m = mb.Module(dict(kind="projector", batch=1, seq=T, in_dim=k, out_dim=n), "bf16")
    m.params.copy_(torch.randn(m.params.numel(), generator=torch.Generator().manual_seed(T), dtype=torch.float32).mul_(0.05).to(torch.bfloat16))
    x, dy = to_dev(synth.normal(8100 + T, (T, k)), "bf16"), to_dev(synth.normal(8101 + T, (T, n)), "bf16")
    outs = []
    for q, alias in ((8, False), (256, False), (64, False), (33, False), (256, True)):
        xin = x.clone()
        y, dx = torch.full_like(dy, float("nan")), xin if alias else torch.full_like(x, float("nan"))
        m.grads.fill_(float("nan"))
        m.step(q, None, xin, y, dy=dy, dx=dx)
        torch.cuda.synchronize()
        outs.append([t.clone().view(torch.int16) for t in (y, dx, m.grads[:m.param_elems])])
    assert not any(torch.isnan(t.view(torch.bfloat16)).any() for t in outs[0])
    for o in outs[1:]:
        assert all(torch.equal(a, b) for a, b in zip(outs[0], o))
    m.destroy()


@pytest.mark.parametrize("dtype,T,k,n", [("bf16", 128, 128, 128), ("bf16", 100, 72, 64), ("f32", 32, 256, 32), ("f32", 20, 28, 132)])
def test_output_of_one_tile_on_an_operand(mb, dtype, T, k, n):
    """A product of one tile of 128 x 128 (fp32: 32 x 32) reads both operands before it stores: its output may lie on
    either, and it must not be dealt out in smaller tiles then."""
    rnd = lambda i, *sh: to_dev(synth.normal(7800 + T + i, sh, 0, 0.3), dtype)
    X, W, dY = rnd(0, T, k), rnd(1, k, n), rnd(2, T, n)
    Y, dX = torch.empty_like(dY), torch.empty_like(X)
    mb.op_linear_fwd(None, 256, dtype, T, k, n, X, W, None, None, Y)
    mb.op_linear_dgrad(None, 256, dtype, T, k, n, dY, W, None, dX)
    side = 128 if dtype == "bf16" else 32
    for which in range(2):
        at = [torch.zeros(max(T * n, T * k, k * n), dtype=X.dtype, device="cuda") for _ in range(3)]
        for buf, t in zip(at, (X, W, dY)):
            buf[:t.numel()] = t.reshape(-1)
        if n <= side:
            bufs = [b.clone() for b in at]
            mb.op_linear_fwd(None, 256, dtype, T, k, n, bufs[0], bufs[1], None, None, bufs[which])
            assert torch.equal(bufs[which][:T * n], Y.reshape(-1))
        if k <= side:
            bufs = [b.clone() for b in at]
            mb.op_linear_dgrad(None, 256, dtype, T, k, n, bufs[2], bufs[1], None, bufs[2 - which])
            assert torch.equal(bufs[2 - which][:T * k], dX.reshape(-1))
