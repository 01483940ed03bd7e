"""Patch stem at the sizes where padded patch rows and the access widths can go wrong: 14 x 14
patches (588 elements, padded in bf16), one patch per sample, patches whose rows need no padding,
widths around a tile, and a caller's tensors that do not start on a 16-byte boundary."""
import numpy as np
import pytest

from oracle import layers as O
from paper_2605_18710_amd import synth
from helpers import quantize, quantize_tree, to_dev, from_dev, assert_close, load_flat_params, read_flat_grads, stem_params

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,g,patch,h,offset", [(1, 1, 14, 64, 0), (3, 5, 14, 136, 0), (2, 24, 14, 264, 0), (2, 3, 16, 64, 0),
                                                (2, 4, 3, 24, 0), (1, 2, 1, 8, 0), (5, 7, 14, 72, 3)])
def test_patch_stem_step(dtype, B, g, patch, h, offset):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_18710_amd import binding as mb
    seed, N, pd = 5200 + 10 * g + patch, g * g, 3 * patch * patch
    p = quantize_tree(stem_params(pd, h, N, seed), dtype)
    img = quantize(synth.uniform(seed + 20, (B, 3, g * patch, g * patch)), dtype)
    dy = quantize(synth.normal(seed + 21, (B * N, h)), dtype)
    tok = O.unfold_patches(img, patch).reshape(B * N, pd)
    y_ref = O.stem_fwd(tok, p, B, N)
    g_ref = O.stem_bwd(tok, p, dy, B, N)
    g_ref = g_ref[-1] if isinstance(g_ref, tuple) else g_ref
    m = mb.Module(dict(kind="patch_stem", batch=B, seq=N, hidden=h, in_dim=pd, patch=patch), dtype)
    try:
        load_flat_params(m, p)

        def at(a):                      # the caller's tensor, `offset` elements into a larger one
            t = to_dev(a, dtype).reshape(-1)
            out = torch.empty(t.numel() + offset, dtype=t.dtype, device="cuda")
            out[offset:] = t
            return out[offset:]
        snaps = []
        for quota in (256, 24):
            m.grads.fill_(float("nan"))
            m.workspace.fill_(255)                 # NaN in both types: nothing may depend on it
            y, x, d = at(np.zeros((B * N, h))), at(img), at(dy)
            m.forward(quota, None, x, y)
            m.backward(quota, None, d)
            torch.cuda.synchronize()
            snaps.append((y.clone(), m.grads.clone()))
        assert all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(*snaps))
        assert_close(from_dev(y).reshape(B * N, h), y_ref.reshape(B * N, h), dtype, "y", roundings=2)
        got = read_flat_grads(m, p)
        for k in p:
            assert_close(got[k], g_ref[k], dtype, k, roundings=2)
    finally:
        m.destroy()


# the position table in the product's epilogue: fewer positions than a tile has rows, one position (a pass of its own), tiles of four
# waves and of eight (the share of the CUs decides; the bits must not follow it), a last tile that is partly past the tokens
@pytest.mark.parametrize("B,g,patch,h", [(300, 1, 14, 256), (130, 2, 16, 640), (40, 7, 14, 520), (9, 24, 14, 1024), (7, 13, 16, 768)])
def test_position_table_in_the_product(B, g, patch, h):
    test_patch_stem_step("bf16", B, g, patch, h, 0)


# rows of patches that pass through LDS and those that do not: the smallest even patch that does and the one below, an odd one, the
# widest image that fits and the next, an image that starts 2 bytes off
@pytest.mark.parametrize("B,g,patch,h,offset", [(2, 9, 2, 16, 0), (2, 9, 4, 24, 0), (1, 7, 6, 24, 0), (1, 5, 5, 8, 0), (1, 64, 16, 8, 0), (1, 65, 16, 8, 0), (2, 6, 8, 16, 1)])
def test_unfolding_by_rows_of_patches(B, g, patch, h, offset):
    test_patch_stem_step("bf16", B, g, patch, h, offset)


# position and bias gradient in one pass: positions that make more than one to a partition and a last partition that is short, samples
# past a batch of eight, a width that ends inside a wave's columns, the most samples of which a lane takes 16 bytes and one more, more samples
# than the pass takes
@pytest.mark.parametrize("dtype,B,g,patch,h", [("bf16", 9, 23, 4, 264), ("bf16", 4, 23, 4, 520), ("bf16", 1, 23, 4, 264), ("bf16", 5, 3, 4, 72), ("f32", 4, 3, 4, 260), ("f32", 3, 24, 2, 132), ("bf16", 17, 3, 4, 72), ("bf16", 33, 3, 4, 72)])
def test_position_and_bias_gradient(dtype, B, g, patch, h):
    test_patch_stem_step(dtype, B, g, patch, h, 0)
