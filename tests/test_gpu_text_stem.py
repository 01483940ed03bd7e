"""Text stem at the sizes where the sort by id, its segments and the access width can go wrong:
position counts around a chunk (2048) and a segment (16), vocabularies on both sides of a digit
(8 bits), one id for everything, no text at all, widths of one and several column tiles, and
tensors that do not start on a 16-byte boundary; and both sides of the rule by which small calls
scan the ids instead of sorting them."""
import numpy as np
import pytest

from oracle import layers as O
from paper_2605_18710_amd import synth
from helpers import quantize, to_dev, from_dev, assert_close

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = [  # B, N, n_img, h, vocab, ids, offset of the caller's tensors in elements
    (1, 1, 0, 8, 1, "mixed", 0),
    (1, 16, 0, 64, 255, "one", 0),
    (1, 17, 1, 64, 256, "mixed", 1),
    (2, 1024, 0, 72, 257, "mixed", 0),
    (1, 2047, 3, 16, 300, "one", 0),
    (3, 683, 1, 2056, 40, "mixed", 0),
    (4, 1100, 1100, 64, 70, "mixed", 0),
    (2, 1500, 700, 40, 65536, "mixed", 0),
    (2, 1500, 0, 24, 16777217, "mixed", 0),
    (5, 900, 11, 1032, 3, "mixed", 3),
    # few positions to many, narrow and wide, small and large vocabularies
    (2, 128, 0, 512, 255, "mixed", 0), (1, 257, 0, 64, 255, "mixed", 0), (1, 256, 0, 520, 255, "mixed", 0),
    (1, 512, 7, 512, 256, "mixed", 1), (1, 640, 0, 64, 300, "one", 0), (1, 641, 7, 64, 256, "one", 0), (1, 512, 0, 520, 257, "mixed", 0),
    (4, 64, 20, 1024, 16384, "one", 0), (4, 64, 20, 64, 16385, "mixed", 0), (1, 32, 0, 8192, 16, "one", 0), (1, 64, 3, 1000, 16, "mixed", 0), (1, 65, 0, 1000, 16, "mixed", 0),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,N,n_img,h,vocab,how,offset", CASES)
def test_text_stem_step(dtype, B, N, n_img, h, vocab, how, offset):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_18710_amd import binding as mb
    seed = 4100 + N + vocab % 97
    ids = synth.integers(seed, (B, N - n_img), 0, vocab) if how == "mixed" else np.full((B, N - n_img), vocab // 2, dtype=np.int32)
    if how == "mixed" and ids.size:
        ids.reshape(-1)[::3] = vocab - 1
    dy = quantize(synth.normal(seed + 1, (B * N, h)), dtype)
    img = quantize(synth.normal(seed + 2, (B * n_img, h)), dtype)
    stem = mb.Module(dict(kind="text_stem", batch=B, seq=N, hidden=h, vocab=vocab, n_img=n_img), dtype)
    used = np.unique(ids)
    try:
        rows = quantize(synth.normal(seed + 3, (max(1, used.size), h), 0, 0.02), dtype)
        stem.params.zero_()
        table = stem.params[:vocab * h].view(vocab, h)
        if used.size:
            table[torch.from_numpy(used.astype(np.int64)).cuda()] = to_dev(rows[:used.size], dtype)
        stem.bind_ids(torch.from_numpy(np.ascontiguousarray(ids).reshape(-1)).cuda() if ids.size else torch.zeros(1, dtype=torch.int32, device="cuda"))

        def at(a):                      # the caller's tensor, `offset` elements into a larger one
            t = to_dev(a, dtype).reshape(-1)
            out = torch.empty(t.numel() + offset + 8, dtype=t.dtype, device="cuda")
            out[offset:offset + t.numel()] = t
            return out[offset:offset + t.numel()]
        x, g, y = at(img), at(dy), at(np.zeros((B * N, h)))
        snaps = []
        for quota in (256, 24):
            stem.grads.fill_(float("nan"))
            dx = at(np.full((B * n_img, h), np.nan))
            stem.forward(quota, None, x if x.numel() else g, y)
            stem.backward(quota, None, g, dx if dx.numel() else None)
            torch.cuda.synchronize()
            snaps.append((stem.grads[:vocab * h].clone(), dx.clone(), y.clone()))
        for a, b in zip(*snaps):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
        d_img, d_text = O.split_tokens(dy, B, n_img, N - n_img)
        ref_y = np.concatenate([img.reshape(B, n_img, h), rows[np.searchsorted(used, ids)].reshape(B, N - n_img, h)], axis=1)
        assert np.array_equal(from_dev(y).reshape(B, N, h), ref_y), "the sequence is a copy"
        assert np.array_equal(from_dev(snaps[0][1]).reshape(B * n_img, h), d_img.reshape(B * n_img, h)), "the image gradient is a copy"
        got = snaps[0][0].view(vocab, h)
        if used.size:
            ref = O.embedding_bwd(np.searchsorted(used, ids).astype(np.int32), d_text, used.size)
            sel = torch.from_numpy(used.astype(np.int64)).cuda()
            # one rounding of a sum of up to 4500 terms in fp32
            assert_close(from_dev(got[sel]), ref, dtype, "table gradient", roundings=4)
            got[sel] = 0
        assert not bool(got.any()), "rows that nobody used"          # NaN counts as non-zero
    finally:
        stem.destroy()


# one workgroup sorts up to 8192 positions where a key and its position fit 32 bits: both sides of both limits, of a
# round (1024 positions), of a wave's share, and of the scan's limits; more rows to a workgroup than it flags at once
ONE_SORT = [(1, 97, 0, 64, 30, "mixed", 0), (1, 97, 0, 64, 8192, "mixed", 0), (1, 96, 5, 64, 8193, "mixed", 0), (1, 96, 0, 64, 24, "one", 0),
            (1, 1024, 0, 8, 300, "mixed", 0), (1, 1025, 1, 8, 300, "mixed", 0), (1, 8192, 0, 8, 524287, "mixed", 0),
            (1, 8192, 0, 8, 524288, "mixed", 0), (3, 2731, 40, 24, 999, "mixed", 1), (1, 8192, 5, 72, 65537, "one", 0),
            (1, 300, 0, 8, 1200007, "mixed", 0), (8, 1024, 196, 128, 70, "mixed", 0)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,N,n_img,h,vocab,how,offset", ONE_SORT)
def test_sort_in_one_launch(dtype, B, N, n_img, h, vocab, how, offset):
    test_text_stem_step(dtype, B, N, n_img, h, vocab, how, offset)
