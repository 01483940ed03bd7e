"""Text stem at the sizes where the embedding gradient's three ways can go wrong, on both sides of the rules between
them.  The scan of small calls (up to 128 positions): widths and positions at its limits.  The sort by one
workgroup (up to 8192 positions, keys and positions in 32 bits): rounds of 1024 positions, digits of 8 bits.  The sort in several
launches (more positions, or more bits): chunks of 2048 positions.  The sums after either sort: segments of 16 positions, one id
for everything, no text at all, widths of one and several column tiles, tensors that do not start on a 16-byte boundary."""
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


# the scan, for more than 96 positions: its limits of positions, vocabulary and width, and the widths at which a thread takes more columns
SCAN = [(1, 128, 0, 512, 2048, "mixed", 0), (1, 128, 0, 512, 2049, "mixed", 0), (1, 128, 3, 520, 500, "mixed", 0), (1, 129, 0, 64, 300, "mixed", 0), (1, 97, 0, 64, 97, "mixed", 0),
        (2, 49, 5, 64, 99, "mixed", 1), (1, 120, 0, 520, 1000, "one", 0), (1, 97, 0, 8, 2047, "one", 0), (1, 64, 0, 2048, 40, "mixed", 0), (1, 63, 0, 2056, 40, "mixed", 0),
        (1, 33, 0, 8184, 16, "mixed", 0)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,N,n_img,h,vocab,how,offset", SCAN)
def test_scan(dtype, B, N, n_img, h, vocab, how, offset):
    test_text_stem_step(dtype, B, N, n_img, h, vocab, how, offset)


@pytest.mark.parametrize("T,h,vocab", [(128, 512, 1000), (97, 64, 128), (100, 600, 2048), (96, 2048, 100), (30, 8192, 50)])
def test_small_calls_add_the_rows_of_an_id_in_ascending_order(T, h, vocab):
    """fp32, every position the same id: the scan has one chain of sums, the sort pieces of 16 positions."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_18710_amd import binding as mb
    stem = mb.Module(dict(kind="text_stem", batch=1, seq=T, hidden=h, vocab=vocab, n_img=0), "f32")
    stem.bind_ids(torch.full((T,), 7, dtype=torch.int32, device="cuda"))
    g = to_dev(synth.normal(4900 + T, (T, h)), "f32")
    y = torch.empty_like(g)
    stem.grads.fill_(float("nan"))
    stem.forward(256, None, g, y)
    stem.backward(256, None, g, None)
    torch.cuda.synchronize()
    acc = torch.zeros(h, device="cuda")
    for t in range(T):
        acc = acc + g[t]
    got = stem.grads[:vocab * h].view(vocab, h)
    assert torch.equal(got[7].view(torch.int32), acc.view(torch.int32))
    assert not bool(got[:7].any()) and not bool(got[8:].any())
    stem.destroy()


# sample lengths and the most image tokens; the counts go from none to that many.  Positions that the scan, the sort by one workgroup and
# the sort in several launches take; of the last: whole chunks, a last chunk of 1 and of 2047 positions, keys of one, two and three digits
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,N,n_img,h,vocab", [(3, 31, 12, 64, 40), (2, 64, 64, 8, 1000), (4, 200, 70, 264, 300), (8, 1024, 196, 64, 70), (1, 8193, 100, 8, 254), (5, 2048, 300, 72, 255),
                                               (3, 3413, 500, 24, 256), (3, 3413, 0, 8, 65536), (2, 5121, 77, 16, 70000), (4, 4096, 196, 40, 3)])
def test_text_stem_with_image_counts(dtype, B, N, n_img, h, vocab):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_18710_amd import binding as mb
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator().manual_seed(N + vocab)
    ids = torch.randint(0, vocab, (B, N), generator=gen, dtype=torch.int32)
    ids[:, ::3] = vocab - 1
    counts = torch.tensor([n_img * b // max(1, B - 1) for b in range(B)], dtype=torch.int32)
    img, dy = torch.randn(B * n_img, h, generator=gen).to(td).cuda(), torch.randn(B * N, h, generator=gen).to(td).cuda()
    stem = mb.Module(dict(kind="text_stem", batch=B, seq=N, hidden=h, vocab=vocab, n_img=n_img), dtype)
    try:
        stem.params[:vocab * h].copy_(torch.randn(vocab * h, generator=gen).to(td))
        stem.bind_ids(ids.cuda())
        stem.bind_image_counts(counts.cuda())
        text = torch.arange(N)[None, :] >= counts[:, None]                       # [B, N]
        sel, at = text.reshape(-1).cuda(), ids[text].long().cuda()
        ref_y = torch.empty_like(dy)
        ref_y[sel] = stem.params[:vocab * h].view(vocab, h)[at]
        ref_y.view(B, N, h)[:, :n_img][~text[:, :n_img].cuda()] = img.view(B, n_img, h)[~text[:, :n_img].cuda()]
        ref_img = torch.where(text[:, :n_img, None].cuda(), torch.zeros((), dtype=td, device="cuda"), dy.view(B, N, h)[:, :n_img])
        ref = torch.zeros(vocab, h, dtype=torch.float64, device="cuda").index_add_(0, at, dy[sel].double())
        snaps = []
        for quota in (256, 24):
            stem.grads.fill_(float("nan"))
            y, dx = torch.full_like(dy, float("nan")), torch.full_like(img, float("nan"))
            stem.forward(quota, None, img if n_img else dy, y)
            stem.backward(quota, None, dy, dx if n_img else None)
            torch.cuda.synchronize()
            assert torch.equal(y, ref_y) and torch.equal(dx.view(B, n_img, h), ref_img)
            snaps.append(stem.grads[:vocab * h].clone())
        assert torch.equal(snaps[0].view(torch.uint8), snaps[1].view(torch.uint8))
        got = snaps[0].view(vocab, h).double()
        assert bool((got[torch.bincount(at, minlength=vocab) == 0] == 0).all()), "rows that nobody used"
        # one rounding of a sum of up to 16000 terms in fp32
        assert_close(got.cpu().numpy(), ref.cpu().numpy(), dtype, "table gradient", roundings=4)
    finally:
        stem.destroy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,N,n_img,h,vocab,how,offset", [(1, 33, 0, 8192, 50, "mixed", 0), (1, 32, 0, 8192, 50, "mixed", 0), (1, 8193, 0, 64, 254, "one", 0), (3, 3413, 2, 264, 257, "mixed", 1)])
def test_limits_of_the_scan_and_of_the_one_workgroup(dtype, B, N, n_img, h, vocab, how, offset):
    test_text_stem_step(dtype, B, N, n_img, h, vocab, how, offset)


# a thread of the one workgroup's launch requests one, two, four or eight keys at once; samples of one position, of image tokens alone
@pytest.mark.parametrize("B,N,n_img", [(1000, 1, 0), (1023, 1, 1), (3, 683, 5), (2, 1025, 1025), (8191, 1, 1), (4, 1025, 100), (2731, 3, 2), (2, 4096, 4000)])
def test_keys_requested_together(B, N, n_img):
    test_text_stem_step("bf16", B, N, n_img, 72, 300, "mixed", 0)
    test_text_stem_with_image_counts("f32", B, N, n_img, 8, 300)
