"""GPU parity: leann_embed against the encoder oracle (bound from the benchmark spec: max-abs 2e-2, bf16 GPU vs
fp32 oracle; a tighter 3e-3 against the oracle's bf16-storage mode)."""
import numpy as np
import pytest

import gemm_plan
import leann_inputs as li
from gpu_util import say, to_dev

pytestmark = pytest.mark.gpu

TOL_FP32 = 2e-2
TOL_BF16_MODE = 3e-3


@pytest.fixture(scope="module")
def L():
    import paper_2506_08276_amd as L
    L.load_library()
    return L


@pytest.fixture(scope="module")
def tiny(L, orc):
    import torch
    cfg = li.TINY
    w = li.encoder_weights(cfg, 7, perturb=True)
    tokens, lengths = li.uniform_chunks(700, 32, 1, 1000, 1, 32, 8)
    lengths[:3] = [1, 32, 31]
    ctx = L.leann_create(cfg, to_dev(w))
    yield dict(cfg=cfg, w=w, tokens=tokens, lengths=lengths, ctx=ctx, t=to_dev(tokens), l=to_dev(lengths))
    L.leann_destroy(ctx)


def test_tiny_ragged_matches_oracle(L, orc, tiny):
    """700 ragged chunks (about 11.5k packed tokens: ~90 row tiles of 128 and a ragged tail)."""
    say("tiny ragged embed, seed 7/8, n=700")
    got = L.leann_embed(tiny["ctx"], tiny["t"], tiny["l"], hidden=128).cpu().numpy()
    e = orc.desc(**tiny["cfg"])
    want = orc.embed(e, tiny["w"], tiny["tokens"], tiny["lengths"])
    want_bf = orc.embed(e, tiny["w"], tiny["tokens"], tiny["lengths"], precision=1)
    assert np.isfinite(got).all()
    assert np.abs(got - want).max() <= TOL_FP32
    assert np.abs(got - want_bf).max() <= TOL_BF16_MODE
    np.testing.assert_allclose(np.linalg.norm(got, axis=1), 1.0, atol=1e-5)


def test_batch_composition_and_pass_invariance(L, tiny):
    """A chunk's embedding is bit-identical whatever shares its batch or its pass."""
    import torch
    say("batch composition invariance")
    full = L.leann_embed(tiny["ctx"], tiny["t"], tiny["l"], hidden=128)
    ids = torch.tensor([5, 699, 0, 5, 123, 77], dtype=torch.int64, device="cuda:0")
    sub = L.leann_embed(tiny["ctx"], tiny["t"], tiny["l"], ids=ids, hidden=128)
    assert torch.equal(sub, full[ids])
    say("pass slicing invariance (64-token passes)")
    L.leann_set_limits(tiny["ctx"], max_tokens_per_pass=64)
    try:
        sliced = L.leann_embed(tiny["ctx"], tiny["t"], tiny["l"], hidden=128)
    finally:
        L.leann_set_limits(tiny["ctx"], max_tokens_per_pass=262144)
    assert torch.equal(sliced, full)
    first = L.leann_embed(tiny["ctx"], tiny["t"], tiny["l"], n_ids=10, hidden=128)
    assert torch.equal(first, full[:10])


@pytest.mark.parametrize("hidden,heads,ffn", [(128, 2, 128), (640, 10, 128)])
def test_pooled_rows_and_few_chunks_against_oracle(L, orc, hidden, heads, ffn):
    """Means over one row, over as many as are read ahead, one more and one fewer, over rows of less than and more than a
    wavefront's pieces; passes of as many chunks as one wavefront scans and of one more."""
    cfg = dict(vocab=500, max_pos=160, hidden=hidden, layers=1, heads=heads, ffn=ffn, ln_eps=1e-12)
    w = li.encoder_weights(cfg, 9, perturb=True)
    tokens, lengths = li.uniform_chunks(65, 130, 1, 500, 1, 130, 4)
    lengths[:12] = [1, 2, 4, 5, 31, 32, 33, 63, 64, 65, 127, 130]
    say(f"pooled rows, hidden {hidden}")
    ctx = L.leann_create(cfg, to_dev(w))
    try:
        t, l = to_dev(tokens), to_dev(lengths)
        got = L.leann_embed(ctx, t, l, hidden=hidden).cpu().numpy()
        few = L.leann_embed(ctx, t, l, n_ids=64, hidden=hidden).cpu().numpy()
        one = L.leann_embed(ctx, t, l, n_ids=1, hidden=hidden).cpu().numpy()
    finally:
        L.leann_destroy(ctx)
    want = orc.embed(orc.desc(**cfg), w, tokens, lengths)
    assert np.abs(got - want).max() <= TOL_FP32
    np.testing.assert_array_equal(few, got[:64])
    np.testing.assert_array_equal(one, got[:1])


@pytest.mark.parametrize("seq", [128, 256])
def test_attention_key_counts(L, orc, seq):
    """Chunks that end before, at and behind every tile of 32 keys, each followed by another chunk's rows: what a chunk's keys end
    with does not depend on what follows, and the oracle gives the same."""
    import torch
    cfg = dict(vocab=500, max_pos=256, hidden=128, layers=2, heads=2, ffn=128, ln_eps=1e-12)
    lengths = np.array([x for e in range(32, seq + 1, 32) for x in (e - 1, e, e + 1) if x <= seq] + [1, 2, 15, 16, 17], np.int32)
    tokens = np.random.default_rng(seq).integers(1, 500, (len(lengths), seq)).astype(np.int32)
    w = li.encoder_weights(cfg, 17, perturb=True)
    say(f"attention key counts, seq {seq}")
    ctx = L.leann_create(cfg, to_dev(w))
    try:
        t, l = to_dev(tokens), to_dev(lengths)
        got = L.leann_embed(ctx, t, l, hidden=128)
        for i in range(len(lengths)):
            alone = L.leann_embed(ctx, t, l, ids=torch.tensor([i], dtype=torch.int64, device="cuda:0"), hidden=128)
            assert torch.equal(alone[0], got[i]), lengths[i]
    finally:
        L.leann_destroy(ctx)
    assert np.abs(got.cpu().numpy() - orc.embed(orc.desc(**cfg), w, tokens, lengths)).max() <= TOL_FP32


def test_padding_content_is_ignored(L, tiny):
    import torch
    say("padding invariance")
    full = L.leann_embed(tiny["ctx"], tiny["t"], tiny["l"], hidden=128)
    junk = tiny["tokens"].copy()
    junk[np.arange(32)[None, :] >= tiny["lengths"][:, None]] = 999
    got = L.leann_embed(tiny["ctx"], to_dev(junk), tiny["l"], hidden=128)
    assert torch.equal(got, full)


def test_empty_and_errors(L, tiny):
    import torch
    say("empty request and invalid inputs")
    out = L.leann_embed(tiny["ctx"], tiny["t"], tiny["l"], n_ids=0, hidden=128)
    assert out.shape == (0, 128)
    bad_tok = tiny["tokens"].copy()
    bad_tok[3, 0] = 1000
    with pytest.raises(L.LeannError) as ei:
        L.leann_embed(tiny["ctx"], to_dev(bad_tok), tiny["l"], hidden=128)
    assert ei.value.status == -1
    bad_len = tiny["lengths"].copy()
    bad_len[4] = 33
    with pytest.raises(L.LeannError):
        L.leann_embed(tiny["ctx"], tiny["t"], to_dev(bad_len), hidden=128)
    with pytest.raises(L.LeannError):
        L.leann_embed(tiny["ctx"], tiny["t"], tiny["l"], ids=torch.tensor([700], dtype=torch.int64, device="cuda:0"),
                      hidden=128)
    with pytest.raises(L.LeannError) as ei:
        L.leann_create(dict(li.TINY, hidden=96, heads=2), to_dev(np.zeros(10, np.float32)))
    assert ei.value.status == -4
    # the context still works after the rejected calls
    ok = L.leann_embed(tiny["ctx"], tiny["t"], tiny["l"], n_ids=4, hidden=128)
    assert torch.isfinite(ok).all()


def test_base_shape_sample_matches_oracle(L, orc):
    """BERT-base shape at seq 256, bf16-exact random weights (config 2); a few chunks the oracle can afford."""
    import torch
    cfg = li.BASE
    say("base-shape sample, seed cfg2")
    w = li.encoder_weights(cfg, li.config_seed(2), bf16_exact=True)
    tokens, lengths = li.uniform_chunks(40, 256, 1, cfg["vocab"], 64, 256, li.config_seed(2) + 1)
    lengths[:5] = [1, 33, 64, 200, 256]
    ctx = L.leann_create(cfg, to_dev(w).to(torch.bfloat16))  # bf16 weight upload path
    try:
        got = L.leann_embed(ctx, to_dev(tokens), to_dev(lengths), hidden=768).cpu().numpy()  # 5466 tokens: tiles of 256 x 256, 256 x 192 and 128 x 192
        L.leann_set_gemm_tiles(ctx, 128, 0)  # the same pass through 128 x 128 tiles: the same bits
        assert np.array_equal(L.leann_embed(ctx, to_dev(tokens), to_dev(lengths), hidden=768).cpu().numpy(), got)
        with pytest.raises(L.LeannError):
            L.leann_set_gemm_tiles(ctx, 192, 0)
    finally:
        L.leann_destroy(ctx)
    ids = np.array([0, 1, 2, 3, 4, 17], np.int64)
    e = orc.desc(**cfg)
    want = orc.embed(e, w, tokens, lengths, ids=ids)
    want_bf = orc.embed(e, w, tokens, lengths, ids=ids, precision=1)
    assert np.isfinite(got).all()
    assert np.abs(got[ids] - want).max() <= TOL_FP32
    assert np.abs(got[ids] - want_bf).max() <= TOL_BF16_MODE
    print("base sample max-abs vs fp32 oracle %.3e, vs bf16-mode oracle %.3e" %
          (np.abs(got[ids] - want).max(), np.abs(got[ids] - want_bf).max()))


def test_small_shape_sample_matches_oracle(L, orc):
    """The 12 x 384 encoder (second throughput point; widths that are not multiples of 256 leave half of the 256-wide
    GEMM tile's last column tile empty) at seq 256; a few chunks against the oracle."""
    import torch
    cfg = li.SMALL
    say("small-shape sample (12 x 384)")
    w = li.encoder_weights(cfg, li.config_seed(2) + 7, bf16_exact=True)
    tokens, lengths = li.uniform_chunks(300, 256, 1, cfg["vocab"], 64, 256, li.config_seed(2) + 8)
    lengths[:4] = [1, 47, 129, 256]
    ctx = L.leann_create(cfg, to_dev(w).to(torch.bfloat16))
    try:
        got = L.leann_embed(ctx, to_dev(tokens), to_dev(lengths), hidden=384).cpu().numpy()
    finally:
        L.leann_destroy(ctx)
    ids = np.array([0, 1, 2, 3, 150, 299], np.int64)
    e = orc.desc(**cfg)
    want = orc.embed(e, w, tokens, lengths, ids=ids)
    want_bf = orc.embed(e, w, tokens, lengths, ids=ids, precision=1)
    assert np.isfinite(got).all()
    assert np.abs(got[ids] - want).max() <= TOL_FP32
    assert np.abs(got[ids] - want_bf).max() <= TOL_BF16_MODE
    print("small sample max-abs vs fp32 oracle %.3e, vs bf16-mode oracle %.3e" %
          (np.abs(got[ids] - want).max(), np.abs(got[ids] - want_bf).max()))


def test_width_256_large_and_small_gemm_tiles(L, orc):
    """hidden = 256: the 256 x 256 GEMM tile with K = 256 (eight K-slabs, the fewest it is launched for: no
    full group of four before the tail) and K = 1024; ragged rows; against the oracle.  The same chunks embedded in
    smaller passes, through the 128 x 128 tile and the stream tiles, give the same bits (all tiles add the K-slabs in one
    order)."""
    import torch
    cfg = dict(layers=3, hidden=256, heads=4, ffn=1024, vocab=2000, max_pos=128, ln_eps=1e-12)
    say("width-256 encoder, large and small GEMM tile")
    w = li.encoder_weights(cfg, li.config_seed(2) + 21, bf16_exact=True)
    tokens, lengths = li.uniform_chunks(600, 128, 1, cfg["vocab"], 16, 128, li.config_seed(2) + 22)
    lengths[:4] = [1, 31, 77, 128]
    ctx = L.leann_create(cfg, to_dev(w).to(torch.bfloat16))
    try:
        t, l = to_dev(tokens), to_dev(lengths)
        passes = {}
        for m, tiles in ((600, {"256x256"}), (100, {"128x128", "stream 64x128"}), (16, {"stream 32x48", "stream 64x64"})):
            reached = gemm_plan.tiles_of_embed(cfg, lengths[:m], 128)
            assert tiles <= {tile for tile, _, _ in reached}, (m, reached)
            passes[m] = L.leann_embed(ctx, t, l, n_ids=m, hidden=256).cpu().numpy()
        assert {(tile, K) for tile, K, _ in gemm_plan.tiles_of_embed(cfg, lengths, 128)} == {("256x256", 256), ("256x256", 1024)}
        got = passes[600]
    finally:
        L.leann_destroy(ctx)
    assert np.array_equal(got[:100], passes[100])
    assert np.array_equal(got[:16], passes[16])
    ids = np.array([0, 1, 2, 3, 50, 99, 599], np.int64)
    e = orc.desc(**cfg)
    want = orc.embed(e, w, tokens, lengths, ids=ids)
    want_bf = orc.embed(e, w, tokens, lengths, ids=ids, precision=1)
    assert np.isfinite(got).all()
    assert np.abs(got[ids] - want).max() <= TOL_FP32
    assert np.abs(got[ids] - want_bf).max() <= TOL_BF16_MODE
    print("width-256 sample max-abs vs fp32 oracle %.3e, vs bf16-mode oracle %.3e" %
          (np.abs(got[ids] - want).max(), np.abs(got[ids] - want_bf).max()))


EVERY_TILE = [(128, 2, 512), (256, 4, 1024), (384, 6, 1536), (768, 12, 3072)]
EVERY_TILE_CHUNKS = (1, 2, 3, 5, 9, 14, 25, 40, 80, 200, 420)


def every_tile_lengths():
    _, lengths = li.uniform_chunks(420, 128, 1, 500, 16, 128, li.config_seed(2) + 30)
    lengths[:3] = [1, 33, 127]
    return lengths


ONE_ROUND = [(512, 8, 128), (640, 10, 1280), (768, 12, 3072), (1024, 16, 1920)]
ONE_ROUND_CHUNKS = (1, 2, 4, 7, 11, 16, 24, 33, 48, 55, 70, 100, 140, 180)


def one_round_lengths():
    lengths = np.full(180, 64, np.int32)
    lengths[0] = 63  # rows = 64 m - 1, one less than whole tiles
    return lengths


@pytest.mark.parametrize("hidden,heads,ffn", EVERY_TILE)
def test_every_gemm_tile_gives_the_same_bits(L, hidden, heads, ffn):
    """Passes from a handful of tokens to tens of thousands, one to 24 K-slabs, row counts that are no multiple of any tile: each
    chunk's embedding equals the one that the 128 x 128 tile alone gives.  Together with the passes of the next test these go through
    every tile from 32 x 16 to 256 x 192 and 256 x 256, with and without GELU (test_gemm_plan.py counts them)."""
    import torch
    cfg = dict(layers=2, hidden=hidden, heads=heads, ffn=ffn, vocab=500, max_pos=128, ln_eps=1e-12)
    say(f"all GEMM tiles, hidden {hidden}")
    w = li.encoder_weights(cfg, li.config_seed(2) + hidden, bf16_exact=True)
    tokens, _ = li.uniform_chunks(420, 128, 1, cfg["vocab"], 16, 128, li.config_seed(2) + 30)
    ctx = L.leann_create(cfg, to_dev(w).to(torch.bfloat16))
    try:
        t, l = to_dev(tokens), to_dev(every_tile_lengths())
        L.leann_set_gemm_tiles(ctx, 128, 0)
        want = L.leann_embed(ctx, t, l, hidden=hidden).cpu().numpy()
        L.leann_set_gemm_tiles(ctx, 256, 2048)
        assert np.isfinite(want).all()
        for m in EVERY_TILE_CHUNKS:
            got = L.leann_embed(ctx, t, l, n_ids=m, hidden=hidden).cpu().numpy()
            assert np.array_equal(got, want[:m]), m
        L.leann_set_gemm_tiles(ctx, 128, 1)  # stream tiles above 64 x 64 and the 128 x 128 tile only
        for m in (9, 80, 420):
            assert np.array_equal(L.leann_embed(ctx, t, l, n_ids=m, hidden=hidden).cpu().numpy(), want[:m]), m
    finally:
        L.leann_destroy(ctx)


@pytest.mark.parametrize("hidden,heads,ffn", ONE_ROUND)
def test_tiles_of_one_round_give_the_same_bits(L, hidden, heads, ffn):
    """Passes that fill the chip once, from one row tile to those that no longer do, with K a multiple of 384 or not (the slabs behind
    its end are zeros), rows at, below and above a tile's edge: the bits of the 128 x 128 tile of the kernel for large passes."""
    import torch
    cfg = dict(layers=1, hidden=hidden, heads=heads, ffn=ffn, vocab=500, max_pos=64, ln_eps=1e-12)
    n, seq = 180, 64
    tokens, _ = li.uniform_chunks(n, seq, 1, cfg["vocab"], 1, seq, 21)
    ctx = L.leann_create(cfg, to_dev(li.encoder_weights(cfg, 22, perturb=True, bf16_exact=True)).to(torch.bfloat16))
    try:
        t, l = to_dev(tokens), to_dev(one_round_lengths())
        L.leann_set_gemm_tiles(ctx, 128, 0)
        want = L.leann_embed(ctx, t, l, hidden=hidden)
        L.leann_set_gemm_tiles(ctx, 256, 2048)
        assert torch.isfinite(want).all()
        for m in ONE_ROUND_CHUNKS:
            say(f"one round of tiles, hidden {hidden}, {m} chunks")
            assert torch.equal(L.leann_embed(ctx, t, l, n_ids=m, hidden=hidden), want[:m]), m
            assert torch.equal(L.leann_embed(ctx, t[1:], l[1:], n_ids=min(m, n - 1), hidden=hidden), want[1:m + 1]), m
    finally:
        L.leann_destroy(ctx)


def weights_of_hard_sums(cfg, seed):
    """Weights whose products are sums of terms of magnitudes from 2^-8 to 2^22 that cancel to a result of order one, so that the
    leading bits of a product already hold what its order of summation and its roundings left over.  Activations come in equal pairs, at random distances
    inside every 64 columns (equal embeddings, scales and rows of the matrix before), and most weights of a pair are opposite.
    Biases from 2^-4 to 2^8 are there from the start of a sum.  {name: fp32 array}, bf16-representable."""
    rng = np.random.Generator(np.random.Philox(seed))
    _, w = li.encoder_weights(cfg, seed, std=1.0, bf16_exact=True, as_dict=True)
    pairs = {}

    def partner(n):  # (p, q): column q[i] holds what column p[i] holds
        if n not in pairs:
            order = np.concatenate([64 * b + rng.permutation(64) for b in range(n // 64)]).reshape(-1, 2)
            pairs[n] = order[:, 0], order[:, 1]
        return pairs[n]

    def equal_rows(a, n):  # of a matrix, or elements of a vector, in blocks of n
        p, q = partner(n)
        for block in a.reshape(-1, n, *a.shape[1:]):
            block[q] = block[p]

    for l in range(cfg["layers"]):
        for name in ("wqkv", "wo", "w1", "w2"):
            a = w[f"l{l}.{name}"]
            a *= 2.0 ** rng.integers(-8, 0, a.shape)  # what does not cancel: of order one in all
            p, q = partner(a.shape[1])
            cancels = rng.random((a.shape[0], p.size)) < 0.7
            big = li.to_bf16_exact(rng.standard_normal(cancels.shape, dtype=np.float32)) * 2.0 ** rng.integers(0, 23, cancels.shape)
            a[:, p] = np.where(cancels, big, a[:, p])
            a[:, q] = np.where(cancels, -big, a[:, q])
            b = w[f"l{l}.b" + name[1:]]
            b[:] = li.to_bf16_exact(rng.standard_normal(b.shape, dtype=np.float32)) * 2.0 ** rng.integers(-4, 9, b.shape)
            equal_rows(a, cfg["ffn"] if name == "w1" else cfg["hidden"])
            equal_rows(b, cfg["ffn"] if name == "w1" else cfg["hidden"])
    p, q = partner(cfg["hidden"])
    for name in ("tok_emb", "pos_emb", "seg_emb"):
        w[name][..., q] = w[name][..., p]
    return {name: a.astype(np.float32) for name, a in w.items()}


def pack_weights(cfg, w):
    return np.concatenate([w[name].reshape(-1) for name, _, _ in li.weight_layout(cfg)]).astype(np.float32)


@pytest.mark.parametrize("hidden,heads,ffn,tiles", [(128, 2, 512, {"32x16", "32x32", "32x64"}), (256, 4, 128, {"32x16", "32x32", "32x64", "64x64"}),
                                                    (768, 12, 3072, {"32x16", "32x32", "32x48", "32x64", "64x64"})])
def test_sums_that_cancel_have_the_same_bits_in_every_tile(L, hidden, heads, ffn, tiles):
    """The smallest passes multiply by MFMA 16x16x32 where the others do by 32x32x16: that one of the former rounds like two of the
    latter is what a chunk's embedding relies on.  Sums whose roundings are a third of them would show a difference; K from 128 to 3072."""
    import torch
    cfg = dict(layers=1, hidden=hidden, heads=heads, ffn=ffn, vocab=300, max_pos=32, ln_eps=1e-12)
    say(f"sums that cancel, hidden {hidden}, ffn {ffn}")
    n, seq = 60, 32
    tokens, lengths = li.uniform_chunks(n, seq, 1, cfg["vocab"], 1, seq, 41)
    lengths[0] = 1
    t, l = to_dev(tokens), to_dev(lengths)
    w = weights_of_hard_sums(cfg, 42)

    def embed(w, counts, large_tile, small_rows):
        ctx = L.leann_create(cfg, to_dev(pack_weights(cfg, w)))
        try:
            L.leann_set_gemm_tiles(ctx, large_tile, small_rows)
            return [L.leann_embed(ctx, t, l, n_ids=m, hidden=hidden) for m in counts]
        finally:
            L.leann_destroy(ctx)

    want = embed(w, (n,), 128, 0)[0]
    assert torch.isfinite(want).all()
    counts = (1, 2, 4, 8, 13, 20, 30, n)
    reached = set().union(*(gemm_plan.tiles_of_embed(cfg, lengths[:m], seq) for m in counts))
    assert {"stream " + tile for tile in tiles} <= {tile for tile, _, _ in reached}
    for m, got in zip(counts, embed(w, counts, 256, 2048)):
        assert torch.equal(got, want[:m]), m
    # another order of the same sums is another result: the FFN's units moved on by eight
    moved = dict(w)
    for name, axis in (("l0.w1", 0), ("l0.b1", 0), ("l0.w2", 1)):
        moved[name] = np.roll(w[name], 8, axis)
    other = embed(moved, (n,), 128, 0)[0]
    assert (other != want).float().mean() > 0.5


def test_weights_that_fit_the_device_once(L):
    """A device that has not the room for the second copy of the layers' matrices: a context is made without it, or a larger pass
    takes its place.  Small and large passes give the bits of a context that has memory."""
    import torch
    cfg = dict(layers=192, hidden=1024, heads=16, ffn=4096, vocab=500, max_pos=256, ln_eps=1e-12)
    matrices = cfg["layers"] * 2 * (4 * 1024 * 1024 + 2 * 1024 * 4096)  # bytes, once: 4.8 GB
    say("weights that fit the device once")
    count = sum(int(np.prod(shape)) for _, shape, _ in li.weight_layout(cfg))
    w = torch.randn(count, generator=torch.Generator("cuda:0").manual_seed(5), device="cuda:0", dtype=torch.bfloat16) * 0.03
    tokens, lengths = li.uniform_chunks(600, 256, 1, cfg["vocab"], 1, 20, 31)
    t, l = to_dev(tokens), to_dev(lengths)
    free = lambda: torch.cuda.mem_get_info()[0]

    def with_room_for(room, use):
        """`use`, while other allocations leave about `room` bytes of the device (up to half a gigabyte more has been seen)."""
        torch.cuda.empty_cache()
        hold = torch.empty(free() - room, dtype=torch.uint8, device="cuda:0")
        try:
            return use()
        finally:
            del hold
            torch.cuda.empty_cache()

    def embed(ctx, counts=(1, 600)):  # 600: workspaces for 153 600 padded rows, 3.1 GB
        return [L.leann_embed(ctx, t, l, n_ids=m, hidden=1024) for m in counts]

    before = free()
    ctx = L.leann_create(cfg, w)
    try:
        assert before - free() >= 2 * matrices - (64 << 20)
        want = embed(ctx)
    finally:
        L.leann_destroy(ctx)

    def without():
        ctx = L.leann_create(cfg, w)
        try:
            return free(), embed(ctx, (1, 8))
        finally:
            L.leann_destroy(ctx)

    left, got = with_room_for(matrices + (3 << 29), without)
    assert left > 1 << 30  # a second copy would have left next to nothing
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1][:8])

    ctx = L.leann_create(cfg, w)
    try:
        assert torch.equal(embed(ctx, (1,))[0], want[0])
        before, got, after = with_room_for(1 << 30, lambda: (free(), embed(ctx), free()))
        assert after > before  # 3.1 GB taken, 4.8 given back
        for a, b in zip(got, want):
            assert torch.isfinite(a).all() and torch.equal(a, b)
    finally:
        L.leann_destroy(ctx)


@pytest.mark.parametrize("hidden,heads,ffn", [(128, 2, 128), (384, 6, 1536), (768, 12, 3072)])
def test_small_passes_of_any_fill_give_the_same_bits(L, hidden, heads, ffn):
    """A small pass requests its operands for the rows that it likely holds, before it knows how many there are: chunks that are
    full, hold one token, or are mixed, from one chunk to a few row tiles, one K-slab to 24, give the bits of the 128 x 128 tile."""
    import torch
    cfg = dict(layers=2, hidden=hidden, heads=heads, ffn=ffn, vocab=500, max_pos=48, ln_eps=1e-12)
    n, seq = 21, 48
    tokens, mixed = li.uniform_chunks(n, seq, 1, cfg["vocab"], 1, seq, 11)
    ctx = L.leann_create(cfg, to_dev(li.encoder_weights(cfg, 12, bf16_exact=True)).to(torch.bfloat16))
    try:
        t = to_dev(tokens)
        for name, lengths in (("full", np.full(n, seq)), ("one token", np.ones(n)), ("mixed", mixed)):
            say(f"small passes, fill {name}, hidden {hidden}")
            l = to_dev(lengths.astype(np.int32))
            L.leann_set_gemm_tiles(ctx, 128, 0)
            want = L.leann_embed(ctx, t, l, hidden=hidden)
            L.leann_set_gemm_tiles(ctx, 256, 2048)
            assert torch.isfinite(want).all()
            for m in (1, 2, 3, 7, 14, n):
                assert torch.equal(L.leann_embed(ctx, t, l, n_ids=m, hidden=hidden), want[:m]), m
    finally:
        L.leann_destroy(ctx)


@pytest.mark.parametrize("hidden,heads,ffn", [(128, 2, 512), (384, 6, 1536)])
def test_pass_without_a_valid_token(L, hidden, heads, ffn):
    """Every requested chunk is outside the store, or its length is: the pass holds no token, whatever product kernel its
    size would pick (one chunk up to passes beyond the small tiles).  The call is an error, and the next one is served."""
    import torch
    cfg = dict(layers=1, hidden=hidden, heads=heads, ffn=ffn, vocab=500, max_pos=64, ln_eps=1e-12)
    tokens, lengths = li.uniform_chunks(40, 64, 1, cfg["vocab"], 16, 64, 3)
    ctx = L.leann_create(cfg, to_dev(li.encoder_weights(cfg, 5)))
    try:
        t, l = to_dev(tokens), to_dev(lengths)
        want = L.leann_embed(ctx, t, l, hidden=hidden)
        for m in (1, 4, 12, 24, 40, 200):
            say(f"no valid token, hidden {hidden}, {m} chunks")
            with pytest.raises(L.LeannError, match="chunk id outside the store"):
                L.leann_embed(ctx, t, l, ids=torch.full((m,), 40, dtype=torch.int64, device="cuda:0"), hidden=hidden)
            with pytest.raises(L.LeannError, match="length outside"):
                L.leann_embed(ctx, t, torch.full_like(l, 65), ids=torch.arange(m, device="cuda:0") % 40, hidden=hidden)
            assert torch.equal(L.leann_embed(ctx, t, l, hidden=hidden), want)
    finally:
        L.leann_destroy(ctx)


@pytest.mark.parametrize("hidden,heads,ffn", [(128, 2, 512), (768, 12, 3072)])
def test_tiles_for_any_fill_give_the_same_bits(L, hidden, heads, ffn):
    """How full the chunks are decides the tiles of passes of more than 4096 padded rows: full, a quarter full, nearly empty and
    mixed chunks, in one pass and in several, give the bits that the 128 x 128 tile alone gives; a bad length in such a
    pass is still an error."""
    import torch
    cfg = dict(layers=2, hidden=hidden, heads=heads, ffn=ffn, vocab=500, max_pos=64, ln_eps=1e-12)
    n, seq = 150, 64
    tokens, mixed = li.uniform_chunks(n, seq, 1, cfg["vocab"], 1, seq, 4)
    ctx = L.leann_create(cfg, to_dev(li.encoder_weights(cfg, 6, bf16_exact=True)).to(torch.bfloat16))
    try:
        t = to_dev(tokens)
        for name, lengths in (("full", np.full(n, seq)), ("quarter", np.full(n, seq // 4)), ("one token", np.ones(n)), ("mixed", mixed)):
            say(f"fill {name}, hidden {hidden}")
            l = to_dev(lengths.astype(np.int32))
            L.leann_set_gemm_tiles(ctx, 128, 0)
            want = L.leann_embed(ctx, t, l, hidden=hidden)
            L.leann_set_gemm_tiles(ctx, 256, 2048)
            assert torch.isfinite(want).all()
            for per_pass in (262144, 75 * seq):
                L.leann_set_limits(ctx, max_tokens_per_pass=per_pass)
                assert torch.equal(L.leann_embed(ctx, t, l, hidden=hidden), want)
        bad = mixed.copy()
        bad[n - 1] = seq + 1
        with pytest.raises(L.LeannError, match="length outside"):
            L.leann_embed(ctx, t, to_dev(bad), hidden=hidden)
    finally:
        L.leann_destroy(ctx)
