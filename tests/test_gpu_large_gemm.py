"""The products of large passes (csrc/gemm_large.h): tiles of 256 x 256 and 256 x 192, whole and ragged in rows and columns, give the
bits of the 128 x 128 tile.  All tiles add the same terms in the same order, so the tolerance is none."""
import numpy as np
import pytest

import gemm_plan
import leann_inputs as li
from gpu_util import say, to_dev

# hidden, heads, FFN width, row counts: K of 8 slabs (the fewest), 12, 20 and 96; widths that are multiples of neither 192 nor 256 (640, 1920,
# 1280); one row more and fewer than whole row tiles, one tile per block and several, blocks without a tile.
SHAPES = [(256, 4, 1024, (20735, 30977, 65536)), (384, 6, 1536, (16129, 24831, 33025, 48640)), (640, 10, 1280, (8191, 12545, 26113)),
          (768, 12, 3072, (11007, 19201))]
SEQ, LAYERS = 256, 8


def lengths_of(rows):
    n = rows // SEQ + 1
    lengths = np.full(n, SEQ, np.int32)
    lengths[-1] = rows - (n - 1) * SEQ
    return lengths if lengths[-1] else lengths[:-1]


def reached(small_rows):
    """{(tile, K, N, with GELU)} of the passes below."""
    out = set()
    for hidden, _, ffn, counts in SHAPES:
        for rows in counts:
            for N, K, gelu in ((3 * hidden, hidden, False), (hidden, hidden, False), (ffn, hidden, True), (hidden, ffn, False)):
                out.add((gemm_plan.tile(rows, N, K, small_rows=small_rows), K, N, gelu))
    return out


@pytest.mark.parametrize("small_rows", [2048, 0])  # 0: as without packed weights
def test_the_passes_reach_both_tiles(small_rows):
    for cols in (192, 256):
        mine = {(K, N, gelu) for tile, K, N, gelu in reached(small_rows) if tile == f"256x{cols}"}
        assert {gelu for _, _, gelu in mine} == {False, True}, cols
        assert any(N % cols for _, N, _ in mine) and any(N % cols == 0 for _, N, _ in mine), cols
        assert 3072 in {K for K, _, _ in mine}, cols
    assert 256 in {K for tile, K, _, _ in reached(small_rows) if tile.startswith("256x")}


def lose_packed_weights(ctx, cfg, largest):
    """A pass whose first workspace finds no memory takes the matrices in operand order for it, and is refused all the same: later calls read
    the rows.  largest: rows of the largest pass so far."""
    import torch
    free = lambda: torch.cuda.mem_get_info()[0]
    n = (1 << 22) // SEQ  # x: 2 to 6 GB
    tokens, lengths = torch.ones((n, SEQ), dtype=torch.int32, device="cuda:0"), torch.ones(n, dtype=torch.int32, device="cuda:0")
    out = torch.empty((n, cfg["hidden"]), dtype=torch.float32, device="cuda:0")
    torch.cuda.empty_cache()
    before = free()
    hold = torch.empty(before - (1 << 30), dtype=torch.uint8, device="cuda:0")
    import paper_2506_08276_amd as L
    try:
        L.leann_set_limits(ctx, max_tokens_per_pass=1 << 22)
        with pytest.raises(L.LeannError) as e:
            L.leann_embed(ctx, tokens, lengths, hidden=cfg["hidden"], out=out)
        assert e.value.status == -2
    finally:
        L.leann_set_limits(ctx, max_tokens_per_pass=1 << 20)
        del hold
        torch.cuda.empty_cache()
    packed = cfg["layers"] * 2 * (4 * cfg["hidden"] ** 2 + 2 * cfg["hidden"] * cfg["ffn"])
    assert free() - before >= 2 * cfg["hidden"] * largest + packed - (8 << 20)  # with the workspace that made room for nothing


@pytest.mark.gpu
@pytest.mark.parametrize("hidden,heads,ffn,counts", SHAPES)
def test_large_tiles_give_the_bits_of_the_128_tile(hidden, heads, ffn, counts):
    """With weights in operand order, and in rows."""
    import torch
    import paper_2506_08276_amd as L
    cfg = dict(layers=LAYERS, hidden=hidden, heads=heads, ffn=ffn, vocab=500, max_pos=SEQ, ln_eps=1e-12)
    n = max(counts) // SEQ + 1
    tokens, _ = li.uniform_chunks(n, SEQ, 1, cfg["vocab"], SEQ, SEQ, 51)
    ctx = L.leann_create(cfg, to_dev(li.encoder_weights(cfg, 52, perturb=True, bf16_exact=True)).to(torch.bfloat16))
    try:
        t = to_dev(tokens)
        want = {}
        for rows in counts:
            say(f"large tiles, hidden {hidden}, {rows} rows")
            l = to_dev(lengths_of(rows))
            L.leann_set_gemm_tiles(ctx, 128, 0)
            want[rows] = L.leann_embed(ctx, t[:len(l)], l, hidden=hidden)
            L.leann_set_gemm_tiles(ctx, 256, 2048)
            assert torch.isfinite(want[rows]).all()
            assert torch.equal(L.leann_embed(ctx, t[:len(l)], l, hidden=hidden), want[rows]), rows
        lose_packed_weights(ctx, cfg, max(counts))
        for rows in counts:
            say(f"large tiles, rows of W, hidden {hidden}, {rows} rows")
            l = to_dev(lengths_of(rows))
            assert torch.equal(L.leann_embed(ctx, t[:len(l)], l, hidden=hidden), want[rows]), rows
    finally:
        L.leann_destroy(ctx)
