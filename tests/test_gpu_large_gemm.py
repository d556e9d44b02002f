"""The products of large passes (csrc/gemm_large.h): tiles of 256 x 256 and 256 x 192, whole and ragged in rows and columns, give the
bits of the 128 x 128 tile.  All tiles add the same terms in the same order, so the tolerance is none."""
import ctypes
import functools
import os
import subprocess
import tempfile

import numpy as np
import pytest

import gemm_plan
import leann_inputs as li
from gpu_util import say, to_dev

# hidden, heads, FFN width, row counts: K of 8 slabs (the fewest), 12 and 20; widths that are multiples of neither 192 nor 256 (640, 1920,
# 1280); one row more and fewer than whole row tiles, one tile per block and several, blocks without a tile.
SHAPES = [(256, 4, 1024, (20735, 30977, 65536)), (384, 6, 1536, (16129, 24831, 33025, 48640)), (640, 10, 1280, (8191, 12545, 26113))]
SEQ = 256


def lengths_of(rows):
    n = rows // SEQ + 1
    lengths = np.full(n, SEQ, np.int32)
    lengths[-1] = rows - (n - 1) * SEQ
    return lengths if lengths[-1] else lengths[:-1]


@functools.lru_cache(None)
def plan():
    source = gemm_plan.SOURCE + """
extern "C" int columns(int rows, int N, int K)
{
    const GemmChoice c = choose_gemm(256, 256, 2048, rows, N, K);
    return c.stream < 0 && c.large == 256 ? c.cols : 0;
}
"""
    with tempfile.TemporaryDirectory() as d:
        open(os.path.join(d, "plan.cpp"), "w").write(source)
        subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(gemm_plan.ROOT, "paper_2506_08276_amd", "csrc"),
                               "-o", os.path.join(d, "plan.so"), os.path.join(d, "plan.cpp")])
        return ctypes.CDLL(os.path.join(d, "plan.so"))


def reached():
    """{(columns of the tile, K, N, with GELU)} of the passes below."""
    out = set()
    for hidden, _, ffn, counts in SHAPES:
        for rows in counts:
            for N, K, gelu in ((3 * hidden, hidden, False), (hidden, hidden, False), (ffn, hidden, True), (hidden, ffn, False)):
                out.add((plan().columns(rows, N, K), K, N, gelu))
    return out


def test_the_passes_reach_both_tiles():
    for cols in (192, 256):
        mine = {(K, N, gelu) for c, K, N, gelu in reached() if c == cols}
        assert {gelu for _, _, gelu in mine} == {False, True}, cols
        assert any(N % cols for _, N, _ in mine) and any(N % cols == 0 for _, N, _ in mine), cols
    assert 256 in {K for c, K, _, _ in reached() if c}


@pytest.mark.gpu
@pytest.mark.parametrize("hidden,heads,ffn,counts", SHAPES)
def test_large_tiles_give_the_bits_of_the_128_tile(hidden, heads, ffn, counts):
    import torch
    import paper_2506_08276_amd as L
    cfg = dict(layers=1, hidden=hidden, heads=heads, ffn=ffn, vocab=500, max_pos=SEQ, ln_eps=1e-12)
    n = max(counts) // SEQ + 1
    tokens, _ = li.uniform_chunks(n, SEQ, 1, cfg["vocab"], SEQ, SEQ, 51)
    ctx = L.leann_create(cfg, to_dev(li.encoder_weights(cfg, 52, perturb=True, bf16_exact=True)).to(torch.bfloat16))
    try:
        t = to_dev(tokens)
        for rows in counts:
            say(f"large tiles, hidden {hidden}, {rows} rows")
            l = to_dev(lengths_of(rows))
            L.leann_set_gemm_tiles(ctx, 128, 0)
            want = L.leann_embed(ctx, t[:len(l)], l, hidden=hidden)
            L.leann_set_gemm_tiles(ctx, 256, 2048)
            assert torch.isfinite(want).all()
            assert torch.equal(L.leann_embed(ctx, t[:len(l)], l, hidden=hidden), want), rows
    finally:
        L.leann_destroy(ctx)
