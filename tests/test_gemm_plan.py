"""CPU checks of the encoder's choice of GEMM tiles (csrc/gemm_plan.h)."""
import pytest

import gemm_plan
import test_gpu_encoder as gpu

WIDTHS = range(128, 1025, 128)
ROWS = sorted({int(1.03 ** i) for i in range(330)} | {31, 32, 33, 63, 64, 65, 127, 128, 129, 2048, 2049})  # 1 to 16 800


def products(d):
    for F in (128, d, 2 * d, 4 * d):
        yield from ((3 * d, d, False), (d, d, False), (F, d, True), (d, F, False))


@pytest.mark.parametrize("d", WIDTHS)
def test_a_stream_tile_is_taken_where_its_blocks_fit_the_chip_at_once(d):
    """One block per CU; the tiles of 64x64 and smaller only
    up to the row limit; the tiles of 256 rows only with K-slabs enough for its pipeline."""
    area = lambda size: size[0] * size[1]
    for N, K, _ in products(d):
        for rows in ROWS:
            name = gemm_plan.tile(rows, N, K)
            size = tuple(int(v) for v in name.split()[-1].split("x"))
            blocks = lambda s: -(-rows // s[0]) * -(-N // s[1])
            if name.startswith("stream"):
                assert blocks(size) <= gemm_plan.CUS
                assert area(size) > 4096 or rows <= 2048
            else:
                assert size[0] == 128 or K >= 256
            assert not gemm_plan.tile(rows, N, K, small_rows=0).startswith("stream")
            assert not gemm_plan.tile(rows, N, K, large_tile=128).startswith("256x")


def test_every_tile_is_taken_by_some_product():
    taken = {(gemm_plan.tile(rows, N, K), gelu) for d in WIDTHS for N, K, gelu in products(d) for rows in ROWS}
    assert taken == {(tile, gelu) for tile in gemm_plan.stream_tiles() + gemm_plan.LARGE_TILES for gelu in (False, True)}


def test_the_passes_that_the_gpu_tests_compare_reach_every_tile():
    """The tests that compare tiles bit for bit launch each of them, with and without GELU, and stream tiles with K both a multiple of
    their loop's 384 and not."""
    every = {(tile, gelu) for tile in gemm_plan.stream_tiles() + gemm_plan.LARGE_TILES for gelu in (False, True)}
    reached = set()
    for shapes, counts, lengths, seq in ((gpu.EVERY_TILE, gpu.EVERY_TILE_CHUNKS, gpu.every_tile_lengths(), 128),
                                         (gpu.ONE_ROUND, gpu.ONE_ROUND_CHUNKS, gpu.one_round_lengths(), 64)):
        for hidden, _, ffn in shapes:
            for m in counts:
                reached |= gemm_plan.tiles_of_embed(dict(hidden=hidden, ffn=ffn), lengths[:m], seq)
    assert {(tile, gelu) for tile, _, gelu in reached} == every
    for tile in gemm_plan.stream_tiles():
        if tile != "stream 32x128":  # taken at K = 128 only
            assert {K % 384 == 0 for t, K, _ in reached if t == tile} == {False, True}, tile
