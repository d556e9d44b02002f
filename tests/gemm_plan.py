"""The encoder's choice of GEMM tiles (csrc/gemm_plan.h, plain host code, compiled here with g++): which tile each product of a
pass goes through, for tests that have to know what they reached."""
import ctypes
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CUS = 256
SOURCE = """
#include "gemm_plan.h"
#define SIZE(W, R, NM, US, US_K) {W * R, W * NM},
static const int sizes[][2] = {LEANN_STREAM_TILES(SIZE)};
extern "C" int tiles() { return sizeof(sizes) / sizeof(sizes[0]); }
extern "C" void tile_size(int tile, int *rows, int *cols) { *rows = sizes[tile][0], *cols = sizes[tile][1]; }
extern "C" void choose(int cus, int large_tile, int small_rows, int rows, int N, int K, int *stream, int *xr, int *large, int *cols)
{
    const GemmChoice c = choose_gemm(cus, large_tile, small_rows, rows, N, K);
    *stream = c.stream, *xr = c.xr, *large = c.large, *cols = c.cols;
}
extern "C" int pass_rows(int max_rows, int tokens) { return max_rows > ASK_ROWS ? tokens : guessed_rows(max_rows); }
"""


@functools.lru_cache(None)
def library():
    with tempfile.TemporaryDirectory() as d:
        open(os.path.join(d, "plan.cpp"), "w").write(SOURCE)
        subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2506_08276_amd", "csrc"),
                               "-o", os.path.join(d, "plan.so"), os.path.join(d, "plan.cpp")])
        return ctypes.CDLL(os.path.join(d, "plan.so"))


LARGE_TILES = ["128x128", "256x256", "256x192"]


def stream_tiles():
    """Names of the stream kernels' tiles."""
    out = []
    for i in range(library().tiles()):
        rows, cols = ctypes.c_int(), ctypes.c_int()
        library().tile_size(i, ctypes.byref(rows), ctypes.byref(cols))
        out.append(f"stream {rows.value}x{cols.value}")
    return out


def tile(rows, N, K, large_tile=256, small_rows=2048):
    """The tile of one product."""
    stream, xr, large, cols = ctypes.c_int(), ctypes.c_int(), ctypes.c_int(), ctypes.c_int()
    library().choose(CUS, large_tile, small_rows, rows, N, K, ctypes.byref(stream), ctypes.byref(xr), ctypes.byref(large), ctypes.byref(cols))
    return stream_tiles()[stream.value] if stream.value >= 0 else f"{large.value}x{cols.value}"


def tiles_of_embed(cfg, lengths, seq, **setting):
    """{(tile, K, with GELU)} of leann_embed's products for chunks of these lengths, one pass of `seq` tokens each."""
    rows = library().pass_rows(len(lengths) * seq, int(sum(lengths)))
    d, F = cfg["hidden"], cfg["ffn"]
    return {(tile(rows, N, K, **setting), K, gelu) for N, K, gelu in ((3 * d, d, False), (d, d, False), (F, d, True), (d, F, False))}
