"""CPU checks of the addresses at which the kernel of large products requests W (csrc/gemm_requests.h), compiled here with g++."""
import os
import subprocess

import pytest

import gemm_plan

# Every request of every wavefront, lane and K-slab of every column tile.  A buffer's bounds are checked against the lane's offset, the only one that a request
# has: it reads all 16 bytes inside of its buffer and of W, or, of columns beyond N, nothing.
SOURCE = """
#include <stdio.h>
#include <stdlib.h>
#include <vector>
#include "gemm_requests.h"
int main(int argc, char **argv)
{
    const int N = atoi(argv[1]), K = atoi(argv[2]), BN = atoi(argv[3]), packed = atoi(argv[4]);
    std::vector<char> seen((size_t)N * K / 8);  // 16-byte pieces of W
    for (int col = 0; col < (N + BN - 1) / BN * BN; col += 32)
        for (int slab = 0; slab < K / 32; ++slab) {
            const WeightSlab w = weight_slab(col, slab, N, K, packed);
            for (int part = 0; part < 2; ++part)
                for (int lane = 0; lane < 64; ++lane) {
                    const int at = weight_offset(lane, part, K, packed);
                    if (at < 0 || w.bytes < 0) return printf("column %d slab %d lane %d: %d of %d\\n", col, slab, lane, at, w.bytes), 1;
                    if (at >= w.bytes && col >= N) continue;  // nothing is fetched
                    const int64_t byte = w.first * 2 + at;
                    if (at + 16 > w.bytes || byte < 0 || byte + 16 > (int64_t)N * K * 2)
                        return printf("column %d slab %d lane %d: %d of %d\\n", col, slab, lane, at, w.bytes), 1;
                    if (seen[byte / 16]++) return printf("column %d slab %d lane %d: twice\\n", col, slab, lane), 1;
                }
        }
    for (char c : seen)
        if (!c) return printf("not all of W\\n"), 1;
    return 0;
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    d = tmp_path_factory.mktemp("requests")
    (d / "walk.cpp").write_text(SOURCE)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(gemm_plan.ROOT, "paper_2506_08276_amd", "csrc"), "-o", str(d / "walk"),
                           str(d / "walk.cpp")])
    return str(d / "walk")


@pytest.mark.parametrize("N,K", [(128, 256), (256, 256), (384, 384), (384, 1536), (640, 1280), (1152, 384), (768, 3072), (1920, 1024)])
@pytest.mark.parametrize("cols", [192, 256])
@pytest.mark.parametrize("packed", [0, 1])
def test_requests_stay_in_w_whatever_the_last_column_tile_reaches(walk, N, K, cols, packed):
    r = subprocess.run([walk, *map(str, (N, K, cols, packed))], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
