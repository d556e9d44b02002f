"""The training rows of leann_build_pq: the seeded permutation, whose steps the device resolves side by side, against the oracle's, which runs them
one after the other."""
import numpy as np
import pytest

import leann_inputs as li
from gpu_util import say, to_dev

pytestmark = pytest.mark.gpu
TRAIN_MAX = 65536


@pytest.fixture(scope="module")
def L():
    import paper_2506_08276_amd as L
    L.load_library()
    return L


@pytest.fixture(scope="module")
def ctx(L):
    ctx = L.leann_create(li.TINY, to_dev(li.encoder_weights(li.TINY, 3)))
    yield ctx
    L.leann_destroy(ctx)


def codebook(L, ctx, x, iters, seed):
    pq = L.leann_build_pq(ctx, to_dev(x), 1, iters, seed)
    try:
        return L.leann_pq_export(ctx, pq)[0].reshape(256, x.shape[1])
    finally:
        L.leann_pq_free(pq)


@pytest.mark.parametrize("n,seed", [(1, 0), (2, 1), (3, 1234567), (255, 9), (256, 2 ** 64 - 1), (257, 5), (1000, 42), (4096, 12), (4097, 13), (5001, 14),
                                    (65535, 3), (65536, 7), (65537, 8), (300001, 2 ** 63 + 11)])
def test_first_training_rows(L, orc, ctx, n, seed):
    """Without an iteration the codebook is the first 256 training rows, exactly."""
    say(f"training rows, n={n} seed={seed}")
    i = np.arange(n)
    x = np.stack([i & 4095, i >> 12], 1).astype(np.float32)  # a row for every number, exact in fp32
    perm = orc.permutation(n, seed)[:min(n, TRAIN_MAX)]
    assert np.array_equal(codebook(L, ctx, x, 0, seed), x[perm[np.arange(256) % len(perm)]])


@pytest.mark.parametrize("n,seed", [(65537, 4), (100003, 6)])
def test_all_training_rows(L, orc, ctx, n, seed):
    """One iteration's means over the training rows: of some 256 rows each, at most 2^17.  A mean's fp32 sum is off by 2^-24 of itself per addition
    in the longest chain, 8 pairwise steps and the rows of one partial sum (fewer than 16): 2e-6 of the largest value.  A wrong row moves the mean
    of a centroid of 256 rows by more, unless the two are 50 apart or less."""
    say(f"all training rows, n={n} seed={seed}")
    x = np.arange(n, dtype=np.float32)[:, None]
    train = x[orc.permutation(n, seed)[:TRAIN_MAX], 0].astype(np.float64)
    cent = train[:256]
    nearest = np.argmin(np.abs(train[:, None] - cent[None, :]), 1)
    want = np.array([train[nearest == c].mean() for c in range(256)])
    assert np.abs(codebook(L, ctx, x, 1, seed)[:, 0] - want).max() <= 2e-6 * n


def numbered_rows(n):
    """A row for every number, exact in fp32, on the device."""
    import torch
    i = torch.arange(n, dtype=torch.int32, device="cuda:0")
    x = torch.empty((n, 2), dtype=torch.float32, device="cuda:0")
    x[:, 0] = i & 4095
    x[:, 1] = i >> 12
    return x


def first_rows(L, ctx, x, seed):
    pq = L.leann_build_pq(ctx, x, 1, 0, seed)
    try:
        cb = np.empty((256, 2), np.float32)
        import ctypes as C
        L.load_library().leann_pq_export(ctx, pq, cb.ctypes.data_as(C.c_void_p), None)
        return cb.astype(np.int64) @ [1, 4096]
    finally:
        L.leann_pq_free(pq)


def test_a_large_table_leaves_no_more_behind_than_its_training(L, orc):
    """The permutation's steps of a table of 6 000 000 rows are 96 MB, its training's scratch 2.4 MB."""
    import torch
    say("memory kept after a large table")
    ctx = L.leann_create(li.TINY, to_dev(li.encoder_weights(li.TINY, 3)))
    try:
        n, seed = 6_000_000, 21
        x = numbered_rows(n)
        first_rows(L, ctx, x[:5000].contiguous(), seed)  # kernels loaded
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        assert np.array_equal(first_rows(L, ctx, x, seed), orc.permutation(n, seed)[:256])
        assert torch.cuda.mem_get_info()[0] > free - (32 << 20)
    finally:
        L.leann_destroy(ctx)


def test_the_host_runs_the_steps_of_the_largest_tables(L, orc, ctx):
    """More than 2^26 rows: 16 bytes each are more than a context keeps."""
    n, seed = (1 << 26) + 1001, 22
    say(f"steps on the host, n={n}")
    assert np.array_equal(first_rows(L, ctx, numbered_rows(n), seed), orc.permutation(n, seed)[:256])


def test_the_host_runs_the_steps_where_the_device_has_no_room(L, orc, ctx):
    """960 MB of steps beside other allocations that leave 300 MB (up to half a gigabyte more has been seen)."""
    import torch
    n, seed = 60_000_000, 23
    say(f"steps on the host for want of memory, n={n}")
    x = numbered_rows(n)
    torch.cuda.empty_cache()
    hold = torch.empty(torch.cuda.mem_get_info()[0] - (300 << 20), dtype=torch.uint8, device="cuda:0")
    try:
        got = first_rows(L, ctx, x, seed)
    finally:
        del hold
        torch.cuda.empty_cache()
    assert np.array_equal(got, orc.permutation(n, seed)[:256])
