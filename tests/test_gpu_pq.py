"""GPU parity: leann_adc / leann_build_pq / PQ import-export against the PQ oracle.

ADC bound (spec: 1e-4 relative): |gpu - oracle| <= 1e-4 * |oracle| (every term of the sum has the same
sign, so the sum's own magnitude is its forward-error scale).  k-means itself is not compared bit for bit (Lloyd iterations amplify rounding); the built table
is judged by its invariants and by its quantisation error against the oracle's.
"""
import numpy as np
import pytest

import leann_inputs as li
from gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import paper_2506_08276_amd as L
    L.load_library()
    return L


@pytest.fixture(scope="module")
def ctx(L):
    c = L.leann_create(li.TINY, to_dev(li.encoder_weights(li.TINY, 1)))
    yield c
    L.leann_destroy(c)


def unit_rows(n, d, seed, clusters=20):
    rng = np.random.default_rng(seed)
    cent = rng.standard_normal((clusters, d))
    x = cent[rng.integers(0, clusters, n)] + 0.4 * rng.standard_normal((n, d))
    return (x / np.linalg.norm(x, axis=1, keepdims=True)).astype(np.float32)


@pytest.mark.parametrize("d,m_sub,n,nc", [(128, 16, 3000, 77), (768, 32, 5000, 1500), (64, 4, 300, 1)])
def test_adc_matches_oracle(L, orc, ctx, d, m_sub, n, nc):
    say(f"adc d={d} m_sub={m_sub} n={n} nc={nc}")
    x = unit_rows(n, d, 3)
    cb, _ = orc.pq_train(x, m_sub, 3, 5)
    codes = orc.pq_encode(x, cb)
    pq = L.leann_pq_import(ctx, cb, codes)
    rng = np.random.default_rng(4)
    nq = 9
    queries = unit_rows(nq, d, 6)
    cand = rng.integers(0, n, size=(nq, nc)).astype(np.uint32)
    cand[0, 0], cand[-1, -1] = 0, n - 1
    got = L.leann_adc(ctx, to_dev(queries), pq, to_dev(cand)).cpu().numpy()
    for qi in range(nq):
        want, l1 = orc.adc(orc.lut(queries[qi], cb), codes, cand[qi])
        assert np.all(np.abs(got[qi] - want) <= 1e-4 * np.maximum(np.abs(want), l1))
    cb2, codes2 = L.leann_pq_export(ctx, pq)
    assert np.array_equal(cb2, cb) and np.array_equal(codes2, codes)
    assert L.leann_pq_info(pq) == (n, d, m_sub)
    # wrapped device-resident codes give the same scores
    import torch
    codes_dev = to_dev(codes)
    pq_w = L.leann_pq_wrap(ctx, cb, codes_dev)
    got_w = L.leann_adc(ctx, to_dev(queries), pq_w, to_dev(cand))
    assert torch.equal(got_w.cpu(), torch.from_numpy(got))
    L.leann_pq_free(pq_w)
    # an id outside the table is reported
    cand[2, 0] = n
    with pytest.raises(L.LeannError):
        L.leann_adc(ctx, to_dev(queries), pq, to_dev(cand))
    L.leann_pq_free(pq)


@pytest.mark.parametrize("m_sub,d", [(32, 768), (16, 128)])
def test_adc_many_queries_several_rounds_per_block(L, orc, ctx, m_sub, d):
    """Launch shapes in which a block of the scorer goes through several rounds of 2048 candidates with its lookup
    table kept in LDS, and a query's candidates are split over several blocks (9000 queries x 4100 candidates: two
    blocks per query, two rounds in the first, a ragged one in the second): sampled queries against the oracle, and
    the whole result against the same candidates scored 1500 at a time (one round per block)."""
    import torch
    n, nq, nc = 5000, 9000, 4100
    say(f"adc multi-round d={d} m_sub={m_sub} nq={nq} nc={nc}")
    x = unit_rows(n, d, 3)
    cb, _ = orc.pq_train(x, m_sub, 2, 5)
    codes = orc.pq_encode(x, cb)
    pq = L.leann_pq_import(ctx, cb, codes)
    queries = unit_rows(nq, d, 8)
    g = torch.Generator(device="cpu").manual_seed(5)
    cand = torch.randint(0, n, (nq, nc), dtype=torch.int32, generator=g)
    qd, cd = to_dev(queries), cand.to("cuda:0")
    got = L.leann_adc(ctx, qd, pq, cd)
    for s0 in range(0, nc, 1500):
        part = L.leann_adc(ctx, qd, pq, cd[:, s0:s0 + 1500].contiguous())
        assert torch.equal(got[:, s0:s0 + 1500], part), s0
    got = got.cpu().numpy()
    cand = cand.numpy().view(np.uint32)
    for qi in (0, 4499, 8999):
        want, l1 = orc.adc(orc.lut(queries[qi], cb), codes, cand[qi])
        assert np.all(np.abs(got[qi] - want) <= 1e-4 * np.maximum(np.abs(want), l1))
    L.leann_pq_free(pq)


@pytest.mark.parametrize("m_sub,d", [(32, 768), (3, 51), (20, 20), (96, 768)])
def test_adc_with_and_without_table_give_the_same_bits(L, ctx, m_sub, d):
    """Calls of at most 256 candidates per query compute the table entries they need, longer ones look them up: the same
    candidates as part of a longer list score bit for bit the same.  A bad id is an error on both ways."""
    import torch
    n, nq = 1000, 5
    say(f"adc direct and by table m_sub={m_sub} d={d}")
    rng = np.random.default_rng(m_sub)
    codes = rng.integers(0, 256, size=(n, m_sub)).astype(np.uint8)
    pq = L.leann_pq_import(ctx, (0.1 * rng.standard_normal((m_sub, 256, d // m_sub))).astype(np.float32), codes)
    q = to_dev(unit_rows(nq, d, 2))
    cand = to_dev(rng.integers(0, n, size=(nq, 300)).astype(np.int32))
    want = L.leann_adc(ctx, q, pq, cand)
    for nc in (1, 15, 16, 17, 64, 256):
        assert torch.equal(L.leann_adc(ctx, q, pq, cand[:, :nc].contiguous()), want[:, :nc]), nc
    for nc in (40, 300):
        bad = cand[:, :nc].clone()
        bad[nq - 1, nc - 1] = n
        with pytest.raises(L.LeannError):
            L.leann_adc(ctx, q, pq, bad)
        assert torch.equal(L.leann_adc(ctx, q, pq, cand[:, :nc].contiguous()), want[:, :nc])
    L.leann_pq_free(pq)


@pytest.mark.parametrize("n,d,m_sub,iters", [(2000, 128, 16, 10), (70000, 48, 2, 3)])
def test_build_pq_invariants_and_error(L, orc, ctx, n, d, m_sub, iters):
    say(f"build_pq n={n} d={d} m_sub={m_sub} iters={iters}")
    x = unit_rows(n, d, 11, clusters=300)
    pq = L.leann_build_pq(ctx, to_dev(x), m_sub, iters, 99)
    cb, codes = L.leann_pq_export(ctx, pq)
    L.leann_pq_free(pq)
    assert cb.shape == (m_sub, 256, d // m_sub) and codes.shape == (n, m_sub) and np.isfinite(cb).all()
    dsub = d // m_sub
    sample = np.random.default_rng(0).choice(n, 500, replace=False)
    err_gpu = 0.0
    for m in range(m_sub):
        sub = x[sample, m * dsub:(m + 1) * dsub].astype(np.float64)
        dist = ((sub[:, None, :] - cb[m][None].astype(np.float64)) ** 2).sum(-1)
        chosen = dist[np.arange(len(sample)), codes[sample, m]]
        assert np.all(chosen <= dist.min(1) + 1e-5)  # every code is a true arg-min of its own codebook
        err_gpu += chosen.sum()
    cb_o, _ = orc.pq_train(x, m_sub, iters, 99)
    dec_o = orc.pq_decode(orc.pq_encode(x[sample], cb_o), cb_o)
    err_orc = ((dec_o.astype(np.float64) - x[sample]) ** 2).sum()
    assert abs(err_gpu - err_orc) <= 0.01 * err_orc  # quantisation error within 1 % of the oracle's
    # same seed, same permutation: the first Lloyd step starts from the same rows, so with iters small and
    # well separated data most centroids agree closely
    close = np.isclose(cb, cb_o, atol=1e-3).all(-1).mean()
    print(f"centroids agreeing with the oracle's to 1e-3: {close:.3f}")
    assert close > 0.5


@pytest.mark.parametrize("n,d,m_sub,offset", [(5, 16, 2, 0), (300, 32, 1, 0), (1000, 51, 3, 0), (777, 20, 20, 0), (640, 40, 2, 0),
                                              (3000, 768, 32, 0), (4097, 48, 2, 4000), (70001, 24, 1, 0)])
def test_build_pq_exact_on_integer_rows(L, ctx, n, d, m_sub, offset):
    """Integer-valued rows: squared distances and sums are exact in fp32, so the nearest centroid (lowest index among
    equals; there are many) and the means have one right value.  Sub-vector lengths 1 to 32, aligned and not, fewer rows
    than centroids, rows far from the origin, non-finite rows, and more rows than are trained on."""
    say(f"build_pq integer rows n={n} d={d} m_sub={m_sub} offset={offset}")
    rng = np.random.default_rng(n + d)
    x = (rng.integers(-6, 7, size=(n, d)) + offset).astype(np.float32)
    dsub = d // m_sub

    def nearest(rows, cb):
        out = np.empty((len(rows), m_sub), np.int64)
        for s in range(0, len(rows), 1000):
            sub = rows[s:s + 1000].reshape(-1, m_sub, 1, dsub).astype(np.float64)
            dist = np.stack([((sub[:, m] - cb[m][None].astype(np.float64)) ** 2).sum(-1) for m in range(m_sub)], 1)
            out[s:s + 1000] = np.where(np.isnan(dist), np.inf, dist).argmin(2)
        return out

    def build(rows, iters):
        pq = L.leann_build_pq(ctx, to_dev(rows), m_sub, iters, 7)
        got = L.leann_pq_export(ctx, pq)
        L.leann_pq_free(pq)
        return got

    cb0, codes0 = build(x, 0)  # the first centroids are rows
    want0 = nearest(x, cb0)
    np.testing.assert_array_equal(codes0, want0)
    if n <= 65536:  # every row is trained on
        cb1, _ = build(x, 1)
        sub = x.reshape(n, m_sub, dsub)
        for m in range(m_sub):
            want = cb0[m].copy()
            for c in np.unique(want0[:, m]):
                own = sub[want0[:, m] == c, m]
                want[c] = own.sum(0, dtype=np.float64).astype(np.float32) / np.float32(len(own))
            np.testing.assert_array_equal(cb1[m], want)
    if n > 256:
        bad = x.copy()
        bad[::97, 0], bad[1::89, d - 1], bad[5, 0] = np.nan, np.inf, -3e38
        cbb, codesb = build(bad, 0)
        with np.errstate(invalid="ignore", over="ignore"):
            want = nearest(bad, cbb)
        rows = np.arange(n) != 5  # 3e38 squared is infinite in fp32 only
        np.testing.assert_array_equal(codesb[rows], want[rows])


@pytest.mark.parametrize("n,d,m_sub", [(300, 64, 8), (1000, 96, 16), (17, 24, 2), (257, 40, 8)])
def test_pq_training_of_rows_at_any_address(L, ctx, n, d, m_sub):
    """Training rows are brought into planes by four elements where they begin at 16 bytes, else one by one, sixteen rows per
    block (here whole blocks, a remainder, fewer): the same table either way."""
    import torch
    say(f"pq training rows, {n} x {d}, {m_sub}")
    x = to_dev(unit_rows(n, d, 12))
    shifted = torch.empty(n * d + 1, dtype=torch.float32, device="cuda:0")[1:].view(n, d)
    shifted.copy_(x)
    tables = []
    for rows in (x, shifted):
        pq = L.leann_build_pq(ctx, rows, m_sub, 3, 5)
        tables.append(L.leann_pq_export(ctx, pq))
        L.leann_pq_free(pq)
    for a, b in zip(*tables):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("n,dsub,longest", [(3000, 4, 255), (3000, 3, 256), (3000, 24, 257), (9000, 32, 6000), (3000, 1, 2999)])
def test_pq_means_of_long_row_lists(L, ctx, n, dsub, longest):
    """Means of centroids with many rows, with as many as are looked through at a time, and one more or fewer: `longest` rows are one
    point and the others lie far from it and from each other.  Integer-valued, so every sum is exact."""
    say(f"pq means n={n} dsub={dsub} longest list {longest}")
    rng = np.random.default_rng(longest)
    x = np.zeros((n, dsub), np.float32)
    x[:, 0] = 100 + 10 * np.arange(n)
    one = rng.permutation(n)[:longest]
    x[one] = 3
    x[one, -1] += rng.integers(-1, 2, longest)  # three points, their nearest centroids the first training rows among them
    cb0, codes0 = codes_of_first_centroids(L, ctx, x, 1)
    pq = L.leann_build_pq(ctx, to_dev(x), 1, 1, 7)
    cb1, _ = L.leann_pq_export(ctx, pq)
    L.leann_pq_free(pq)
    want = cb0[0].copy()
    for c in np.unique(codes0):
        own = x[codes0[:, 0] == c]
        want[c] = own.sum(0, dtype=np.float64).astype(np.float32) / np.float32(len(own))
    np.testing.assert_array_equal(cb1[0], want)


def nearest_by_fp32_sums(rows, cb):
    """Codes by the definition: s(c) = sum over j, ascending, of (x_j - c_j)^2 in fp32 with fused multiply-adds; the smallest
    finite sum, the lowest index among equals, 0 if there is none.  The fused operation is emulated in float64: the
    product of two fp32 values is exact there, and the sum is rounded to odd, so that the rounding to fp32 is the only one
    (53 >= 24 + 2 bits)."""
    m_sub, _, dsub = cb.shape
    out = np.empty((len(rows), m_sub), np.int64)
    with np.errstate(over="ignore", invalid="ignore"):
        for m in range(m_sub):
            x = rows[:, m * dsub:(m + 1) * dsub]
            s = np.zeros((len(rows), 256), np.float32)
            for j in range(dsub):
                t = (x[:, j, None] - cb[m, None, :, j]).astype(np.float64)  # fp32 subtraction
                p, a = t * t, s.astype(np.float64)
                h = p + a
                v = h - p
                err = (p - (h - v)) + (a - v)
                bits = h.view(np.int64)
                even = np.isfinite(err) & (err != 0) & ((bits & 1) == 0)
                s = np.where(even, bits + np.where(err > 0, 1, -1), bits).view(np.float64).astype(np.float32)
            s = np.where(np.isfinite(s), s, np.inf)
            out[:, m] = s.argmin(1)  # the first of the smallest; index 0 where all are infinite
    return out


def test_tables_trained_by_several_threads(L, ctx):
    """Calls on one context from several threads, their sizes growing: each table is the one that a call alone gives."""
    import threading
    say("pq training, three threads")
    rows = [to_dev(unit_rows(n, 48, n)) for n in (700, 3000, 9000)]

    def train(x):
        pq = L.leann_build_pq(ctx, x, 6, 3, 5)
        out = L.leann_pq_export(ctx, pq)
        L.leann_pq_free(pq)
        return out

    got = [None] * 3

    def work(i):
        got[i] = train(rows[i])

    threads = [threading.Thread(target=work, args=(i,)) for i in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for x, (cb, codes) in zip(rows, got):
        cb1, codes1 = train(x)
        np.testing.assert_array_equal(cb, cb1)
        np.testing.assert_array_equal(codes, codes1)


def test_scratch_beyond_what_is_kept_is_given_back(L, ctx):
    """65536 training rows of 4224 elements are more than the 1 GiB that a context keeps; a small table comes out as ever afterwards."""
    import torch
    say("pq scratch above the bound")
    small = to_dev(unit_rows(700, 48, 1))

    def train(x, m_sub):
        pq = L.leann_build_pq(ctx, x, m_sub, 1, 5)
        out = L.leann_pq_export(ctx, pq)
        L.leann_pq_free(pq)
        return out

    before = train(small, 6)
    large = torch.randn((65536, 4224), device="cuda:0", generator=torch.Generator("cuda:0").manual_seed(3))
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    train(large, 132)
    assert torch.cuda.mem_get_info()[0] > free - (64 << 20)
    for a, b in zip(before, train(small, 6)):
        np.testing.assert_array_equal(a, b)


def test_scratch_is_given_back_when_memory_runs_out(L):
    """A search with room for more stored embeddings than any card holds is refused; the scratch of an earlier training is free again
    then.  Without that demand the same search, and another training, give what they gave before."""
    import torch
    say("pq scratch given back to a search")
    cfg = dict(li.TINY, layers=1)
    n = 65536
    ctx = L.leann_create(cfg, to_dev(li.encoder_weights(cfg, 1)))
    try:
        emb = to_dev(unit_rows(n, cfg["hidden"], 2))
        t, l = to_dev(np.ones((n, 8), np.int32)), to_dev(np.full(n, 8, np.int32))
        row_ptr, col_idx = to_dev(np.arange(n + 1, dtype=np.int64)), to_dev(((np.arange(n) + 1) % n).astype(np.int32))

        def train():
            pq = L.leann_build_pq(ctx, emb, 16, 1, 5)
            return pq, L.leann_pq_export(ctx, pq)

        def search(pq):
            return L.leann_search(ctx, emb[:3].contiguous(), (row_ptr, col_idx, 0), pq, t, l, 10, 3, 0.5, 4)[:2]

        pq, table = train()
        found = search(pq)
        scratch = n * (4 * cfg["hidden"] + 5 * 16 + 8)
        free = torch.cuda.mem_get_info()[0]
        L.leann_set_call_memo(ctx, 1 << 30)  # times 4 * hidden bytes
        with pytest.raises(L.LeannError) as e:
            search(pq)
        assert e.value.status == -2
        assert torch.cuda.mem_get_info()[0] >= free + scratch - (8 << 20)  # the memo's index of 4 bytes per node has been allocated
        L.leann_set_call_memo(ctx, 0)
        for a, b in zip(found, search(pq)):
            assert torch.equal(a, b)
        again, table1 = train()
        for a, b in zip(table, table1):
            np.testing.assert_array_equal(a, b)
        L.leann_pq_free(again)
        L.leann_pq_free(pq)
    finally:
        L.leann_destroy(ctx)


def codes_of_first_centroids(L, ctx, x, m_sub):
    """(codebook, codes) after no training round: the centroids are 256 of the rows."""
    pq = L.leann_build_pq(ctx, to_dev(x), m_sub, 0, 7)
    got = L.leann_pq_export(ctx, pq)
    L.leann_pq_free(pq)
    return got


@pytest.mark.parametrize("dsub,longest", [(3, 1.5e19), (3, 1.7e19), (16, 1.7e19), (24, 2.2e19)])
def test_pq_codes_where_products_overflow(L, ctx, dsub, longest):
    """Rows so long that |c|^2 and |x|^2 are finite in fp32 and |c|^2 - 2 x.c is not, next to shorter ones; in the last
    case the squares of some overflow too."""
    say(f"pq codes of long rows, dsub {dsub} up to {longest}")
    rng = np.random.default_rng(dsub)
    x = rng.standard_normal((1500, 2, dsub))
    norm = np.exp(rng.uniform(np.log(3e18), np.log(longest), (1500, 2, 1)))
    x = (x / np.linalg.norm(x, axis=2, keepdims=True) * norm).astype(np.float32).reshape(1500, 2 * dsub)
    cb, codes = codes_of_first_centroids(L, ctx, x, 2)
    np.testing.assert_array_equal(codes, nearest_by_fp32_sums(x, cb))


@pytest.mark.parametrize("dsub,offset", [(1, 0.0), (5, 0.0), (8, 3.0), (24, 0.0), (32, 0.0), (32, 100.0)])
def test_pq_codes_of_near_ties(L, ctx, dsub, offset):
    """Clusters whose rows (and so some of their centroids) lie 1e-5 to 0.3 apart: gaps between the two nearest centroids
    on both sides of what the matrix cores can tell apart, and far below it.  Bit for bit the codes of the fp32 sums."""
    say(f"pq codes of near ties, dsub {dsub} offset {offset}")
    rng = np.random.default_rng(dsub)
    cent = rng.standard_normal((100, 2 * dsub))
    spread = np.exp(rng.uniform(np.log(1e-5), np.log(0.3), (100, 1)))
    own = rng.integers(0, 100, 3000)
    x = (offset + cent[own] + spread[own] * rng.standard_normal((3000, 2 * dsub))).astype(np.float32)
    cb, codes = codes_of_first_centroids(L, ctx, x, 2)
    np.testing.assert_array_equal(codes, nearest_by_fp32_sums(x, cb))


@pytest.mark.parametrize("n,dsub,m_sub", [(5000, 2, 100), (1500, 3, 40), (4097, 4, 33), (700, 1, 200), (9000, 1, 7), (65, 2, 300)])
def test_pq_codes_of_many_subspaces(L, ctx, n, dsub, m_sub):
    """Few and many runs of rows, numbers of them that are no multiple of the XCDs, and sub-vectors of one element: every code is
    that of the fp32 sums."""
    say(f"pq codes n={n} dsub={dsub} m_sub={m_sub}")
    x = np.random.default_rng(n).standard_normal((n, dsub * m_sub)).astype(np.float32)
    cb, codes = codes_of_first_centroids(L, ctx, x, m_sub)
    np.testing.assert_array_equal(codes, nearest_by_fp32_sums(x, cb))


def test_build_pq_rejects_bad_shapes(L, ctx):
    say("build_pq bad shapes")
    x = to_dev(np.zeros((10, 130), np.float32))
    with pytest.raises(L.LeannError):
        L.leann_build_pq(ctx, x, 4, 1, 0)      # 130 % 4 != 0
    with pytest.raises(L.LeannError):
        L.leann_build_pq(ctx, x, 2, 1, 0)      # sub-vector longer than 32
