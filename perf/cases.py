"""The work a user of this framework has it do, as cases that can be timed and compared.

Every case goes through the public entry points of `paper_2506_08276_amd`:

- `embed`   leann_embed: chunks of token ids to embeddings (the recomputation step, and a query's own embedding);
- `search`  leann_search / leann_search_updates: queries to their k nearest chunks, with recomputed, partly stored or
            fully stored embeddings, with and without pending updates;
- `adc`     leann_adc: approximate scores of candidate nodes from the PQ table;
- `pq`      leann_build_pq + leann_pq_export: training the PQ table and taking it home;
- `graph`   leann_build_graph: the proximity graph by insertion.

A program keeps one encoder per shape for its life: the contexts below are made once per process, with fixed weights;
chunks, queries, graphs, tables and updates come from the seed.  Index structures that a search reads are made here with
torch and `leann_inputs`, so that two versions of the framework search the very same index.
"""
import math

import numpy as np
import torch

import leann_inputs as li
import paper_2506_08276_amd as L

DEV = "cuda:0"
SHAPES = {"base": li.BASE, "small": li.SMALL}
_encoders = {}


def listed():
    """The cases."""
    return [
        # a query's text on its way into a search: one chunk, nothing but latency
        dict(name="embed one query", kind="embed", shape="base", n=1, seq=128),
        # what one query sends through the encoder per round (a dozen ragged chunks)
        dict(name="embed one flush", kind="embed", shape="base", n=13, seq=128),
        # the lighter encoder on a batch of documents; widths that are not multiples of 256
        dict(name="embed small encoder", kind="embed", shape="small", n=300, seq=256),
        # indexing, and the rounds of a large query batch: the encoder's throughput case
        dict(name="embed large batch", kind="embed", shape="base", n=2048, seq=256),
        # interactive use: one query at a time, everything recomputed
        dict(name="search one query", kind="search", shape="base", n=12288, seq=128, nq=1, ef=84, k=3, alpha=0.05,
             batch=64, stored=0.0, updates=False),
        # batch use: many queries in flight, everything recomputed
        dict(name="search batch", kind="search", shape="base", n=12288, seq=128, nq=200, ef=128, k=3, alpha=0.05,
             batch=64, stored=0.0, updates=False),
        # hub embeddings kept, soft deletes and an add buffer pending
        dict(name="search hubs stored, updates", kind="search", shape="base", n=12288, seq=128, nq=48, ef=96, k=3,
             alpha=0.1, batch=32, stored=0.1, updates=True),
        # every embedding kept: queues, graph, codes and scoring without the encoder
        dict(name="search all stored", kind="search", shape="base", n=12288, seq=128, nq=500, ef=200, k=3, alpha=0.05,
             batch=64, stored=1.0, updates=False),
        # the neighbours of one hop
        dict(name="adc one hop", kind="adc", n=500_000, d=768, m_sub=32, nq=1, nc=64),
        # re-ranking long candidate lists of many queries over a table larger than the caches
        dict(name="adc many candidates", kind="adc", n=16_000_000, d=768, m_sub=32, nq=1024, nc=16384),
        # offline: the PQ table of a collection
        dict(name="pq table", kind="pq", n=100_000, d=768, m_sub=32, iters=6),
        # offline: the graph of a collection, hubs keeping 64 neighbours and the others 16
        dict(name="graph construction", kind="graph", n=8192, d=768, efC=128, M=64, m=16, batch=1024, ramp=8),
    ]


def _log(rng, lo, hi):
    """A whole number in [lo, hi], spread over the logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the ranges that the listed ones stand for."""
    kind = rng.choice(["embed", "embed", "search", "search", "adc", "pq", "graph"])
    if kind == "embed":
        return dict(kind=kind, shape=rng.choice(["base", "base", "small"]), n=_log(rng, 1, 2048), seq=rng.randint(16, 256))
    if kind == "search":
        stored = rng.choice([0.0, 0.0, 0.1, 1.0])
        return dict(kind=kind, shape=rng.choice(["base", "small"]), n=_log(rng, 3000, 12288), seq=rng.randint(48, 128),
                    nq=_log(rng, 1, 500 if stored == 1.0 else 128), ef=_log(rng, 64, 200 if stored == 1.0 else 128), k=rng.choice([1, 3]),
                    alpha=rng.choice([0.05, 0.1, 0.2]), batch=rng.choice([16, 32, 64, 128]), stored=stored,
                    updates=rng.random() < 0.3)
    if kind == "adc":
        m_sub = rng.choice([16, 32, 32, 48])
        return dict(kind=kind, n=_log(rng, 5000, 16_000_000), d=m_sub * rng.choice([8, 16, 24]), m_sub=m_sub,
                    nq=_log(rng, 1, 1024), nc=_log(rng, 1, 16384))
    if kind == "pq":
        d, m_sub = rng.choice([(768, 32), (384, 32), (128, 16), (768, 48), (384, 16)])
        return dict(kind=kind, n=_log(rng, 1000, 100_000), d=d, m_sub=m_sub, iters=rng.randint(2, 6))
    M = rng.choice([16, 32, 64])
    return dict(kind="graph", n=_log(rng, 500, 8192), d=rng.choice([128, 384, 768]), efC=rng.choice([48, 96, 128]), M=M,
                m=rng.choice([M, max(4, M // 4)]), batch=rng.choice([64, 256, 1024]), ramp=8)


# ------------------------------------------------------------------ what a program has in hand
def _weights(cfg, seed):
    """Packed random-init weights as a {name: bf16 tensor} dict in packed order: N(0, 0.02) matrices, zero biases."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    out = {}
    for name, shape, kind in li.weight_layout(cfg):
        if kind == "matrix":
            out[name] = (torch.randn(shape, generator=g, device=DEV) * 0.02).bfloat16()
        else:
            out[name] = torch.full(shape, 1.0 if kind == "gamma" else 0.0, device=DEV).bfloat16()
    return out


def encoder(shape):
    """(context, weights) of an encoder shape; made once per process."""
    if shape not in _encoders:
        w = _weights(SHAPES[shape], li.config_seed(2) + len(shape))
        packed = torch.cat([t.reshape(-1) for t in w.values()])
        _encoders[shape] = (L.leann_create(SHAPES[shape], packed), w)
    return _encoders[shape]


class _Pq:
    """A PQ handle that is freed with the state that holds it."""

    def __init__(self, handle):
        self.handle = handle

    def __del__(self):
        if L is not None:
            L.leann_pq_free(self.handle)


def embed_with_torch(cfg, w, tokens, lengths, mat=torch.bfloat16, acc=torch.float32, block=1024):
    """The encoder in plain torch on padded blocks; `mat`: type of the matrix products, `acc`: of everything else."""
    d, H, S = cfg["hidden"], cfg["heads"], tokens.shape[1]
    cast = {k: v.to(mat if k.split(".")[-1] in ("wqkv", "wo", "w1", "w2") else acc) for k, v in w.items()}
    out = []
    for s in range(0, tokens.shape[0], block):
        tok, n_tok = tokens[s:s + block].long(), lengths[s:s + block].long()
        b = tok.shape[0]
        valid = torch.arange(S, device=DEV)[None, :] < n_tok[:, None]

        def norm(x, name):
            return torch.nn.functional.layer_norm(x, (d,), cast[name + "_g"], cast[name + "_b"], cfg["ln_eps"])

        def linear(x, name):
            return (x.to(mat) @ cast[name].t()).to(acc)

        x = norm(cast["tok_emb"][tok * valid] + cast["pos_emb"][:S] + cast["seg_emb"], "emb_ln").reshape(b * S, d)
        mask = torch.zeros((b, 1, 1, S), dtype=acc, device=DEV).masked_fill(~valid[:, None, None, :], -float("inf"))
        for layer in range(cfg["layers"]):
            p = f"l{layer}."
            qkv = (linear(x, p + "wqkv") + cast[p + "bqkv"]).reshape(b, S, 3, H, d // H).permute(2, 0, 3, 1, 4).contiguous()
            att = torch.softmax(qkv[0] @ qkv[1].transpose(-1, -2).contiguous() / math.sqrt(d // H) + mask, -1) @ qkv[2]
            att = att.transpose(1, 2).reshape(b * S, d)
            x = norm(x + linear(att, p + "wo") + cast[p + "bo"], p + "ln1")
            hid = torch.nn.functional.gelu(linear(x, p + "w1") + cast[p + "b1"])
            x = norm(x + linear(hid, p + "w2") + cast[p + "b2"], p + "ln2")
        e = (x.reshape(b, S, d) * valid[:, :, None]).sum(1) / n_tok[:, None]
        out.append(e / e.norm(dim=1, keepdim=True).clamp_min(1e-12))
    return torch.cat(out)


def _clustered(g, n, d):
    """Unit vectors around n / 25 centres (what a proximity graph and a PQ table are built for)."""
    cent = torch.randn((max(2, n // 25), d), generator=g, device=DEV)
    x = cent[torch.randint(0, cent.shape[0], (n,), generator=g, device=DEV)] + 0.7 * torch.randn((n, d), generator=g, device=DEV)
    return (x / x.norm(dim=1, keepdim=True)).contiguous()


def _codebook(emb, m_sub, g, iters=5):
    """Lloyd's iterations per subspace, all subspaces at once; (codebook fp32 [m][256][dsub], codes u8 [n][m])."""
    n, d = emb.shape
    x = emb.reshape(n, m_sub, d // m_sub).transpose(0, 1).contiguous()
    cb = x[:, torch.randperm(n, generator=g, device=DEV)[:256]].contiguous()
    for it in range(iters + 1):
        dist = (cb * cb).sum(2)[:, None, :] - 2 * (x @ cb.transpose(1, 2).contiguous())
        code = dist.argmin(2)
        if it == iters:
            return cb.cpu().numpy(), code.t().to(torch.uint8).contiguous().cpu().numpy()
        own = torch.nn.functional.one_hot(code, 256).float().transpose(1, 2).contiguous()
        count = own.sum(2, keepdim=True)
        cb = torch.where(count > 0, (own @ x) / count.clamp_min(1), cb)


def _prepare_embed(case, g, seed):
    cfg = SHAPES[case["shape"]]
    n, seq = case["n"], case["seq"]
    ctx, _ = encoder(case["shape"])
    tokens = torch.randint(1, cfg["vocab"], (n, seq), generator=g, device=DEV, dtype=torch.int32)
    lengths = torch.randint((seq + 3) // 4, seq + 1, (n,), generator=g, device=DEV, dtype=torch.int32)
    # lengths keep their mean over the batch, so that a batch of few chunks is as much work with one seed as with another
    lengths[n // 2:n // 2 * 2] = seq + (seq + 3) // 4 - lengths[:n // 2]
    if n % 2:
        lengths[-1] = (5 * seq + 7) // 8
    return dict(ctx=ctx, tokens=tokens, lengths=lengths, hidden=cfg["hidden"])


def _prepare_search(case, g, seed):
    cfg = SHAPES[case["shape"]]
    n, seq, nq, k = case["n"], case["seq"], case["nq"], case["k"]
    ctx, w = encoder(case["shape"])
    space = li.make_latent_space(cfg["vocab"], seed + 1)
    corpus = li.latent_corpus(space, n, seq, seq // 4, seq, seed + 2)
    tokens = torch.from_numpy(corpus["tokens"]).to(DEV)
    lengths = torch.from_numpy(corpus["lengths"]).to(DEV)
    emb = embed_with_torch(cfg, w, tokens, lengths)
    nbr, sim = li.knn_graph(emb, 32)
    entry, _ = li.max_in_degree_node(nbr)
    lists, _, _ = li.navigable_fixture(emb, nbr, sim, hub_frac=0.02, hub_deg=64, low_deg=16)
    row_ptr, col_idx = li.to_csr(lists)
    graph = (torch.from_numpy(row_ptr.view(np.int64)).to(DEV), torch.from_numpy(col_idx.view(np.int32)).to(DEV), entry)
    pq = _Pq(L.leann_pq_import(ctx, *_codebook(emb, 32, g)))
    st = dict(ctx=ctx, tokens=tokens, lengths=lengths, graph=graph, pq=pq, cache=None, deleted=None, buffer=None)
    alive = torch.ones(n, dtype=torch.bool, device=DEV)
    exact = emb
    if case["updates"]:
        alive = torch.rand(n, generator=g, device=DEV) >= 0.05
        bits = np.packbits((~alive).cpu().numpy(), bitorder="little")
        bits = np.concatenate([bits, np.zeros(-len(bits) % 4, np.uint8)]).view(np.int32)
        st["deleted"] = torch.from_numpy(bits.copy()).to(DEV)
        nb = n // 50
        extra = emb[torch.randint(0, n, (nb,), generator=g, device=DEV)] + 0.01 * torch.randn((nb, emb.shape[1]), generator=g, device=DEV)
        extra = (extra / extra.norm(dim=1, keepdim=True)).contiguous()
        st["buffer"] = (torch.arange(n, n + nb, dtype=torch.int32, device=DEV), extra)
        exact, alive = torch.cat([emb, extra]), torch.cat([alive, torch.ones(nb, dtype=torch.bool, device=DEV)])
    if case["stored"] > 0:
        rows, slot_of = li.hub_slots(row_ptr, col_idx, case["stored"])
        st["cache"] = (torch.from_numpy(slot_of).to(DEV), emb[torch.from_numpy(rows).to(DEV)].contiguous())
    # Queries are fresh variants of the corpus' families.  They are taken from the eighth of them whose k + 1 nearest
    # chunks are furthest apart: where two chunks are equally near, either is a right answer.
    qtok, qlen, _ = li.latent_queries(space, corpus, 8 * (nq + 8), seed + 3)
    q = embed_with_torch(cfg, w, torch.from_numpy(qtok).to(DEV), torch.from_numpy(qlen).to(DEV))
    score = (q @ exact.t()).masked_fill(~alive, -float("inf"))
    top = torch.topk(score, k + 1, dim=1).values
    clear = (top[:, :-1] - top[:, 1:]).amin(1)
    st["queries"] = q[torch.sort(torch.topk(clear, nq + 8).indices).values[:nq]].contiguous()
    return st


def _prepare_adc(case, g, seed):
    ctx, _ = encoder("base")
    n, d, m = case["n"], case["d"], case["m_sub"]
    codes = torch.randint(0, 256, (n, m), generator=g, device=DEV, dtype=torch.uint8)
    cb = (torch.randn((m, 256, d // m), generator=g, device=DEV) * 0.05).cpu().numpy()
    q = torch.randn((case["nq"], d), generator=g, device=DEV)
    cand = torch.randint(0, n, (case["nq"], case["nc"]), generator=g, device=DEV, dtype=torch.int32)
    return dict(ctx=ctx, codes=codes, pq=_Pq(L.leann_pq_wrap(ctx, cb, codes)), cand=cand,
                queries=(q / q.norm(dim=1, keepdim=True)).contiguous())


def _prepare_pq(case, g, seed):
    ctx, _ = encoder("base")
    return dict(ctx=ctx, emb=_clustered(g, case["n"], case["d"]), m_sub=case["m_sub"], iters=case["iters"], seed=seed)


def _prepare_graph(case, g, seed):
    ctx, _ = encoder("base")
    n = case["n"]
    hub = None
    if case["m"] < case["M"]:
        hub = (torch.rand(n, generator=g, device=DEV) < 0.02).to(torch.uint8)
    return dict(ctx=ctx, emb=_clustered(g, n, case["d"]), hub=hub, efC=case["efC"], M=case["M"], m=case["m"],
                batch=case["batch"], ramp=case["ramp"])


_PREPARE = {"embed": _prepare_embed, "search": _prepare_search, "adc": _prepare_adc, "pq": _prepare_pq,
            "graph": _prepare_graph}


def prepare(case, seed):
    """What a user's program has in hand before the call, on the GPU."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    st = _PREPARE[case["kind"]](case, g, seed)
    st["case"] = dict(case)
    return st


def run(st):
    """One pass; its outputs."""
    c, kind = st["case"], st["case"]["kind"]
    if kind == "embed":
        return L.leann_embed(st["ctx"], st["tokens"], st["lengths"], hidden=st["hidden"])
    if kind == "search":
        args = (st["ctx"], st["queries"], st["graph"], st["pq"].handle, st["tokens"], st["lengths"], c["ef"], c["k"],
                c["alpha"], c["batch"])
        if c["updates"]:
            ids, scores, _ = L.leann_search_updates(*args, cache=st["cache"], deleted_bits=st["deleted"], buffer=st["buffer"])
        else:
            ids, scores, _ = L.leann_search(*args, cache=st["cache"])
        return {"ids": ids, "scores": scores}
    if kind == "adc":
        return L.leann_adc(st["ctx"], st["queries"], st["pq"].handle, st["cand"])
    if kind == "pq":
        pq = _Pq(L.leann_build_pq(st["ctx"], st["emb"], st["m_sub"], st["iters"], st["seed"]))
        codebook, codes = L.leann_pq_export(st["ctx"], pq.handle)
        return {"codebook": codebook, "codes": codes}
    row_ptr, col_idx = L.leann_build_graph(st["ctx"], st["emb"], st["efC"], st["M"], st["m"], st["hub"], st["batch"], st["ramp"])
    # the number of edges depends on the vectors: the list is filled up to the room that the caller gives it
    return {"row_ptr": row_ptr, "col_idx": torch.nn.functional.pad(col_idx, (0, c["n"] * c["M"] - col_idx.numel()))}


def _encoder_work(cfg, chunks, mean_len, passes=1):
    d, F, layers = cfg["hidden"], cfg["ffn"], cfg["layers"]
    per_token = layers * (2.0 * (4 * d * d + 2 * d * F) + 4.0 * mean_len * d)
    weights = 2.0 * layers * (4 * d * d + 2 * d * F)
    return dict(flops=chunks * mean_len * per_token, bytes=passes * weights + chunks * (mean_len * (4 + 2 * d) + 4 * d))


def work(case):
    """Bytes and operations of one pass that the path cannot do without."""
    kind = case["kind"]
    if kind == "embed":
        return _encoder_work(SHAPES[case["shape"]], case["n"], 0.625 * case["seq"])
    if kind == "search":
        # Every entry of the full exact queue has had its exact score taken and has been expanded: at least ef exact
        # scores and ef hops of about 16 neighbours per query; chunks that several queries ask for count once.
        cfg, nq, ef, n = SHAPES[case["shape"]], case["nq"], case["ef"], case["n"]
        exact = nq * ef * cfg["hidden"]
        bytes_ = nq * ef * (16 * (4 + 32) + 16) + 4.0 * exact
        flops = 2.0 * exact + nq * ef * 16 * 32
        if case["stored"] < 1.0:
            e = _encoder_work(cfg, min(nq * ef, n) * (1.0 - case["stored"]), 0.625 * case["seq"])
            bytes_, flops = bytes_ + e["bytes"], flops + e["flops"]
        if case["updates"]:
            bytes_ += 4.0 * (n // 50) * cfg["hidden"]
            flops += 2.0 * nq * (n // 50) * cfg["hidden"]
        return dict(bytes=bytes_, flops=flops)
    if kind == "adc":
        per = case["m_sub"] + 8
        return dict(bytes=float(case["nq"] * case["nc"] * per + case["nq"] * case["d"] * 4 + 1024 * case["d"]),
                    flops=float(case["nq"] * (case["nc"] * case["m_sub"] + 768 * case["d"])))
    if kind == "pq":
        n, d, nt = case["n"], case["d"], min(case["n"], 65536)
        return dict(bytes=float(case["iters"] * 4 * nt * d + 4 * n * d + n * case["m_sub"]),
                    flops=768.0 * d * (n + case["iters"] * nt))
    # graph: every inserted node meets at least efC others (a full queue) and each meeting reads their vectors once
    n, d, efC = case["n"], case["d"], min(case["efC"], case["n"] // 2)
    return dict(bytes=4.0 * n * d * efC + 4.0 * n * case["m"], flops=2.0 * n * efC * d)


def tolerance(case):
    """How far another correct implementation at the same precision can be."""
    kind = case["kind"]
    if kind == "embed":
        return {"rel": 1e-2}
    if kind == "search":
        return {"rel": 1e-4, "differ": 0.01}
    if kind == "adc":
        return {"rel": 4e-7}
    if kind == "pq":
        return {"rel": 2e-6, "differ": 1e-4}
    return "exact"
