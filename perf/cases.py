"""Cases whose speed is tracked: what a serving engine has this framework do.

Each case is one public call, or the few that belong together, at sizes from
this repository's workloads and tests or generic ones.  ``match`` identifies
the reusable prefix of arriving prompts (hash, then lookup); ``retrieve``
moves staged chunks into the paged KV pool; ``store`` moves finished chunks
out of it; ``staged`` retrieves chunks that still lie in host memory; ``pass``
is a whole pass of ``StagingPath`` over a small batch.

A case's structure (prompt lengths, which request reuses which prefix) is
fixed by the case; token ids, block tables and KV contents come from the seed.
"""
import math

import numpy as np
import torch

import paper_2609_35065_amd as kv
import workloads as W
from paper_2609_35065_amd.pipeline import StagingPath

VOCAB = 32000
CHUNK = 256            # tokens of a staged chunk
POOL_FACTOR = 1.25     # paged blocks per live block
GAMMA = 0x9E3779B97F4A7C15


def _kv(name, op, requests, tokens, **more):
    c = {"name": name, "op": op, "requests": requests, "tokens": tokens, "lengths": "equal", "prefix": 1.0,
         "prefixes": requests, "layers": 32, "heads": 8, "dim": 128, "elem": 2, "block": 16, "layout": "kv_first",
         "pad": 0}
    c.update(more)
    return c


def listed():
    return [
        # one short prompt arrives: the smallest call, all latency
        {"name": "match-1x1000", "op": "match", "requests": 1, "tokens": 1000, "lengths": "equal", "prefix": 0.5,
         "prefixes": 1, "staged_chunks": 4096},
        # a full admission queue of equal prompts: the batch of the capacity sweep
        {"name": "match-1024x1024", "op": "match", "requests": 1024, "tokens": 1024, "lengths": "equal",
         "prefix": 0.9, "prefixes": 16, "staged_chunks": 65536},
        # one long document: the longest chain of block hashes
        {"name": "match-1x65536", "op": "match", "requests": 1, "tokens": 65536, "lengths": "equal", "prefix": 1.0,
         "prefixes": 1, "staged_chunks": 4096},
        # one arriving request reuses three chunks (32-layer bf16 KV): the smallest retrieve in ordinary use
        _kv("retrieve-1x1024", "retrieve", 1, 1024, prefix=0.75),
        # the benchmark batch: 8 shared prefixes, 64 requests
        _kv("retrieve-64x4096", "retrieve", 64, 4096, prefix=0.5, prefixes=8),
        # ragged prompts over popular prefixes, one KV head per GPU (4 KiB segments), as a tensor-parallel shard
        _kv("retrieve-lognormal-1head", "retrieve", 256, 2048, lengths="lognormal", prefix=0.75, prefixes=32,
            heads=1),
        # head size 80 (20 KiB segments, not a power of two), a prefix of its own for each request
        _kv("retrieve-32x2048-d80", "retrieve", 32, 2048, prefix=0.75, dim=80),
        # one decoding request has filled one more chunk: the smallest store
        _kv("store-1x256", "store", 1, 256),
        # the 512 chunks the benchmark batch stores: the largest call
        _kv("store-64x2048", "store", 64, 2048),
        # 8-bit KV, both planes of a block together, ragged prompts
        _kv("store-16-lognormal-fp8", "store", 16, 2048, lengths="lognormal", heads=4, elem=1, layout="block_first"),
        # one request whose prefix lies in host memory: copies over the link, scatter behind them
        _kv("staged-1x2048", "staged", 1, 2048),
        # a few requests arrive: hash, lookup, claims, jobs, retrieve, store and index update in one pass
        _kv("pass-8x1024", "pass", 8, 1024, prefix=0.5, prefixes=2),
    ]


def _log_between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["match", "match", "match", "retrieve", "retrieve", "retrieve", "retrieve", "store", "store",
                     "store", "staged", "pass"])
    if op == "match":
        tokens = _log_between(rng, 256, 65536)
        requests = _log_between(rng, 1, max(1, min(1024, (1 << 20) // tokens)))
        return {"op": op, "requests": requests, "tokens": tokens, "lengths": rng.choice(["equal", "lognormal"]),
                "prefix": round(rng.uniform(0.25, 1.0), 2), "prefixes": rng.randint(1, requests),
                "staged_chunks": _log_between(rng, 4096, 65536)}
    shape = {"layers": rng.choice([24, 32, 40, 48]), "heads": rng.choice([1, 1, 2, 4, 8, 8]),
             "dim": rng.choice([64, 80, 96, 128, 128, 128]), "elem": rng.choice([1, 2, 2, 2, 2, 4]),
             "block": rng.choice([16, 16, 16, 32]), "layout": rng.choice(["kv_first", "block_first"]),
             "pad": rng.choice([0, 0, 0, 16, 4096])}
    slot = 2 * shape["layers"] * CHUNK * shape["heads"] * shape["dim"] * shape["elem"]
    cap = {"retrieve": 4 << 30, "store": 4 << 30, "staged": 512 << 20, "pass": 1 << 30}[op]
    chunks = _log_between(rng, 1, max(1, min(2048, cap // slot)))
    requests = _log_between(rng, 1, chunks)
    if op in ("staged", "pass"):
        requests = min(requests, 16)
    tokens = max(CHUNK, chunks * CHUNK // requests + rng.randint(0, 255))
    c = {"op": op, "requests": requests, "tokens": tokens, "lengths": rng.choice(["equal", "lognormal"]),
         "prefix": round(rng.uniform(0.5, 1.0), 2), "prefixes": rng.randint(1, requests)}
    c.update(shape)
    return c


# ---------------------------------------------------------------------------
# structure of a case: a function of the case alone
# ---------------------------------------------------------------------------

def _structure(c):
    """(lengths, prefix id, prefix tokens) per request.  Lognormal lengths have
    sigma 0.8 around the case's mean, clipped to 256 .. 4 times the mean; they
    share prefixes by Zipf(1.1), equal ones evenly."""
    R, n = c["requests"], c["tokens"]
    rng = np.random.default_rng([R, n, c["prefixes"]])
    if c["lengths"] == "equal":
        lengths = np.full(R, n, np.int64)
        pid = np.arange(R) % c["prefixes"]
    else:
        mu = math.log(n) - 0.8 ** 2 / 2
        lengths = np.clip(rng.lognormal(mu, 0.8, R), CHUNK, 4 * n).astype(np.int64)
        if c["op"] in ("staged", "pass"):
            lengths = np.minimum(lengths, 2 * n)
        p = 1.0 / np.arange(1, c["prefixes"] + 1) ** 1.1
        pid = rng.choice(c["prefixes"], R, p=p / p.sum())
    pre = (c["prefix"] * lengths / CHUNK).astype(np.int64) * CHUNK
    if c["op"] in ("retrieve", "staged"):
        pre = np.maximum(pre, CHUNK)   # every request reuses something
    return lengths, pid.astype(np.int32), pre


def _prefix_chunks(pid, pre, prefixes):
    """Chunks of each prefix stream (its longest use) and the first slot of each."""
    n = np.zeros(prefixes, np.int64)
    np.maximum.at(n, pid, pre // CHUNK)
    return n, np.concatenate([[0], np.cumsum(n)])


def _slot_bytes(c):
    return 2 * c["layers"] * CHUNK * c["heads"] * c["dim"] * c["elem"]


def work(case):
    lengths, pid, pre = _structure(case)
    nch, _ = _prefix_chunks(pid, pre, case["prefixes"])
    unique, hits, total = int(nch.sum()), int((pre // CHUNK).sum()), int((lengths // CHUNK).sum())
    meta = 4 * int(lengths.sum()) + 8 * int((lengths // 16).sum()) + 20 * total + 24 * case["requests"]
    if case["op"] == "match":
        return {"bytes": meta, "flops": 0}
    slot = _slot_bytes(case)
    moved = {"retrieve": unique + hits, "store": 2 * total, "staged": 2 * unique + hits,
             "pass": unique + hits + 2 * (total - hits)}[case["op"]]
    return {"bytes": moved * slot, "flops": 0}


def tolerance(case):
    return "exact"   # hashes are whole numbers and KV is moved as it is


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _tokens(c, seed):
    """Token ids of the batch, requests back to back: each request's prefix
    tokens from its prefix stream, the rest its own."""
    lengths, pid, pre = _structure(c)
    rng = np.random.default_rng([seed, 1])
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    toks = rng.integers(0, VOCAB, int(off[-1]), dtype=np.int32)
    nch, _ = _prefix_chunks(pid, pre, c["prefixes"])
    streams = [rng.integers(0, VOCAB, int(k) * CHUNK, dtype=np.int32) for k in nch]
    for r in range(c["requests"]):
        toks[off[r]:off[r] + pre[r]] = streams[pid[r]][:pre[r]]
    return toks, off, streams, pid, pre, nch


def _offsets(tok_off):
    nb = np.diff(tok_off) // 16
    nc = nb // (CHUNK // 16)
    return (np.concatenate([[0], np.cumsum(nb)]).astype(np.int64),
            np.concatenate([[0], np.cumsum(nc)]).astype(np.int64))


def _filler_keys(n, seed):
    """Keys of chunks that other requests left in the index."""
    return np.random.default_rng([seed, 2]).integers(1, 2 ** 63, n, dtype=np.int64).view(np.uint64)


def _fill(t, elem, gen):
    """KV values (normal) of the case's element type in a byte buffer."""
    if elem == 2:
        t.view(torch.bfloat16).normal_(generator=gen)
    elif elem == 4:
        t.view(torch.float32).normal_(generator=gen)
    else:
        for s in range(0, t.numel(), 1 << 30):
            v = t[s:s + (1 << 30)]
            v.view(torch.float8_e4m3fn).copy_(torch.empty(v.numel(), dtype=torch.bfloat16, device=t.device)
                                              .normal_(generator=gen))
    return t


class _State:
    pass


def _pool(c, seed, lengths):
    """Paged pool (one tensor per layer, views of one buffer), its layout and
    the requests' block tables: blocks in random order, as a used pool hands
    them out."""
    B = c["block"]
    nblk = lengths // B + (lengths % B > 0)
    live = int(nblk.sum())
    NB = max(live + 1, int(live * POOL_FACTOR))
    perm = np.random.default_rng([seed, 3]).permutation(NB).astype(np.int32)
    bt = np.full((lengths.size, int(nblk.max())), -1, np.int32)
    at = 0
    for r, n in enumerate(nblk):
        bt[r, :n] = perm[at:at + n]
        at += n
    return NB, bt


def _copy_state(case, seed, jobs_of, host=False):
    c, s = case, _State()
    lengths, pid, pre = _structure(c)
    nch, first = _prefix_chunks(pid, pre, c["prefixes"])
    NB, bt = _pool(c, seed, lengths)
    jobs, slots = jobs_of(lengths, pid, pre, first)
    seg = c["block"] * c["heads"] * c["dim"] * c["elem"]
    row = seg + c["pad"]
    strides = (NB * row, row) if c["layout"] == "kv_first" else (row, 2 * row)
    s.layout = kv.make_layout(c["layers"], c["heads"], c["dim"], c["elem"], c["block"], CHUNK, NB, slots, *strides)
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    s.pool = _fill(torch.empty(c["layers"] * 2 * NB * row, dtype=torch.uint8, device="cuda"), c["elem"], gen)
    s.layers = list(s.pool.view(c["layers"], -1))
    s.staging = _fill(torch.empty(slots * _slot_bytes(c), dtype=torch.uint8, device="cuda"), c["elem"], gen)
    s.host = None
    if host:
        s.host = torch.empty(s.staging.numel(), dtype=torch.uint8, pin_memory=True)
        s.host.copy_(s.staging)
        s.staging.zero_()
    s.bt, s.bt_stride, s.num_reqs = torch.from_numpy(bt).cuda(), bt.shape[1], bt.shape[0]
    s.h_jobs = np.array(jobs, np.int32).reshape(-1, 4)
    return s


def _retrieve_jobs(lengths, pid, pre, first):
    return ([(first[pid[r]] + j, r, j, 0) for r in range(lengths.size) for j in range(pre[r] // CHUNK)],
            int(first[-1]))


def _store_jobs(lengths, pid, pre, first):
    jobs = [(r, j) for r in range(lengths.size) for j in range(lengths[r] // CHUNK)]
    return [(i, r, j, 0) for i, (r, j) in enumerate(jobs)], len(jobs)


def prepare(case, seed):
    op = case["op"]
    if op == "match":
        s = _State()
        toks, off, streams, _, _, nch = _tokens(case, seed)
        blk_off, chunk_off = _offsets(off)
        s.num_reqs, s.bpc = case["requests"], CHUNK // 16
        s.tokens, s.tok_off = torch.from_numpy(toks).cuda(), torch.from_numpy(off).cuda()
        s.blk_off, s.chunk_off = torch.from_numpy(blk_off).cuda(), torch.from_numpy(chunk_off).cuda()
        s.block_hash = torch.zeros(max(int(blk_off[-1]), 1), dtype=torch.int64, device="cuda")
        s.chunk_slot = torch.zeros(max(int(chunk_off[-1]), 1), dtype=torch.int32, device="cuda")
        s.hit = torch.zeros(s.num_reqs, dtype=torch.int32, device="cuda")
        # the index: the prefixes' chunks and those of earlier requests
        soff = np.concatenate([[0], np.cumsum(nch * CHUNK)]).astype(np.int64)
        sblk, schunk = _offsets(soff)
        h = torch.zeros(max(int(sblk[-1]), 1), dtype=torch.int64, device="cuda")
        flat = np.concatenate(streams) if int(soff[-1]) else np.zeros(1, np.int32)
        kv.kv_hash_prefix(torch.from_numpy(flat).cuda(), torch.from_numpy(soff).cuda(), nch.size, 0,
                          torch.from_numpy(sblk).cuda(), h)
        keys = kv.kv_chunk_keys(h.cpu().numpy().view(np.uint64), sblk, s.bpc, schunk)
        filler = _filler_keys(max(0, case["staged_chunks"] - keys.size), seed)
        keys = np.concatenate([keys, filler])
        s.index = kv.kv_index_create(keys.size)
        kv.kv_index_insert(s.index, keys, np.arange(keys.size, dtype=np.int32))
        return s
    if op == "pass":
        return _prepare_pass(case, seed)
    s = _copy_state(case, seed, _store_jobs if op == "store" else _retrieve_jobs, host=op == "staged")
    s.store = op == "store"
    if not s.store:
        s.h_jobs = kv.kv_group_jobs_by_slot(s.h_jobs)
    s.d_jobs = torch.from_numpy(s.h_jobs).cuda()
    if op == "staged":
        s.pipeline = kv.KvPipeline(64)
        s.copy_stream = torch.cuda.Stream()
    return s


def _prepare_pass(c, seed):
    toks, off, streams, pid, pre, nch = _tokens(c, seed)
    lengths = np.diff(off)
    NB, bt = _pool(c, seed, lengths)
    staged = [(p, j) for p in range(c["prefixes"]) for j in range(int(nch[p]))]
    misses = int((lengths // CHUNK - pre // CHUNK).sum())
    w = W.Workload(name="pass", shape=W.KVShape(c["layers"], c["heads"], c["dim"], c["elem"], c["block"], CHUNK),
                   seed=seed, tokens=toks, tok_off=off, prefix_id=pid, prefix_tokens=pre, prefix_streams=streams,
                   prestage_chunks=staged, num_slots=len(staged) + max(misses, 1), num_blocks=NB, block_tables=bt,
                   paged_layout=c["layout"], block_pad=c["pad"])
    s = _State()
    s.path = StagingPath(w)
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    for t in [s.path.staging] + s.path.layers:
        _fill(t, c["elem"], gen)
    s.path.prestage()
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def _words(t):
    """A byte buffer's contents as whole numbers, without a copy."""
    return t.view(torch.int64) if t.numel() % 8 == 0 else t


def run(state):
    s = state
    if hasattr(s, "path"):
        s.path.run_pass(evict_stored=True)
        p = s.path
        return {"block_hash": p.block_hash, "chunk_slot": p.chunk_slot, "hit": p.hit, "staging": _words(p.staging),
                "layers": [_words(t) for t in p.layers]}
    if hasattr(s, "index"):
        kv.kv_hash_prefix(s.tokens, s.tok_off, s.num_reqs, 0, s.blk_off, s.block_hash)
        kv.kv_lookup(s.index, s.block_hash, s.blk_off, s.num_reqs, s.bpc, s.chunk_off, s.chunk_slot, s.hit)
        return {"block_hash": s.block_hash, "chunk_slot": s.chunk_slot, "hit": s.hit}
    n = len(s.h_jobs)
    if s.host is not None:
        # the copies may start once earlier work no longer reads the slots they fill
        s.copy_stream.wait_stream(torch.cuda.current_stream())
        kv.kv_retrieve_pipelined(s.pipeline, s.layout, s.host, s.staging, s.layers, s.bt, s.bt_stride, s.num_reqs,
                                 s.h_jobs, s.d_jobs, 4, s.copy_stream)
        return {"pool": _words(s.pool), "staging": _words(s.staging)}
    if s.store:
        kv.kv_store_gather(s.layout, s.staging, s.layers, s.bt, s.bt_stride, s.num_reqs, s.d_jobs, n)
        return {"staging": _words(s.staging)}
    kind = kv.kv_retrieve_plan(s.layout, s.h_jobs)
    kv.kv_retrieve_scatter_as(kind, s.layout, s.staging, s.layers, s.bt, s.bt_stride, s.num_reqs, s.d_jobs, n)
    return {"pool": _words(s.pool)}


# ---------------------------------------------------------------------------
# the same in plain numpy, 64-bit whole numbers
# ---------------------------------------------------------------------------

def _mix(z):
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def _hashes(toks, off):
    """Block hashes of a ragged batch: the chain runs over all requests at once."""
    blk_off, _ = _offsets(off)
    nb = np.diff(blk_off)
    out = np.zeros(int(blk_off[-1]), np.uint64)
    h = np.zeros(nb.size, np.uint64)
    pos = (np.arange(1, 17, dtype=np.uint64) << np.uint64(32))
    for b in range(int(nb.max()) if nb.size else 0):
        r = np.nonzero(nb > b)[0]
        at = off[r][:, None] + 16 * b + np.arange(16)
        d = _mix(toks[at].astype(np.uint32).astype(np.uint64) + pos).sum(axis=1, dtype=np.uint64)
        h[r] = _mix(h[r] ^ d ^ np.uint64(GAMMA))
        out[blk_off[r] + b] = h[r]
    return out


def exact(case, seed):
    """Hashes and lookup results; the copies move bytes and compute nothing."""
    if case["op"] != "match":
        return None
    toks, off, streams, _, _, nch = _tokens(case, seed)
    out = _hashes(toks, off)
    soff = np.concatenate([[0], np.cumsum(nch * CHUNK)]).astype(np.int64)
    sh = _hashes(np.concatenate(streams), soff) if int(soff[-1]) else np.zeros(0, np.uint64)
    bpc = CHUNK // 16
    keys = sh[bpc - 1::bpc]   # the streams are whole chunks
    keys = np.concatenate([keys, _filler_keys(max(0, case["staged_chunks"] - keys.size), seed)])
    slots = {int(k): i for i, k in enumerate(keys)}
    blk_off, chunk_off = _offsets(off)
    slot = np.zeros(max(int(chunk_off[-1]), 1), np.int32)
    hit = np.zeros(case["requests"], np.int32)
    for r in range(case["requests"]):
        got = [slots.get(int(out[blk_off[r] + (j + 1) * bpc - 1]), -1) for j in range(chunk_off[r + 1] - chunk_off[r])]
        slot[chunk_off[r]:chunk_off[r + 1]] = got
        hit[r] = got.index(-1) if -1 in got else len(got)
    return {"block_hash": out.view(np.int64), "chunk_slot": slot, "hit": hit}
