"""What the framework's speed is measured on: joins, candidate lists, verification, search and
index builds over string collections of the shapes this repository's workloads have (DNA reads
and long DNA, protein-like strings with a threshold per string, text), from a handful of strings
to the largest collection the benchmark runs.

Inputs are drawn on the GPU from the seed alone: clusters of mutated copies of hidden strings
(the near-duplicates a join is run to find) and unrelated strings, as
``paper_1810_08833_amd/datagen.py`` draws them on the host.
"""
import math

import numpy as np
import torch

import paper_1810_08833_amd as mj

#: Letters, Zipf exponent of their frequencies (None: uniform) and q-gram length of each kind.
ALPHABETS = {"dna": (4, None), "protein": (25, 1.1), "text": (37, 1.0)}
MAX_SYMBOLS = 260_000_000  # of a DNA collection: 50,000 strings of 5,000 symbols
MEAN_QUERY = 5500          # indexed strings and queries have lengths U[1000, 10000]


def listed():
    dna = dict(data="dna", copies=10, reps=1)
    return [
        # a few strings, checked against each other inside some larger program: latency
        dict(dna, name="join_dna_60", op="join", n=60, copies=5, mean=1000, spread=0.2, rate_lo=0.02,
             rate_hi=0.10, indel=0.667, q=4, k=60, t_div=1, packed=False),
        # one small set of reads (the small benchmark workload)
        dict(dna, name="join_dna_1k", op="join", n=1000, mean=1000, spread=0.2, rate_lo=0.02,
             rate_hi=0.10, indel=0.667, q=4, k=60, t_div=1, packed=False),
        # an ordinary set of long reads, one byte a symbol, odd counts
        dict(dna, name="join_dna_7k", op="join", n=7001, copies=7, mean=3001, spread=0.5,
             rate_lo=0.01, rate_hi=0.05, indel=0.8, q=5, k=101, t_div=2, packed=False),
        # the long-read benchmark workload, 2-bit packed
        dict(dna, name="join_dna_50k", op="join", n=50_000, mean=5000, spread=0.5, rate_lo=0.01,
             rate_hi=0.06, indel=0.8, q=5, k=150, t_div=2, packed=True),
        # protein-like strings: ragged lengths, a threshold per string, seven repetitions
        dict(name="join_protein_20k", op="join", data="protein", n=20_000, copies=10, q=4, reps=7,
             t_div=1),
        dict(name="join_protein_200k", op="join", data="protein", n=200_000, copies=10, q=4, reps=7,
             t_div=1),
        # the headline workload
        dict(name="join_text_300k", op="join", data="text", n=300_000, copies=10, q=6, k=120, reps=4,
             t_div=2),
        # candidates alone, for a program with a verifier of its own
        dict(name="candidates_text_30k", op="candidates", data="text", n=30_000, copies=10, q=6,
             k=120, reps=4, t_div=2),
        # verification alone, of pairs that another filter proposed
        dict(dna, name="verify_dna_20k", op="verify", n=4000, mean=5000, spread=0.5, rate_lo=0.01,
             rate_hi=0.06, indel=0.8, q=5, k=150, t_div=2, packed=False, pairs=20_011),
        # one query against a resident index: latency
        dict(name="search_1", op="search", data="dna", n=200_000, queries=1, q=5, reps=1, t_div=2),
        # a full batch against the largest index (5.5 G symbols)
        dict(name="search_4096", op="search", data="dna", n=1_000_000, queries=4096, q=5, reps=1,
             t_div=2),
        # a collection indexed, then asked once
        dict(name="index_20k", op="index", data="dna", n=20_000, queries=64, q=5, reps=1, t_div=2),
    ]


def _log_between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_dna(rng, n):
    """A DNA collection of n strings: partitions of 16 symbols or more in small sets, of 33 or
    more in large ones, so that unrelated strings seldom share one."""
    large = n > 2000
    mean = _log_between(rng, 600, min(6000, max(601, MAX_SYMBOLS // n)))
    return dict(data="dna", n=n, copies=rng.randint(3, 12), reps=1, mean=mean,
                spread=round(rng.uniform(0.1, 0.6), 2), rate_lo=0.01, rate_hi=round(rng.uniform(0.04, 0.1), 3),
                indel=round(rng.uniform(0.5, 0.9), 2), q=5 if large else 4,
                k=max(8, int(mean * rng.uniform(0.02, 0.06))), t_div=2 if large else 1,
                packed=rng.random() < 0.5)


def draw(rng):
    op = rng.choice(["join", "join", "join", "candidates", "verify", "search", "search", "index"])
    if op == "search":
        return dict(op=op, data="dna", n=_log_between(rng, 2000, 800_000),
                    queries=_log_between(rng, 1, 4096), q=5, reps=1, t_div=2)
    if op == "index":
        return dict(op=op, data="dna", n=_log_between(rng, 500, 60_000),
                    queries=_log_between(rng, 1, 1000), q=5, reps=1, t_div=2)
    if op == "verify":
        return dict(_draw_dna(rng, _log_between(rng, 300, 20_000)), op=op,
                    pairs=_log_between(rng, 100, 150_000))
    data = rng.choice(["dna", "protein", "text"])
    if data == "dna":
        return dict(_draw_dna(rng, _log_between(rng, 60, 50_000)), op=op)
    if data == "protein":
        return dict(op=op, data=data, n=_log_between(rng, 1000, 190_000), copies=rng.randint(4, 12),
                    q=4, reps=rng.randint(3, 7), t_div=1)
    return dict(op=op, data=data, n=_log_between(rng, 1000, 280_000), copies=rng.randint(4, 12), q=6,
                k=rng.randint(80, 130), reps=rng.randint(1, 4), t_div=2)


# ---------------------------------------------------------------- inputs, on the GPU
def _symbols(gen, count, data):
    sigma, zipf = ALPHABETS[data]
    if zipf is None:
        return torch.randint(0, sigma, (count,), generator=gen, device="cuda", dtype=torch.uint8)
    w = torch.arange(1, sigma + 1, dtype=torch.float64) ** -zipf
    cdf = (torch.cumsum(w, 0) / w.sum()).float().cuda()
    u = torch.rand(count, generator=gen, device="cuda")
    return torch.searchsorted(cdf, u, right=True).clamp_(max=sigma - 1).to(torch.uint8)


def _offsets(lens):
    off = torch.zeros(lens.numel() + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(lens, 0, out=off[1:])
    return off


def _take(chars, offsets, ids):
    """The strings `ids` of a collection, in that order."""
    lens = offsets[ids + 1] - offsets[ids]
    off = _offsets(lens)
    at = torch.repeat_interleave(offsets[ids] - off[:-1], lens)
    at += torch.arange(at.numel(), device="cuda")
    return chars[at], off


def _mutated(gen, chars, offsets, rates, indel, data):
    """Each string with independent edits at its rate: a share `indel` of them insertions and
    deletions in equal parts, the rest substitutions by another symbol."""
    sigma = ALPHABETS[data][0]
    lens = offsets[1:] - offsets[:-1]
    total = chars.numel()
    u = torch.rand(total, generator=gen, device="cuda") / torch.repeat_interleave(rates, lens)
    ins, dele, sub = u < indel / 2, (u >= indel / 2) & (u < indel), (u >= indel) & (u < 1)
    other = torch.randint(1, sigma, (total,), generator=gen, device="cuda", dtype=torch.int16)
    body = torch.where(sub, ((chars + other) % sigma).to(torch.uint8), chars)
    del u, other, sub
    count = 1 + ins.to(torch.int64) - dele.to(torch.int64)
    at = _offsets(count)
    new = torch.empty(int(at[-1]), dtype=torch.uint8, device="cuda")
    new[at[:-1][ins]] = _symbols(gen, int(ins.sum()), data)
    own = ~dele
    new[(at[:-1] + ins)[own]] = body[own]
    return new, at[offsets]


def _lengths(gen, count, case):
    if case["data"] == "protein":
        v = torch.exp(math.log(400) + 0.8 * torch.randn(count, generator=gen, device="cuda"))
        return v.round().clamp_(50, 5000).to(torch.int64)
    if case["data"] == "text":
        v = 1200 + 300 * torch.randn(count, generator=gen, device="cuda")
        return v.round().clamp_(300, 3000).to(torch.int64)
    m = case["mean"]
    v = m * (1 + case["spread"] * (torch.rand(count, generator=gen, device="cuda") * 2 - 1))
    return v.round().clamp_(min=1).to(torch.int64)


def _collection(gen, case):
    """Symbols, offsets and cluster of every string: all clustered for DNA, a fifth of the
    protein-like strings and a tenth of the texts, the others unrelated."""
    n, copies, data = case["n"], case["copies"], case["data"]
    share, lo, hi, indel = {"dna": (1.0, case.get("rate_lo"), case.get("rate_hi"), case.get("indel")),
                            "protein": (0.2, 0.03, 0.12, 0.667),
                            "text": (0.1, 0.02, 0.10, 0.667)}[data]
    members = int(round(n * share))
    clusters = -(-members // copies)
    off = _offsets(_lengths(gen, clusters, case))
    chars = _symbols(gen, int(off[-1]), data)
    of = torch.arange(members, device="cuda") // copies
    chars, off = _take(chars, off, of)
    rates = lo + (hi - lo) * torch.rand(members, generator=gen, device="cuda")
    chars, off = _mutated(gen, chars, off, rates, indel, data)
    if members == n:
        return chars, off, of
    rest = _offsets(_lengths(gen, n - members, case))
    chars = torch.cat([chars, _symbols(gen, int(rest[-1]), data)])
    off = torch.cat([off, off[-1] + rest[1:]])
    of = torch.cat([of, torch.full((n - members,), -1, device="cuda")])
    order = torch.randperm(n, generator=gen, device="cuda")
    chars, off = _take(chars, off, order)
    return chars, off, of[order]


def _strings(chars, offsets, data, packed=False):
    if not packed:
        return mj.DeviceStrings(chars, offsets, ALPHABETS[data][0])
    words = torch.zeros((chars.numel() + 15) // 16, dtype=torch.int32, device="cuda")
    for j in range(16):
        part = chars[j::16].to(torch.int32) << (2 * j)
        words[:part.numel()] |= part
    return mj.DeviceStrings(words, offsets, ALPHABETS[data][0], mj.PACK_2BIT)


def _indexed(gen, case):
    """Unrelated DNA strings to index, and queries: every other one a mutated copy."""
    n, nq = case["n"], case["queries"]
    off = _offsets(torch.randint(1000, 10_001, (n,), generator=gen, device="cuda"))
    chars = _symbols(gen, int(off[-1]), "dna")
    known = (nq + 1) // 2
    src = torch.randint(0, n, (known,), generator=gen, device="cuda")
    qc, qo = _take(chars, off, src)
    rates = 0.05 + 0.10 * torch.rand(known, generator=gen, device="cuda")
    qc, qo = _mutated(gen, qc, qo, rates, 0.667, "dna")
    if nq > known:
        fresh = _offsets(torch.randint(1000, 10_001, (nq - known,), generator=gen, device="cuda"))
        qc = torch.cat([qc, _symbols(gen, int(fresh[-1]), "dna")])
        qo = torch.cat([qo, qo[-1] + fresh[1:]])
    k = -(-(qo[1:] - qo[:-1]) // 10)
    return _strings(chars, off, "dna"), _strings(qc, qo, "dna"), k.to(torch.int32)


# ---------------------------------------------------------------- the context a program keeps
_kept = {}


def _context(case):
    """A program that works on collections of one kind keeps one context for all of them."""
    key = tuple(sorted((k, v) for k, v in case.items() if k != "name"))
    if key not in _kept:
        _kept.clear()
        _kept[key] = mj.Context()
    return _kept[key]


def _room(case):
    """Pairs that the caller's array for the results holds: more than a collection of this kind
    gives (every copy with every other copy of its cluster, for candidates unrelated pairs too)."""
    if case["op"] in ("search", "index"):
        return 64 + 4 * case["queries"]
    if case["op"] == "candidates":
        return 1024 + 16 * case["n"]
    return 1024 + case["n"] * case["copies"]


def _put(state, pairs):
    """The pairs in the caller's array, and how many they are."""
    count = min(len(pairs), len(state["found"]))
    state["found"][:count] = pairs[:count]
    return state["found"], len(pairs)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    ctx = _context(case)
    state = {"op": case["op"], "ctx": ctx, "found": np.zeros(_room(case), dtype=np.uint64)}
    if case["op"] in ("search", "index"):
        strings, queries, k = _indexed(gen, case)
        # T follows each string's own threshold, a tenth of its length
        lens = strings.offsets[1:] - strings.offsets[:-1]
        params = mj.Params(q=case["q"], k_per_string=(-(-lens // 10)).to(torch.int32),
                           t_div=case["t_div"], reps=case["reps"])
        state.update(queries=queries, k=k)
        if case["op"] == "search":
            state["index"] = mj.Index(strings, params, ctx=ctx)
        else:
            state.update(strings=strings, params=params)
        return state
    chars, offsets, cluster = _collection(gen, case)
    k = case.get("k", -1)
    per_string = None
    if k < 0:
        per_string = (-(-(offsets[1:] - offsets[:-1]) * 8 // 100)).to(torch.int32)
    state["strings"] = _strings(chars, offsets, case["data"], case.get("packed", False))
    state["params"] = mj.Params(q=case["q"], k=k, k_per_string=per_string, t_div=case["t_div"],
                                reps=case["reps"])
    if case["op"] == "verify":
        # three quarters of the pairs from one cluster, the others of unrelated strings
        rng = np.random.default_rng(int(seed))
        n, copies = case["n"], case["copies"]
        a = rng.integers(0, n, case["pairs"])
        near = np.minimum(a // copies * copies + rng.integers(0, copies, case["pairs"]), n - 1)
        b = np.where(rng.random(case["pairs"]) < 0.75, near, rng.integers(0, n, case["pairs"]))
        b = np.where(a == b, (a + 1) % n, b)
        a, b = np.minimum(a, b).astype(np.uint64), np.maximum(a, b).astype(np.uint64)
        state["pairs"] = (a << np.uint64(32)) | b
    return state


def run(state):
    op, ctx = state["op"], state["ctx"]
    if op == "verify":
        return mj.verify(state["strings"], state["params"], state["pairs"], ctx=ctx)
    if op in ("search", "index"):
        index = state["index"] if op == "search" else mj.Index(state["strings"], state["params"], ctx=ctx)
        pairs, stats = index.search(state["queries"], k_per_query=state["k"])
        found, count = _put(state, pairs)
        out = {"pairs": found, "count": count, "candidates": stats["candidates"],
               "indexed": index.records}
        if op == "index":
            index.close()
        return out
    call = mj.join if op == "join" else mj.candidates
    pairs, stats = call(state["strings"], state["params"], ctx=ctx)
    found, count = _put(state, pairs)
    return {"pairs": found, "count": count, "candidates": stats["candidates"],
            "records": stats["records"]}


def work(case):
    """Symbols and offsets read once, results written once.  The arithmetic is all on whole
    numbers (hashes, comparisons, bit-parallel edit distance): no floating-point operations."""
    n = case["n"]
    if case["op"] in ("search", "index"):
        queries = case["queries"] * (MEAN_QUERY + 8 + 4)
        # a mutated copy's source is read at 2 bits a symbol to verify it, a record's key probed
        found = case["queries"] * (MEAN_QUERY // 4) // 2
        probes = case["queries"] * (MEAN_QUERY // 20) * 16
        built = n * (MEAN_QUERY + 8 + 4) if case["op"] == "index" else 0
        return {"bytes": float(queries + found + probes + built), "flops": 0.0}
    mean = {"protein": 540, "text": 1200}.get(case["data"]) or case["mean"]
    size = mean / 4 if case.get("packed") else mean
    out = n * 8
    if case["op"] == "verify":
        out = case["pairs"] * 9
    elif case["op"] == "candidates":
        out = n * 8 * 4
    return {"bytes": float(n * (size + 8) + out), "flops": 0.0}


def exact(case, seed):
    """Every output is a whole number, compared as such: there is nothing to round."""
    return None
