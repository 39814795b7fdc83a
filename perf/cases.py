"""The work that programs have this library do, as cases that can be timed.

Every case is one call (or one short sequence of calls) through the public
entry points: self searches from one small sample to a pooled repertoire,
their Hamming and paired-chain forms, queries of one set, of many sets and of
a server's requests against a reference index, and the build of such an index.
Sequences follow the recipe of the repository's seeded generator (lengths
round(Normal(15, 2)) in [8, 24], C...F frame, Zipf interior, 30% mutants of
other sequences), drawn on the GPU.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2403_09010_amd import Context, Server

DEV = "cuda:0"
MAX_LEN, MIN_LEN = 24, 8
CODE_C, CODE_F = 1, 4
FRESH = 0.7      # fresh sequences; the others are mutants of another one
REF_MUT = 0.1    # query sequences that are mutants of a reference sequence
INDEL, MAX_SCORE = 8, 8
MEAN_LEN = 15.0


def listed():
    return [
        # one small sample, the smallest call (launches and latency)
        dict(name="self_10k_k1", kind="self", n=10_000, k=1, hamming=False, host=False),
        # one sample of a cohort, an odd size, host arrays in and out
        dict(name="self_100k_k2_host", kind="self", n=100_003, k=2, hamming=False, host=True),
        # one deep repertoire: the headline self search
        dict(name="self_1m_k2", kind="self", n=1_000_000, k=2, hamming=False, host=False),
        # the same with three deletions
        dict(name="self_1m_k3", kind="self", n=1_000_000, k=3, hamming=False, host=False),
        # a pooled cohort, the largest call
        dict(name="self_10m_k2", kind="self", n=10_000_000, k=2, hamming=False, host=False),
        # comparison with Hamming-only tools on a large set
        dict(name="hamming_2m_k1", kind="self", n=2_000_003, k=1, hamming=True, host=False),
        # both chains of single-cell receptors
        dict(name="paired_1m_k2", kind="paired", n=1_000_000, k=2),
        # one request of a service alone: a small host set, rescored, against a large database
        dict(name="query_3k_weighted", kind="query", n=3_000, ref=5_000_000, k=2, weighted=True, host=True),
        # one repertoire against a database, device arrays
        dict(name="query_200k", kind="query", n=200_000, ref=2_000_000, k=2, weighted=False, host=False),
        # many patients' sets against a database in one call
        dict(name="batch_20", kind="batch", sets=20, lo=1_000, hi=200_000, ref=2_000_000, k=2),
        # a queue of requests of mixed sizes at a server
        dict(name="serve_16", kind="serve", sets=16, lo=100, hi=50_000, ref=5_000_000),
        # a database indexed anew and queried once
        dict(name="build_2m", kind="build", n=5_000, ref=2_000_000, k=2),
    ]


def _size(rng, lo, hi):
    """An integer in [lo, hi], spread over its logarithm (odd as often as even)."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["self", "self", "self", "paired", "query", "query", "batch", "serve", "build"])
    if kind == "self":
        k = rng.choice([1, 2, 2, 3])
        hi = {1: 10_000_000, 2: 8_000_000, 3: 1_000_000}[k]
        return dict(kind=kind, n=_size(rng, 10_000, hi), k=k, hamming=rng.random() < 0.2,
                    host=rng.random() < 0.3)
    if kind == "paired":
        return dict(kind=kind, n=_size(rng, 10_000, 1_000_000), k=rng.choice([1, 2, 2]))
    if kind == "query":
        weighted = rng.random() < 0.5
        return dict(kind=kind, n=_size(rng, 3_000, 200_000), ref=_size(rng, 200_000, 5_000_000),
                    k=2 if weighted else rng.choice([1, 2, 2]), weighted=weighted,
                    host=rng.random() < 0.5)
    if kind == "batch":
        return dict(kind=kind, sets=rng.randint(2, 20), lo=1_000, hi=_size(rng, 5_000, 200_000),
                    ref=_size(rng, 200_000, 2_000_000), k=2)
    if kind == "serve":
        return dict(kind=kind, sets=rng.randint(2, 16), lo=100, hi=_size(rng, 1_000, 50_000),
                    ref=_size(rng, 200_000, 5_000_000))
    return dict(kind=kind, n=_size(rng, 1_000, 20_000), ref=_size(rng, 100_000, 2_000_000),
                k=rng.choice([1, 2, 2]))


# ------------------------------------------------------------------ inputs
# A set of sequences is a padded (codes uint8[n, 24], lengths int64[n]) pair
# until it is handed over as CSR.

def _residue_cdf():
    perm = random.Random(12345).sample(range(20), 20)
    p = [0.0] * 20
    for r, code in enumerate(perm):
        p[code] = 1.0 / (r + 1)
    return torch.tensor(p, dtype=torch.float32, device=DEV).cumsum(0) / sum(p)


def _residues(g, *shape):
    u = torch.rand(*shape, generator=g, device=DEV)
    return torch.bucketize(u, _residue_cdf(), right=True, out_int32=True).clamp_(max=19).to(torch.uint8)


def _below(g, hi, n):
    """n integers, the t-th uniform in [0, hi[t])."""
    u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
    return torch.minimum((u * hi).long(), hi - 1)


def _fresh(g, n):
    ln = torch.randn(n, generator=g, device=DEV).mul_(2.0).add_(15.0).round_()
    ln = ln.clamp_(MIN_LEN, MAX_LEN).long()
    codes = _residues(g, n, MAX_LEN)
    codes[:, 0] = CODE_C
    codes.scatter_(1, (ln - 1)[:, None], CODE_F)
    return codes, ln


def _edit(g, codes, ln):
    """One interior edit of every sequence: substitution, insertion or deletion."""
    n = len(ln)
    kind = torch.randint(0, 3, (n,), generator=g, device=DEV)
    kind[(kind == 1) & (ln >= MAX_LEN)] = 0
    kind[(kind == 2) & (ln <= MIN_LEN)] = 0
    pos = 1 + _below(g, torch.where(kind == 1, ln - 1, ln - 2), n)
    new = _residues(g, n)
    old = codes.gather(1, pos[:, None])[:, 0]
    new = torch.where((kind == 0) & (new == old), (new + 1) % 20, new).to(torch.uint8)
    at = torch.arange(MAX_LEN, device=DEV)[None, :]
    src = at - ((kind == 1)[:, None] & (at > pos[:, None])).long()
    src = src + ((kind == 2)[:, None] & (at >= pos[:, None])).long()
    out = codes.gather(1, src.clamp_(0, MAX_LEN - 1))
    keep = out.gather(1, pos[:, None])[:, 0]
    out.scatter_(1, pos[:, None], torch.where(kind == 2, keep, new)[:, None])
    return out, ln + (kind == 1).long() - (kind == 2).long()


def _mutants(g, codes, ln):
    """One or two edits of every sequence."""
    codes, ln = _edit(g, codes, ln)
    c2, l2 = _edit(g, codes, ln)
    two = torch.rand(len(ln), generator=g, device=DEV) < 0.5
    return torch.where(two[:, None], c2, codes), torch.where(two, l2, ln)


def _grow(g, n, make, mutate):
    """n records: fresh ones, then three generations of mutants of all before, shuffled."""
    base = max(1, n - int((1 - FRESH) * n))
    cols = make(base)
    while len(cols[0]) < n:
        m = min(n - len(cols[0]), max(1, int((1 - FRESH) * n) // 3))
        u = torch.randint(0, len(cols[0]), (m,), generator=g, device=DEV)
        cols = [torch.cat(x) for x in zip(cols, mutate([c[u] for c in cols]))]
    perm = torch.randperm(n, generator=g, device=DEV)
    return [c[perm] for c in cols]


def _sequences(g, n):
    return _grow(g, n, lambda m: list(_fresh(g, m)), lambda cols: list(_mutants(g, *cols)))


def _paired(g, n):
    def mutate(cols):
        ca, la, cb, lb = cols
        ma, na = _mutants(g, ca, la)
        mb, nb = _mutants(g, cb, lb)
        a = torch.rand(len(la), generator=g, device=DEV) < 0.5
        return [torch.where(a[:, None], ma, ca), torch.where(a, na, la),
                torch.where(a[:, None], cb, mb), torch.where(a, lb, nb)]
    return _grow(g, n, lambda m: [*_fresh(g, m), *_fresh(g, m)], mutate)


def _queries(g, n, ref):
    codes, ln = _sequences(g, n)
    hit = torch.rand(n, generator=g, device=DEV) < REF_MUT
    u = torch.randint(0, len(ref[1]), (n,), generator=g, device=DEV)
    mc, ml = _mutants(g, ref[0][u], ref[1][u])
    return torch.where(hit[:, None], mc, codes), torch.where(hit, ml, ln)


def _csr(codes, ln, host=False):
    mask = torch.arange(MAX_LEN, device=DEV)[None, :] < ln[:, None]
    flat = codes[mask]
    offs = torch.zeros(len(ln) + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(ln, 0, out=offs[1:])
    return (flat.cpu().numpy(), offs.cpu().numpy()) if host else (flat, offs)


def _costs():
    r = random.Random(8)
    c = np.zeros((20, 20), dtype=np.uint8)
    for a in range(20):
        for b in range(a + 1, 20):
            c[a, b] = c[b, a] = r.choice((3, 4))
    return c


def _sizes(case):
    """The set sizes of a batch or a queue: log-uniform over the range, the same for every seed."""
    n = case["sets"]
    q = [(x + 0.5) / n for x in range(n)]
    random.Random(5).shuffle(q)
    return [int(round(case["lo"] * (case["hi"] / case["lo"]) ** t)) for t in q]


_CTX = None


def _context():
    """The one context that a program keeps for all its searches."""
    global _CTX
    if _CTX is None:
        _CTX = Context(0)
    return _CTX


def prepare(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    ctx = _context()
    st = dict(case=case, ctx=ctx)
    kind = case["kind"]
    if kind == "self":
        st["set"] = _csr(*_sequences(g, case["n"]), host=case["host"])
    elif kind == "paired":
        ca, la, cb, lb = _paired(g, case["n"])
        st["a"], st["b"] = _csr(ca, la), _csr(cb, lb)
    else:
        ref = _sequences(g, case["ref"])
        if kind in ("batch", "serve"):
            st["sets"] = [_csr(*_queries(g, n, ref), host=kind == "serve") for n in _sizes(case)]
        else:
            st["set"] = _csr(*_queries(g, case["n"], ref), host=case.get("host", False))
        st["subst"] = _costs()
        if kind == "build":
            st["ref"] = _csr(*ref)
        else:
            st["index"] = ctx.build_index(*_csr(*ref), case.get("k", 2))
        if kind == "serve":
            st["server"] = Server(st["index"], k=2, subst=st["subst"], indel=INDEL,
                                  max_score=MAX_SCORE)
    host = case.get("host", kind == "serve")
    sizes = _sizes(case) if kind in ("batch", "serve") else [case["n"]]
    st["out"] = [_arrays(case, n, host) for n in sizes]
    torch.cuda.synchronize()
    return st


def _rate(case):
    """Triplets per sequence that the recipe gives, with room to spare."""
    k, m = case.get("k", 2), (case["ref"] if "ref" in case else case["n"]) / 1e6
    if "ref" in case:
        return 0.2 + 0.15 * m
    return {1: 0.25, 2: 0.45 + 0.06 * m, 3: 0.6 + 1.3 * m}[k]


def _arrays(case, n, host):
    """The arrays in which a program collects the triplets of n sequences."""
    cap = int(1.25 * _rate(case) * n) + 2000
    if host:
        return [np.zeros(cap, dtype=t) for t in (np.uint32, np.uint32, np.uint8)]
    return [torch.zeros(cap, dtype=t, device=DEV) for t in (torch.int32, torch.int32, torch.uint8)]


def _collect(outs, results):
    """The results copied to the program's own arrays, and their counts."""
    for bufs, r in zip(outs, results):
        for b, x in zip(bufs, (r.i, r.j, r.d)):
            b[:len(x)] = x
    return {"n": np.array([len(r) for r in results]), "triplets": outs}


def run(st):
    case, ctx = st["case"], st["ctx"]
    kind = case["kind"]
    if kind == "self":
        rs = [ctx.self_search(*st["set"], case["k"], hamming=case["hamming"])]
    elif kind == "paired":
        rs = [ctx.paired_self_search(st["a"], st["b"], case["k"])]
    elif kind == "query" and case["weighted"]:
        rs = [ctx.query_weighted(st["index"], *st["set"], st["subst"], INDEL, MAX_SCORE)]
    elif kind == "query":
        rs = [ctx.query(st["index"], *st["set"], case["k"])]
    elif kind == "batch":
        rs = ctx.query_batch(st["index"], st["sets"], case["k"])
    elif kind == "serve":
        ids = [st["server"].submit(*s) for s in st["sets"]]
        rs = [st["server"].poll(x)[0] for x in ids]
    else:
        index = ctx.build_index(*st["ref"], case["k"])
        rs = [ctx.query(index, *st["set"], case["k"])]
        index.free()
    return _collect(st["out"], rs)


def work(case):
    """Codes and offsets read once, triplets (9 bytes) written once. A query
    reads of the index at least one 64-byte line per variant it looks up; a
    build reads the reference and writes 8 bytes per variant of it."""
    kind, k = case["kind"], case.get("k", 2)
    per_seq = MEAN_LEN + 8
    variants = sum(math.comb(int(MEAN_LEN), m) for m in range(k + 1)) * 0.82
    pairs = _rate(case) * 9
    if kind == "self":
        b = case["n"] * (per_seq + pairs)
    elif kind == "paired":
        b = case["n"] * (2 * per_seq + pairs)
    else:
        n = sum(_sizes(case)) if kind in ("batch", "serve") else case["n"]
        b = n * (per_seq + pairs + 64 * variants)
        if kind == "build":
            b += case["ref"] * (per_seq + 16 + 8 * variants)
    return {"bytes": float(b), "flops": 0.0}


# ------------------------------------------------------------------ reference

def _levenshtein(a, la, b, lb):
    """Unit-cost edit distance of each row pair, by the full programme."""
    n = len(la)
    row = torch.arange(MAX_LEN + 1, device=DEV, dtype=torch.int64)[None, :].repeat(n, 1)
    out = torch.where((la == 0)[:, None], row, 0)
    at = torch.arange(1, MAX_LEN + 1, device=DEV)
    for x in range(1, MAX_LEN + 1):
        t = torch.minimum(row[:, :-1] + (a[:, x - 1:x] != b).long(), row[:, 1:] + 1)
        t = torch.cat([torch.full((n, 1), x, device=DEV, dtype=torch.int64), t], 1)
        # insertions: new[y] = min over z <= y of t[z] + (y - z)
        shift = torch.cat([at.new_zeros(1), at])[None, :]
        row = torch.cummin(t - shift, 1).values + shift
        out = torch.where((la == x)[:, None], row, out)
    return out.gather(1, lb[:, None])[:, 0]


def exact(case, seed):
    """The triplets by brute force, where every pair can be looked at: pairs
    whose lengths and residue counts allow the distance, then the full
    programme."""
    if case["kind"] != "self" or case["n"] > 30_000:
        return None
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    codes, ln = _sequences(g, case["n"])
    n, k = case["n"], case["k"]
    valid = torch.arange(MAX_LEN, device=DEV)[None, :] < ln[:, None]
    bag = torch.zeros(n, 20, device=DEV)
    bag.scatter_add_(1, codes.long(), valid.float())
    found = []
    for x in range(0, n, 512):
        y = min(n, x + 512)
        near = (bag[x:y, None, :] - bag[None, x:, :]).abs_().sum(2) <= 2 * k
        i, j = near.nonzero(as_tuple=True)
        i, j = i + x, j + x
        keep = (i < j) & ((ln[i] - ln[j]).abs() <= (0 if case["hamming"] else k))
        i, j = i[keep], j[keep]
        if case["hamming"]:
            d = ((codes[i] != codes[j]) & valid[i]).sum(1)
        else:
            d = _levenshtein(codes[i], ln[i], codes[j], ln[j])
        found.append(torch.stack([i, j, d])[:, d <= k])
    r = torch.cat(found, 1)
    out = _arrays(case, n, case["host"])
    for b, x in zip(out, r):
        b[:len(x)] = x.cpu().numpy() if case["host"] else x
    return {"n": np.array([r.shape[1]]), "triplets": [out]}
