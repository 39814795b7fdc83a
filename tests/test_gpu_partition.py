"""The automatic grouping of self searches (variants partitioned into hash bins,
each filtered and grouped by one workgroup) against the sorted grouping path,
at the sizes where its plan changes and on inputs that overflow its bins."""
import numpy as np
import pytest

import cdr3gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def paths():
    from paper_2403_09010_amd import Context
    from paper_2403_09010_amd.symdel import OPT_PATH
    a, b = Context(0), Context(0)
    b.set_option(OPT_PATH, 2)
    yield a, b
    a.close()
    b.close()


def csr(strings):
    offs = np.zeros(len(strings) + 1, dtype=np.int64)
    offs[1:] = np.cumsum([len(s) for s in strings])
    return np.frombuffer(b"".join(strings), dtype=np.uint8).copy(), offs


def strings_of(seed, n):
    c, o = cdr3gen.generate(seed, n)
    return [c[o[t]:o[t + 1]].tobytes() for t in range(n)]


def same(paths, c, o, k, hamming=False):
    print(f"[partition] {len(o) - 1} sequences k={k} hamming={hamming}", flush=True)
    a = paths[0].self_search(c, o, k, hamming=hamming)
    b = paths[1].self_search(c, o, k, hamming=hamming)
    assert len(a) == len(b)
    assert np.array_equal(a.i, b.i) and np.array_equal(a.j, b.j) and np.array_equal(a.d, b.d)
    sa, sb = paths[0].stats(), paths[1].stats()
    assert sa["n_keys"] == sb["n_keys"] and sa["n_sort_passes"] == 0
    return sa


# one bin; bins at their smallest; around 2^21 variants (one region per bin,
# then eight); around 2^24 (small and large workgroups); 2^12 bins; two levels
@pytest.mark.parametrize("n,k", [(1, 2), (37, 0), (300, 2), (20_800, 2), (20_950, 2), (166_000, 2),
                                 (168_500, 2), (1_250_000, 2), (470_000, 3), (2_100_000, 1)])
def test_plan_sizes(paths, n, k):
    same(paths, *cdr3gen.generate(100 + n % 97, n), k)


def test_hamming(paths):
    same(paths, *cdr3gen.generate(5, 60_000), 2, hamming=True)


@pytest.mark.parametrize("length", [1, 2, 3, 23, 24])
def test_lengths(paths, length):
    rng = np.random.default_rng(length)
    pick = rng.integers(0, 3 if length > 3 else 20, (400, length)).astype(np.uint8)
    for k in (0, 1, 2, 3):
        same(paths, *csr([bytes(x) for x in pick]), k)


# small inputs are sized by an estimate: the most variants a sequence can have,
# and sequences that are refused in between
@pytest.mark.parametrize("n,k", [(1, 3), (40, 3), (2_000, 2), (9_000, 2), (30_000, 1)])
def test_estimated_sizes(paths, n, k):
    from paper_2403_09010_amd import SymdelError
    rng = np.random.default_rng(n)
    rows = np.argsort(rng.random((n, 20)), axis=1).astype(np.uint8)
    rows = np.concatenate([rows, rows[:, :4]], axis=1)  # 24 residues, no two neighbours alike
    rows[n // 2:, 3] = rows[:n - n // 2, 7]
    c, o = csr([bytes(x) for x in rows])
    same(paths, c, o, k)
    for bad, name in ((np.full(1, 20, np.uint8), "SD_E_ALPHABET"), (np.zeros(0, np.uint8), "SD_E_LENGTH"),
                      (np.zeros(25, np.uint8), "SD_E_LENGTH")):
        with pytest.raises(SymdelError) as e:
            paths[0].self_search(np.concatenate([c, bad]), np.append(o, o[-1] + len(bad)), k)
        assert e.value.name == name


def test_sequences_sorted_by_length(paths):
    # consecutive long sequences: workgroups hold more variants than the mean
    s = sorted(strings_of(9, 30_000), key=len)
    same(paths, *csr(s), 2)
    same(paths, *csr(s), 3)


def test_every_element_shared(paths):
    # each sequence twice: every element passes the filter, so bins are
    # grouped in several rounds
    s = strings_of(7, 60_000)
    assert same(paths, *csr(s + s), 2)["n_big_segments"] == 0


def test_overflowing_bins(paths):
    # 2,000 copies of one sequence among 200,000: its variants' bins overflow
    # their regions and are grouped by a sort
    s = strings_of(8, 200_000)
    assert same(paths, *csr(s + [s[17]] * 2_000), 1)["n_big_segments"] > 0


def test_overflow_area_too_small(paths):
    # copies only: the overflow area overflows and the sorted path takes over
    s = strings_of(11, 3)
    from paper_2403_09010_amd.symdel import OPT_PATH  # noqa: F401
    print("[partition] copies of three sequences", flush=True)
    c, o = csr([s[t % 3] for t in range(9_000)])
    a, b = paths[0].self_search(c, o, 1), paths[1].self_search(c, o, 1)
    assert np.array_equal(a.i, b.i) and np.array_equal(a.j, b.j) and np.array_equal(a.d, b.d)


def test_wide_ids(paths):
    # more than 2^24 sequences: 32 id bits and 32 hash bits
    same(paths, *cdr3gen.generate(13, (1 << 24) + 3), 0)


# 32 id bits on two levels; 2^18 bins, which the first level shares out further
@pytest.mark.parametrize("n,k,least", [((1 << 24) + 5, 1, 51_200 << 12), (3_850_000, 3, 51_200 << 15)])
def test_large_plans(n, k, least):
    from paper_2403_09010_amd import Context
    from paper_2403_09010_amd.symdel import OPT_PATH
    with Context(0) as a, Context(0) as b:
        b.set_option(OPT_PATH, 2)
        assert same((a, b), *cdr3gen.generate(15, n), k)["n_keys"] > least


def test_budget_without_room_for_two_levels(paths):
    # the sorted path fits, two levels do not: their generator does not run for nothing
    from paper_2403_09010_amd import Context
    from paper_2403_09010_amd.symdel import OPT_TIMING
    c, o = cdr3gen.generate(16, 2_300_000)
    want = paths[0].self_search(c, o, 2)
    nk = paths[0].stats()["n_keys"]
    assert nk > 51_200 << 12
    print(f"[partition] a budget of 22 bytes for each of {nk} variants", flush=True)
    with Context(0, hbm_budget=22 * nk) as ctx:
        ctx.set_option(OPT_TIMING, 1)
        got = ctx.self_search(c, o, 2)
        names = [s["name"] for s in ctx.stats()["stages"]]
    assert np.array_equal(got.i, want.i) and np.array_equal(got.j, want.j)
    assert "vargen_hash" in names and "vargen_part" not in names


def same_paired(paths, a, b, k):
    print(f"[partition] {len(a[1]) - 1} paired records k={k}", flush=True)
    x = paths[0].paired_self_search(a, b, k)
    y = paths[1].paired_self_search(a, b, k)
    assert len(x) == len(y)
    assert np.array_equal(x.i, y.i) and np.array_equal(x.j, y.j) and np.array_equal(x.d, y.d)
    # the sorted path writes repeated variants of a record too
    assert paths[0].stats()["n_keys"] <= paths[1].stats()["n_keys"]


# joined strings around the 32 and 64 positions where the generator's halves,
# rotations and masks change form, down to one residue per chain
@pytest.mark.parametrize("la,lb", [(1, 1), (1, 24), (24, 1), (24, 24), (15, 15), (15, 16), (16, 16),
                                   (23, 9)])
def test_paired_lengths(paths, la, lb):
    rng = np.random.default_rng(la * 25 + lb)
    a, b = (csr([bytes(x) for x in rng.integers(0, 3, (300, n)).astype(np.uint8)]) for n in (la, lb))
    for k in (0, 1, 2, 3):
        same_paired(paths, a, b, k)


@pytest.mark.parametrize("n", [1, 2_000, 40_000, 250_000])
def test_paired_sizes(paths, n):
    same_paired(paths, *cdr3gen.paired(n % 89, n), 2)


@pytest.fixture(scope="module")
def query_paths():
    from paper_2403_09010_amd import Context
    from paper_2403_09010_amd.symdel import OPT_JOIN_ELEMS
    a, b = Context(0), Context(0)
    b.set_option(OPT_JOIN_ELEMS, 1)  # the general path
    yield a, b
    a.close()
    b.close()


def same_query(paths, idx, q, k, subst=None):
    print(f"[partition] {len(q[1]) - 1} queries k={k} weighted={subst is not None}", flush=True)
    if subst is not None:
        x, y = (c.query_weighted(idx, *q, subst, 8, 8) for c in paths)
    else:
        x, y = (c.query(idx, *q, k) for c in paths)
    assert len(x) == len(y)
    assert np.array_equal(x.i, y.i) and np.array_equal(x.j, y.j) and np.array_equal(x.d, y.d)
    assert paths[0].stats()["n_keys"] == paths[1].stats()["n_keys"]


# looked up one by one, joined with few and with many elements per workgroup,
# and single queries; every radius up to the index's
@pytest.mark.parametrize("nref,k,sizes", [(3_000, 3, (1, 9, 1_500)), (40, 2, (1, 700)),
                                          (60_000, 2, (1, 900, 30_000)), (300_000, 2, (60_000,))])
def test_query_sizes(query_paths, nref, k, sizes):
    ref = cdr3gen.generate(nref % 83, nref)
    idx = query_paths[0].build_index(*ref, k)
    for n in sizes:
        q = cdr3gen.generate_query(n % 71, n, *ref, ref_mut_frac=0.3)
        for kk in range(k + 1):
            same_query(query_paths, idx, q, kk)
        if k == 2:
            same_query(query_paths, idx, q, k, cdr3gen.cost_matrix())
    idx.free()


def test_query_copies(query_paths):
    # variants shared by thousands of references, of queries, and of both
    s = strings_of(17, 1_000)
    many = csr([s[5]] * 9_000 + s)
    few = csr([s[5]] * 3 + s[:50])
    for ref, queries in ((many, (few, csr(s * 20))), (csr(strings_of(18, 50_000)), (many,))):
        idx = query_paths[0].build_index(*ref, 1)
        for q in queries:
            same_query(query_paths, idx, q, 1)
        idx.free()


@pytest.fixture(scope="module")
def build_paths():
    from paper_2403_09010_amd import Context
    from paper_2403_09010_amd.symdel import OPT_SORT_ITEMS
    a, b = Context(0), Context(0)
    b.set_option(OPT_SORT_ITEMS, 16)
    yield a, b
    a.close()
    b.close()


def same_index(paths, ref, k, queries):
    """Indexes built bin by bin and by digit passes: the same sizes and answers."""
    print(f"[index] {len(ref[1]) - 1} references k={k}", flush=True)
    a, b = (c.build_index(*ref, k) for c in paths)
    assert a.info() == b.info()
    for q in queries:
        x, y = paths[0].query(a, *q, k), paths[0].query(b, *q, k)
        assert len(x) == len(y)
        assert np.array_equal(x.i, y.i) and np.array_equal(x.j, y.j) and np.array_equal(x.d, y.d)
    a.free()
    b.free()


# 2^1 to 2^8 bins, one level up to 2^12 bins, two levels, every radius; queries
# that look their variants up, and that join whole bins
@pytest.mark.parametrize("n,k", [(1, 2), (65, 0), (700, 3), (9_000, 1), (60_000, 2), (300_000, 2),
                                 (100_000, 3), (900_000, 2)])
def test_index_sizes(build_paths, n, k):
    ref = cdr3gen.generate(n % 89, n)
    same_index(build_paths, ref, k, [cdr3gen.generate_query(3, min(n, 3_000), *ref, ref_mut_frac=0.5),
                                     cdr3gen.generate_query(4, min(n, 40_000), *ref, ref_mut_frac=0.9)])


# variants shared by so many references that bins hold more than a workgroup
# sorts, that a region overflows, and that most elements are in such bins
@pytest.mark.parametrize("copies,rest", [(7_000, 60_000), (9_000, 3_000), (30_000, 300_000),
                                         (50_000, 10)])
def test_index_copies(build_paths, copies, rest):
    s = strings_of(19, rest)
    ref = csr(s[:rest // 2] + [s[0]] * copies + [s[1][:1]] * 3 + s[rest // 2:])
    same_index(build_paths, ref, 2, [csr(s[:3] + s[-500:]), csr(s[-min(rest, 30_000):])])


# batches of device sets are packed where they lie: set sizes around a
# workgroup's 256 sequences, empty sets, one set, tiles of several sets
@pytest.mark.parametrize("sizes", [(0, 1, 255, 0, 256, 257, 1, 0), (700,), (0, 0), (1,) * 70,
                                   (3_000, 40_000, 900)])
def test_batch_device_sets(query_paths, sizes):
    import torch
    ctx = query_paths[0]
    ref = cdr3gen.generate(29, 8_000)
    idx = ctx.build_index(*ref, 2)
    none = (np.zeros(0, np.uint8), np.zeros(1, np.int64))
    sets = [cdr3gen.generate_query(600 + x, n, *ref, ref_mut_frac=0.4) if n else none
            for x, n in enumerate(sizes)]
    dev = [tuple(torch.from_numpy(a).cuda() for a in q) for q in sets]
    for q, r in zip(sets, ctx.query_batch(idx, dev, 2)):
        want = ctx.query(idx, *q, 2)
        assert len(r) == len(want)
        for a, b in zip(r.numpy(), want.numpy()):
            assert np.array_equal(a, b)
    idx.free()


# offsets of a device set that the kernel must refuse without reading past them
@pytest.mark.parametrize("at,value,name", [(0, 3, "SD_E_INVAL"), (5, -9, "SD_E_INVAL"),
                                           (40, 1 << 40, "SD_E_INVAL"),
                                           (-1, 1 << 40, "SD_E_LENGTH")])
def test_batch_device_offsets_refused(query_paths, at, value, name):
    import torch
    from paper_2403_09010_amd import SymdelError
    ctx = query_paths[0]
    ref = cdr3gen.generate(29, 3_000)
    idx = ctx.build_index(*ref, 1)
    good = cdr3gen.generate_query(7, 300, *ref)
    bad = good[1].copy()
    bad[at] = value
    sets = [tuple(torch.from_numpy(a).cuda() for a in q) for q in (good, (good[0], bad), good)]
    with pytest.raises(SymdelError) as e:
        ctx.query_batch(idx, sets, 1)
    assert e.value.name == name
    assert len(ctx.query_batch(idx, sets[::2], 1)) == 2
    idx.free()


# two offsets that agree with each other, past the codes' end
@pytest.mark.parametrize("at", [60, 1, 253, 256])
def test_batch_device_offsets_beyond_the_codes(query_paths, at):
    import torch
    from paper_2403_09010_amd import SymdelError
    ctx = query_paths[0]
    ref = cdr3gen.generate(29, 3_000)
    idx = ctx.build_index(*ref, 1)
    good = csr([bytes([x % 20] * 10) for x in range(300)])
    bad = good[1].copy()
    bad[at], bad[at + 1] = 3_400, 3_410
    sets = [tuple(torch.from_numpy(a).cuda() for a in q) for q in (good, (good[0], bad), good)]
    with pytest.raises(SymdelError) as e:
        ctx.query_batch(idx, sets, 1)
    assert e.value.name == "SD_E_INVAL"
    idx.free()


# codes at any alignment, part of a workgroup and whole ones, against the host's
# own copy of the same sequences
@pytest.mark.parametrize("n,shift", [(1, 3), (255, 1), (256, 15), (257, 8), (1_000, 7)])
def test_unaligned_codes(paths, n, shift):
    import torch
    c, o = cdr3gen.generate(n, n)
    c = c.copy()
    c[o[n // 2]:o[n // 2] + 2] = (0, 19)  # the residue codes' ends
    dev = torch.zeros(len(c) + shift, dtype=torch.uint8, device="cuda")
    dev[shift:] = torch.from_numpy(c).cuda()
    for k in (0, 2):
        a = paths[0].self_search(dev[shift:], torch.from_numpy(o).cuda(), k)
        b = paths[1].self_search(c, o, k)
        assert len(a) == len(b)
        for x, y in zip(a.numpy(), b.numpy()):
            assert np.array_equal(x, y)


# blocks of freed indexes serve the next ones: sizes that fit, nearly fit and do
# not, two indexes at a time, and one that outlives its context
@pytest.mark.parametrize("sizes", [(40_000, 40_100, 39_000), (60_000, 500, 60_000), (1, 30_000, 1)])
def test_index_memory_kept(sizes):
    from paper_2403_09010_amd import Context
    ctx, fresh = Context(0), Context(0)
    for n in sizes:
        ref = cdr3gen.generate(31, n)
        q = cdr3gen.generate_query(5, 2_000, *ref, ref_mut_frac=0.6)
        a, b = ctx.build_index(*ref, 2), ctx.build_index(*ref, 1)
        c = fresh.build_index(*ref, 2)
        assert a.info() == c.info()
        x, y = ctx.query(a, *q, 2), fresh.query(c, *q, 2)
        assert np.array_equal(x.i, y.i) and np.array_equal(x.j, y.j) and np.array_equal(x.d, y.d)
        a.free()
        z = ctx.query(b, *q, 1)
        keep = y.d <= 1
        assert np.array_equal(z.i, y.i[keep]) and np.array_equal(z.j, y.j[keep])
        b.free()
    ctx.close()
    x = fresh.query(c, *q, 2)
    assert np.array_equal(x.i, y.i) and np.array_equal(x.j, y.j)
    last = fresh
    last.close()
    c.free()


def test_query_copies_after_a_larger_set(query_paths):
    # copies overflow their bins' regions; the slots that a cut run leaves behind
    # hold elements of the larger set before, whose last ids the smaller one has not
    rng = np.random.default_rng(41)
    pick = [bytes(x) for x in rng.integers(0, 20, (80_000, 11)).astype(np.uint8)]
    long = bytes(rng.permutation(20).astype(np.uint8)) + b"\1\5\3\7"
    ctx = query_paths[0]
    idx = ctx.build_index(*csr(pick[60_000:] + [long]), 2)
    large = csr(pick[:60_000] + [long] * 5_000)
    small = csr([long] * 5_000 + pick[:59_000])
    want = query_paths[1].query(idx, *small, 2)
    for turn in range(4):
        print(f"[partition] copies after a larger set, turn {turn}", flush=True)
        ctx.query(idx, *large, 2)
        got = ctx.query(idx, *small, 2)
        assert np.array_equal(got.i, want.i) and np.array_equal(got.j, want.j)
    idx.free()


def not_slower(binned, general, call, check):
    """Median times of call(ctx) on two contexts in turn, after one call of each."""
    import time
    import torch
    check(call(binned), call(general))
    times = {binned: [], general: []}
    for _ in range(7):
        for ctx in times:
            torch.cuda.synchronize()
            t = time.perf_counter()
            call(ctx)
            torch.cuda.synchronize()
            times[ctx].append(time.perf_counter() - t)
    a, b = (float(np.median(t)) for t in times.values())
    print(f"[partition] {a * 1e3:.3f} ms, the path that sorts {b * 1e3:.3f}", flush=True)
    assert a < 1.25 * b


def equal(a, b):
    for x, y in zip(a.numpy(), b.numpy()):
        assert np.array_equal(x, y)


# copies that bins, lists and hash sets were not sized for take no longer than where
# all candidates are sorted
@pytest.mark.parametrize("n,clones,copies,k", [(100_000, 1, 3_000, 2), (300_000, 20, 300, 3)])
def test_copies_take_no_longer(paths, n, clones, copies, k):
    import torch
    s = strings_of(23, n)
    q = [torch.from_numpy(a).cuda() for a in csr(s + [x for x in s[:clones] for _ in range(copies)])]
    not_slower(*paths, lambda ctx: ctx.self_search(*q, k), equal)


# the first search of a context, whose bins are sized for sequences without copies
@pytest.mark.parametrize("n,copies,k", [(10_000, 300, 2), (10_000, 1_000, 1), (3_000, 200, 3),
                                        (40_000, 40, 2)])
def test_first_search_with_copies(paths, n, copies, k):
    from paper_2403_09010_amd import Context
    s = strings_of(29, n)
    c, o = csr(s + [s[9]] * copies)
    print(f"[partition] the first search of a context: {n} sequences, {copies} copies, k={k}", flush=True)
    with Context(0) as ctx:
        equal(ctx.self_search(c, o, k), paths[1].self_search(c, o, k))


@pytest.fixture(scope="module")
def sorting():
    """The automatic path, and contexts whose candidates are sorted by either kind of passes."""
    from paper_2403_09010_amd import Context
    from paper_2403_09010_amd.symdel import OPT_PAIR_SORT
    ctxs = [Context(0) for _ in range(3)]
    for x in (1, 2):
        ctxs[x].set_option(OPT_PAIR_SORT, x)
    yield ctxs
    for c in ctxs:
        c.close()


# references with thousands and hundreds of copies, copies among the queries, queries
# that are all in the index, with three deletions too
@pytest.mark.parametrize("nref,copies,k,queries,qcopies", [
    (200_000, 9_000, 2, 50, 3), (200_000, 9_000, 2, 3_000, 300), (200_000, 9_000, 2, 200_000, 0),
    (200_000, 500, 2, 3_000, 300), (300_000, 0, 2, 30_000, 3_000), (300_000, 0, 2, 30_000, 30_000),
    (300_000, 0, 1, 100_000, 5_000), (100_000, 0, 3, 1_000, 0), (100_000, 0, 3, 20_000, 0)])
def test_query_copies_take_no_longer(sorting, nref, copies, k, queries, qcopies):
    import torch
    s = strings_of(23, nref)
    idx = sorting[0].build_index(*csr([s[5]] * copies + s), k)
    q = [torch.from_numpy(a).cuda() for a in csr([s[5]] * qcopies + s[:queries])]
    n = len(sorting[0].query(idx, *q, k))
    print(f"[partition] {nref} references, {queries} queries, {n} pairs", flush=True)
    general = sorting[2 if n >= 1 << 20 else 1]
    not_slower(sorting[0], general, lambda ctx: ctx.query(idx, *q, k), equal)
    idx.free()


# the first queries with copies: one search finds out how many there are, one puts them
@pytest.mark.parametrize("copies,queries,qcopies", [(500, 50, 3), (2_000, 50, 3), (500, 3_000, 30)])
def test_first_query_with_copies(sorting, copies, queries, qcopies):
    from paper_2403_09010_amd import Context
    from paper_2403_09010_amd.symdel import OPT_TIMING
    s = strings_of(31, 100_000)
    q = csr([s[5]] * qcopies + s[:queries])
    with Context(0) as ctx:
        ctx.set_option(OPT_TIMING, 1)
        idx = ctx.build_index(*csr([s[5]] * copies + s), 2)
        print(f"[partition] {copies} copies, {queries} queries", flush=True)
        found = ctx.query(idx, *q, 2)
        stages = [x["name"] for x in ctx.stats()["stages"]]
        idx.free()
    idx = sorting[1].build_index(*csr([s[5]] * copies + s), 2)
    equal(found, sorting[1].query(idx, *q, 2))
    idx.free()
    assert stages.count("join") <= 2, stages
