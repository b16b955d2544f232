"""HIP path vs the CPU oracle, element by element (needs a gfx950 GPU).

B and the unions are compared as integers, J bit for bit (binary64), |X_i|
exactly.  Sizes here finish in seconds on the oracle and still span several
128-column tiles, many row batches and ragged tails.
"""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1911_04200_amd as jas  # noqa: E402
from paper_1911_04200_amd import jas as cabi  # noqa: E402


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).cuda()


def gpu_all_pairs(ids, off, U, batch_bits=0, dmin=0, upper=False, flags=0):
    db, st = jas.encode(dev(ids), dev(off), universe_bits=U, batch_bits=batch_bits, dense_min_degree=dmin)
    out = jas.gram(db, upper=upper, flags=flags)
    torch.cuda.synchronize()
    res = {k: v.cpu().numpy() for k, v in out.items()}
    db.close()
    return res, st


def assert_matches(res, ref, upper=False):
    n = ref["card"].size
    assert np.array_equal(res["card"], ref["card"]), "|X_i|"
    if upper:
        iu = np.triu_indices(n)
        want = {"B": ref["inter"][iu], "den": ref["union"][iu], "J": ref["J"][iu]}
    else:
        want = {"B": ref["inter"], "den": ref["union"], "J": ref["J"]}
    bad = np.argwhere(res["B"] != want["B"])
    assert bad.size == 0, f"B differs at {bad[:5].tolist()}"
    assert np.array_equal(res["den"], want["den"]), "unions differ"
    assert np.array_equal(res["J"].view(np.uint64), want["J"].view(np.uint64)), "J differs"


@pytest.fixture(scope="module")
def tiny():
    spec = synth.workload("tiny")
    ids, off = synth.generate(spec)
    return spec, ids, off, oracle.all_pairs(ids, off)


# (batch_bits, dense_min_degree, upper): one batch .. 2^20 batches, every row packed .. no row packed
VARIANTS = [(24, 0, False), (24, 0, True), (16, 2, False), (10, 3, False), (4, 5, True), (24, 1000, False),
            (12, 8, False), (20, 4, True)]


@pytest.mark.parametrize("bb,dmin,upper", VARIANTS)
@pytest.mark.parametrize("path", ["popcount", "mfma"])
def test_tiny_workload(tiny, bb, dmin, upper, path):
    spec, ids, off, ref = tiny
    flags = cabi.JAS_FORCE_POPCOUNT if path == "popcount" else cabi.JAS_FORCE_MFMA
    res, st = gpu_all_pairs(ids, off, spec.universe_bits, bb, dmin, upper, flags)
    assert_matches(res, ref, upper)
    assert st["n_ids"] == ids.size
    assert st["n_pairs"] == int(ref["card"].sum())


SCALED = {
    # structure of each workload at sizes the oracle finishes in seconds
    "paperlike": dict(n=300, size_scale=0.004, pool_scale=0.004),
    "precision": dict(n=257, size_scale=0.01, pool_scale=0.01),
    "batching": dict(n=400, size_scale=0.004, pool_scale=0.004),
    "serving_db": dict(n=200, size_scale=0.01, pool_scale=0.005),
}


@pytest.mark.parametrize("name", sorted(SCALED))
@pytest.mark.parametrize("dmin", [0, 2, 6])
def test_scaled_workloads(name, dmin):
    spec = synth.scaled(synth.workload(name), **SCALED[name])
    ids, off = synth.generate(spec)
    ref = oracle.all_pairs(ids, off)
    res, st = gpu_all_pairs(ids, off, spec.universe_bits, synth.BATCH_BITS[name], dmin, upper=(dmin == 6))
    assert_matches(res, ref, upper=(dmin == 6))
    assert st["n_packed_rows"] + st["n_list_rows"] == st["n_shared_rows"] > 0
    if dmin == 2:
        assert st["n_packed_rows"] == st["n_shared_rows"]
    elif dmin == 6:
        assert st["n_list_rows"] > 0
    else:
        assert st["dense_min_degree"] >= 2


# The paper's synthetic indicator matrices (Sec. V-A3): each entry 1 with
# probability p.  From rows of degree ~0.3 (row lists) to p = 1, where every
# set holds every row (B = m, J = 1); one batch of all rows and 16 batches.
BERNOULLI_CASES = [(1e-3, 16, 300), (1e-2, 14, 200), (0.1, 12, 150), (0.5, 10, 130), (1.0, 9, 70)]


@pytest.mark.parametrize("p,rows_log2,n", BERNOULLI_CASES)
@pytest.mark.parametrize("batches", [1, 16])
@pytest.mark.parametrize("path", ["auto", "popcount"])
def test_bernoulli_matrices(p, rows_log2, n, batches, path):
    spec = synth.bernoulli(p, rows_log2, n, seed=batches)
    ids, off = synth.generate(spec)
    ref = oracle.all_pairs(ids, off)
    flags = cabi.JAS_FORCE_POPCOUNT if path == "popcount" else 0
    bb = rows_log2 - (batches.bit_length() - 1)
    res, st = gpu_all_pairs(ids, off, rows_log2, bb, 0, flags=flags)
    assert_matches(res, ref)
    if p == 1.0:
        assert np.all(res["B"] == 1 << rows_log2) and np.all(res["J"] == 1.0)
        assert st["n_packed_rows"] == 1 << rows_log2


# Vertex similarity (Sec. II-F): the sets are the neighbourhoods of an R-MAT
# graph (hubs of degree ~ n/5 next to isolated vertices), A its adjacency.
@pytest.mark.parametrize("dmin", [0, 2, 1 << 20])
def test_graph_neighbourhood_similarity(dmin):
    ids, off = synth.rmat_graph(10, 16, seed=2)
    ref = oracle.all_pairs(ids, off)
    res, st = gpu_all_pairs(ids, off, 10, 10, dmin)
    assert_matches(res, ref)


def test_graph_link_prediction_queries():
    ids, off = synth.rmat_graph(12, 8, seed=3)
    n = off.size - 1
    db, _ = jas.encode(dev(ids), dev(off), universe_bits=12, batch_bits=12, keep_ids=True)
    # queries: neighbourhoods of some vertices, one with an edge added, and an empty set
    qs = [ids[int(off[v]):int(off[v + 1])] for v in (0, 17, 4095)]
    qs.append(np.union1d(qs[1], np.array([5], np.uint64)))
    qs.append(np.zeros(0, np.uint64))
    qo = np.zeros(len(qs) + 1, np.uint64)
    qo[1:] = np.cumsum([q.size for q in qs])
    qi = np.concatenate(qs).astype(np.uint64)
    out = jas.query(db, dev(qi), dev(qo))
    torch.cuda.synchronize()
    ref = oracle.cross(qi, qo, ids, off)
    assert np.array_equal(out["B"].cpu().numpy(), ref["inter"])
    assert np.array_equal(out["den"].cpu().numpy(), ref["union"])
    assert np.array_equal(out["J"].cpu().numpy().view(np.uint64), ref["J"].view(np.uint64))
    db.close()


def test_duplicates_and_empty_sets():
    spec = synth.scaled(synth.workload("tiny"), n=40, dup_rate=0.3)
    ids, off = synth.generate(spec)
    # make sets 3, 17 and 39 empty and set 20 a copy of set 5
    sets = [ids[int(off[i]):int(off[i + 1])] for i in range(40)]
    sets[3] = sets[17] = sets[39] = np.zeros(0, np.uint64)
    sets[20] = sets[5].copy()
    off2 = np.zeros(41, np.uint64)
    off2[1:] = np.cumsum([s.size for s in sets])
    ids2 = np.concatenate(sets)
    ref = oracle.all_pairs(ids2, off2)
    for dmin in (0, 4):
        res, _ = gpu_all_pairs(ids2, off2, 24, 14, dmin)
        assert_matches(res, ref)
    assert res["J"][3, 17] == 1.0 and res["J"][3, 5] == 0.0 and res["J"][5, 20] == 1.0


def encode_timed(ids, off, U, **kw):
    """Encode and Gram with the library's timers on; returns (result, stats, timer names)."""
    cabi.jas_timing_report()
    cabi.jas_timing_enable(True)
    try:
        res, st = gpu_all_pairs(ids, off, U, **kw)
    finally:
        names = set(cabi.jas_timing_report())
        cabi.jas_timing_enable(False)
    return res, st, names


def csr(sets):
    off = np.zeros(len(sets) + 1, np.uint64)
    off[1:] = np.cumsum([s.size for s in sets])
    return np.concatenate(sets).astype(np.uint64), off


@pytest.mark.parametrize("case", ["uniform", "uniform_u24", "narrow_ids", "one_hot_id"])
def test_bucket_ranges_and_fallback(case):
    """Keys are sorted on their top ID bits only and each range of whole buckets is
    finished in LDS (keys held in 32 bits relative to the range's first bucket when
    they fit, as with U=24 here, else in 64); a bucket too large for LDS (IDs crowded
    into a narrow range, or one ID repeated many times) must take the full sort and
    give the same result."""
    rng = np.random.default_rng({"uniform": 1, "uniform_u24": 4, "narrow_ids": 2, "one_hot_id": 3}[case])
    if case.startswith("uniform"):
        U, n = (36, 90) if case == "uniform" else (24, 90)
        core = rng.integers(0, 1 << U, 4000, dtype=np.uint64)
        sets = [np.concatenate([rng.choice(core, int(rng.integers(0, 3000))),
                                rng.integers(0, 1 << U, int(rng.integers(0, 3000)), dtype=np.uint64)])
                for _ in range(n)]
    elif case == "narrow_ids":
        U, n = 40, 60
        sets = [rng.choice(1 << 12, int(rng.integers(500, 2500)), replace=False).astype(np.uint64)
                for _ in range(n)]
    else:
        U, n = 32, 40
        sets = [rng.integers(0, 1 << 32, 2000, dtype=np.uint64) for _ in range(n)]
        sets[7] = np.concatenate([sets[7], np.full(20000, 12345, np.uint64)])
        sets[9] = np.concatenate([sets[9], np.array([12345], np.uint64)])
    ids, off = csr(sets)
    ref = oracle.all_pairs(ids, off)
    res, st, names = encode_timed(ids, off, U, dmin=0)
    assert_matches(res, ref)
    assert st["n_pairs"] == int(ref["card"].sum())
    if case == "uniform":  # relative keys need 37 bits
        assert "local_cls_wide" in names and "host:classify_fallback" not in names
    elif case == "uniform_u24":  # relative keys fit 32 bits
        assert "local_cls" in names and "local_cls_wide" not in names and "host:classify_fallback" not in names
    else:
        assert "host:classify_fallback" in names and "cls_write" in names


def max_range_len(ids, off, U, stride):
    """Longest range [first bucket edge >= c*stride, first edge >= (c+1)*stride)
    of the keys sorted by their top ID bits, as the encoder forms them."""
    n = off.size - 1
    N = ids.size
    sbits = max(1, int(np.ceil(np.log2(n))))
    # the encoder's choice of sorted top bits: buckets of about 512 keys, or
    # about 1024 when a range's keys still fit 32 bits (4 bits for its span)
    tb = min(U, int(np.ceil(np.log2(-(-N // 512)))))
    fewer = min(U, int(np.ceil(np.log2(-(-N // 1024)))))
    if fewer > 0 and (U - fewer) + 4 + sbits <= 32:
        tb = fewer
    bucket = np.sort(ids >> np.uint64(U - tb), kind="stable")
    edges = np.flatnonzero(np.diff(bucket)) + 1
    edges = np.concatenate([[0], edges, [N]])
    starts = [edges[np.searchsorted(edges, min(c * stride, N))] for c in range(-(-N // stride) + 1)]
    return int(np.max(np.diff(starts)))


@pytest.mark.parametrize("declined", [False, True])
def test_first_sort_pass_forms_the_keys(monkeypatch, declined):
    """With a global sort the digits are counted from the IDs alone and the
    sort's first pass forms the keys (id << s | sample) itself, the sample of
    each tile found once; when the single-pass sort declines (a digit total
    above its look-back counts, forced here by a lowered test limit), the keys
    are formed by a kernel of their own and sorted by reduce-then-scan
    passes.  Both give the oracle's result."""
    spec = synth.scaled(synth.workload("paperlike"), n=300, size_scale=0.004, pool_scale=0.004)
    ids, off = synth.generate(spec)
    # a few empty sets and many short ones, so that tiles hold several samples
    sets = [ids[int(off[i]):int(off[i + 1])] for i in range(spec.n)]
    sets[1] = sets[7] = np.zeros(0, np.uint64)
    sets[20:120] = [s[:37] for s in sets[20:120]]
    ids, off = csr(sets)
    if declined:
        monkeypatch.setenv("JAS_TEST_SCATTER_LIMIT", "100")
    ref = oracle.all_pairs(ids, off)
    res, st, names = encode_timed(ids, off, spec.universe_bits)
    assert_matches(res, ref)
    assert "count_digits" in names
    if declined:
        assert "build_keys" in names and "radix_scatter" in names and "radix_onesweep" not in names
    else:
        assert "build_keys" not in names and "radix_onesweep" in names


def test_concurrent_encodes_on_two_streams():
    """Two host threads encode different collections on their own streams at
    once (each encode puts its row-list pairs on the library's side stream
    while it packs on its own stream); both results are the oracle's."""
    import threading

    cases = []
    for k, name in enumerate(("paperlike", "precision")):
        spec = synth.scaled(synth.workload(name), **SCALED[name])
        ids, off = synth.generate(spec)
        cases.append((spec, ids, off, oracle.all_pairs(ids, off)))
    results, errors = [None, None], []

    def work(k):
        try:
            spec, ids, off, _ = cases[k]
            st = torch.cuda.Stream()
            with torch.cuda.stream(st):
                for _ in range(3):
                    db, _ = jas.encode(dev(ids), dev(off), universe_bits=spec.universe_bits, dense_min_degree=6)
                    out = jas.gram(db)
                    st.synchronize()
                    results[k] = {key: v.cpu().numpy() for key, v in out.items()}
                    db.close()
        except Exception as e:  # reported by the main thread
            errors.append(repr(e))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for k in range(2):
        assert_matches(results[k], cases[k][3])


@pytest.mark.parametrize("N", [6145, 8192, 8193, 16384, 16385, 24577])
def test_scatter_tile_edges(N):
    """Entry counts around the single-pass scatter's 8192-entry tiles (the
    global sort runs from 6145 entries on), with set boundaries exactly on,
    just before and just after tile boundaries and empty sets there, so that
    the first pass's per-tile samples (first and last entry of each tile, the
    starts inside it) meet every case."""
    rng = np.random.default_rng(N)
    U = 30
    cuts = sorted({0, N} | {c for t in range(8192, N, 8192) for c in (t - 1, t, t + 1) if 0 < c < N}
                  | {int(x) for x in rng.integers(1, N, 6)})
    sizes = [b - a for a, b in zip(cuts, cuts[1:])]
    sets = []
    for k, sz in enumerate(sizes):
        sets.append(rng.integers(0, 1 << U, sz, dtype=np.uint64))
        if k % 3 == 1:
            sets.append(np.zeros(0, np.uint64))  # an empty set at this boundary
    # shared IDs, so that rows of several samples exist
    pool = rng.integers(0, 1 << U, 64, dtype=np.uint64)
    for st in sets:
        if st.size:
            st[: min(st.size, 5)] = rng.choice(pool, min(st.size, 5))
    ids, off = csr(sets)
    assert ids.size == N
    ref = oracle.all_pairs(ids, off)
    res, st, names = encode_timed(ids, off, U)
    assert_matches(res, ref)
    assert "radix_onesweep" in names and "count_digits" in names


@pytest.mark.parametrize("N", [(1 << 24) - 1, 1 << 24, (1 << 24) + 1, (1 << 24) + 16383])
def test_scatter_large_tiles(N):
    """From 2^24 keys on the scatter's tiles hold 32 keys per thread (16384 in
    all, reordered in LDS in halves), or 24 in the pass that forms the keys:
    sizes just below that, exactly whole tiles, one key more and one key less
    than another tile, through jas_relabel (sorted keys: ranks against
    numpy's) and an encode of three sets (against the oracle)."""
    rng = np.random.default_rng(N)
    ids = rng.integers(0, 1 << 30, N, dtype=np.uint64)
    out = torch.empty(N, dtype=torch.int64, device="cuda")
    D, _ = cabi.jas_relabel(dev(ids), N, 30, None, out)
    distinct, rank = np.unique(ids, return_inverse=True)
    assert D == distinct.size
    assert np.array_equal(out.cpu().numpy(), rank)
    off = np.array([0, N // 3, N // 3 + 1, N], np.uint64)
    res, st = gpu_all_pairs(ids, off, 30, upper=True)
    assert_matches(res, oracle.all_pairs(ids, off), upper=True)


@pytest.mark.parametrize("rows", [380, 747, 748, 760])
def test_pair_sort_tile_sizes(rows):
    """17 M to 34 M pair words of 700 samples, two passes, below and above 2^25
    words, where tiles hold 64 words per thread."""
    rng = np.random.default_rng(rows)
    n, deg = 700, 300
    member = np.zeros((n, rows), np.int32)
    for r in range(rows):
        member[rng.choice(n, deg, replace=False), r] = 1
    ids = np.sort(rng.choice(1 << 24, rows, replace=False).astype(np.uint64))
    cids, off = csr([ids[m != 0] for m in member])
    db, st = jas.encode(dev(cids), dev(off), universe_bits=24, dense_min_degree=1000)
    out = jas.gram(db)
    pairs = torch.from_numpy(cabi.jas_db_read(db, cabi.JAS_DB_LIST_PAIRS).view(np.int32)).cuda()
    torch.cuda.synchronize()
    db.close()
    assert st["n_list_pairs"] == rows * deg * (deg - 1) // 2
    assert bool((pairs[1:] >> 16 >= pairs[:-1] >> 16).all())
    assert np.array_equal(out["B"].cpu().numpy(), member @ member.T)


@pytest.mark.parametrize("U", [9, 10, 14, 17, 18, 19, 26, 40, 55])
def test_lds_pass_widths(U):
    """The ID bits a range leaves for LDS are sorted in the fewest passes of at
    most 9 bits: universes whose ranges need one pass up to six, with keys in
    32 or 64 bits, repeats and sets of one ID."""
    rng = np.random.default_rng(U)
    n = 40
    sets = [rng.integers(0, 1 << U, int(rng.integers(1, 700)), dtype=np.uint64) for _ in range(n)]
    core = rng.integers(0, 1 << U, 90, dtype=np.uint64)
    sets = [np.concatenate([x, rng.choice(core, 30)]) for x in sets]
    sets[3] = core[:1].copy()
    ids, off = csr(sets)
    res, st = gpu_all_pairs(ids, off, U)
    assert_matches(res, oracle.all_pairs(ids, off))


def test_every_id_bit_sorted_globally():
    """A small universe and many entries (U = 8, 90,000 entries with repeats):
    the global sort covers every ID bit, so each bucket is one ID with its
    keys in sample order and the ranges (from 4096-key strides) are finished
    in LDS with no sort passes."""
    rng = np.random.default_rng(21)
    sets = [rng.integers(0, 256, 300, dtype=np.uint64) for _ in range(300)]
    sets[4] = np.zeros(0, np.uint64)
    ids, off = csr(sets)
    assert -(-ids.size // 512) > 128  # ceil(log2(N / 512)) >= U
    ref = oracle.all_pairs(ids, off)
    cabi.jas_timing_report()
    cabi.jas_timing_enable(True)
    try:
        res, st = gpu_all_pairs(ids, off, 8)
    finally:
        rep = cabi.jas_timing_report()
        cabi.jas_timing_enable(False)
    assert_matches(res, ref)
    assert rep["range_starts"][0] == 1 and "local_cls" in rep and "host:classify_fallback" not in rep


@pytest.mark.parametrize("U,per_cluster,tries", [(36, 26, 1), (36, 36, 2), (28, 36, 2)])
def test_longer_ranges_when_a_bucket_is_large(U, per_cluster, tries):
    """Clusters of IDs make buckets of 90 * per_cluster keys.  With 26 per
    cluster (~2300 keys) some 3072-key-stride range exceeds the 4096 keys the
    four-blocks-per-CU kernel holds, so the kernel for 6144-key ranges runs;
    with 36 (~3200 keys) some range exceeds even 6144 keys at that stride and
    the encoder tries 2048.  Either way the ranges are finished in LDS, with
    keys held in 64 bits there for U = 36 and in 32 for U = 28 (where the
    encoder sorts one top bit fewer, as the 32-bit keys still fit)."""
    rng = np.random.default_rng(11)
    n = 90
    sets = []
    for _ in range(n):
        parts = [rng.integers(0, 1 << U, 2000, dtype=np.uint64)]
        for k in range(8):
            parts.append((np.uint64(k << (U - 4)) + rng.choice(1 << 20, per_cluster, replace=False)).astype(np.uint64))
        sets.append(np.concatenate(parts))
    ids, off = csr(sets)
    if tries == 1:
        assert 6144 >= max_range_len(ids, off, U, 3072) > 4096
    else:
        assert max_range_len(ids, off, U, 3072) > 6144 >= max_range_len(ids, off, U, 2048) > 4096
    ref = oracle.all_pairs(ids, off)
    cabi.jas_timing_report()
    cabi.jas_timing_enable(True)
    try:
        res, st = gpu_all_pairs(ids, off, U)
    finally:
        rep = cabi.jas_timing_report()
        cabi.jas_timing_enable(False)
    assert_matches(res, ref)
    assert rep["range_starts"][0] == tries and "host:classify_fallback" not in rep
    assert ("local_cls_wide" if U == 36 else "local_cls") in rep


@pytest.mark.parametrize("case", ["uniform", "uniform_u24", "narrow_ids"])
def test_query_index_on_both_classification_paths(case):
    """With JAS_KEEP_IDS the distinct keys form the query index, whether the
    ranges were finished in LDS (keys held in 64 or in 32 bits there) or the
    full sort had to run."""
    rng = np.random.default_rng(7)
    if case.startswith("uniform"):
        U, n = (36, 70) if case == "uniform" else (24, 70)
        core = rng.integers(0, 1 << U, 3000, dtype=np.uint64)
        sets = [np.concatenate([rng.choice(core, int(rng.integers(0, 2500))),
                                rng.integers(0, 1 << U, int(rng.integers(0, 2500)), dtype=np.uint64)])
                for _ in range(n)]
    else:
        U, n = 40, 60
        sets = [rng.choice(1 << 12, int(rng.integers(500, 2500)), replace=False).astype(np.uint64)
                for _ in range(n)]
    ids, off = csr(sets)
    cabi.jas_timing_report()
    cabi.jas_timing_enable(True)
    try:
        db, st = jas.encode(dev(ids), dev(off), universe_bits=U, keep_ids=True)
        torch.cuda.synchronize()
    finally:
        names = set(cabi.jas_timing_report())
        cabi.jas_timing_enable(False)
    assert ("host:classify_fallback" in names) == (case == "narrow_ids")
    assert ("local_cls_wide" in names) == (case == "uniform")
    qsets = [sets[3], sets[11][::2], np.concatenate([sets[20][:50], np.array([(1 << U) - 1], np.uint64)])]
    qi, qo = csr(qsets)
    out = jas.query(db, dev(qi), dev(qo))
    torch.cuda.synchronize()
    res = {k: v.cpu().numpy() for k, v in out.items()}
    db.close()
    ref = oracle.cross(qi, qo, ids, off)
    assert np.array_equal(res["q_card"], ref["q_card"])
    assert np.array_equal(res["B"], ref["inter"])
    assert np.array_equal(res["J"].view(np.uint64), ref["J"].view(np.uint64))


def test_pack_long_and_short_rows():
    """Word rows whose 64 rows hold 64 samples or more on average are packed a
    row per wave, the others an entry per thread; both must give the oracle."""
    rng = np.random.default_rng(21)
    n = 200
    core = rng.choice(1 << 30, 700, replace=False).astype(np.uint64)  # rows of degree ~150-200
    sets = [np.concatenate([rng.choice(core, int(rng.integers(500, 700)), replace=False),
                            rng.integers(0, 1 << 30, int(rng.integers(0, 400)), dtype=np.uint64)])
            for _ in range(n)]
    ids, off = csr(sets)
    ref = oracle.all_pairs(ids, off)
    for dmin in (2, 100):
        res, st = gpu_all_pairs(ids, off, 30, 0, dmin)
        assert st["n_packed_rows"] > 0
        assert_matches(res, ref)


@pytest.mark.parametrize("n,dmin", [(300, 1000), (10300, 0)])
def test_row_lists_by_sample_and_by_row(n, dmin):
    """Rows kept as lists are summed sample by sample (their pairs sorted by the
    smaller sample, an LDS row of counters per sample, up to 10240 samples; long
    and short runs of one sample take different flushes) or, for more samples,
    pair by pair per row."""
    rng = np.random.default_rng(n)
    pool = rng.choice(1 << 20, 3000, replace=False).astype(np.uint64)
    sets = [np.unique(rng.choice(pool, int(rng.integers(0, 7)))) for _ in range(n)]
    sets[5] = pool[:40].copy()  # one sample in many rows
    sets[0] = pool[:2500].copy()  # a long run of pairs (0, b): counted without a touched list
    ids, off = csr(sets)
    ref = oracle.all_pairs(ids, off)
    res, st = gpu_all_pairs(ids, off, 20, 0, dmin)
    assert st["n_list_rows"] > 0
    assert_matches(res, ref)
    res, _ = gpu_all_pairs(ids, off, 20, 0, dmin, upper=True)
    assert_matches(res, ref, upper=True)


@pytest.mark.parametrize("rows,most", [(1, 200), (5, 60), (64, 40), (65, 200), (130, 120)])
def test_few_long_list_rows(rows, most):
    """Few list rows of many samples: several waves deal out the pairs of the same
    64 rows, and the pairs of one sample cross many short counting chunks."""
    rng = np.random.default_rng(rows)
    n = 200
    ids = np.sort(rng.choice(1 << 20, rows, replace=False).astype(np.uint64))
    deg = np.concatenate([[most], rng.integers(0, most + 1, rows - 1)]).astype(int)
    holders = [set(rng.choice(n, d, replace=False).tolist()) for d in deg]
    sets = [np.array([x for x, h in zip(ids, holders) if s in h], dtype=np.uint64) for s in range(n)]
    cids, off = csr(sets)
    ref = oracle.all_pairs(cids, off)
    res, st = gpu_all_pairs(cids, off, 20, 0, 1000)
    assert st["n_packed_rows"] == 0 and st["n_list_rows"] > 0
    assert_matches(res, ref)


@pytest.mark.parametrize("n", [1, 2, 3, 255, 256, 511, 512, 1023, 1024, 1025])
def test_upper_outputs_at_block_edges(n):
    rng = np.random.default_rng(n)
    sets = [np.unique(rng.integers(0, 2000, int(rng.integers(0, 12)))).astype(np.uint64) for _ in range(n)]
    ids, off = csr(sets)
    res, _ = gpu_all_pairs(ids, off, 11, upper=True)
    assert_matches(res, oracle.all_pairs(ids, off), upper=True)


@pytest.mark.parametrize("run", [3, 37, 38, 40, 1500])
def test_pair_runs_counted_directly_or_in_lds(run):
    """Runs of one smaller sample just below and above n / 8 pairs (300 samples),
    alone and among long ones, full and upper layout."""
    rng = np.random.default_rng(run)
    n, sets = 300, [[] for _ in range(300)]
    nid = 0
    for a in range(0, 290, 2):
        for k in range(run if a % 10 else 2 * run):
            b = int(rng.integers(a + 1, n)) if k % 3 else a + 1
            sets[a].append(nid)
            sets[b].append(nid)
            nid += 1
    ids, off = csr([np.array(s, dtype=np.uint64) for s in sets])
    ref = oracle.all_pairs(ids, off)
    for upper in (False, True):
        res, st = gpu_all_pairs(ids, off, 20, 0, 1000, upper=upper)
        assert st["n_list_pairs"] == nid
        assert_matches(res, ref, upper=upper)


@pytest.mark.parametrize("n,rows,deg", [(20, 64 * 4096 + 5, (2, 5)), (200, 64 * 4096 - 63, (2, 5)), (300, 700, (90, 102)),
                                        (1100, 700, (90, 102)), (1100, 130, (300, 700)), (10300, 200, (80, 110))])
@pytest.mark.parametrize("word_bits", [32, 64])
def test_packed_words_on_every_split(n, rows, deg, word_bits):
    """W word by word: a wave, 4 or 8 waves per row of it, entries dealt out one by
    one (up to 6144 in a row of W) or a packed row per wave, one and two column
    chunks, a last word row that is not full."""
    rng = np.random.default_rng(rows)
    ids = np.sort(rng.choice(1 << 24, rows, replace=False).astype(np.uint64))
    d = rng.integers(deg[0], deg[1] + 1, rows)
    r = np.repeat(np.arange(rows), d)
    smp = np.concatenate([rng.choice(n, k, replace=False) for k in d]) if rows < 1000 else None
    if smp is None:  # distinct by steps below n / deg
        k = np.arange(r.size) - np.repeat(np.cumsum(d) - d, d)
        smp = (np.repeat(rng.integers(0, n, rows), d) + k * (n // (deg[1] + 1))) % n
    order = np.lexsort((r, smp))
    off = np.zeros(n + 1, np.uint64)
    off[1:] = np.cumsum(np.bincount(smp, minlength=n))
    db, st = jas.encode(dev(ids[r[order]]), dev(off), universe_bits=24, dense_min_degree=2, word_bits=word_bits)
    W = cabi.jas_db_read(db, cabi.JAS_DB_WORDS)
    db.close()
    want = np.zeros((-(-rows // 64), -(-n // 128) * 128), np.uint64)
    np.bitwise_or.at(want, (r // 64, smp), np.uint64(1) << (r % 64).astype(np.uint64))
    assert st["n_packed_rows"] == rows and np.array_equal(W.reshape(want.shape), want)
    halves = want.view(np.uint32).reshape(want.shape[0], -1, 2) if word_bits == 32 else want[:, :, None]
    z = np.count_nonzero(halves, axis=1).astype(np.int64)
    assert st["nnz_words"] == z.sum() and st["word_pairs_F"] == (z * (z + 1) // 2).sum()


@pytest.mark.parametrize("deg", [(2, 2), (2, 9), (30, 60), (43, 44), (64, 65), (150, 200)])
def test_list_pairs_word_by_word(deg):
    """Pairs of list rows from two samples to more than one LDS stage of pairs
    (896) and from few to many rows per wave, with gaps between the rows (IDs of
    one sample): every stored pair word, ordered by the smaller sample."""
    rng = np.random.default_rng(deg[1])
    n, rows = 211, 700 if deg[1] < 100 else 150
    ids = rng.choice(1 << 24, rows, replace=False).astype(np.uint64)
    holders = [np.sort(rng.choice(n, int(rng.integers(deg[0], deg[1] + 1)), replace=False)) for _ in range(rows)]
    member = np.zeros((n, rows), bool)
    for r, h in enumerate(holders):
        member[h, r] = True
    sets = [np.unique(np.concatenate([ids[member[s]], rng.integers(1 << 24, 1 << 25, 20).astype(np.uint64)]))
            for s in range(n)]
    cids, off = csr(sets)
    db, st = jas.encode(dev(cids), dev(off), universe_bits=25, dense_min_degree=1000)
    pairs = cabi.jas_db_read(db, cabi.JAS_DB_LIST_PAIRS)
    out = jas.gram(db)
    torch.cuda.synchronize()
    db.close()
    assert_matches({k: v.cpu().numpy() for k, v in out.items()}, oracle.all_pairs(cids, off))
    uniq, inv = np.unique(cids, return_inverse=True)
    smp = np.repeat(np.arange(n), np.diff(off.astype(np.int64)))
    want = []
    for r in np.flatnonzero(np.bincount(inv) > 1):
        h = np.sort(smp[inv == r])
        i, j = np.triu_indices(h.size, 1)
        want.append((h[i] << 16 | h[j]).astype(np.uint32))
    want = np.concatenate(want)
    assert st["n_list_pairs"] == want.size
    assert np.all(np.diff((pairs >> np.uint32(16)).astype(np.int64)) >= 0)
    assert np.array_equal(np.sort(pairs), np.sort(want))


@pytest.mark.parametrize("rows", [1, 31, 33, 64, 65, 129])
@pytest.mark.parametrize("word_bits", [32, 64])
@pytest.mark.parametrize("dmin", [0, 2])
def test_single_batch_word_rows(rows, word_bits, dmin):
    """One batch packs its rows without the batch tables; sizes from the degree
    histogram (dmin 0) and from the device (dmin 2) give the same db as several
    batches do."""
    rng = np.random.default_rng(rows)
    pool = np.sort(rng.choice(1 << 20, rows, replace=False).astype(np.uint64))
    sets = [pool[rng.random(rows) < 0.9] for _ in range(140)]
    sets[0], sets[1] = pool, pool
    ids, off = csr(sets)
    ref = oracle.all_pairs(ids, off)
    for batch_bits in (0, 20, 14):
        db, st = jas.encode(dev(ids), dev(off), universe_bits=20, batch_bits=batch_bits, dense_min_degree=dmin,
                            word_bits=word_bits)
        out = jas.gram(db)
        torch.cuda.synchronize()
        db.close()
        assert_matches({k: v.cpu().numpy() for k, v in out.items()}, ref)
        assert st["n_packed_rows"] + st["n_list_rows"] == rows and st["n_rows"] == rows
        if batch_bits != 14 and st["n_packed_rows"]:
            assert st["n_batches"] == 1 and st["n_word_rows"] == -(-st["n_packed_rows"] // word_bits)


@pytest.mark.parametrize("N", [3000, 300000])
def test_id_outside_universe_among_many(N):
    """Checked after the sort has run on it, with and without global sort passes;
    the next call is not affected."""
    rng = np.random.default_rng(N)
    ids = rng.integers(0, 1 << 30, N).astype(np.uint64)
    off = np.array([0, N // 3, N], dtype=np.uint64)
    bad = ids.copy()
    bad[N // 2] = 1 << 40
    with pytest.raises(jas.JasError) as e:
        gpu_all_pairs(bad, off, 30)
    assert e.value.status == cabi.JAS_EINVAL
    res, _ = gpu_all_pairs(ids, off, 30)
    assert_matches(res, oracle.all_pairs(ids, off))


@pytest.mark.parametrize("n,N", [(300, 20000), (300, 2000000), (12, 2000000)])
def test_budgeted_sorts_clear_between_passes(n, N):
    """With a memory budget the sorts keep one pass's look-back words: several
    passes of keys and of pairs (n > 256) give the same result."""
    rng = np.random.default_rng(N)
    pool = rng.integers(0, 1 << 34, N // 20).astype(np.uint64)
    sets = [np.unique(np.concatenate([rng.choice(pool, N // n // 2), rng.integers(0, 1 << 34, N // n // 2).astype(np.uint64)]))
            for _ in range(n)]
    ids, off = csr(sets)
    outs = []
    for budget in (0, 1 << 34):
        db, st = jas.encode(dev(ids), dev(off), universe_bits=34, dense_min_degree=1000, hbm_budget_bytes=budget)
        outs.append((jas.gram(db, upper=True), st))
        torch.cuda.synchronize()
        db.close()
    for k, v in outs[0][0].items():
        assert torch.equal(v, outs[1][0][k]), k
    assert outs[0][1] == outs[1][1] and outs[0][1]["list_pairs"] > 0


@pytest.mark.parametrize("n", [3, 63, 64, 65, 128, 191, 449])
def test_full_outputs_mirror_across_tiles(n):
    """The full layout's lower triangle, union sizes and similarities come from the
    upper triangle tile by tile: every entry, at the edges of a tile."""
    rng = np.random.default_rng(n)
    sets = [np.unique(rng.integers(0, 300, int(rng.integers(0, 80)))).astype(np.uint64) for _ in range(n)]
    ids, off = csr(sets)
    res, _ = gpu_all_pairs(ids, off, 9)
    assert_matches(res, oracle.all_pairs(ids, off))


@pytest.mark.parametrize("n", [1, 2, 127, 128, 129, 255, 257])
@pytest.mark.parametrize("path", ["popcount", "mfma"])
def test_tile_edges(n, path):
    flags = cabi.JAS_FORCE_POPCOUNT if path == "popcount" else cabi.JAS_FORCE_MFMA
    rng = np.random.default_rng(n)
    core = rng.choice(1 << 20, 3000, replace=False).astype(np.uint64)
    sets = [np.concatenate([rng.choice(core, int(rng.integers(0, 2000)), replace=False),
                            rng.integers(0, 1 << 20, int(rng.integers(0, 300))).astype(np.uint64)])
            for _ in range(n)]
    off = np.zeros(n + 1, np.uint64)
    off[1:] = np.cumsum([s.size for s in sets])
    ids = np.concatenate(sets) if n else np.zeros(0, np.uint64)
    ref = oracle.all_pairs(ids, off)
    res, _ = gpu_all_pairs(ids, off, 20, 12, 0, flags=flags)
    assert_matches(res, ref)
    res, _ = gpu_all_pairs(ids, off, 20, 0, 0, upper=True, flags=flags)
    assert_matches(res, ref, upper=True)


def test_all_sets_empty():
    off = np.zeros(6, np.uint64)
    ids = np.zeros(0, np.uint64)
    db, st = jas.encode(dev(np.zeros(1, np.uint64))[:0], dev(off), universe_bits=16)
    out = jas.gram(db)
    torch.cuda.synchronize()
    assert st["n_pairs"] == 0
    assert np.all(out["B"].cpu().numpy() == 0)
    assert np.all(out["J"].cpu().numpy() == 1.0)
    assert np.all(out["den"].cpu().numpy() == 0)
    db.close()
    ref = oracle.all_pairs(ids, off)
    assert np.all(ref["J"] == 1.0)


def test_zero_sets():
    db, st = jas.encode(dev(np.zeros(1, np.uint64))[:0], dev(np.zeros(1, np.uint64)), universe_bits=16)
    assert db.n == 0
    out = jas.gram(db)
    assert out["B"].numel() == 0
    db.close()


@pytest.mark.parametrize("U,n", [(63, 2), (62, 3), (1, 3), (2, 5), (40, 1024)])
def test_universe_extremes(U, n):
    rng = np.random.default_rng(U * 1000 + n)
    top = (1 << U) - 1
    base = np.array([top, top - 1, 0, top // 2, top // 3], dtype=np.uint64)[: min(5, 1 << U)]
    sets = [np.unique(np.concatenate([rng.choice(base, int(rng.integers(0, base.size + 1))),
                                      rng.integers(0, top, 3, dtype=np.uint64, endpoint=True)]))
            for _ in range(n)]
    off = np.zeros(n + 1, np.uint64)
    off[1:] = np.cumsum([s.size for s in sets])
    ids = np.concatenate(sets)
    ref = oracle.all_pairs(ids, off)
    res, _ = gpu_all_pairs(ids, off, U, 0, 0)
    assert_matches(res, ref)


def test_id_outside_universe_is_rejected():
    ids = np.array([1, 2, 1 << 20], dtype=np.uint64)
    with pytest.raises(jas.JasError) as e:
        jas.encode(dev(ids), dev(np.array([0, 3], np.uint64)), universe_bits=20)
    assert e.value.status == cabi.JAS_EINVAL


@pytest.mark.parametrize("dmin", [4, 1000])
def test_budgets_around_the_smallest_that_is_enough(dmin):
    """Budgets from enough down to far too small, on the null stream: refused ones
    leave nothing behind that the encode after them could meet."""
    rng = np.random.default_rng(dmin)
    pool = rng.integers(0, 1 << 30, 10000, dtype=np.uint64)
    sets = [np.concatenate([rng.choice(pool, 1500), rng.integers(0, 1 << 30, 1500, dtype=np.uint64)]) for _ in range(64)]
    ids, off = csr(sets)
    d, o = dev(ids), dev(off)
    ref = oracle.all_pairs(ids, off)
    enough, refused = 1 << 25, 0
    for budget in [int((1 << 25) * 0.93 ** k) for k in range(60)]:
        try:
            db, _ = jas.encode(d, o, universe_bits=30, dense_min_degree=dmin, hbm_budget_bytes=budget)
            db.close()
            assert not refused, "a smaller budget was enough"
            enough = budget
        except jas.JasError as e:
            assert e.status == cabi.JAS_ENOMEM
            refused += 1
            if refused % 8 == 1:
                db, _ = jas.encode(d, o, universe_bits=30, dense_min_degree=dmin, hbm_budget_bytes=enough)
                assert np.array_equal(jas.gram(db)["B"].cpu().numpy(), ref["inter"])
                db.close()
    assert refused > 20


def test_budget_is_enforced():
    spec = synth.workload("tiny")
    ids, off = synth.generate(spec)
    with pytest.raises(jas.JasError) as e:
        jas.encode(dev(ids), dev(off), universe_bits=24, hbm_budget_bytes=1 << 20)
    assert e.value.status == cabi.JAS_ENOMEM


def test_host_pointers_match_device_path(tiny):
    spec, ids, off, ref = tiny
    opts = cabi.jas_encode_opts(24, 16, 0, cabi.JAS_HOST_PTRS, 0)
    db, st = cabi.jas_encode(ids, off, 32, opts)
    B = np.empty((32, 32), np.int32)
    card = np.empty(32, np.int64)
    den = np.empty((32, 32), np.int64)
    J = np.empty((32, 32), np.float64)
    cabi.jas_gram(db, cabi.JAS_HOST_PTRS, None, B, card, den, J)
    db.close()
    assert_matches({"B": B, "card": card, "den": den, "J": J}, ref)


@pytest.mark.parametrize("name", ["precision", "paperlike"])
def test_mfma_equals_popcount_on_dense_tiles(name):
    spec = synth.scaled(synth.workload(name), n=384, size_scale=0.01, pool_scale=0.01)
    ids, off = synth.generate(spec)
    db, st = jas.encode(dev(ids), dev(off), universe_bits=spec.universe_bits, batch_bits=synth.BATCH_BITS[name])
    a = jas.gram(db, flags=cabi.JAS_FORCE_POPCOUNT)
    b = jas.gram(db, flags=cabi.JAS_FORCE_MFMA)
    c = jas.gram(db)
    torch.cuda.synchronize()
    assert st["n_word_rows"] > 0
    assert torch.equal(a["B"], b["B"]) and torch.equal(a["B"], c["B"])
    assert torch.equal(a["J"], b["J"])
    db.close()
    ref = oracle.all_pairs(ids, off)
    assert_matches({k: v.cpu().numpy() for k, v in b.items()}, ref)


def test_gram_autotuner_keeps_results_exact():
    spec = synth.scaled(synth.workload("precision"), n=300, size_scale=0.01, pool_scale=0.01)
    ids, off = synth.generate(spec)
    db, st = jas.encode(dev(ids), dev(off), universe_bits=spec.universe_bits, dense_min_degree=2)
    assert st["n_word_rows"] > 0
    plain = jas.gram(db, upper=True)
    tuned = jas.gram(db, upper=True, flags=cabi.JAS_TUNE)    # times every tile variant, then runs the fastest
    again = jas.gram(db, upper=True)                          # the kept choice
    torch.cuda.synchronize()
    for k in ("B", "den", "J", "card"):
        assert torch.equal(plain[k], tuned[k]) and torch.equal(plain[k], again[k]), k
    db.close()
    ref = oracle.all_pairs(ids, off)
    assert_matches({k: v.cpu().numpy() for k, v in tuned.items()}, ref, upper=True)


@pytest.mark.parametrize("n", [130, 300, 513])
def test_every_mfma_tile_variant_is_exact(n):
    """Each MFMA tile variant (128 x 128 and 256 x 256 tiles, word rows per
    step, K split) gives the oracle's B, C and J, with ragged column tiles."""
    spec = synth.scaled(synth.workload("precision"), n=n, size_scale=0.01, pool_scale=0.01)
    ids, off = synth.generate(spec)
    db, st = jas.encode(dev(ids), dev(off), universe_bits=spec.universe_bits, dense_min_degree=2)
    assert st["n_word_rows"] > 0
    ref = oracle.all_pairs(ids, off)
    nv = cabi.jas_gram_variants()
    assert nv >= 2
    for v in range(nv):
        for upper in (False, True):
            out = jas.gram(db, upper=upper, flags=cabi.JAS_GRAM_VARIANT(v))
            torch.cuda.synchronize()
            assert_matches({k: x.cpu().numpy() for k, x in out.items()}, ref, upper=upper)
    with pytest.raises(cabi.JasError):
        jas.gram(db, flags=cabi.JAS_GRAM_VARIANT(nv))
    db.close()


@pytest.mark.parametrize("n,rows", [(2, 1), (63, 64), (65, 65), (128, 129), (129, 1000), (192, 1025), (257, 2100)])
def test_fp4_row_pairs_and_diagonal_tiles(n, rows):
    """The fp4 kernel reads word rows in pairs, several pairs ahead, and skips
    the half of a diagonal tile below the diagonal: word row counts of 1, 2,
    3, odd and one past a block's 16, columns around 64, 128 and 256."""
    rng = np.random.default_rng(100 * n + rows)
    every = rng.choice(1 << 20, rows, replace=False).astype(np.uint64)
    A = rng.random((rows, n)) < 0.4
    A[:, :2] = True  # every row is shared, so the word rows are ceil(rows / 64)
    ids, off = csr([every[A[:, j]] for j in range(n)])
    ref = oracle.all_pairs(ids, off)
    db, st = jas.encode(dev(ids), dev(off), universe_bits=20, dense_min_degree=2)
    assert st["n_word_rows"] == -(-rows // 64)
    for upper in (False, True):
        out = jas.gram(db, upper=upper, flags=cabi.JAS_FORCE_MFMA)
        torch.cuda.synchronize()
        assert_matches({k: x.cpu().numpy() for k, x in out.items()}, ref, upper=upper)
    db.close()


@pytest.mark.parametrize("word_rows", [1008, 1024, 1041])
def test_fp4_blocks_of_few_and_many_word_rows(word_rows):
    """Blocks of fewer than 1024 word rows add 32 columns in a row, longer ones
    every other column.  With 276 tile pairs, the last tile ragged, the fixed
    splits give blocks of all the rows, of half of them and shorter ones."""
    n, degree, rows = 2900, 6, 64 * word_rows
    rng = np.random.default_rng(word_rows)
    cols = np.sort(rng.integers(0, n - degree, (rows, degree)), axis=1) + np.arange(degree)  # distinct
    every = rng.choice(1 << 20, rows, replace=False).astype(np.uint64)
    order = np.lexsort((np.repeat(every, degree), cols.ravel()))
    ids = np.repeat(every, degree)[order]
    off = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(cols.ravel(), minlength=n), out=off[1:])
    want = np.zeros(n * n, np.int64)
    for a in range(degree):
        for b in range(a + 1, degree):
            want += np.bincount(cols[:, a] * n + cols[:, b], minlength=n * n)
    upper = np.triu_indices(n)
    want = want.reshape(n, n)
    np.fill_diagonal(want, np.diff(off))
    db, st = jas.encode(dev(ids), dev(off), universe_bits=20, dense_min_degree=2)
    assert st["n_word_rows"] == word_rows
    for flags in [cabi.JAS_FORCE_MFMA] + [cabi.JAS_GRAM_VARIANT(v) for v in range(cabi.jas_gram_variants())]:
        B = jas.gram(db, upper=True, flags=flags)["B"].cpu().numpy()
        assert np.array_equal(B, want[upper]), flags
    db.close()


def test_repeat_runs_are_identical():
    spec = synth.scaled(synth.workload("precision"), n=300, size_scale=0.01, pool_scale=0.01)
    ids, off = synth.generate(spec)
    db, _ = jas.encode(dev(ids), dev(off), universe_bits=spec.universe_bits, dense_min_degree=4)
    a = jas.gram(db)["B"].cpu().numpy()
    b = jas.gram(db)["B"].cpu().numpy()
    c = jas.gram(db, flags=cabi.JAS_FORCE_POPCOUNT)["B"].cpu().numpy()
    assert np.array_equal(a, c)
    db.close()
    assert np.array_equal(a, b)


# --- query path -------------------------------------------------------------
@pytest.mark.parametrize("query_only", [False, True])
def test_query_matches_oracle(query_only):
    """A query against every database set; with JAS_QUERY_ONLY the db holds only the
    query index (less device memory, the same answers) and jas_gram refuses it."""
    spec = synth.scaled(synth.workload("serving_db"), n=150, size_scale=0.01, pool_scale=0.005)
    ids, off = synth.generate(spec)
    db, st = jas.encode(dev(ids), dev(off), universe_bits=spec.universe_bits, batch_bits=26, keep_ids=True,
                        dense_min_degree=5, query_only=query_only)
    if query_only:
        full, st_full = jas.encode(dev(ids), dev(off), universe_bits=spec.universe_bits, batch_bits=26,
                                   keep_ids=True, dense_min_degree=5)
        assert st["device_bytes"] < st_full["device_bytes"]
        assert st["n_packed_rows"] == 0 and st["n_list_rows"] == 0 and st["n_pairs"] == st_full["n_pairs"]
        full.close()
        with pytest.raises(cabi.JasError) as e:
            jas.gram(db)
        assert e.value.status == cabi.JAS_EINVAL
    qspec = synth.scaled(synth.query_spec(spec, 0, 9), size_scale=0.01)
    qi, qo = synth.generate(qspec)
    # add DB sets 0 and 7, an empty set, and a set with repeats and IDs absent from the DB
    extra = [ids[int(off[0]):int(off[1])], ids[int(off[7]):int(off[8])], np.zeros(0, np.uint64),
             np.array([5, 5, 5, (1 << 36) - 1, 123456789], np.uint64)]
    sets = [qi[int(qo[i]):int(qo[i + 1])] for i in range(9)] + extra
    qoff = np.zeros(len(sets) + 1, np.uint64)
    qoff[1:] = np.cumsum([s.size for s in sets])
    qids = np.concatenate(sets)
    ref = oracle.cross(qids, qoff, ids, off)
    out = jas.query(db, dev(qids), dev(qoff))
    torch.cuda.synchronize()
    res = {k: v.cpu().numpy() for k, v in out.items()}
    db.close()
    assert np.array_equal(res["q_card"], ref["q_card"])
    assert np.array_equal(res["B"], ref["inter"])
    assert np.array_equal(res["den"], ref["union"])
    assert np.array_equal(res["J"].view(np.uint64), ref["J"].view(np.uint64))


def check_query(db, qsets, ids, off, flags=0):
    qi, qo = csr(qsets)
    out = jas.query(db, dev(qi), dev(qo), flags=flags)
    torch.cuda.synchronize()
    res = {k: v.cpu().numpy() for k, v in out.items()}
    ref = oracle.cross(qi, qo, ids, off)
    assert np.array_equal(res["q_card"], ref["q_card"])
    assert np.array_equal(res["B"], ref["inter"]) and np.array_equal(res["den"], ref["union"])
    assert np.array_equal(res["J"].view(np.uint64), ref["J"].view(np.uint64))


@pytest.mark.parametrize("sizes", [[1], [0, 15, 16, 17], [511, 512, 513, 0], [4095, 4097, 1], [32768], [32768, 32769],
                                   [20000] * 60])
def test_query_set_sizes_on_both_paths(sizes):
    """Requests whose sets have at most 32768 IDs and 2^20 in all are made sets
    through LDS hash tables, the others by a sort: sizes around a block's share
    and both limits, with repeats inside a set and IDs the database lacks."""
    rng = np.random.default_rng(sum(sizes))
    pool = rng.integers(0, 1 << 36, 60000, dtype=np.uint64)
    sets = [rng.choice(pool, 3000) for _ in range(60)]
    ids, off = csr(sets)
    db, _ = jas.encode(dev(ids), dev(off), universe_bits=36, keep_ids=True)
    q = [np.concatenate([rng.choice(pool, z // 2), rng.integers(0, 1 << 36, z - z // 2, dtype=np.uint64)]) for z in sizes]
    check_query(db, q, ids, off)
    for k, z in enumerate(sizes):  # one ID throughout, and IDs in a row
        q[k] = np.full(z, pool[k], np.uint64) if k % 2 else np.arange(z, dtype=np.uint64) << np.uint64(20)
    check_query(db, q, ids, off)
    if max(sizes) > 0:  # an ID outside the universe is refused on either path
        q[int(np.argmax(sizes))][-1] = 1 << 36
        with pytest.raises(jas.JasError) as e:
            check_query(db, q, ids, off)
        assert e.value.status == cabi.JAS_EINVAL
    db.close()


@pytest.mark.parametrize("sizes", [[32768] + [1] * 4000, [0] * 3 + [20000] + [0] * 3000 + [17, 16, 15],
                                   [0] * 50 + [40000] + [3, 0] * 1000])
def test_query_sets_of_unequal_sizes(sizes):
    """One large set among many small or empty ones, through the tables and through the sort."""
    rng = np.random.default_rng(len(sizes))
    pool = rng.integers(0, 1 << 30, 30000, dtype=np.uint64)
    ids, off = csr([rng.choice(pool, 2000) for _ in range(20)])
    db, _ = jas.encode(dev(ids), dev(off), universe_bits=30, keep_ids=True)
    check_query(db, [rng.choice(pool, z) for z in sizes], ids, off)
    db.close()


@pytest.mark.parametrize("set_ids", [100, 40000])
def test_query_of_more_sets_than_a_launch_has_blocks(set_ids):
    """2^22 + 5 sets, all but two empty: slices and sets past the grid's size are taken in turn."""
    rng = np.random.default_rng(set_ids)
    pool = rng.integers(0, 1 << 30, 30000, dtype=np.uint64)
    ids, off = csr([rng.choice(pool, 2000) for _ in range(3)])
    db, _ = jas.encode(dev(ids), dev(off), universe_bits=30, keep_ids=True)
    nq, at = (1 << 22) + 5, (12345, (1 << 22) + 3)
    sizes = np.zeros(nq, np.int64)
    sizes[list(at)] = set_ids, 7
    qo = np.zeros(nq + 1, np.uint64)
    qo[1:] = np.cumsum(sizes)
    qi = rng.choice(pool, int(qo[-1]))
    out = jas.query(db, dev(qi), dev(qo))
    torch.cuda.synchronize()
    B, card = out["B"].cpu().numpy(), out["q_card"].cpu().numpy()
    db.close()
    ref = oracle.cross(qi, np.array([0, set_ids, set_ids + 7], np.uint64), ids, off)
    assert np.array_equal(B[list(at)], ref["inter"]) and np.array_equal(card[list(at)], ref["q_card"])
    assert B.any(axis=1).sum() <= 2 and np.count_nonzero(card) == 2


@pytest.mark.parametrize("n", [10300, 16384, 16385])
def test_query_rows_of_more_than_64_kb_of_lds(n):
    """From about 10300 samples on a block's row of counters and its table pass 64 KB
    of LDS; past 16384 samples the counters are in memory."""
    rng = np.random.default_rng(n)
    pool = rng.integers(0, 1 << 24, 4000, dtype=np.uint64)
    ids, off = csr([rng.choice(pool, 5) for _ in range(n)])
    db, _ = jas.encode(dev(ids), dev(off), universe_bits=24, keep_ids=True, query_only=True)
    check_query(db, [rng.choice(pool, 700), pool, pool[:0], pool[-1:]], ids, off)
    check_query(db, [rng.choice(pool, 33000), pool[:9]], ids, off)
    db.close()


@pytest.mark.parametrize("n", [513, 3000, 20000])
def test_query_ids_most_samples_hold(n):
    """A database ID in every one of n samples: beyond the 512 entries a thread
    reads itself, the block reads the run (with the row of B in LDS up to 16384
    samples, else in memory), next to IDs of other lengths and of none."""
    rng = np.random.default_rng(n)
    hubs = np.array([7, 1 << 19, (1 << 20) - 1], np.uint64)  # the universe's last ID ends the key array
    sets = [np.concatenate([hubs[: 1 + i % 3] if i else hubs, rng.integers(8, 1 << 18, 5, dtype=np.uint64)])
            for i in range(n)]
    ids, off = csr(sets)
    db, _ = jas.encode(dev(ids), dev(off), universe_bits=20, keep_ids=True, query_only=True)
    check_query(db, [hubs, np.array([7, 9, 7], np.uint64), np.zeros(0, np.uint64),
                     rng.integers(0, 1 << 20, 40000, dtype=np.uint64)], ids, off)
    check_query(db, [hubs[::-1].copy(), sets[5]], ids, off)
    db.close()


def test_query_row_equals_gram_row():
    spec = synth.scaled(synth.workload("batching"), n=120, size_scale=0.004, pool_scale=0.004)
    ids, off = synth.generate(spec)
    db, _ = jas.encode(dev(ids), dev(off), universe_bits=spec.universe_bits, batch_bits=26, keep_ids=True)
    g = jas.gram(db)
    rows = [3, 50, 119]
    qs = [ids[int(off[i]):int(off[i + 1])] for i in rows]
    qoff = np.zeros(4, np.uint64)
    qoff[1:] = np.cumsum([s.size for s in qs])
    out = jas.query(db, dev(np.concatenate(qs)), dev(qoff))
    torch.cuda.synchronize()
    assert torch.equal(out["B"], g["B"][rows])
    assert torch.equal(out["J"], g["J"][rows])
    db.close()


def test_query_requires_index_and_rejects_bad_ids():
    spec = synth.workload("tiny")
    ids, off = synth.generate(spec)
    db, _ = jas.encode(dev(ids), dev(off), universe_bits=24)
    with pytest.raises(jas.JasError):
        jas.query(db, dev(ids[:10]), dev(np.array([0, 10], np.uint64)))
    db.close()
    db, _ = jas.encode(dev(ids), dev(off), universe_bits=24, keep_ids=True)
    with pytest.raises(jas.JasError) as e:
        jas.query(db, dev(np.array([1 << 24], np.uint64)), dev(np.array([0, 1], np.uint64)))
    assert e.value.status == cabi.JAS_EINVAL
    db.close()


def test_gram_captured_in_a_graph_replays_exactly():
    spec = synth.scaled(synth.workload("paperlike"), n=200, size_scale=0.004, pool_scale=0.004)
    ids, off = synth.generate(spec)
    db, st = jas.encode(dev(ids), dev(off), universe_bits=spec.universe_bits, batch_bits=26, dense_min_degree=4)
    assert st["n_list_rows"] > 0 and st["n_packed_rows"] > 0
    eager = jas.gram(db)
    torch.cuda.synchronize()
    n = spec.n
    B = torch.full((n, n), -7, dtype=torch.int32, device="cuda")
    card = torch.empty(n, dtype=torch.int64, device="cuda")
    den = torch.empty((n, n), dtype=torch.int64, device="cuda")
    J = torch.empty((n, n), dtype=torch.float64, device="cuda")
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        cabi.jas_gram(db, 0, side, B, card, den, J)  # warm the path outside the capture
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        cabi.jas_gram(db, 0, torch.cuda.current_stream(), B, card, den, J)
    for rep in range(3):
        B.fill_(-1)
        J.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(B, eager["B"]), f"replay {rep}"
        assert torch.equal(J, eager["J"]) and torch.equal(den, eager["den"]) and torch.equal(card, eager["card"])
        _ = (eager["B"].float() * 2).sum().item()  # eager work between replays
    db.close()
