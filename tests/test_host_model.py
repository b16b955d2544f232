"""The library's own host and device code run on the CPU under AddressSanitizer
(tests/host_model): which memory its kernels touch, when its buffers are given
back, and what is still running when a call returns.  Every buffer has exactly
the size asked for and holds 0xFF bytes at first, and with lazy streams every
kernel runs as late as the host's waits allow.  No GPU.
"""
import os
import subprocess
import sys

import pytest

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "host_model"))
import model  # noqa: E402

PRELUDE = r"""
import sys
import numpy as np
import model
jas, lib = model.attach(sys.argv[1])

def collection(n, total, universe_bits, share, seed=3):
    # about total IDs in n sets, part of each from one pool of a twentieth as many
    rng = np.random.default_rng(seed)
    pool = rng.integers(0, 1 << universe_bits, max(8, total // 20))
    sets = []
    for _ in range(n):
        k = max(1, int(total / n * rng.uniform(.5, 1.5)))
        m = int(k * share)
        sets.append(np.concatenate([rng.choice(pool, m), rng.integers(0, 1 << universe_bits, k - m)]))
    off = np.zeros(n + 1, np.uint64)
    off[1:] = np.cumsum([s.size for s in sets])
    return np.concatenate(sets).astype(np.uint64), off

def intersections(ids, off):
    n = off.size - 1
    smp = np.repeat(np.arange(n), np.diff(off).astype(np.int64))
    pairs = np.unique(np.stack([ids.astype(np.int64), smp]), axis=1)
    row = np.unique(pairs[0], return_inverse=True)[1]
    A = np.zeros((int(row.max()) + 1 if row.size else 1, n), np.float32)
    A[row, pairs[1]] = 1
    return (A.T @ A).astype(np.int32)

def gram(db, n):
    B = np.zeros((n, n), np.int32)
    jas.jas_gram(db, jas.JAS_FORCE_POPCOUNT, None, B)
    lib.model_drain()
    return B
"""


@pytest.fixture(scope="module")
def library(tmp_path_factory):
    if model.compiler() is None:
        pytest.skip("clang's AddressSanitizer runtime is not installed")
    return model.build(str(tmp_path_factory.mktemp("host_model")))


def run(library, script, *args):
    lib, rt = library
    r = subprocess.run([sys.executable, "-c", PRELUDE + script + "\nprint('DONE')", lib, *map(str, args)],
                       env=model.environment(rt), capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.endswith("DONE\n"), (r.stdout[-2000:], r.stderr[:6000])
    return r.stdout


REFUSED = r"""
n, total, ubits, share, batch, dmin, flags, wb = [int(a) for a in sys.argv[2:5]] + [float(sys.argv[5])] + [int(a) for a in sys.argv[6:10]]
ids, off = collection(n, total, ubits, share)
want = intersections(ids, off)
opts = jas.jas_encode_opts(ubits, batch, dmin, flags, 0, wb)
refused = []
lib.model_lazy(1)
for k in [-1] + list(range(lib.model_allocations() + 1000)):
    lib.model_fail_at(k)
    try:
        db, _ = jas.jas_encode(ids, off, n, opts)
    except jas.JasError as e:
        assert e.status == jas.JAS_ENOMEM and "refused" in e.message, str(e)
        refused.append((k, e.message, lib.model_pending()))
        lib.model_drain()  # (what is still enqueued uses freed buffers, if any were given back too early)
        continue
    lib.model_fail_at(-1)
    assert np.array_equal(gram(db, n), want)
    db.close()
    if k >= 0:
        break  # no allocation is left to refuse
assert k > 15
lib.model_drain()
assert lib.model_live() == 0
"""
NOTHING_LEFT = "assert not [r for r in refused if r[2]], refused"


@pytest.mark.parametrize("dmin", [5, 1000])
def test_encode_refused_at_every_allocation(library, dmin):
    """Every allocation of an encode on the null stream refused in turn: work of
    the library's own stream is waited for before its buffers are given back."""
    run(library, REFUSED, 64, 16000, 30, 0.5, 0, dmin, 0, 64)


def test_query_keys_of_a_refused_encode(library):
    """The same with a query index: its keys are still being written when a later
    allocation is refused, so they are not idle when they go back."""
    run(library, REFUSED, 64, 16000, 30, 0.5, 0, 1000, 2, 64)


def test_nothing_runs_after_a_refused_encode(library):
    """Once an encode is back with an error, no kernel of it is left to read the
    caller's IDs."""
    run(library, REFUSED + NOTHING_LEFT, 64, 16000, 30, 0.5, 24, 6, 2, 32)


CALLS_REFUSED = r"""
rng = np.random.default_rng(5)
ids, off = collection(40, 20000, 30, 0.5)
db, _ = jas.jas_encode(ids, off, 40, jas.jas_encode_opts(30, 0, 0, jas.JAS_KEEP_IDS | jas.JAS_QUERY_ONLY, 0, 64))
lib.model_drain()
q = np.concatenate([rng.choice(ids, 40000), rng.integers(0, 1 << 30, 1000).astype(np.uint64)])  # one set, sorted
qoff = np.array([0, q.size], np.uint64)
long_ids = rng.integers(0, 1 << 62, 30000).astype(np.uint64)
crowded = rng.integers(0, 1 << 14, 30000).astype(np.uint64)

def query(flags):
    B, card = np.zeros(40, np.int32), np.zeros(1, np.int64)
    jas.jas_query(db, q, qoff, 1, flags, None, B, card)
    return card[0] == np.unique(q).size and B[7] == np.intersect1d(q, ids[int(off[7]):int(off[8])]).size

def relabel(x):
    out = np.zeros(x.size, np.uint64)
    u, inv = np.unique(x, return_inverse=True)
    return jas.jas_relabel(x, x.size, 62, None, out)[0] == u.size and np.array_equal(out, inv)

lib.model_lazy(1)
for call in (lambda: query(0), lambda: query(jas.JAS_HOST_PTRS), lambda: relabel(long_ids), lambda: relabel(crowded)):
    for k in range(1000):
        lib.model_fail_at(k)
        try:
            ok = call()
        except jas.JasError as e:
            assert e.status == jas.JAS_ENOMEM and lib.model_pending() == 0, (k, str(e), lib.model_pending())
            continue
        assert ok and k > 5
        break
"""


def test_nothing_runs_after_a_refused_query_or_relabelling(library):
    """Nor of a query (which writes the caller's B first) or a relabelling."""
    run(library, CALLS_REFUSED)


REFUSED_BY_A_PLAN = r"""
n, ubits = 40, 30
ids, off = collection(n, 16000, ubits, 0.5)
plan = jas.jas_plan_create(ids, off, n, jas.jas_encode_opts(ubits, 0, 4, 0, 0, 64), 0.1)
want = intersections(ids, off)
for bad in (False, True, False):
    x = ids.copy()
    if bad:
        x[100] |= np.uint64(1 << ubits)
    jas.jas_plan_encode(plan, x, off)
    B = gram(plan.db, n)
    assert np.array_equal(B, want) != bad
    if bad:
        assert not B[~np.eye(n, dtype=bool)].any()
    try:
        jas.jas_plan_check(plan)
        assert not bad
    except jas.JasError as e:
        assert bad and e.status == jas.JAS_EINVAL, str(e)
"""


def test_a_plan_classifies_nothing_after_a_failed_sort(library):
    """Keys that were not all placed (an ID >= 2^U, or a look-back that gave up)
    are not classified: no rows, the error as before, and the next collection is
    encoded as ever."""
    run(library, REFUSED_BY_A_PLAN)


SAME_PAIRS = r"""
n, upper = int(sys.argv[2]), int(sys.argv[3])
rng = np.random.default_rng(n)
# two samples share nearly all list rows, a few others some
sets = [rng.integers(1 << 20, 1 << 21, 3) for _ in range(n)]
a, b = n // 3, n // 2
rows = rng.choice(1 << 20, 6000, replace=False)
for s in (a, b):
    sets[s] = np.concatenate([sets[s], rows])
for s in rng.choice(n, 40, replace=False):
    sets[s] = np.concatenate([sets[s], rows[:2]])
off = np.zeros(n + 1, np.uint64)
off[1:] = np.cumsum([s.size for s in sets])
ids = np.concatenate(sets).astype(np.uint64)
db, st = jas.jas_encode(ids, off, n, jas.jas_encode_opts(21, 0, 1000, 0, 0, 64))
B = np.zeros(n * (n + 1) // 2 if upper else n * n, np.int32)
before = lib.model_atomic_adds()
jas.jas_gram(db, jas.JAS_ACCUMULATE | (jas.JAS_UPPER if upper else 0), None, B, np.zeros(n, np.int64))
lib.model_drain()
adds = lib.model_atomic_adds() - before
at = np.flatnonzero(B)
i = at // n if not upper else np.searchsorted(np.cumsum(np.arange(n, 0, -1)), at, side="right")
j = at % n if not upper else at - (i * n - i * (i - 1) // 2) + i
want = {}
smp = np.repeat(np.arange(n), np.diff(off).astype(np.int64))
order = np.lexsort((smp, ids))
rows_of = np.split(smp[order], np.flatnonzero(np.diff(ids[order])) + 1)
for r in rows_of:
    r = np.unique(r)
    for x in range(r.size):
        for y in r[x + 1:]:
            want[(int(r[x]), int(y))] = want.get((int(r[x]), int(y)), 0) + 1
assert {(int(p), int(q)): int(v) for p, q, v in zip(i, j, B[at])} == want
assert st["n_list_pairs"] > 7000 and want[(a, b)] >= 6000
print(adds, "additions for", st["n_list_pairs"], "pairs;", len(want), "different")
assert adds < 2 * len(want) + st["n_list_pairs"] // 16
"""


@pytest.mark.parametrize("n, upper", [(3000, 0), (8192, 1), (8193, 0), (10240, 1)])
def test_pairs_of_the_same_two_samples(library, n, upper):
    """Samples with many rows of their own: their pair words are equal, and B gets
    few additions for them (each would wait for the one before it)."""
    print(run(library, SAME_PAIRS, n, upper))


RUNS = r"""
n, long_runs = 1024, [int(x) for x in sys.argv[2:]]
rng = np.random.default_rng(len(long_runs))
# a row for every pair word: runs of 0 to 5 words with the long ones among them
words = rng.integers(0, 6, n)
words[n - 1] = 0
words[np.linspace(5, n - 30, len(long_runs)).astype(int)] = long_runs
x = np.repeat(np.arange(n), words)
y = rng.integers(x + 1, np.minimum(x + 8, n))
row = rng.permutation(x.size)
smp, ids = np.concatenate([x, y]), np.concatenate([row, row])
order = np.lexsort((ids, smp))
off = np.zeros(n + 1, np.uint64)
np.cumsum(np.bincount(smp, minlength=n), out=off[1:])
db, st = jas.jas_encode(ids[order].astype(np.uint64), off, n, jas.jas_encode_opts(20, 0, 1000, 0, 0, 64))
assert st["n_list_pairs"] == x.size
B = np.zeros((n, n), np.int32)
before = lib.model_barriers()
jas.jas_gram(db, jas.JAS_ACCUMULATE, None, B, np.zeros(n, np.int64))
lib.model_drain()
print(lib.model_barriers() - before, "waits for", x.size, "words in", (words > 0).sum(), "runs")
want = np.zeros((n, n), np.int32)
np.add.at(want, (x, y), 1)
assert np.array_equal(B, want)
"""


def test_short_runs_of_pairs_are_not_counted_one_by_one(library):
    """A run of a quarter of n words among hundreds of short ones: none is worth the
    waits that counting it by itself takes (0.106 ms for 0.006)."""
    waits = int(run(library, RUNS, 300).split()[0])
    assert waits < 40


@pytest.mark.parametrize("long_runs", [(511, 512, 513), (1023, 1024, 1025, 2047), (5000, 700, 3000, 1500), (9000,)])
@pytest.mark.parametrize("blocks", ["library", "library_of_many_passes"])
def test_runs_of_pairs_of_every_length(request, blocks, long_runs):
    """Runs around the shortest that is counted in LDS and around a chunk's length,
    between short ones, in chunks of 1024 words and in a few long ones."""
    run(request.getfixturevalue(blocks), RUNS, *long_runs)


UNEQUAL_SETS = r"""
rng = np.random.default_rng(11)
ids, off = collection(4, 3000, 20, 0.5)
db, _ = jas.jas_encode(ids, off, 4, jas.jas_encode_opts(20, 0, 0, jas.JAS_KEEP_IDS | jas.JAS_QUERY_ONLY, 0, 64))
members = [np.unique(ids[int(off[j]):int(off[j + 1])]) for j in range(4)]
for sizes in ([0] * 16500 + [32768] + [0] * 16500, [32768] + [0] * 9, [0, 31, 0, 0, 16, 1, 15, 17, 0]):
    nq = len(sizes)
    qoff = np.zeros(nq + 1, np.uint64)
    qoff[1:] = np.cumsum(sizes)
    q = rng.choice(ids, int(qoff[-1]))
    B, card = np.full((nq, 4), -1, np.int32), np.full(nq, -1, np.int64)
    jas.jas_query(db, q, qoff, nq, 0, None, B, card)
    assert not card[np.diff(qoff) == 0].any() and not B[np.diff(qoff) == 0].any()
    for k in np.flatnonzero(np.diff(qoff)):
        s = np.unique(q[int(qoff[k]):int(qoff[k + 1])])
        assert card[k] == s.size and all(B[k, j] == np.intersect1d(s, members[j]).size for j in range(4)), k
"""


def test_query_sets_of_unequal_sizes(library):
    """A request of one large set and many small or empty ones takes as many blocks
    as there are sets and shares of IDs (the largest set's number for every set is
    more than a launch may have)."""
    run(library, UNEQUAL_SETS)


ONE_SHARE = r"""
# 5000 IDs the hash deals to the first of their 313 blocks
x = np.arange(1 << 22, dtype=np.uint64)
h = ((x ^ (x >> np.uint64(32))) * np.uint64(0x9E3779B97F4A7C15)) >> np.uint64(32)
q = x[(h * np.uint64(313)) >> np.uint64(32) == 0][:5000]
assert q.size == 5000
ids = np.concatenate([q[::3], q[:10], x[:2000]])
off = np.array([0, q[::3].size, ids.size], np.uint64)
db, _ = jas.jas_encode(ids, off, 2, jas.jas_encode_opts(22, 0, 0, jas.JAS_KEEP_IDS | jas.JAS_QUERY_ONLY, 0, 64))
B, card = np.zeros(2, np.int32), np.zeros(1, np.int64)
jas.jas_query(db, q, np.array([0, q.size], np.uint64), 1, 0, None, B, card)
assert card[0] == q.size and B[0] == q[::3].size and B[1] == np.intersect1d(q, ids[int(off[1]):]).size
print(lib.model_atomic_swaps(), "slots looked at")
assert lib.model_atomic_swaps() < 1 << 20
"""


def test_query_ids_that_fill_one_table(library):
    """A block whose table is full leaves the request to the sort without looking at
    every slot for each ID that is left (256 threads do so once)."""
    print(run(library, ONE_SHARE))


CROWDED_IDS = r"""
rng = np.random.default_rng(2)
N = 30000
low = rng.integers(0, 1 << 30, N).astype(np.uint64)
few = rng.choice(low[:500], N)
groups = rng.choice(rng.integers(0, 1 << 62, 300), N).astype(np.uint64) + rng.integers(0, 100, N).astype(np.uint64)
two = np.where(np.arange(N) % 2 == 0, low, low + np.uint64(1 << 61))
prefix = np.uint64(5 << 40)

def passes(ids, ubits):
    out, before = np.zeros(N, np.uint64), lib.model_launches(b"k_radix_onesweep")
    u, inv = np.unique(ids, return_inverse=True)
    d, bits = jas.jas_relabel(ids, N, ubits, None, out)
    assert d == u.size and bits == max(1, int(u.size - 1).bit_length()) and np.array_equal(out, inv.astype(np.uint64))
    return lib.model_launches(b"k_radix_onesweep") - before

alone = passes(low, 30)
assert passes(low, 62) == alone and passes(low + prefix, 62) == alone and passes(low + np.uint64(1 << 63), 64) == alone
one = passes(np.full(N, 77, np.uint64), 62)
assert one == 1, one  # sorted on the one bit that is left
assert passes(two, 62) == 8, passes(two, 62)  # every bit, and nothing before
for ids in (few, few + prefix, groups):
    passes(ids, 63)
"""


def test_relabelling_of_ids_that_share_their_top_bits(library):
    """Crowded IDs are sorted as if the universe ended at the highest bit in which
    two of them differ, or, where that does not help, on every bit at once."""
    run(library, CROWDED_IDS)


BUDGET = r"""
plan, n, total, ubits, share, batch, dmin, flags, wb, budget = [float(a) if "." in a else int(a) for a in sys.argv[2:12]]
ids, off = collection(n, total, ubits, share)
opts = jas.jas_encode_opts(ubits, batch, dmin, flags, budget, wb)
if plan:
    p = jas.jas_plan_create(ids, off, n, opts, 0.25)
    jas.jas_plan_encode(p, ids, off)
    jas.jas_plan_check(p)
    db = p.db
else:
    db, _ = jas.jas_encode(ids, off, n, opts)
assert np.array_equal(gram(db, n), intersections(ids, off))
"""


@pytest.mark.parametrize("call", [
    "0 10 2000 20 0.5 0 3 0 64 560244", "0 10 2000 20 0.5 0 50 2 64 609668", "0 64 8000 30 0.5 0 2 0 64 670468",
    "0 300 60000 36 0.7 26 7 0 64 4572944", "0 64 200000 30 0.01 0 2 0 64 4028696", "0 64 200000 36 0.01 0 2 2 64 5543584",
    "1 40 20000 30 0.5 22 2 0 32 1319600", "1 40 20000 30 0.5 0 4 0 64 1757740", "1 300 60000 36 0.7 0 1000 0 64 5379348"])
def test_memory_budgets_that_were_enough_are(library, call):
    """The smallest budgets that an encode or a plan took with 8-bit sort passes,
    one pass's look-back words and counters without slots of their own (bytes, for
    collections of few and many sets, rows of both forms, batches, a query index)."""
    run(library, BUDGET, *call.split())


SMALL_PRODUCT = r"""
# two sets of the same IDs and 298 empty ones: 1024 word rows, 6 tile pairs
x = np.arange(65536, dtype=np.uint64)
off = np.full(301, 2 * x.size, np.uint64)
off[:2] = [0, x.size]
db, st = jas.jas_encode(np.concatenate([x, x]), off, 300, jas.jas_encode_opts(16, 0, 2, 0, 0, 64))
assert st["w_rows"] == 1024, st
jas.jas_gram(db, jas.JAS_FORCE_MFMA, None, np.zeros((300, 300), np.int32))
print(lib.model_blocks(b"k_gram_fp4"), "blocks")
assert lib.model_launches(b"k_gram_fp4") == 1 and lib.model_blocks(b"k_gram_fp4") < 192
"""


def test_small_products_take_few_blocks(library):
    """Each block adds whole tiles to B: 1024 word rows of 300 samples are not cut
    into as many blocks as run at once (16 rows each, 0.035 ms for 0.023)."""
    run(library, SMALL_PRODUCT)


@pytest.fixture(scope="module")
def library_of_many_passes(tmp_path_factory):
    """The library with one key per bucket instead of 512, and the large tiles from
    32 K keys on: 100,000 keys are then sorted as 50 M are, in passes of 9 bits and
    tiles of 24, 32 and 64 keys per thread.  A tile's look-back words have to be
    clear when it publishes its own.  Pair words are counted in few, long chunks."""
    if model.compiler() is None:
        pytest.skip("clang's AddressSanitizer runtime is not installed")
    publish = "            status_store(status + onesweep::status_index(tile, tid, kDigits), (tile == 0 ? kFlagP : kFlagA) | tc);"
    return model.build(str(tmp_path_factory.mktemp("many_passes")), changes=[
        ("jas_internal.hpp", "constexpr uint64_t kBucketKeys = 512;", "constexpr uint64_t kBucketKeys = 1;"),
        ("gram.hip", "constexpr uint64_t kPairBlocks = 4096;", "constexpr uint64_t kPairBlocks = 3;"),
        ("radix.hip", "const uint64_t two_tiles = (uint64_t)4 * 256 * kOsNT;", "const uint64_t two_tiles = 1024;"),
        # (a plan classifies the keys of a refused collection too: see the IDs outside the universe)
        ("encode.hip", "    if (dsz && (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 7u)) {", "    if (false) {"),
        ("radix.hip", publish, "            if (status_load(status + onesweep::status_index(tile, tid, kDigits))) abort();\n" + publish)])


MANY_PASSES = r"""
total, ubits, dmin, passes = [int(a) for a in sys.argv[2:6]]
n = 60
ids, off = collection(n, total, ubits, 0.5)
want = intersections(ids, off)
def count(f):
    before = lib.model_launches(b"k_radix_onesweep")
    B = f()
    assert np.array_equal(B, want)
    return lib.model_launches(b"k_radix_onesweep") - before
def encode(budget):
    db, st = jas.jas_encode(ids, off, n, jas.jas_encode_opts(ubits, 0, dmin, 0, budget, 64))
    assert dmin == 2 or st["n_list_pairs"] > 1 << 16  # pairs in the largest tiles
    B = gram(db, n)
    db.close()
    return B
pair_passes = 1 if dmin > 2 else 0
assert count(lambda: encode(0)) == passes + pair_passes
assert total > 200000 or count(lambda: encode(1 << 40)) == passes + pair_passes
for budget in (0, 1 << 40) if total <= 100000 else ():
    plan = jas.jas_plan_create(ids, off, n, jas.jas_encode_opts(ubits, 0, dmin, 0, budget, 64), 0.1)
    for _ in range(2 if total < 10000 else 1):
        jas.jas_plan_encode(plan, ids, off)
        assert np.array_equal(gram(plan.db, n), want)
        jas.jas_plan_check(plan)
    plan.close()
out = np.zeros(ids.size, np.uint64)
u, inv = np.unique(ids, return_inverse=True)
assert jas.jas_relabel(ids, ids.size, ubits, None, out)[0] == u.size and np.array_equal(out, inv.astype(np.uint64))
"""


@pytest.mark.parametrize("total, dmin, passes", [(9000, 2, 2), (75000, 1000, 2), (150000, 2, 2), (300000, 2, 3)])
def test_sorts_of_many_passes(library_of_many_passes, total, dmin, passes):
    """Sorts on 14 to 19 top bits (7 + 7, 9 + 8, 9 + 9, 7 + 7 + 5) with the look-back words
    of two passes cleared in turn, or of one where memory is limited; tiles of 16
    keys per thread, or 24 in the first pass and 32 in the next (64 for pair words)."""
    run(library_of_many_passes, MANY_PASSES, total, 50, dmin, passes)


OUTSIDE = r"""
# 13 sorted bits in passes of 7 and 6: bit 40 of an ID lies in the last pass's 7-bit digit, not in the 6 bits it sorts
n, ubits = 50, 40
ids, off = collection(n, 7600, ubits, 0.3)
assert 6144 < ids.size <= 1 << 13
opts = jas.jas_encode_opts(ubits, 0, 4, 0, 0, 64)
plan = jas.jas_plan_create(ids, off, n, opts, 0.1)
bad = ids.copy()
bad[::ids.size // 200] |= np.uint64(1 << ubits)
for call in (lambda: jas.jas_encode(bad, off, n, opts), lambda: (jas.jas_plan_encode(plan, bad, off), jas.jas_plan_check(plan))):
    try:
        call()
        raise SystemExit("an ID outside the universe was accepted")
    except jas.JasError as e:
        assert e.status == jas.JAS_EINVAL, str(e)
jas.jas_plan_encode(plan, ids, off)
jas.jas_plan_check(plan)
"""


def test_ids_outside_the_universe_are_sorted_by_the_digits_they_are_counted_by(library_of_many_passes):
    """IDs >= 2^U are refused after the sort: until then every place of the sorted
    keys is written, also where the last pass is narrower than the others (a plan
    classifies them before the host sees the flag)."""
    run(library_of_many_passes, OUTSIDE)
