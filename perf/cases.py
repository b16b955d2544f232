"""The library's work as its users have it done: cases to time and compare.

A case is a dict of plain values.  `listed()` names the ones that are always
measured, `draw(rng)` gives one more of the same ranges, `prepare(case, seed)`
makes what a program has in hand before the call (inputs on the GPU, a query
database, an encode plan), `run(state)` is one pass through the public entry
points, `work(case)` what that pass cannot do without and `exact(case, seed)`
its results by plain torch in 64 bits.

Every input is made on the GPU from the seed.  Sets follow the collections
this project is measured on: part of a set from one of a few shared pools of
IDs (without repeats), the rest uniform over the universe ("pool"); indicator
matrices whose entries are 1 with one probability ("bernoulli"); the
neighbourhoods of a power-law graph ("graph"); and the k-mers of mutated
copies of a few genomes ("kmer").
"""
import math

import numpy as np
import torch

from paper_1911_04200_amd import api, jas

DEVICE = "cuda"
CHUNK = 1 << 26  # entries made at a time


def listed():
    return [
        # A first look at a few small samples: latency, launches and read-backs count.
        dict(name="pairs_tiny", kind="pool", n=32, universe_bits=24, size_lo=1e3, size_hi=1e5, share_lo=0.0,
             share_hi=0.8, pools=1, pool_log2=16, batch_bits=24, upper=False, word_bits=64),
        # All pairs of the vertices of a small power-law graph: few IDs, many outputs.
        dict(name="pairs_graph", kind="graph", n=8192, edge_factor=64, upper=False, word_bits=64),
        # The paper's synthetic matrix at p = 1e-3 (32M rows, 10k samples): every row goes to the row lists.
        dict(name="pairs_sparse", kind="bernoulli", n=10000, universe_bits=25, density=1e-3, upper=True,
             word_bits=64),
        # Large genome collection: 1024 samples of about a million k-mers in twenty groups, wide universe.
        dict(name="pairs_paperlike", kind="pool", n=1024, universe_bits=40, size_lo=2e5, size_hi=6e6, share_lo=0.3,
             share_hi=0.9, pools=20, pool_log2=22, batch_bits=26, upper=False, word_bits=64),
        # One core pool shared by every sample: dense packed rows, the matrix units' case.
        dict(name="pairs_precision", kind="pool", n=4096, universe_bits=32, size_lo=1e5, size_hi=1e6, share_lo=0.7,
             share_hi=0.7, pools=1, pool_log2=22, batch_bits=32, upper=False, word_bits=64),
        # Many samples in many groups, packed upper layout: row lists at full size.
        dict(name="pairs_batching", kind="pool", n=10000, universe_bits=36, size_lo=1e3, size_hi=1e6, share_lo=0.3,
             share_hi=0.9, pools=50, pool_log2=22, batch_bits=26, upper=True, word_bits=64),
        # One of the eight parts of the p = 1e-2 matrix streamed through the GPU: encode, add to B, finish.
        dict(name="stream_part", kind="bernoulli", n=10000, universe_bits=22, density=1e-2, upper=True, word_bits=64,
             accumulate=True),
        # A service that encodes collection after collection of one shape: a plan, replayed as one HIP graph.
        dict(name="plan_replay", kind="pool", n=1000, universe_bits=36, size_lo=1e3, size_hi=1e5, share_lo=0.3,
             share_hi=0.9, pools=5, pool_log2=19, batch_bits=26, upper=True, word_bits=64, plan=True),
        # The smallest request against a resident database: one query set, latency.
        dict(name="query_one", kind="pool", n=4096, universe_bits=36, size_lo=1e5, size_hi=1e6, share_lo=0.3,
             share_hi=0.9, pools=32, pool_log2=22, batch_bits=26, nq=1, q_lo=1e4, q_hi=1e4, noalloc=False),
        # A serving call: 32 query sets of ten thousand to a million IDs.
        dict(name="query_batch", kind="pool", n=4096, universe_bits=36, size_lo=1e5, size_hi=1e6, share_lo=0.3,
             share_hi=0.9, pools=32, pool_log2=22, batch_bits=26, nq=32, q_lo=1e4, q_hi=1e6, noalloc=False),
        # Link prediction: a few vertices' neighbourhoods against every vertex of a graph, no allocation.
        dict(name="query_links", kind="graph", n=1 << 20, edge_factor=16, nq=16, noalloc=True),
        # Long k-mers from sequences to similarities: front end, exact relabelling, all pairs.
        dict(name="kmer31_pairs", kind="kmer", n=128, length=1 << 20, pieces=4, k=31, canonical=True, upper=False,
             word_bits=64),
    ]


def draw(rng):
    def log(lo, hi):
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    what = rng.choice(["pool", "pool", "pool", "bernoulli", "graph", "plan", "query", "query", "links", "kmer"])
    upper, wb = rng.random() < 0.5, rng.choice([64, 64, 64, 32])
    if what in ("pool", "plan"):
        n = int(log(3, 1000 if what == "plan" else 10000))
        total = log(1e4, 3e7 if what == "plan" else 1e9)
        hi = max(8.0, min(2e6, 3.0 * total / n))
        c = dict(kind="pool", n=n, universe_bits=rng.randint(24, 40), size_lo=max(1.0, hi * log(0.01, 0.5)), size_hi=hi,
                 share_lo=round(rng.uniform(0.0, 0.5), 2), share_hi=round(rng.uniform(0.5, 0.9), 2),
                 pools=int(log(1, min(50, n))), pool_log2=min(22, max(5, math.ceil(math.log2(hi)) + rng.randint(0, 2))),
                 batch_bits=rng.choice([0, 20, 26]), upper=upper, word_bits=wb)
        return dict(c, plan=True) if what == "plan" else c
    if what == "bernoulli":
        n, u, p = int(log(100, 10000)), rng.randint(16, 25), log(1e-4, 1e-1)
        while n * 2.0 ** u * p > 4e8 or n * 2.0 ** u * n > 4.2e14 and n * p > 25 or n * n * p * p * 2.0 ** u > 4e9 and n * p < 25:
            u -= 1
        return dict(kind="bernoulli", n=n, universe_bits=u, density=p, upper=upper, word_bits=wb,
                    accumulate=rng.random() < 0.5)
    if what == "graph":
        return dict(kind="graph", n=1 << rng.randint(6, 13), edge_factor=int(log(4, 64)), upper=upper, word_bits=wb)
    if what == "query":
        n = int(log(100, 8192))
        hi = log(1e3, min(1e6, 5e8 / n))
        return dict(kind="pool", n=n, universe_bits=rng.randint(28, 40), size_lo=0.1 * hi, size_hi=hi, share_lo=0.3,
                    share_hi=0.9, pools=int(log(1, 32)), pool_log2=22, batch_bits=26, nq=int(log(1, 64)), q_lo=100.0,
                    q_hi=log(1e3, 1e5), noalloc=rng.random() < 0.5)
    if what == "links":
        return dict(kind="graph", n=1 << rng.randint(14, 20), edge_factor=int(log(4, 16)), nq=int(log(1, 32)),
                    noalloc=rng.random() < 0.5)
    return dict(kind="kmer", n=int(log(2, 128)), length=int(log(1e4, 1e6)), pieces=rng.randint(1, 8),
                k=rng.choice([19, 21, 31]), canonical=rng.random() < 0.7, upper=upper, word_bits=wb)


# ---------------------------------------------------------------------------
# Inputs.
def _gen(seed):
    return torch.Generator(device=DEVICE).manual_seed(seed)


def _csr(sizes):
    off = np.zeros(len(sizes) + 1, dtype=np.int64)
    np.cumsum(sizes, out=off[1:])
    return off


def _below(width, gen):
    """A uniform integer in [0, width) for every entry of width."""
    u = torch.rand(width.shape, generator=gen, device=DEVICE, dtype=torch.float64)
    return torch.minimum((u * width).to(torch.int64), width - 1)


def _strata(t, k, m, gen):
    """Entry t of k ascending, distinct values below m: one in each of k equal stretches of [0, m)."""
    lo = t * m // k
    return lo + _below((t + 1) * m // k - lo, gen)


def _spread(g, bits):
    """A fixed bijection of the integers below 2^bits."""
    mask, h = (1 << bits) - 1, max(1, bits // 2)
    g = (g * 0x2545F4914F6CDD1D) & mask
    g = g ^ (g >> h)
    g = (g * 0x9E3779B97F4A7C1) & mask
    return g ^ (g >> h)


def _entries(sizes):
    """(first entry, one past, set of every entry, place in its set), CHUNK entries or whole sets at a time."""
    off = _csr(sizes)
    doff = torch.from_numpy(off).to(DEVICE)
    a = 0
    while a < len(sizes):
        b = int(np.searchsorted(off, off[a] + CHUNK, side="right")) - 1
        b = min(len(sizes), max(b, a + 1))
        lens = doff[a + 1:b + 1] - doff[a:b]
        s = torch.repeat_interleave(torch.arange(a, b, device=DEVICE), lens, output_size=int(off[b] - off[a]))
        yield int(off[a]), int(off[b]), s, torch.arange(int(off[a]), int(off[b]), device=DEVICE) - doff[s]
        a = b


def _pool_sets(sizes, parts, group, universe_bits, pool_log2, gen):
    """IDs of the sets: set i has parts[i] of the IDs of pool group[i], the rest uniform."""
    ids = torch.empty(max(int(sizes.sum()), 1), dtype=torch.int64, device=DEVICE)
    k, c = torch.from_numpy(parts).to(DEVICE), torch.from_numpy(group).to(DEVICE)
    for a, b, s, t in _entries(sizes):
        ks = k[s]
        shared = t < ks
        g = _strata(torch.minimum(t, ks), (ks + 1), 1 << pool_log2, gen) + (c[s] << pool_log2)
        v = torch.randint(0, 1 << universe_bits, (b - a,), generator=gen, device=DEVICE)
        ids[a:b] = torch.where(shared, _spread(g, universe_bits), v)
    return ids


def _pool_case(n, lo, hi, share, groups, c, rng, gen):
    sizes = np.exp(rng.uniform(math.log(lo), math.log(hi), n)).astype(np.int64)
    sizes = np.minimum(np.maximum(sizes, 1), 1 << (c["universe_bits"] - 1))
    parts = np.minimum((sizes * rng.uniform(share[0], share[1], n)).astype(np.int64), (1 << c["pool_log2"]) - 1)
    group = rng.integers(0, groups, n) % max(1, 1 << (c["universe_bits"] - c["pool_log2"]))
    return _pool_sets(sizes, parts, group, c["universe_bits"], c["pool_log2"], gen), _csr(sizes)


def _bernoulli(c, rng, gen):
    m = 1 << c["universe_bits"]
    sizes = rng.binomial(m, c["density"], c["n"]).astype(np.int64)
    ids = torch.empty(max(int(sizes.sum()), 1), dtype=torch.int64, device=DEVICE)
    k = torch.from_numpy(sizes).to(DEVICE)
    for a, b, s, t in _entries(sizes):
        ids[a:b] = _strata(t, k[s], m, gen)
    return ids, _csr(sizes)


def _graph(c, gen):
    """Neighbourhoods of an undirected R-MAT graph (quadrants 0.57, 0.19, 0.19, 0.05): ascending, no repeats."""
    bits = c["n"].bit_length() - 1
    e = c["edge_factor"] * c["n"]
    u = torch.zeros(e, dtype=torch.int64, device=DEVICE)
    v = torch.zeros(e, dtype=torch.int64, device=DEVICE)
    for _ in range(bits):
        r = torch.rand(e, generator=gen, device=DEVICE)
        u = 2 * u + (r >= 0.76)
        v = 2 * v + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    u, v = _spread(u, bits), _spread(v, bits)
    keep = u != v
    u, v = u[keep], v[keep]
    key = torch.unique(torch.cat([u << bits | v, v << bits | u]))
    deg = torch.bincount(key >> bits, minlength=c["n"]).cpu().numpy()
    return key & (c["n"] - 1), _csr(deg)


def _genomes(c, rng, gen):
    """n copies of one of four random genomes, one base in a hundred substituted, each cut into pieces: 2-bit words."""
    n, L = c["n"], c["length"]
    refs = torch.randint(0, 4, (4, L), generator=gen, device=DEVICE, dtype=torch.uint8)
    bases = refs[torch.from_numpy(rng.integers(0, 4, n)).to(DEVICE)]
    hit = torch.rand((n, L), generator=gen, device=DEVICE) < 0.01
    sub = torch.randint(1, 4, (n, L), generator=gen, device=DEVICE, dtype=torch.uint8)
    bases = torch.where(hit, (bases + sub) & 3, bases).reshape(-1)
    bases = torch.nn.functional.pad(bases, (0, -bases.numel() % 32)).reshape(-1, 32)
    words = torch.zeros(bases.shape[0], dtype=torch.int64, device=DEVICE)
    for j in range(32):
        words |= bases[:, j].to(torch.int64) << (2 * j)
    cuts = np.sort(rng.integers(1, L, (n, c["pieces"] - 1)), axis=1) + L * np.arange(n)[:, None]
    starts = np.concatenate([L * np.arange(n)[:, None], cuts], axis=1).reshape(-1)
    seq_off = np.concatenate([starts, [n * L]]).astype(np.uint64)
    return words, seq_off, (np.arange(n + 1) * c["pieces"]).astype(np.uint64)


def _sets(c, seed):
    """The case's sets: (ids, host offsets)."""
    rng, gen = np.random.default_rng(seed), _gen(seed)
    if c["kind"] == "bernoulli":
        return _bernoulli(c, rng, gen)
    if c["kind"] == "graph":
        return _graph(c, gen)
    return _pool_case(c["n"], c["size_lo"], c["size_hi"], (c["share_lo"], c["share_hi"]), c["pools"], c, rng, gen)


def _queries(c, seed, ids, off):
    """The case's query sets: new sets of the pools, or vertices' neighbourhoods with a few new edges."""
    rng, gen = np.random.default_rng(seed + 1), _gen(seed + 1)
    if c["kind"] == "pool":
        return _pool_case(c["nq"], c["q_lo"], c["q_hi"], (0.0, 0.9), c["pools"], c, rng, gen)
    picked = rng.choice(c["n"], c["nq"], replace=False)
    parts = [torch.cat([ids[off[i]:off[i + 1]], torch.from_numpy(rng.integers(0, c["n"], 2)).to(DEVICE)]) for i in picked]
    return torch.cat(parts), _csr([p.numel() for p in parts])


def _universe(c):
    return 2 * c["k"] if c["kind"] == "kmer" else c["n"].bit_length() - 1 if c["kind"] == "graph" else c["universe_bits"]


def _opts(c, flags=0, universe_bits=0):
    return jas.jas_encode_opts(universe_bits or _universe(c), c.get("batch_bits", 0), 0, flags, 0, c.get("word_bits", 64))


def _device(off):
    return torch.from_numpy(np.asarray(off, dtype=np.int64)).to(DEVICE)


def _outputs(c, rows=None):
    n = c["n"]
    length = rows * n if rows else n * (n + 1) // 2 if c["upper"] else n * n
    return {"B": torch.empty(length, dtype=torch.int32, device=DEVICE),
            "card": torch.empty(rows or n, dtype=torch.int64, device=DEVICE),
            "den": torch.empty(length, dtype=torch.int64, device=DEVICE),
            "J": torch.empty(length, dtype=torch.float64, device=DEVICE)}


# ---------------------------------------------------------------------------
def prepare(case, seed):
    c = dict(case)
    if c["kind"] == "kmer":
        words, seq_off, smp_off = _genomes(c, np.random.default_rng(seed), _gen(seed))
        off = jas.jas_kmer_offsets(seq_off, smp_off, c["k"])
        return dict(case=c, words=words, seq_off=seq_off, off=_device(off),
                    ids=torch.empty(max(int(off[-1]), 1), dtype=torch.int64, device=DEVICE))
    ids, off = _sets(c, seed)
    state = dict(case=c, ids=ids, off=_device(off))
    if "nq" in c:  # the resident database, as a server keeps it
        q_ids, q_off = _queries(c, seed, ids, off)
        db, _ = jas.jas_encode(ids, state["off"], c["n"], _opts(c, jas.JAS_KEEP_IDS | jas.JAS_QUERY_ONLY))
        return dict(case=c, db=db, ids=q_ids, off=_device(q_off))
    if c.get("accumulate"):
        state["out"] = _outputs(c)
    if c.get("plan"):  # one captured step, replayed for every collection of this shape
        state["plan"] = plan = jas.jas_plan_create(ids, state["off"], c["n"], _opts(c), 0.25)
        state["out"] = out = _outputs(c)
        flags = jas.JAS_UPPER if c["upper"] else 0
        torch.cuda.synchronize()
        state["graph"] = graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            jas.jas_plan_encode(plan, ids, state["off"])
            jas.jas_gram(plan.db, flags, None, out["B"], out["card"], out["den"], out["J"])
    return state


def run(state):
    c = state["case"]
    n, ids, off = c["n"], state["ids"], state["off"]
    if c.get("plan"):
        state["graph"].replay()
        return state["out"]
    if "nq" in c:
        if not c["noalloc"]:
            return api.query(state["db"], ids, off)
        out = _outputs(c, c["nq"])
        jas.jas_query_noalloc(state["db"], ids, off, c["nq"], 0, None, out["B"], out["card"], out["den"], out["J"])
        return out
    universe = _universe(c)
    if c["kind"] == "kmer":
        jas.jas_kmers(state["words"], state["seq_off"], c["k"], jas.JAS_CANONICAL if c["canonical"] else 0, None, ids)
        if universe + (n - 1).bit_length() > 64:
            _, universe = jas.jas_relabel(ids, ids.numel(), universe, None, ids)
    if c.get("accumulate"):
        out = state["out"]
        flags = jas.JAS_UPPER if c["upper"] else 0
        out["B"].zero_()
        out["card"].zero_()
        db, _ = jas.jas_encode(ids, off, n, _opts(c))
        jas.jas_gram(db, flags | jas.JAS_ACCUMULATE, None, out["B"], out["card"])
        db.close()
        jas.jas_finalize(n, flags, None, out["B"], out["card"], out["den"], out["J"])
        return out
    db, _ = jas.jas_encode(ids, off, n, _opts(c, universe_bits=universe))
    out = api.gram(db, upper=c["upper"])
    db.close()
    return out


# ---------------------------------------------------------------------------
def _mean_size(lo, hi):
    return (hi - lo) / math.log(hi / lo) if hi > lo else lo


def _rmat_squares(c):
    """The sum of the squared degrees an R-MAT graph would have if no edge came twice."""
    return (2.0 * c["edge_factor"] * c["n"]) ** 2 * (0.76 ** 2 + 0.24 ** 2) ** (c["n"].bit_length() - 1)


def work(case):
    """Every ID read once, every output written once, and one multiply-add for every pair of samples and shared row."""
    c, n = case, case["n"]
    if "nq" in c:
        if c["kind"] == "pool":
            total = c["nq"] * _mean_size(c["q_lo"], c["q_hi"])
            held = 0.45 * total * n * 0.6 * _mean_size(c["size_lo"], c["size_hi"]) / (c["pools"] * 2.0 ** c["pool_log2"])
        else:
            total = c["nq"] * (2.0 * c["edge_factor"] + 2)
            held = total * _rmat_squares(c) / (2.0 * c["edge_factor"] * n)
        # a query ID, the place where it is looked up and the samples found there
        return {"bytes": 8 * total + 16 * total + 8 * held + 20.0 * c["nq"] * n, "flops": 2 * held}
    outs = 20.0 * (n * (n + 1) // 2 if c.get("upper") else n * n) + 16.0 * n
    if c["kind"] == "kmer":
        total = float(n) * c["length"]
        return {"bytes": total / 4 + 16 * total + outs, "flops": total * n / 4}
    if c["kind"] == "bernoulli":
        total = n * 2.0 ** c["universe_bits"] * c["density"]
        pairs = 2.0 ** c["universe_bits"] * (n * c["density"]) ** 2 / 2
    elif c["kind"] == "graph":
        total = 2.0 * c["edge_factor"] * n
        pairs = _rmat_squares(c) / 2
    else:
        total = n * _mean_size(c["size_lo"], c["size_hi"])
        part = total * (c["share_lo"] + c["share_hi"]) / 2
        pairs = part * part / (2.0 * c["pools"] * 2.0 ** c["pool_log2"])
    return {"bytes": 8 * total + outs, "flops": 2 * pairs}


# ---------------------------------------------------------------------------
def _incidence(ids, off):
    """Distinct (row, set) pairs of CSR sets, as rows numbered 0 .. and sets."""
    sets = torch.repeat_interleave(torch.arange(len(off) - 1, device=DEVICE), _device(np.diff(off)))
    rows = torch.unique(ids[:sets.numel()], return_inverse=True)[1]
    n = len(off) - 1
    key = torch.unique(rows * n + sets)
    return key // n, key % n


def _kmer_ids(c, seed):
    """The k-mer IDs by the definition: a base-4 number, first base most significant."""
    words, seq_off, smp_off = _genomes(c, np.random.default_rng(seed), _gen(seed))
    b = ((words[:, None] >> (2 * torch.arange(32, device=DEVICE))) & 3).reshape(-1)
    k, out, sizes = c["k"], [], []
    for s in range(c["n"]):
        have = 0
        for p in range(int(smp_off[s]), int(smp_off[s + 1])):
            q = b[int(seq_off[p]):int(seq_off[p + 1])]
            if q.numel() < k:
                continue
            m = q.numel() - k + 1
            f, r = torch.zeros(m, dtype=torch.int64, device=DEVICE), torch.zeros(m, dtype=torch.int64, device=DEVICE)
            for j in range(k):
                f = 4 * f + q[j:j + m]
                r = r + ((3 - q[j:j + m]) << (2 * j))
            out.append(torch.minimum(f, r) if c["canonical"] else f)
            have += m
        sizes.append(have)
    return (torch.cat(out) if out else b[:0]), _csr(sizes)


def exact(case, seed):
    c, n = dict(case), case["n"]
    if "nq" in c:
        if c["nq"] * n > 8192:
            return None
        ids, off = _sets(c, seed)
        q_ids, q_off = _queries(c, seed, ids, off)
        sets = [torch.unique(q_ids[q_off[i]:q_off[i + 1]]) for i in range(c["nq"])]
        inter = torch.zeros((c["nq"], n), dtype=torch.float64, device=DEVICE)
        card = torch.zeros(n, dtype=torch.float64, device=DEVICE)
        for j in range(n):
            x = torch.unique(ids[off[j]:off[j + 1]])
            card[j] = x.numel()
            for i, q in enumerate(sets):
                at = torch.searchsorted(x, q).clamp(max=x.numel() - 1)
                inter[i, j] = (x[at] == q).sum()
        q_card = torch.tensor([float(q.numel()) for q in sets], dtype=torch.float64, device=DEVICE)
        union = q_card[:, None] + card - inter
        J = inter / union
        return {"J": J.reshape(-1) if c["noalloc"] else J}
    if c["kind"] == "kmer":
        if c["n"] * c["length"] > 2e6:
            return None
        ids, off = _kmer_ids(c, seed)
    else:
        total = (n * _mean_size(c["size_lo"], c["size_hi"]) if c["kind"] == "pool" else
                 n * 2.0 ** c["universe_bits"] * c["density"] if c["kind"] == "bernoulli" else 1e6)
        if total > 5e6 or total * n * n > 1e14:
            return None
        ids, off = _sets(c, seed)
    rows, sets = _incidence(ids, off)
    inter = torch.zeros((n, n), dtype=torch.float64, device=DEVICE)
    step = max(1, (1 << 28) // n)  # rows of the indicator matrix at a time
    top = int(rows.max()) + 1 if rows.numel() else 0
    for a in range(0, top, step):
        lo, hi = (int(v) for v in torch.searchsorted(rows, torch.tensor([a, a + step], device=DEVICE)))
        A = torch.zeros((min(step, top - a), n), dtype=torch.float64, device=DEVICE)
        A[rows[lo:hi] - a, sets[lo:hi]] = 1.0
        inter += A.T @ A
    card = torch.bincount(sets, minlength=n).to(torch.float64)
    union = card[:, None] + card - inter
    J = torch.where(union == 0, torch.ones_like(union), inter / union.clamp(min=1))
    if not c["upper"]:
        return {"J": J.reshape(-1) if c.get("plan") or c.get("accumulate") else J}
    i, j = torch.triu_indices(n, n, device=DEVICE).unbind(0)
    return {"J": J[i, j]}
