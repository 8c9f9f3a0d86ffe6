"""Work that users of the Smith-Waterman database search have it do, as cases
that can be timed: a resident database and one call of a public entry point.

A case names an operation, a database (its number of sequences and the shape
of their lengths) and the query lengths and gap penalties:

  op  search      one query against every sequence, device buffers
      host        the same call over host buffers (query up, scores down)
      batch       many queries in one batched call, device buffers
      topk        one search, its k best hits and where their alignments end
      mode        global or semi-global scores
      traceback   the alignments of a query's best hits (host result)

  db  small       lengths log-normal, mean 350, clip 20..2,000 (the smallest
                  configuration of the benchmark: 2,000 sequences)
      plain       lengths log-normal, mean 355, clip 20..35,000, the longest
                  set to 35,000 (a Swiss-Prot-like protein database)
      longmix     2 % of the sequences of 10,000..35,000 residues, the rest
                  log-normal
      dna         nucleotide sequences, log-normal, mean 1,500, clip 30..12,000

Residues are drawn from the background composition (bases uniformly).  As in
a real database the query has relatives: a dozen sequences carry a stretch of
it at 30..100 % identity, so a few scores are far above the rest (and, for
queries of some hundred residues, above the range of the 16-bit kernels).
"""
import math

import numpy as np
import torch

import paper_2203_11100_amd as sw
import swinputs

RELATIVES = 12


def listed():
    return [
        # one short query against a small database: the latency of a call
        {"name": "small", "op": "search", "db": "small", "n_seqs": 2000, "m": 144,
         "go": 10, "ge": 2},
        # the same database kind through host buffers, as a script calls it
        {"name": "host-call", "op": "host", "db": "plain", "n_seqs": 20001, "m": 211,
         "go": 10, "ge": 2},
        # one query of the plain workload's shortest, a middle and its longest
        # length against the whole database
        {"name": "search-144", "op": "search", "db": "plain", "n_seqs": 200000, "m": 144,
         "go": 10, "ge": 2},
        {"name": "search-977", "op": "search", "db": "plain", "n_seqs": 200000, "m": 977,
         "go": 10, "ge": 2},
        {"name": "search-5478", "op": "search", "db": "plain", "n_seqs": 200000, "m": 5478,
         "go": 10, "ge": 2},
        # a database with a heavy tail of long sequences (the long-pair kernel)
        {"name": "long-mix", "op": "search", "db": "longmix", "n_seqs": 12500, "m": 2000,
         "go": 10, "ge": 2},
        # a file of queries of every length in one batched call
        {"name": "batch", "op": "batch", "db": "plain", "n_seqs": 100000, "m": 5000, "queries": 24,
         "go": 10, "ge": 2},
        # a search report: the best hits with their alignment ends, gaps read
        # as 10 + 2 k
        {"name": "topk", "op": "topk", "db": "plain", "n_seqs": 100000, "m": 457, "k": 1000,
         "go": 12, "ge": 2},
        # then the alignments of the ten best
        {"name": "traceback", "op": "traceback", "db": "plain", "n_seqs": 20001, "m": 310, "k": 10,
         "go": 10, "ge": 2},
        # the other alignment modes
        {"name": "global", "op": "mode", "db": "plain", "n_seqs": 100000, "m": 310,
         "mode": "global", "go": 10, "ge": 2},
        {"name": "semiglobal", "op": "mode", "db": "small", "n_seqs": 30000, "m": 975,
         "mode": "semiglobal", "go": 10, "ge": 2},
        # nucleotides: +5 / -4, gaps 16 / 4
        {"name": "dna", "op": "search", "db": "dna", "n_seqs": 3000, "m": 1001,
         "go": 16, "ge": 4},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: every operation and database kind, sizes spread over
    the logarithm of their ranges, no larger than the largest listed one."""
    op = rng.choice(["search", "search", "search", "host", "batch", "topk", "mode", "traceback"])
    db = rng.choice(["small", "plain", "plain", "plain", "longmix", "dna"])
    if op in ("batch", "mode", "traceback") and db in ("longmix", "dna"):
        db = "plain"
    lo, hi = {"small": (1500, 30000), "plain": (2000, 200000), "longmix": (2000, 15000),
              "dna": (1000, 6000)}[db]
    c = {"op": op, "db": db, "n_seqs": _log_uniform(rng, lo, hi), "m": _log_uniform(rng, 30, 5478)}
    c["go"], c["ge"] = (16, 4) if db == "dna" else rng.choice([(10, 2), (10, 2), (12, 2), (11, 1)])
    if op == "mode":
        c["mode"] = rng.choice(["global", "semiglobal"])
        c["m"] = _log_uniform(rng, 30, 2000)
        c["n_seqs"] = min(c["n_seqs"], 100000)
    if op == "topk":
        c["k"] = _log_uniform(rng, 1, 1000)
    if op == "traceback":
        c["k"] = _log_uniform(rng, 1, 25)
        c["m"] = _log_uniform(rng, 30, 1500)
        c["n_seqs"] = min(c["n_seqs"], 20001)
    if op == "batch":
        c["queries"] = _log_uniform(rng, 2, 24)
        c["n_seqs"] = min(c["n_seqs"], 100000)
        c["m"] = max(c["m"], 100)
    return c


def _lengths(case, rng):
    n, db = case["n_seqs"], case["db"]
    if db == "small":
        return swinputs.lognormal_lengths(n, 350.0, 0.75, 20, 2000, rng)
    if db == "dna":
        return swinputs.lognormal_lengths(n, 1500.0, 0.8, 30, 12000, rng)
    if db == "longmix":
        n_long = max(1, n // 50)
        lens = np.concatenate([swinputs.lognormal_lengths(n - n_long, 350.0, 0.75, 20, 9999, rng),
                               rng.integers(10000, 35001, size=n_long)])
        return lens[rng.permutation(n)].astype(np.int64)
    lens = swinputs.lognormal_lengths(n, 355.0, 0.75, 20, 35000, rng)
    lens[int(np.argmax(lens))] = 35000
    return lens


def _query_lengths(case):
    """The queries' lengths: one, or (batches) spread evenly over 50 .. m."""
    if case["op"] != "batch":
        return [case["m"]]
    k = case["queries"]
    return [50 + (case["m"] - 50) * i // (k - 1) for i in range(k)]


def _residues(case, n, gen):
    """n residue codes, drawn on the GPU, as a host array."""
    if case["db"] == "dna":
        codes = torch.randint(0, 4, (n,), dtype=torch.uint8, device="cuda", generator=gen)
    else:
        cdf = np.cumsum(swinputs.BACKGROUND_FREQS)
        cdf[-1] = 1.0
        lut = np.searchsorted(cdf, (np.arange(65536) + 0.5) / 65536.0, side="right")
        lut = torch.from_numpy(lut.astype(np.uint8)).cuda()
        codes = lut[torch.randint(0, 65536, (n,), dtype=torch.int32, device="cuda", generator=gen)]
    return codes.cpu().numpy()


def _inputs(case, seed):
    """Database (residues, offsets), queries, matrix and the sequences that
    carry a stretch of the first query, from the seed alone."""
    rng = np.random.default_rng([seed, 7])
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    lens = _lengths(case, rng)
    offs = np.zeros(len(lens) + 1, dtype=np.int64)
    np.cumsum(lens, out=offs[1:])
    res = _residues(case, int(offs[-1]), gen)
    queries = [_residues(case, m, gen) for m in _query_lengths(case)]
    # the relatives: the whole query where it fits, else a stretch of it
    q = queries[-1]
    ids = rng.choice(len(lens), RELATIVES, replace=False)
    for t, sid in enumerate(ids):
        n = min(len(q), int(lens[sid]))
        at_q = int(rng.integers(0, len(q) - n + 1))
        at = int(offs[sid]) + int(rng.integers(0, int(lens[sid]) - n + 1))
        identity = 0.3 + 0.7 * t / (RELATIVES - 1)
        keep = rng.random(n) < identity
        res[at:at + n][keep] = q[at_q:at_q + n][keep]
    matrix = swinputs.dna_matrix(5, 4, -2) if case["db"] == "dna" else swinputs.blosum62()
    return res, offs, queries, matrix, ids


def prepare(case, seed):
    res, offs, queries, matrix, ids = _inputs(case, seed)
    st = dict(case)
    st.update(handle=sw.Database(res, offs), matrix=matrix)
    n = len(offs) - 1
    op = case["op"]
    if op in ("host", "traceback"):
        st["query"] = queries[0]
        if op == "traceback":     # the hits that a report would align
            rest = np.setdiff1d(np.arange(min(n, 4 * RELATIVES)), ids)
            st["seqs"] = np.concatenate([ids[::-1], rest])[:case["k"]].astype(np.int32)
    elif op == "batch":
        st["qoffs"] = np.concatenate([[0], np.cumsum([len(q) for q in queries])]).astype(np.int64)
        st["query"] = torch.from_numpy(np.concatenate(queries)).cuda()
        st["out"] = torch.empty((len(queries), n), dtype=torch.int32, device="cuda")
    else:
        st["query"] = torch.from_numpy(queries[0]).cuda()
        st["out"] = torch.empty(n, dtype=torch.int32, device="cuda")
        if op == "topk":
            st["hits"] = torch.empty((min(case["k"], n), 4), dtype=torch.int32, device="cuda")
    return st


def run(st):
    db, q, s, go, ge = st["handle"], st["query"], st["matrix"], st["go"], st["ge"]
    op = st["op"]
    if op == "search":
        db.search_async(q, s, go, ge, st["out"])
        return st["out"]
    if op == "host":
        return db.search(q, s, go, ge)
    if op == "batch":
        db.search_batch_async(q, st["qoffs"], s, go, ge, st["out"])
        return st["out"]
    if op == "topk":
        db.search_topk_async(q, s, go, ge, st["k"], st["out"], st["hits"])
        return st["out"], st["hits"]
    if op == "mode":
        db.search_mode_async(q, s, go, ge, st["mode"], st["out"])
        return st["out"]
    found = db.traceback(q, s, go, ge, st["seqs"])
    ops = np.frombuffer("".join(a["ops"] for a in found).encode(), dtype=np.uint8)
    room = np.zeros(16 * len(q) * len(found), dtype=np.uint8)   # their number varies with the inputs
    room[:len(ops)] = ops
    return (np.array([[a["seq"], a["score"], a["query_begin"], a["query_end"], a["db_begin"],
                       a["db_end"]] for a in found], dtype=np.int32), room)


def _expected_residues(case):
    """Residues of the database, from its recipe."""
    n = case["n_seqs"]
    if case["db"] == "dna":
        return 1480.0 * n
    if case["db"] == "longmix":
        return 348.0 * (n - n // 50) + 22500.0 * max(1, n // 50)
    if case["db"] == "small":
        return 347.0 * n
    return 355.0 * n + 25000.0


def work(case):
    """Residues and queries read once, scores written once; ten operations a
    cell of Gotoh's recurrence (one add, three subtractions, six maxima)."""
    n, qs = case["n_seqs"], _query_lengths(case)
    if case["op"] == "traceback":
        k = case["k"]
        res = 355.0 * k
        return {"bytes": res + sum(qs) + 24.0 * k + 355.0 * k, "flops": 10.0 * sum(qs) * res}
    res = _expected_residues(case)
    out = 4.0 * n * len(qs) + 16.0 * case.get("k", 0)
    return {"bytes": res + sum(qs) + out, "flops": 10.0 * sum(qs) * res}


def exact(case, seed):
    """Local scores by the recurrence in 64-bit integers, anti-diagonal by
    anti-diagonal over groups of sequences of similar length; None for other
    operations and for cases that take too long this way."""
    if case["op"] not in ("search", "host"):
        return None
    lens = _lengths(case, np.random.default_rng([seed, 7]))
    m, n = case["m"], case["n_seqs"]
    if m * float((lens + m).sum()) > 3e10 or m + int(lens.max()) > 40000:
        return None
    res, offs, queries, matrix, _ = _inputs(case, seed)
    go, ge = case["go"], case["ge"]
    low = -(1 << 40)
    table = torch.full((25, 25), low, dtype=torch.int64)
    table[:24, :24] = torch.from_numpy(matrix.astype(np.int64))
    table = table.cuda()
    q = torch.from_numpy(queries[0].astype(np.int64)).cuda()
    res_d = torch.from_numpy(np.append(res, 24).astype(np.uint8)).cuda()
    order = np.argsort(lens, kind="stable")[::-1]
    out = torch.zeros(n, dtype=torch.int64, device="cuda")
    group = max(1, min(4096, 8_000_000 // m))
    at = 0
    while at < n:
        size = min(group, 64) if at == 0 else group      # the longest ones apart
        ids = order[at:at + size].copy()
        at += size
        L = int(lens[ids].max())
        b = len(ids)
        # codes reversed along the query: cell (i, j = d - i) reads column
        # m - 1 - i + d of the padded codes flipped by rows
        pos = torch.arange(L, device="cuda")[None, :]
        start = torch.from_numpy(offs[ids]).cuda()[:, None]
        ln = torch.from_numpy(lens[ids]).cuda()[:, None]
        codes = torch.full((b, L + 2 * m), 24, dtype=torch.uint8, device="cuda")
        codes[:, m:m + L] = res_d[torch.where(pos < ln, start + pos, len(res_d) - 1)]
        z = lambda v: torch.full((b, m + 1), v, dtype=torch.int64, device="cuda")  # noqa: E731
        h1, h2, e, f, best = z(0), z(0), z(low), z(low), z(0)
        rows = q.flip(0)[None, :].expand(b, m)            # row i at place m - 1 - i
        for d in range(m + L - 1):
            # places 0 .. m - 1 hold rows m - 1 .. 0; place m is the top border
            s = table[rows, codes[:, d + 1:d + 1 + m].long()]
            e2 = torch.maximum(e[:, :m] - ge, h1[:, :m] - go)
            f2 = torch.maximum(f[:, 1:] - ge, h1[:, 1:] - go)
            h = torch.clamp(torch.maximum(torch.maximum(h2[:, 1:] + s, e2), f2), min=0)
            h2, h1 = h1, h2
            h1[:, :m] = h
            h1[:, m] = 0
            e[:, :m] = e2
            f[:, :m] = f2
            best = torch.maximum(best, h1)
        out[torch.from_numpy(ids).cuda()] = best.max(dim=1).values
    return out
