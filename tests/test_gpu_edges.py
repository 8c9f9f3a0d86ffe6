"""GPU parity where several of the packed kernels' resources meet their limits at
once: contexts with persistent kernels and long pairs side by side, the
allocation-free search with fewer row buffers than it would take (and under
capture), batches whose long pairs keep a profile slot for every one of 16 waves,
and boundary rows that wrap beside guarded scores; against the oracle."""
import sys

import numpy as np
import pytest

import oracle.cpu as ocpu
import swinputs

pytestmark = pytest.mark.gpu

B62 = swinputs.blosum62()


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module")
def sw():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2203_11100_amd as lib
    return lib


def _mix(seed, n_short, n_long, longest=20000):
    rng = np.random.default_rng(seed)
    lens = np.concatenate([swinputs.lognormal_lengths(n_short, 350.0, 0.75, 20, 2047, rng),
                           rng.integers(2048, longest + 1, n_long)]).astype(np.int64)
    lens[-1] = longest
    res, offs = swinputs.make_database(rng.permutation(lens), rng)
    return res, offs, rng


def _relatives(res, offs, q, rng, n=4):
    sizes = np.diff(offs)
    for sid in rng.choice(len(sizes), n, replace=False):
        k = min(len(q), int(sizes[sid]))
        res[offs[sid]:offs[sid] + k] = q[:k]


def _same(got, want, what):
    bad = np.nonzero(got != want)[0]
    assert len(bad) == 0, (what, [(int(i), int(got[i]), int(want[i])) for i in bad[:5]])


def test_contexts_with_long_pairs_at_once(sw):
    import torch
    res, offs, rng = _mix(1, 3000, 40)
    qs = [swinputs.random_residues(m, rng) for m in (40, 300, 700, 1500)]
    _relatives(res, offs, qs[2], rng)
    want = [ocpu.search(q, res, offs, B62, 10, 2) for q in qs]
    say("four contexts at once")
    with sw.Database(res, offs) as db:
        ctxs = [db.context() for _ in qs]
        try:
            dq = [torch.from_numpy(q).cuda() for q in qs]
            outs = [torch.empty(len(offs) - 1, dtype=torch.int32, device="cuda") for _ in qs]
            streams = [torch.cuda.Stream() for _ in qs]
            torch.cuda.synchronize()
            for turn in range(4):       # each context takes every query, several in flight
                for k, (c, s) in enumerate(zip(ctxs, streams)):
                    outs[k].fill_(-7)
                torch.cuda.synchronize()
                for k, (c, s) in enumerate(zip(ctxs, streams)):
                    j = (k + turn) % len(qs)
                    c.search_async(dq[j], B62, 10, 2, outs[k], s)
                torch.cuda.synchronize()
                for k in range(len(qs)):
                    _same(outs[k].cpu().numpy(), want[(k + turn) % len(qs)], (turn, k))
        finally:
            for c in ctxs:
                c.close()


# 32 MiB hold nine rows of 400,000 columns: queries of several passes keep fewer pairs
# in flight than waves, on fewer workgroups than pairs
@pytest.mark.parametrize("m", [100, 1000, 3000])
def test_noalloc_with_few_row_buffers(sw, m):
    import torch
    rng = np.random.default_rng(m)
    lens = np.concatenate([[400_000], rng.integers(2048, 5000, 60), rng.integers(20, 900, 300)])
    res, offs = swinputs.make_database(lens.astype(np.int64), rng)
    q = swinputs.random_residues(m, rng)
    _relatives(res, offs, q, rng)
    out = torch.full((len(lens),), -7, dtype=torch.int32, device="cuda")
    say("allocation-free, few rows, m=%d" % m)
    with sw.Database(res, offs) as db:
        for go, ge in ((10, 2), (10, 0)):       # windows of the long sequence; whole pairs
            for _ in range(2):
                out.fill_(-7)
                db.search_async_noalloc(torch.from_numpy(q).cuda(), B62, go, ge, out)
                torch.cuda.synchronize()
                _same(out.cpu().numpy(), ocpu.search(q, res, offs, B62, go, ge), (m, go, ge))


def test_noalloc_under_capture(sw):
    import torch
    res, offs, rng = _mix(5, 2000, 12, 9000)
    qs = [swinputs.random_residues(300, rng) for _ in range(3)]
    _relatives(res, offs, qs[1], rng)
    want = [ocpu.search(q, res, offs, B62, 10, 2) for q in qs]
    say("capture of the allocation-free search")
    with sw.Database(res, offs) as db:
        dq = torch.from_numpy(qs[0]).cuda()
        out = torch.full((len(offs) - 1,), -7, dtype=torch.int32, device="cuda")
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            db.search_async_noalloc(dq, B62, 10, 2, out, s)     # code objects loaded
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            db.search_async_noalloc(dq, B62, 10, 2, out, s)
        for turn in range(6):
            dq.copy_(torch.from_numpy(qs[turn % 3]))
            out.fill_(-7)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            _same(out.cpu().numpy(), want[turn % 3], ("replay", turn))
            db.search_async(dq, B62, 10, 2, out)                # the program's own work between
            torch.cuda.synchronize()
            _same(out.cpu().numpy(), want[turn % 3], ("eager", turn))


# batches: very long sequences against queries of one pass and of many, so that 16
# waves keep their own profile slots, and matrices that need the guard in bins whose
# boundary rows wrap
@pytest.mark.parametrize("hot", [False, True])
def test_batches_of_very_long_sequences(sw, hot):
    rng = np.random.default_rng(12)
    lens = np.concatenate([rng.integers(8192, 12000, 24), rng.integers(2048, 8192, 60),
                           rng.integers(20, 2047, 1500)]).astype(np.int64)
    res, offs = swinputs.make_database(rng.permutation(lens), rng)
    qs = [swinputs.random_residues(m, rng) for m in (30, 64, 129, 500, 1100, 2500)]
    for q in qs[2:5]:
        _relatives(res, offs, q, rng, 3)
    mat = B62
    if hot:
        mat = rng.integers(-128, 1, (24, 24)).astype(np.int8)
        mat[np.arange(24), np.arange(24)] = 127
    say("batch of very long sequences, hot %s" % hot)
    with sw.Database(res, offs) as db:
        for _ in range(2):
            got = db.search_batch(qs, mat, 12, 2)
            for q, row in zip(qs, got):
                _same(row, ocpu.search(q, res, offs, mat, 12, 2), len(q))
