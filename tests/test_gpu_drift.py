"""GPU parity of the inter-task kernel's two cell forms at the edges of the
rule that chooses between them, against the oracle."""
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


def _db(seed, top):
    """Short sequences of every length up to `top`, a few of them copies."""
    rng = np.random.default_rng(seed)
    lens = np.concatenate([[0, 1, 95, 96, 97, top, top - 1], rng.integers(1, 400, 500),
                           rng.integers(400, top, 60)]).astype(np.int64)
    res, offs = swinputs.make_database(lens, rng)
    return res, offs, rng


def _hot():
    """Entries from -128 to 127: a score passes the limit within 17 cells."""
    mat = np.random.default_rng(5).integers(-128, 1, (24, 24)).astype(np.int8)
    mat[np.arange(24), np.arange(24)] = 127
    return mat


# gaps from none to past what the drift form takes (2,048 columns: 13 and 14),
# and open penalties past the 16-bit range
@pytest.mark.parametrize("m,go,ge", [(1, 10, 2), (13, 10, 0), (300, 0, 0), (700, 13, 13),
                                     (700, 14, 14), (700, 300, 12), (333, 100000, 3),
                                     (333, 100000, 100000), (2500, 11, 1)])
@pytest.mark.parametrize("limit", [32767, 60])
def test_gap_ranges(sw, m, go, ge, limit):
    res, offs, rng = _db(m, 2047)
    q = swinputs.random_residues(m, rng)
    big = int(np.argmax(np.diff(offs)))
    n = min(m, 2047)
    res[offs[big]:offs[big] + n] = q[:n]           # a score up to the range's own
    say("m=%d gaps %d/%d limit %d" % (m, go, ge, limit))
    want = ocpu.search(q, res, offs, B62, go, ge)
    with sw.Database(res, offs) as db:
        db.set_option(sw.SW_OPT_OFFLOAD_BINS, 0)   # every bin in the inter-task kernel
        db.set_option(sw.SW_OPT_SAT_LIMIT, limit)
        got = db.search(q, B62, go, ge)
        st = db.stats()
    bad = np.nonzero(got != want)[0]
    assert len(bad) == 0, [(int(i), int(got[i]), int(want[i])) for i in bad[:5]]
    assert st["n_rescored"] == int((want >= min(limit, 2048)).sum())


# scores that would leave the 16-bit range (the guard), bins long enough that
# the rows' drift starts again, and longer than the drift form takes
@pytest.mark.parametrize("m,t_long,ge", [(64, 0, 1), (900, 0, 2), (1500, 6000, 2), (400, 20000, 2)])
def test_guarded_scores_and_long_bins(sw, m, t_long, ge):
    top = 2047 if t_long == 0 else t_long - 1
    res, offs, rng = _db(m, top)
    q = swinputs.random_residues(m, rng)
    lens = np.diff(offs)
    for i in np.argsort(lens)[-40::3]:             # copies of the query, repeated
        n = int(lens[i])
        res[offs[i]:offs[i] + n] = np.resize(q, n)
    say("guard: m=%d t_long=%d" % (m, t_long))
    for mat in (_hot(), B62):
        want = ocpu.search(q, res, offs, mat, 12, ge)
        with sw.Database(res, offs, long_threshold=t_long) as db:
            db.set_option(sw.SW_OPT_OFFLOAD_BINS, 0)
            got = db.search(q, mat, 12, ge)
            st = db.stats()
        bad = np.nonzero(got != want)[0]
        assert len(bad) == 0, [(int(i), int(got[i]), int(want[i])) for i in bad[:5]]
        assert st["n_rescored"] == int((want >= 2048).sum())


# batches: both cell forms, matrices with and without the guard in one launch
# (long bins), boundary rows given out round and round (a long bin fills them),
# queries of a single strip (more entries in flight than waves) and of many
@pytest.mark.parametrize("go,ge,matrix", [(10, 2, "b62"), (10, 0, "b62"), (12, 4, "b62"),
                                          (20, 14, "b62"), (12, 2, "hot")])
@pytest.mark.parametrize("lens", [[1, 7, 13], [5] * 40, [300, 23, 2600, 900, 24], [1500, 1400]])
def test_batches(sw, go, ge, matrix, lens):
    res, offs, rng = _db(sum(lens), 8191)          # default threshold: short and long bins
    qs = [swinputs.random_residues(m, rng) for m in lens]
    sizes = np.diff(offs)
    for i in np.argsort(sizes)[-30::3]:
        n = int(sizes[i])
        res[offs[i]:offs[i] + n] = np.resize(qs[0], n)
    mat = _hot() if matrix == "hot" else B62
    say("batch %s gaps %d/%d %s" % (lens[:5], go, ge, matrix))
    with sw.Database(res, offs) as db:
        got = db.search_batch(qs, mat, go, ge)
        for _ in range(2):                          # the captured graph again
            assert (db.search_batch(qs, mat, go, ge) == got).all()
    for q, row in zip(qs, got):
        want = ocpu.search(q, res, offs, mat, go, ge)
        bad = np.nonzero(row != want)[0]
        assert len(bad) == 0, [(int(i), int(row[i]), int(want[i])) for i in bad[:5]]


# global and semi-global: the packed form and, past its 16-bit range, the int32
# one; queries that fill their strips and that leave rows above them
@pytest.mark.parametrize("m", [1, 16, 42, 97, 640, 2300])
@pytest.mark.parametrize("go,ge,matrix", [(10, 2, "b62"), (0, 0, "b62"), (11, 1, "b62"),
                                          (40, 10, "b62"), (3000, 3, "b62"), (9000, 5, "b62"),
                                          (100000, 7, "b62"), (12, 2, "hot")])
def test_modes(sw, m, go, ge, matrix):
    res, offs, rng = _db(m + go, 2047)
    q = swinputs.random_residues(m, rng)
    sizes = np.diff(offs)
    for i in np.argsort(sizes)[-20::2]:
        n = int(sizes[i])
        res[offs[i]:offs[i] + n] = np.resize(q, n)
    mat = _hot() if matrix == "hot" else B62
    say("modes m=%d gaps %d/%d %s" % (m, go, ge, matrix))
    with sw.Database(res, offs) as db:
        for mode in ("global", "semiglobal"):
            got = db.search_mode(q, mat, go, ge, mode)
            want = ocpu.search_mode(q, res, offs, mat, go, ge, mode)
            bad = np.nonzero(got != want)[0]
            assert len(bad) == 0, (mode, [(int(i), int(got[i]), int(want[i])) for i in bad[:5]])
