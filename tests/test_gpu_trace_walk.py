"""GPU parity of the traceback's walk on the device at the edges of its tiles,
against the oracle's traceback."""
import sys

import numpy as np
import pytest

import oracle
import swinputs

pytestmark = pytest.mark.gpu

B62 = swinputs.blosum62()


@pytest.fixture(scope="module")
def sw():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2203_11100_amd as lib
    return lib


def _same(got, q, res, offs, go, ge):
    for al in got:
        b = res[offs[al["seq"]]:offs[al["seq"] + 1]]
        want = oracle.sw_gotoh_traceback(q, b, B62, go, ge)
        assert (al["score"], al["query_begin"], al["db_begin"], al["query_end"], al["db_end"],
                al["ops"]) == want, (al["seq"], len(b))


# whole copies of the query (diagonals of many tiles), copies with 63..200 residues
# left out or put in (gaps across tiles), for every code word the kernel leaves
@pytest.mark.parametrize("rows", [0, 2, 4, 8])
@pytest.mark.parametrize("m,go,ge", [(63, 10, 2), (64, 2, 0), (65, 1, 1), (500, 3, 0), (513, 12, 1)])
def test_long_diagonals_and_gaps(sw, rows, m, go, ge):
    rng = np.random.default_rng(m + rows)
    q = swinputs.random_residues(m, rng)
    seqs = [q, np.concatenate([swinputs.random_residues(77, rng), q])]
    for cut in (1, 63, 64, 65, 200):
        at = m // 3
        seqs.append(np.concatenate([q[:at], q[at + cut:]]))
        seqs.append(np.concatenate([q[:at], swinputs.random_residues(cut, rng), q[at:]]))
    offs = np.concatenate([[0], np.cumsum([len(s) for s in seqs])]).astype(np.int64)
    res = np.concatenate(seqs).astype(np.uint8)
    print("walk m=%d gaps %d/%d rows %d" % (m, go, ge, rows), file=sys.stderr, flush=True)
    with sw.Database(res, offs) as db:
        db.set_option(sw.SW_OPT_INTRA_ROWS, rows)
        _same(db.traceback(q, B62, go, ge, list(range(len(seqs)))), q, res, offs, go, ge)


# more runs than come down with the ends
def test_many_runs(sw):
    rng = np.random.default_rng(3)
    lens = rng.integers(250, 350, 300).astype(np.int64)
    res, offs = swinputs.make_database(lens, rng)
    q = swinputs.random_residues(300, rng)
    with sw.Database(res, offs) as db:
        got = db.traceback(q, B62, 0, 0, list(range(len(lens))))
    assert sum(len([1 for x, y in zip(a["ops"], a["ops"][1:]) if x != y]) for a in got) > 8192
    _same(got, q, res, offs, 0, 0)


# what a sequence's codes take beside its own columns: nothing for an empty one, and
# the columns between neighbours once
def test_code_memory_and_empty_sequences(sw):
    import torch
    rng = np.random.default_rng(8)
    lens = np.array([0, 12, 0, 40, 1, 0], np.int64)
    res, offs = swinputs.make_database(lens, rng)
    m = 1_000_000                                    # a column: a megabyte
    q = swinputs.random_residues(m, rng)
    with sw.Database(res, offs) as db:
        db.search(q[:100], B62, 10, 2)
        for seqs, columns in (([0, 2, 5, 0], 0), ([1, 0, 3, 4], 12 + 40 + 1 + 4 * 63)):
            before = torch.cuda.mem_get_info()[0]
            got = db.traceback(q, B62, 10, 2, seqs)
            used = before - torch.cuda.mem_get_info()[0]
            print("traceback of %s: %d MB" % (seqs, used / 1e6), file=sys.stderr, flush=True)
            assert used <= (columns + 80) * 1_000_448      # profile, runs, rounding
            for al, sid in zip(got, seqs):
                assert al["seq"] == sid
                if lens[sid] == 0:
                    assert (al["score"], al["query_begin"], al["query_end"], al["db_begin"],
                            al["db_end"], al["ops"]) == (0, -1, -1, -1, -1, "")
                else:
                    b = res[offs[sid]:offs[sid + 1]]
                    at = al["query_begin"] - 100 if al["query_begin"] > 100 else 0
                    part = q[at:al["query_end"] + 1]
                    want = oracle.sw_gotoh_traceback(part, b, B62, 10, 2)
                    assert al["score"] == want[0] and al["ops"] == want[5]
    # groups of neighbours, empty ones among them, equal each alone
    lens = np.array([70, 0, 200, 64, 0, 63, 1, 300], np.int64)
    res, offs = swinputs.make_database(lens, rng)
    q = swinputs.random_residues(130, rng)
    with sw.Database(res, offs) as db:
        some = [t for t in range(8) if lens[t]]
        _same(db.traceback(q, B62, 4, 1, some), q, res, offs, 4, 1)
        together = db.traceback(q, B62, 4, 1, list(range(8)) * 2)
        for t, al in enumerate(together):
            assert al == db.traceback(q, B62, 4, 1, [t % 8])[0]
