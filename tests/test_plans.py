"""The host's rules for the packed kernels (csrc/plans.h), compiled and called:
which calls the 16-bit forms take, and that at the edge of the rules every value
of the recurrence stays where the kernels' maxima order integers."""
import numpy as np
import pytest

import plans_shim as plans
import swinputs
from test_drift_cells import drift_plan

B62 = swinputs.blosum62()
DNA = swinputs.dna_matrix(5, 4, -2)
TOP, GLOBAL, SEMI = 31743, 1, 2


def _hot():
    mat = np.random.default_rng(5).integers(-128, 1, (24, 24)).astype(np.int8)
    mat[np.arange(24), np.arange(24)] = 127
    return mat


def test_drift_rule_is_the_one_the_cell_model_checks():
    rng = np.random.default_rng(1)
    for _ in range(4000):
        mat = (B62, DNA, _hot())[int(rng.integers(3))]
        m, cols = int(rng.integers(1, 6000)), int(rng.choice([96, 400, 2048, 8192, 20000]))
        ge = int(rng.choice([0, 1, 2, 4, 10, 12, 13, 14, 28, 100]))
        go = ge + int(rng.choice([0, 8, 3000]))
        limit, R = int(rng.choice([0, 40, 2048])), int(rng.choice([12, 14, 16, 20, 32]))
        got = plans.drift(m, cols, R, mat, go, ge, limit)
        group, guard = drift_plan(m, cols, R, mat, go, ge, limit)
        assert got["group"] == group
        if group:
            assert bool(got["guard"]) == guard
            assert got["c2"] == min(go - ge, 2048) * 0x10001
            assert got["group2"] == (ge * R * group) * 0x10001 and ge * R * group < 65536


def test_drift_edge_at_the_default_limit():
    for R in (12, 14, 16, 18, 20):
        for m in (100, 700, 5000):
            assert plans.drift(m, 2048, R, B62, 12, 12)["group"] >= 1
            assert plans.drift(m, 2048, R, B62, 13, 13)["group"] == 0


def test_pair_bytes_hold_every_score():
    for mat in (B62, DNA, _hot(), np.full((24, 24), -128, np.int8)):
        lo, hi = int(mat.min()), int(mat.max())
        for limit in (0, 2048):
            for ge in list(range(0, 140)) + [1000, 5000, 100000]:
                f = plans.pair(mat, ge, limit)
                if f["add"] < 0:
                    continue
                assert 0 <= lo + f["add"] and hi + f["add"] <= 255
                assert f["add"] == 2 * ge + f["bias"] and 0 <= f["code_byte"] <= 255
                # a superstep's drift and what a score past the limit can gain
                assert 2560 + min(limit, 2048) + 136 * max(hi, 0) + ge * 88 <= TOP
    assert plans.pair(B62, 122)["add"] >= 0 and plans.pair(B62, 123)["add"] < 0


def _values(q, b, matrix, go, ge, mode, base, pad, pad_score, lanes=None):
    """Every 16-bit value of a global or semi-global matrix in its drift frame:
    base + ge * (row + column), the query's rows behind `pad` rows of the top
    border; b holds -1 where the sequence has ended.  lanes = R: the long-pair
    kernel's frame, in which (semi-global) the columns count from the superstep."""
    m, n = len(q), len(b)
    neg = -(1 << 40)
    w = lambda k: go + (k - 1) * ge if k > 0 else 0                     # noqa: E731
    H = np.array([-w(j) if mode == GLOBAL else 0 for j in range(n + 1)], np.int64)
    F = np.full(n + 1, neg, np.int64)
    cols = np.arange(n)
    low, high, c = [], [], go - ge
    for i in range(1, m + 1):
        row = i - 1 + pad
        off = (cols + row // lanes % 64) // 64 * 64 if lanes and mode == SEMI else 0
        tilde = lambda x, r=row: x + base + ge * (r + cols - off)       # noqa: E731
        sc = np.where(b >= 0, matrix[q[i - 1], np.maximum(b, 0)].astype(np.int64), pad_score)
        F = np.maximum(F - ge, H - go)                                  # F(i, j)
        d = H[:-1] + sc
        h = np.empty(n + 1, np.int64)
        h[0] = -w(i)                                                    # H(i, 0)
        # E(i, j) = max over k < j of H(i, k) - go - (j - k - 1) ge, where opening a
        # gap after a cell that came from E never pays
        g = np.concatenate([h[:1], np.maximum(d, F[1:])])
        e = np.maximum.accumulate(g + ge * np.arange(n + 1))[:-1] - go - ge * cols
        h[1:] = np.maximum(g[1:], e)
        for x in (tilde(d), tilde(h[1:]), tilde(h[1:]) - c, tilde(F[1:]), tilde(e)):
            low.append(int(x.min()))
            high.append(int(x.max()))
        H = h
    return min(low), max(high)


def _worst(matrix, m, n, rng):
    """Query and sequences that gain, and lose, the most."""
    a, b = np.unravel_index(int(np.argmax(matrix)), matrix.shape)
    x, y = np.unravel_index(int(np.argmin(matrix)), matrix.shape)
    yield np.full(m, a), np.full(n, b)
    yield np.full(m, x), np.full(n, y)
    yield np.full(m, a), np.concatenate([np.full(n // 2, b), np.full(n - n // 2, -1)])
    yield rng.integers(0, 20, m), rng.integers(0, 20, n)


def _edge(ok, lo, hi):
    """The largest value in [lo, hi] for which ok holds (ok(lo) does)."""
    while lo < hi:
        mid = (lo + hi + 1) // 2
        lo, hi = (mid, hi) if ok(mid) else (lo, mid - 1)
    return lo


# calls at the last query length, and with the last opening penalty, that the
# rule still gives to the packed forms
@pytest.mark.parametrize("mode", [GLOBAL, SEMI])
@pytest.mark.parametrize("go,ge,matrix,cols", [(10, 2, "b62", 700), (40, 10, "b62", 400),
                                               (12, 2, "hot", 260), (9, 0, "dna", 300)])
def test_mode_values_stay_in_range(mode, go, ge, matrix, cols):
    mat = {"b62": B62, "dna": DNA, "hot": _hot()}[matrix]
    rng = np.random.default_rng(go)
    strips = lambda m, g=go: plans.mode(m, cols, mat, g, ge, mode)["R"] > 0             # noqa: E731
    wave = lambda m, g=go, R=4: plans.mode_pairs(m, cols, mat, g, ge, mode, R)["add"] >= 0  # noqa: E731
    for ok, lanes, pad_score in ((strips, None, -64), (wave, 4, -2 * ge)):
        m = _edge(ok, 1, 600)
        g = _edge(lambda v: ok(m, v), go, 31000)
        for gap in (go, g):
            p = (plans.mode_pairs(m, cols, mat, gap, ge, mode, 4) if lanes
                 else plans.mode(m, cols, mat, gap, ge, mode))
            for q, b in _worst(mat, m, cols, rng):
                lo, hi = _values(q, b, mat, gap, ge, mode, p["base"], p["pad"], pad_score, lanes)
                assert 0 <= lo and hi <= TOP, (m, gap, lanes, lo, hi)


def test_pair_rows_fit_what_is_launched():
    for n_pass in (1, 2, 3, 8, 40):
        for W in (1, 8, 16):
            for grid in (1, 15, 256):
                for items in (grid, 4000):
                    for stride in (5000, 35_000, 1 << 24):
                        for have in (-1, 1, 7, 3000):
                            r = plans.rows(n_pass, W, grid, items, stride, have)
                            assert r["ring"] >= 1 and 1 <= r["grid"] <= grid
                            if n_pass == 1:
                                assert r["rows"] == 0 and r["grid"] == grid
                                continue
                            assert r["rows"] == r["ring"] * r["grid"]
                            if have > 0:
                                assert r["rows"] <= have
                                continue
                            assert r["grid"] == grid
                            assert r["rows"] <= max(min(items, 1024), (512 << 20) // (8 * stride))
    # the usual case holds every pair that the waves can be at
    assert plans.rows(2, 16, 15, 1000, 35_000) == {"ring": 9, "grid": 15, "rows": 135}


def test_pair_launch_leaves_cus_to_the_bins_and_fits():
    rng = np.random.default_rng(2)
    for _ in range(20000):
        m = int(np.exp(rng.uniform(0, 11)))
        items = float(int(np.exp(rng.uniform(0, 10))))
        longest = float(int(np.exp(rng.uniform(3, 13))))
        cols = items * longest * rng.uniform(0.05, 1.0)
        beside = float(rng.choice([0, 0, 1e-6, 1e-4, 1e-2]))
        rows, waves = int(rng.choice([0, 0, 2, 4, 8])), int(rng.choice([0, 0, 1, 2, 4, 8]))
        own, cus = bool(rng.integers(2)), int(rng.choice([256, 256, 32, 1]))
        bins = np.sort(rng.integers(96, 2048, int(rng.choice([0, 5, 400]))))[::-1] if beside else ()
        R, W, grid = plans.launch(m, items, cols, longest, beside, cus, rows, waves, own, bins)
        assert R in (2, 4, 8) and W in (1, 2, 4, 8, 16) and (not rows or R == rows)
        assert not waves or W == waves
        P = -(-m // (64 * R))
        assert plans.lds(R, W, P, own) <= 160 * 1024
        assert 1 <= grid <= items
        if W >= 8:      # one workgroup a CU, and CUs for the bins
            assert grid <= (max(1, cus * 7 // 8) if beside else cus)


def test_pair_launch_spreads_few_passes_over_the_device():
    # 47 residues, 881 windows of up to 4,402 columns beside 2 % of the work: every
    # wave filled would be 56 workgroups
    R, W, grid = plans.launch(47, 881, 3.2e6, 4402, 1.8e8 / 8.5e12)
    assert R == 2 and grid == 224
    # 300 pairs alone: as many CUs as there are
    for m in (977, 2000, 5000):
        assert plans.launch(m, 300, 5.5e6, 34971)[2] == 256
    # few pairs beside many bins keep to few CUs
    assert plans.launch(457, 355, 9.8e5, 7067, 3.2e10 / 8.5e12)[2] <= 48
    # bins that take as long as the pairs start at once: 142 of 400 columns, 960 pairs
    assert plans.launch(30, 960, 3.84e5, 400, 2.57e-5, bins=[400] * 142)[2] <= 256 - 142
    # a short query's wave has few rows, or its chain is longer than it has to be
    assert plans.launch(50, 16, 1.9e5, 35000, 1e-4, own=True)[0] == 2


def test_binary16_pairs_take_fewer_waves_for_many_short_pairs():
    # 20,001 plain sequences, 5,484 pairs of 529 columns on average, windows of 5,156
    assert plans.half_rows(977, 5484, 2.9e6, 5156, 4, 4) == (8, 2)
    assert plans.half_rows(2500, 5548, 2.9e6, 6808, 4, 4) == (8, 2)
    # long pairs, few of them: the shortest chain, as it was
    assert plans.half_rows(2500, 1494, 8.8e6, 6808, 4, 4) == (4, 4)
    assert plans.half_rows(977, 1, 35000, 35000, 4, 4) == (4, 4)


def test_binary16_pairs_keep_their_rows_where_others_are_slower():
    # {m, pairs, their columns, longest, bins' residues, form}: measured with the other
    # form that an estimate of full rounds names 1.14, 1.18, 1.18 and 1.30 times as long
    for m, items, cols, longest, beside, form in (
            (690, 3394, 1.38e7, 4845, 1.57e7, (4, 4)), (2500, 3458, 1.88e7, 6808, 1.55e7, (4, 4)),
            (1400, 1494, 7.33e6, 5615, 0, (8, 4)), (310, 1513, 2.39e6, 4433, 1.2e5, (2, 4))):
        assert plans.half_rows(m, items, cols, longest, *form, beside) == form, m
    # 100,000 plain sequences: the bins are the search (2.18 ms, 2.29 with 4 x 2)
    assert plans.half_rows(310, 2237, 3.03e6, 4433, 2, 4, 2.95e7) == (2, 4)
    # and 1.4 to 2.8 times shorter with other rows
    assert plans.half_rows(450, 5164, 2.8e6, 4585, 2, 4, 1.53e6) == (4, 2)
    assert plans.half_rows(450, 10000, 4e6, 400, 2, 4) == (8, 1)
    assert plans.half_rows(2000, 5548, 2.91e6, 6266, 8, 4, 1.34e6) == (8, 2)


def test_batches_bound_by_their_longest_half_bin_fill_the_simds():
    plain = dict(cols=5.6e5, longest=8188)       # 100,000 plain sequences
    # kernel ms of the forms, each forced, for two queries of a length
    for m, ms in ((144, {(12, 12): 2.94, (14, 12): 3.65, (16, 12): 4.03, (18, 12): 3.26,
                         (20, 12): 3.53, (12, 16): 3.22, (14, 16): 3.73, (24, 12): 4.06}),
                  (200, {(12, 12): 4.34, (14, 12): 4.22, (16, 12): 4.74, (18, 12): 4.17,
                         (20, 12): 4.87, (12, 16): 4.55, (14, 16): 4.73}),
                  (256, {(12, 12): 5.86, (14, 12): 5.15, (16, 12): 4.81, (18, 12): 5.33,
                         (20, 12): 5.76, (12, 16): 5.39, (14, 16): 5.25, (16, 16): 4.87}),
                  (400, {(12, 12): 8.87, (14, 12): 8.37, (16, 12): 8.42, (18, 12): 8.38,
                         (20, 12): 7.03, (12, 16): 8.39, (14, 16): 8.75, (16, 16): 7.87})):
        form = plans.batch([m, m], **plain)
        assert form in ms and ms[form] <= 1.12 * min(ms.values()), (m, form)
    # many queries: the work decides, and taller strips cost less a row
    assert plans.batch([50 + 215 * i for i in range(24)], **plain) in ((24, 12), (16, 16), (20, 12))
    assert plans.batch([300, 300], **plain, rows=14, waves=16) == (14, 16)
    assert plans.batch([300, 300], **plain, rows=32, waves=8) is None
