"""The drift form of the packed 16-bit cells and the strip stream of the
inter-task kernel, as models on the CPU.

Cells: every value carries base + ge * (row + column); the model computes
them with numpy uint16, the scores of a strip's rows against a batch of
sequences, with the range rule of the host (groups of strips whose drift
starts again, the guard) and checks scores against the oracle and every
value against 0 .. 31743, the range in which the kernel's maxima order
integers.

Stream: waves take the strips of a workgroup's bins round robin and wait for
the strip above through progress words; random interleavings check that a
strip reads a chunk only as the strip above left it, that every bin is scored
once and that every wave ends.
"""
import random

import numpy as np
import pytest

import swinputs
from oracle import cpu as ocpu

B62 = swinputs.blosum62()
BASE, TOP, EXACT = 2560, 31743, 2048


def drift_plan(m, cols, R, matrix, go, ge, limit):
    """The host's rule: (strips per group, guard), or (0, _) for the other form."""
    max_s = max(0, int(matrix.max()))
    top = TOP - BASE - 256
    score = max(min(-(-m // R) * R, cols) * max_s, limit)
    guarded = limit + (R + 8) * max_s

    def groups(highest):
        if ge == 0:
            return 1 << 30 if highest <= top else 0
        return int((top - highest) / ge - cols - R - 8) // R if top >= highest else 0
    g, guard = groups(score), False
    if g < 1:
        g, guard = groups(guarded), True
    return min(max(g, 0), -(-m // R)), guard


def drift_scores(q, seqs, matrix, go, ge, R, limit, plan):
    """uint16 model of the kernel: scores (or -1 at the limit) of each sequence."""
    group, guard = plan
    n = max(len(s) for s in seqs)
    cols = (n + 3) // 4 * 4
    b = len(seqs)
    code = np.full((b, cols), -1, np.int64)
    for k, s in enumerate(seqs):
        code[k, :len(s)] = s
    m, c = len(q), min(go - ge, EXACT)
    strips = -(-m // R)
    up_h = np.zeros((cols, b), np.int64)
    up_f = np.zeros((cols, b), np.int64)
    best = np.zeros(b, np.int64)
    seen = [TOP, 0]

    def keep(v):
        seen[0], seen[1] = min(seen[0], int(v.min())), max(seen[1], int(v.max()))
        return v
    for s in range(strips):
        ig = s % group
        z0 = BASE + ge * ig * R
        H = np.array([[z0 + ge * (k - 1)] * b for k in range(R)])
        E = np.array([[z0 + ge * k] * b for k in range(R)])
        A = np.zeros((R + 2, b), np.int64)
        sbest = np.zeros(b, np.int64)
        hdiag = np.full(b, z0 - 2 * ge)
        delta = 65535 if s == 0 else ge * R * group if ig == 0 else 0
        for j in range(cols):
            z = z0 + ge * j
            h_up, f_up = up_h[j].copy(), up_f[j].copy()
            if delta or guard:
                h_up = np.minimum(np.maximum(np.maximum(h_up - delta, 0), z - ge), z - ge + limit)
                f_up = np.minimum(np.maximum(f_up - delta, 0), z - ge + limit)
            hd, hdiag, F = hdiag, h_up, f_up
            for k in range(R):
                i = s * R + k
                sc = (np.where(code[:, j] >= 0, matrix[q[i], np.maximum(code[:, j], 0)], -64)
                      if i < m else np.full(b, -64))
                h = keep(np.maximum(np.maximum(hd + sc + 2 * ge, E[k]), F))
                keep(hd + sc + 2 * ge)
                t = keep(h - c)
                if k == 0 and not j & 1:
                    x = keep(np.maximum(A[1], h) - z)
                if j & 1:
                    below = H[k + 1] if k + 1 < R else np.zeros(b, np.int64)
                    A[k] = np.maximum(np.maximum(A[k + 2], h), below)
                    if k == 0:
                        sbest = np.maximum(np.maximum(sbest, x), keep(A[0] - z))
                E[k] = np.maximum(np.maximum(E[k], t), z + ge * (k + 1))
                F = np.maximum(F, t)
                hd = H[k].copy()
                H[k] = h
            up_h[j], up_f[j] = H[R - 1], F
            if guard and j % 4 == 3:
                over = sbest >= limit
                for k in range(R):
                    zk = z0 + ge * (j + 1 + k)
                    E[k][over], H[k][over], A[k][over] = zk, zk - ge, zk - ge
                hdiag = np.where(over, z0 + ge * (j + 1) - 2 * ge, hdiag)
        for k in range(1, R):
            sbest = np.maximum(sbest, A[k] - (z0 + ge * (cols - 1 + k)))
        best = np.maximum(best, sbest)
    assert 0 <= seen[0] and seen[1] <= TOP, seen
    return np.where(best < limit, best, -1)


@pytest.mark.parametrize("m,R,go,ge,limit,matrix", [
    (1, 12, 10, 2, 2048, "b62"), (29, 12, 12, 2, 2048, "b62"), (40, 14, 11, 1, 40, "b62"),
    (33, 16, 10, 0, 2048, "b62"), (45, 12, 120, 100, 2048, "b62"), (26, 14, 3000, 2, 2048, "b62"),
    (60, 12, 30, 28, 2048, "hot"), (70, 20, 10, 2, 2048, "hot"), (50, 12, 5, 5, 0, "b62")])
def test_drift_cells_match_the_oracle(m, R, go, ge, limit, matrix):
    rng = np.random.default_rng(m)
    mat = B62
    if matrix == "hot":      # scores that pass the limit within a few cells
        mat = rng.integers(-128, 128, (24, 24)).astype(np.int8)
        mat[3, 3] = 127
    q = swinputs.random_residues(m, rng)
    seqs = [swinputs.random_residues(int(n), rng) for n in rng.integers(1, 90, 24)]
    seqs[0] = q.copy()
    seqs[1] = np.repeat(q, 2)
    if matrix == "hot":
        q[:] = 3
        seqs[2] = np.full(80, 3, np.uint8)
    plan = drift_plan(m, 96, R, mat, go, ge, min(limit, EXACT))
    assert plan[0] >= 1
    got = drift_scores(q, seqs, mat, go, ge, R, min(limit, EXACT), plan)
    offs = np.concatenate([[0], np.cumsum([len(s) for s in seqs])]).astype(np.int64)
    want = ocpu.search(q, np.concatenate(seqs), offs, mat, go, ge)
    assert (got == np.where(want < min(limit, EXACT), want, -1)).all()
    # the drift starting again every strip, and the guard where it is not needed
    for other in ((1, plan[1]), (plan[0], True)):
        assert (drift_scores(q, seqs, mat, go, ge, R, min(limit, EXACT), other) == got).all()


DONE = (1 << 23) - 1


def run_stream(W, S, chunks, seed, workgroups, RING):
    """Random interleaving of the waves of some workgroups; raises on a wrong
    read, a bin scored twice or not at all, or no progress."""
    rng = random.Random(seed)
    queue, scored, word = [0], [0] * len(chunks), 1 << 32

    def behind(a, b):      # a < b as progress words
        return (a - b) % word >= word // 2

    def wave(G, w):
        n, s = divmod(w, S)
        k, before = 0, (w - 1) % W
        while True:
            here, there = (k << 23) % word, ((k if w else k - 1) << 23) % word
            slot, b = n % RING, -1
            if s == 0:
                while (k or w) and behind(G["prog"][before], there):
                    yield False
                if not G["end"]:
                    while G["free"][slot] != n:
                        yield False
                    b = queue[0]
                    queue[0] += 1
                    if b >= len(chunks):
                        b, G["end"] = -1, True
                    G["bin"][slot] = b
            else:
                while behind(G["prog"][before], there + 1):
                    yield False
                if not G["end"]:
                    b = G["bin"][slot]
            yield True
            if b < 0:
                G["prog"][w] = (here + DONE) % word
                return
            G["prog"][w] = here
            C = chunks[b]
            for c in range(-1, C):            # -1: the fetch of chunk 0 alone
                nxt = min(c + 1, C - 1)
                while s and behind(G["prog"][before], there + nxt + 1):
                    yield False
                if s and c + 1 < C:
                    assert G["rows"].get((b, nxt)) == s - 1, "chunk read out of turn"
                yield True
                if c >= 0:
                    G["rows"][b, c] = s
                    G["prog"][w] = (here + c + 1) % word
            G["fin"][slot] += 1
            if G["fin"][slot] == S:
                scored[b] += 1
                G["fin"][slot], G["free"][slot] = 0, n + RING
            s, n, k = (s + W) % S, n + (s + W) // S, k + 1

    waves = []
    for _ in range(workgroups):
        G = {"prog": [word - 1] * W, "bin": [None] * RING, "fin": [0] * RING,
             "free": list(range(RING)), "rows": {}, "end": False}
        waves += [(wave(G, w), rng.random() ** 3) for w in range(W)]
    idle = 0
    while waves:
        t = rng.randrange(len(waves))
        if rng.random() > waves[t][1] + 0.05:
            continue
        try:
            idle = 0 if next(waves[t][0]) else idle + 1
        except StopIteration:
            del waves[t]
        assert idle < 100_000, "no wave can go on"
    assert scored == [1] * len(chunks)


@pytest.mark.parametrize("W", [1, 2, 4, 8, 12, 16])
def test_strip_stream_scores_every_bin_once(W):
    for t in range(30):
        r = random.Random(100 * W + t)
        S = r.choice([1, 2, 3, 5, 7, 11, 12, 13, 16, 17, 31, 40])
        chunks = [r.choice([2, 3, 5, 8, 24]) for _ in range(r.randint(1, 12))]
        run_stream(W, S, chunks, t, r.choice([1, 1, 2, 3]), r.choice([4, 16]))
