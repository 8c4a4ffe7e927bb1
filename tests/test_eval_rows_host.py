"""Host emulation of the row evaluation's words (csrc/eval.hip, RowCfg and
k_eval_rows): points and queries are packed with the constants of the source,
and the row that the point word and the query word select must stand for the
digits themselves, for every prime at the largest net the rows take (all digit
positions of the word in use)."""
import os
import re

import numpy as np
import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_0808_0487_amd", "csrc", "eval.hip")
LARGEST = {2: 26, 3: 16, 5: 10, 7: 9}


def row_cfg(p):
    body = re.search(r"struct RowCfg<%d> \{(.*?)\};" % p, open(SRC).read(), re.S).group(1)
    return {k: int(v) for k, v in re.findall(r"(\w+) = (\d+)", body)}


@pytest.mark.parametrize("p", [2, 3, 5, 7])
def test_words_select_the_row_of_the_digits(p):
    """Of a word: the first digits' difference b = (q0 - x0) mod p (p = 2: of
    two digits), and the first digit after them that differs."""
    c, m = row_cfg(p), LARGEST[p]
    K, ND, DB = c["K"], c["ND"], c["DB"]
    D = {2: 32, 3: 20, 5: 13, 7: 11}[p]
    g = np.random.default_rng(p)
    n = 4000
    X = g.integers(0, p, size=(m, n))
    Qd = np.concatenate([g.integers(0, p, size=(m, n)), g.integers(0, p, size=(D - m, n))])
    for i in range(n):  # agree with the point on a prefix of any length
        k = g.integers(K, m + 1)
        Qd[K:k, i] = X[K:k, i]
    hx, hq = np.zeros(n, dtype=np.uint64), np.zeros(n, dtype=np.uint64)
    for f in range(K, m):
        hx |= X[f].astype(np.uint64) << np.uint64(32 - DB * (f - K + 1))
    for f in range(K, K + ND):
        if f < D:
            hq |= Qd[f].astype(np.uint64) << np.uint64(32 - DB * (f - K + 1))
    if p == 2:
        hx |= ((X[0] * 2 + X[1]).astype(np.uint64) << np.uint64(4)) | np.uint64(1)
        hq |= (Qd[0] * 2 + Qd[1]).astype(np.uint64) << np.uint64(4)
        b = ((hx ^ hq) >> np.uint64(4)) & np.uint64(3)
        want_b = (X[0] * 2 + X[1]) ^ (Qd[0] * 2 + Qd[1])
    else:
        hx |= (X[0] + 1).astype(np.uint64)
        sel = hx & np.uint64(c["FMASK"])
        # byte 1 + x0 of the query's table holds (q0 - x0) mod p, byte 0 zero
        tab = np.zeros((n, 8), dtype=np.int64)
        for x0 in range(p):
            tab[:, 1 + x0] = (Qd[0] - x0) % p
        b = tab[np.arange(n), sel.astype(np.int64)]
        want_b = (Qd[0] - X[0]) % p
    assert np.array_equal(b.astype(np.int64), want_b)
    z = hx ^ hq
    assert np.all(z != 0)
    clz = 32 - np.frexp(z.astype(np.float64))[1]
    group = clz // DB
    Xd = np.concatenate([X, np.zeros((D - m, n), dtype=X.dtype)])
    diff = Xd[K:K + ND] != Qd[K:K + ND] if K + ND <= D else Xd[K:] != Qd[K:]
    first = np.where(diff.any(0), diff.argmax(0), ND)
    assert np.array_equal(np.minimum(group, ND), first)
