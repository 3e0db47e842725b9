"""Groups of tiny column blocks (a wave each, several per work item) with 33
to 64 panel rows, or more than 8 update tiles: the rows past 32 are products
with the block's inverse.  Such blocks are grouped on levels with at least
512 of them only, so every case holds more, of at most 8 and of 9 to 16
columns.

Systems: two leaves of w columns, uncoupled, and a root of r, dense
otherwise, many of each shape in one matrix, in this order.  A = L0 L0^T or
L0 D0 L0^T with L0's diagonal in [1, 2] and other entries uniform in [-1, 1]
/ sqrt(m), m = 2 w + r.

Bound for A - L D L^T: every entry is a sum of at most m products, formed in
FP64 and stored once per step in the factor's precision, at most m + 2
roundings of the sum of the magnitudes; the products with the inverse (a
condition number below 8) have eight times that: 8 (m + 2) u (|L||D||L^T|).
"""
import numpy as np
import pytest

from planted import unit_lower

pytestmark = pytest.mark.gpu


def _pattern(shapes):
    """Lower triangles by column; (colptr, rowind, first row of every system)."""
    rows, count, first = [], [], [0]
    for w, r in shapes:
        for c in range(2 * w + r):
            i = np.arange(c, 2 * w + r)
            i = i[(c >= w) | (i < w) | (i >= 2 * w)]
            rows.append(i + first[-1])
            count.append(len(i))
        first.append(first[-1] + 2 * w + r)
    return np.concatenate([[0], np.cumsum(count)]).astype(np.int64), np.concatenate(rows).astype(np.int32), np.array(first)


def _gather(mats, colptr, rowind, first):
    col = np.repeat(np.arange(len(colptr) - 1), np.diff(colptr))
    q = np.searchsorted(first, col, side="right") - 1
    out = np.empty(len(rowind))
    for s, M in enumerate(mats):
        lo, hi = colptr[first[s]], colptr[first[s + 1]]
        out[lo:hi] = M[rowind[lo:hi] - first[s], col[lo:hi] - first[s]]
    assert q[-1] == len(mats) - 1
    return out


def _mask(w, m):
    M = np.tril(np.ones((m, m)))
    M[w:2 * w, :w] = 0.0
    return M


def _unpack(sv, F, first):
    """Every system's panels as a dense lower matrix, original numbering."""
    out = [np.zeros((b - a, b - a)) for a, b in zip(first[:-1], first[1:])]
    for k in range(sv["ncblk"]):
        f, ld, o = int(sv["fcol"][k]), int(sv["stride"][k]), int(sv["panel_off"][k])
        w = int(sv["lcol"][k]) - f + 1
        rows = sv["perm"][np.concatenate([np.arange(sv["frow"][b], sv["lrow"][b] + 1)
                                          for b in range(sv["bptr"][k], sv["bptr"][k + 1])])]
        cols = sv["perm"][f:f + w]
        q = np.searchsorted(first, cols[0], side="right") - 1
        out[q][np.ix_(rows - first[q], cols - first[q])] = F[o:o + ld * w].reshape(w, ld).T
    return [np.tril(M) for M in out]


def _tall(sv):
    """Blocks that are grouped with 33 to 64 panel rows: (of at most 8 columns, of 9 to 16)."""
    lvl = np.zeros(sv["ncblk"], int)
    for k in range(sv["ncblk"]):
        for j in sv["utgt"][sv["uptr"][k]:sv["uptr"][k + 1]]:
            lvl[j] = max(lvl[j], lvl[k] + 1)
    w = sv["lcol"] - sv["fcol"] + 1
    tall = (w <= 16) & (sv["stride"] > 32) & (sv["stride"] <= 64)
    tall &= np.bincount(lvl[tall], minlength=lvl.max() + 1)[lvl] >= 512
    return (tall & (w <= 8)).sum(), (tall & (w > 8)).sum()


# (shapes, split width): panels of 33, 64, 33, 64, 47 rows; 14 facing blocks of 4
CASES = {"two_sizes": ([(5, 28), (8, 56), (9, 24), (16, 48), (13, 34)] * 230, 256),
         "many_targets": ([(4, 56)] * 1030 + [(3, 32)] * 10, 4)}


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("method,precision", [("llt", "fp64"), ("llt", "fp32_ir"), ("ldlt", "fp64"), ("ldlt", "fp32_ir")])
def test_tall(method, precision, case):
    import torch
    from paper_1405_2636_amd import Solver
    shapes, split = CASES[case]
    print("tall tiny blocks", method, precision, case, flush=True)
    rng = np.random.default_rng(5)
    colptr, rowind, first = _pattern(shapes)
    mats = []
    for w, r in shapes:
        m = 2 * w + r
        L = np.tril(rng.uniform(-1, 1, (m, m)), -1) / np.sqrt(m) * _mask(w, m) + np.diag(rng.uniform(1, 2, m))
        d = rng.choice([-1.0, 1.0], m) if method == "ldlt" else np.ones(m)
        mats.append((L * d) @ L.T)
    s = Solver(int(first[-1]), colptr, rowind, method=method, precision=precision, amalg_pct=0, split_width=split,
               user_perm=np.arange(first[-1], dtype=np.int32))
    sv, inf = s.symbolic(), s.info()
    few, more = _tall(sv)
    assert few + more >= 1024 and few >= 460 and (more >= 460 or split == 4)
    assert inf["ntasks"] < inf["ncblk"] - 0.4 * (few + more)   # (two of them per item)
    u = 2.0 ** -53 if precision == "fp64" else 2.0 ** -24
    for _ in range(2):
        s.factorize(torch.tensor(_gather(mats, colptr, rowind, first), device="cuda"))
        for A, L, (w, r) in zip(mats, _unpack(sv, s.factor_values().cpu().numpy(), first), shapes):
            d = np.diag(L).copy() if method == "ldlt" else np.ones(len(L))
            if method == "ldlt":
                np.fill_diagonal(L, 1.0)
            tol = 8 * (len(L) + 2) * u * ((abs(L) * abs(d)) @ abs(L).T)
            assert np.max(np.tril(abs(A - (L * d) @ L.T)) - tol * (1 + 2 ** -20)) <= 0, (w, r)


def test_tall_replaced_pivots(orc):
    """Static pivots in such blocks: A = L0 D0 L0^T in small integers with
    zero pivots whose columns of L0 are empty, the replacement a power of two:
    every step is exact, and the factor equals the oracle's bit for bit."""
    import torch
    from paper_1405_2636_amd import Solver
    shapes = [(5, 28), (16, 48), (9, 55)] * 350
    rng = np.random.default_rng(9)
    colptr, rowind, first = _pattern(shapes)
    mats = []
    for q, (w, r) in enumerate(shapes):
        m = 2 * w + r
        zeros = {q % w, w + q % (w - 1), 2 * w + q % r}
        L = unit_lower(rng, m, zeros, per_col=2) * _mask(w, m)
        d = rng.choice([-1.0, 1.0, 2.0, -2.0], m)
        d[list(zeros)] = 0.0
        mats.append((L * d) @ L.T)
    values = _gather(mats, colptr, rowind, first)
    eps = 2.0 ** -20 / np.max(np.abs(values))
    assert eps * np.max(np.abs(values)) == 2.0 ** -20
    kw = dict(amalg_pct=0, user_perm=np.arange(first[-1], dtype=np.int32))
    print("tall tiny blocks, replaced pivots", flush=True)
    s = Solver(int(first[-1]), colptr, rowind, method="ldlt", static_pivot_eps=eps, **kw)
    assert min(_tall(s.symbolic())) >= 300
    sym = orc.analyze(int(first[-1]), colptr, rowind, **kw)
    P, nrep = orc.factor_ldlt(sym, colptr, rowind, values, pivot_eps=eps, return_nrep=True)
    assert nrep == 3 * len(shapes)
    s.factorize(torch.tensor(values, device="cuda"))
    assert s.info()["pivots_replaced"] == nrep
    assert np.array_equal(s.factor_values().cpu().numpy(), P)
