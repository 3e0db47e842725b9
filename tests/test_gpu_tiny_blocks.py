"""Groups of tiny column blocks (at most 16 columns and 64 panel rows, up to
8 blocks of one dependency level per work item, a wave each): the factor of
a batch of small grids, enough of them for full and partial groups on the
lower levels and single blocks on the upper ones, against the oracle's
factor of the same block-diagonal matrix, factored twice.  L D L^T with the
sign of every second system turned (negative pivots).

Bound: every system is diagonally dominant (ghost edges) and a row of its
factor sums at most n terms, so the factor's error is at most a small multiple
of n u ||F||; 64 (n + 1) u max|F| elementwise, n the largest system's size,
holds it with room for the atomic updates' order."""
import numpy as np
import pytest

from gen import grid_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count,hi", [(900, 10), (250, 26)])   # small panels; panels past 32 rows
@pytest.mark.parametrize("method,precision", [("llt", "fp64"), ("llt", "fp32_ir"), ("ldlt", "fp64"), ("ldlt", "bf16x3_ir")])
def test_groups(orc, method, precision, count, hi):
    import torch
    from paper_1405_2636_amd import Solver
    ps = grid_batch(count, seed=77, lo=1, hi=hi)
    print("tiny blocks", method, precision, sum(p.n for p in ps), flush=True)
    s = Solver.batch([(p.n, p.colptr, p.rowind) for p in ps], method=method, precision=precision, graph=False, tune=False)
    off = np.concatenate([[0], np.cumsum([p.n for p in ps])])
    eoff = np.concatenate([[0], np.cumsum([p.nnz for p in ps])])
    colptr = np.concatenate([[0]] + [p.colptr[1:] + e for p, e in zip(ps, eoff)]).astype(np.int64)
    rowind = np.concatenate([p.rowind + o for p, o in zip(ps, off)]).astype(np.int32)
    values = np.concatenate([p.values * (-1 if method == "ldlt" and q % 2 else 1) for q, p in enumerate(ps)])
    n = int(off[-1])
    sym = orc.analyze(n, colptr, rowind)
    F = (orc.factor if method == "llt" else orc.factor_ldlt)(sym, colptr, rowind, values)
    inf = s.info()
    assert inf["nsmall"] > 1024 and inf["ntasks"] < inf["nsmall"]   # groups of several blocks
    u = 2.0 ** -53 if precision == "fp64" else 2.0 ** -24 if precision == "fp32_ir" else 2.0 ** -16
    for _ in range(2):
        s.factorize(torch.tensor(values, device="cuda"))
        G = s.factor_values().cpu().numpy()
        assert np.max(np.abs(G - F)) <= 64 * (max(p.n for p in ps) + 1) * u * np.max(np.abs(F))
    b = np.random.default_rng(3).uniform(-1, 1, n)
    x, info = s.solve(torch.tensor(b, device="cuda"))
    assert info["omega"] <= 1e-14
