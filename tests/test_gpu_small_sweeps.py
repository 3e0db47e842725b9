"""Small blocks in the triangular sweeps (width <= 32, at most 128 panel
rows): tiny ones (width <= 8, at most 32 panel rows) by 16 lanes, the others
by a wave, at the edges of both, in one block-diagonal matrix.  A system is
two leaves of w columns and a root of r, all dense but for the leaves' zero
coupling, in this order (no amalgamation), so its leaves are blocks of width
w with r rows below.  Checked through an unrefined solve (no step to hide an
error) against dense solves in FP64, for blocks of 1, 4 and 8 right-hand
sides, full and partial.

Bound: the rows are dominant by a factor of two, so the condition number is
at most 3; a factorization and two sweeps of at most m = 160 terms a row
leave an error below 64 m u max|x|."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

# (w, r): widths and panel rows at and next to 8, 16, 32 and 32, 64, 128
SHAPES = [(1, 1), (1, 31), (2, 15), (7, 25), (8, 24), (8, 8), (8, 25), (9, 23), (3, 60), (8, 120), (9, 1), (16, 16),
          (15, 64), (17, 65), (31, 97), (32, 96), (32, 97), (33, 95), (32, 1), (25, 63), (30, 34)]


def _system(w, r, rng, sym):
    n = 2 * w + r
    A = rng.uniform(-1, 1, (n, n))
    A[:w, w:2 * w] = A[w:2 * w, :w] = 0.0
    if sym:
        A = (A + A.T) / 2
    np.fill_diagonal(A, 0.0)
    np.fill_diagonal(A, 2 * np.maximum(np.abs(A).sum(0), np.abs(A).sum(1)) + 1)
    return A


def _check(shapes, method, precision, nrhs, m0):
    import torch
    from paper_1405_2636_amd import Solver
    rng = np.random.default_rng(nrhs)
    mats = [_system(w, r, rng, method != "lu") * (-1 if method == "ldlt" and q % 2 else 1)
            for q, (w, r) in enumerate(shapes)]
    A = sp.csc_matrix(sp.block_diag(mats))
    A.sort_indices()
    n = A.shape[0]
    s = Solver(n, A.indptr, A.indices, method=method, precision=precision, amalg_pct=0, user_perm=np.arange(n, dtype=np.int32),
               ir_max_iter=0, ir_tol=1.0)
    s.factorize(torch.tensor(A.data, device="cuda"))
    b = rng.uniform(-1, 1, (nrhs, n))
    x, _ = s.solve(torch.tensor(b, device="cuda"))
    x = x.cpu().numpy()
    u = 2.0 ** -53 if precision == "fp64" else 2.0 ** -24
    o = 0
    for (w, r), M in zip(shapes, mats):
        m = len(M)
        ref = np.linalg.solve(M, b[:, o:o + m].T).T
        assert np.max(np.abs(x[:, o:o + m] - ref)) <= 64 * max(m0, m) * u * np.max(np.abs(ref)), (w, r)
        o += m


MODES = pytest.mark.parametrize("method,precision", [("llt", "fp64"), ("ldlt", "fp64"), ("lu", "fp64"), ("llt", "fp32_ir"),
                                                     ("ldlt", "fp32_ir"), ("lu", "fp32_ir")])


@pytest.mark.parametrize("nrhs", [1, 2, 4, 5, 8, 13, 17])
@MODES
def test_shapes(method, precision, nrhs):
    print("small sweeps", method, precision, nrhs, flush=True)
    _check(SHAPES, method, precision, nrhs, 160)


@pytest.mark.parametrize("many", [0, 1])
@pytest.mark.parametrize("nrhs", [1, 3, 8, 17])
@MODES
def test_wide(method, precision, nrhs, many):
    """Wider blocks, next to multiples of 16 and 64: the diagonal and
    off-diagonal steps, on levels of few blocks and of many."""
    print("wide blocks", method, precision, nrhs, many, flush=True)
    _check([(47, 33), (64, 65), (65, 200), (130, 65)] + [(33, 40)] * (64 * many), method, precision, nrhs, 0)
