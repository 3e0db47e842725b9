"""More right-hand sides than one launch of the sweeps takes (2^18): the
sweeps run in parts, the last of 1 (which takes the item lists of a single
right-hand side), 3 or 9.  The unrefined solution of every right-hand side
against a dense solve in FP64.

Bound: the rows are dominant by a factor of two, so the condition number is
at most 3; a factorization and two sweeps of at most n terms a row leave an
error below 64 n u max|x|."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("extra", [1, 3, 9])
@pytest.mark.parametrize("method", ["llt", "lu"])
def test_parts(method, extra):
    import torch
    from paper_1405_2636_amd import Solver
    n, nrhs = 78, (1 << 18) + extra   # leaves of 3 (a small block), 33 and 2 columns, a root of 40
    rng = np.random.default_rng(extra)
    A = rng.uniform(-1, 1, (n, n))
    A[:3, 3:38] = A[3:38, :3] = A[3:36, 36:38] = A[36:38, 3:36] = 0.0
    if method == "llt":
        A = (A + A.T) / 2
    np.fill_diagonal(A, 0.0)
    np.fill_diagonal(A, 2 * np.maximum(np.abs(A).sum(0), np.abs(A).sum(1)) + 1)
    keep = A.T != 0.0
    print("many right-hand sides", method, nrhs, flush=True)
    s = Solver(n, np.concatenate([[0], np.cumsum(keep.sum(1))]), np.nonzero(keep)[1], method=method, amalg_pct=0,
               user_perm=np.arange(n, dtype=np.int32), ir_max_iter=0, ir_tol=1.0)
    s.factorize(torch.tensor(A.T[keep], device="cuda"))
    b = torch.rand(nrhs, n, generator=torch.Generator(device="cuda").manual_seed(extra), device="cuda", dtype=torch.float64)
    ref = torch.linalg.solve(torch.tensor(A), b.cpu().T).T
    x, _ = s.solve(b)
    err = (x.cpu() - ref).abs().amax(1)
    assert bool((err <= 64 * n * 2.0 ** -53 * ref.abs().amax(1)).all()), int(err.argmax())
