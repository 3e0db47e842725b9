"""Diagonal blocks of every width class of the block factorization (32-column
row blocks and tiles, tiles stepped over 8, 16 or 32 columns, one to eight
tiles, whole and ragged last tiles) in every method and storage precision,
against the oracle's factor, and the kept inverses through a solve without
refinement.

Matrices: dense, off-diagonal entries uniform in [-1, 1], |a_ii| = 2 n
(negative for every third row in L D L^T and L U), identity order: one
column block of width n up to 256, pieces above.  Their eigenvalues lie
within a factor 3 of 2 n in magnitude (Gershgorin: the off-diagonal row sums
are below n), so the factor's error is at most about its backward error:
(n + 1) u ||F||_F for the products, a small factor for the inverted tiles
and for the oracle's own rounding.  Bounds: 32 (n + 1) sqrt(n) u max|F|
elementwise, and 64 (n + 1) u for the componentwise backward error of the
unrefined solve (two triangular products)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

WIDTHS = [1, 2, 7, 8, 9, 16, 17, 31, 32, 33, 40, 63, 64, 65, 97, 128, 129, 160, 191, 224, 225, 250, 255, 256, 257, 400]


@pytest.mark.parametrize("method,precision", [("llt", "fp64"), ("llt", "fp32_ir"), ("ldlt", "fp64"), ("ldlt", "fp32_ir"),
                                              ("lu", "fp64"), ("lu", "fp32_ir")])
def test_widths(orc, method, precision):
    import torch
    from paper_1405_2636_amd import Solver
    u = 2.0 ** -53 if precision == "fp64" else 2.0 ** -24
    for n in WIDTHS:
        rng = np.random.default_rng(n)
        A = rng.uniform(-1, 1, (n, n))
        if method != "lu":
            A = np.tril(A) + np.tril(A, -1).T
        d = np.where((np.arange(n) % 3 == 1) & (method != "llt"), -2.0 * n, 2.0 * n)
        np.fill_diagonal(A, d)
        colptr = np.arange(n + 1, dtype=np.int64) * n
        rowind = np.tile(np.arange(n, dtype=np.int32), n)
        values = np.ascontiguousarray(A.T).ravel()   # column by column
        perm = np.arange(n, dtype=np.int32)
        sym = orc.analyze(n, colptr, rowind, user_perm=perm)
        F = {"llt": orc.factor, "ldlt": orc.factor_ldlt, "lu": orc.factor_lu}[method](sym, colptr, rowind, values)
        F = np.concatenate(F[:2]) if method == "lu" else F
        for fuse in ([True, False] if n <= 40 else [True]):
            print(method, precision, n, fuse, flush=True)
            s = Solver(n, colptr, rowind, method=method, precision=precision, user_perm=perm, ir_max_iter=0, fuse_small=fuse)
            s.factorize(torch.tensor(values, device="cuda"))
            G = s.factor_values().cpu().numpy()
            err = np.max(np.abs(G - F)) / np.max(np.abs(F))
            assert err <= 32 * (n + 1) * np.sqrt(n) * u, (n, fuse, err)
            x, info = s.solve(torch.tensor(rng.uniform(-1, 1, n), device="cuda"), raise_on_noconv=False)
            assert info["omega"] <= 64 * (n + 1) * u, (n, fuse, info)
