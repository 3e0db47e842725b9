"""A block of 128 columns or more, alone on its level, whose panel has more
than 16384 rows below it (L U: 8192): too many for the block substitution,
its panel solves are 16-row wave tiles of the product with the inverse.

Matrix: the first block's panel dense, L0 (and U0) as in the factor, with
diagonals in [1, 2] and other entries uniform in [-1, 1] / sqrt(n); below it
twice the identity, which fills.  The first panel's residual is checked entry
by entry against 64 sqrt(w) u (|L||U|)_ij (sums of w products with roundings of
independent signs, eight standard deviations, times the condition number,
below 8, of the block whose inverse multiplies); all others through the
componentwise backward error of an unrefined solve, at most 8 sqrt(n) u."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("method,precision,split,n", [("llt", "fp64", 256, 16700), ("ldlt", "fp32_ir", 128, 16640),
                                                      ("lu", "fp64", 200, 8420)])
def test_long_panel(method, precision, split, n):
    import torch
    from paper_1405_2636_amd import Solver
    w = -(-n // -(-n // split))   # balanced pieces, the first one the widest
    gen = torch.Generator(device="cuda").manual_seed(n)
    opts = dict(generator=gen, device="cuda", dtype=torch.float64)

    def panel():
        m = (2 * torch.rand(n, w, **opts) - 1) / np.sqrt(n)
        m[:w] = torch.tril(m[:w], -1) + torch.diag(1 + torch.rand(w, **opts))
        return m

    L = panel()
    U = {"llt": lambda: L, "ldlt": lambda: L * torch.where(torch.arange(w, device="cuda") % 3 == 1, -1.0, 1.0),
         "lu": panel}[method]()
    Ac, Ar = L @ U[:w].T, U @ L[:w].T   # A's first columns, and rows transposed
    keep = torch.tril(torch.ones(n, w, dtype=torch.bool, device="cuda")) | (method == "lu")
    extra = w if method == "lu" else 0   # entries above the diagonal of a later column
    tail = torch.cat([Ar[w:, :extra], 2 * torch.ones(n - w, 1, dtype=torch.float64, device="cuda")], 1)
    values = torch.cat([Ac.T[keep.T], tail.ravel()])
    later = np.concatenate([np.tile(np.arange(extra), (n - w, 1)), np.arange(w, n)[:, None]], 1)
    rowind = np.concatenate([np.nonzero(keep.T.cpu().numpy())[1], later.ravel()]).astype(np.int32)
    count = np.concatenate([keep.sum(0).cpu().numpy(), np.full(n - w, extra + 1)])
    print("long panel", method, precision, n, w, flush=True)
    s = Solver(n, np.concatenate([[0], np.cumsum(count)]), rowind, method=method, precision=precision, split_width=split,
               user_perm=np.arange(n, dtype=np.int32), ir_max_iter=0, ir_tol=1.0, trace=True)
    sv = s.symbolic()
    assert sv["lcol"][0] == w - 1 and sv["stride"][0] == n and (sv["perm"] == np.arange(n)).all()
    s.factorize(values)
    _, k = s.trace()
    solves = (k[:, 0] == 1) & (k[:, 1] == 0)
    assert k[solves, 3].max() == 16 * (4 // -(-w // 64)) and not ((k[:, 0] == 4) & (k[:, 1] == 0)).any()
    assert ((k[:, 0] == 4) & (k[:, 1] > 0)).any()
    F = s.factor_values()
    P = F[:n * w].view(w, n).T.clone()
    G, H = P.clone(), P.clone()
    G[:w] = torch.tril(P[:w])
    if method != "llt":
        G[:w].fill_diagonal_(1.0)
    H = G if method == "llt" else G * torch.diagonal(P[:w])
    if method == "lu":
        pe = F.numel() // 2
        H = torch.cat([torch.triu(P[:w]).T, F[pe:pe + n * w].view(w, n).T[w:]])
    u = 2.0 ** -53 if precision == "fp64" else 2.0 ** -24
    tol = 64 * np.sqrt(w) * u
    assert bool(((G @ H[:w].T - Ac).abs() <= tol * (G.abs() @ H[:w].abs().T)).all())
    if method == "lu":
        assert bool(((H @ G[:w].T - Ar).abs() <= tol * (H.abs() @ G[:w].abs().T)).all())
    x, info = s.solve(torch.tensor(np.random.default_rng(1).uniform(-1, 1, n), device="cuda"))
    assert info["omega"] <= 8 * np.sqrt(n) * u, info
