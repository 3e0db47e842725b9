"""Update tiles larger than 64 x 64 (128 x 128 and 256 x 64) with inner
dimensions of 32 and more, of single and of merged pieces, in every method
and storage precision: 128 x 128 asked for (tile = 1: every level takes it),
and 256 x 64 on levels with too much work for 64 x 64 tiles.

Matrices: arrows, A = L0 U0 (L0 L0^T, L0 D0 L0^T), with leaves of w dense
columns, uncoupled to each other, and a dense root of r.  L0's and U0^T's
diagonals are in [1, 2], their other entries uniform in [-1, 1] / sqrt(K), K
the longest row: condition numbers are small, and the products carry as much
of A as the diagonals do.  Checked: A - L U of the GPU's factor, entry by
entry, in FP64.

Bound: a sum of K products with roundings of independent signs is off by at
most 8 sqrt(K) u times the sum of the magnitudes, (|L||U|)_ij, eight standard
deviations for the millions of entries; the panel solves multiply by inverted
diagonal blocks, whose condition number, below 8, multiplies that:
64 sqrt(K) u (|L||U|)_ij.  In split BF16 every product is off by 2^-16 of
itself besides: 64 * 2^-15 sqrt((L^2)(U^2))_ij."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


class Arrow:
    """A as blocks: Ac[q] leaf q's columns ((w + r) x w), Ar[q] its rows
    transposed, Ass the root; pattern and values by column (symmetric methods:
    the lower triangle)."""

    def __init__(self, torch, leaves, w, r, method, seed):
        self.leaves, self.w, self.r, self.n, self.method = leaves, w, r, leaves * w + r, method
        gen = torch.Generator(device="cuda").manual_seed(seed)
        opts = dict(generator=gen, device="cuda", dtype=torch.float64)

        def block(rows, cols):
            m = (2 * torch.rand(rows, cols, **opts) - 1) / np.sqrt(self.n)
            m[:cols] = torch.tril(m[:cols], -1) + torch.diag(1 + torch.rand(cols, **opts))
            return m

        shapes = [(w + r, w)] * leaves + [(r, r)]
        L = [block(*s) for s in shapes]
        if method == "llt":
            U = L
        elif method == "ldlt":
            U = [m * torch.where(torch.rand(m.shape[1], **opts) < 0.3, -1.0, 1.0) for m in L]
        else:
            U = [block(*s) for s in shapes]
        self.Ac, self.Ar, self.Ass = self.products(L, U)
        full = method == "lu"
        s0 = leaves * w
        # (columns as rows of the transposed blocks, what is kept of them, their first rows in A)
        parts = [(self.Ac[q].T, np.concatenate([np.arange(w) + q * w, np.arange(r) + s0]), w) for q in range(leaves)]
        root = torch.cat([a[w:].T for a in self.Ar] + [self.Ass]) if full else self.Ass
        parts.append((root.T, np.arange(0 if full else s0, self.n), r))
        rowind, count, values = [], [], []
        for At, rows, c in parts:
            keep = np.ones(At.shape, bool) if full else np.triu(np.ones(At.shape, bool))
            rowind.append(rows[np.nonzero(keep)[1]])
            count.append(keep.sum(1))
            values.append(At.contiguous()[torch.tensor(keep, device="cuda")])
        self.rowind = np.concatenate(rowind).astype(np.int32)
        self.colptr = np.concatenate([[0], np.cumsum(np.concatenate(count))]).astype(np.int64)
        self.values = torch.cat(values)

    def products(self, L, U):
        w = self.w
        Ac = [l @ u[:w].T for l, u in zip(L[:-1], U[:-1])]
        Ar = [u @ l[:w].T for l, u in zip(L[:-1], U[:-1])]
        Ass = L[-1] @ U[-1].T
        for l, u in zip(L[:-1], U[:-1]):
            Ass += l[w:] @ u[w:].T
        return Ac, Ar, Ass

    def blocks(self, torch, sv, panel):
        """The panels (panel(offset, stride, width): stride x width) as the
        leaves' (w + r) x w blocks and the root's square."""
        w, r, s0, perm = self.w, self.r, self.leaves * self.w, sv["perm"].astype(np.int64)
        assert (perm[s0:] == np.arange(s0, self.n)).all()
        out = [torch.zeros(w + r, w, dtype=torch.float64, device="cuda") for _ in range(self.leaves)]
        out.append(torch.zeros(r, r, dtype=torch.float64, device="cuda"))
        for k in range(sv["ncblk"]):
            f, wk = int(sv["fcol"][k]), int(sv["lcol"][k] - sv["fcol"][k] + 1)
            rows = perm[np.concatenate([np.arange(sv["frow"][b], sv["lrow"][b] + 1)
                                        for b in range(sv["bptr"][k], sv["bptr"][k + 1])])]
            P, cols = panel(int(sv["panel_off"][k]), int(sv["stride"][k]), wk), perm[f:f + wk]
            leaf = np.minimum(cols // w, self.leaves)   # (the last leaf and the root are one supernode)
            for q in np.unique(leaf):
                c, i = np.nonzero(leaf == q)[0], np.nonzero(rows >= q * w)[0]
                at = np.where((rows[i] < s0) | (q == self.leaves), rows[i] - q * w, rows[i] - s0 + w)
                out[q][torch.tensor(at, device="cuda")[:, None], torch.tensor(cols[c] - q * w, device="cuda")] = P[i][:, c]
        return out

    def error(self, torch, s, precision):
        """The largest |A - L U|_ij over its bound."""
        F, sv = s.factor_values(), s.symbolic()
        pe, w = s.info()["panel_entries"], self.w

        def lower(o, ld, wk):    # unit diagonal but for L L^T
            P = F[o:o + ld * wk].view(wk, ld).T.clone()
            P[:wk] = torch.tril(P[:wk])
            if self.method != "llt":
                P[:wk].fill_diagonal_(1.0)
            return P

        def upper(o, ld, wk):    # U^T
            P = F[o:o + ld * wk].view(wk, ld).T
            if self.method == "llt":
                return lower(o, ld, wk)
            if self.method == "ldlt":
                return lower(o, ld, wk) * torch.diagonal(P[:wk])
            return torch.cat([torch.triu(P[:wk]).T, F[pe + o:pe + o + ld * wk].view(wk, ld).T[wk:]])

        L, U = self.blocks(torch, sv, lower), self.blocks(torch, sv, upper)
        u = 2.0 ** -53 if precision == "fp64" else 2.0 ** -24
        mag = self.products([m.abs() for m in L], [m.abs() for m in U])
        sq = self.products([m * m for m in L], [m * m for m in U])
        got = self.products(L, U)
        worst = 0.0
        for g, a, m, v in zip(*([*p[0], *(p[1] if self.method == "lu" else []), p[2]]
                                for p in (got, (self.Ac, self.Ar, self.Ass), mag, sq))):
            tol = 64 * np.sqrt(self.n) * u * m
            if precision == "bf16x3_ir":
                tol += 64 * 2.0 ** -15 * torch.sqrt(v)
            worst = max(worst, float(((g - a).abs() / tol).max()))
        return worst


def _factor(torch, a, method, precision, **kw):
    from paper_1405_2636_amd import Solver
    print("wide tiles", method, precision, a.leaves, a.w, a.r, kw, flush=True)
    s = Solver(a.n, a.colptr, a.rowind, method=method, precision=precision, amalg_pct=0,
               user_perm=np.arange(a.n, dtype=np.int32), trace=True, **kw)
    s.factorize(a.values)
    t, k = s.trace()
    sv = s.symbolic()
    width = sv["lcol"] - sv["fcol"] + 1
    wide = (k[:, 0] == 2) & (k[:, 3] > 64 * 64) & (width[k[:, 1]] >= 32)
    return s, t, k, wide


MODES = [("llt", "fp64"), ("llt", "fp32_ir"), ("llt", "bf16x3_ir"), ("ldlt", "fp64"), ("ldlt", "fp32_ir"),
         ("ldlt", "bf16x3_ir"), ("lu", "fp64"), ("lu", "fp32_ir")]


@pytest.mark.parametrize("opts", [dict(merge_split=1), dict(merge_split=4), dict(deterministic=True)])
@pytest.mark.parametrize("method,precision", MODES)
def test_asked_for(method, precision, opts):
    import torch
    for leaves, w, r, split in ((5, 150, 301, 64), (3, 45, 517, 256), (9, 33, 130, 256)):
        a = Arrow(torch, leaves, w, r, method, 7 + w)
        s, _, k, wide = _factor(torch, a, method, precision, tile=1, split_width=split, **opts)
        assert wide.any()
        assert a.error(torch, s, precision) <= 1.0


# (leaves, columns of a leaf, root): more than 8192 tiles of 64 x 64 (FP32: 1024) on the leaves' two levels
@pytest.mark.parametrize("method,precision,leaves,w,r,two_per_cu", [
    ("llt", "fp64", 40, 512, 1300, True), ("ldlt", "fp64", 40, 300, 1310, False), ("lu", "fp64", 20, 300, 1310, False),
    ("llt", "fp32_ir", 12, 300, 933, False), ("llt", "bf16x3_ir", 12, 300, 933, False),
    ("ldlt", "fp32_ir", 12, 300, 933, False), ("ldlt", "bf16x3_ir", 12, 300, 933, False),
    ("lu", "fp32_ir", 12, 300, 933, False)])
def test_default_shape(method, precision, leaves, w, r, two_per_cu):
    """256 x 64 on levels with many tiles, merged pieces among them; work
    enough for two workers on a CU in the first case."""
    import torch
    a = Arrow(torch, leaves, w, r, method, r)
    s, t, k, wide = _factor(torch, a, method, precision)
    assert k[wide, 3].max() == 256 * 64
    if two_per_cu:   # items in work at once
        at = np.concatenate([t[:, 1], t[:, 2]])
        step = np.concatenate([np.ones(len(t), int), -np.ones(len(t), int)])
        order = np.lexsort((step, at))
        assert np.cumsum(step[order]).max() > torch.cuda.get_device_properties(0).multi_processor_count
    assert a.error(torch, s, precision) <= 1.0
