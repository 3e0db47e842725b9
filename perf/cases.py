"""The work that programs have this solver do, as measurable cases.

Four kinds, each through the package's public entry points:

* ``step``: the values of an analysed matrix change, and it is solved with
  them (a Newton or time step): ``Solver.factorize`` then ``Solver.solve``;
* ``solve``: the factor stays and new right-hand sides come in (a linear
  time loop, a preconditioner, many load cases): ``Solver.solve`` or
  ``Solver.solve_noalloc``;
* ``batch``: many small independent systems analysed as one handle, all of
  them factored and solved at once: ``Solver.batch``;
* ``adjoint``: a differentiable solve, forward and backward:
  ``solve_autograd``.

The matrices: finite-volume diffusion with a lognormal coefficient per cell
on 2-D and 3-D grids (symmetric positive definite), convection-diffusion
(unsymmetric) and clamped trilinear elasticity with a lognormal modulus per
element (three unknowns per node).  Their sizes run from the 64 x 64 grid to
the 100^3 grid, with odd and unequal sides.
"""
import numpy as np
import torch

from paper_1405_2636_amd import Solver, solve_autograd


def listed():
    return [
        # the smallest call: one 64 x 64 grid, bound by launches and the length of its dependency chain
        dict(name="step_grid2d_64", kind="step", op="diffusion", nx=64, ny=64, nz=1,
             method="llt", precision="fp64", nrhs=1),
        # a whole 2-D problem: little arithmetic per unknown, many narrow column blocks
        dict(name="step_grid2d_701x503", kind="step", op="diffusion", nx=701, ny=503, nz=1,
             method="llt", precision="fp64", nrhs=1),
        # an ordinary 3-D time step with uneven sides
        dict(name="step_grid3d_41x37x43", kind="step", op="diffusion", nx=41, ny=37, nz=43,
             method="llt", precision="fp64", nrhs=1),
        # the benchmark's size: 1e6 unknowns, 3.8e12 flops
        dict(name="step_grid3d_100", kind="step", op="diffusion", nx=100, ny=100, nz=100,
             method="llt", precision="fp64", nrhs=1),
        # the factor held in FP32, FP64 accuracy by refinement
        dict(name="step_grid3d_63x65x61_f32", kind="step", op="diffusion", nx=63, ny=65, nz=61,
             method="llt", precision="fp32_ir", nrhs=1),
        # split-BF16 products, the fastest factorization of a large problem
        dict(name="step_grid3d_80_bf16x3", kind="step", op="diffusion", nx=80, ny=80, nz=80,
             method="llt", precision="bf16x3_ir", nrhs=1),
        # unsymmetric transport with a few right-hand sides
        dict(name="step_convection_50x47x49_lu", kind="step", op="convection", nx=50, ny=47, nz=49,
             method="lu", precision="fp64", nrhs=4),
        # structural analysis: eight load cases, L D L^T
        dict(name="step_elastic_18x20x19_ldlt", kind="step", op="elastic", nx=18, ny=20, nz=19,
             method="ldlt", precision="fp64", nrhs=8),
        # many small systems at once, sides 16 to 96
        dict(name="batch_256", kind="batch", nsys=256, lo=16, hi=96, mix=7, precision="fp64"),
        # a linear time loop: one right-hand side per step, the factor kept
        dict(name="solve_grid3d_72x70x69", kind="solve", op="diffusion", nx=72, ny=70, nz=69,
             method="llt", precision="fp64", nrhs=1, noalloc=False),
        # many load cases on one factor, not a multiple of the block of right-hand sides
        dict(name="solve_grid3d_48_13rhs", kind="solve", op="diffusion", nx=48, ny=48, nz=48,
             method="llt", precision="fp64", nrhs=13, noalloc=False),
        # inverse problem: gradients with respect to the values and the right-hand side
        dict(name="adjoint_grid3d_36x35x34", kind="adjoint", op="diffusion", nx=36, ny=35, nz=34,
             method="llt", precision="fp64", nrhs=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _sides(rng, op):
    """Sides of a grid: 2-D 20 to 700, 3-D 10 to 80, elasticity 5 to 26 free nodes, each side by itself within 20%."""
    if op == "elastic":
        s, dim = _log_int(rng, 6, 24), 3
    else:
        dim = rng.choice((2, 3, 3))
        s = _log_int(rng, 24, 640) if dim == 2 else _log_int(rng, 11, 74)
    side = [max(4, int(round(s * rng.uniform(0.83, 1.08)))) for _ in range(dim)]
    return side + [1] * (3 - dim)


def draw(rng):
    kind = rng.choice(("step", "step", "step", "solve", "solve", "batch", "adjoint"))
    if kind == "batch":
        lo = rng.randint(8, 24)
        return dict(kind="batch", nsys=_log_int(rng, 8, 400), lo=lo, hi=rng.randint(lo + 8, 96),
                    mix=rng.randint(0, 1 << 20), precision=rng.choice(("fp64", "fp64", "fp32_ir")))
    if kind == "adjoint":
        nx, ny, nz = _sides(rng, "diffusion")
        return dict(kind="adjoint", op="diffusion", nx=nx, ny=ny, nz=nz, method=rng.choice(("llt", "ldlt")),
                    precision=rng.choice(("fp64", "fp32_ir")), nrhs=rng.choice((1, 1, 3)))
    op = rng.choice(("diffusion", "diffusion", "convection", "elastic"))
    nx, ny, nz = _sides(rng, op)
    method = "lu" if op == "convection" else rng.choice(("llt", "ldlt"))
    precision = rng.choice(("fp64", "fp64", "fp32_ir", "bf16x3_ir"))
    nrhs = rng.choice((1, 1, 1, 2, 4, 8, _log_int(rng, 3, 24)))
    case = dict(kind=kind, op=op, nx=nx, ny=ny, nz=nz, method=method, precision=precision, nrhs=nrhs)
    if kind == "solve":
        n = nx * ny * nz * (3 if op == "elastic" else 1)
        case["noalloc"] = n * nrhs < 1_000_000 and rng.random() < 0.3
    return case


# ---------------------------------------------------------------- matrices
# A matrix is held as a table: row c of `near` lists, in ascending order, the
# rows that column c may have (-1: outside the grid), and `val` their values.
def _grid_near(nx, ny, nz):
    """The grid neighbours of every cell (x fastest), the cell itself among them, ascending."""
    i = np.arange(nx * ny * nz, dtype=np.int64)
    x, y, z = i % nx, i // nx % ny, i // (nx * ny)
    cols = []
    for ok, step in ((z > 0, -nx * ny), (y > 0, -nx), (x > 0, -1), (i >= 0, 0), (x < nx - 1, 1), (y < ny - 1, nx),
                     (z < nz - 1, nx * ny)):
        if nz > 1 or abs(step) != nx * ny or step == 0:
            cols.append(np.where(ok, i + step, -1))
    return np.stack(cols, 1)


def _node_near(mx, my, mz):
    """The unknowns coupled to every unknown of a trilinear mesh of mx x my x mz free nodes, three each."""
    i = np.arange(mx * my * mz, dtype=np.int64)
    x, y, z = i % mx, i // mx % my, i // (mx * my)
    cols = []
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                ok = (x + dx >= 0) & (x + dx < mx) & (y + dy >= 0) & (y + dy < my) & (z + dz >= 0) & (z + dz < mz)
                node = i + dx + mx * (dy + my * dz)
                cols += [np.where(ok, 3 * node + e, -1) for e in range(3)]
    return np.repeat(np.stack(cols, 1), 3, axis=0)


def _near(case):
    return (_node_near if case["op"] == "elastic" else _grid_near)(case["nx"], case["ny"], case["nz"])


def _stiffness(nu=0.3):
    """24 x 24 stiffness of the unit trilinear cube with unit modulus (2 x 2 x 2 Gauss points)."""
    lam, mu = nu / ((1 + nu) * (1 - 2 * nu)), 0.5 / (1 + nu)
    elast = np.zeros((6, 6))
    elast[:3, :3] = lam
    elast[range(6), range(6)] += [2 * mu] * 3 + [mu] * 3
    corner = [((a >> 0) & 1, (a >> 1) & 1, (a >> 2) & 1) for a in range(8)]
    out = np.zeros((24, 24))
    pts = (0.5 - 0.5 / 3 ** 0.5, 0.5 + 0.5 / 3 ** 0.5)
    for p in ((u, v, w) for u in pts for v in pts for w in pts):
        strain = np.zeros((6, 24))
        for a, c in enumerate(corner):
            f = [p[d] if c[d] else 1 - p[d] for d in range(3)]
            s = [1.0 if c[d] else -1.0 for d in range(3)]
            gx, gy, gz = s[0] * f[1] * f[2], f[0] * s[1] * f[2], f[0] * f[1] * s[2]
            strain[:, 3 * a:3 * a + 3] = [[gx, 0, 0], [0, gy, 0], [0, 0, gz], [0, gz, gy], [gz, 0, gx], [gy, gx, 0]]
        out += strain.T @ elast @ strain / 8
    return (out + out.T) / 2


def _elastic_values(mx, my, mz, gen):
    """Values of the table of `_node_near`, modulus lognormal(0, 0.5) per element, the outer nodes clamped."""
    modulus = torch.exp(0.5 * torch.randn((mz + 1, my + 1, mx + 1), generator=gen, dtype=torch.float64, device="cuda"))
    ke = torch.tensor(_stiffness(), device="cuda")
    val = torch.zeros((mz, my, mx, 3, 27, 3), dtype=torch.float64, device="cuda")
    corner = [((a >> 0) & 1, (a >> 1) & 1, (a >> 2) & 1) for a in range(8)]
    for b, cb in enumerate(corner):      # the column's node
        x, y, z = (1 - cb[0]), (1 - cb[1]), (1 - cb[2])
        part = modulus[z:z + mz, y:y + my, x:x + mx, None, None]
        for a, ca in enumerate(corner):  # the row's node
            off = (ca[0] - cb[0] + 1) + 3 * ((ca[1] - cb[1] + 1) + 3 * (ca[2] - cb[2] + 1))
            val[..., off, :] += part * ke[3 * a:3 * a + 3, 3 * b:3 * b + 3].T
    return val.reshape(3 * mx * my * mz, 81)


def _diffusion_values(near, gen, faces):
    """Harmonic-mean face weights of a lognormal(0, 0.5) coefficient per cell; a missing neighbour is a Dirichlet face."""
    coef = torch.exp(0.5 * torch.randn(near.shape[0], generator=gen, dtype=torch.float64, device="cuda"))
    here = coef[:, None]
    there = torch.where(near >= 0, coef[near.clamp(min=0)], here)
    weight = 2 * here * there / (here + there)
    own = near == torch.arange(near.shape[0], device="cuda")[:, None]
    weight = torch.where(own, torch.zeros_like(weight), weight)
    val = torch.where(own, weight.sum(1, keepdim=True).expand_as(weight), -weight)
    assert near.shape[1] == faces + 1
    return torch.where(near >= 0, val, torch.zeros_like(val))


def _convection_values(near, gen, faces):
    """Central differences: row i couples to its upper neighbour by -1 + b/2 and to its lower one by -1 - b/2."""
    half = faces // 2
    vel = torch.rand((near.shape[0], half), generator=gen, dtype=torch.float64, device="cuda") - 0.5
    val = torch.zeros(near.shape, dtype=torch.float64, device="cuda")
    val[:, half] = float(faces)
    src = near.clamp(min=0)
    for k in range(half):
        axis = half - 1 - k              # column k of the table is the lower neighbour along `axis`
        # table entry (row near[c, k], column c): seen from that row, c is its upper neighbour
        val[:, k] = -1 + 0.5 * vel[src[:, k], axis]
        val[:, 2 * half - k] = -1 - 0.5 * vel[src[:, 2 * half - k], axis]
    return torch.where(near >= 0, val, torch.zeros_like(val))


def _values(case, near, gen):
    if case["op"] == "elastic":
        return torch.where(near >= 0, _elastic_values(case["nx"], case["ny"], case["nz"], gen), 0.0)
    faces = 6 if case["nz"] > 1 else 4
    return (_convection_values if case["op"] == "convection" else _diffusion_values)(near, gen, faces)


def _csc(near, lower=False):
    """Compressed columns of a table, and which of its entries are stored."""
    keep = near >= 0
    if lower:
        keep &= near >= np.arange(near.shape[0])[:, None]
    colptr = np.zeros(near.shape[0] + 1, np.int64)
    np.cumsum(keep.sum(1), out=colptr[1:])
    return colptr, near[keep].astype(np.int32), keep


def _batch_sides(case):
    rng = np.random.default_rng(case["mix"])
    return [(int(a), int(b)) for a, b in rng.integers(case["lo"], case["hi"] + 1, (case["nsys"], 2))]


def _batch_near(case):
    """The members' tables and one table of them all."""
    parts, whole, off = [], [], 0
    for nx, ny in _batch_sides(case):
        t = _grid_near(nx, ny, 1)
        parts.append(t)
        whole.append(np.where(t >= 0, t + off, -1))
        off += t.shape[0]
    return parts, np.concatenate(whole)


def _gen(seed):
    return torch.Generator("cuda").manual_seed(int(seed))


def _inputs(case, seed, near):
    """The table's values, the right-hand side(s) and, for the adjoint, the gradient that comes in."""
    gen, t = _gen(seed), torch.as_tensor(near, device="cuda")
    val = _diffusion_values(t, gen, 4) if case["kind"] == "batch" else _values(case, t, gen)
    nrhs = case.get("nrhs", 1)
    shape = (near.shape[0],) if nrhs == 1 else (nrhs, near.shape[0])
    b, g = (2 * torch.rand(shape, generator=gen, dtype=torch.float64, device="cuda") - 1 for _ in range(2))
    return val, b, g


def prepare(case, seed):
    if case["kind"] == "batch":
        parts, near = _batch_near(case)
        solver = Solver.batch([(t.shape[0],) + _csc(t)[:2] for t in parts], precision=case["precision"])
        keep = near >= 0
    else:
        near = _near(case)
        colptr, rowind, keep = _csc(near, lower=case["kind"] == "adjoint")
        solver = Solver(near.shape[0], colptr, rowind, method=case["method"], precision=case["precision"])
    val, b, g = _inputs(case, seed, near)
    values = val[torch.as_tensor(keep, device="cuda")]
    if case["kind"] == "solve":
        solver.factorize(values)
    if case["kind"] == "adjoint":
        values.requires_grad_()
        b.requires_grad_()
    return dict(kind=case["kind"], noalloc=case.get("noalloc", False), solver=solver, values=values, b=b, g=g)


def run(state):
    solver, values, b = state["solver"], state["values"], state["b"]
    if state["kind"] == "adjoint":
        x = solve_autograd(solver, values, b)
        gv, gb = torch.autograd.grad(x, (values, b), state["g"])
        return {"x": x.detach(), "grad_values": gv, "grad_b": gb}
    if state["kind"] != "solve":
        solver.factorize(values)
    x, _ = (solver.solve_noalloc if state["noalloc"] else solver.solve)(b.clone())
    return {"x": x}


def work(case):
    """Factorization: the algorithmic flops of the elimination order, the factor written once.  A solve reads the
    factor in each of its two sweeps (4 flops per entry and right-hand side; L U has two factors, one per sweep)."""
    if case["kind"] == "batch":
        parts, near = _batch_near(case)
        info = Solver.batch([(t.shape[0],) + _csc(t)[:2] for t in parts], precision=case["precision"]).info()
        nnz = int((near >= 0).sum())
    else:
        colptr, rowind, _ = _csc(_near(case), lower=case["kind"] == "adjoint")
        info = Solver(len(colptr) - 1, colptr, rowind, method=case["method"], precision=case["precision"]).info()
        nnz = len(rowind)
    nrhs, solves = case.get("nrhs", 1), 2 if case["kind"] == "adjoint" else 1
    factor = info["nnz_l"] * (8 if case["precision"] == "fp64" else 4)
    entry, vectors = 8 * nnz, 16 * info["n"] * nrhs
    size = solves * (2 * factor + vectors + entry)
    flops = solves * 4.0 * info["nnz_l"] * nrhs
    if case["kind"] != "solve":
        size += factor * (2 if case.get("method") == "lu" else 1) + entry
        flops += info["flops_alg"]
    if case["kind"] == "adjoint":
        size += entry
    return {"bytes": size, "flops": flops}


# ---------------------------------------------------------------- 64-bit results
def _solve64(near, val, b):
    """A x = b in 64 bits, A given by its rows: conjugate gradients (symmetric) or BiCGSTAB, with a diagonal
    preconditioner, restarted on the true residual until that no longer falls."""
    idx, n = near.clamp(min=0), near.shape[0]
    diag = (val * (near == torch.arange(n, device="cuda")[:, None])).sum(1)

    def mul(v):
        return (val * v[idx]).sum(1)

    def bicgstab(r, tol):
        d, r0, p, rho = torch.zeros_like(r), r.clone(), r.clone(), r @ r
        for k in range(20000):
            ph = p / diag
            v = mul(ph)
            alpha = rho / (r0 @ v)
            s = r - alpha * v
            sh = s / diag
            t = mul(sh)
            om = (t @ s) / (t @ t)
            d = d + alpha * ph + om * sh
            r = s - om * t
            new = r0 @ r
            if k % 10 == 9 and not float(r.norm()) > tol:
                break
            p, rho = r + (new / rho) * (alpha / om) * (p - om * v), new
        return d

    def cg(r, tol):
        d, z = torch.zeros_like(r), r / diag
        p, rho = z.clone(), r @ z
        for k in range(20000):
            v = mul(p)
            alpha = rho / (p @ v)
            d, r = d + alpha * p, r - alpha * v
            z = r / diag
            new = r @ z
            if k % 20 == 19 and not float(r.norm()) > tol:
                break
            p, rho = z + (new / rho) * p, new
        return d

    symmetric = bool(torch.equal(val, _transposed(near, val)))
    x, last = torch.zeros_like(b), float("inf")
    for _ in range(6):
        r = b - mul(x)
        size = float(r.norm())
        if size > 0.5 * last or size == 0.0:
            break
        last = size
        x = x + (cg if symmetric else bicgstab)(r, 1e-9 * size)
    return x


def _transposed(near, val):
    """The table of the transposed matrix (the pattern is symmetric, its rows ascending)."""
    n, k = near.shape
    keep = near >= 0
    row = near[keep]
    col = torch.arange(n, device="cuda")[:, None].expand(n, k)[keep]
    out = torch.zeros_like(val)
    out[keep] = val[keep][torch.argsort(row * n + col, stable=True)]
    return out


def exact(case, seed):
    near = _batch_near(case)[1] if case["kind"] == "batch" else _near(case)
    val, b, g = _inputs(case, seed, near)
    near = torch.as_tensor(near, device="cuda")
    rows = _transposed(near, val)        # the table lists columns: `rows` lists the rows of A

    def solve(v):
        return _solve64(near, rows, v) if v.dim() == 1 else torch.stack([_solve64(near, rows, u) for u in v])

    x = solve(b)
    if case["kind"] != "adjoint":
        return {"x": x}
    db = solve(g)
    keep = (near >= 0) & (near >= torch.arange(near.shape[0], device="cuda")[:, None])
    row = near[keep]
    col = torch.arange(near.shape[0], device="cuda")[:, None].expand_as(near)[keep]
    xs, ds = x.reshape(-1, x.shape[-1]), db.reshape(-1, x.shape[-1])
    gv = -(ds[:, row] * xs[:, col]).sum(0)
    gv = torch.where(row == col, gv, gv - (ds[:, col] * xs[:, row]).sum(0))
    return {"x": x, "grad_values": gv, "grad_b": db}
