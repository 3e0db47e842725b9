"""Workers of the scheduler kernel: two per compute unit where the work is
longer than the elimination chain, one where the chain is.  Small blocks of
L U are not fused: the work of a batch of small systems is its work items.
Counted from the trace: items in work at once."""
import numpy as np
import pytest

from gen import convection_diffusion, grid_batch

pytestmark = pytest.mark.gpu


def _at_once(s):
    t, _ = s.trace()
    at, step = np.concatenate([t[:, 1], t[:, 2]]), np.repeat([1, -1], len(t))
    return np.cumsum(step[np.lexsort((step, at))]).max()   # (an item that ends as another starts: ended first)


@pytest.mark.parametrize("method", ["llt", "ldlt", "lu"])
def test_batch_of_small_systems(method):
    import torch
    from paper_1405_2636_amd import Solver
    ps = grid_batch(400, seed=21, lo=8, hi=48)
    print("workers", method, sum(p.n for p in ps), flush=True)
    s = Solver.batch([(p.n, p.colptr, p.rowind) for p in ps], method=method, graph=False, tune=False, trace=True)
    s.factorize(torch.tensor(np.concatenate([p.values for p in ps]), device="cuda"))
    assert _at_once(s) > torch.cuda.get_device_properties(0).multi_processor_count
    x, info = s.solve(torch.tensor(np.concatenate([p.b[:, 0] for p in ps]), device="cuda"))
    assert info["omega"] <= 1e-14


@pytest.mark.parametrize("method", ["llt", "ldlt", "lu"])
def test_chain(method):
    import torch
    from paper_1405_2636_amd import Solver
    p = convection_diffusion((14, 13, 12), seed=2, cmax=0.0 if method != "lu" else 0.5)
    print("workers", method, p.n, flush=True)
    s = Solver(p.n, p.colptr, p.rowind, method=method, trace=True)
    s.factorize(torch.tensor(p.values, device="cuda"))
    assert _at_once(s) <= torch.cuda.get_device_properties(0).multi_processor_count
    x, info = s.solve(torch.ones(p.n, dtype=torch.float64, device="cuda"))
    assert info["omega"] <= 1e-14
