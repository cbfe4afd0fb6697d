"""The two-stage kernels at every tile depth that their rule picks (2 to 16
planes), against the oracle: thin boxes whose tile counts make each depth the
cheapest, with a ragged last tile in z and in y.  The same shapes through the
adjoint, whose kernels keep the stage outputs and accumulate the potential's
gradient.  Tolerances: 1e-12 (complex128) and 1e-5 (complex64) of the largest
value, as for the other paths; the gradient as in test_gpu_adjoint.py.
"""
import numpy as np
import pytest
import torch

from oracle import adjoint as oadj
from oracle import integrate
from paper_1908_02456_amd import workloads as W

pytestmark = pytest.mark.gpu

# (nz, ny, nx) by the depth picked
FIRST = {2: (7, 12, 4), 3: (7, 513, 4), 4: (7, 682, 4), 5: (9, 683, 4), 6: (11, 681, 4), 8: (13, 681, 4),
         12: (17, 681, 4), 16: (26, 683, 4)}
OTHER = {2: (7, 11, 4), 3: (7, 513, 4), 4: (7, 681, 4), 5: (9, 683, 4), 6: (11, 682, 4), 8: (7, 1027, 4),
         12: (10, 1025, 4), 16: (26, 681, 4)}


def _solver():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1908_02456_amd.solver import Solver
    return Solver


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("order", ["first", "zeroth", "dirichlet"])
@pytest.mark.parametrize("depth", sorted(FIRST))
def test_two_stage_path_at_each_depth(depth, order, dtype):
    Solver = _solver()
    shape = (FIRST if order == "first" else OTHER)[depth]
    print("case: depth", depth, shape, order, dtype, flush=True)
    h, dt, steps = 0.25, 0.004, 3
    psi0 = W.random_complex(shape, seed=51)
    V = W.random_potential(shape, seed=52, scale=2.0)
    st = integrate.make_setup(shape, h, dt, 1, order, s0=1.5, s1=1.5)
    ref, ref_aux, _ = integrate.run(st, psi0, V, steps)
    s = Solver(shape, h, dt, order=order, s0=1.5, s1=1.5, dtype=dtype, path="fused")
    psi = torch.from_numpy(psi0).to(s.cdtype).cuda()
    aux = s.new_aux()
    s.step(psi, aux, torch.from_numpy(V).to(s.rdtype).cuda(), steps)
    tol = 1e-12 if dtype == "c128" else 1e-5
    assert np.abs(psi.cpu().numpy() - ref).max() <= tol * np.abs(ref).max()
    if order == "first":
        flat = integrate.pack_aux(st, ref_aux)
        assert np.abs(aux.cpu().numpy()[:flat.size] - flat).max() <= tol * np.abs(flat).max()


@pytest.mark.parametrize("order", ["first", "zeroth"])
@pytest.mark.parametrize("depth", sorted(FIRST))
def test_adjoint_at_each_depth(depth, order):
    Solver = _solver()
    shape = (FIRST if order == "first" else OTHER)[depth]
    print("case: adjoint depth", depth, shape, order, flush=True)
    h, dt, steps = 0.3, 0.01, 2
    psi0 = W.random_complex(shape, seed=53)
    V = W.random_potential(shape, seed=54, scale=2.0)
    st = integrate.make_setup(shape, h, dt, 1, order, s0=1.5, s1=1.5)
    J, gpsi, gV = oadj.adjoint_run(st, psi0, V, steps, "energy")
    s = Solver(shape, h, dt, order=order, s0=1.5, s1=1.5, path="fused")
    Jg, gp, gv = s.adjoint(torch.from_numpy(psi0).cuda(), torch.from_numpy(V).cuda(), steps, "energy")
    assert abs(Jg - J) < 1e-12 * abs(J)
    assert np.abs(gp.cpu().numpy() - gpsi).max() < 1e-12 * np.abs(gpsi).max()
    terms = dt * np.abs(gpsi).max() * np.abs(psi0).max()
    assert np.abs(gv.cpu().numpy() - gV).max() < 1e-12 * max(np.abs(gV).max(), terms)
