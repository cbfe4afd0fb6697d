"""The tile depth that a context's launches run at, as abc_tile_depth and
abc_batch_tile_depth tell it, and parity at depths that few shapes reach: the
two-stage kernels of the first order at 5 and 12 planes (5 is what 96^3 takes)
with the adjoint's, and the staged sweep at each of its depths.  Every case
asserts the depth, with a ragged last tile in z.  Tolerances: 1e-12 (complex128)
and 1e-5 (complex64) of the largest value, as for the other paths; the gradient
as in test_gpu_adjoint.py.
"""
import numpy as np
import pytest
import torch

from oracle import adjoint as oadj
from oracle import integrate
from paper_1908_02456_amd import workloads as W

pytestmark = pytest.mark.gpu


def _cls():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1908_02456_amd.solver import Batch, Solver
    return Batch, Solver


def _check(s, st, psi0, V, steps):
    ref, ref_aux, _ = integrate.run(st, psi0, V, steps)
    psi, aux = torch.from_numpy(psi0).to(s.cdtype).cuda(), s.new_aux()
    s.step(psi, aux, torch.from_numpy(V).to(s.rdtype).cuda(), steps)
    tol = 1e-12 if s.cdtype == torch.complex128 else 1e-5
    assert np.abs(psi.cpu().numpy() - ref).max() <= tol * np.abs(ref).max()
    if st.order == "first":
        flat = integrate.pack_aux(st, ref_aux)
        assert np.abs(aux.cpu().numpy()[:flat.size] - flat).max() <= tol * np.abs(flat).max()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("depth,shape", [(5, (13, 515, 4)), (12, (18, 683, 4))])
def test_first_order_two_stage(depth, shape, dtype):
    _, Solver = _cls()
    print("case: depth", depth, shape, dtype, flush=True)
    h, dt = 0.25, 0.004
    st = integrate.make_setup(shape, h, dt, 1, "first", s1=1.5)
    s = Solver(shape, h, dt, order="first", s1=1.5, dtype=dtype, path="fused")
    assert s.tile_depth() == depth
    _check(s, st, W.random_complex(shape, seed=91), W.random_potential(shape, seed=92, scale=2.0), 3)


@pytest.mark.parametrize("depth,shape", [(5, (13, 515, 4)), (12, (18, 683, 4))])
def test_first_order_adjoint(depth, shape):
    _, Solver = _cls()
    print("case: adjoint depth", depth, shape, flush=True)
    h, dt, steps = 0.3, 0.01, 2
    psi0 = W.random_complex(shape, seed=93)
    V = W.random_potential(shape, seed=94, scale=2.0)
    st = integrate.make_setup(shape, h, dt, 1, "first", s1=1.5)
    J, gpsi, gV = oadj.adjoint_run(st, psi0, V, steps, "energy")
    s = Solver(shape, h, dt, order="first", s1=1.5, path="fused")
    assert s.tile_depth() == depth
    Jg, gp, gv = s.adjoint(torch.from_numpy(psi0).cuda(), torch.from_numpy(V).cuda(), steps, "energy")
    assert abs(Jg - J) < 1e-12 * abs(J)
    assert np.abs(gp.cpu().numpy() - gpsi).max() < 1e-12 * np.abs(gpsi).max()
    terms = dt * np.abs(gpsi).max() * np.abs(psi0).max()
    assert np.abs(gv.cpu().numpy() - gV).max() < 1e-12 * max(np.abs(gV).max(), terms)


@pytest.mark.parametrize("dtype,R,depth,shape", [
    ("c128", 1, 2, (7, 341, 30)), ("c128", 1, 3, (47, 41, 30)), ("c128", 1, 4, (19, 305, 30)),
    ("c128", 1, 6, (22, 386, 30)), ("c128", 1, 8, (34, 341, 30)), ("c64", 1, 3, (47, 41, 30)),
    ("c64", 1, 6, (22, 386, 30)), ("c128", 2, 3, (58, 65, 30)), ("c64", 2, 3, (16, 386, 30)),
    ("c128", 3, 3, (10, 410, 30)), ("c64", 3, 3, (16, 386, 30)), ("c128", 3, 6, (37, 410, 30)),
    ("c128", 3, 16, (57, 386, 66))])
def test_staged_sweep(dtype, R, depth, shape):
    _, Solver = _cls()
    print("case: staged depth", depth, shape, "R", R, dtype, flush=True)
    h, dt = 0.25, 0.004
    st = integrate.make_setup(shape, h, dt, R, "first", s1=1.5)
    s = Solver(shape, h, dt, radius=R, order="first", s1=1.5, dtype=dtype, path="staged")
    assert s.tile_depth() == depth
    _check(s, st, W.random_complex(shape, seed=95), W.random_potential(shape, seed=96, scale=2.0), 1)


def test_depth_of_a_batch_and_under_a_limit():
    # a batch of one box takes the depth that the box takes alone; tuning returns
    # and leaves the depth in use, which the group reports
    Batch, Solver = _cls()
    print("case: batch depth", flush=True)
    shape = (40, 24, 70)  # few tiles: 2 planes under every limit
    cfg = dict(shape=shape, h=0.25, dt=0.004, order="first", s1=1.5, window=0)
    b, s = Batch([cfg]), Solver(shape, 0.25, 0.004, order="first", s1=1.5, window=0, path="fused")
    assert b.groups() == [2] and s.tile_depth() == 2
    psi, V = torch.zeros(shape, dtype=torch.complex128, device="cuda"), torch.zeros(shape, dtype=torch.float64, device="cuda")
    assert b.tune([psi], [b.new_aux(0)], [V]) == [2]
    assert s.tune(psi, s.new_aux(), V) in (4, 8, 16) and s.tile_depth() == 2


def test_depth_of_the_other_paths():
    _, Solver = _cls()
    print("case: depth, other paths", flush=True)
    one = dict(order="first", dtype="c64", path="onepass", window=0)
    assert Solver((40, 48, 32), 0.25, 0.002, **one).tile_depth() == 8
    assert Solver((96, 96, 96), 0.25, 0.002, batch=8, **one).tile_depth() == 24
    assert Solver((12, 12, 12), 0.25, 0.002, order="periodic").tile_depth() == 0
    assert Solver((12, 12, 12), 0.25, 0.002, order="first", batch=3, path="staged").tile_depth() == 0
