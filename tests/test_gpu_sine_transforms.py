"""The mean field's sine transforms at the edges of their matrix tiles and of
their plane classes (64, 96 and 128 points a side in LDS, rocBLAS beyond), with
one field or both switched on, against the oracle's sparse solves.

Tolerance as in test_gpu_skyrme.py: the solves stop at a relative residual of
1e-14 and the condition number of -Delta_h on these thin boxes is below 1e3, so
the potential is held at 1e-11 of its largest value.  R = 1 solves are exact
after one iteration of the sine-transform inverse (at most 3 allowed for
rounding).
"""
import numpy as np
import pytest
import torch

from oracle import integrate
from paper_1908_02456_amd import workloads as W

pytestmark = pytest.mark.gpu

BOTH = dict(t0=-1.0, t3=0.5, v0=-0.8, a=0.7, e2=0.3, tol=1e-14, maxit=3000)
SHAPES = [(3, 16, 16), (5, 17, 15), (16, 15, 17), (4, 64, 64), (3, 65, 33), (3, 20, 97), (3, 96, 96), (3, 128, 128),
          (3, 112, 130), (3, 129, 128), (3, 7, 200), (65, 5, 6), (256, 4, 5), (257, 4, 5)]


def _check(shape, R, mf, batch=2):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1908_02456_amd.solver import Solver
    print("case: sine transforms", shape, "R", R, mf["v0"], mf["e2"], flush=True)
    h = 0.3
    psi0 = W.random_complex(shape + (batch,), seed=61)
    V = W.random_potential(shape, seed=62)
    st = integrate.make_setup(shape, h, 0.002, R, "dirichlet", t0=mf["t0"], t3=mf["t3"], v0=mf["v0"], a_y=mf["a"],
                              e2=mf["e2"])
    ref = V + integrate.meanfield(st, psi0)
    s = Solver(shape, h, 0.002, radius=R, order="dirichlet", batch=batch, meanfield=mf)
    psi, Vt = torch.from_numpy(psi0).cuda(), torch.from_numpy(V).cuda()
    for _ in range(2):  # from zero, then from its own solution
        got = s.effective_potential(psi, Vt).cpu().numpy()
        assert np.abs(got - ref).max() < 1e-11 * np.abs(ref).max()
    n, iy, ic = s.potential_iterations()
    assert n == 2 and s.potential_unconverged() == 0
    if R == 1:
        assert (1 if mf["v0"] else 0) <= iy <= 6 and (1 if mf["e2"] else 0) <= ic <= 6
    if not mf["v0"]:
        assert iy == 0
    if not mf["e2"]:
        assert ic == 0


@pytest.mark.parametrize("shape", SHAPES)
def test_both_fields(shape):
    _check(shape, 1, BOTH)


@pytest.mark.parametrize("off", ["v0", "e2"])
@pytest.mark.parametrize("shape", [(5, 17, 15), (3, 7, 200)])
def test_one_field(shape, off):
    _check(shape, 1, dict(BOTH, **{off: 0.0}))


@pytest.mark.parametrize("R", [2, 3])
@pytest.mark.parametrize("shape", [(7, 33, 18), (7, 8, 200)])
def test_wider_stencils(shape, R):
    _check(shape, R, BOTH)
