"""The one-pass sweep at the tile depths that complex64 picks (8 planes, 16 and
24 for boxes with many tiles) and with the high x face inside a lane pair or between
two (odd and even rows, full rows), against the oracle: ragged tiles in y and z,
the shortest boxes that the first order takes.  Tolerances: 1e-12 (complex128)
and 1e-5 (complex64) of the largest value, as for the other paths.
"""
import numpy as np
import pytest
import torch

from oracle import integrate
from paper_1908_02456_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", ["first", "zeroth", "dirichlet"])
@pytest.mark.parametrize("shape,dtype", [((13, 17, 9), "c64"), ((13, 18, 10), "c64"), ((21, 1021, 9), "c64"),
                                         ((26, 1021, 10), "c64"), ((33, 1017, 127), "c64"), ((26, 1021, 128), "c64"),
                                         ((47, 1021, 9), "c64"), ((43, 1018, 127), "c64"), ((48, 1021, 128), "c64"),
                                         ((21, 13, 9), "c128"), ((22, 14, 10), "c128"), ((37, 15, 127), "c128"),
                                         ((22, 14, 128), "c128")])
def test_onepass_tiles(shape, dtype, order):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1908_02456_amd.solver import Solver
    print("case:", shape, order, dtype, flush=True)
    h, dt, steps = 0.25, 0.004, 2
    psi0 = W.random_complex(shape, seed=81)
    V = W.random_potential(shape, seed=82, scale=2.0)
    st = integrate.make_setup(shape, h, dt, 1, order, s0=1.5, s1=1.5)
    ref, ref_aux, _ = integrate.run(st, psi0, V, steps)
    s = Solver(shape, h, dt, order=order, s0=1.5, s1=1.5, dtype=dtype, path="onepass")
    psi = torch.from_numpy(psi0).to(s.cdtype).cuda()
    aux = s.new_aux()
    s.step(psi, aux, torch.from_numpy(V).to(s.rdtype).cuda(), steps)
    tol = 1e-12 if dtype == "c128" else 1e-5
    assert np.abs(psi.cpu().numpy() - ref).max() <= tol * np.abs(ref).max()
    if order == "first":
        flat = integrate.pack_aux(st, ref_aux)
        assert np.abs(aux.cpu().numpy()[:flat.size] - flat).max() <= tol * np.abs(flat).max()
