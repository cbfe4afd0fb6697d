"""Box form, one orbital: the steps read one triangle of the operator only where
the set-up has found it symmetric (rows scaled by 1 / (i A_ii) in the first order)
up to the rounding of the product's sums, sqrt(n_Gamma) 2^-53 of its norm.  The
measure is checked against the exported operator: equal, but for the rounding
of the scaled entries (2^-52 of the norm).
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _solver():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1908_02456_amd.solver import Solver
    return Solver


@pytest.mark.parametrize("order,shape,R,h,s0", [("zeroth", (24, 24, 23), 1, 0.05, 1.0), ("zeroth", (24, 24, 23), 1, 1.0, 100.0),
                                                ("zeroth", (16, 17, 16), 3, 0.05, 1.0), ("zeroth", (16, 17, 16), 3, 1.0, 0.01),
                                                ("first", (24, 25, 24), 1, 0.05, 1.0), ("first", (24, 25, 24), 1, 1.0, 0.01),
                                                ("first", (3, 40, 40), 1, 0.25, 1.0)])
def test_triangle_only_where_symmetric(order, shape, R, h, s0):
    Solver = _solver()
    print("case: box symmetry", order, shape, "R", R, "h", h, "s", s0, flush=True)
    s = Solver(shape, h, 1e-4 * h * h, radius=R, order=order, form="box", s0=s0, s1=s0)
    n = s.box_info()["n_gamma"]
    assert n >= 3000
    if order == "first":
        op = s.export(1, 2 * n * n).reshape(n, 2 * n)
        op = op[:, :n] / (1j * np.diag(op[:, n:])).real[:, None]
    else:
        op = s.export(1, n * n).reshape(n, n)
    want = np.linalg.norm(op - op.T) / np.linalg.norm(op)
    got = s.export(4, 1)[0]
    print("  asymmetry", got.real, "from the exported operator", want, flush=True)
    assert abs(got.real - want) <= 2.0 ** -52
    assert got.real <= np.sqrt(n) * 2.0 ** -53 and got.imag == 1.0


@pytest.mark.parametrize("kw", [dict(order="zeroth"), dict(order="first", shape=(24, 24, 24), batch=2),
                                dict(order="first", shape=(18, 18, 18), radius=3)])
def test_full_product_elsewhere(kw):
    Solver = _solver()
    print("case: full product", kw, flush=True)
    kw = dict(kw)
    s = Solver(kw.pop("shape", (10, 10, 10)), 0.25, 0.002, form="box", **kw)
    assert s.export(4, 1)[0] == -1.0
