"""Device memory that the adjoint takes while it runs: X and lambda, the
checkpoints, and per segment step a state (the first is its checkpoint) and three
vectors; four more where the staged kernels do the reverse step.  Sampled from
another thread while the call runs (it holds its one allocation throughout).
"""
import math
import threading

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw,extra", [(dict(order="first", window=0), 0), (dict(order="dirichlet", radius=2), 4)])
@pytest.mark.parametrize("stride", [0, 100])
def test_adjoint_takes_what_it_uses(kw, extra, stride):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1908_02456_amd.solver import Solver
    n, steps = 96, 100
    print("case: adjoint memory", n, kw, "stride", stride, flush=True)
    s = Solver((n,) * 3, 0.2, 0.002, **kw)
    psi = torch.rand((n,) * 3, dtype=torch.complex128, device="cuda")
    V = torch.zeros((n,) * 3, dtype=torch.float64, device="cuda")
    s.adjoint(psi, V, 2, "prob")
    torch.cuda.synchronize()
    idle, low, stop = torch.cuda.mem_get_info()[0], [], threading.Event()

    def sample():
        while not stop.is_set():
            low.append(torch.cuda.mem_get_info()[0])

    t = threading.Thread(target=sample)
    t.start()
    try:
        for _ in range(3):
            s.adjoint(psi, V, steps, "prob", stride)
    finally:
        stop.set()
        t.join()
    seg = stride or math.ceil(math.sqrt(steps))
    seg = min(seg, steps)
    states = 2 + extra + math.ceil(steps / seg) + (seg - 1) + 3 * seg
    # the face variables of X, lambda, the checkpoints and the segment's states
    states += (2 + math.ceil(steps / seg) + (seg - 1)) * s.aux_elems / n ** 3
    took = (idle - min(low)) / (16 * n ** 3)
    print("  states", states, "taken", took, "samples", len(low), flush=True)
    # the samples have met the allocation; the rounding to pages (up or, where the
    # process holds free ones, down): less than one and a half states
    assert took > 0.9 * states
    assert took < states + 1.5
