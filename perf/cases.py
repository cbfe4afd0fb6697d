"""Performance cases of the absorbing-boundary time stepper, through its public entry points.

Each case is one call (or one short sequence of calls) as a simulation program makes it in its time loop:
`Solver.step`, `Solver.diagnostics`, `Batch.step` and the `abc_objective` gradient.  `exact` restates the
method in 64-bit torch, without the package, for the same inputs.

Kinds of cases
  faces     one orbital in a box closed by the per-face operators (or by zero boundary values)
  orbitals  a batch of orbitals sharing a mean field (local, or with the Yukawa and Coulomb solves)
  box       the paper's dense box-form operators
  uneven    independent boxes of mixed sizes and orders in one call
  gradient  forward run and reverse sweep behind torch.autograd
"""
import math

import numpy as np
import torch

from paper_1908_02456_amd.autograd import abc_objective
from paper_1908_02456_amd.solver import Batch, Solver

DEVICE = "cuda"


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------

def _faces(shape, steps, order="first", radius=1, window=0, dtype="c128", h=0.2, dt=0.002, records=False):
    """window: kernel half-width; -1 asks for the exact sections."""
    nz, ny, nx = shape
    return {"kind": "faces", "nz": nz, "ny": ny, "nx": nx, "h": h, "dt": dt, "steps": steps, "order": order,
            "radius": radius, "window": window, "dtype": dtype, "records": records}


def _orbitals(shape, batch, steps, dtype, long_range, order="first"):
    nz, ny, nx = shape
    return {"kind": "orbitals", "nz": nz, "ny": ny, "nx": nx, "h": 0.2, "dt": 0.002, "steps": steps, "order": order,
            "batch": batch, "dtype": dtype, "long_range": long_range}


def _box(shape, steps, order, batch=1, radius=1):
    nz, ny, nx = shape
    return {"kind": "box", "nz": nz, "ny": ny, "nx": nx, "h": 0.25, "dt": 0.005, "steps": steps, "order": order,
            "batch": batch, "radius": radius}


def _uneven(count, steps, layout, lo=48, hi=160):
    return {"kind": "uneven", "count": count, "steps": steps, "layout": layout, "lo": lo, "hi": hi, "h": 0.2, "dt": 0.002}


def _gradient(shape, steps, objective="energy"):
    nz, ny, nx = shape
    return {"kind": "gradient", "nz": nz, "ny": ny, "nx": nx, "h": 0.2, "dt": 0.002, "steps": steps,
            "objective": objective}


def listed():
    return [
        # one step and a diagnostics record of a small box, the size of the paper's 3D test: a loop that looks at
        # every step, bound by launches and latency
        dict(_faces((31, 29, 33), 1, h=0.1, dt=0.001, records=True), name="small_one_step"),
        # the headline workload between two looks at the state
        dict(_faces((128, 128, 128), 20), name="well_128_c128"),
        # the same with the FP32 stencil
        dict(_faces((128, 128, 128), 20, dtype="c64"), name="well_128_c64"),
        # the large zero-boundary box that reflections are measured against
        dict(_faces((256, 256, 256), 4, order="dirichlet"), name="reference_256"),
        # the paper's seven points per axis
        dict(_faces((128, 128, 128), 10, radius=3), name="seven_point_128"),
        # the windowed face operator, which absorbs better than the local one
        dict(_faces((128, 128, 128), 10, window=8), name="window8_128"),
        # the exact face sections, which absorb best among the face forms; an uneven box
        dict(_faces((128, 110, 121), 5, window=-1), name="exact_sections"),
        # the mean-field batch of 32 orbitals
        dict(_orbitals((96, 96, 96), 32, 5, "c64", False), name="tdhf_96_32orb_c64"),
        # a small nucleus' orbitals with the Yukawa and Coulomb fields solved every step
        dict(_orbitals((61, 61, 61), 8, 5, "c128", True), name="long_range_61_8orb"),
        # the paper's dense operators on the largest box that they suit in a loop
        dict(_box((32, 32, 32), 5, "first"), name="box_form_32"),
        # a parameter scan: boxes of sizes 48 to 160, zeroth and first order
        dict(_uneven(12, 4, 4), name="uneven_12"),
        # optimisation of a potential: forward and reverse.  The energy, since over so few steps the probability's
        # gradient with respect to the potential cancels to its terms' rounding
        dict(_gradient((96, 96, 96), 48), name="gradient_96"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["faces", "faces", "faces", "wide", "orbitals", "box", "uneven", "gradient"])
    if kind == "faces":
        order = rng.choice(["dirichlet", "zeroth", "first", "first"])
        shape = [_log_int(rng, 24, 160) for _ in range(3)]
        return _faces(shape, rng.choice([1, 4, 10]), order=order, radius=rng.choice([1, 1, 2, 3]),
                      dtype=rng.choice(["c128", "c128", "c64"]), records=rng.random() < 0.25)
    if kind == "wide":
        order = rng.choice(["zeroth", "first"])
        shape = [_log_int(rng, 40, 128) for _ in range(3)]
        return _faces(shape, rng.choice([2, 5]), order=order, radius=rng.choice([1, 1, 3]),
                      window=rng.choice([2, 4, 8, 12, -1]), dtype=rng.choice(["c128", "c64"]))
    if kind == "orbitals":
        long_range = rng.random() < 0.5
        n = 80 if long_range else 96
        shape = [_log_int(rng, 24, n) for _ in range(3)]
        return _orbitals(shape, rng.choice([2, 4, 8, 15, 32]) if not long_range else rng.choice([2, 4, 8, 15]),
                         rng.choice([1, 3, 5]), rng.choice(["c64", "c128"]), long_range,
                         order=rng.choice(["zeroth", "first"]))
    if kind == "box":
        shape = [_log_int(rng, 10, 30) for _ in range(3)]
        return _box(shape, rng.choice([1, 3, 5]), rng.choice(["zeroth", "first"]), batch=rng.choice([1, 1, 8, 32]))
    if kind == "uneven":
        return _uneven(rng.randint(4, 12), rng.choice([1, 2, 4]), rng.randrange(1000), lo=32, hi=rng.choice([96, 128, 160]))
    shape = [_log_int(rng, 32, 100) for _ in range(3)]
    return _gradient(shape, _log_int(rng, 8, 48))


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _axis(n, h):
    return (torch.arange(n, dtype=torch.float64, device=DEVICE) - 0.5 * (n - 1)) * h


def _packet(shape, h, center, k, width=1.0):
    """exp(-|x - c|^2 / 2 width^2) exp(i k.x); center and k as (z, y, x)."""
    f = []
    for n, c, q in zip(shape, center, k):
        x = _axis(n, h)
        f.append(torch.polar(torch.exp(-(x - c) ** 2 / (2 * width * width)), q * x))
    return (f[0][:, None, None] * f[1][None, :, None] * f[2][None, None, :]).contiguous()


def _well(shape, h, amplitude, center):
    f = [torch.exp(-(_axis(n, h) - c) ** 2 / 2) for n, c in zip(shape, center)]
    return (-amplitude * f[0][:, None, None] * f[1][None, :, None] * f[2][None, None, :]).contiguous()


def _packet_and_well(shape, h, rng):
    """A Gaussian well near the centre and a packet that reaches the faces."""
    ext = [n * h for n in shape]
    width = min(1.0, min(ext) / 5)
    psi = _packet(shape, h, [rng.uniform(-0.15, 0.15) * e for e in ext], rng.uniform(-3.0, 3.0, 3), width)
    V = _well(shape, h, rng.uniform(1.0, 5.0), rng.uniform(-0.5, 0.5, 3))
    return psi, V


def _oscillator(shape, h, count, rng):
    """The lowest Cartesian oscillator states, each boosted by a random plane wave, [z][y][x][orbital]."""
    top = 0
    states = []
    while len(states) < count:
        states += [(a, b, top - a - b) for a in range(top, -1, -1) for b in range(top - a, -1, -1)]
        top += 1
    states = states[:count]
    axes = []
    for d, n in enumerate(shape):
        x = _axis(n, h)
        f = [math.pi ** -0.25 * torch.exp(-0.5 * x * x)]
        f.append(math.sqrt(2.0) * x * f[0])
        for m in range(1, top):
            f.append(math.sqrt(2.0 / (m + 1)) * x * f[m] - math.sqrt(m / (m + 1)) * f[m - 1])
        q = torch.as_tensor(rng.uniform(-1.2, 1.2, count), device=DEVICE)
        f = torch.stack([f[s[d]] for s in states], dim=1)
        f = f / torch.sqrt(h * (f * f).sum(0, keepdim=True))
        axes.append(torch.polar(torch.ones_like(f), q[None, :] * x[:, None]) * f)
    return (axes[0][:, None, None] * axes[1][None, :, None] * axes[2][None, None, :]).contiguous()


def _half(case):
    """(window, fejer) of the Solver for the case's window."""
    w = case["window"]
    return (max(case["nz"], case["ny"], case["nx"]) - 1, False) if w < 0 else (w, True)


def _shape(case):
    return case["nz"], case["ny"], case["nx"]


def _uneven_layout(case):
    """Sizes and orders of the boxes; a third of the boxes are not cubes."""
    r = np.random.default_rng(case["layout"])
    size = lambda: int(round(math.exp(r.uniform(math.log(case["lo"]), math.log(case["hi"])))))  # noqa: E731
    out = []
    for i in range(case["count"]):
        n = size()
        shape = (n, size(), size()) if i % 3 == 2 else (n, n, n)
        out.append((shape, "first" if r.random() < 0.5 else "zeroth"))
    return out


LOCAL = (-1.0, 0.5)
YUKAWA = {"v0": 0.3, "a": 0.7, "e2": 0.2}


def _inputs(case, seed):
    """Fields of the case in FP64, in the case's order of draws."""
    rng = np.random.default_rng(seed)
    if case["kind"] == "uneven":
        return [_packet_and_well(shape, case["h"], rng) for shape, _ in _uneven_layout(case)]
    shape = _shape(case)
    if case["kind"] == "orbitals" or case.get("batch", 1) > 1:
        psi = _oscillator(shape, case["h"], case["batch"], rng)
        return psi, _well(shape, case["h"], rng.uniform(1.0, 5.0), rng.uniform(-0.5, 0.5, 3))
    return _packet_and_well(shape, case["h"], rng)


def prepare(case, seed):
    kind = case["kind"]
    fields = _inputs(case, seed)
    if kind == "uneven":
        b = Batch([{"shape": shape, "h": case["h"], "dt": case["dt"], "order": order} for shape, order in _uneven_layout(case)])
        return {"case": case, "batch": b, "psi": [f[0] for f in fields], "V": [f[1] for f in fields],
                "aux": [b.new_aux(i) for i in range(b.n)]}
    psi, V = fields
    opts = {"order": case.get("order", "first"), "radius": case.get("radius", 1), "dtype": case.get("dtype", "c128"),
            "batch": case.get("batch", 1)}
    if kind == "faces":
        opts["window"], opts["fejer"] = _half(case)
    elif kind == "box":
        opts["form"] = "box"
    elif kind == "orbitals":
        opts["meanfield"] = dict(t0=LOCAL[0], t3=LOCAL[1], **YUKAWA) if case["long_range"] else LOCAL
    s = Solver(_shape(case), case["h"], case["dt"], **opts)
    st = {"case": case, "solver": s, "psi": psi.to(s.cdtype), "V": V.to(s.rdtype)}
    if kind != "gradient":
        st["aux"] = s.new_aux() if s.aux_elems else None
    return st


def run(state):
    case = state["case"]
    steps = case["steps"]
    if case["kind"] == "uneven":
        state["batch"].step(state["psi"], state["aux"], state["V"], steps)
        return {"psi": state["psi"], "aux": [a for a, (_, order) in zip(state["aux"], _uneven_layout(case)) if order == "first"]}
    s, psi, V = state["solver"], state["psi"], state["V"]
    if case["kind"] == "gradient":
        psi0, V0 = psi.detach().requires_grad_(), V.detach().requires_grad_()
        J = abc_objective(s, psi0, V0, steps, case["objective"])
        gpsi, gV = torch.autograd.grad(J, (psi0, V0))
        return {"J": J.detach(), "grad_psi": gpsi, "grad_V": gV}
    aux = state["aux"]
    s.step(psi, aux, V, steps)
    out = {"psi": psi}
    if aux is not None:
        # behind an FP32 stencil the FP64 auxiliary variables are FP32 results: a program records them as such
        out["aux"] = aux.to(s.cdtype)
    if case.get("records"):
        out["record"] = s.diagnostics(psi, aux, V)
    return out


def _gamma_count(shape, R):
    return math.prod(shape) - math.prod(max(n - 2 * R, 0) for n in shape)


def work(case):
    """State in and out and the potential once per step (a step maps the whole state, which no cache level near the
    cores holds), the auxiliary variables likewise, a dense operator once per stage; the stencil's, the face
    kernels' and the dense products' operations."""
    steps = case["steps"]
    if case["kind"] == "uneven":
        total = {"bytes": 0, "flops": 0}
        for shape, order in _uneven_layout(case):
            w = work(_faces(shape, steps, order=order))
            total = {k: total[k] + w[k] for k in total}
        return total
    shape, R, batch = _shape(case), case.get("radius", 1), case.get("batch", 1)
    n = math.prod(shape)
    c = 8 if case.get("dtype") == "c64" else 16
    step_bytes = n * (2 * c * batch + c // 2)
    step_flops = 4 * n * batch * 2 * (7 * R + 6)
    order = case.get("order", "first")
    if case["kind"] == "box":
        g = _gamma_count(shape, R)
        step_bytes += 4 * 16 * g * g + (32 * g * batch if order == "first" else 0)
        step_flops += 4 * 8 * g * g * batch
    elif order in ("zeroth", "first"):
        face = 2 * R * batch * (shape[0] * shape[1] + shape[0] * shape[2] + shape[1] * shape[2])
        if order == "first":
            step_bytes += 32 * face
        w = case.get("window", 0)
        taps = R * (2 * w + 1) ** 2 if w >= 0 else R + 10 * math.log2(4 * max(shape))
        step_flops += 4 * 8 * face * taps
    if case.get("long_range"):
        step_bytes += n * 2 * c // 2
        step_flops += 2 * 2 * 6 * n * sum(shape) // 3
    if case["kind"] == "gradient":
        # forward, reverse, and one pass more for what the reverse sweep needs of the forward states
        return {"bytes": 3 * steps * step_bytes, "flops": 3 * steps * step_flops}
    return {"bytes": steps * step_bytes, "flops": steps * step_flops}


# ---------------------------------------------------------------------------
# The method in 64-bit torch
# ---------------------------------------------------------------------------

WEIGHTS = {1: (-2.0, 1.0), 2: (-5 / 2, 4 / 3, -1 / 12), 3: (-49 / 18, 3 / 2, -3 / 20, 1 / 90)}
S1 = 1.0


def _minus_half_laplacian(y, h, R):
    c = WEIGHTS[R]
    out = 3 * c[0] * y
    for axis in range(3):
        n = y.shape[axis]
        for k in range(1, min(R, n - 1) + 1):
            out = out.clone()
            out.narrow(axis, 0, n - k).add_(y.narrow(axis, k, n - k), alpha=c[k])
            out.narrow(axis, k, n - k).add_(y.narrow(axis, 0, n - k), alpha=c[k])
    return out * (-0.5 / (h * h))


def _symbol_1d(theta, h, R):
    c = WEIGHTS[R]
    return (-c[0] - sum(2 * c[k] * torch.cos(k * theta) for k in range(1, R + 1))) / (2 * h * h)


def _half_line(R, h, s, P):
    """Half-line map of the exterior of one face per transverse mode, (P/2+1, P/2+1, R, R): the solution of
    X = (D - U X L)^-1 on the blocked exterior line, by doubling."""
    c = WEIGHTS[R]
    th = 2 * math.pi * torch.arange(P // 2 + 1, dtype=torch.float64, device=DEVICE) / P
    t = _symbol_1d(th, h, R)
    shift = (t[:, None] + t[None, :]).reshape(-1) - 1j * s
    a = [-v / (2 * h * h) for v in c]
    D = torch.zeros(shift.numel(), R, R, dtype=torch.complex128, device=DEVICE)
    U = torch.zeros(R, R, dtype=torch.complex128, device=DEVICE)
    H = torch.zeros(R, R, dtype=torch.complex128, device=DEVICE)
    for i in range(R):
        for j in range(R):
            D[:, i, j] = a[abs(i - j)]
            if j <= i:
                U[i, j] = a[R + j - i]
            if i + j + 1 <= R:
                H[i, j] = a[i + j + 1]
        D[:, i, i] += shift

    def mul(p, q):
        return (p[:, :, :, None] * q[:, None, :, :]).sum(2)

    up, low, first, mid = U.expand_as(D).clone(), U.T.expand_as(D).clone(), D.clone(), D.clone()
    for _ in range(60):
        inv = torch.linalg.inv(mid)
        p, q = mul(mul(up, inv), low), mul(mul(low, inv), up)
        up, low = -mul(mul(up, inv), up), -mul(mul(low, inv), low)
        first, mid = first - p, mid - p - q
        if float(up.abs().max()) < 1e-40 or float(low.abs().max()) < 1e-40:
            break
    Y = torch.linalg.inv(first)
    Hb = H.expand_as(Y)
    k = -mul(mul(Hb, Y), Hb.transpose(1, 2))
    return k.reshape(P // 2 + 1, P // 2 + 1, R, R), H


class _Faces:
    """Convolution along each face (zero-padded FFT) and the normal-line block."""

    def __init__(self, shape, h, R, order, w, fejer):
        P = 64
        while P < max(64.0, 4.0 * (w + 1), 60.0 / (math.sqrt(S1) * h) + 2.0 * w):
            P *= 2
        sym, H = _half_line(R, h, S1, P)
        if order == "first":
            self.a = -1j * (H @ H.T)
            eye = torch.eye(R, dtype=torch.complex128, device=DEVICE)
            inv = torch.linalg.inv(sym.reshape(-1, R, R))
            sym = S1 * eye - (self.a[None, :, :, None] * inv[:, None, :, :]).sum(2).reshape(sym.shape)
        i = torch.arange(P, device=DEVICE)
        i = torch.minimum(i, P - i)
        k = torch.fft.ifft2(sym[i][:, i], dim=(0, 1))
        p = torch.arange(-w, w + 1, device=DEVICE)
        k = k[p % P][:, p % P]
        if fejer:
            f = 1 - p.abs().double() / (w + 1)
            k = k * (f[:, None] * f[None, :])[:, :, None, None]
        self.R, self.w, self.k, self.spectra = R, w, k, {}

    def slab(self, y, f):
        axis, n = 2 - f // 2, y.shape[2 - f // 2]
        at = [i if f % 2 == 0 else n - 1 - i for i in range(self.R)]
        return torch.stack([y.select(axis, i) for i in at], 0)

    def add(self, out, slab, f):
        axis, n = 2 - f // 2, out.shape[2 - f // 2]
        for i in range(self.R):
            out.select(axis, i if f % 2 == 0 else n - 1 - i).add_(slab[i])

    def convolve(self, slab):
        if self.w == 0:
            return torch.stack([sum(self.k[0, 0, i, j] * slab[j] for j in range(self.R)) for i in range(self.R)], 0)
        n1, n2 = slab.shape[1], slab.shape[2]
        w1, w2 = min(self.w, n1 - 1), min(self.w, n2 - 1)
        L1, L2 = n1 + w1, n2 + w2
        if (n1, n2) not in self.spectra:
            z = torch.zeros(self.R, self.R, L1, L2, dtype=torch.complex128, device=DEVICE)
            p1, p2 = torch.arange(-w1, w1 + 1, device=DEVICE), torch.arange(-w2, w2 + 1, device=DEVICE)
            part = self.k[(p1 + self.w)][:, (p2 + self.w)].permute(2, 3, 0, 1)
            for i in range(self.R):
                for j in range(self.R):
                    z[i, j].index_put_((p1[:, None] % L1, p2[None, :] % L2), part[i, j], accumulate=True)
            self.spectra[n1, n2] = torch.fft.fft2(z)
        S = self.spectra[n1, n2]
        tail = slab.dim() - 3
        x = torch.fft.fft2(slab, s=(L1, L2), dim=(1, 2))
        y = []
        for i in range(self.R):
            y.append(sum(S[i, j].reshape(S.shape[2:] + (1,) * tail) * x[j] for j in range(self.R)))
        return torch.fft.ifft2(torch.stack(y, 0), dim=(1, 2))[:, :n1, :n2]

    def local(self, slab):
        return torch.stack([sum(self.a[i, j] * slab[j] for j in range(self.R)) for i in range(self.R)], 0)


class _BoxForm:
    """Dense operators of the boundary-element formula over the box's boundary layer."""

    def __init__(self, shape, h, R, order):
        nz, ny, nx = shape
        z, y, x = torch.meshgrid(*(torch.arange(n, device=DEVICE) for n in shape), indexing="ij")
        near = torch.zeros(shape, dtype=torch.bool, device=DEVICE)
        for q, n in ((z, nz), (y, ny), (x, nx)):
            near |= (q < R) | (q > n - 1 - R)
        G = torch.stack([z[near], y[near], x[near]], 1)
        ext = []
        for axis, n in enumerate(shape):
            o = [a for a in range(3) if a != axis]
            u, v = torch.meshgrid(torch.arange(shape[o[0]], device=DEVICE), torch.arange(shape[o[1]], device=DEVICE), indexing="ij")
            for q in list(range(-R, 0)) + list(range(n, n + R)):
                e = torch.empty(u.numel(), 3, dtype=torch.long, device=DEVICE)
                e[:, axis], e[:, o[0]], e[:, o[1]] = q, u.reshape(-1), v.reshape(-1)
                ext.append(e)
        E = torch.cat(ext)
        c = torch.tensor(WEIGHTS[R], dtype=torch.float64, device=DEVICE)
        H = torch.zeros(len(G), len(E), dtype=torch.float64, device=DEVICE)
        for i in range(0, len(G), 1024):
            d = (G[i:i + 1024, None] - E[None]).abs()
            far = d.sum(2)
            on = (d.amax(2) == far) & (far <= R)
            H[i:i + 1024] = torch.where(on, -c[far.clamp(max=R)] / (2 * h * h), 0.0)
        L = 16
        while L < 2 * (max(shape) + 2 * R) + math.ceil(35.0 / (math.sqrt(S1) * h)):
            L *= 2
        t = _symbol_1d(2 * math.pi * torch.arange(L, dtype=torch.float64, device=DEVICE) / L, h, R)
        g = torch.fft.ifftn(1.0 / (t[:, None, None] + t[None, :, None] + t[None, None, :] - 1j * S1)).reshape(-1)

        def table(P, Q):
            out = torch.empty(len(P), len(Q), dtype=torch.complex128, device=DEVICE)
            for i in range(0, len(P), 512):
                d = (P[i:i + 512, None] - Q[None]) % L
                out[i:i + 512] = g[(d[..., 0] * L + d[..., 1]) * L + d[..., 2]]
            return out

        def real_times(A, B):
            return torch.complex(A @ B.real, A @ B.imag)

        eye = torch.eye(len(G), dtype=torch.complex128, device=DEVICE)
        def solve(A, X):
            lu, piv = torch.linalg.lu_factor(A)
            return torch.cat([torch.linalg.lu_solve(lu, piv, part.contiguous()) for part in X.split(256, dim=1)], 1)

        S = real_times(H, real_times(H, table(E, E)).T.contiguous())
        K = -solve(eye - real_times(H, table(E, G)), S)
        self.G, self.M = G, K
        if order == "first":
            A = -1j * (H @ H.T)
            self.A, self.B = A, S1 * eye - solve(K, A).T.contiguous()

    def of(self, y):
        return y[self.G[:, 0], self.G[:, 1], self.G[:, 2]]

    def add(self, out, v):
        out.index_put_((self.G[:, 0], self.G[:, 1], self.G[:, 2]), v, accumulate=True)


def _field(rho, h, mu2, scale):
    """(-Delta_h + mu2) W = scale rho with zero values outside (three points per axis), by sine transforms."""
    out, total = scale * rho, mu2
    sines = []
    for axis, n in enumerate(rho.shape):
        j = torch.arange(1, n + 1, dtype=torch.float64, device=DEVICE)
        sines.append(math.sqrt(2.0 / (n + 1)) * torch.sin(math.pi * j[:, None] * j[None, :] / (n + 1)))
        lam = (2 - 2 * torch.cos(math.pi * j / (n + 1))) / (h * h)
        total = total + lam.reshape([-1 if a == axis else 1 for a in range(3)])
    for turn in range(2):
        for axis, S in enumerate(sines):
            out = (out.movedim(axis, -1) @ S).movedim(-1, axis)
        if turn == 0:
            out = out / total
    return out


def _taylor(case, shape, order, ops, psi, V, steps):
    """Steps of the fourth-order Taylor propagator from (psi, zero auxiliary variables)."""
    h, dt, R = case["h"], case["dt"], case.get("radius", 1)
    batched = psi.dim() == 4
    box = isinstance(ops, _BoxForm)
    aux = None
    if order == "first":
        aux = [torch.zeros_like(ops.of(psi))] if box else [torch.zeros_like(ops.slab(psi, f)) for f in range(6)]
    for _ in range(steps):
        U = V
        if case["kind"] == "orbitals":
            rho = (psi.real ** 2 + psi.imag ** 2).sum(3)
            U = U + LOCAL[0] * rho + LOCAL[1] * rho * rho
            if case["long_range"]:
                U = U + _field(rho, h, 1.0 / YUKAWA["a"] ** 2, 4 * math.pi * YUKAWA["v0"] * YUKAWA["a"])
                U = U + _field(rho, h, 0.0, 2 * math.pi * YUKAWA["e2"])
        U = U[..., None] if batched else U
        y, f = psi, aux
        out, out_f = psi, aux
        for k in range(1, 5):
            dy = _minus_half_laplacian(y, h, R) + U * y
            df = None
            if order == "zeroth":
                if box:
                    ops.add(dy, ops.M @ ops.of(y))
                else:
                    for i in range(6):
                        ops.add(dy, ops.convolve(ops.slab(y, i)), i)
            elif order == "first":
                if box:
                    ops.add(dy, f[0])
                    df = [ops.B @ f[0] + ops.A @ ops.of(y)]
                else:
                    for i in range(6):
                        ops.add(dy, f[i], i)
                    df = [ops.convolve(f[i]) + ops.local(ops.slab(y, i)) for i in range(6)]
            y = (-1j * dt / k) * dy
            out = out + y
            if df is not None:
                f = [(dt / k) * v for v in df]
                out_f = [p + v for p, v in zip(out_f, f)]
        psi, aux = out, out_f
    return psi, aux


def _operators(case, shape, order, window=0, fejer=True):
    if order == "dirichlet":
        return None
    if case["kind"] == "box":
        return _BoxForm(shape, case["h"], case["radius"], order)
    return _Faces(shape, case["h"], case.get("radius", 1), order, window, fejer)


def _flat(aux):
    return torch.cat([a.reshape(-1) for a in aux])


def exact(case, seed):
    fields = _inputs(case, seed)
    if case["kind"] == "uneven":
        psis, auxs = [], []
        for (shape, order), (psi, V) in zip(_uneven_layout(case), fields):
            psi, aux = _taylor(case, shape, order, _operators(case, shape, order), psi, V, case["steps"])
            psis.append(psi)
            if order == "first":
                auxs.append(_flat(aux))
        return {"psi": psis, "aux": auxs}
    shape, order, (psi, V) = _shape(case), case.get("order", "first"), fields
    # a program holds its inputs in the state's type
    if case.get("dtype") == "c64":
        psi, V = psi.to(torch.complex64).to(torch.complex128), V.float().double()
    ops = _operators(case, shape, order, *(_half(case) if case["kind"] == "faces" else ()))
    h3 = case["h"] ** 3
    if case["kind"] == "gradient":
        psi0, V0 = psi.requires_grad_(), V.requires_grad_()
        end = psi0
        # one checkpoint per step: the state alone is kept, each step is run again in the reverse sweep
        aux = [torch.zeros_like(ops.slab(psi, f)) for f in range(6)]
        states = [(psi.detach(), [a.detach() for a in aux])]
        with torch.no_grad():
            for _ in range(case["steps"]):
                states.append(_one_step(case, ops, *states[-1], V.detach()))
        end = states[-1][0].requires_grad_()
        Vl = V.detach().requires_grad_()
        J = h3 * (end * end.conj()).real.sum() if case["objective"] == "prob" else \
            h3 * (end.conj() * (_minus_half_laplacian(end, case["h"], 1) + Vl * end)).sum().real
        lam, gV = torch.autograd.grad(J, (end, Vl), allow_unused=True)
        gV = torch.zeros_like(V) if gV is None else gV
        mu = [torch.zeros_like(a) for a in aux]
        for y, f in reversed(states[:-1]):
            y, f, Vl = y.detach().requires_grad_(), [a.detach().requires_grad_() for a in f], V.detach().requires_grad_()
            y2, f2 = _one_step(case, ops, y, f, Vl)
            g = torch.autograd.grad([y2] + f2, [y, Vl] + f, [lam] + mu)
            lam, gV, mu = g[0], gV + g[1], list(g[2:])
        return {"J": J.detach(), "grad_psi": lam, "grad_V": gV}
    end, aux = _taylor(case, shape, order, ops, psi, V, case["steps"])
    out = {"psi": end}
    if order == "first":
        out["aux"] = _flat(aux)
    if case.get("records"):
        norm = h3 * (end.abs() ** 2).sum()
        lyap = norm
        if order == "first":
            q = torch.linalg.inv(1j * ops.a)
            for a in aux:
                qa = torch.stack([sum(q[i, j] * a[j] for j in range(ops.R)) for i in range(ops.R)], 0)
                lyap = lyap + h3 * (a.conj() * qa).sum().real
        Hy = _minus_half_laplacian(end, case["h"], case["radius"]) + V * end
        energy = h3 * (end.conj() * Hy).sum().real
        out["record"] = torch.stack([norm, lyap, energy, torch.zeros_like(norm)])
    return out


def _one_step(case, ops, psi, aux, V):
    """A step of _taylor with every operation differentiable, for the gradient."""
    y, f = psi, aux
    out, out_f = psi, aux
    for k in range(1, 5):
        dy = _minus_half_laplacian(y, case["h"], 1) + V * y
        dy = dy.clone()
        for i in range(6):
            ops.add(dy, f[i], i)
        df = [ops.convolve(f[i]) + ops.local(ops.slab(y, i)) for i in range(6)]
        y = (-1j * case["dt"] / k) * dy
        f = [(case["dt"] / k) * v for v in df]
        out, out_f = out + y, [p + v for p, v in zip(out_f, f)]
    return out, out_f
