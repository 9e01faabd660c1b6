"""Timed cases of the framework's public entry points.

Each case is a plain dict whose ``op`` names a path:

  step        set a phonon field, solve (M^T M) u = Phi, action S_F and force dS_F/dx: what every
              evaluation of the fermion force of a hybrid Monte Carlo update does
  autograd    the same through the differentiable ``fermion_action`` (forward and backward)
  green       G xi for a block of Rademacher vectors: the solves of a measurement
  apply       one operator or preconditioner apply on a block of right-hand sides
  batch       many independent systems of uneven size solved together
  trajectory  one hybrid Monte Carlo update of the field, shortened to a few steps
  estimators  space-time averages from given pairs (xi, G xi): Green's function and four-point products
  ssh         set field, preconditioned solve, action and force of the SSH-type coupling

Fields, pseudofermions and random vectors follow the recipes of the repository's workloads (iid,
shifted iid, autoregressive in imaginary time, checkerboard density wave), drawn on the device from
the seed alone.  Solves run to relative residuals near 1e-13, where two correct solvers agree to the
digits a double comparison needs (the condition number turns a residual of 1e-8 into a solution
error of 1e-6); the tolerance only scales the iteration count.

``exact`` forms the same results in plain float64 torch: the operator from reshapes and rolls, textbook
conjugate gradients, torch's FFT for circulants and cross-correlations, autograd for the SSH force.
"""

import cmath
import math

import torch

from paper_2203_01291_amd.hmc import PhononHMC
from paper_2203_01291_amd.measure import GreenMeasurement
from paper_2203_01291_amd.solver import FermionBatch, FermionSolver, fermion_action
from paper_2203_01291_amd.ssh import SSHSolver

F64 = torch.float64

# Model parameters of the workloads: (dtau, mu, omega, alpha) by field recipe.
_MODEL = {"iid": (0.1, 0.0, 1.0, 1.0), "cdw": (0.1, 0.0, 0.5, 1.5), "ar1": (0.05, -0.2, 1.0, 1.2),
          "shift": (0.05, 0.0, 1.0, 1.5)}


# ------------------------------------------------------------------- the cases
def listed():
    return [
        # The smallest lattice of the workloads, FP64, one pseudofermion: launches and waits.
        dict(name="step_L4", op="step", L=4, Ltau=40, field="iid", nrhs=1, prec="f64", precond=True,
             a1=1.0, a2=1.0, tol=1e-13),
        # Both pseudofermion fields of a mid-size density-wave lattice, FP64 with the paper's orders.
        dict(name="step_L16_cdw", op="step", L=16, Ltau=160, field="cdw", nrhs=2, prec="f64", precond=True,
             a1=1.0, a2=1.0, tol=1e-13),
        # The benchmark's lattice: one FP32-refined preconditioned solve.
        dict(name="step_L32", op="step", L=32, Ltau=400, field="ar1", nrhs=1, prec="f32_refined",
             precond=True, a1=0.15, a2=12.0, tol=1e-13),
        # The largest lattice, one right-hand side.
        dict(name="step_L64", op="step", L=64, Ltau=400, field="shift", nrhs=1, prec="f32_refined",
             precond=True, a1=0.05, a2=12.0, tol=1e-13),
        # A ragged lattice through autograd, plain FP64 conjugate gradients, three right-hand sides.
        dict(name="autograd_L18", op="autograd", L=18, Ltau=84, field="iid", nrhs=3, prec="f64",
             precond=False, a1=1.0, a2=1.0, tol=1e-13),
        # A measurement's block of ten random vectors.
        dict(name="green_L32_x10", op="green", L=32, Ltau=160, field="iid", nrhs=10, prec="f32_refined",
             precond=True, a1=0.15, a2=12.0, tol=1e-13),
        # The operator beyond the last-level cache: many right-hand sides sharing one large field.
        dict(name="apply_MTM_L64_x40", op="apply", kind="MTM", L=64, Ltau=400, field="shift", nrhs=40,
             dtype="f64", a1=1.0, a2=1.0),
        # The preconditioner on ten FP32 vectors of the benchmark's lattice.
        dict(name="apply_FFT_L32_x10", op="apply", kind="FFT", L=32, Ltau=400, field="ar1", nrhs=10,
             dtype="f32", a1=0.15, a2=12.0),
        # Uneven systems in one call, pseudofermion-like right-hand sides.
        dict(name="batch_24x12", op="batch", nsys=24, Lmin=8, Lmax=24, Ltau=100, nrhs=12, precond=True,
             a1=1.0, a2=1.0, tol=1e-13),
        # An update of a mid-size lattice, four steps instead of the usual hundred.
        dict(name="trajectory_L16", op="trajectory", L=16, Ltau=160, field="cdw", steps=4, tol=1e-13,
             prec="f32_refined", a1=0.25, a2=4.0),
        # The estimators of ten random vectors on the benchmark's lattice.
        dict(name="estimators_L32_x10", op="estimators", L=32, Ltau=400, nrhs=10),
        # The SSH-type coupling, FP64, preconditioned by the adiabatic preconditioner.
        dict(name="ssh_L20", op="ssh", L=20, Ltau=120, field="iid", g=0.2, nrhs=2, prec="f64", precond=True,
             a1=0.25, a2=4.0, tol=1e-13),
    ]


def _log_int(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, step * int(round(v / step))))


def _slices_ok(Ltau):
    """Imaginary-time extents every path of the framework takes."""
    H = Ltau // 2
    half = any(H % h == 0 and H // h <= 32 for h in (1, 2, 3, 4, 5, 8, 10, 16, 20))
    return Ltau % 2 == 0 and half and any(Ltau % p == 0 and Ltau // p <= 64 for p in range(1, 65))


def _slices(rng, lo, hi):
    want = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min((T for T in range(lo, hi + 1) if _slices_ok(T)), key=lambda T: abs(T - want))


def draw(rng):
    """One more case: sides 4 to 64 (every even side), 20 to 400 slices, 1 to 40 right-hand sides."""
    op = rng.choice(["step", "step", "step", "autograd", "green", "apply", "apply", "batch", "trajectory",
                     "estimators", "ssh"])
    a1, a2 = rng.choice([(1.0, 1.0), (0.25, 4.0), (0.15, 12.0)])
    field = rng.choice(["iid", "cdw", "ar1", "shift"])
    prec = rng.choice(["f64", "f32_refined"])
    if op in ("step", "autograd", "green"):
        L, T = _log_int(rng, 4, 48, 2), _slices(rng, 20, 160)
        most = max(1, min(12 if op == "green" else 4, 1000000 // (L * L * T)))
        return dict(op=op, L=L, Ltau=T, field=field, nrhs=_log_int(rng, 1, most), prec=prec,
                    precond=rng.random() < 0.75, a1=a1, a2=a2, tol=1e-13)
    if op == "apply":
        L, T = _log_int(rng, 4, 64, 2), _slices(rng, 20, 400)
        most = max(1, min(40, 60000000 // (L * L * T)))
        return dict(op=op, kind=rng.choice(["M", "MT", "MTM", "F", "FT", "FFT"]), L=L, Ltau=T, field=field,
                    nrhs=_log_int(rng, 1, most), dtype=rng.choice(["f64", "f32"]), a1=a1, a2=a2)
    if op == "batch":
        lo = rng.choice([4, 6, 8])
        return dict(op=op, nsys=_log_int(rng, 3, 24), Lmin=lo, Lmax=rng.choice([12, 16, 20]), Ltau=_slices(rng, 20, 100),
                    nrhs=_log_int(rng, 1, 12), precond=rng.random() < 0.5, a1=1.0, a2=1.0, tol=1e-13)
    if op == "trajectory":
        return dict(op=op, L=_log_int(rng, 4, 16, 2), Ltau=_slices(rng, 20, 120), field=field,
                    steps=rng.randint(1, 4), tol=1e-13, prec=prec, a1=a1, a2=a2)
    if op == "estimators":
        L, T = _log_int(rng, 4, 48, 2), _slices(rng, 20, 200)
        return dict(op=op, L=L, Ltau=T, nrhs=_log_int(rng, 2, 10))
    return dict(op=op, L=_log_int(rng, 4, 20, 2), Ltau=_slices(rng, 20, 120), field="iid", g=0.2,
                nrhs=_log_int(rng, 1, 4), prec=prec, precond=rng.random() < 0.75, a1=a1, a2=a2, tol=1e-13)


# ------------------------------------------------------------------- inputs
def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _generator(seed):
    return torch.Generator(device=_device()).manual_seed(int(seed))


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, dtype=F64, device=_device())


def _signs(g, *shape):
    return (torch.randint(0, 2, shape, generator=g, device=_device()) * 2 - 1).to(F64)


def _ar1(g, T, N, sigma):
    """Stationary autoregressive process along tau (coefficient 0.95), independent sites."""
    noise, rho = _randn(g, T, N), 0.95
    out = torch.empty_like(noise)
    out[0] = sigma * noise[0]
    for k in range(1, T):
        out[k] = rho * out[k - 1] + sigma * math.sqrt(1 - rho * rho) * noise[k]
    return out


def _field(kind, g, L, T):
    N = L * L
    if kind == "iid":
        return _randn(g, T, N)
    if kind == "shift":
        return _randn(g, T, N) + 0.5
    if kind == "ar1":
        return _ar1(g, T, N, 1.0 / math.sqrt(_MODEL[kind][2]))
    s = torch.arange(L, device=_device())
    sign = (1.0 - 2.0 * ((s[:, None] + s[None, :]) % 2)).to(F64).reshape(N)
    return 0.8 * sign + _ar1(g, T, N, 0.3)


def _inputs(case, seed):
    """The host-side draws of a case, as a dict of tensors (and the models they belong to)."""
    g, op = _generator(seed), case["op"]
    if op == "batch":
        systems, sides = [], torch.Generator().manual_seed(int(case["nsys"]) * 7919 + int(case["Ltau"]))
        for _ in range(case["nsys"]):
            L = case["Lmin"] + 2 * int(torch.randint(0, (case["Lmax"] - case["Lmin"]) // 2 + 1, (), generator=sides))
            m = _Plain(dict(case, L=L, field="iid"))
            x = _field("iid", g, L, case["Ltau"])
            phi = _randn(g, case["nrhs"], case["Ltau"], L * L)
            systems.append((m, x, m.at(x).MT(phi).contiguous()))
        return dict(systems=systems)
    L, T = case["L"], case["Ltau"]
    if op == "estimators":
        xi = _signs(g, case["nrhs"], T, L * L)
        return dict(xi=xi, gxi=(0.5 * xi + 0.3 * _randn(g, case["nrhs"], T, L * L)).contiguous())
    x0 = _field(case["field"], g, L, T)
    if op == "apply":
        v = _randn(g, case["nrhs"], T, L * L)
        return dict(x=x0, v=v if case["dtype"] == "f64" else v.float())
    if op == "green":
        return dict(x=x0, xi=_signs(g, case["nrhs"], T, L * L))
    if op == "trajectory":
        return dict(x=x0, R=_randn(g, 2, T, L * L), Rp=_randn(g, T, L * L))
    phi = _randn(g, case["nrhs"], T, L * L)
    Phi = _plain(case).at(x0).MT(phi).contiguous()
    return dict(x=(x0 + 0.1 * _randn(g, T, L * L)).contiguous(), Phi=Phi)


# ------------------------------------------------------------------- the timed path
class _Lattice:
    def __init__(self, L, T, m):
        self.L, self.Ltau, self.dtau, self.t, self.mu, self.alpha = L, T, m.dtau, 1.0, m.mu, m.alpha


def _solver(case, max_rhs):
    m = _plain(case)
    return FermionSolver(case["L"], case["Ltau"], m.dtau, 1.0, m.mu, m.alpha, max_rhs=max_rhs)


def prepare(case, seed):
    d, op = _inputs(case, seed), case["op"]
    st = dict(case=case, **d)
    if op == "batch":
        st = dict(case=case, batch=FermionBatch([(_Lattice(m.L, m.T, m), x, b) for m, x, b in d["systems"]]))
    elif op in ("step", "autograd"):
        st["solver"] = _solver(case, case["nrhs"])
    elif op in ("green", "estimators"):
        st["solver"] = _solver(dict(case, field=case.get("field", "iid")), case["nrhs"])
        st["meas"] = GreenMeasurement(st["solver"])
        if op == "green":
            st["solver"].set_field(d["x"], case["a1"], case["a2"])
    elif op == "apply":
        st["solver"] = _solver(case, case["nrhs"])
        st["solver"].set_field(d["x"], case["a1"], case["a2"])
        st["out"] = torch.empty_like(d["v"])
    elif op == "trajectory":
        st["solver"] = _solver(case, 2)
        om = _plain(case).omega
        st["hmc"] = PhononHMC(st["solver"], om, om, 1.0 / (100.0 * om), Nt=case["steps"], nt=10, nfields=2,
                              a1=case["a1"], a2=case["a2"], force_tol=case["tol"], action_tol=case["tol"],
                              precond=True, prec=case["prec"])
        st["work"], st["p"] = torch.empty_like(d["x"]), torch.empty_like(d["x"])
    else:
        m = _plain(case)
        st["solver"] = SSHSolver(case["L"], case["Ltau"], m.dtau, 1.0, m.mu, m.alpha, case["g"], max_rhs=case["nrhs"])
        if case["precond"]:
            st["pc"] = _solver(case, case["nrhs"])
            st["solver"].attach_preconditioner(st["pc"], case["a1"], case["a2"])
    return st


def run(st):
    case, op = st["case"], st["case"]["op"]
    if op == "batch":
        st["batch"].solve(tol=case["tol"], precond=case["precond"], a1=case["a1"], a2=case["a2"])
        return list(st["batch"].u)
    if op == "estimators":
        return dict(average=st["meas"].green_average(st["xi"], st["gxi"]),
                    pairs=st["meas"].pair_products(st["xi"], st["gxi"]))
    if op == "green":
        return st["meas"].green_vectors(st["xi"], tol=case["tol"], precond=case["precond"], prec=case["prec"])[0]
    s = st["solver"]
    if op == "apply":
        if case["kind"] in ("M", "MT", "MTM"):
            return s.matvec(st["v"], case["kind"], out=st["out"])
        return s.precond(st["v"], case["kind"], out=st["out"])
    if op == "trajectory":
        x = st["work"].copy_(st["x"])
        h = st["hmc"].trajectory(x, st["R"], st["Rp"], 0.0, p_out=st["p"])
        return dict(x=x, p=st["p"], H_i=h["H_i"], H_f=h["H_f"])
    how = dict(tol=case["tol"], prec=case["prec"], precond=case["precond"])
    if op == "autograd":
        x = st["x"].detach().requires_grad_(True)
        S = fermion_action(x, st["Phi"], s, a1=case["a1"], a2=case["a2"], **how)
        S.backward()
        return dict(S=S.detach(), grad=x.grad)
    if op == "step":
        s.set_field(st["x"], case["a1"], case["a2"])
    else:
        s.set_field(st["x"])
    u, _ = s.solve(st["Phi"], **how)
    return dict(u=u, S=s.action(st["Phi"], u), grad=s.force(u))


# ------------------------------------------------------------------- needed work
def work(case):
    """Inputs read once and outputs written once; for solves the operations of a nominal iteration
    count that grows with the inverse temperature (40 operations per unknown and iteration)."""
    op = case["op"]
    if op == "batch":
        Ls = range(case["Lmin"], case["Lmax"] + 1, 2)
        unknowns = case["nsys"] * case["Ltau"] * sum(L * L for L in Ls) / len(Ls)
        return dict(bytes=8 * unknowns * (1 + 2 * case["nrhs"]),
                    flops=40 * unknowns * case["nrhs"] * (40 + 40 * 0.1 * case["Ltau"]))
    d = case["L"] ** 2 * case["Ltau"]
    if op == "estimators":
        n = case["nrhs"]
        transforms = 2 * n + 1 + 4 * (n * (n - 1) // 2) + n + 3
        return dict(bytes=8 * d * (2 * n + 4), flops=2.5 * d * math.log2(d) * transforms)
    if op == "apply":
        w, n = (8 if case["dtype"] == "f64" else 4), case["nrhs"]
        each = {"M": 10, "MT": 10, "MTM": 20}.get(case["kind"], 60 if case["kind"] == "FFT" else 30)
        return dict(bytes=w * d * (2 * n + (1 if len(case["kind"]) and case["kind"][0] == "M" else 0)), flops=each * d * n)
    beta = _MODEL[case["field"]][0] * case["Ltau"]
    iters = 40 + 40 * beta
    n = case.get("nrhs", 2)
    if op == "trajectory":
        return dict(bytes=8 * d * 6, flops=40 * d * 2 * iters * (case["steps"] + 2))
    return dict(bytes=8 * d * (2 + 2 * n), flops=40 * d * n * iters)


# ------------------------------------------------------------------- plain float64 reference
class _Plain:
    """M of a lattice in plain torch: at(x) installs a field; vectors are [..., Ltau, N]."""

    def __init__(self, case):
        self.L, self.T = case["L"], case["Ltau"]
        self.dtau, self.mu, self.omega, self.alpha = _MODEL[case["field"]]
        self.ch, self.sh = math.cosh(self.dtau), math.sinh(self.dtau)

    def at(self, x):
        self.E = torch.exp(-self.dtau * (self.alpha * x - self.mu))
        return self

    def _plaq(self, v):
        v = v.reshape(v.shape[:-2] + (self.L // 2, 2, self.L // 2, 2))
        v = self.ch * v + self.sh * v.flip(-1)
        v = self.ch * v + self.sh * v.flip(-3)
        return v.reshape(v.shape[:-4] + (self.L, self.L))

    def _odd(self, v):
        return self._plaq(v.roll((-1, -1), (-2, -1))).roll((1, 1), (-2, -1))

    def C(self, v):
        g = v.reshape(v.shape[:-1] + (self.L, self.L))
        return self._plaq(self._odd(g)).reshape(v.shape)

    def CT(self, v):
        g = v.reshape(v.shape[:-1] + (self.L, self.L))
        return self._odd(self._plaq(g)).reshape(v.shape)

    def moved(self, v):
        """B_tau v~_{tau-1} with the antiperiodic wrap."""
        s = v.roll(1, -2)
        s[..., 0, :].neg_()
        return self.E * self.C(s)

    def M(self, v):
        return v - self.moved(v)

    def MT(self, w):
        s = self.CT(self.E * w).roll(-1, -2)
        s[..., -1, :].neg_()
        return w - s

    def MTM(self, v):
        return self.MT(self.M(v))

    def force(self, x, u):
        y = self.moved(u)
        return (-2.0 * self.dtau * self.alpha * (u - y) * y).sum(0)


class _PlainSSH(_Plain):
    """The SSH-type operator: every bond of the four families with its own hopping."""

    def __init__(self, case):
        super().__init__(case)
        self.g = case["g"]

    def at(self, x):
        super().at(x)
        g = x.reshape(self.T, self.L, self.L)
        self.f = []
        for axis, odd in ((-1, 0), (-2, 0), (-1, 1), (-2, 1)):
            s = g.roll(-odd, axis)
            lo = s.reshape(self._pairs(s.shape, axis)).unbind(axis if axis == -1 else -2)
            tb = self.dtau * (1.0 - self.g * (lo[1] - lo[0]))
            d = -1 if axis == -1 else -2
            self.f.append((axis, odd, torch.stack((tb, tb), d)))
        return self

    def _pairs(self, shape, axis):
        h = self.L // 2
        return shape[:-2] + ((self.L, h, 2) if axis == -1 else (h, 2, self.L))

    def _family(self, v, k):
        axis, odd, tb = self.f[k]
        s = v.roll(-odd, axis)
        s = s.reshape(self._pairs(s.shape, axis))
        s = torch.cosh(tb) * s + torch.sinh(tb) * s.flip(-1 if axis == -1 else -2)
        return s.reshape(v.shape).roll(odd, axis)

    def _through(self, v, order):
        g = v.reshape(v.shape[:-1] + (self.L, self.L))
        for k in order:
            g = self._family(g, k)
        return g.reshape(v.shape)

    def C(self, v):
        return self._through(v, (3, 2, 1, 0))

    def CT(self, v):
        return self._through(v, (0, 1, 2, 3))

    def force(self, x, u):
        """d/dx of -|M(x) u|^2 at fixed u, which is dS_F/dx."""
        z = x.detach().clone().requires_grad_(True)
        with torch.enable_grad():
            self.at(z)
            (-(self.M(u) ** 2).sum()).backward()
        self.at(x)
        return z.grad


class _Series:
    """The truncated Chebyshev series F, F^T and F F^T of a field, all frequencies side by side."""

    def __init__(self, m, a1, a2):
        self.m, T, dev = m, m.T, m.E.device
        self.dbar = m.E.mean(0)
        self.lo = float(self.dbar.min()) * math.exp(-4.0 * m.dtau)
        self.db = float(self.dbar.max()) * math.exp(4.0 * m.dtau) - self.lo
        self.c = torch.zeros(T, 1024, dtype=torch.complex128, device=dev)
        for w in range(T):
            n = min(1024, max(1, math.floor(self.db * (a1 / (2 * math.pi * (min(w, T - 1 - w) + 0.5) / T) + a2))))
            th = math.pi * (torch.arange(2 * n, dtype=F64, device=dev) + 0.5) / (2 * n)
            f = 1.0 / (1.0 - cmath.exp(-2j * math.pi * (w + 0.5) / T) * (self.lo + (torch.cos(th) + 1.0) * self.db / 2.0))
            k = torch.arange(n, dtype=F64, device=dev)
            self.c[w, :n] = (torch.cos(k[:, None] * th) * f).sum(1) / n
            self.c[w, 0] *= 0.5
        self.most = int((self.c.abs().sum(0) > 0).sum())
        self.twist = torch.exp(-1j * math.pi * torch.arange(T, dtype=F64, device=dev) / T)[:, None]

    def _A(self, v, transpose):
        b = self.m.CT(self.dbar * v) if transpose else self.dbar * self.m.C(v)
        return (2.0 / self.db) * (b - self.lo * v) - v

    def _blocks(self, v, transpose):
        c = self.c.conj() if transpose else self.c
        out, old, cur = c[:, :1] * v, v, None
        for k in range(1, self.most):
            old, cur = (v, self._A(v, transpose)) if k == 1 else (cur, 2.0 * self._A(cur, transpose) - old)
            out = out + c[:, k:k + 1] * cur
        return out

    def __call__(self, v, kind):
        z = torch.fft.fft(self.twist * v, dim=-2)
        if kind in ("FT", "FFT"):
            z = self._blocks(z, True)
        if kind in ("F", "FFT"):
            z = self._blocks(z, False)
        return (self.twist.conj() * torch.fft.ifft(z, dim=-2)).real


def _plain(case):
    return (_PlainSSH if case["op"] == "ssh" else _Plain)(case)


def _dot(a, b):
    return (a * b).sum((-2, -1), keepdim=True)


def _cg(m, b, tol=1e-15, most=60000):
    """Textbook conjugate gradients on M^T M, restarted from its true residual until it stops falling."""
    u, bb = torch.zeros_like(b), _dot(b, b)
    for _ in range(3):
        r = b - m.MTM(u)
        p, rr = r.clone(), _dot(r, r)
        for k in range(most):
            if k % 50 == 0 and bool((rr <= tol * tol * bb).all()):
                break
            q = m.MTM(p)
            a = rr / _dot(p, q).clamp_min(1e-300)
            u = u + a * p
            r = r - a * q
            new = _dot(r, r)
            p = r + (new / rr.clamp_min(1e-300)) * p
            rr = new
    return u


def _boson_force(m, x):
    return (m.dtau * m.omega ** 2 * x + (2 * x - x.roll(1, 0) - x.roll(-1, 0)) / m.dtau - m.dtau * m.alpha)


def _circulant(eig, v):
    return torch.fft.ifft(eig[:, None] * torch.fft.fft(v, dim=0), dim=0).real


def _hamiltonian(m, x, p, eig, SF):
    SB = 0.5 * m.dtau * (m.omega ** 2 * (x * x).sum() + (((x.roll(-1, 0) - x) / m.dtau) ** 2).sum())
    return SB - m.dtau * m.alpha * x.sum() + SF + 0.5 * (p * _circulant(1.0 / eig, p)).sum()


def _trajectory(case, d):
    m, x = _plain(case), d["x"].clone()
    om, T = m.omega, m.T
    w = torch.arange(T, dtype=F64, device=x.device)
    stiff = 4.0 / m.dtau ** 2 * torch.sin(math.pi * w / T) ** 2
    eig = m.dtau * (2 * om * om + stiff) / (2 * om * om)
    dt, h = 1.0 / (100.0 * om), 1.0 / (1000.0 * om)
    Phi = m.at(x).MT(d["R"])
    p = _circulant(eig.sqrt(), d["Rp"])
    H_i = _hamiltonian(m, x, p, eig, 0.5 * (d["R"] ** 2).sum())
    kick = lambda: 0.5 * m.force(x, _cg(m.at(x), Phi))  # noqa: E731
    F = kick()
    for _ in range(case["steps"]):
        p = p - 0.5 * dt * F
        for _ in range(10):
            p = p - 0.5 * h * _boson_force(m, x)
            x = x + h * _circulant(1.0 / eig, p)
            p = p - 0.5 * h * _boson_force(m, x)
        u = _cg(m.at(x), Phi)
        F = 0.5 * m.force(x, u)
        p = p - 0.5 * dt * F
    H_f = _hamiltonian(m, x, p, eig, 0.5 * (Phi * u).sum())
    return dict(x=x, p=p, H_i=float(H_i), H_f=float(H_f))


def _estimators(case, d):
    L, T, n = case["L"], case["Ltau"], case["nrhs"]
    xi, gx = (d[k].reshape(n, T, L, L) for k in ("xi", "gxi"))
    ax, cal = (-3, -2, -1), float(T * L * L)

    def corr(a, b):
        return torch.fft.ifftn(torch.fft.fftn(a, dim=ax).conj() * torch.fft.fftn(b, dim=ax), dim=ax).real

    avg, pairs = 0.0, torch.zeros(3, T, L, L, dtype=F64, device=xi.device)
    for a, b in zip(xi, gx):
        avg = avg + corr(torch.cat([a, -a]), torch.cat([b, -b]))[:T] / (2 * cal * n)
    for a in range(n):
        for b in range(a + 1, n):
            pairs[0] += corr(xi[a] * xi[b], gx[a] * gx[b])
            pairs[1] += corr(xi[a] * gx[a], xi[b] * gx[b])
            pairs[2] += corr(xi[a] * gx[b], xi[b] * gx[a])
    return dict(average=avg, pairs=pairs / (cal * (n * (n - 1) // 2)))


def exact(case, seed):
    d, op = _inputs(case, seed), case["op"]
    if op == "batch":
        return [_cg(m.at(x), b) for m, x, b in d["systems"]]
    if op == "estimators":
        return _estimators(case, d)
    if op == "trajectory":
        return _trajectory(case, d)
    m = _plain(case).at(d["x"])
    if op == "apply":
        if case["kind"] in ("F", "FT", "FFT"):
            series = _Series(m, case["a1"], case["a2"])
            return torch.stack([series(v.double(), case["kind"]) for v in d["v"]])
        return torch.stack([getattr(m, case["kind"])(v.double()) for v in d["v"]])
    if op == "green":
        return _cg(m, m.MT(d["xi"]))
    u = _cg(m, d["Phi"])
    S, grad = (d["Phi"] * u).sum((-2, -1)), m.force(d["x"], u)
    return dict(S=S.sum(), grad=grad) if op == "autograd" else dict(u=u, S=S, grad=grad)
