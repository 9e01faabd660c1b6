"""z = F F^T r as the solvers apply it: after one iteration from a zero guess the iterate is alpha z,
z = F F^T b, so it shows the preconditioner inside a solve itself."""

import numpy as np
import pytest
import torch

from oracle import lattice as OL
from oracle import precond as OP
from paper_2203_01291_amd.solver import FermionSolver

pytestmark = pytest.mark.gpu


def _solver(lat, max_rhs):
    return FermionSolver(lat.L, lat.Ltau, lat.dtau, lat.t, lat.mu, lat.alpha, max_rhs=max_rhs)


# Blocks applied as matrices gain for few right-hand sides and long series only: a matrix's rows serve one
# vector after the other.  A field handed over through set_fields has no matrices and runs the same kernels
# otherwise, so the iterates agree to the last bit exactly where no matrix was used.
@pytest.mark.parametrize("L,Ltau,a,nrhs,matrices", [
    (16, 160, (1.0, 1.0), 1, ["f64", "f32_refined"]), (16, 160, (1.0, 1.0), 4, ["f64", "f32_refined"]),
    (16, 160, (1.0, 1.0), 16, []), (16, 160, (1.0, 1.0), 17, []), (16, 160, (0.15, 12.0), 8, []),
    (12, 100, (1.0, 1.0), 40, []), (32, 160, (1.0, 1.0), 2, ["f64", "f32_refined"]),
    (24, 100, (1.0, 1.0), 8, ["f64"]), (24, 100, (1.0, 1.0), 32, [])])
@pytest.mark.parametrize("prec", ["f64", "f32_refined"])
def test_matrices_by_right_hand_sides(L, Ltau, a, nrhs, matrices, prec):
    lat = OL.Lattice(L, Ltau, 0.1, 1.0, 0.0, 1.0)
    rng = np.random.default_rng(L + Ltau + nrhs)
    b = torch.from_numpy(rng.standard_normal((nrhs, Ltau, lat.N))).cuda()
    x = torch.from_numpy(rng.standard_normal((Ltau, lat.N))).cuda()
    s = _solver(lat, nrhs)
    how = dict(tol=1e-30, maxiter=1, max_outer=1, precond=True, prec=prec)
    s.set_fields(x, rhs_per_field=nrhs, a1=a[0], a2=a[1])
    series, _ = s.solve(b, **how)
    s.set_field(x, *a)
    u, st = s.solve(b, **how)
    assert all(v["iters"] == 1 for v in st)
    assert torch.equal(u, series) == (prec not in matrices)


# One iteration's iterate over its norm, per right-hand side.
def _direction(solver, b, prec, **kw):
    u, st = solver.solve(b, tol=1e-30, maxiter=1, max_outer=1, precond=True, prec=prec, **kw)
    assert all(v["iters"] == 1 for v in st)
    u = u.cpu().numpy()
    return u / np.sqrt((u * u).sum((1, 2), keepdims=True))


def _close(got, b, pcs, prec):
    for r, pc in enumerate(pcs):
        ref = pc.apply_FFt(b[r])
        ref /= np.sqrt((ref * ref).sum())
        # rounding of a series of a few tens of terms in each precision, as for a single apply
        assert np.max(np.abs(got[r] - ref)) < (1e-12 if prec == "f64" else 1e-5) * np.max(np.abs(ref)), r


# A shared field (series, matrices where they gain), a field per right-hand side (series only) and another
# shared field after it, whose solve must not meet a matrix of an earlier one.  In one launch: one wave per
# frequency with and without matrices (L = 4, 6, 8), several frequencies per workgroup (L = 22), Ltau / 2
# odd (L = 10).  In slots: every form of the series kernel, with and without matrices.
@pytest.mark.parametrize("L,Ltau", [(4, 2), (4, 100), (4, 128), (6, 56), (8, 32), (10, 18), (22, 4),
                                    (8, 100), (10, 160), (16, 80), (20, 60), (24, 40), (30, 40), (32, 40), (34, 8),
                                    (48, 6)])
@pytest.mark.parametrize("prec", ["f64", "f32_refined"])
def test_direction_of_a_solve(L, Ltau, prec):
    lat = OL.Lattice(L, Ltau, 0.1, 1.0, -0.1, 1.1)
    rng = np.random.default_rng(11 * L + Ltau)
    xs = rng.standard_normal((2, Ltau, lat.N)) * np.array([1.0, 0.5])[:, None, None]
    b = rng.standard_normal((2, Ltau, lat.N))
    C = OL.sparse_C(lat).tocsr()
    pcs = [OP.Preconditioner(lat, x, 1.0, 1.0, C=C) for x in xs]
    xg, bg = torch.from_numpy(xs).cuda(), torch.from_numpy(b).cuda()
    s = _solver(lat, 2)
    s.set_field(xg[0])
    _close(_direction(s, bg[:1].contiguous(), prec), b, pcs[:1], prec)
    _close(_direction(s, bg, prec), b, pcs[:1] * 2, prec)
    s.set_fields(xg)
    _close(_direction(s, bg, prec), b, pcs, prec)
    s.set_field(xg[1])
    _close(_direction(s, bg, prec), b, pcs[1:] * 2, prec)


# Solves captured with and without the field, replayed after eager changes of it, against eager solves of
# handles that never met another field.
@pytest.mark.parametrize("prec", ["f64", "f32_refined"])
def test_direction_under_capture(prec):
    lat = OL.Lattice(16, 80, 0.1, 1.0, 0.0, 1.0)
    rng = np.random.default_rng(3)
    xs = [torch.from_numpy(c * rng.standard_normal((lat.Ltau, lat.N))).cuda() for c in (1.0, 0.4, 1.3)]
    b = torch.from_numpy(rng.standard_normal((1, lat.Ltau, lat.N))).cuda()
    how = dict(tol=1e-30, maxiter=1, max_outer=1, precond=True, prec=prec)
    want = []
    for x in xs:
        s = _solver(lat, 1)
        s.set_field(x)
        want.append(s.solve(b, **how)[0])
    s = _solver(lat, 1)
    x, u = xs[0].clone(), torch.zeros_like(b)
    s.set_field(x)
    st = torch.empty(4, dtype=torch.float64, device="cuda")
    s.solve_async(b, u, stats=st, zero_guess=True, **how)
    torch.cuda.synchronize()
    solve_only, both = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(solve_only):
        s.solve_async(b, u, stats=st, zero_guess=True, **how)
    with torch.cuda.graph(both):
        s.set_field(x)
        s.solve_async(b, u, stats=st, zero_guess=True, **how)

    def same(a, k):  # series or matrix: the same operator to rounding
        assert float((a - want[k]).norm() / want[k].norm()) < (1e-12 if prec == "f64" else 1e-5)

    for k in (1, 2, 0, 0, 2):
        s.set_field(xs[k])
        solve_only.replay()
        same(u, k)
        same(s.solve(b, **how)[0], k)
        x.copy_(xs[(k + 1) % 3])
        both.replay()
        same(u, (k + 1) % 3)
        same(s.solve(b, **how)[0], (k + 1) % 3)


# In the workgroups of a batch, at the shapes of the tests of whole solves.
@pytest.mark.parametrize("shapes", [[(4, 6, 2), (6, 8, 1)], [(10, 42, 2), (12, 40, 1), (8, 100, 1)],
                                    [(24, 60, 1), (16, 32, 2)], [(32, 20, 1), (22, 24, 1)], [(4, 20, 1100)]])
@pytest.mark.parametrize("tune", [False, True])
def test_direction_of_a_batch(shapes, tune):
    from paper_2203_01291_amd.solver import FermionBatch
    systems, host = [], []
    for n, (L, Ltau, nrhs) in enumerate(shapes):
        lat = OL.Lattice(L, Ltau, 0.1, 1.0, 0.1, 1.0)
        rng = np.random.default_rng(17 * n + L)
        x = rng.standard_normal((Ltau, lat.N))
        b = rng.standard_normal((nrhs, Ltau, lat.N))
        systems.append((lat, torch.from_numpy(x).cuda(), torch.from_numpy(b).cuda()))
        host.append((b, OP.Preconditioner(lat, x, 1.0, 1.0, C=OL.sparse_C(lat).tocsr())))
    batch = FermionBatch(systems)
    if tune:
        batch.tune(tol=1e-30, maxiter=1, precond=True)
    stats = batch.solve(tol=1e-30, maxiter=1, precond=True)
    assert all(st["iters"] == 1 for st in stats)
    for (b, pc), u in zip(host, batch.u):
        u = u.cpu().numpy()[:3]
        _close(u / np.sqrt((u * u).sum((1, 2), keepdims=True)), b, [pc] * len(u), "f32_refined")


# The SSH solve takes the adiabatic preconditioner of its on-site factor.
@pytest.mark.parametrize("L,Ltau,nrhs", [(6, 56, 1), (16, 80, 2), (32, 40, 1)])
@pytest.mark.parametrize("prec", ["f64", "f32_refined"])
def test_direction_of_an_ssh_solve(L, Ltau, nrhs, prec):
    from paper_2203_01291_amd.ssh import SSHSolver
    lat = OL.Lattice(L, Ltau, 0.1, 1.0, -0.1, 0.9)
    rng = np.random.default_rng(L)
    x = 0.6 * rng.standard_normal((Ltau, lat.N))
    b = rng.standard_normal((nrhs, Ltau, lat.N))
    s = SSHSolver(L, Ltau, 0.1, 1.0, -0.1, 0.9, 0.2, max_rhs=nrhs)
    s.attach_preconditioner(_solver(lat, nrhs), 1.0, 1.0)
    s.set_field(torch.from_numpy(x).cuda())
    pc = OP.Preconditioner(lat, x, 1.0, 1.0, C=OL.sparse_C(lat).tocsr())
    _close(_direction(s, torch.from_numpy(b).cuda(), prec), b, [pc] * nrhs, prec)


# An apply of its own is a function of the field and its input: the same bits before and after solves,
# which use matrices.
@pytest.mark.parametrize("L,Ltau", [(6, 56), (16, 80), (32, 60)])
def test_apply_does_not_depend_on_solves(L, Ltau):
    lat = OL.Lattice(L, Ltau, 0.1, 1.0, 0.0, 1.0)
    rng = np.random.default_rng(L)
    v = torch.from_numpy(rng.standard_normal((1, Ltau, lat.N))).cuda()
    s = _solver(lat, 1)
    s.set_field(torch.from_numpy(rng.standard_normal((Ltau, lat.N))).cuda())
    before = [s.precond(w, "FFT") for w in (v, v.float())]
    for prec in ("f64", "f32_refined"):
        s.solve(v, tol=1e-2, precond=True, prec=prec)
    for w, ref in zip((v, v.float()), before):
        assert torch.equal(s.precond(w, "FFT"), ref)


# Many vectors, on either side of the split series kernel's line, as applies and inside a solve.
@pytest.mark.parametrize("L,Ltau,nrhs", [(14, 20, 200), (16, 20, 140), (16, 20, 200), (24, 20, 26), (24, 20, 52),
                                         (26, 20, 52), (28, 20, 52), (30, 20, 26), (30, 20, 52)])
@pytest.mark.parametrize("prec", ["f64", "f32_refined"])
def test_series_of_many_vectors(L, Ltau, nrhs, prec):
    lat = OL.Lattice(L, Ltau, 0.1, 1.0, 0.1, 1.0)
    rng = np.random.default_rng(5 * L + nrhs)
    x = rng.standard_normal((Ltau, lat.N))
    b = rng.standard_normal((nrhs, Ltau, lat.N))
    s = _solver(lat, nrhs)
    s.set_field(torch.from_numpy(x).cuda())
    pc = OP.Preconditioner(lat, x, 1.0, 1.0, C=OL.sparse_C(lat).tocsr())
    some = [0, 1, nrhs // 2, nrhs - 1]
    bg = torch.from_numpy(b).cuda()
    got = s.precond(bg if prec == "f64" else bg.float(), "FFT").double().cpu().numpy()
    for r in some:
        ref = pc.apply_FFt(b[r])
        assert np.max(np.abs(got[r] - ref)) < (1e-12 if prec == "f64" else 1e-5) * np.max(np.abs(ref)), r
    _close(_direction(s, bg, prec)[some], b[some], [pc] * len(some), prec)
