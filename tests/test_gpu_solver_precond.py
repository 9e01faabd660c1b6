"""z = F F^T r as the solvers apply it: after one iteration from a zero guess the iterate is alpha z,
z = F F^T b, so it shows the preconditioner inside a solve itself."""

import numpy as np
import pytest
import torch

from oracle import lattice as OL
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
