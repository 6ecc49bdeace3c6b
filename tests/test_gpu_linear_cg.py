"""The fused passes of the linear CG (implicit adjoint, backward Euler) in every dimension: the adjoint
state against the oracle's Hessian at the returned field, on grids whose partial rows are absorbed
directly and on grids that fold them first, in both precisions; the stopping rules."""
import numpy as np
import pytest

from gpe_inputs import Problem, gaussian, harmonic_potential, random_field
from oracle import gpe_oracle as O

pytestmark = pytest.mark.gpu


def _case(torch, prob, dtype):
    from paper_1611_02045_amd import gpe
    V = harmonic_potential(prob, (1.0, 1.4, 2.0))
    plan64 = gpe.Plan.from_problem(prob, "f64")
    phi = torch.from_numpy(gaussian(prob, (0.6, 0.8, 1.0))).to("cuda:0")
    Vd = torch.from_numpy(V).to("cuda:0")
    rep = plan64.pcg_solve(Vd, phi, tol=1e-10, max_iter=4000)
    assert rep["status"] == 0
    plan = plan64 if dtype == "f64" else gpe.Plan.from_problem(prob, dtype)
    return plan, V, phi, Vd.to(plan.real_dtype)


@pytest.mark.parametrize("dtype,tol,bound", [("f64", 1e-11, 1e-10), ("f32", 1e-3, 4e-3)])
@pytest.mark.parametrize("n,beta", [
    ((256,), 100.0),
    ((40,), 20.0),            # partial waves
    ((64, 32), 50.0),
    ((160, 80), 100.0),
    ((32, 16, 16), 50.0),
    ((64, 64, 64), 200.0),    # 512 rows of the z pass: folded before they are absorbed
    ((128, 128, 64), 400.0),  # and 512 of the x pass
], ids=str)
def test_adjoint_solves_the_projected_system(n, beta, dtype, tol, bound):
    torch = pytest.importorskip("torch")
    prob = Problem(len(n), n, (6.0,) * len(n), beta, 0.2 if len(n) > 1 else 0.0)
    plan, V, phi, Vd = _case(torch, prob, dtype)
    rhs = random_field(prob, 9, envelope=0.1)
    mu, rep = plan.adjoint_solve(phi.to(plan.complex_dtype), Vd, torch.from_numpy(rhs).to("cuda:0", plan.complex_dtype),
                                 tol=tol, max_iter=2000)
    assert rep["status"] == 0 and rep["res_inf"] <= tol
    p, m = phi.cpu().numpy(), mu.cpu().numpy().astype(np.complex128)
    lam = O.chemical_potential(prob, V, p)
    want = O.project_gauge(prob, p, rhs)
    got = O.project_gauge(prob, p, O.hessian_apply(prob, V, p, m) - lam * m)
    assert O.norm(prob, got - want) <= bound * O.norm(prob, want)
    # the solution lies in the tangent space
    assert O.norm(prob, m - O.project_gauge(prob, p, m)) <= bound * O.norm(prob, m)


def test_adjoint_stops():
    """A zero right-hand side returns zero at once; the iteration cap is kept; an excited state (an
    indefinite Hessian) is refused."""
    torch = pytest.importorskip("torch")
    from paper_1611_02045_amd import gpe
    prob = Problem(2, (64, 32), (6.0, 6.0), 50.0, 0.2)
    plan, V, phi, Vd = _case(torch, prob, "f64")
    mu, rep = plan.adjoint_solve(phi, Vd, torch.zeros_like(phi))
    assert rep["status"] == 0 and rep["iters"] == 0 and float(mu.abs().max()) == 0.0
    rhs = torch.from_numpy(random_field(prob, 9, envelope=0.1)).to("cuda:0")
    for cap in (1, 15, 16, 17):
        _, rep = plan.adjoint_solve(phi, Vd, rhs, tol=1e-14, max_iter=cap)
        assert rep["status_name"] == "not_converged" and rep["iters"] == cap
    flat = Problem(2, (64, 32), (6.0, 6.0), 0.0, 0.0)
    x = O.coordinates(flat)[0]
    excited = torch.from_numpy((x * gaussian(flat)) / O.norm(flat, x * gaussian(flat))).to("cuda:0")
    with pytest.raises(gpe.GpeError):
        gpe.Plan.from_problem(flat, "f64").adjoint_solve(
            excited, torch.from_numpy(harmonic_potential(flat)).to("cuda:0"), rhs, tol=1e-10, max_iter=500)
