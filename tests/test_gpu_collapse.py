"""Partial rows beyond what a consumer absorbs, folded by the collapse first: the phase-A rows of the PCG (maxima
and sums, filled by two passes), for a lone instance and in a batch, and both sums of the linear CG.  That the
grids here have that many rows is asserted from the tile rule in test_part_rows.py."""
import numpy as np
import pytest

from gpe_inputs import Problem, gaussian, harmonic_potential, random_field
from oracle import gpe_oracle as O

pytestmark = pytest.mark.gpu

# (n, count): FP64 solves with more phase-A rows (x pass) per instance than its consumer absorbs
PCG_CASES = [((128, 128, 128), 1), ((1024, 1024), 2)]
# n: FP64 adjoints with more rows of the first (x) and last (z) pass than theirs
LINEAR_CASES = [(128, 128, 128)]


@pytest.mark.parametrize("n,count", PCG_CASES, ids=str)
def test_pcg_trajectory_matches_oracle(n, count):
    torch = pytest.importorskip("torch")
    from paper_1611_02045_amd import gpe
    its = 3
    probs = [Problem(len(n), n, (8.0, 6.0, 7.0)[: len(n)], 30.0 + 20.0 * i, 0.4) for i in range(count)]
    Vs = [harmonic_potential(p, (1.0, 1.2, 0.9)) for p in probs]
    phis = [gaussian(p, (1.4, 1.1, 0.8)) for p in probs]
    pd = [torch.from_numpy(p).to("cuda:0") for p in phis]
    _, reps = gpe.pcg_solve_batched(probs, [torch.from_numpy(V).to("cuda:0") for V in Vs], pd, "f64", tol=1e-30,
                                    max_iter=its)
    for i in range(count):
        ref = O.pcg(probs[i], Vs[i], phis[i], tol_res=1e-30, max_iter=its)
        assert reps[i]["iters"] == its
        # FP64 rounding of three iterations from a smooth start
        assert abs(reps[i]["E"] - ref.E) < 1e-11 * abs(ref.E)
        assert np.max(np.abs(pd[i].cpu().numpy() - ref.phi)) < 1e-9 * np.max(np.abs(ref.phi))


@pytest.mark.parametrize("n", LINEAR_CASES, ids=str)
def test_adjoint_solves_the_projected_system(n):
    torch = pytest.importorskip("torch")
    from paper_1611_02045_amd import gpe
    prob = Problem(3, n, (6.0,) * 3, 400.0, 0.2)
    V = harmonic_potential(prob, (1.0, 1.4, 2.0))
    plan = gpe.Plan.from_problem(prob, "f64")
    phi, Vd = (torch.from_numpy(a).to("cuda:0") for a in (gaussian(prob, (0.6, 0.8, 1.0)), V))
    assert plan.pcg_solve(Vd, phi, tol=1e-10, max_iter=4000)["status"] == 0
    rhs = random_field(prob, 9, envelope=0.1)
    tol = 1e-11
    mu, rep = plan.adjoint_solve(phi, Vd, torch.from_numpy(rhs).to("cuda:0"), tol=tol, max_iter=2000)
    assert rep["status"] == 0 and rep["res_inf"] <= tol
    p, m = phi.cpu().numpy(), mu.cpu().numpy()
    lam = O.chemical_potential(prob, V, p)
    want = O.project_gauge(prob, p, rhs)
    got = O.project_gauge(prob, p, O.hessian_apply(prob, V, p, m) - lam * m)
    # ten times the tolerance of the tracked residual
    assert O.norm(prob, got - want) <= 10 * tol * O.norm(prob, want)
