"""Solves that end within their first chunks of iterations: wherever they end, and whatever the chunk, they return
the bits of the solve that is polled after every iteration, and one from a converged field costs little more than
one of no iterations."""
import statistics
import time

import pytest

from gpe_inputs import Problem, gaussian, harmonic_potential

pytestmark = pytest.mark.gpu


def _near(torch, n, dtype="f64"):
    """A plan, its potential and a start near the ground state."""
    from paper_1611_02045_amd import gpe
    prob = Problem(len(n), n, (6.0,) * len(n), 60.0, 0.2)
    plan = gpe.Plan.from_problem(prob, dtype)
    V = torch.from_numpy(harmonic_potential(prob, (1.0, 1.3, 1.6))).to("cuda:0", plan.real_dtype)
    phi0 = torch.from_numpy(gaussian(prob)).to("cuda:0", plan.complex_dtype)
    phi = phi0.clone()
    plan.pcg_solve(V, phi, tol=1e-9 if dtype == "f64" else 1e-4, max_iter=2000)
    return prob, plan, V, phi, phi + 1e-3 * phi0


@pytest.mark.parametrize("n", [(64, 32), (16, 16, 16)], ids=str)
@pytest.mark.parametrize("graph", [0, 1])
def test_end_is_independent_of_the_chunk(n, graph):
    torch = pytest.importorskip("torch")
    _, plan, V, _, start = _near(torch, n)
    ends = set()
    for tol in (1e-1, 1e-3, 1e-4, 2e-5, 5e-6, 1e-6, 2e-7, 1e-8, 1e-9, 1e-10, 1e-11):
        for max_iter in (400, 9):
            want = None
            for check_every in (1, 2, 3, 4, 6, 16, 17, 64):
                phi = start.clone()
                rep = plan.pcg_solve(V, phi, tol=tol, max_iter=max_iter, check_every=check_every, use_graph=graph,
                                     refresh_every=0)
                got = (rep["iters"], rep["status"], rep["E"], rep["res_inf"])
                want = want or (got, phi)
                assert got == want[0] and torch.equal(phi, want[1]), (tol, max_iter, check_every)
            ends.add(want[0][0])
    assert len(ends) >= 6 and min(ends) == 0 and max(ends) > 16  # in and behind a first chunk of 16


def test_batch_ends_are_independent_of_the_chunk():
    """Instances that end in the first chunk beside one that does not."""
    torch = pytest.importorskip("torch")
    from paper_1611_02045_amd import gpe
    prob, _, V, done, near = _near(torch, (64, 32))
    far = torch.from_numpy(gaussian(prob, (2.0, 0.7))).to("cuda:0")
    want = None
    for check_every in (1, 2, 8, 16, 50):
        phis = [p.clone() for p in (done, far, near, done)]
        _, reps = gpe.pcg_solve_batched([prob] * 4, [V] * 4, phis, "f64", tol=2e-9, max_iter=400, check_every=check_every,
                                        refresh_every=0)
        got = [(r["iters"], r["status"], r["E"]) for r in reps]
        want = want or (got, phis)
        assert got == want[0]
        assert all(torch.equal(a, b) for a, b in zip(phis, want[1]))


def test_converged_start_costs_no_second_chunk():
    """Both calls queue one chunk; the converged one may not add a graph and a second chunk (2.1 times the other then,
    1.1 without)."""
    torch = pytest.importorskip("torch")
    _, plan, V, phi, _ = _near(torch, (64, 64, 64))

    def cost(**opts):
        took = []
        for _ in range(25):
            p = phi.clone()
            torch.cuda.synchronize()
            t = time.perf_counter()
            plan.pcg_solve(V, p, **opts)
            took.append(time.perf_counter() - t)
        return statistics.median(took[5:])

    assert cost(tol=2e-9, max_iter=400) < 1.5 * cost(tol=0.0, max_iter=0)
