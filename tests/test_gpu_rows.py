"""Partial rows between the passes of 2-D and 3-D solves: trajectories against the FP64 oracle at row counts
on both sides of the line between rows absorbed as they are and rows collapsed first, for a lone instance and
in a batch, with rows shared by two passes (phase A) and partly filled ones (the direction passes)."""
import numpy as np
import pytest

from gpe_inputs import Problem, gaussian, harmonic_potential
from oracle import gpe_oracle as O

pytestmark = pytest.mark.gpu


def _problem(n, beta):
    prob = Problem(len(n), n, (8.0, 6.0, 7.0)[: len(n)], beta, 0.4)
    return prob, harmonic_potential(prob, (1.0, 1.2, 0.9)), gaussian(prob, (1.4, 1.1, 0.8))


@pytest.mark.parametrize("n,count", [
    ((16, 8), 1),         # one workgroup per pass
    ((640, 128), 1),      # unequal row counts of the passes
    ((256, 512), 1),      # 256 direction rows or fewer
    ((512, 1024), 1),     # 512: the most that a lone instance absorbs
    ((1024, 1024), 1),    # collapsed
    ((64, 64, 64), 1),    # 384 in three passes
    ((64, 64, 64), 2),    # the same in a batch: collapsed
    ((16, 128, 8), 3),
], ids=str)
def test_trajectory_matches_oracle(n, count):
    torch = pytest.importorskip("torch")
    from paper_1611_02045_amd import gpe
    its = 4
    probs, Vs, phis = zip(*[_problem(n, 30.0 + 20.0 * i) for i in range(count)])
    Vd = [torch.from_numpy(V).to("cuda:0") for V in Vs]
    pd = [torch.from_numpy(p).to("cuda:0") for p in phis]
    _, reps = gpe.pcg_solve_batched(list(probs), Vd, pd, "f64", tol=1e-30, max_iter=its)
    for i in range(count):
        ref = O.pcg(probs[i], Vs[i], phis[i], tol_res=1e-30, max_iter=its)
        assert reps[i]["iters"] == its
        # FP64 rounding of four iterations from a smooth start
        assert abs(reps[i]["E"] - ref.E) < 1e-11 * abs(ref.E)
        got = pd[i].cpu().numpy()
        assert np.max(np.abs(got - ref.phi)) < 1e-9 * np.max(np.abs(ref.phi))
