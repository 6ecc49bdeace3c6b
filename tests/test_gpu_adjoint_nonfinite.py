"""Non-finite input of the implicit adjoint is reported as such: not as a converged solve with mu = 0 (a NaN
right-hand side), nor as an indefinite Hessian (a NaN potential)."""
import numpy as np
import pytest

from gpe_inputs import Problem, gaussian, harmonic_potential, random_field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [(64,), (40,), (64, 32), (16, 16, 8)], ids=str)
@pytest.mark.parametrize("where", ["rhs nan", "rhs inf", "V nan"])
def test_status(n, dtype, where):
    torch = pytest.importorskip("torch")
    from paper_1611_02045_amd import gpe
    prob = Problem(len(n), n, (5.0,) * len(n), 20.0, 0.1 if len(n) > 1 else 0.0)
    plan = gpe.Plan.from_problem(prob, dtype)
    phi = torch.from_numpy(gaussian(prob)).to("cuda:0", plan.complex_dtype)
    V, rhs = harmonic_potential(prob), random_field(prob, 3, envelope=0.1)
    if where == "V nan":
        V.flat[5] = np.nan
    else:
        rhs.flat[7] = np.nan if where == "rhs nan" else np.inf
    with pytest.raises(gpe.GpeError) as err:
        plan.adjoint_solve(phi, torch.from_numpy(V).to("cuda:0", plan.real_dtype),
                           torch.from_numpy(rhs).to("cuda:0", plan.complex_dtype), max_iter=40)
    assert err.value.status == -4


def test_nan_gradient_of_a_ground_state_is_refused():
    torch = pytest.importorskip("torch")
    from paper_1611_02045_amd import autograd, gpe
    prob = Problem(2, (32, 32), (5.0, 5.0), 20.0, 0.0)
    V = torch.from_numpy(harmonic_potential(prob)).to("cuda:0").requires_grad_()
    phi = autograd.ground_state(V, 20.0, 0.0, torch.from_numpy(gaussian(prob)).to("cuda:0"),
                                autograd.Grid(2, prob.n, prob.L))
    with pytest.raises(gpe.GpeError):
        (phi.abs().square().sum() * float("nan")).backward()
