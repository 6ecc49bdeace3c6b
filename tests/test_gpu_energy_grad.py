"""The energy's backward in the passes of one H apply, against the FP64 oracle: every dimension, rows read
by partial and whole waves, both precisions, the scaled device form and its double backward."""
import numpy as np
import pytest

from gpe_inputs import Problem, harmonic_potential, random_field
from oracle import gpe_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,tol", [("f64", 2e-12), ("f32", 2e-5)])
@pytest.mark.parametrize("n", [(8,), (40,), (256,), (1024,), (8, 8), (64, 16), (80, 40), (640, 64), (512, 256),
                               (8, 16, 8), (64, 32, 64), (40, 16, 80)], ids=str)
def test_energy_gradient_matches_oracle(n, dtype, tol):
    torch = pytest.importorskip("torch")
    from paper_1611_02045_amd import gpe
    prob = Problem(len(n), n, (5.0, 4.0, 3.0)[: len(n)], 120.0, 0.6 if len(n) > 1 else 0.0)
    V = harmonic_potential(prob, (1.0, 1.3, 0.8))
    phi = random_field(prob, 3, envelope=0.05)
    plan = gpe.Plan.from_problem(prob, dtype)
    P, W = torch.from_numpy(phi).to("cuda:0", plan.complex_dtype), torch.from_numpy(V).to("cuda:0", plan.real_dtype)
    h = O.cell(prob)
    parts = O.energy_parts(prob, V, phi)
    rot = -O.inner(prob, phi, O.angular_momentum(prob, phi)).real if prob.dim > 1 else 0.0
    want = (2.0 * h * O.hamiltonian(prob, V, phi), h * np.abs(phi) ** 2, parts.interaction / prob.beta, rot)
    scale = abs(parts.kinetic) + abs(parts.potential) + abs(parts.interaction) + abs(parts.rotation)

    def check(got, f):
        gphi, gV, db, do = got
        assert np.max(np.abs(gphi.cpu().numpy() - f * want[0])) < tol * abs(f) * np.max(np.abs(want[0]))
        assert np.max(np.abs(gV.cpu().numpy() - f * want[1])) < tol * abs(f) * np.max(np.abs(want[1]))
        assert abs(float(db) - f * want[2]) < tol * abs(f) * want[2]
        # <phi, L_z phi> cancels: its error is that of its terms, bounded by the kinetic energy times the box
        assert abs(float(do) - f * want[3]) < tol * abs(f) * 10.0 * scale

    check(plan.energy_grad(P, W), 1.0)
    f = -1.75  # exact in both precisions
    check(plan.energy_grad_scaled(P, W, torch.tensor(f, dtype=plan.real_dtype, device="cuda:0")), f)
    g2 = plan.energy_grad(P, W, want_V=False)
    assert g2[1] is None
    E = plan.energy_value(P, W)
    assert E.is_cuda and E.dtype == plan.real_dtype and abs(float(E) - parts.total) < tol * scale


def test_energy_autograd_forms():
    """backward(), a factor, and create_graph (the products with the incoming gradient stay differentiable)."""
    torch = pytest.importorskip("torch")
    from paper_1611_02045_amd.autograd import Grid, energy
    prob = Problem(2, (32, 16), (4.0, 4.0), 30.0, 0.4)
    grid = Grid(2, prob.n, prob.L)
    phi = torch.from_numpy(random_field(prob, 3, envelope=0.1)).to("cuda:0").requires_grad_(True)
    V = torch.from_numpy(harmonic_potential(prob)).to("cuda:0").requires_grad_(True)
    b, o = (torch.tensor(x, dtype=torch.float64, device="cuda:0", requires_grad=True) for x in (30.0, 0.4))
    leaves = (phi, V, b, o)
    one = torch.autograd.grad(energy(phi, V, b, o, grid), leaves)
    k = torch.tensor(3.0, dtype=torch.float64, device="cuda:0", requires_grad=True)
    three = torch.autograd.grad(k * energy(phi, V, b, o, grid), leaves, create_graph=True)
    for x, y in zip(one, three):
        assert torch.allclose(3.0 * x, y, rtol=1e-13, atol=0.0)
    dk, = torch.autograd.grad(three[3], k)
    assert torch.allclose(dk, one[3], rtol=1e-13)
    with pytest.raises(RuntimeError):  # not finite
        energy((phi * float("nan")).detach(), V, b, o, grid)


def test_energy_backward_accepts_any_incoming_gradient():
    """A batch of incoming gradients (no storage of its own), a lazily negated one and one on another stream
    give the products of the plain one, exactly (powers of two)."""
    torch = pytest.importorskip("torch")
    from paper_1611_02045_amd import autograd as A
    prob = Problem(2, (64, 32), (5.0, 4.0), 120.0, 0.6)
    V = torch.from_numpy(harmonic_potential(prob, (1.0, 1.3))).cuda().requires_grad_()
    phi = torch.from_numpy(random_field(prob, 3, envelope=0.05)).cuda().requires_grad_()
    grid = A.Grid(prob.dim, prob.n, prob.L)
    b, o = (torch.tensor(x, dtype=torch.float64, device="cuda:0", requires_grad=True) for x in (prob.beta, prob.omega))
    E = A.energy(phi, V, b, o, grid)
    one = torch.ones((), dtype=torch.float64, device="cuda:0")
    args = (phi, V, b, o)
    want = torch.autograd.grad(E, args, one, retain_graph=True)
    rows = torch.autograd.grad(E, args, torch.stack([one, -2.0 * one]), retain_graph=True, is_grads_batched=True)
    for w, r in zip(want, rows):
        assert torch.equal(r[0], w) and torch.equal(r[1], -2.0 * w)
    neg = torch.complex(one, 2.0 * one).conj().imag
    assert neg.is_neg()
    for w, r in zip(want, torch.autograd.grad(E, args, neg, retain_graph=True)):
        assert torch.equal(r, -2.0 * w)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        E2 = A.energy(phi, V, b, o, grid)
        got = torch.autograd.grad(E2, args, 4.0 * one)
    torch.cuda.current_stream().wait_stream(side)
    for w, r in zip(want, got):
        assert torch.equal(r, 4.0 * w)
