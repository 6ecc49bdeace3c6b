"""Lines of 5 * 2^k points in 320-thread workgroups (whole waves): H apply and energy against the FP64
oracle at the edges of that tile's rule: the fewest and most workgroups that take it, lines that do not
divide into it, each axis."""
import numpy as np
import pytest

from gpe_inputs import Problem, harmonic_potential, random_field
from oracle import gpe_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,count", [
    ((640, 128), 1),       # 32 workgroups of four 640-point x lines: the fewest that take the tile
    ((640, 64), 1),        # 16: they do not
    ((128, 640), 1),       # the same along y
    ((640, 640), 2),       # 320 workgroups: more than one per CU (FP32 only)
    ((320, 320), 7),       # 280
    ((80, 160), 5),        # 160 lines of 80 points, 80 of 160
    ((40, 40), 40),        # 64 lines a workgroup, more than a field has
    ((40, 80, 40), 3),
], ids=str)
def test_wide_lines_match_oracle(n, count, dtype):
    torch = pytest.importorskip("torch")
    from paper_1611_02045_amd import gpe
    prob = Problem(len(n), n, (8.0, 6.0, 5.0)[: len(n)], 300.0, 0.7)
    V = harmonic_potential(prob, (1.0, 1.3, 0.8))
    base = random_field(prob, 11, envelope=0.01)
    plan = gpe.Plan.from_problem(prob, dtype)
    Vd = torch.from_numpy(V).to("cuda:0", plan.real_dtype)
    phi = torch.stack([torch.from_numpy(base * (1.0 + i / count)).to("cuda:0", plan.complex_dtype) for i in range(count)])
    tol = 2e-12 if dtype == "f64" else 2e-5
    out = plan.apply_H_batched(phi, Vd)
    for i in sorted({0, count // 2, count - 1}):
        ref = O.hamiltonian(prob, V, base * (1.0 + i / count))
        err = float(np.max(np.abs(out[i].cpu().numpy() - ref)) / np.max(np.abs(ref)))
        assert err < tol, (i, err)
    ref = O.energy_parts(prob, V, base)
    scale = abs(ref.kinetic) + abs(ref.potential) + abs(ref.interaction) + abs(ref.rotation)
    assert abs(plan.energy(phi[0].contiguous(), Vd) - ref.total) < tol * scale
