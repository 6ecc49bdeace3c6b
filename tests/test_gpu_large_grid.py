"""Energy and its derivatives on grids whose passes write more partial rows than 1 << 18 doubles hold, against the
closed form for a plane wave: E = |k|^2/2 + V0 + beta/(2 vol), dE/dbeta = 1/(2 vol), dE/dV = h^d/vol."""
import math

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,dtype,bound", [((320, 320, 320), "f64", 1e-12), ((512, 512, 512), "f32", 1e-5)])
def test_plane_wave(n, dtype, bound):
    torch = pytest.importorskip("torch")
    from paper_1611_02045_amd import gpe
    L, beta, V0, modes = 4.0, 100.0, 1.5, (3, -2, 5)
    plan = gpe.Plan(3, n, (L,) * 3, beta, 0.0, dtype)
    k = [m * math.pi / L for m in modes]
    axes = [torch.exp(1j * q * (-L + torch.arange(m, device="cuda:0", dtype=torch.float64) * (2 * L / m)))
            for q, m in zip(k, n)]
    vol = (2 * L) ** 3
    phi = (axes[2][:, None, None] * axes[1][None, :, None] * axes[0][None, None, :] / math.sqrt(vol)).to(plan.complex_dtype)
    V = torch.full(plan.shape, V0, device="cuda:0", dtype=plan.real_dtype)
    kin, rho = 0.5 * sum(q * q for q in k), 1.0 / vol
    E, parts = plan.energy(phi, V, parts=True)
    assert abs(E - (kin + V0 + 0.5 * beta * rho)) <= bound * E
    assert abs(parts["kinetic"] - kin) <= bound * kin
    _, gV, db, _ = plan.energy_grad(phi, V)
    cell = vol / math.prod(n)
    assert abs(db - 0.5 * rho) <= bound * rho
    assert float((gV - cell * rho).abs().max()) <= bound * cell * rho
