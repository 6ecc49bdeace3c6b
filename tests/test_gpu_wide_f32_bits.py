"""320-thread passes (lines of 5 * 2^k points) against the 256-thread ones that they stand for: an FP32 solve
returns the same bits, on either side of the line between few and many workgroups.

Checksums of the fields after six iterations, one for each preconditioner named below, taken from the build of
commit c631a72, whose passes had 256 threads at most.  The inputs are formed by correctly rounded operations."""
import zlib

import numpy as np
import pytest
import torch

from gpe_inputs import Problem

pytestmark = pytest.mark.gpu

PRECONDS = ("none", "combined")
# (grid, instances): crc32 for each preconditioner
GOLDEN = {
    ((320, 320), 1): (3636817847, 897610318),
    ((320, 320), 4): (2546821411, 705757633),
    ((320, 320), 8): (4065729396, 932803356),
    ((512, 160), 1): (3543796802, 4087235474),
    ((160, 160), 9): (2630751278, 1369461616),
    ((256, 160), 16): (1273767467, 2915079165),
    ((1024, 320), 1): (2298033982, 340156804),
    ((640, 640), 1): (2182253210, 2383020931),
    ((64, 64, 80), 1): (2886708131, 3685534378),
    ((128, 32, 40), 1): (219503151, 1213324671),
    ((40, 32, 80), 5): (3448885174, 2661190930),
}


def solve_crc(n, count, precond):
    from paper_1611_02045_amd import gpe
    dim = len(n)
    ax = np.meshgrid(*[np.arange(m) for m in reversed(n)], indexing="ij")[::-1]  # x, y, z
    env = sum(np.abs(a - m // 2) * 12 // m for a, m in zip(ax, n))
    V = sum((1 + k) * ((a - m // 2) / (m / 16.0)) ** 2 for k, (a, m) in enumerate(zip(ax, n)))
    phis = []
    for b in range(count):
        re = 2.0 ** -env * (1 + ((7 * ax[0] + 5 * ax[1] + 3 * b) % 31 - 15) / 64.0)
        im = 2.0 ** -env * (((11 * ax[0] + 9 * ax[-1] + b) % 29 - 14) / 64.0)
        phis.append(torch.from_numpy(re + 1j * im).to("cuda:0", torch.complex64))
    Vs = [torch.from_numpy(V).to("cuda:0", torch.float32)] * count
    gpe.pcg_solve_batched([Problem(dim, n, (8.0,) * dim, 64.0, 0.25)] * count, Vs, phis, "f32", max_iter=6, tol=0.0,
                          precond=precond)
    return zlib.crc32(torch.stack(phis).cpu().numpy().tobytes())


@pytest.mark.parametrize("n,count", list(GOLDEN))
def test_wide_solve_returns_the_pinned_bits(n, count):
    assert tuple(solve_crc(n, count, p) for p in PRECONDS) == GOLDEN[n, count]
