"""Host checks of the partial rows (no GPU needed).  Over every grid the library takes, in both types, the rows that
the passes of one field write fit what a plan allocates, at the tile of the rule and at every tile that a
measurement can record.  And the grids that the GPU tests take for their row counts have these counts."""
import os
import shutil
import subprocess

import pytest

from conftest import ROOT

PROGRAM = r"""
#include <cstdio>
#include "launch.hpp"
#include "internal.hpp"
using namespace gpe;
int main() {
    const int sizes[13] = {8, 16, 32, 40, 64, 80, 128, 160, 256, 320, 512, 640, 1024};
    long grids = 0, beyond = 0, bad = 0;
    for (int dim = 1; dim <= 3; ++dim)
        for (int i = 0; i < 13; ++i)
            for (int j = 0; j < (dim > 1 ? 13 : 1); ++j)
                for (int k = 0; k < (dim > 2 ? 13 : 1); ++k)
                    for (int cb = 8; cb <= 16; cb += 8) {
                        gpe_problem_t p = {};
                        p.dim = dim;
                        p.n[0] = sizes[i]; p.n[1] = sizes[j]; p.n[2] = sizes[k];
                        for (double& L : p.L) L = 1.0;
                        const Geo g = make_geo(p);
                        size_t rows = 0;  // the most that launches over one field can ask for
                        for (int a = 0; a < dim; ++a) {
                            int most = pass_blocks_per_field(g, a, cb, 1, false);
                            for (int C = fewest_tuned_lines(g, a, cb); C * (g.n[a] / 8) <= max_pass_threads(g, a); C *= 2) {
                                if (!valid_lines(g, a, cb, C)) continue;
                                record_tuned_lines(g, a, cb, 1, C);
                                most = std::max(most, pass_blocks_per_field(g, a, cb, 1, false));
                            }
                            rows += most;
                        }
                        ++grids;
                        beyond += 4 * rows > (1u << 18);
                        if (4 * rows > field_part_doubles(g, cb)) ++bad;
                    }
    std::printf("%ld %ld %ld\n", grids, beyond, bad);
    return 0;
}
"""

# rows of the x, y and z passes of an FP64 batch of B, and the most that its consumers absorb
COUNTS = r"""
#include <cstdio>
#include <cstdlib>
#include "rows.hpp"
#include "internal.hpp"
using namespace gpe;
int main(int argc, char** argv) {
    gpe_problem_t p = {};
    const int B = std::atoi(argv[1]);
    p.dim = argc - 2;
    for (int a = 0; a < p.dim; ++a) p.n[a] = std::atoi(argv[2 + a]);
    for (double& L : p.L) L = 1.0;
    const Geo g = make_geo(p);
    std::printf("%d", absorb_rows(B));
    for (int a = 0; a < p.dim; ++a) std::printf(" %d", pass_blocks_per_field(g, a, 16, B, true));
    return 0;
}
"""


def _host_program(tmp_path, text):
    lib = os.path.join(ROOT, "paper_1611_02045_amd")
    if shutil.which("hipcc") is None or not os.path.exists(os.path.join(lib, "libgpe.so")):
        pytest.skip("needs hipcc and the built library")
    src, exe = tmp_path / "rows.hip", tmp_path / "rows"
    src.write_text(text)
    subprocess.run(["hipcc", "-std=c++17", "-O1", "-w", "--offload-host-only", "-x", "hip", "-I", os.path.join(lib, "csrc"),
                    str(src), "-o", str(exe), "-L", lib, "-l:libgpe.so", f"-Wl,-rpath,{lib}"], check=True, timeout=300)
    return lambda *args: list(map(int, subprocess.run([str(exe), *map(str, args)], capture_output=True, text=True,
                                                      check=True, timeout=120).stdout.split()))


def test_grids_of_the_collapse_tests(tmp_path):
    from test_gpu_collapse import LINEAR_CASES, PCG_CASES
    rows = _host_program(tmp_path, COUNTS)
    for n, count in PCG_CASES:
        most, nx, *_ = rows(count, *n)
        assert nx > most, (n, count, nx)
    for n in LINEAR_CASES:
        most, nx, _, nz = rows(1, *n)
        assert nx > most and nz > most, (n, nx, nz)


def test_rows_of_every_grid_fit(tmp_path):
    grids, beyond, bad = _host_program(tmp_path, PROGRAM)()
    assert grids == 2 * (13 + 13 ** 2 + 13 ** 3)
    assert beyond > 0  # grids that a fixed 1 << 18 doubles would not hold
    assert bad == 0
