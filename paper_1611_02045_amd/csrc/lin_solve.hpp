// Queueing of the linear CG's passes (lin_passes.hpp), compiled once per precision.
#pragma once

#include "lin_passes.hpp"

namespace gpe {

constexpr int kLinDiagBlocks = 256;

template <typename T>
hipError_t lin_solve(LinCtx<T>& c, LinS& h, int check_every) {
    const Geo& g = *c.g;
    const bool f64 = sizeof(T) == 8;
    const bool spectral = c.kind == GPE_P_KINETIC || c.kind == GPE_P_COMBINED;
    const int scaled = c.kind == GPE_P_COMBINED ? 1 : 0;
    const int cb = (int)sizeof(C2<T>);
    const size_t region = lin_region_doubles(g);
    LinS *const S_dir = c.S, *const S_upd = c.S + 1;
    const void* twx = c.tw->get(0, f64);
    const Partials none{nullptr, 0, 0, 0};
    const int last = g.dim - 1;
    const int nq = pass_blocks_per_field(g, last, cb, 1, true);
    const int nz = spectral ? pass_blocks_per_field(g, 0, cb, 1, true) : kLinDiagBlocks;
    const Partials pq{c.rows, nq, nq, 0}, pz{c.rows + 2 * region, nz, nz, 0};
    const Partials qview = nq <= absorb_rows(1) ? pq : Partials{c.rows + region, (nq + kCollapseRows - 1) / kCollapseRows, 0, 0};
    hipError_t e;
    // x, r update (or only the first residual's z when the state says init), preconditioner
    auto update = [&]() -> hipError_t {
        if (!spectral) {
            hipLaunchKernelGGL(k_lin_upd_diag<T>, dim3(kLinDiagBlocks), dim3(256), 0, c.s, c.f, S_dir, S_upd, g.N,
                               c.kind == GPE_P_POTENTIAL ? 1 : 0, qview, pz.parts);
            return hipGetLastError();
        }
        if (g.dim == 1) {
            OpLinUpd<T, true> op{c.f, S_dir, S_upd, qview, scaled};
            return launch_pass<T, 0>(g, 1, twx, op, pz, c.s);
        }
        OpLinUpd<T, false> op{c.f, S_dir, S_upd, qview, scaled};
        hipError_t ee = launch_pass<T, 0>(g, 1, twx, op, none, c.s);
        if (ee == hipSuccess) ee = op_kinetic_middle(g, f64, *c.tw, c.f.w, &S_upd->alpha, c.s);
        if (ee != hipSuccess) return ee;
        OpLinPost<T> post{c.f, S_upd, scaled};
        return launch_pass<T, 0>(g, 1, twx, post, pz, c.s);
    };
    auto direction = [&](const Partials& zview) -> hipError_t {
        if (g.dim == 1) {
            OpLinApply<T, 0, true, true> op{c.f, S_upd, S_dir, zview};
            return launch_pass<T, 0>(g, 1, twx, op, pq, c.s);
        }
        OpLinApply<T, 0, true, false> ox{c.f, S_upd, S_dir, zview};
        hipError_t ee = launch_pass<T, 0>(g, 1, twx, ox, none, c.s);
        if (ee != hipSuccess) return ee;
        if (g.dim == 2) {
            OpLinApply<T, 1, false, true> oy{c.f, S_dir, nullptr, none};
            return launch_pass<T, 1>(g, 1, c.tw->get(1, f64), oy, pq, c.s);
        }
        if ((ee = op_apply_y(g, f64, *c.tw, c.f.p, c.f.w, c.omega, c.s)) != hipSuccess) return ee;
        OpLinApply<T, 2, false, true> oz{c.f, S_dir, nullptr, none};
        return launch_pass<T, 2>(g, 1, c.tw->get(2, f64), oz, pq, c.s);
    };
    auto collapse_z = [&] { return absorbable<Z_K, 0u>(pz, c.rows + 3 * region, 1, 1, g, c.s); };
    h.omega = c.omega;
    h.it = 0;
    h.done = h.status = h.first = 0;
    h.init = 1;
    LinS both[2] = {h, h};
    if ((e = hipMemcpyAsync(c.S, both, sizeof(both), hipMemcpyHostToDevice, c.s)) != hipSuccess) return e;
    if ((e = update()) != hipSuccess) return e;
    Partials zview = collapse_z();
    for (int64_t it = 0; it <= h.max_it; it += check_every) {
        for (int k = 0; k < check_every; ++k) {
            if ((e = direction(zview)) != hipSuccess) return e;
            (void)absorbable<Q_K, 0u>(pq, c.rows + region, 1, 1, g, c.s);
            if ((e = update()) != hipSuccess) return e;
            zview = collapse_z();
        }
        hipLaunchKernelGGL(k_lin_test, dim3(1), dim3(256), 0, c.s, S_upd, S_dir, zview);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if ((e = hipMemcpyAsync(&h, S_dir, sizeof(h), hipMemcpyDeviceToHost, c.s)) != hipSuccess) return e;
        if ((e = hipStreamSynchronize(c.s)) != hipSuccess) return e;
        if (h.done) break;
    }
    return hipSuccess;
}

}  // namespace gpe
