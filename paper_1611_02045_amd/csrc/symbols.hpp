// Symbols shared by the operators and the linear solvers.
#pragma once

#include "passes.hpp"

namespace gpe {

// Rotation coefficient of the directional symbol along AX for the line (i1, i2):
// R = -omega L_z = i omega (x d_y - y d_x) acts as +omega y xi along x and -omega x mu along y.
template <int AX>
__device__ __forceinline__ double rot_coef(const Geo& g, const LineCtx& lc, double omega) {
    if (g.dim < 2 || omega == 0.0) return 0.0;
    if (AX == 0) return omega * coord_of(lc.i1, g.L[1], g.h[1]);
    if (AX == 1) return -omega * coord_of(lc.i1, g.L[0], g.h[0]);
    return 0.0;
}

// Pointwise factor of P_V: (alpha + V + beta rho)^{-1/2} (kind 1) or its square.
template <typename T>
__device__ __forceinline__ T pv_scale(int kind, double alpha, T V, T rho, double beta) {
    const double d = alpha + (double)V + beta * (double)rho;
    return kind == 1 ? (T)(1.0 / sqrt(d)) : (T)(1.0 / d);
}

}  // namespace gpe
