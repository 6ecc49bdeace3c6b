// Standalone operators of the solver as chains of directional passes:
//   * H_phi phi and L f = (T + V - omega L_z) f            (Sections 2-3)
//   * the energy E(phi) and its parts                     (Section 2)
//   * the preconditioners P_Delta, P_V, P_C, P_C1, P_C2   (Section 5.5)
#include <algorithm>
#include <cmath>
#include <vector>

#include "internal.hpp"
#include "launch.hpp"
#include "symbols.hpp"

namespace gpe {

// ---------------------------------------------------------------------------------------------
// Directional part of L (and H): out = acc + F_a^{-1}[sigma_a F_a f], sigma_a = xi^2/2 + rot*xi,
// and on the pass with `pointwise` set also + (V + beta|f|^2) f (beta term only for the
// nonlinear H).  The pointwise part goes with the x pass, where V is read contiguously; the
// strided passes then read only f and the running sum.
// ---------------------------------------------------------------------------------------------
// Every input is read ahead of the first store: `acc` and `out` may be one buffer, so a read after a
// store is a memory round trip of its own (the y pass took eight in a row: 2.7 of its 5.5 us on a
// 256^2 FP64 field).
template <typename T, int AX>
struct OpApply {
    static constexpr bool FWD = true, INV = true, SCALARS = false, PREFETCH = true, WIDE = false, FIXED = true;
    static constexpr int K = 0;
    static constexpr unsigned MAXMASK = 0;
    const C2<T>* f;
    const C2<T>* acc;  // strided passes: the running sum (nullptr: none)
    C2<T>* out;
    const T* V;        // used by the pass with `pointwise` set
    double beta, omega;
    int pointwise, nonlinear;
    double kin = 1.0;  // weight of the kinetic symbol (0: rotation part only)
    // only the x pass carries the pointwise part: the strided passes keep no copy of f
    static constexpr bool PW = AX == 0;
    struct State {
        C2<T> f0[8];
        C2<T> a[PW ? 1 : 8];
        T V[PW ? 8 : 1];
    };
    __device__ void prefetch(const Geo&, const LineCtx& lc, State& st) const {
#pragma unroll
        for (int s = 0; s < 8; ++s) st.f0[s] = f[lc.at(s)];
    }
    // the x pass starts the sum, the strided passes continue it
    __device__ void prefetch_tail(const Geo&, const LineCtx& lc, State& st) const {
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int64_t i = lc.at(s);
            if constexpr (PW) {
                st.V[s] = pointwise && V ? V[i - lc.off_b] : (T)0;
            } else {
                st.a[s] = acc ? acc[i] : mk((T)0, (T)0);
            }
        }
    }
    __device__ void load(const Geo&, const LineCtx&, State& st, C2<T> (&v)[8], double (&)[1]) const {
#pragma unroll
        for (int s = 0; s < 8; ++s) v[s] = st.f0[s];
    }
    template <int LG>
    __device__ void spectral(const Geo& g, const LineCtx& lc, State&, C2<T> (&v)[8], double (&)[1], C2<T>*,
                             const C2<T>*) const {
        const double rot = rot_coef<AX>(g, lc, omega);
        const double inv = 1.0 / lc.M;  // 1/M (exact for M = 2^k)
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const double xi = freq_of(lc.k(s), lc.M, g.dk[AX]);
            v[s] = scl(v[s], (T)((0.5 * kin * xi * xi + rot * xi) * inv));
        }
    }
    __device__ void store(const Geo&, const LineCtx& lc, State& st, C2<T> (&v)[8], double (&)[1]) const {
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            C2<T> o = v[s];
            if constexpr (PW) {
                if (pointwise && V) {
                    T w = st.V[s];
                    if (nonlinear) w += (T)beta * abs2(st.f0[s]);
                    o = add(o, scl(st.f0[s], w));
                }
            } else {
                o = add(o, st.a[s]);
            }
            out[lc.at(s)] = o;
        }
    }
};

// Fields of one part of a batched apply.  The passes share phi and the running sum between launches;
// when phi, the sum and the output of a whole batch exceed the 256 MB last-level cache, every pass
// after the first takes them from HBM.  A batch is therefore applied in equal parts of at most
// kApplyPartBytes of those three, which reuse one region for the sum.  Measured (us, whole batch;
// parts of at most 100, 160, 230 MB): 64 x 512^2 FP32 165; 155, 147, 142.  32 x 512^2 FP64 142; 162,
// 138, 130.  32 x 640^2 FP64 302; 376, 302, 286.  256 x 256^2 FP32 145; 142, 130, 125.  Three-pass
// (3-D) batches gain little (4 x 128^3 FP64 196; 212, 211, 187).
constexpr int64_t kApplyPartBytes = int64_t(224) << 20;
int64_t apply_part_most(const Geo& g, int complex_bytes) {
    return std::max<int64_t>(1, kApplyPartBytes / (3 * (int64_t)complex_bytes * g.N));
}
static int apply_part(const Geo& g, int complex_bytes, int B) {
    const int64_t most = apply_part_most(g, complex_bytes);
    const int64_t parts = (B + most - 1) / most;
    return (int)((B + parts - 1) / parts);
}

// One part: B of the batch's fields.  Tiles follow the whole batch (Cx, Cy, Cz lines per workgroup).
template <typename T>
static hipError_t apply_part_t(const Geo& g, int B, const Twiddles& tw, const C2<T>* F, const T* V, C2<T>* out,
                               C2<T>* tmp, double beta, double omega, bool nl, bool plane, const int C[3],
                               hipStream_t s) {
    const bool f64 = sizeof(T) == 8;
    Partials none{nullptr, 0, 0, 0};
    hipError_t e;
    if (plane) {
        // whole xy-planes in LDS, the xy-part into tmp, then the z pass
        if ((e = op_apply_plane(g, f64, B, tw, F, V, tmp, beta, omega, nl, s)) != hipSuccess) return e;
        OpApply<T, 2> oz{F, tmp, out, nullptr, beta, omega, 0, nl};
        return launch_pass<T, 2>(g, B, tw.get(2, f64), oz, none, s, nullptr, C[2]);
    }
    // x-pass (with the pointwise part) into tmp, then the y (and z) passes accumulate.
    OpApply<T, 0> ox{F, nullptr, tmp, V, beta, omega, 1, nl};
    if ((e = launch_pass<T, 0>(g, B, tw.get(0, f64), ox, none, s, nullptr, C[0])) != hipSuccess) return e;
    OpApply<T, 1> oy{F, tmp, g.dim == 2 ? out : tmp, nullptr, beta, omega, 0, nl};
    if ((e = launch_pass<T, 1>(g, B, tw.get(1, f64), oy, none, s, nullptr, C[1])) != hipSuccess || g.dim == 2) return e;
    OpApply<T, 2> oz{F, tmp, out, nullptr, beta, omega, 0, nl};
    return launch_pass<T, 2>(g, B, tw.get(2, f64), oz, none, s, nullptr, C[2]);
}

template <typename T>
static hipError_t apply_t(const Geo& g, int B, const Twiddles& tw, const void* f, const void* V, void* out,
                          void* tmp, double beta, double omega, bool nl, hipStream_t s) {
    const bool f64 = sizeof(T) == 8;
    const C2<T>* F = (const C2<T>*)f;
    C2<T>* O = (C2<T>*)out;
    if (g.dim == 1) {
        OpApply<T, 0> op{F, nullptr, O, (const T*)V, beta, omega, 1, nl};
        return launch_pass<T, 0>(g, B, tw.get(0, f64), op, Partials{nullptr, 0, 0, 0}, s);
    }
    const bool plane = plane_preferred(g, f64, B);
    if (plane && g.dim == 2) return op_apply_plane(g, f64, B, tw, f, V, out, beta, omega, nl, s);  // all of H f
    int C[3] = {0, 0, 0};
    for (int a = 0; a < g.dim; ++a) C[a] = pass_lines_per_block(g, a, (int)sizeof(C2<T>), B, false);
    const int part = apply_part(g, (int)sizeof(C2<T>), B);
    for (int b = 0; b < B; b += part) {
        const int64_t off = (int64_t)b * g.N;
        const hipError_t e = apply_part_t<T>(g, std::min(part, B - b), tw, F + off, (const T*)V, O + off, (C2<T>*)tmp,
                                             beta, omega, nl, plane, C, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// out = R f with R = -L_z (rotation symbol with omega = 1, no kinetic, no potential); dim >= 2.
template <typename T>
static hipError_t rotation_t(const Geo& g, const Twiddles& tw, const void* f, void* out, void* tmp, hipStream_t s) {
    const bool f64 = sizeof(T) == 8;
    const C2<T>* F = (const C2<T>*)f;
    Partials none{nullptr, 0, 0, 0};
    hipError_t e;
    OpApply<T, 0> ox{F, nullptr, (C2<T>*)tmp, nullptr, 0.0, 1.0, 0, 0, 0.0};
    if ((e = launch_pass<T, 0>(g, 1, tw.get(0, f64), ox, none, s)) != hipSuccess) return e;
    // the y pass completes R (no z part in 3-D: L_z acts in the xy-planes)
    OpApply<T, 1> oy{F, (const C2<T>*)tmp, (C2<T>*)out, nullptr, 0.0, 1.0, 1, 0, 0.0};
    return launch_pass<T, 1>(g, 1, tw.get(1, f64), oy, none, s);
}

hipError_t op_rotation(const Geo& g, bool f64, const Twiddles& tw, const void* f, void* out, void* tmp, hipStream_t s) {
    return f64 ? rotation_t<double>(g, tw, f, out, tmp, s) : rotation_t<float>(g, tw, f, out, tmp, s);
}

hipError_t op_apply(const Geo& g, bool f64, int B, const Twiddles& tw, const void* f, const void* V, void* out,
                    void* tmp, double beta, double omega, bool nonlinear, hipStream_t s) {
    return f64 ? apply_t<double>(g, B, tw, f, V, out, tmp, beta, omega, nonlinear, s)
               : apply_t<float>(g, B, tw, f, V, out, tmp, beta, omega, nonlinear, s);
}

// ---------------------------------------------------------------------------------------------
// Interpolation onto the grid with twice the points per axis and the same box (the nested grids
// of Section 6), one axis per pass, by the trigonometric interpolant of the discretisation with
// the Nyquist coefficient split evenly between the frequencies -M/2 and +M/2.  At the coarse
// points the interpolant is the input itself; at the midpoints x_j + h/2 it is the input shifted
// by half a cell, F^{-1}[e^{i pi p / M} F f] over -M/2 < p < M/2, the split Nyquist pair adding
// cos(pi/2) = 0 there.  The pass writes both: out[2j] = f[j], out[2j + 1] = the shifted value.
// The pass geometry is the source's (axes before AX already doubled); out has twice its points.
// ---------------------------------------------------------------------------------------------
template <typename T, int AX>
struct OpProlong {
    static constexpr bool FWD = true, INV = true, SCALARS = false, PREFETCH = false, WIDE = false;
    static constexpr int K = 0;
    static constexpr unsigned MAXMASK = 0;
    const C2<T>* f;
    C2<T>* out;
    double hr, hi;  // e^{i pi / M} (host FP64) for the pass's line length M
    struct State {};
    __device__ void load(const Geo&, const LineCtx& lc, State&, C2<T> (&v)[8], double (&)[1]) const {
#pragma unroll
        for (int s = 0; s < 8; ++s) v[s] = f[lc.at(s)];
    }
    // e^{i pi p / M} from the transform's table tw[e] = e^{-2 pi i e / M}: conj(tw[floor(p/2) mod M]),
    // times e^{i pi / M} for odd p.
    template <int LG>
    __device__ void spectral(const Geo&, const LineCtx& lc, State&, C2<T> (&v)[8], double (&)[1], C2<T>*,
                             const C2<T>* tw) const {
        const T inv = (T)(1.0 / lc.M);  // 1/M (exact for M = 2^k)
        const C2<T> half{(T)hr, (T)hi};
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int j = lc.k(s);
            const int p = j < (lc.M >> 1) ? j : j - lc.M;
            if (2 * p == -lc.M) {
                v[s] = C2<T>{(T)0, (T)0};
            } else {
                const int q = (p - (p & 1)) >> 1;
                const C2<T> t = tw[q < 0 ? q + lc.M : q];
                C2<T> m{t.x, -t.y};
                if (p & 1) m = mul(m, half);
                v[s] = scl(mul(v[s], m), inv);
            }
        }
    }
    __device__ void store(const Geo& g, const LineCtx& lc, State&, C2<T> (&v)[8], double (&)[1]) const {
        // source offset s (within its instance) -> even output offset: x: 2s; y: 2s - x;
        // z: 2s - (y n_x + x); the odd neighbour is one output step further along AX.
        const int64_t nx = g.n[0], nxy = (int64_t)g.n[0] * g.n[1];
        const int64_t keep = AX == 0 ? 0 : (AX == 1 ? (int64_t)lc.i1 : (int64_t)lc.i2 * nx + lc.i1);
        const int64_t step = AX == 0 ? 1 : (AX == 1 ? nx : nxy);
        C2<T>* o = out + 2 * lc.off_b;
        const int64_t e0 = 2 * (lc.at(0) - lc.off_b) - keep;  // the points of a thread are TPL apart
        const int64_t de = 2 * (int64_t)lc.TPL * lc.stride;
        // the inputs are re-read (cached): keeping them across the transforms put them in scratch memory in
        // FP64, where even the eight of them ahead of the first store cost more than the trips between the
        // stores that they save (128^3 FP64: 180 us read one by one, 219 ahead; FP32 89, 87)
        constexpr bool kAhead = sizeof(T) == 4;
        C2<T> f0[8];
        if constexpr (kAhead) {
#pragma unroll
            for (int s = 0; s < 8; ++s) f0[s] = f[lc.at(s)];
        }
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            o[e0 + s * de] = kAhead ? f0[s] : f[lc.at(s)];
            o[e0 + s * de + step] = v[s];
        }
    }
};

// g with axes [0, upto) doubled (the geometry of the source of the pass along `upto`).
static Geo doubled_upto(const Geo& g, int upto) {
    Geo d = g;
    for (int a = 0; a < upto; ++a) {
        d.n[a] *= 2;
        d.lg[a] += 1;
        d.N *= 2;
        d.h[a] *= 0.5;
        d.cell *= 0.5;
    }
    return d;
}

template <typename T, int AX>
static OpProlong<T, AX> prolong_op(const Geo& g, const C2<T>* src, C2<T>* dst) {
    const double a = 3.141592653589793238462643383279502884 / g.n[AX];
    return OpProlong<T, AX>{src, dst, std::cos(a), std::sin(a)};
}

template <typename T>
static hipError_t prolong_t(const Geo& g, const Twiddles& tw, const void* in, void* out, void* tmp, hipStream_t s) {
    const bool f64 = sizeof(T) == 8;
    Partials none{nullptr, 0, 0, 0};
    hipError_t e;
    const C2<T>* src = (const C2<T>*)in;
    C2<T>* dst = (C2<T>*)out;
    C2<T>* t = (C2<T>*)tmp;
    if (g.dim == 1) return launch_pass<T, 0>(g, 1, tw.get(0, f64), prolong_op<T, 0>(g, src, dst), none, s);
    // 2-D: x into tmp (2N), y into out.  3-D: x into the last quarter of out, y into tmp (4N),
    // z into out (the x result is dead by then; passes on one stream run in order).
    C2<T>* xo = g.dim == 2 ? t : dst + 6 * g.N;
    if ((e = launch_pass<T, 0>(g, 1, tw.get(0, f64), prolong_op<T, 0>(g, src, xo), none, s)) != hipSuccess) return e;
    const Geo g1 = doubled_upto(g, 1);
    if (g.dim == 2) return launch_pass<T, 1>(g1, 1, tw.get(1, f64), prolong_op<T, 1>(g1, xo, dst), none, s);
    if ((e = launch_pass<T, 1>(g1, 1, tw.get(1, f64), prolong_op<T, 1>(g1, xo, t), none, s)) != hipSuccess) return e;
    const Geo g2 = doubled_upto(g, 2);
    return launch_pass<T, 2>(g2, 1, tw.get(2, f64), prolong_op<T, 2>(g2, t, dst), none, s);
}

hipError_t op_prolong(const Geo& g, bool f64, const Twiddles& tw, const void* in, void* out, void* tmp, hipStream_t s) {
    return f64 ? prolong_t<double>(g, tw, in, out, tmp, s) : prolong_t<float>(g, tw, in, out, tmp, s);
}

// ---------------------------------------------------------------------------------------------
// Tile measurement: for each axis, the directional pass (forward transform, kinetic multiplier,
// inverse transform, store) over B fields is timed for every valid number of lines per workgroup,
// and the fastest is recorded for the grid, point size and batch size.
// ---------------------------------------------------------------------------------------------
template <typename T, int AX>
static hipError_t tune_axis(const Geo& g, int B, const Twiddles& tw, const C2<T>* f, C2<T>* out, hipStream_t s,
                            int& best_C, double& best_us) {
    const int cb = (int)sizeof(C2<T>);
    const int TPL = g.n[AX] / 8;
    OpApply<T, AX> op{f, nullptr, out, nullptr, 0.0, 0.0, 0, 0};
    Partials none{nullptr, 0, 0, 0};
    hipEvent_t e0, e1;
    hipError_t e;
    if ((e = hipEventCreate(&e0)) != hipSuccess) return e;
    if ((e = hipEventCreate(&e1)) != hipSuccess) return e;
    best_C = 0;
    best_us = 0.0;
    for (int C = fewest_tuned_lines(g, AX, cb); C * TPL <= max_pass_threads(g, AX) && e == hipSuccess; C *= 2) {
        if (!valid_lines(g, AX, cb, C)) continue;
        constexpr int kWarm = 2, kReps = 10;
        for (int r = 0; r < kWarm && e == hipSuccess; ++r) e = launch_pass<T, AX>(g, B, tw.get(AX, sizeof(T) == 8), op, none, s, nullptr, C);
        if (e == hipSuccess) e = hipEventRecord(e0, s);
        for (int r = 0; r < kReps && e == hipSuccess; ++r) e = launch_pass<T, AX>(g, B, tw.get(AX, sizeof(T) == 8), op, none, s, nullptr, C);
        if (e == hipSuccess) e = hipEventRecord(e1, s);
        if (e == hipSuccess) e = hipEventSynchronize(e1);
        float ms = 0.0f;
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
        const double us = 1e3 * ms / kReps;
        if (e == hipSuccess && (best_C == 0 || us < best_us)) {
            best_C = C;
            best_us = us;
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (e == hipSuccess && best_C > 0) record_tuned_lines(g, AX, cb, B, best_C);
    return e;
}

template <typename T>
static hipError_t autotune_t(const Geo& g, int B, const Twiddles& tw, void* f, void* out, hipStream_t s, int tiles[3],
                             double us[3]) {
    const C2<T>* F = (const C2<T>*)f;
    C2<T>* O = (C2<T>*)out;
    hipError_t e = tune_axis<T, 0>(g, B, tw, F, O, s, tiles[0], us[0]);
    if (e == hipSuccess && g.dim > 1) e = tune_axis<T, 1>(g, B, tw, F, O, s, tiles[1], us[1]);
    if (e == hipSuccess && g.dim > 2) e = tune_axis<T, 2>(g, B, tw, F, O, s, tiles[2], us[2]);
    return e;
}

hipError_t op_autotune(const Geo& g, bool f64, int B, const Twiddles& tw, void* f, void* out, hipStream_t s,
                       int tiles[3], double us[3]) {
    return f64 ? autotune_t<double>(g, B, tw, f, out, s, tiles, us) : autotune_t<float>(g, B, tw, f, out, s, tiles, us);
}

// ---------------------------------------------------------------------------------------------
// Energy: forward transforms only; Parseval turns <phi, F^{-1} sigma F phi> into
// (1/M) sum sigma |F phi|^2 per line.  Sums: {kinetic, rotation, potential, quartic}.
// ---------------------------------------------------------------------------------------------
template <typename T, int AX>
struct OpEnergy {
    static constexpr bool FWD = true, INV = false, SCALARS = false, PREFETCH = true, WIDE = false;
    static constexpr int K = 4;
    static constexpr unsigned MAXMASK = 0;
    const C2<T>* phi;
    const T* V;
    double omega;
    struct State {
        C2<T> f0[8];
        T V[AX == 0 ? 8 : 1];
    };
    __device__ void prefetch(const Geo&, const LineCtx& lc, State& st) const {
#pragma unroll
        for (int s = 0; s < 8; ++s) st.f0[s] = phi[lc.at(s)];
    }
    __device__ void prefetch_tail(const Geo&, const LineCtx& lc, State& st) const {
        if constexpr (AX == 0) {
#pragma unroll
            for (int s = 0; s < 8; ++s) st.V[s] = V[lc.at(s)];
        }
    }
    __device__ void load(const Geo&, const LineCtx&, State& st, C2<T> (&v)[8], double (&)[K]) const {
#pragma unroll
        for (int s = 0; s < 8; ++s) v[s] = st.f0[s];
    }
    template <int LG>
    __device__ void spectral(const Geo& g, const LineCtx& lc, State&, C2<T> (&v)[8], double (&acc)[4], C2<T>*,
                             const C2<T>*) const {
        const double rot = rot_coef<AX>(g, lc, omega);
        const double inv = 1.0 / lc.M;  // 1/M (exact for M = 2^k)
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const double xi = freq_of(lc.k(s), lc.M, g.dk[AX]);
            const double w = (double)abs2(v[s]) * inv;
            acc[0] += 0.5 * xi * xi * w;
            acc[1] += rot * xi * w;
        }
    }
    __device__ void store(const Geo&, const LineCtx&, State& st, C2<T> (&)[8], double (&acc)[4]) const {
        if constexpr (AX == 0) {
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const double r = (double)abs2(st.f0[s]);
                acc[2] += (double)st.V[s] * r;
                acc[3] += r * r;
            }
        }
    }
};

// Sum the per-block partials of up to three passes and scale into {kin, pot, inter, rot}.  host
// (nullable): the same in mapped host memory; E (nullable): their sum in the field precision.
template <typename T>
__global__ __launch_bounds__(256) void k_energy_collect(const double* p0, int n0, const double* p1, int n1,
                                                        const double* p2, int n2, double cell, double beta,
                                                        double* dst, double* host, T* E) {
    __shared__ double red[16 * 4 + 8];
    double v[4] = {0, 0, 0, 0};
    const double* ps[3] = {p0, p1, p2};
    const int ns[3] = {n0, n1, n2};
    for (int q = 0; q < 3; ++q) {
        if (!ps[q]) continue;
        for (int blk = threadIdx.x; blk < ns[q]; blk += blockDim.x)
            for (int k = 0; k < 4; ++k) v[k] += ps[q][(size_t)blk * 4 + k];
    }
    __shared__ double T4[4];
    block_reduce<4>(v, red, T4);
    if (threadIdx.x == 0) {
        const double h[4] = {cell * T4[0],                // <phi, T phi>
                             cell * T4[2],                // <phi, V phi>
                             0.5 * beta * cell * T4[3],   // beta/2 h^d sum |phi|^4
                             cell * T4[1]};               // <phi, R phi> = -omega Re<phi, L_z phi>
        for (int k = 0; k < 4; ++k) {
            dst[k] = h[k];
            if (host) host[k] = h[k];
        }
        if (E) *E = (T)(h[0] + h[1] + h[2] + h[3]);
    }
}

// Row regions of the passes along axes [0, axes) of one field, K sums per row: the tiles C and row counts nb,
// settled once for the launches and their consumer (another thread may record a tile meanwhile).  Fails when the
// rows exceed the buffer.
static hipError_t field_rows(const Geo& g, int complex_bytes, int axes, int K, const Reduce& red, int C[3], int nb[3]) {
    size_t rows = 0;
    for (int a = 0; a < axes; ++a) {
        C[a] = pass_lines_per_block(g, a, complex_bytes, 1, false);
        nb[a] = (int)(lines_per_field(g, a) / C[a]);
        rows += (size_t)nb[a];
    }
    return sizeof(double) * rows * K <= red.parts.bytes ? hipSuccess : hipErrorInvalidValue;
}

template <typename T>
static hipError_t energy_t(const Geo& g, const Twiddles& tw, const void* phi, const void* V, double beta,
                           double omega, Reduce& red, double* dst, double* host, void* E, hipStream_t s) {
    const bool f64 = sizeof(T) == 8;
    const int cb = (int)sizeof(C2<T>);
    const C2<T>* P = (const C2<T>*)phi;
    double* parts = (double*)red.parts.ptr;
    const double* pp[3] = {nullptr, nullptr, nullptr};
    int nn[3] = {0, 0, 0}, C[3];
    hipError_t e;
    if ((e = field_rows(g, cb, g.dim, 4, red, C, nn)) != hipSuccess) return e;
    size_t off = 0;
    for (int ax = 0; ax < g.dim; ++ax) {
        Partials pr{parts + off, 0, 0, 0};
        if (ax == 0) e = launch_pass<T, 0>(g, 1, tw.get(0, f64), OpEnergy<T, 0>{P, (const T*)V, omega}, pr, s, nullptr, C[0]);
        else if (ax == 1) e = launch_pass<T, 1>(g, 1, tw.get(1, f64), OpEnergy<T, 1>{P, (const T*)V, omega}, pr, s, nullptr, C[1]);
        else e = launch_pass<T, 2>(g, 1, tw.get(2, f64), OpEnergy<T, 2>{P, (const T*)V, omega}, pr, s, nullptr, C[2]);
        if (e != hipSuccess) return e;
        pp[ax] = parts + off;
        off += (size_t)nn[ax] * 4;
    }
    hipLaunchKernelGGL(k_energy_collect<T>, dim3(1), dim3(256), 0, s, pp[0], nn[0], pp[1], nn[1], pp[2], nn[2],
                       g.cell, beta, dst, host, (T*)E);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Backward of the energy in the passes of one H apply: the gradient 2 h^d H phi (the last pass scales
// what it writes), h^d |phi|^2 and the sums of dE/dbeta = h^d/2 sum |phi|^4 (x pass) and dE/domega = <phi, -L_z phi>
// (Parseval, on the transforms that the apply makes anyway).  E is affine in beta and omega, so both
// derivatives are the energy's own sums at beta = omega = 1.  gE (nullable): a factor in device memory.
// A separate apply, scaling, density and energy took 8 launches and 23 s N bytes in 2-D against 3 launches
// and 12 s N here: 640^2 FP64, 58 us of kernels then, 32 now.
// ---------------------------------------------------------------------------------------------
template <typename T, int AX, bool LAST>
struct OpEnergyGrad {
    static constexpr bool FWD = true, INV = true, SCALARS = false, PREFETCH = true, WIDE = false, FIXED = true;
    static constexpr int K = AX < 2 ? 2 : 0;  // {quartic, rotation}
    static constexpr int KA = K > 0 ? K : 1;
    static constexpr unsigned MAXMASK = 0;
    static constexpr bool PW = AX == 0;
    const C2<T>* f;
    const C2<T>* acc;  // strided passes: the running sum
    C2<T>* out;
    const T* V;
    T* gV;             // x pass, nullable
    const T* gE;       // nullable
    double beta, omega;
    struct State {
        C2<T> f0[8];
        C2<T> a[PW ? 1 : 8];
        T V[PW ? 8 : 1];
    };
    __device__ void prefetch(const Geo&, const LineCtx& lc, State& st) const {
#pragma unroll
        for (int s = 0; s < 8; ++s) st.f0[s] = f[lc.at(s)];
    }
    __device__ void prefetch_tail(const Geo&, const LineCtx& lc, State& st) const {
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            if constexpr (PW) st.V[s] = V[lc.at(s)];
            if constexpr (!PW) st.a[s] = acc[lc.at(s)];
        }
    }
    __device__ void load(const Geo&, const LineCtx&, State& st, C2<T> (&v)[8], double (&)[KA]) const {
#pragma unroll
        for (int s = 0; s < 8; ++s) v[s] = st.f0[s];
    }
    template <int LG>
    __device__ void spectral(const Geo& g, const LineCtx& lc, State&, C2<T> (&v)[8], double (&sum)[KA], C2<T>*,
                             const C2<T>*) const {
        const double one = rot_coef<AX>(g, lc, 1.0);  // rotation symbol at omega = 1
        const double rot = rot_coef<AX>(g, lc, omega);
        const double inv = 1.0 / lc.M;  // 1/M (exact for M = 2^k)
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const double xi = freq_of(lc.k(s), lc.M, g.dk[AX]);
            if constexpr (K > 0) sum[1] += one * xi * ((double)abs2(v[s]) * inv);
            v[s] = scl(v[s], (T)((0.5 * xi * xi + rot * xi) * inv));
        }
    }
    __device__ void store(const Geo& g, const LineCtx& lc, State& st, C2<T> (&v)[8], double (&sum)[KA]) const {
        const T scale = (T)(2.0 * g.cell), cell = (T)g.cell;
        const T ge = gE ? *gE : (T)1;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int64_t i = lc.at(s);
            C2<T> o = v[s];
            if constexpr (PW) {
                const T r = abs2(st.f0[s]);
                o = add(o, scl(st.f0[s], st.V[s] + (T)beta * r));
                sum[0] += (double)r * (double)r;
                if (gV) gV[i] = gE ? ge * (cell * r) : cell * r;
            } else {
                o = add(o, st.a[s]);
            }
            if constexpr (LAST) {
                o = scl(o, scale);
                if (gE) o = scl(o, ge);
            }
            out[i] = o;
        }
    }
};

// {dE/dbeta, dE/domega} from the partial rows of the x and y passes, into dst (FP64) or, times *gE, into the
// field-precision scalars db and dw (nullable).
template <typename T>
__global__ __launch_bounds__(256) void k_grad_collect(const double* p0, int n0, const double* p1, int n1, double cell,
                                                      double* dst, T* db, T* dw, const T* gE) {
    __shared__ double red[8 * 2];
    double v[2] = {0.0, 0.0};
    for (int i = threadIdx.x; i < n0; i += blockDim.x) {
        v[0] += p0[2 * (size_t)i];
        v[1] += p0[2 * (size_t)i + 1];
    }
    for (int i = threadIdx.x; i < n1; i += blockDim.x) v[1] += p1[2 * (size_t)i + 1];
    block_reduce_to<2, 0u>(v, red, [=](int k, double t) {
        const double x = k == 0 ? 0.5 * cell * t : cell * t;
        if (dst) dst[k] = x;
        T* const to = k == 0 ? db : dw;
        if (to) *to = gE ? *gE * (T)x : (T)x;
    });
}

template <typename T>
static hipError_t energy_grad_t(const Geo& g, const Twiddles& tw, const void* phi, const void* V, void* gphi, void* gV,
                                double beta, double omega, Reduce& red, double* dst, void* db, void* dw,
                                const void* gE, void* tmp, hipStream_t s) {
    const bool f64 = sizeof(T) == 8;
    const int cb = (int)sizeof(C2<T>);
    const C2<T>* F = (const C2<T>*)phi;
    C2<T>*const O = (C2<T>*)gphi, *const W = (C2<T>*)tmp;
    const T *const Vt = (const T*)V, *const ge = (const T*)gE;
    int nn[3] = {0, 0, 0}, C[3];
    hipError_t e = field_rows(g, cb, std::min(g.dim, 2), 2, red, C, nn);
    if (e != hipSuccess) return e;
    const int n0 = nn[0], n1 = nn[1];
    double* const p0 = (double*)red.parts.ptr;
    double* const p1 = p0 + 2 * (size_t)n0;
    const Partials r0{p0, n0, n0, 0}, r1{p1, n1, n1, 0}, none{nullptr, 0, 0, 0};
    if (g.dim == 1) {
        OpEnergyGrad<T, 0, true> ox{F, nullptr, O, Vt, (T*)gV, ge, beta, omega};
        e = launch_pass<T, 0>(g, 1, tw.get(0, f64), ox, r0, s, nullptr, C[0]);
    } else {
        OpEnergyGrad<T, 0, false> ox{F, nullptr, W, Vt, (T*)gV, ge, beta, omega};
        e = launch_pass<T, 0>(g, 1, tw.get(0, f64), ox, r0, s, nullptr, C[0]);
        if (e == hipSuccess && g.dim == 2) {
            OpEnergyGrad<T, 1, true> oy{F, W, O, nullptr, nullptr, ge, beta, omega};
            e = launch_pass<T, 1>(g, 1, tw.get(1, f64), oy, r1, s, nullptr, C[1]);
        } else if (e == hipSuccess) {
            OpEnergyGrad<T, 1, false> oy{F, W, W, nullptr, nullptr, ge, beta, omega};
            e = launch_pass<T, 1>(g, 1, tw.get(1, f64), oy, r1, s, nullptr, C[1]);
            OpEnergyGrad<T, 2, true> oz{F, W, O, nullptr, nullptr, ge, beta, omega};
            if (e == hipSuccess) e = launch_pass<T, 2>(g, 1, tw.get(2, f64), oz, none, s);
        }
    }
    if (e != hipSuccess || !(dst || db || dw)) return e;
    hipLaunchKernelGGL(k_grad_collect<T>, dim3(1), dim3(256), 0, s, p0, n0, p1, n1, g.cell, dst, (T*)db, (T*)dw, ge);
    return hipGetLastError();
}

hipError_t op_energy_grad(const Geo& g, bool f64, const Twiddles& tw, const void* phi, const void* V, void* gphi,
                          void* gV, double beta, double omega, Reduce& red, double* dst, void* db, void* dw,
                          const void* gE, void* tmp, hipStream_t s) {
    return f64 ? energy_grad_t<double>(g, tw, phi, V, gphi, gV, beta, omega, red, dst, db, dw, gE, tmp, s)
               : energy_grad_t<float>(g, tw, phi, V, gphi, gV, beta, omega, red, dst, db, dw, gE, tmp, s);
}

hipError_t op_energy(const Geo& g, bool f64, const Twiddles& tw, const void* phi, const void* V, double beta,
                     double omega, Reduce& red, double* dst, hipStream_t s, double* host, void* E) {
    return f64 ? energy_t<double>(g, tw, phi, V, beta, omega, red, dst, host, E, s)
               : energy_t<float>(g, tw, phi, V, beta, omega, red, dst, host, E, s);
}

__global__ void k_lambda_tilde(const double* parts, double* dst) {
    if (threadIdx.x == 0) *dst = parts[0] + parts[1] + 2.0 * parts[2];
}

hipError_t op_lambda_tilde(const double* parts, double* dst, hipStream_t s) {
    hipLaunchKernelGGL(k_lambda_tilde, dim3(1), dim3(64), 0, s, parts, dst);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Preconditioners.  Scaling kinds: 0 none, 1 by (alpha + V + beta|phi|^2)^{-1/2}, 2 by its inverse.
// The spectral multiplier 1/(alpha + |k|^2/2) (with the 1/N of the inverse transforms) is applied
// in the pass that does both the forward and the inverse transform (the last axis).
// ---------------------------------------------------------------------------------------------
template <typename T, int AX, bool F, bool I>
struct OpPre {
    static constexpr bool FWD = F, INV = I, SCALARS = false, PREFETCH = true, WIDE = false, FIXED = true;
    static constexpr int K = 0;
    static constexpr unsigned MAXMASK = 0;
    // only the x passes scale: the prologue's and the epilogue's V and phi (1-D does both)
    static constexpr bool PRE = AX == 0 && F, POST = AX == 0 && I;
    const C2<T>* in;
    C2<T>* out;
    const C2<T>* phi;
    const T* V;
    const double* alpha;
    double beta;
    int pre, post;
    struct State {
        C2<T> f0[8], ph[PRE || POST ? 8 : 1];
        T V[PRE || POST ? 8 : 1];
    };
    __device__ void scale_inputs(const LineCtx& lc, State& st) const {
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int64_t i = lc.at(s);
            st.V[s] = V[i];
            st.ph[s] = phi[i];
        }
    }
    __device__ void prefetch(const Geo&, const LineCtx& lc, State& st) const {
#pragma unroll
        for (int s = 0; s < 8; ++s) st.f0[s] = in[lc.at(s)];
        if constexpr (PRE)
            if (pre) scale_inputs(lc, st);
    }
    __device__ void prefetch_tail(const Geo&, const LineCtx& lc, State& st) const {
        if constexpr (POST)
            if (post && !(PRE && pre)) scale_inputs(lc, st);
    }
    __device__ void load(const Geo&, const LineCtx&, State& st, C2<T> (&v)[8], double (&)[1]) const {
        const double a = *alpha;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            v[s] = st.f0[s];
            if constexpr (PRE)
                if (pre) v[s] = scl(v[s], pv_scale<T>(pre, a, st.V[s], abs2(st.ph[s]), beta));
        }
    }
    template <int LG>
    __device__ void spectral(const Geo& g, const LineCtx& lc, State&, C2<T> (&v)[8], double (&)[1], C2<T>*,
                             const C2<T>*) const {
        if (!(F && I)) return;
        const double a = *alpha;
        // frequencies of the other (already transformed) axes
        double ko = 0.0;
        if (AX == 1) {
            const double xi = freq_of(lc.i1, g.n[0], g.dk[0]);
            ko = xi * xi;
        } else if (AX == 2) {
            const double xi = freq_of(lc.i1, g.n[0], g.dk[0]);
            const double mu = freq_of(lc.i2, g.n[1], g.dk[1]);
            ko = xi * xi + mu * mu;
        }
        const double invN = 1.0 / (double)g.N;  // 1/N (exact for powers of two)
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const double k = freq_of(lc.k(s), lc.M, g.dk[AX]);
            v[s] = scl(v[s], (T)(invN / (a + 0.5 * (ko + k * k))));
        }
    }
    __device__ void store(const Geo&, const LineCtx& lc, State& st, C2<T> (&v)[8], double (&)[1]) const {
        const double a = post ? *alpha : 0.0;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            C2<T> o = v[s];
            if constexpr (POST)
                if (post) o = scl(o, pv_scale<T>(post, a, st.V[s], abs2(st.ph[s]), beta));
            out[lc.at(s)] = o;
        }
    }
};

template <typename T>
__global__ void k_precond_diag(const C2<T>* r, C2<T>* out, const C2<T>* phi, const T* V, const double* alpha,
                               double beta, int kind, int64_t N) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    C2<T> v = r[i];
    if (kind == GPE_P_POTENTIAL) v = scl(v, pv_scale<T>(2, *alpha, V[i], abs2(phi[i]), beta));
    out[i] = v;
}

// The middle passes of P_Delta on a field transformed along x, in place: forward y (z), the multiplier
// 1/(alpha + |k|^2/2) with the 1/N of the inverse transforms, inverse (z) y.
template <typename T>
static hipError_t kinetic_middle(const Geo& g, const Twiddles& tw, C2<T>* w, const double* alpha, hipStream_t s) {
    const bool f64 = sizeof(T) == 8;
    Partials none{nullptr, 0, 0, 0};
    hipError_t e;
    if (g.dim == 2) {
        OpPre<T, 1, true, true> y{w, w, nullptr, nullptr, alpha, 0.0, 0, 0};
        return launch_pass<T, 1>(g, 1, tw.get(1, f64), y, none, s);
    }
    OpPre<T, 1, true, false> y1{w, w, nullptr, nullptr, alpha, 0.0, 0, 0};
    if ((e = launch_pass<T, 1>(g, 1, tw.get(1, f64), y1, none, s)) != hipSuccess) return e;
    OpPre<T, 2, true, true> z{w, w, nullptr, nullptr, alpha, 0.0, 0, 0};
    if ((e = launch_pass<T, 2>(g, 1, tw.get(2, f64), z, none, s)) != hipSuccess) return e;
    OpPre<T, 1, false, true> y2{w, w, nullptr, nullptr, alpha, 0.0, 0, 0};
    return launch_pass<T, 1>(g, 1, tw.get(1, f64), y2, none, s);
}

hipError_t op_kinetic_middle(const Geo& g, bool f64, const Twiddles& tw, void* w, const double* alpha_dev,
                             hipStream_t s) {
    return f64 ? kinetic_middle<double>(g, tw, (C2<double>*)w, alpha_dev, s)
               : kinetic_middle<float>(g, tw, (C2<float>*)w, alpha_dev, s);
}

// The y part of L added to `out` (3-D: the pass between the first and the last), in place.
hipError_t op_apply_y(const Geo& g, bool f64, const Twiddles& tw, const void* f, void* out, double omega,
                      hipStream_t s) {
    const Partials none{nullptr, 0, 0, 0};
    if (f64) {
        OpApply<double, 1> oy{(const C2<double>*)f, (const C2<double>*)out, (C2<double>*)out, nullptr, 0.0, omega, 0, 0};
        return launch_pass<double, 1>(g, 1, tw.get(1, true), oy, none, s);
    }
    OpApply<float, 1> oy{(const C2<float>*)f, (const C2<float>*)out, (C2<float>*)out, nullptr, 0.0, omega, 0, 0};
    return launch_pass<float, 1>(g, 1, tw.get(1, false), oy, none, s);
}

// Full multi-dimensional P_Delta with pre/post scalings: x forward, middle axes, x inverse.
template <typename T>
static hipError_t kinetic_chain(const Geo& g, const Twiddles& tw, const C2<T>* r, C2<T>* out, C2<T>* tmp,
                                const C2<T>* phi, const T* V, const double* alpha, double beta, int pre,
                                int post, hipStream_t s) {
    const bool f64 = sizeof(T) == 8;
    Partials none{nullptr, 0, 0, 0};
    hipError_t e;
    if (g.dim == 1) {
        OpPre<T, 0, true, true> op{r, out, phi, V, alpha, beta, pre, post};
        return launch_pass<T, 0>(g, 1, tw.get(0, f64), op, none, s);
    }
    OpPre<T, 0, true, false> x1{r, tmp, phi, V, alpha, beta, pre, 0};
    if ((e = launch_pass<T, 0>(g, 1, tw.get(0, f64), x1, none, s)) != hipSuccess) return e;
    if ((e = kinetic_middle<T>(g, tw, tmp, alpha, s)) != hipSuccess) return e;
    OpPre<T, 0, false, true> x2{tmp, out, phi, V, alpha, beta, 0, post};
    return launch_pass<T, 0>(g, 1, tw.get(0, f64), x2, none, s);
}

template <typename T>
static hipError_t precond_t(const Geo& g, const Twiddles& tw, int kind, const void* phi, const void* V,
                            const double* alpha, double beta, const void* r, void* out, void* tmp, hipStream_t s) {
    const C2<T>* R = (const C2<T>*)r;
    C2<T>* O = (C2<T>*)out;
    const C2<T>* P = (const C2<T>*)phi;
    const T* Vt = (const T*)V;
    if (kind == GPE_P_NONE || kind == GPE_P_POTENTIAL) {
        const int64_t N = g.N;
        hipLaunchKernelGGL(k_precond_diag<T>, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, R, O, P, Vt, alpha,
                           beta, kind, N);
        return hipGetLastError();
    }
    int pre = 0, post = 0;
    if (kind == GPE_P_COMBINED) pre = post = 1;  // P_V^{1/2} P_Delta P_V^{1/2}
    if (kind == GPE_P_C1) post = 2;              // P_V P_Delta
    if (kind == GPE_P_C2) pre = 2;               // P_Delta P_V
    return kinetic_chain<T>(g, tw, R, O, (C2<T>*)tmp, P, Vt, alpha, beta, pre, post, s);
}

hipError_t op_precond(const Geo& g, bool f64, const Twiddles& tw, int kind, const void* phi, const void* V,
                      const double* alpha_dev, double beta, const void* r, void* out, void* tmp, hipStream_t s) {
    return f64 ? precond_t<double>(g, tw, kind, phi, V, alpha_dev, beta, r, out, tmp, s)
               : precond_t<float>(g, tw, kind, phi, V, alpha_dev, beta, r, out, tmp, s);
}

// Minimum of alpha + V + beta |phi|^2 (SPD check of P_V), two-level deterministic reduction.
template <typename T>
__global__ void k_min_diag(const C2<T>* phi, const T* V, const double* alpha, double beta, int64_t N,
                           double* parts) {
    __shared__ double red[16 + 4];
    double m[1] = {1e300};
    const double a = *alpha;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (int64_t)gridDim.x * blockDim.x)
        m[0] = fmin(m[0], a + (double)V[i] + beta * (double)abs2(phi[i]));
    m[0] = -m[0];
    __shared__ double o1[1];
    block_reduce<1, 1u>(m, red, o1);
    if (threadIdx.x == 0) parts[blockIdx.x] = -o1[0];
}

__global__ __launch_bounds__(256) void k_min_collect(const double* parts, int n, double* dst) {
    __shared__ double red[8];
    double m[1] = {-1e300};
    for (int i = threadIdx.x; i < n; i += blockDim.x) m[0] = fmax(m[0], -parts[i]);
    block_reduce_to<1, 1u>(m, red, [dst](int, double t) { *dst = -t; });
}

hipError_t op_min_diag(const Geo& g, bool f64, const void* phi, const void* V, const double* alpha_dev,
                       double beta, Reduce& red, double* dst, hipStream_t s) {
    const int blocks = 256;
    double* parts = (double*)red.parts.ptr;
    if (f64)
        hipLaunchKernelGGL(k_min_diag<double>, dim3(blocks), dim3(256), 0, s, (const C2<double>*)phi,
                           (const double*)V, alpha_dev, beta, g.N, parts);
    else
        hipLaunchKernelGGL(k_min_diag<float>, dim3(blocks), dim3(256), 0, s, (const C2<float>*)phi,
                           (const float*)V, alpha_dev, beta, g.N, parts);
    hipLaunchKernelGGL(k_min_collect, dim3(1), dim3(256), 0, s, parts, blocks, dst);
    return hipGetLastError();
}

}  // namespace gpe
