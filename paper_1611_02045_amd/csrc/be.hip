// Backward Euler discretisation of the normalised gradient flow (the BESP schemes of Section 4, run
// in Section 6 as BE_nu with a preconditioned Krylov inner solver).
//
// Outer step n (||phi_n|| = 1): lambda_n = <phi_n, H_{phi_n} phi_n>; stop when
// ||H_{phi_n} phi_n - lambda_n phi_n||_inf <= tol; otherwise solve
//   (I/dt + H_{phi_n} - s lambda_n) phit = phi_n / dt,   H_{phi_n} = L + beta |phi_n|^2 (frozen),
// with s = 1 for the scheme with the Lagrange multiplier (the multiplier on the new iterate, the
// reading under which the scheme is the plain one with the effective step dt / (1 - dt lambda_n))
// and s = 0 for the plain scheme, then phi_{n+1} = phit / ||phit||.  The inner solve is
// preconditioned linear CG from phit = phi_n (the operator is Hermitian, and positive definite
// when 1/dt > s (lambda_n - lambda_1)); the preconditioner is P_nu of Section 5.5 with the shift
// 1/dt of the BESP literature the paper cites.  The inner solve is the chain of fused passes of
// lin_passes.hpp: every CG scalar stays on the device; the host polls the inner state every
// `check_every` iterations and reads a few scalars per outer step.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <string>

#include "internal.hpp"
#include "linear.hpp"
#include "lin_passes.hpp"
#include "plan.hpp"

namespace gpe {

// The inner solve's start phit = phi and its residual phi / dt - A phi = s lambda phi - H phi.
template <typename T>
__global__ void k_be_start(C2<T>* x, C2<T>* r, const C2<T>* phi, const C2<T>* hphi, T slam, int64_t N) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const C2<T> p = phi[i];
    x[i] = p;
    r[i] = sub(scl(p, slam), hphi[i]);
}

// Per-block maxima of |Hphi - lambda phi| (lambda = sc[0] / sc[1]).
template <typename T>
__global__ __launch_bounds__(256) void k_be_resmax(const C2<T>* hphi, const C2<T>* phi, const double* sc, double* parts,
                                                   int64_t N) {
    __shared__ double red[4];
    __shared__ double out[1];
    const T lam = (T)(sc[0] / sc[1]);
    double m[1] = {0.0};
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (int64_t)gridDim.x * blockDim.x) {
        const C2<T> r = sub(hphi[i], scl(phi[i], lam));
        m[0] = fmax(m[0], (double)abs2(r));
    }
    block_reduce<1, 1u>(m, red, out);
    if (threadIdx.x == 0) parts[blockIdx.x] = out[0];
}

// sc[4] = sqrt(max of the parts); sc[5] = lambda = sc[0] / sc[1].
__global__ void k_be_scalars(const double* parts, int nb, double* sc) {
    __shared__ double red[4];
    __shared__ double out[1];
    double m[1] = {0.0};
    for (int b = threadIdx.x; b < nb; b += blockDim.x) m[0] = fmax(m[0], parts[b]);
    block_reduce<1, 1u>(m, red, out);
    if (threadIdx.x == 0) {
        sc[4] = sqrt(out[0]);
        sc[5] = sc[0] / sc[1];
    }
}

// phi = x / sqrt(nx2[0]).
template <typename T>
__global__ void k_be_normalise(C2<T>* phi, const C2<T>* x, const double* nx2, int64_t N) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N) phi[i] = scl(x[i], (T)(1.0 / sqrt(nx2[0])));
}

}  // namespace gpe

using namespace gpe;

#define HIPCHK(expr)                                                                    \
    do {                                                                                \
        hipError_t _e = (expr);                                                         \
        if (_e != hipSuccess) {                                                         \
            set_error(std::string("HIP error in " #expr ": ") + hipGetErrorString(_e)); \
            return GPE_EHIP;                                                            \
        }                                                                               \
    } while (0)

constexpr int64_t kBeInnerMax = 10000;

template <typename T>
static int be_impl(gpe_plan_t* plan, const void* V, void* phi_inout, double dt, int lambda_term,
                   const gpe_pcg_opts_t* o, double inner_tol, int64_t* inner_total, gpe_pcg_report_t* report,
                   hipStream_t s) {
    const auto t0 = std::chrono::steady_clock::now();
    const Geo& g = plan->g;
    const int64_t N = g.N;
    const size_t cf = sizeof(C2<T>) * (size_t)N;
    HIPCHK(plan->tmp.ensure(7 * cf + 2 * sizeof(LinS) +
                            (64 + kDotBlocks * 4 + lin_rows_doubles(g)) * sizeof(double) + 256));
    char* base = (char*)plan->tmp.ptr;
    const double beta = plan->prob.beta, omega = plan->prob.omega, invdt = 1.0 / dt;
    C2<T>* phi = (C2<T>*)phi_inout;
    C2<T>* hphi = (C2<T>*)(base + 0 * cf);
    LinCtx<T> c{};
    c.g = &g;
    c.tw = &plan->tw;
    c.omega = omega;
    c.kind = o->precond;
    c.f.phi = phi;
    c.f.V = (const T*)V;
    c.f.x = (C2<T>*)(base + 1 * cf);
    c.f.r = (C2<T>*)(base + 2 * cf);
    c.f.z = (C2<T>*)(base + 3 * cf);
    c.f.p = (C2<T>*)(base + 4 * cf);
    c.f.q = (C2<T>*)(base + 5 * cf);
    c.f.w = (C2<T>*)(base + 6 * cf);
    c.S = (LinS*)(base + 7 * cf);
    // [0..1] <phi,H phi>, <phi,phi>; [4] ||r||_inf; [5] lambda; [12] <x,x> (an inner product request
    // writes 4 consecutive slots)
    double* sc = (double*)(base + 7 * cf + 2 * sizeof(LinS));
    double* parts = sc + 64;
    c.rows = parts + kDotBlocks * 4;
    c.s = s;
    // normalise the start
    HIPCHK(field_dots<T>(N, g.cell, parts, 1, phi, phi, 0, nullptr, nullptr, 0, sc + 12, s));
    hipLaunchKernelGGL(k_be_normalise<T>, dim3(nblk(N)), dim3(256), 0, s, phi, phi, sc + 12, N);
    HIPCHK(hipGetLastError());
    int64_t inner = 0, n = 0;
    int st = GPE_NOT_CONVERGED;
    double hs[6] = {};  // sc[0..5]: [1] ||phi||^2, [4] ||r||_inf, [5] lambda
    for (n = 0;; ++n) {
        // lambda_n and the residual of phi_n
        HIPCHK(op_apply(g, sizeof(T) == 8, 1, plan->tw, phi, V, hphi, c.f.w, beta, omega, true, s));
        HIPCHK(field_dots<T>(N, g.cell, parts, 2, phi, hphi, 0, phi, phi, 0, sc, s));
        hipLaunchKernelGGL(k_be_resmax<T>, dim3(kDotBlocks), dim3(256), 0, s, hphi, phi, sc, parts, N);
        hipLaunchKernelGGL(k_be_scalars, dim3(1), dim3(256), 0, s, parts, kDotBlocks, sc);
        HIPCHK(hipGetLastError());
        HIPCHK(hipMemcpyAsync(hs, sc, sizeof(hs), hipMemcpyDeviceToHost, s));
        HIPCHK(hipStreamSynchronize(s));
        if (!std::isfinite(hs[4]) || !std::isfinite(hs[5])) {
            st = GPE_ENONFINITE;
            set_error("non-finite value in the backward Euler iteration");
            break;
        }
        if (hs[4] <= o->tol_res_inf) {
            st = GPE_OK;
            break;
        }
        if (n >= o->max_iter) break;
        const double slam = lambda_term ? hs[5] : 0.0;
        hipLaunchKernelGGL(k_be_start<T>, dim3(nblk(N)), dim3(256), 0, s, c.f.x, c.f.r, phi, hphi, (T)slam, N);
        LinS cs;
        std::memset(&cs, 0, sizeof(cs));
        cs.beta = beta;
        cs.cell = g.cell;
        cs.nphi2 = hs[1];
        cs.shift = invdt - slam;
        cs.alpha = invdt;
        cs.rr0 = hs[1] * invdt * invdt;  // ||phi / dt||^2
        cs.tol2 = inner_tol * inner_tol;
        cs.max_it = kBeInnerMax;
        HIPCHK(lin_solve<T>(c, cs, std::max(1, o->check_every)));
        inner += cs.it;
        if (cs.status == -1) {
            st = GPE_EINVAL;
            set_error("the backward Euler operator is not positive definite (reduce dt)");
            break;
        }
        if (cs.status == -4) {
            st = GPE_ENONFINITE;
            set_error("non-finite value in the inner solve");
            break;
        }
        // phi_{n+1} = phit / ||phit||
        HIPCHK(field_dots<T>(N, g.cell, parts, 1, c.f.x, c.f.x, 0, nullptr, nullptr, 0, sc + 12, s));
        hipLaunchKernelGGL(k_be_normalise<T>, dim3(nblk(N)), dim3(256), 0, s, phi, c.f.x, sc + 12, N);
        HIPCHK(hipGetLastError());
    }
    if (inner_total) *inner_total = inner;
    if (report) {
        std::memset(report, 0, sizeof(*report));
        report->status = st;
        report->iters = n;
        report->res_inf = hs[4];
        report->lambda = hs[5];
        double* ed = (double*)plan->red.scalars.ptr;
        double h[4] = {0.0, 0.0, 0.0, 0.0};
        HIPCHK(op_energy(g, sizeof(T) == 8, plan->tw, phi, V, beta, omega, plan->red, ed, s));
        HIPCHK(hipMemcpyAsync(h, ed, sizeof(h), hipMemcpyDeviceToHost, s));
        HIPCHK(hipStreamSynchronize(s));
        report->E = h[0] + h[1] + h[2] + h[3];
        report->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    }
    return st;
}

extern "C" int gpe_be_solve(gpe_plan_t* plan, const void* V, void* phi_inout, double dt, int lambda_term,
                            const gpe_pcg_opts_t* opts, double inner_tol, int64_t* inner_iters,
                            gpe_pcg_report_t* report, void* stream) {
    if (!plan || !V || !phi_inout || !opts) { set_error("NULL argument"); return GPE_EINVAL; }
    if (!(dt > 0.0) || !std::isfinite(dt)) { set_error("dt must be positive"); return GPE_EINVAL; }
    if (!(inner_tol > 0.0) || !(opts->tol_res_inf > 0.0) || opts->max_iter < 0) {
        set_error("need inner_tol > 0, tol_res_inf > 0 and max_iter >= 0");
        return GPE_EINVAL;
    }
    if (opts->precond < GPE_P_NONE || opts->precond > GPE_P_COMBINED) {
        set_error("the inner CG needs a symmetric preconditioner (none, kinetic, potential or combined)");
        return GPE_EINVAL;
    }
    return plan->f64() ? be_impl<double>(plan, V, phi_inout, dt, lambda_term, opts, inner_tol, inner_iters, report,
                                         (hipStream_t)stream)
                       : be_impl<float>(plan, V, phi_inout, dt, lambda_term, opts, inner_tol, inner_iters, report,
                                        (hipStream_t)stream);
}
