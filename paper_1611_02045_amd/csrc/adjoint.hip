// Implicit adjoint of a converged ground state (second-order conditions of Section 2).
//
// At a ground state phi* (H phi* = lambda phi*, ||phi*|| = 1) the tangent linearisation of the
// stationarity condition is A dphi = -Pi (d_theta H) phi* dtheta with
//   A = Pi (1/2 nabla^2 E(phi*) - lambda) Pi,   1/2 nabla^2 E[f] = H f + 2 beta Re(conj(phi) f) phi,
// on {phi*, i phi*}^perp in the real inner product Re<.,.> (the sphere's normal and the global
// phase, a null direction of the Hessian, are projected out; A is SPD there at a local minimum).
// For a loss with d l = Re<g, d phi>, the adjoint state mu solves A mu = Pi g and
// d l / d theta = -Re<mu, (d_theta H) phi*> (plus the loss's own explicit dependence).
// The solve is linear preconditioned CG with the projected combined preconditioner Pi P_C Pi, as a chain
// of fused passes (lin_passes.hpp); every CG scalar lives in device memory, so iterations are queued
// without host round trips and the host only polls a convergence flag.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <string>

#include "internal.hpp"
#include "plan.hpp"
#include "linear.hpp"
#include "lin_passes.hpp"

namespace gpe {

// f <- f - (c0 phi + c1 i phi) / ||phi||^2 with c = {Re<phi,f>, Re<i phi,f>} (device).
template <typename T>
__global__ void k_project(C2<T>* f, const C2<T>* phi, const double* c, const double* nphi2, int64_t N) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const T c0 = (T)(c[0] / *nphi2), c1 = (T)(c[1] / *nphi2);
    const C2<T> p = phi[i];
    // c0 phi + c1 (i phi) = (c0 p.x - c1 p.y, c0 p.y + c1 p.x)
    f[i] = mk(f[i].x - (c0 * p.x - c1 * p.y), f[i].y - (c0 * p.y + c1 * p.x));
}

// grad_V = -h^d Re(conj(mu) phi) (the adjoint part of dl/dV_k).
template <typename T>
__global__ void k_grad_V(const C2<T>* mu, const C2<T>* phi, T* gV, T cell, int64_t N) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N) gV[i] = -cell * redot(mu[i], phi[i]);
}

// v = |phi|^2 phi (the field (d_beta H) phi).
template <typename T>
__global__ void k_cubic(const C2<T>* phi, C2<T>* v, int64_t N) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N) v[i] = scl(phi[i], abs2(phi[i]));
}

template <typename T>
struct AdjCtx {
    const Geo* g;
    double* parts;  // kDotBlocks * 4
    hipStream_t s;
};

template <typename T>
static hipError_t dots(AdjCtx<T>& c, int nq, const C2<T>* a0, const C2<T>* b0, int i0, const C2<T>* a1,
                       const C2<T>* b1, int i1, double* dst) {
    return field_dots<T>(c.g->N, c.g->cell, c.parts, nq, a0, b0, i0, a1, b1, i1, dst, c.s);
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

template <typename T>
static int adjoint_impl(gpe_plan_t* plan, const void* phi_star, const void* V, const void* rhs, void* mu,
                        const gpe_pcg_opts_t* o, gpe_pcg_report_t* report, hipStream_t s) {
    const auto t0 = std::chrono::steady_clock::now();
    const Geo& g = plan->g;
    const int64_t N = g.N;
    const size_t cf = sizeof(C2<T>) * (size_t)N;
    HIPCHK(plan->tmp.ensure(6 * cf + 2 * sizeof(LinS) +
                            (64 + kDotBlocks * 4 + lin_rows_doubles(g)) * sizeof(double) + 256));
    char* base = (char*)plan->tmp.ptr;
    const C2<T>* phi = (const C2<T>*)phi_star;
    LinCtx<T> l{};
    l.g = &g;
    l.tw = &plan->tw;
    l.omega = plan->prob.omega;
    l.kind = GPE_P_COMBINED;
    l.f.phi = phi;
    l.f.V = (const T*)V;
    l.f.x = (C2<T>*)mu;
    l.f.r = (C2<T>*)(base + 0 * cf);
    l.f.z = (C2<T>*)(base + 1 * cf);
    l.f.p = (C2<T>*)(base + 2 * cf);
    l.f.q = (C2<T>*)(base + 3 * cf);
    l.f.w = (C2<T>*)(base + 4 * cf);
    C2<T>* hphi = (C2<T>*)(base + 5 * cf);
    l.S = (LinS*)(base + 6 * cf);
    double* sc = (double*)(base + 6 * cf + 2 * sizeof(LinS));  // [0..1] projections, [8] lambda~, [12] <phi,H phi>,
    l.rows = sc + 64 + kDotBlocks * 4;                         // [13] ||phi||^2, [16..19] energy parts
    l.s = s;
    AdjCtx<T> c{&g, sc + 64, s};
    // lambda and ||phi||^2 (fresh), lambda~ for the preconditioner
    HIPCHK(op_apply(g, sizeof(T) == 8, 1, plan->tw, phi_star, V, hphi, l.f.w, plan->prob.beta, plan->prob.omega, true, s));
    HIPCHK(dots<T>(c, 2, phi, hphi, 0, phi, phi, 0, sc + 12));
    HIPCHK(op_energy(g, sizeof(T) == 8, plan->tw, phi_star, V, plan->prob.beta, plan->prob.omega, plan->red, sc + 16, s));
    HIPCHK(op_lambda_tilde(sc + 16, sc + 8, s));
    // x = 0, r = Pi rhs
    hipLaunchKernelGGL(k_zero_c<T>, dim3(nblk(N)), dim3(256), 0, s, l.f.x, N);
    hipLaunchKernelGGL(k_copy_c<T>, dim3(nblk(N)), dim3(256), 0, s, (const C2<T>*)rhs, l.f.r, N);
    HIPCHK(dots<T>(c, 2, phi, l.f.r, 0, phi, l.f.r, 1, sc));
    hipLaunchKernelGGL(k_project<T>, dim3(nblk(N)), dim3(256), 0, s, l.f.r, phi, sc, sc + 13, N);
    HIPCHK(hipGetLastError());
    double h[6];
    HIPCHK(hipMemcpyAsync(h, sc + 8, sizeof(h), hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    LinS hs;
    std::memset(&hs, 0, sizeof(hs));
    hs.alpha = h[0];
    hs.lam = h[4] / h[5];
    hs.nphi2 = h[5];
    hs.beta = plan->prob.beta;
    hs.cell = g.cell;
    hs.tol2 = o->tol_res_inf * o->tol_res_inf;
    hs.max_it = o->max_iter;
    hs.hess = 1;
    HIPCHK(lin_solve<T>(l, hs, std::max(1, o->check_every)));
    const auto t1 = std::chrono::steady_clock::now();
    int st = hs.status == 0 ? GPE_OK : hs.status == 1 ? GPE_NOT_CONVERGED : hs.status == -4 ? GPE_ENONFINITE : GPE_EINVAL;
    if (report) {
        std::memset(report, 0, sizeof(*report));
        report->status = st;
        report->iters = hs.it;
        report->lambda = hs.lam;
        report->res_inf = hs.rr0 == 0.0 ? 0.0 : std::sqrt(hs.rr / hs.rr0);
        report->seconds = std::chrono::duration<double>(t1 - t0).count();
    }
    if (st == GPE_EINVAL) set_error("the projected Hessian is not positive definite (phi_star is not a local minimum)");
    if (st == GPE_ENONFINITE) set_error("non-finite value in the adjoint iteration");
    return st;
}

extern "C" int gpe_adjoint_solve(gpe_plan_t* plan, const void* phi_star, const void* V, const void* rhs, void* mu,
                                 const gpe_pcg_opts_t* opts, gpe_pcg_report_t* report, void* stream) {
    if (!plan || !phi_star || !V || !rhs || !mu || !opts) { set_error("NULL argument"); return GPE_EINVAL; }
    if (mu == rhs || mu == phi_star) { set_error("mu must not alias rhs or phi_star"); return GPE_EINVAL; }
    if (!(opts->tol_res_inf > 0.0) || opts->max_iter < 1) { set_error("need tol > 0 and max_iter >= 1"); return GPE_EINVAL; }
    return plan->f64() ? adjoint_impl<double>(plan, phi_star, V, rhs, mu, opts, report, (hipStream_t)stream)
                       : adjoint_impl<float>(plan, phi_star, V, rhs, mu, opts, report, (hipStream_t)stream);
}

// Parameter gradients of the adjoint part: grad_V = -h^d Re(conj(mu) phi) (device, nullable),
// *dl_dbeta = -Re<mu, |phi|^2 phi>, *dl_domega = +Re<mu, L_z phi> (host, nullable).
template <typename T>
static int param_grads_impl(gpe_plan_t* plan, const void* phi, const void* mu, void* grad_V, double* dl_dbeta,
                            double* dl_domega, hipStream_t s) {
    const Geo& g = plan->g;
    const int64_t N = g.N;
    const size_t cf = sizeof(C2<T>) * (size_t)N;
    HIPCHK(plan->tmp.ensure(2 * cf + 64 * sizeof(double) + kDotBlocks * 4 * sizeof(double) + 256));
    char* base = (char*)plan->tmp.ptr;
    double* sc = (double*)(base + 2 * cf);
    AdjCtx<T> c{&g, sc + 64, s};
    C2<T>* v = (C2<T>*)base;
    C2<T>* w = (C2<T>*)(base + cf);
    if (grad_V)
        hipLaunchKernelGGL(k_grad_V<T>, dim3(nblk(N)), dim3(256), 0, s, (const C2<T>*)mu, (const C2<T>*)phi, (T*)grad_V,
                           (T)g.cell, N);
    double h[2] = {0.0, 0.0};
    if (dl_dbeta) {
        hipLaunchKernelGGL(k_cubic<T>, dim3(nblk(N)), dim3(256), 0, s, (const C2<T>*)phi, v, N);
        HIPCHK(dots<T>(c, 1, (const C2<T>*)mu, v, 0, nullptr, nullptr, 0, sc));
        HIPCHK(hipMemcpyAsync(&h[0], sc, sizeof(double), hipMemcpyDeviceToHost, s));
    }
    if (dl_domega && g.dim >= 2) {
        HIPCHK(op_rotation(g, sizeof(T) == 8, plan->tw, phi, v, w, s));  // v = -L_z phi
        HIPCHK(dots<T>(c, 1, (const C2<T>*)mu, v, 0, nullptr, nullptr, 0, sc + 4));
        HIPCHK(hipMemcpyAsync(&h[1], sc + 4, sizeof(double), hipMemcpyDeviceToHost, s));
    }
    HIPCHK(hipStreamSynchronize(s));
    if (dl_dbeta) *dl_dbeta = -h[0];
    if (dl_domega) *dl_domega = g.dim >= 2 ? -h[1] : 0.0;
    return GPE_OK;
}

extern "C" int gpe_adjoint_param_grads(gpe_plan_t* plan, const void* phi_star, const void* mu, void* grad_V,
                                       double* dl_dbeta, double* dl_domega, void* stream) {
    if (!plan || !phi_star || !mu) { set_error("NULL argument"); return GPE_EINVAL; }
    return plan->f64() ? param_grads_impl<double>(plan, phi_star, mu, grad_V, dl_dbeta, dl_domega, (hipStream_t)stream)
                       : param_grads_impl<float>(plan, phi_star, mu, grad_V, dl_dbeta, dl_domega, (hipStream_t)stream);
}
