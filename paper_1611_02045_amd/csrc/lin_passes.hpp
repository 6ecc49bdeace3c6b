// One iteration of the preconditioned linear CG of the implicit adjoint and of backward Euler,
//   A x = b,  A f = Pi [L f + w(phi) f + 2 beta Re(conj(phi) f) phi]   (adjoint, w = beta|phi|^2 - lambda)
//             A f = L f + (1/dt - s lambda + beta|phi|^2) f            (backward Euler, Pi = 1)
// as a chain of fused passes, like the PCG iteration's (pcg_passes.hpp):
//
//   dir    p = Pi z + b p, then the x part of L p plus V p            [x pass; absorbs the sums of `post`:
//          convergence test and b]
//   apply  the y (z) part of L p and the pointwise part -> q; <p,q> and the projections of q  [last axis]
//   upd    x += a p, r -= a Pi q, P_V^{1/2} prologue, forward x       [x pass; absorbs the sums of `apply`: a]
//   (middle passes of P_Delta: op_kinetic_middle)
//   post   inverse x, P_V^{1/2} epilogue -> z; <r,r>, <r,z> and the projections of r and z  [x pass]
//
// The projections Pi are applied where their field is next read: with c = <phi, q>/||phi||^2 (and i phi)
// <p, Pi q> = <p, q> - c <p, phi>, so no pass over the fields is spent on them.  One iteration takes 5 launches
// (8 in 3-D).  The passes of a small grid are latency chains of 5.5-7.5 us each, so their number sets
// the time: with kernels of its own for each inner product, update, projection and scalar an adjoint
// iteration took 17 launches (13 in backward Euler).  256^2 FP64: 86 us an adjoint iteration then, 40
// now; 58 and 32 us an inner iteration of backward Euler.  Every sum is reduced in a fixed order, and every
// workgroup of a pass runs the same scalar logic (FP64) on the same rows; the state has two slots
// (S_dir after `dir`, S_upd after `upd`), so no pass writes a slot that it reads.
#pragma once

#include "internal.hpp"
#include "rows.hpp"
#include "symbols.hpp"

namespace gpe {

struct alignas(16) LinS {
    double lam, beta, omega, cell, nphi2;  // chemical potential, parameters, h^d, ||phi||^2
    double shift;                          // backward Euler: 1/dt - s lambda
    double alpha;                          // shift of the preconditioner
    double rz, rr, rr0, a, b;              // <r,z>, <r,r>, its reference, the CG coefficients
    double c0, c1, d0, d1;                 // components of q and of z along phi and i phi
    double tol2;
    int64_t it, max_it;
    int32_t done, status;                  // status -1: not positive definite, -4: non-finite, 1: max_it
    int32_t init;                          // the next `upd` only forms the first residual's z
    int32_t first;                         // the next `dir` starts the iteration (b = 0)
    int32_t update;                        // within `upd`: x and r are updated
    int32_t hess;                          // adjoint (projections, Hessian)
    int32_t pad[3];
};

// Sums of `apply` and of `post` (Im: along i phi).
enum : int { Q_PQ = 0, Q_PHIQ, Q_IPHIQ, Q_PPHI, Q_PIPHI, Q_K };
enum : int { Z_RR = 0, Z_RZ, Z_RPHI, Z_RIPHI, Z_PHIZ, Z_IPHIZ, Z_K };

template <typename T>
struct LinFields {
    const C2<T>* phi;
    const T* V;
    C2<T>*x, *r, *z, *p, *q, *w;
};

// Im(conj(a) b) = Re(conj(i a) b)
template <typename T>
__device__ __forceinline__ T imdot(C2<T> a, C2<T> b) { return a.x * b.y - a.y * b.x; }

// f - c0 phi - c1 (i phi)
template <typename T>
__device__ __forceinline__ C2<T> without_phi(C2<T> f, C2<T> ph, T c0, T c1) {
    return mk(f.x - (c0 * ph.x - c1 * ph.y), f.y - (c0 * ph.y + c1 * ph.x));
}

// Convergence test and the CG coefficient, from the sums of `post`.
__device__ __forceinline__ void lin_dir(LinS& S, const double* t) {
    if (S.done) return;
    const double w = S.cell;
    S.d0 = S.hess ? w * t[Z_PHIZ] / S.nphi2 : 0.0;
    S.d1 = S.hess ? w * t[Z_IPHIZ] / S.nphi2 : 0.0;
    const double rz = w * (t[Z_RZ] - S.d0 * t[Z_RPHI] - S.d1 * t[Z_RIPHI]), rr = w * t[Z_RR];
    S.rr = rr;
    if (S.first) {
        S.first = 0;
        S.b = 0.0;
        if (S.hess) S.rr0 = rr;  // relative to the projected right-hand side
        if (!isfinite(rr) || !isfinite(rz)) {
            S.status = -4;
            S.done = 1;
        }
        // zero right-hand side, or an initial guess that already solves the system
        if (S.hess ? !(S.rr0 > 0.0) : rr <= S.tol2 * S.rr0) S.done = 1;
        S.rz = rz;
        return;
    }
    S.it += 1;
    if (!(rz == rz) || !(rr == rr)) {
        S.status = -4;
        S.done = 1;
    } else if (rr <= S.tol2 * S.rr0) {
        S.status = 0;
        S.done = 1;
    } else if (S.it >= S.max_it) {
        S.status = 1;
        S.done = 1;
    } else {
        S.b = rz / S.rz;
        S.rz = rz;
    }
}

// The step, from the sums of `apply`.
__device__ __forceinline__ void lin_upd(LinS& S, const double* t) {
    if (S.done) return;
    S.update = S.init ? 0 : 1;
    if (S.init) {
        S.init = 0;
        S.first = 1;
        return;
    }
    const double w = S.cell;
    S.c0 = S.hess ? w * t[Q_PHIQ] / S.nphi2 : 0.0;
    S.c1 = S.hess ? w * t[Q_IPHIQ] / S.nphi2 : 0.0;
    const double pq = w * (t[Q_PQ] - S.c0 * t[Q_PPHI] - S.c1 * t[Q_PIPHI]);
    if (!(pq > 0.0)) {
        S.status = pq != pq ? -4 : -1;  // -1: the operator is not positive definite
        S.done = 1;
        return;
    }
    S.a = S.rz / pq;
}

// Take the state and the rows in, run `fn` on thread 0, publish from block 0.
template <int K, int NV, class F>
__device__ __forceinline__ void lin_begin(const LinS* in, LinS* out, const Partials& P, int blk, double* red, LinS* s,
                                          const IntakeAbsorbOf<LinS, K, NV, 0u>& it, F fn) {
    __shared__ double tot[K];
    it.st.store(in, 0, s);
    it.rows.reduce(P, 0, red, tot);  // ends with a barrier: s and tot are visible
    if (threadIdx.x == 0) {
        double t[K];
#pragma unroll
        for (int k = 0; k < K; ++k) t[k] = tot[k];
        fn(*s, t);
    }
    __syncthreads();
    state_publish(out, 0, blk, s);
}

constexpr int kLinRows = 16;  // rows per thread held in registers

// q's pointwise part beyond V p, and the sums of `apply` at one point.
template <typename T>
__device__ __forceinline__ C2<T> lin_apply_point(const LinS& s, C2<T> o, C2<T> p, C2<T> ph, double* acc) {
    const T w = s.hess ? (T)s.beta * abs2(ph) - (T)s.lam : (T)s.shift + (T)s.beta * abs2(ph);
    o = add(o, scl(p, w));
    if (s.hess) {
        o = add(o, scl(ph, (T)2 * (T)s.beta * redot(ph, p)));
        acc[Q_PHIQ] += (double)redot(ph, o);
        acc[Q_IPHIQ] += (double)imdot(ph, o);
        acc[Q_PPHI] += (double)redot(p, ph);
        acc[Q_PIPHI] += (double)imdot(ph, p);
    }
    acc[Q_PQ] += (double)redot(p, o);
    return o;
}

// The sums of `post` at one point.
template <typename T>
__device__ __forceinline__ void lin_post_sums(const LinS& s, C2<T> r, C2<T> z, C2<T> ph, double* acc) {
    acc[Z_RR] += (double)abs2(r);
    acc[Z_RZ] += (double)redot(r, z);
    if (s.hess) {
        acc[Z_RPHI] += (double)redot(ph, r);
        acc[Z_RIPHI] += (double)imdot(ph, r);
        acc[Z_PHIZ] += (double)redot(ph, z);
        acc[Z_IPHIZ] += (double)imdot(ph, z);
    }
}

// ---------------------------------------------------------------------------------------------
// dir (FIRST, x) and apply (LAST): the passes of q = A p.  1-D does both in one.
// ---------------------------------------------------------------------------------------------
template <typename T, int AX, bool FIRST, bool LAST>
struct OpLinApply {
    using ScalarState = LinS;
    static constexpr bool FWD = true, INV = true, SCALARS = true, PREFETCH = true, WIDE = true;
    static constexpr int K = LAST ? Q_K : 0;
    static constexpr int KA = K > 0 ? K : 1;
    static constexpr unsigned MAXMASK = 0;
    LinFields<T> f;
    const LinS* Sin;  // FIRST: S_upd; otherwise S_dir
    LinS* Sout;       // FIRST: S_dir
    Partials rows;    // FIRST: the sums of `post`
    using Intake = std::conditional_t<FIRST, IntakeAbsorbOf<LinS, Z_K, kLinRows, 0u>, IntakeStateOf<LinS>>;
    __device__ void intake(int, int, Intake& it) const {
        it.st.issue(Sin, 0);
        if constexpr (FIRST) it.rows.issue(rows, 0);
    }
    struct State {
        C2<T> p[8];
        C2<T> ph[8];             // phi
        C2<T> z[FIRST ? 8 : 1];  // z
        C2<T> w[FIRST ? 1 : 8];  // the parts of L p so far
        T V[FIRST ? 8 : 1];
    };
    __device__ void prefetch(const Geo&, const LineCtx& lc, State& st) const {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int64_t i = lc.at(q);
            st.p[q] = f.p[i];
            if constexpr (FIRST) {
                st.z[q] = f.z[i];
                st.ph[q] = f.phi[i];
            }
        }
    }
    __device__ void prefetch_tail(const Geo&, const LineCtx& lc, State& st) const {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int64_t i = lc.at(q);
            if constexpr (FIRST) st.V[q] = f.V[i];
            if constexpr (!FIRST) {
                st.w[q] = f.w[i];
                st.ph[q] = f.phi[i];
            }
        }
    }
    __device__ void begin(const Geo&, int, int blk, double* red, LinS* s, Intake& it) const {
        if constexpr (FIRST)
            lin_begin(Sin, Sout, rows, blk, red, s, it, [](LinS& S, const double* t) { lin_dir(S, t); });
        else
            state_copy(Sin, 0, s, it.st);
    }
    __device__ void load(const Geo&, const LineCtx& lc, State& st, C2<T> (&v)[8], double (&)[KA]) const {
        if constexpr (FIRST) {
            const LinS& s = *lc.ls;
            const T d0 = (T)s.d0, d1 = (T)s.d1, b = (T)s.b;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                C2<T> p = s.hess ? without_phi(st.z[q], st.ph[q], d0, d1) : st.z[q];
                if (s.b != 0.0) p = add(p, scl(st.p[q], b));  // the first p is not read
                st.p[q] = p;
                f.p[lc.at(q)] = p;
            }
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = st.p[q];
    }
    template <int LG>
    __device__ void spectral(const Geo& g, const LineCtx& lc, State&, C2<T> (&v)[8], double (&)[KA], C2<T>*,
                             const C2<T>*) const {
        const double rot = rot_coef<AX>(g, lc, lc.ls->omega);
        const double inv = 1.0 / lc.M;  // 1/M (exact for M = 2^k)
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const double xi = freq_of(lc.k(q), lc.M, g.dk[AX]);
            v[q] = scl(v[q], (T)((0.5 * xi * xi + rot * xi) * inv));
        }
    }
    __device__ void store(const Geo&, const LineCtx& lc, State& st, C2<T> (&v)[8], double (&acc)[KA]) const {
        const LinS& s = *lc.ls;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            C2<T> o = v[q];
            if constexpr (FIRST) o = add(o, scl(st.p[q], st.V[q]));
            if constexpr (!FIRST) o = add(o, st.w[q]);
            if constexpr (LAST)
                f.q[lc.at(q)] = lin_apply_point(s, o, st.p[q], st.ph[q], acc);
            else
                f.w[lc.at(q)] = o;
        }
    }
};

// ---------------------------------------------------------------------------------------------
// upd (x): the step, then the preconditioner's prologue and forward x; with ONE (1-D) also its
// multiplier, inverse and epilogue, and the sums of `post`.
// ---------------------------------------------------------------------------------------------
template <typename T, bool ONE>
struct OpLinUpd {
    using ScalarState = LinS;
    static constexpr bool FWD = true, INV = ONE, SCALARS = true, PREFETCH = true, WIDE = true;
    static constexpr int K = ONE ? Z_K : 0;
    static constexpr int KA = K > 0 ? K : 1;
    static constexpr unsigned MAXMASK = 0;
    LinFields<T> f;
    const LinS* Sin;  // S_dir
    LinS* Sout;       // S_upd
    Partials rows;    // the sums of `apply`
    int scaled;       // P_V^{1/2} on both sides
    using Intake = IntakeAbsorbOf<LinS, Q_K, kLinRows, 0u>;
    __device__ void intake(int, int, Intake& it) const {
        it.st.issue(Sin, 0);
        it.rows.issue(rows, 0);
    }
    struct State {
        C2<T> x[8], r[8], p[8], q[8], ph[8];
        T V[8];
    };
    __device__ void prefetch(const Geo&, const LineCtx& lc, State& st) const {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int64_t i = lc.at(k);
            st.x[k] = f.x[i];
            st.r[k] = f.r[i];
            st.p[k] = f.p[i];
            st.q[k] = f.q[i];
            st.ph[k] = f.phi[i];
            st.V[k] = f.V[i];
        }
    }
    __device__ void prefetch_tail(const Geo&, const LineCtx&, State&) const {}
    __device__ void begin(const Geo&, int, int blk, double* red, LinS* s, Intake& it) const {
        lin_begin(Sin, Sout, rows, blk, red, s, it, [](LinS& S, const double* t) { lin_upd(S, t); });
    }
    __device__ void load(const Geo&, const LineCtx& lc, State& st, C2<T> (&v)[8], double (&)[KA]) const {
        const LinS& s = *lc.ls;
        const T a = (T)s.a, c0 = (T)s.c0, c1 = (T)s.c1;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int64_t i = lc.at(k);
            if (s.update) {
                const C2<T> q = s.hess ? without_phi(st.q[k], st.ph[k], c0, c1) : st.q[k];
                f.x[i] = add(st.x[k], scl(st.p[k], a));
                st.r[k] = sub(st.r[k], scl(q, a));
                f.r[i] = st.r[k];
            }
            v[k] = scaled ? scl(st.r[k], pv_scale<T>(1, s.alpha, st.V[k], abs2(st.ph[k]), s.beta)) : st.r[k];
        }
    }
    template <int LG>
    __device__ void spectral(const Geo& g, const LineCtx& lc, State&, C2<T> (&v)[8], double (&)[KA], C2<T>*,
                             const C2<T>*) const {
        if constexpr (ONE) {
            const double invN = 1.0 / lc.M;  // 1/M (exact for M = 2^k)
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const double xi = freq_of(lc.k(k), lc.M, g.dk[0]);
                v[k] = scl(v[k], (T)(invN / (lc.ls->alpha + 0.5 * xi * xi)));
            }
        }
    }
    __device__ void store(const Geo&, const LineCtx& lc, State& st, C2<T> (&v)[8], double (&acc)[KA]) const {
        if constexpr (!ONE) {
#pragma unroll
            for (int k = 0; k < 8; ++k) f.w[lc.at(k)] = v[k];
        } else {
            const LinS& s = *lc.ls;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                C2<T> z = v[k];
                if (scaled) z = scl(z, pv_scale<T>(1, s.alpha, st.V[k], abs2(st.ph[k]), s.beta));
                f.z[lc.at(k)] = z;
                lin_post_sums(s, st.r[k], z, st.ph[k], acc);
            }
        }
    }
};

// ---------------------------------------------------------------------------------------------
// post (x): inverse x, epilogue -> z, and its sums.
// ---------------------------------------------------------------------------------------------
template <typename T>
struct OpLinPost {
    using ScalarState = LinS;
    static constexpr bool FWD = false, INV = true, SCALARS = true, PREFETCH = true, WIDE = true;
    static constexpr int K = Z_K;
    static constexpr unsigned MAXMASK = 0;
    LinFields<T> f;
    const LinS* Sin;  // S_upd
    int scaled;
    using Intake = IntakeStateOf<LinS>;
    __device__ void intake(int, int, Intake& it) const { it.st.issue(Sin, 0); }
    struct State {
        C2<T> w[8], r[8], ph[8];
        T V[8];
    };
    __device__ void prefetch(const Geo&, const LineCtx& lc, State& st) const {
#pragma unroll
        for (int k = 0; k < 8; ++k) st.w[k] = f.w[lc.at(k)];
    }
    __device__ void prefetch_tail(const Geo&, const LineCtx& lc, State& st) const {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int64_t i = lc.at(k);
            st.r[k] = f.r[i];
            st.ph[k] = f.phi[i];
            st.V[k] = f.V[i];
        }
    }
    __device__ void begin(const Geo&, int, int, double*, LinS* s, Intake& it) const { state_copy(Sin, 0, s, it.st); }
    __device__ void load(const Geo&, const LineCtx&, State& st, C2<T> (&v)[8], double (&)[K]) const {
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = st.w[k];
    }
    template <int LG>
    __device__ void spectral(const Geo&, const LineCtx&, State&, C2<T> (&)[8], double (&)[K], C2<T>*,
                             const C2<T>*) const {}
    __device__ void store(const Geo&, const LineCtx& lc, State& st, C2<T> (&v)[8], double (&acc)[K]) const {
        const LinS& s = *lc.ls;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            C2<T> z = v[k];
            if (scaled) z = scl(z, pv_scale<T>(1, s.alpha, st.V[k], abs2(st.ph[k]), s.beta));
            f.z[lc.at(k)] = z;
            lin_post_sums(s, st.r[k], z, st.ph[k], acc);
        }
    }
};

// upd and post for the diagonal preconditioners (identity, P_V): one pointwise sweep.
template <typename T>
__global__ __launch_bounds__(256) void k_lin_upd_diag(LinFields<T> f, const LinS* Sin, LinS* Sout, int64_t N, int pv,
                                                     Partials rows, double* out) {
    __shared__ double red[(256 / 64 + 1) * 16 + 4];
    __shared__ LinS s;
    IntakeAbsorbOf<LinS, Q_K, kLinRows, 0u> it;
    it.st.issue(Sin, 0);
    it.rows.issue(rows, 0);
    lin_begin(Sin, Sout, rows, (int)blockIdx.x, red, &s, it, [](LinS& S, const double* t) { lin_upd(S, t); });
    if (s.done) return;
    const T a = (T)s.a, c0 = (T)s.c0, c1 = (T)s.c1;
    double acc[Z_K] = {};
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (int64_t)gridDim.x * blockDim.x) {
        const C2<T> ph = f.phi[i];
        C2<T> r = f.r[i];
        const T V = f.V[i];
        if (s.update) {
            const C2<T> q0 = f.q[i], p = f.p[i], x = f.x[i];
            const C2<T> q = s.hess ? without_phi(q0, ph, c0, c1) : q0;
            f.x[i] = add(x, scl(p, a));
            r = sub(r, scl(q, a));
            f.r[i] = r;
        }
        const C2<T> z = pv ? scl(r, pv_scale<T>(2, s.alpha, V, abs2(ph), s.beta)) : r;
        f.z[i] = z;
        lin_post_sums(s, r, z, ph, acc);
    }
    double* P = out + (size_t)blockIdx.x * Z_K;
    block_reduce_to<Z_K, 0u>(acc, red, [P](int k, double t) { P[k] = t; });
}

// The state after the sums pending at the end of a chunk (what `dir` will find), for the host's poll.
static __global__ __launch_bounds__(256) void k_lin_test(const LinS* Sin, LinS* Sout, Partials rows) {
    __shared__ double red[(256 / 64 + 1) * 16 + 4];
    __shared__ LinS s;
    IntakeAbsorbOf<LinS, Z_K, kLinRows, 0u> it;
    it.st.issue(Sin, 0);
    it.rows.issue(rows, 0);
    lin_begin(Sin, Sout, rows, 0, red, &s, it, [](LinS& S, const double* t) { lin_dir(S, t); });
}

// The linear CG of one field: fields, device state and row regions.
template <typename T>
struct LinCtx {
    const Geo* g;
    const Twiddles* tw;
    LinFields<T> f;
    double omega;
    int kind;         // gpe_precond_t: none, kinetic, potential or combined
    LinS* S;          // two slots: S_dir, S_upd
    double* rows;     // lin_rows_doubles(g)
    hipStream_t s;
};

// Doubles of the row regions: `apply` and `post`, each with its collapse.
inline size_t lin_region_doubles(const Geo& g) {
    int64_t nb = 512;
    for (int a = 0; a < g.dim; ++a) nb = std::max<int64_t>(nb, lines_per_field(g, a));
    return (size_t)nb * Z_K;
}
inline size_t lin_rows_doubles(const Geo& g) { return 4 * lin_region_doubles(g); }

// Solves from f.x with the residual in f.r: the state `h` (parameters, tolerances; init and counters are
// set here) goes to the device, chunks of check_every iterations are queued and polled, and h returns
// the final state.
template <typename T>
hipError_t lin_solve(LinCtx<T>& c, LinS& h, int check_every);
extern template hipError_t lin_solve<double>(LinCtx<double>&, LinS&, int);
extern template hipError_t lin_solve<float>(LinCtx<float>&, LinS&, int);

}  // namespace gpe
