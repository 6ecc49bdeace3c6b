// One-dimensional problems: whole PCG iterations in one workgroup per instance.
//
// A 1-D field is one line of at most 1024 points, so an instance's state (phi, L phi, r, p, L phat, V) fits
// the registers of the line's M/8 threads, and every sum of an iteration is a workgroup reduction.  The
// kernel runs `iters` iterations (Algorithm 2: the step, residual and convergence test, preconditioner,
// direction, L phat and the line-search sums, as in pcg_passes.hpp, with the same scalar logic) and
// touches global memory only when it starts and ends.  What bounds an iteration is the chain of one or two
// waves: as two launches, with the state's trips through memory and two row reductions, it took 25 us at
// 256 points in FP64; the solve of that line to 1e-10 (57 iterations) went from 1673 us to 596.
//
// Element by element the arithmetic is that of the two launches: which product of a sum is rounded and which
// fused is written out wherever the compiler chose otherwise in this kernel than in those, so that FP32 solves
// return the same bits (the transform of the scaled residual starts in the block that scales it, as there, hence
// the compile-time SPECTRAL).
#include "pcg_passes.hpp"

namespace gpe {

// The line transform for a compile-time size (LG, see ct_points), else the run-time one.
template <typename T, int DIR, int LG, bool FIXED = false>
__device__ __forceinline__ void line_fft1(C2<T> (&v)[8], C2<T>* buf, const C2<T>* tw, int t, int lg, int M, bool wave) {
    if constexpr (LG > 0)
        fft_line_ct<T, DIR, ct_lg(LG), !ct_f5(LG) && ct_lg(LG) <= 9, ct_f5(LG), 0, FIXED, true>(v, buf, tw, t);
    else
        fft_line<T, DIR>(v, buf, tw, t, lg, M, wave);
}

// Threads of the workgroup: whole waves (partial ones reduce slowly), except for lines of 5 * 2^k points,
// which take exactly M/8.  Threads beyond the line's M/8 hold further lines of zeros, with LDS slots of
// their own: they run the same transforms and add nothing to the sums.
inline int line_threads(const Geo& g) { return g.f5[0] ? g.n[0] / 8 : std::max(64, g.n[0] / 8); }
inline size_t line_lds(const Geo& g, size_t point) {
    const int lines = line_threads(g) / (g.n[0] / 8);
    return point * ((size_t)g.n[0] + (size_t)lines * line_stride(g.n[0])) + 16;
}

template <typename T, int LG, bool SPECTRAL>
__global__ __launch_bounds__(128) void k_pcg_line(IterFields<T> f, Geo g, const C2<T>* __restrict__ twg, Scal* S,
                                                 double* rows, int row_stride, int iters, int pre,
                                                 int post) {
    extern __shared__ double4 smem_raw[];
    __shared__ double red[(128 / 64 + 1) * 16 + 4];
    __shared__ double tot_a[A_K], tot_b[B_K];
    __shared__ Scal s_local;
    Scal& s = s_local;
    const int lg = LG > 0 ? ct_lg(LG) : g.lg[0], M = LG > 0 ? ct_points(LG) : g.n[0], TPL = M >> 3;
    const int b = g.imap ? g.imap[blockIdx.x] : g.b0 + (int)blockIdx.x;
    C2<T>* tw = reinterpret_cast<C2<T>*>(smem_raw);
    const int c = threadIdx.x / TPL, t = threadIdx.x - c * TPL;
    C2<T>* buf = tw + M + (size_t)c * line_stride(M);
    const bool on = c == 0;
    const bool wave = blockDim.x <= 64;
    const int64_t base = (int64_t)b * g.N;
    double* row = rows + (size_t)b * row_stride;

    StateChunk ch;
    ch.issue(S, b);
    for (int k = threadIdx.x; k < B_K; k += blockDim.x) tot_b[k] = row[k];
    const C2<T> zero = mk((T)0, (T)0);
    C2<T> ph[8], lph[8], rp[8], pp[8], lp[8];
    T V[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int64_t i = base + t + q * TPL;
        ph[q] = on ? f.phi[i] : zero;
        lph[q] = on ? f.Lphi[i] : zero;
        rp[q] = on ? f.rp[i] : zero;
        pp[q] = on ? f.pp[i] : zero;
        lp[q] = on ? f.lp[i] : zero;
        V[q] = on ? f.V[i] : (T)0;
    }
    for (int i = threadIdx.x; i < M; i += blockDim.x) tw[i] = twg[i];
    state_copy(S, b, &s, ch);  // ends with a barrier: the tables and totals are visible too

    for (int it = 0; it < iters; ++it) {
        int kb = -1;
        if (s.line_search == 2 && !s.done && s.b_phase && blockDim.x >= 64 && threadIdx.x < 64) kb = full_scan_wave(s, tot_b);
        finish<B_K>(&s, tot_b, 0, [kb](Scal& S1, const double* tt) {
            if (!S1.done && S1.b_phase) {
                fin_step(S1, tt, kb);
                S1.b_phase = 0;
            }
        });
        if (s.done) break;
        C2<T> v[8], r[8];
        double d[8], acc[A_K];
#pragma unroll
        for (int k = 0; k < A_K; ++k) acc[k] = 0.0;
        {
            const T lam = (T)s.lam, beta = (T)s.beta;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                if (s.has_step) {
                    const C2<T> np = add(scl(ph[q], (T)s.c_phi), scl(pp[q], (T)s.c_p));
                    lph[q] = add(scl(lph[q], (T)s.c_L), scl(lp[q], (T)s.c_Lp));
                    acc[A_DPHI] = fmax(acc[A_DPHI], (double)abs2(sub(np, ph[q])));
                    ph[q] = np;
                }
                const T rho = FixedDots<LG == 0>::phi2(ph[q]);
                const double r2 = rho;
                acc[A_A] += (double)redot_fixed<false>(ph[q], lph[q]);
                acc[A_Q4] += r2 * r2;
                acc[A_N2] += r2;
                r[q] = add(lph[q], scl(ph[q], beta * rho - lam));
                res_sums<T>(acc, r[q]);
                d[q] = on ? pv_diag(s, (double)V[q], (double)rho) : 1.0;
                v[q] = scl(r[q], pscale<T>(pre, d[q]));
            }
        }
        if constexpr (SPECTRAL) {
            line_fft1<T, -1, LG>(v, buf, tw, t, lg, M, wave);
            const double invN = 1.0 / M;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const double k = freq_of(t + q * TPL, M, s.dk[0]);
                v[q] = scl(v[q], (T)(invN / (s.lamt + 0.5 * k * k)));
            }
            line_fft1<T, +1, LG, true>(v, buf, tw, t, lg, M, wave);
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            v[q] = on ? scl(v[q], pscale<T>(post, d[q])) : zero;  // P r
            cg_sums<T, 0, FixedDots<LG == 0>>(acc, r[q], v[q], rp[q], pp[q], ph[q]);
        }
        block_reduce<A_K, A_MAXMASK>(acc, red, tot_a);
        finish<A_K>(&s, tot_a, 0, [](Scal& S1, const double* tt) {
            if (!S1.done) fin_residual(S1, tt);
            if (!S1.done) {
                fin_direction(S1, tt);
                if (!S1.done) S1.b_phase = 1;
            }
        });
#pragma unroll
        for (int q = 0; q < 8; ++q) rp[q] = r[q];
        if (s.done) break;
        const T inv = (T)(1.0 / s.pnorm), bcg = (T)s.beta_cg, rho0 = (T)s.rho;
        C2<T> u[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            pp[q] = sub(scl(pp[q], bcg), add(v[q], scl(ph[q], rho0)));
            u[q] = v[q] = scl(pp[q], inv);
        }
        line_fft1<T, -1, LG>(v, buf, tw, t, lg, M, wave);
        const double invM = 1.0 / M;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const double xi = freq_of(t + q * TPL, M, s.dk[0]);
            v[q] = scl(v[q], (T)((0.5 * xi * xi) * invM));
        }
        line_fft1<T, +1, LG>(v, buf, tw, t, lg, M, wave);
        double bs[B_K];
#pragma unroll
        for (int k = 0; k < B_K; ++k) bs[k] = 0.0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const C2<T> o = on ? add(v[q], scl(u[q], V[q])) : zero;
            lp[q] = o;
            linesearch_sums<T, 0, FixedDots<LG == 0>>(bs, ph[q], u[q], o);
        }
        block_reduce<B_K, B_MAXMASK>(bs, red, tot_b);
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int64_t i = base + t + q * TPL;
        if (on) {
            f.phi[i] = ph[q];
            f.Lphi[i] = lph[q];
            f.rp[i] = rp[q];
            f.pp[i] = pp[q];
            f.lp[i] = lp[q];
        }
    }
    for (int k = threadIdx.x; k < B_K; k += blockDim.x) row[k] = tot_b[k];
    state_publish(S, b, 0, &s);
}

template <typename T>
hipError_t enqueue_line(const IterCtx<T>& c, int iters, hipStream_t s) {
    const Geo& g = c.g;
    int pre = 0, post = 0;
    const bool spectral = c.precond != GPE_P_NONE && c.precond != GPE_P_POTENTIAL;
    if (c.precond == GPE_P_COMBINED) pre = post = 1;
    if (c.precond == GPE_P_C1) post = 2;
    if (c.precond == GPE_P_C2 || c.precond == GPE_P_POTENTIAL) pre = 2;
    const int Bl = g.bl > 0 ? g.bl : c.B;
    const LaunchEvents* ev =
        c.timer ? c.timer->next("pcg_iteration_x", 21.0 * (double)sizeof(T) * (double)g.N * (double)c.B) : nullptr;
    // compile-time transforms at the sizes where the passes have them (640 points, 24 FP32 iterations with the
    // combined preconditioner: 740 us with the run-time one, 628)
    using K = decltype(&k_pcg_line<T, 0, true>);
    const K variants[2][6] = {
        {k_pcg_line<T, 0, false>, k_pcg_line<T, 6, false>, k_pcg_line<T, 7, false>, k_pcg_line<T, 8, false>,
         k_pcg_line<T, 9, false>, k_pcg_line<T, 107, false>},
        {k_pcg_line<T, 0, true>, k_pcg_line<T, 6, true>, k_pcg_line<T, 7, true>, k_pcg_line<T, 8, true>,
         k_pcg_line<T, 9, true>, k_pcg_line<T, 107, true>}};
    const int lg = g.lg[0];
    const K kern = variants[spectral ? 1 : 0][g.f5[0] ? (lg == 7 ? 5 : 0) : lg >= 6 && lg <= 9 ? lg - 5 : 0];
    launch_timed(ev, kern, dim3((unsigned)Bl), dim3((unsigned)line_threads(g)), line_lds(g, sizeof(C2<T>)), s, c.f, g,
                 (const C2<T>*)c.tw->get(0, sizeof(T) == 8), c.S + c.B,
                 c.parts + (size_t)R_B * c.region_doubles, (int)B_K, iters, pre, post);
    return hipGetLastError();
}

template hipError_t enqueue_line<double>(const IterCtx<double>&, int, hipStream_t);
template hipError_t enqueue_line<float>(const IterCtx<float>&, int, hipStream_t);

}  // namespace gpe
