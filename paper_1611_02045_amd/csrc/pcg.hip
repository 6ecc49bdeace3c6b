// Host side of one PCG iteration (its passes: pcg_passes.hpp), the pointwise first pass of the diagonal
// preconditioners, and the collapse of partial rows.
#include "pcg_passes.hpp"

namespace gpe {

GPE_PCG_X_PASSES(GPE_LAUNCH_EXTERN, double)
GPE_PCG_YZ_PASSES(GPE_LAUNCH_EXTERN, double)
GPE_PCG_X_PASSES(GPE_LAUNCH_EXTERN, float)
GPE_PCG_YZ_PASSES(GPE_LAUNCH_EXTERN, float)

// ---------------------------------------------------------------------------------------------
// Diagonal preconditioners (identity, P_V): [step], the pending retraction, residual, P r and all
// phase-A sums in one pointwise sweep (fixed chunks per block: deterministic partials).
// ---------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void k_resid_diag(IterFields<T> f, const Scal* Sin, Scal* Sout, int64_t N, int nbpi,
                                                   int pre, Partials pb, Partials pr, int b0, const int* imap) {
    __shared__ double red[(256 / 64 + 1) * 16 + 8];
    __shared__ Scal s;
    const int bi = blockIdx.x / nbpi;  // instance within the launch
    const int b = imap ? imap[bi] : b0 + bi;
    const int blk = blockIdx.x - bi * nbpi;
    IntakeStep it;
    intake_step(Sin, pb, b, it);
    begin_step(Sin, Sout, pb, b, blk, red, &s, it);
    if (s.done) return;
    double acc[A_K];
#pragma unroll
    for (int k = 0; k < A_K; ++k) acc[k] = 0.0;
    const T lam = (T)s.lam, beta = (T)s.beta;
    const int64_t chunk = (N + nbpi - 1) / nbpi;
    const int64_t lo = (int64_t)blk * chunk, hi = min(N, lo + chunk);
    const int64_t off = (int64_t)b * N;
    for (int64_t j = lo + threadIdx.x; j < hi; j += blockDim.x) {
        const int64_t i = off + j;
        C2<T> ph = f.phi[i];
        C2<T> lph = f.Lphi[i];
        apply_step<T>(f, s, i, ph, lph, acc);
        const T rho = abs2(ph);
        const C2<T> r = add(lph, scl(ph, beta * rho - lam));
        f.r[i] = r;
        const C2<T> prv = scl(r, pscale<T>(pre, pv_diag(s, (double)f.V[i], (double)rho)));
        f.pr[i] = prv;
        res_sums<T>(acc, r);
        cg_sums<T>(acc, r, prv, f.rp[i], f.pp[i], ph);
    }
    double* P = pr.parts + ((size_t)b * pr.row_stride() + pr.off + blk) * A_K;
    block_reduce_to<A_K, A_MAXMASK>(acc, red, [P](int k, double t) { P[k] = t; });
}

// ---------------------------------------------------------------------------------------------
// Host: enqueue one iteration for B instances (2-D and 3-D; 1-D: pcg_line.hip).
// ---------------------------------------------------------------------------------------------
template <typename T>
hipError_t enqueue_iteration(const IterCtx<T>& c, hipStream_t s) {
    const Geo& g = c.g;
    const bool f64 = sizeof(T) == 8;
    const int cb = (int)sizeof(C2<T>);
    const IterFields<T>& f = c.f;
    Scal* S_step = c.S;
    Scal* S_dir = c.S + c.B;
    // launched instances: [g.b0, g.b0 + Bl), or g.imap[0 .. Bl) (converged instances are not launched)
    const int Bl = g.bl > 0 ? g.bl : c.B;
    hipError_t e;
    // the view a consumer absorbs: the region itself, or its collapse into a row per kCollapseRows
    auto consumable = [&](const Partials& p, int rc, int K) -> Partials {
        double* const to = c.parts + (size_t)rc * c.region_doubles;
        return K == A_K ? absorbable<A_K, A_MAXMASK>(p, to, c.B, Bl, g, s)
                        : absorbable<B_K, B_MAXMASK>(p, to, c.B, Bl, g, s);
    };
    const Partials none{nullptr, 0, 0, 0};
    // algorithmic bytes of a launch: `reals` real numbers of sizeof(T) per grid point and instance
    const double unit = (double)sizeof(T) * (double)g.N * (double)c.B;
    auto tick = [&](const char* name, double reals) -> const LaunchEvents* {
        return c.timer ? c.timer->next(name, reals * unit) : nullptr;
    };
    // The direction passes (x, y, z) share one region of B-sum rows, each pass at its own offset
    // within an instance's rows; the step absorbs them at the next iteration's start, through their
    // collapse when they are many.
    const int nbx = pass_blocks_per_field(g, 0, cb, c.B, true);
    const int nby = pass_blocks_per_field(g, 1, cb, c.B, true);
    const int nbz = g.dim >= 3 ? pass_blocks_per_field(g, 2, cb, c.B, true) : 0;
    const int nbB = nbx + nby + nbz;
    double* const partsB = c.parts + (size_t)R_B * c.region_doubles;
    const Partials pb0{partsB, nbx, nbB, 0}, pb1{partsB, nby, nbB, nbx}, pb2{partsB, nbz, nbB, nbx + nby};
    const Partials pbAll{partsB, nbB, nbB, 0};
    const int nbBc = (nbB + kCollapseRows - 1) / kCollapseRows;
    const Partials sb = nbB <= absorb_rows(c.B) ? pbAll : Partials{c.parts + (size_t)R_BC * c.region_doubles, nbBc, nbBc, 0};
    // ---- phase A ----
    int pre = 0, post = 0;
    const bool spectral_p = c.precond == GPE_P_KINETIC || c.precond == GPE_P_COMBINED || c.precond == GPE_P_C1 ||
                            c.precond == GPE_P_C2;
    if (c.precond == GPE_P_COMBINED) pre = post = 1;
    if (c.precond == GPE_P_C1) post = 2;
    if (c.precond == GPE_P_C2 || c.precond == GPE_P_POTENTIAL) pre = 2;
    Partials pa;  // the phase-A rows
    if (!spectral_p) {
        // diagonal P (identity or P_V): one pointwise kernel for residual, P r and every sum
        const int nbpi = c.pointwise_blocks;
        pa = Partials{c.parts + (size_t)R_A * c.region_doubles, nbpi, nbpi, 0};
        launch_timed(tick("step_resid_diag", 21), k_resid_diag<T>, dim3((unsigned)(nbpi * Bl)), dim3(256), 0, s, f,
                     S_dir, S_step, g.N, nbpi, pre, sb, pa, g.b0, g.imap);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    } else {
        pa = Partials{c.parts + (size_t)R_A * c.region_doubles, nbx, nbx, 0};
        OpResid<T> op{f, S_dir, S_step, sb, pre};
        if ((e = launch_pass<T, 0>(g, c.B, c.tw->get(0, f64), op, pa, s, tick("step_resid_fwd_x", 17))) != hipSuccess)
            return e;
        if (g.dim == 2) {
            OpPMid<T, 1, true, true> y{f.w, S_step};
            if ((e = launch_pass<T, 1>(g, c.B, c.tw->get(1, f64), y, none, s, tick("precond_y", 4))) != hipSuccess)
                return e;
        } else {
            OpPMid<T, 1, true, false> y1{f.w, S_step};
            if ((e = launch_pass<T, 1>(g, c.B, c.tw->get(1, f64), y1, none, s, tick("precond_fwd_y", 4))) != hipSuccess)
                return e;
            OpPMid<T, 2, true, true> z{f.w, S_step};
            if ((e = launch_pass<T, 2>(g, c.B, c.tw->get(2, f64), z, none, s, tick("precond_z", 4))) != hipSuccess)
                return e;
            OpPMid<T, 1, false, true> y2{f.w, S_step};
            if ((e = launch_pass<T, 1>(g, c.B, c.tw->get(1, f64), y2, none, s, tick("precond_inv_y", 4))) != hipSuccess)
                return e;
        }
        OpPLast<T> op3{f, S_step, post};
        if ((e = launch_pass<T, 0>(g, c.B, c.tw->get(0, f64), op3, pa, s, tick("precond_inv_x", 13))) != hipSuccess)
            return e;
    }
    const Partials pdir = consumable(pa, R_AC, A_K);
    // ---- phase B ----
    // Whether 256-thread workgroups of a pass over half of the batch would be one per CU or fewer.  Such launches
    // have the form for few workgroups, which rounds the x product of <phat, L phat> and <phi, L phat> where the others
    // round the y product; the 320-thread form, which has both kinds, rounds as they did.
    auto few_blocks = [&](int ax) {
        const int64_t half = c.B - c.B / 2;
        return lines_per_field(g, ax) / pass_lines_rule(g, ax, cb, (int)half, false) * half <= device_cus();
    };
    if (g.dim == 2) {
        OpLp<T, 0, true, false> ox{f, S_step, S_dir, pdir};
        if ((e = launch_pass<T, 0>(g, c.B, c.tw->get(0, f64), ox, pb0, s,
                tick("test_dir_Lp_x", 11))) != hipSuccess)
            return e;
        OpLp<T, 1, false, true> oy{f, S_dir, nullptr, none, few_blocks(1)};
        if ((e = launch_pass<T, 1>(g, c.B, c.tw->get(1, f64), oy, pb1, s,
                tick("Lp_y_linesearch", 8))) != hipSuccess)
            return e;
    } else {
        OpLp<T, 0, true, false> ox{f, S_step, S_dir, pdir};
        if ((e = launch_pass<T, 0>(g, c.B, c.tw->get(0, f64), ox, pb0, s,
                tick("test_dir_Lp_x", 11))) != hipSuccess)
            return e;
        OpLp<T, 1, false, false> oy{f, S_dir, nullptr, none};
        if ((e = launch_pass<T, 1>(g, c.B, c.tw->get(1, f64), oy, pb1, s, tick("Lp_y", 8))) != hipSuccess) return e;
        OpLp<T, 2, false, true> oz{f, S_dir, nullptr, none, few_blocks(2)};
        if ((e = launch_pass<T, 2>(g, c.B, c.tw->get(2, f64), oz, pb2, s,
                tick("Lp_z_linesearch", 8))) != hipSuccess)
            return e;
    }
    (void)consumable(pbAll, R_BC, B_K);
    return hipGetLastError();
}

template hipError_t enqueue_iteration<double>(const IterCtx<double>&, hipStream_t);
template hipError_t enqueue_iteration<float>(const IterCtx<float>&, hipStream_t);

}  // namespace gpe
