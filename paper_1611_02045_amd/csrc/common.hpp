// Shared device/host definitions of libgpe: complex arithmetic, grid geometry, per-instance
// solver scalars and the deterministic block reduction used by every reducing kernel.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gpe {

// ------------------------------------------------------------------------------------------------
// Complex numbers stored interleaved (re, im); alignment gives 8/16-byte vector loads.
// ------------------------------------------------------------------------------------------------
template <typename T>
struct alignas(2 * sizeof(T)) C2 {
    T x, y;
};

template <typename T> __host__ __device__ __forceinline__ C2<T> mk(T a, T b) { C2<T> r; r.x = a; r.y = b; return r; }
template <typename T> __host__ __device__ __forceinline__ C2<T> add(C2<T> a, C2<T> b) { return mk(a.x + b.x, a.y + b.y); }
template <typename T> __host__ __device__ __forceinline__ C2<T> sub(C2<T> a, C2<T> b) { return mk(a.x - b.x, a.y - b.y); }
template <typename T> __host__ __device__ __forceinline__ C2<T> scl(C2<T> a, T s) { return mk(a.x * s, a.y * s); }
template <typename T> __host__ __device__ __forceinline__ C2<T> mul(C2<T> a, C2<T> b) {
    return mk(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// a * conj(b)
template <typename T> __host__ __device__ __forceinline__ C2<T> mulc(C2<T> a, C2<T> b) {
    return mk(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}
template <typename T> __host__ __device__ __forceinline__ T abs2(C2<T> a) { return a.x * a.x + a.y * a.y; }
// Re(conj(a) b)
template <typename T> __host__ __device__ __forceinline__ T redot(C2<T> a, C2<T> b) { return a.x * b.x + a.y * b.y; }
// a * (i s): multiplication by a purely imaginary number
template <typename T> __host__ __device__ __forceinline__ C2<T> muli(C2<T> a, T s) { return mk(-a.y * s, a.x * s); }

// ------------------------------------------------------------------------------------------------
// Grid geometry of one problem (Section 3).
// ------------------------------------------------------------------------------------------------
struct Geo {
    int dim;
    int n[3];       // points per axis (1 for unused axes)
    int lg[3];      // log2 of the power-of-two part of n (n = 2^lg, or 5 * 2^lg when f5)
    int f5[3];      // 1 when n = 5 * 2^lg (a radix-5 stage ends the line transform)
    int pow2;       // every axis is a power of two (the line decomposition uses shifts only)
    int b0, bl;     // a launch covers instances [b0, b0 + bl) of the B laid out (bl = 0: all of them),
                    // or, when imap is set, the bl instances imap[0 .. bl) (device, each < B); tiles and
                    // partial-row strides always follow the full B
    const int* imap;
    double L[3];    // half-widths
    double h[3];    // spacings 2L/n
    double dk[3];   // frequency spacings pi/L
    double cell;    // h^d
    int64_t N;      // points per field
};

// Frequency xi of transform index j on an axis of n points and half-width L (Nyquist kept), given
// the spacing dk = pi/L.
__device__ __forceinline__ double freq_of(int j, int n, double dk) {
    int p = (j < (n >> 1)) ? j : j - n;
    return (double)p * dk;
}
// Grid coordinate x_k = -L + k h.
__device__ __forceinline__ double coord_of(int k, double L, double h) { return -L + (double)k * h; }

// ------------------------------------------------------------------------------------------------
// Per-instance solver state (FP64).  One struct per instance, resident in device memory.
// ------------------------------------------------------------------------------------------------
struct alignas(16) Scal {
    // problem parameters (per instance: batched solves mix boxes, beta and omega)
    double beta, omega, cell;
    double L[3], h[3], dk[3];  // dk = pi/L
    // scalars of the current iterate phi_n
    double a;          // <phi, L phi>, L = T + V - omega L_z (tracked field)
    double aR;         // <phi, R phi>, R = -omega L_z
    double q4;         // h^d sum |phi|^4
    double nrm2;       // ||phi||^2
    double lam;        // lambda_n
    double lamt;       // lambda~_n (preconditioner shift)
    double E;          // E(phi_n)
    double E_prev;     // E(phi_{n-1})
    double res;        // ||r_n||_inf
    double dphi;       // ||phi_n - phi_{n-1}||_inf
    // conjugate-gradient memory
    double rPr_prev;   // <r_{n-1}, P_{n-1} r_{n-1}>
    // direction (after the preconditioner reductions)
    double beta_cg, rho, pnorm, d1, d2, rPr_cur;
    double aR_next;    // <phi_{n+1}, R phi_{n+1}> predicted by the step
    int32_t restarted, dim;
    // step (after the line search)
    double theta, c_phi, c_p, c_L, c_Lp, dE;
    // counters and flags
    int64_t n, restarts, halvings, iters_fp32;
    int32_t done, status, have_prev, linesearch_fail;  // linesearch_fail: consecutive failures
    int32_t stagnant, nonfinite, b_phase, precision;   // b_phase: direction partials are pending
    // options copied per instance
    double tol_res, tol_energy, theta_default;
    int32_t method, beta_rule, max_halvings, precond;
    int64_t max_iter;
    // stagnation tracking (mixed precision)
    double best_res, best_E;
    int64_t best_n;
    double switch_res;
    int32_t stall_window, has_step;   // has_step: a retraction step is pending (applied by phase A)
    int32_t line_search, pad0;        // 0 decrease test, 1 Armijo test, 2 full line search
    // history
    double* hist;      // device ring of rows of 8 doubles, nullable
    int64_t hist_cap;
};

enum : int { ST_OK = 0, ST_NOT_CONVERGED = 1, ST_LINESEARCH = -5, ST_NONFINITE = -4 };

// ------------------------------------------------------------------------------------------------
// Deterministic block reduction of K doubles.  Entry k is summed, or max-reduced when bit k of
// MASK is set.  Inside a full wave the K entries are reduced by a transposing butterfly: at
// each of the first log2(K') exchanges (K' = K rounded up to a power of two) a lane keeps half of
// its entries and trades the other half with its partner; after log2(64 / K') plain steps
// lane l holds entry l / (64 / K') reduced over the wave, for K' - 1 + log2(64 / K') exchanges in
// total instead of 6 K.  Partners are 32 and 16 lanes apart in the first two exchanges, where the
// half-wave and row swaps trade two registers in one instruction and leave both addends in place (no
// selects), and within a row of 16 lanes (data-parallel primitives) after that: through LDS
// (ds_bpermute) an exchange of one double costs four selects, two LDS trips and their wait, and the
// reduction of 16 sums took 1.1 us of each small pass.  Blocks whose size is not a multiple of 64 take a masked xor
// tree per entry (lanes beyond the block's last thread contribute the identity).  The waves are then
// combined in a fixed order by the first K threads, which hand each total to `sink(k, total)`.
// `red` is LDS scratch of at least (blockDim/64 + 1) * K doubles; v is clobbered.  Must be called by
// every thread of the block, in uniform control flow; the sink's writes need a barrier before another
// thread reads them.
// ------------------------------------------------------------------------------------------------
struct U2 {
    unsigned x, y;
};
__device__ __forceinline__ U2 bits_of(double v) { return __builtin_bit_cast(U2, v); }
__device__ __forceinline__ double of_bits(unsigned lo, unsigned hi) { return __builtin_bit_cast(double, U2{lo, hi}); }

// Lanes of the upper half (OFF = 32: the wave's, 16: each row pair's) of `a` trade places with those of
// the lower half of `b`: afterwards a and b hold, in the lower half's lanes, a of both halves, and in the
// upper half's lanes, b of both.
template <int OFF>
__device__ __forceinline__ void swap_halves(double& a, double& b) {
    static_assert(OFF == 32 || OFF == 16, "half-wave or row swap");
    const U2 p = bits_of(a), q = bits_of(b);
    if constexpr (OFF == 32) {
        const auto lo = __builtin_amdgcn_permlane32_swap(p.x, q.x, false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap(p.y, q.y, false, false);
        a = of_bits(lo[0], hi[0]);
        b = of_bits(lo[1], hi[1]);
    } else {
        const auto lo = __builtin_amdgcn_permlane16_swap(p.x, q.x, false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(p.y, q.y, false, false);
        a = of_bits(lo[0], hi[0]);
        b = of_bits(lo[1], hi[1]);
    }
}

// The partner's value within a row of 16 lanes: lane xor 8 (rotation by 8), the mirror image within
// eight lanes (its bit 2 differs), lane xor 2, lane xor 1.
template <int OFF>
__device__ __forceinline__ double row_partner(double v) {
    static_assert(OFF == 8 || OFF == 4 || OFF == 2 || OFF == 1, "partner within a row");
    constexpr int ctrl = OFF == 8 ? 0x128 : OFF == 4 ? 0x141 : OFF == 2 ? 0x4E : 0xB1;
    const U2 p = bits_of(v);
    return of_bits((unsigned)__builtin_amdgcn_mov_dpp((int)p.x, ctrl, 0xF, 0xF, true),
                   (unsigned)__builtin_amdgcn_mov_dpp((int)p.y, ctrl, 0xF, 0xF, true));
}

// v and its partner's value at distance OFF, in an order that is the same in both lanes where the
// hardware swap gives it (OFF >= 16).
template <int OFF>
__device__ __forceinline__ void partner_pair(double& a, double& b) {
    if constexpr (OFF >= 16) {
        b = a;
        swap_halves<OFF>(a, b);
    } else {
        b = row_partner<OFF>(a);
    }
}

// Whether any / all of the entries congruent to j modulo HALF are max-reduced (bits of mask below K).
__host__ __device__ constexpr bool any_max(unsigned mask, int j, int half, int K) {
    for (int e = j; e < K; e += half)
        if ((mask >> e) & 1u) return true;
    return false;
}
__host__ __device__ constexpr bool all_max(unsigned mask, int j, int half, int K) {
    for (int e = j; e < K; e += half)
        if (!((mask >> e) & 1u)) return false;
    return true;
}

// One exchange of the transposing butterfly (HALF entries traded with the lane at distance OFF),
// then the next; template recursion keeps every register index a compile-time constant.  Entry
// base + j is in u[j]; only an index that some lane holds a max entry at pays for the choice.
template <int HALF, int OFF, int K, unsigned MASK, int KP, int J = 0>
__device__ __forceinline__ void butterfly_round(double (&u)[KP], int lane, int& base) {
    if constexpr (HALF >= 1) {
        const bool up = (lane & OFF) != 0;
        double a, b;
        if constexpr (OFF >= 16) {
            a = u[J];
            b = u[J + HALF];
            swap_halves<OFF>(a, b);
        } else {
            a = up ? u[J + HALF] : u[J];
            b = row_partner<OFF>(up ? u[J] : u[J + HALF]);
        }
        if constexpr (!any_max(MASK, J, HALF, K)) {
            u[J] = a + b;
        } else if constexpr (all_max(MASK, J, HALF, K)) {
            u[J] = fmax(a, b);
        } else {
            const bool mx = (MASK >> (base + (up ? HALF : 0) + J)) & 1u;
            u[J] = mx ? fmax(a, b) : a + b;
        }
        if constexpr (J + 1 < HALF) {
            butterfly_round<HALF, OFF, K, MASK, KP, J + 1>(u, lane, base);
        } else {
            base += up ? HALF : 0;
            butterfly_round<HALF / 2, OFF / 2, K, MASK, KP>(u, lane, base);
        }
    }
}

// The plain steps at distances OFF, OFF / 2, ..., 1.
template <int OFF, int K, unsigned MASK>
__device__ __forceinline__ void plain_steps(double& u, bool mx) {
    if constexpr (OFF >= 1) {
        double a = u, b;
        partner_pair<OFF>(a, b);
        if constexpr (!any_max(MASK, 0, 1, K)) {
            u = a + b;
        } else if constexpr (all_max(MASK, 0, 1, K)) {
            u = fmax(a, b);
        } else {
            u = mx ? fmax(a, b) : a + b;
        }
        plain_steps<OFF / 2, K, MASK>(u, mx);
    }
}

template <int K, unsigned MASK, class Sink>
__device__ __forceinline__ void block_reduce_to(double (&v)[K], double* red, Sink sink) {
    static_assert(K >= 1 && K <= 32, "block_reduce handles 1..32 entries");
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int nw = (blockDim.x + 63) >> 6;
    if ((blockDim.x & 63u) == 0) {
        constexpr int KP = K <= 1 ? 1 : K <= 2 ? 2 : K <= 4 ? 4 : K <= 8 ? 8 : K <= 16 ? 16 : 32;
        double u[KP];
#pragma unroll
        for (int k = 0; k < KP; ++k) u[k] = k < K ? v[k] : 0.0;  // padding entries are sums of zeros
        int base = 0;  // first entry index still held by this lane
        butterfly_round<KP / 2, 32, K, MASK>(u, lane, base);
        plain_steps<32 / KP, K, MASK>(u[0], (MASK >> base) & 1u);
        __syncthreads();
        if ((lane & (64 / KP - 1)) == 0 && base < K) red[wave * K + base] = u[0];
    } else {
        const int nact = min(64, (int)blockDim.x - wave * 64);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            double s = v[k];
            constexpr unsigned mask = MASK;
            const bool mx = (mask >> k) & 1u;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                double o = __shfl_xor(s, off, 64);
                if ((lane ^ off) >= nact) o = mx ? -1e300 : 0.0;
                s = mx ? fmax(s, o) : s + o;
            }
            v[k] = s;
        }
        __syncthreads();
        if (lane == 0) {
#pragma unroll
            for (int k = 0; k < K; ++k) red[wave * K + k] = v[k];
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < K; k += blockDim.x) {
        const bool mx = (MASK >> k) & 1u;
        double s = red[k];
        for (int w = 1; w < nw; ++w) {
            const double o = red[w * K + k];
            s = mx ? fmax(s, o) : s + o;
        }
        sink(k, s);
    }
}

// block_reduce_to with the totals in `out` (LDS, K doubles), visible to every thread on return.
template <int K, unsigned MASK = 0u>
__device__ __forceinline__ void block_reduce(double (&v)[K], double* red, double* out) {
    block_reduce_to<K, MASK>(v, red, [out](int k, double s) { out[k] = s; });
    __syncthreads();
}

}  // namespace gpe
