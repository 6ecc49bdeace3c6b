// Partial rows and per-instance scalar state between the passes of the iterative solvers: how a pass
// takes them in, publishes them, and how many rows are folded ahead of their consumer.
#pragma once

#include "launch.hpp"

namespace gpe {

// ---------------------------------------------------------------------------------------------
// Scalar state of an instance (S: the PCG's Scal, the linear solvers' LinS) and the partial rows of its
// producers, as the passes take them in
// ---------------------------------------------------------------------------------------------
// The state of instance b travels as 16-byte chunks, one per thread, so that a block fetches it
// in one round trip.
template <class S>
constexpr int kStateChunks = (int)(sizeof(S) / sizeof(uint4));

// The state of instance b, fetched by the first threads (one chunk each) at the start of a pass
// and stored into LDS in begin().
template <class S>
struct StateChunkOf {
    static_assert(sizeof(S) % sizeof(uint4) == 0, "the state is copied in 16-byte chunks");
    uint4 ch;
    __device__ __forceinline__ void issue(const S* in, int b) {
        if (threadIdx.x < kStateChunks<S>) ch = reinterpret_cast<const uint4*>(in + b)[threadIdx.x];
    }
    __device__ __forceinline__ void store(const S* in, int b, S* s) const {
        uint4* dst = reinterpret_cast<uint4*>(s);
        if (threadIdx.x < kStateChunks<S>) dst[threadIdx.x] = ch;
        for (int c = threadIdx.x + blockDim.x; c < kStateChunks<S>; c += blockDim.x)  // blocks < 28 threads
            dst[c] = reinterpret_cast<const uint4*>(in + b)[c];
    }
};

// The partial rows (K <= 16 sums) of instance b in a region, fetched at the start of a pass in an
// (entry, row group) layout: thread t reads entry k = t % 16 of rows t / 16 + j G (G = blockDim / 16,
// j < NV) into registers.  reduce() folds them (and any rows beyond NV G), combines the four row
// groups of each wave by two exchanges and the waves through LDS, in a fixed order.  Blocks that
// are not whole waves fetch nothing early and reduce row by row.  Rows may be stale (a region
// whose sums are not pending), never out of bounds.
template <int K, int NV, unsigned mask>
struct RowFetch {
    static_assert(K >= 1 && K <= 16, "up to 16 sums per row");
    double v[NV];
    __device__ __forceinline__ static bool fast() { return (blockDim.x & 63u) == 0; }
    __device__ __forceinline__ void issue(const Partials& P, int b) {
        if (!fast() || !P.parts || P.nb <= 0) return;
        const int k = threadIdx.x & 15, grp = threadIdx.x >> 4, G = blockDim.x >> 4;
        const double id = ((mask >> k) & 1u) ? -1e300 : 0.0;
        const double* rows = P.parts + (size_t)b * P.row_stride() * K;
        const int kc = k < K ? k : K - 1;
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int r = grp + j * G;
            const double x = rows[(size_t)min(r, P.nb - 1) * K + kc];  // clamped: always in bounds
            v[j] = (k < K && r < P.nb) ? x : id;
        }
    }
    __device__ __forceinline__ void reduce(const Partials& P, int b, double* red, double* tot) const {
        if (!P.parts || P.nb <= 0) {
            for (int k = threadIdx.x; k < K; k += blockDim.x) tot[k] = ((mask >> k) & 1u) ? -1e300 : 0.0;
            __syncthreads();
            return;
        }
        const double* rows = P.parts + (size_t)b * P.row_stride() * K;
        if (!fast()) {
            reduce_partials<K, mask>(rows, P.nb, red, tot);
            return;
        }
        const int k = threadIdx.x & 15, grp = threadIdx.x >> 4, G = blockDim.x >> 4;
        const bool mx = (mask >> k) & 1u;
        double a = v[0];
#pragma unroll
        for (int j = 1; j < NV; ++j) a = mx ? fmax(a, v[j]) : a + v[j];
        if (k < K)
            for (int r = grp + NV * G; r < P.nb; r += G) a = mx ? fmax(a, rows[(size_t)r * K + k]) : a + rows[(size_t)r * K + k];
        double o;
        partner_pair<16>(a, o);
        a = mx ? fmax(a, o) : a + o;
        partner_pair<32>(a, o);
        a = mx ? fmax(a, o) : a + o;
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
        if (lane < 16) red[wave * 16 + lane] = a;
        __syncthreads();
        if (threadIdx.x < K) {
            double t = red[threadIdx.x];
            for (int w = 1; w < nw; ++w) t = mx ? fmax(t, red[w * 16 + threadIdx.x]) : t + red[w * 16 + threadIdx.x];
            tot[threadIdx.x] = t;
        }
        __syncthreads();
    }
};

// What a pass that only reads the state fetches early.
template <class S>
struct IntakeStateOf {
    StateChunkOf<S> st;
};
// What a pass that absorbs a region of K-sum rows fetches early (NV rows per thread in registers).
template <class S, int K, int NV, unsigned MASK>
struct IntakeAbsorbOf {
    StateChunkOf<S> st;
    RowFetch<K, NV, MASK> rows;
};

// Copy the fetched state into LDS and barrier.
template <class S>
__device__ __forceinline__ void state_copy(const S* in, int b, S* s, const StateChunkOf<S>& ch) {
    ch.store(in, b, s);
    __syncthreads();
}

// Block 0 of the instance writes the LDS state to out[b] (after a barrier that made it final).
template <class S>
__device__ __forceinline__ void state_publish(S* out, int b, int blk, const S* s) {
    if (blk != 0) return;
    const uint4* src = reinterpret_cast<const uint4*>(s);
    uint4* dst = reinterpret_cast<uint4*>(out + b);
    for (int c = threadIdx.x; c < kStateChunks<S>; c += blockDim.x) dst[c] = src[c];
}

// ---------------------------------------------------------------------------------------------
// Collapse the per-block partial rows of each instance, kCollapseRows of them into one row in each
// workgroup (fixed order), so that the consuming pass's workgroups reduce few rows.  The fold is
// bound by one trip of the rows through memory: a workgroup reads its rows 16 lanes to a row, four
// loads per thread in flight at once.  One workgroup per instance folding every row took 6.1 us for
// the 1024 rows of a 128^3 pass and 8.0 us for its 3072 direction rows, this split 4.5 and 4.6 us (a launch
// that does nothing takes about 2).
// ---------------------------------------------------------------------------------------------
constexpr int kCollapseRows = 64;
template <int K, unsigned MASK>
__global__ __launch_bounds__(256) void k_collapse(const double* parts, int nb, int stride, double* out, int split,
                                                 int b0, const int* imap) {
    __shared__ double red[(256 / 64) * 16];
    __shared__ double tot[K];
    const int bi = blockIdx.x / split, part = blockIdx.x - bi * split;
    const int b = imap ? imap[bi] : b0 + bi;
    const int first = part * kCollapseRows;
    const Partials rows{const_cast<double*>(parts) + (size_t)first * K, min(kCollapseRows, nb - first), stride, 0};
    RowFetch<K, kCollapseRows / 16, MASK> f;
    f.issue(rows, b);
    f.reduce(rows, b, red, tot);
    for (int k = threadIdx.x; k < K; k += blockDim.x) out[((size_t)b * split + part) * K + k] = tot[k];
}

// Rows per instance up to which the consumers of a batch of B absorb a region as it is.  Every workgroup
// of the consumer reads all of its instance's rows, where a collapse costs one launch of 4.5 us and its gap: a lone
// instance takes up to 512 rows (32 iterations, with collapse -> without, us: 640^2 FP64 4833 -> 4622, 1024 x
// 512 FP64 4550 -> 4190, 64^3 unchanged), more instances, whose consumers have several workgroups per CU, 256
// (eight FP64 at 640^2, 320 rows: 16250 collapsed, 16660 not).
inline int absorb_rows(int B) { return B == 1 ? 512 : 256; }

// The rows a consumer absorbs: the region itself up to absorb_rows(), else its collapse into `to` (queued
// here), a row per kCollapseRows.  B: the instances of the batch, Bl of them launched.
template <int K, unsigned MASK>
inline Partials absorbable(const Partials& p, double* to, int B, int Bl, const Geo& g,
                           hipStream_t s) {
    if (p.nb <= absorb_rows(B)) return p;
    const int split = (p.nb + kCollapseRows - 1) / kCollapseRows;
    hipLaunchKernelGGL((k_collapse<K, MASK>), dim3((unsigned)(Bl * split)), dim3(256), 0, s, p.parts, p.nb,
                       p.row_stride(), to, split, g.b0, g.imap);
    return Partials{to, split, split, 0};
}

}  // namespace gpe
