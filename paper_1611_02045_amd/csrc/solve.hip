// Host driver of the PG / PCG ground-state solver (Algorithms 1-2) and its C ABI entry points.
//
// A solve runs one or two phases.  FP64 mode: one FP64 phase to tol.  Mixed mode: an FP32 phase
// (fields and transforms in FP32, every scalar in FP64) until ||r||_inf <= switch_res, a
// stagnation of the residual, or a failed line search; then the iterate is promoted to FP64,
// L phi is recomputed from it, the CG memory is reset and an FP64 phase finishes to tol.
// Within a phase, iterations are queued in chunks of `check_every`; the host polls the
// per-instance scalars one chunk behind (kernels of a finished instance return immediately).
// Every `refresh_every` iterations L phi and its scalars are recomputed from phi, bounding the
// drift of the linearity update.  The reported E, lambda and ||r||_inf are recomputed in FP64
// from the final iterate.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "internal.hpp"
#include "launch.hpp"
#include "pcg.hpp"
#include "plan.hpp"
#include "solver.hpp"

namespace gpe {

// ---------------------------------------------------------------------------------------------
// Small kernels of the driver
// ---------------------------------------------------------------------------------------------
template <typename TI, typename TO>
__global__ void k_convert(const TI* in, TO* out, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = (TO)in[i];
}

template <typename T>
__global__ void k_zero(T* p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = (T)0;
}

// Per-instance sum of |phi|^2 over fixed chunks (deterministic partials: nbpi per instance).
template <typename T>
__global__ __launch_bounds__(256) void k_norm_partial(const C2<T>* phi, int64_t N, int nbpi, double* parts) {
    __shared__ double red[8];
    const int b = blockIdx.x / nbpi, blk = blockIdx.x - b * nbpi;
    const int64_t chunk = (N + nbpi - 1) / nbpi, lo = (int64_t)blk * chunk, hi = min(N, lo + chunk);
    double v[1] = {0.0};
    for (int64_t j = lo + threadIdx.x; j < hi; j += blockDim.x) v[0] += (double)abs2(phi[(int64_t)b * N + j]);
    __shared__ double o1[1];
    block_reduce<1>(v, red, o1);
    if (threadIdx.x == 0) parts[blockIdx.x] = o1[0];
}

// Scale instance b by 1/||phi||, each block reducing the instance's partials itself (same order).
template <typename T>
__global__ __launch_bounds__(256) void k_norm_apply(C2<T>* phi, int64_t N, int nbpi, const double* parts,
                                                    const Scal* S) {
    __shared__ double red[8];
    __shared__ double inv;
    const int b = blockIdx.x / nbpi, blk = blockIdx.x - b * nbpi;
    double v[1] = {0.0};
    for (int k = threadIdx.x; k < nbpi; k += blockDim.x) v[0] += parts[(size_t)b * nbpi + k];
    __shared__ double o1[1];
    block_reduce<1>(v, red, o1);
    if (threadIdx.x == 0) inv = 1.0 / sqrt(S[b].cell * o1[0]);
    __syncthreads();
    const int64_t chunk = (N + nbpi - 1) / nbpi, lo = (int64_t)blk * chunk, hi = min(N, lo + chunk);
    for (int64_t j = lo + threadIdx.x; j < hi; j += blockDim.x) {
        const int64_t i = (int64_t)b * N + j;
        phi[i] = scl(phi[i], (T)inv);
    }
}

// Fill the scalars of a (re)started iterate from the energy parts computed with beta = 1:
// parts = {<phi,T phi>, <phi,V phi>, 1/2 h^d sum|phi|^4, <phi,R phi>}.
__global__ void k_scal_from_parts(Scal* S, const double* parts, int restart_cg) {
    if (threadIdx.x != 0) return;
    Scal& s = *S;
    const double kin = parts[0], pot = parts[1], q4 = 2.0 * parts[2], rot = parts[3];
    s.a = kin + pot + rot;
    s.aR = rot;
    s.q4 = q4;
    s.lam = s.a + s.beta * q4;
    s.lamt = kin + pot + s.beta * q4;
    const double E = s.a + 0.5 * s.beta * q4;
    if (restart_cg) {
        s.nrm2 = 1.0;
        s.have_prev = 0;
        s.has_step = 0;
        s.E_prev = E;
        s.best_res = 1e300;
        s.best_E = 1e300;
        s.best_n = s.n;
    }
    s.E = E;
}

// Fresh FP64 check of a final iterate: lambda = Re<phi, H phi>/||phi||^2, ||H phi - lambda phi||_inf.
template <typename T>
__global__ __launch_bounds__(256) void k_verify_dot(const C2<T>* phi, const C2<T>* hphi, int64_t N, double* parts) {
    __shared__ double red[16];
    double v[2] = {0.0, 0.0};
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (int64_t)gridDim.x * blockDim.x) {
        v[0] += (double)redot(phi[i], hphi[i]);
        v[1] += (double)abs2(phi[i]);
    }
    __shared__ double o2[2];
    block_reduce<2>(v, red, o2);
    if (threadIdx.x < 2) parts[blockIdx.x * 2 + threadIdx.x] = o2[threadIdx.x];
}

template <typename T>
__global__ __launch_bounds__(256) void k_verify_res(const C2<T>* phi, const C2<T>* hphi, int64_t N, const double* dots,
                                                    int ndot, double* maxparts, double* lam_out) {
    __shared__ double red[16];
    __shared__ double lam_s;
    double v[2] = {0.0, 0.0};
    for (int k = threadIdx.x; k < ndot; k += blockDim.x) {
        v[0] += dots[2 * k];
        v[1] += dots[2 * k + 1];
    }
    __shared__ double t2[2];
    block_reduce<2>(v, red, t2);
    if (threadIdx.x == 0) {
        lam_s = t2[0] / t2[1];
        if (blockIdx.x == 0) *lam_out = lam_s;
    }
    __syncthreads();
    const double lam = lam_s;
    double m[1] = {0.0};
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (int64_t)gridDim.x * blockDim.x) {
        const C2<T> p = phi[i], h = hphi[i];
        const double rx = (double)h.x - lam * (double)p.x, ry = (double)h.y - lam * (double)p.y;
        m[0] = fmax(m[0], sqrt(rx * rx + ry * ry));
    }
    __shared__ double o1[1];
    block_reduce<1, 1u>(m, red, o1);
    if (threadIdx.x == 0) maxparts[blockIdx.x] = o1[0];
}

// Maximum of n partials (one workgroup; a single thread's loop over 256 of them took 15 us).
__global__ __launch_bounds__(256) void k_max_collect(const double* parts, int n, double* dst) {
    __shared__ double red[8];
    double m[1] = {0.0};
    for (int i = threadIdx.x; i < n; i += blockDim.x) m[0] = fmax(m[0], parts[i]);
    block_reduce_to<1, 1u>(m, red, [dst](int, double t) { *dst = t; });
}

static unsigned blocks_for(int64_t n) { return (unsigned)((n + 255) / 256); }

template <typename TI, typename TO>
static hipError_t convert(const void* in, void* out, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL((k_convert<TI, TO>), dim3(blocks_for(n)), dim3(256), 0, s, (const TI*)in, (TO*)out, n);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Workspace of one precision: 8 complex fields + V for B instances.
// ---------------------------------------------------------------------------------------------
template <typename T>
static IterFields<T> carve(DevBuf& buf, int64_t BN, hipError_t* err) {
    const size_t cf = sizeof(C2<T>) * (size_t)BN;
    const size_t need = 8 * cf + sizeof(T) * (size_t)BN + 256;
    *err = buf.ensure(need);
    IterFields<T> f{};
    if (*err != hipSuccess) return f;
    char* p = (char*)buf.ptr;
    C2<T>** slots[8] = {&f.phi, &f.Lphi, &f.r, &f.rp, &f.pp, &f.pr, &f.lp, &f.w};
    for (int k = 0; k < 8; ++k) *slots[k] = (C2<T>*)(p + k * cf);
    f.V = (T*)(p + 8 * cf);
    return f;
}

// Recompute L phi and the scalars of the current iterate (instance-wise, B = 1 per call).
template <typename T>
static hipError_t refresh_instance(const Geo& g, const Twiddles& tw, IterFields<T>& f, int64_t off, Scal* Sd,
                                   double beta, double omega, Reduce& red, bool restart_cg, hipStream_t s) {
    const bool f64 = sizeof(T) == 8;
    hipError_t e;
    // L phi into Lphi (w as the transform intermediate)
    if ((e = op_apply(g, f64, 1, tw, f.phi + off, f.V + off, f.Lphi + off, f.w + off, beta, omega, false, s)) !=
        hipSuccess)
        return e;
    // Mid-phase refreshes stop here: the scalars already describe the iterate that the pending
    // step produces, and L phi (fresh) is only combined linearly by that step.
    if (!restart_cg) return hipSuccess;
    double* parts = (double*)red.scalars.ptr + 16;
    if ((e = op_energy(g, f64, tw, f.phi + off, f.V + off, 1.0, omega, red, parts, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_scal_from_parts, dim3(1), dim3(64), 0, s, Sd, parts, 1);
    return hipGetLastError();
}

template <typename T>
static hipError_t normalize_all(IterFields<T>& f, int B, int64_t N, Scal* Sd, Reduce& red, hipStream_t s) {
    const int nbpi = (int)std::max<int64_t>(1, std::min<int64_t>(256, N / 2048));
    double* parts = (double*)red.parts.ptr;
    hipLaunchKernelGGL(k_norm_partial<T>, dim3(nbpi * B), dim3(256), 0, s, f.phi, N, nbpi, parts);
    hipLaunchKernelGGL(k_norm_apply<T>, dim3(nbpi * B), dim3(256), 0, s, f.phi, N, nbpi, parts, Sd);
    return hipGetLastError();
}

template <typename T>
static hipError_t zero_cg_memory(IterFields<T>& f, int64_t BN, hipStream_t s) {
    hipLaunchKernelGGL(k_zero<T>, dim3(blocks_for(2 * BN)), dim3(256), 0, s, (T*)f.rp, 2 * BN);
    hipLaunchKernelGGL(k_zero<T>, dim3(blocks_for(2 * BN)), dim3(256), 0, s, (T*)f.pp, 2 * BN);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// One phase for B instances of one grid.
// ---------------------------------------------------------------------------------------------
// A non-blocking stream of default priority ordered after the work queued on another stream;
// synchronised and destroyed with the object.
struct PrivateStream {
    hipStream_t s = nullptr;
    hipError_t create_after(hipStream_t other) {
        std::lock_guard<std::mutex> lock(capture_mutex());
        hipError_t e = hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
        if (e != hipSuccess) {
            s = nullptr;
            return e;
        }
        hipEvent_t ev;
        if ((e = hipEventCreateWithFlags(&ev, hipEventDisableTiming)) != hipSuccess) return e;
        e = hipEventRecord(ev, other);
        if (e == hipSuccess) e = hipStreamWaitEvent(s, ev, 0);
        (void)hipEventDestroy(ev);
        return e;
    }
    ~PrivateStream() {
        if (s) {
            (void)hipStreamSynchronize(s);
            std::lock_guard<std::mutex> lock(capture_mutex());
            (void)hipStreamDestroy(s);
        }
    }
};

// An instantiated graph captured from work queued on one stream.  Every graph call of the library
// (capture and instantiation, launch, destruction) holds capture_mutex: instantiating a graph and
// destroying its executable allocate and free the device memory that holds the graph's kernel
// arguments, which the mutex keeps out of other host threads' capture windows like every other
// allocation and free, and no two host threads run graph calls at once.  Captures only kernel
// launches: no memory-set or copy nodes.
struct GraphExec {
    hipGraphExec_t exec = nullptr;
    template <class F>
    hipError_t capture(hipStream_t s, F enqueue) {
        std::lock_guard<std::mutex> lock(capture_mutex());
        hipError_t e = hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal);
        if (e != hipSuccess) return e;
        hipError_t qe = enqueue();
        hipGraph_t g = nullptr;
        e = hipStreamEndCapture(s, &g);
        if (qe != hipSuccess || e != hipSuccess) {
            if (g) (void)hipGraphDestroy(g);
            return qe != hipSuccess ? qe : e;
        }
        e = hipGraphInstantiate(&exec, g, nullptr, nullptr, 0);
        (void)hipGraphDestroy(g);
        if (e != hipSuccess) exec = nullptr;
        return e;
    }
    hipError_t launch(hipStream_t s) {
        std::lock_guard<std::mutex> lock(capture_mutex());
        return hipGraphLaunch(exec, s);
    }
    void reset() {
        if (exec) {
            std::lock_guard<std::mutex> lock(capture_mutex());
            (void)hipGraphExecDestroy(exec);
        }
        exec = nullptr;
    }
    ~GraphExec() { reset(); }
};

// Copies the states of B instances into mapped host memory (one workgroup each).
__global__ __launch_bounds__(64) void k_poll(const Scal* S, Scal* host) {
    static_assert(sizeof(Scal) % sizeof(uint4) == 0, "copied in 16-byte chunks");
    const uint4* src = reinterpret_cast<const uint4*>(S + blockIdx.x);
    uint4* dst = reinterpret_cast<uint4*>(host + blockIdx.x);
    for (int c = threadIdx.x; c < (int)(sizeof(Scal) / sizeof(uint4)); c += 64) dst[c] = src[c];
}

// Slots of mapped host memory for the states, each with the event that tells when its copy is complete: two for
// the ends of chunks, kMarks for the quarters of the first one.  The memory is the caller's: its allocation and
// release in each solve took 40 us.
struct PollSlots {
    static constexpr int kMarks = 3, kSlots = 2 + kMarks;
    int B = 0;
    Scal *host = nullptr, *dev = nullptr;
    hipEvent_t ev[kSlots] = {};
    hipStream_t stream = nullptr;
    bool used[kSlots] = {};
    hipError_t init(HostBuf& buf, int count, hipStream_t s) {
        B = count;
        stream = s;
        hipError_t e = buf.ensure(kSlots * sizeof(Scal) * (size_t)B);
        if (e != hipSuccess) return e;
        host = (Scal*)buf.ptr;
        dev = (Scal*)buf.dev;
        std::lock_guard<std::mutex> lock(capture_mutex());
        for (int k = 0; k < kSlots && e == hipSuccess; ++k) e = hipEventCreateWithFlags(&ev[k], hipEventDisableTiming);
        return e;
    }
    hipError_t queue(const Scal* S, int slot) {
        used[slot] = true;
        hipLaunchKernelGGL(k_poll, dim3((unsigned)B), dim3(64), 0, stream, S, dev + (size_t)slot * B);
        const hipError_t e = hipGetLastError();
        return e != hipSuccess ? e : hipEventRecord(ev[slot], stream);
    }
    // whether the slot's copy is complete (an error of the device is left to wait())
    bool ready(int slot) const {
        if (!used[slot]) return false;
        const bool yes = hipEventQuery(ev[slot]) != hipErrorNotReady;
        if (!yes) (void)hipGetLastError();  // "not ready" is no error of a later launch
        return yes;
    }
    bool all_done(int slot) const {
        return std::all_of(host + (size_t)slot * B, host + (size_t)(slot + 1) * B, [](const Scal& s) { return s.done != 0; });
    }
    // whether every instance of slot b is done, or will be after as many iterations again as from slot a to b, its
    // residual falling as it did there (within a factor of ten)
    bool ending(int a, int b) const {
        for (int k = 0; k < B; ++k) {
            const Scal &p = host[(size_t)a * B + k], &q = host[(size_t)b * B + k];
            if (!q.done && !(q.res * q.res <= 10.0 * q.tol_res * p.res)) return false;
        }
        return true;
    }
    hipError_t wait(int slot, std::vector<Scal>& out) {
        const hipError_t e = hipEventSynchronize(ev[slot]);
        if (e == hipSuccess) std::copy(host + (size_t)slot * B, host + (size_t)(slot + 1) * B, out.begin());
        return e;
    }
    // queued kernels may still write the slots (and use what its owner frees after it)
    ~PollSlots() {
        if (std::any_of(used, used + kSlots, [](bool u) { return u; })) (void)hipStreamSynchronize(stream);
        std::lock_guard<std::mutex> lock(capture_mutex());
        for (hipEvent_t x : ev)
            if (x) (void)hipEventDestroy(x);
    }
};

template <typename T>
hipError_t run_phase(PhaseArgs& pa, IterFields<T> f, std::vector<Scal>& host_S, hipStream_t s_caller) {
    const Geo& g = pa.g;
    const int B = pa.B;
    const int64_t N = g.N;
    hipError_t e;
    // Graph capture is not possible on the legacy default stream (the usual caller's stream): with
    // graphs the phase runs on a private stream that first waits for the caller's queued work (or on the
    // stream of a batch's part as it is); the loop below ends with a synchronisation of that stream, so
    // nothing is left queued on it.
    // (1-D: a chunk is one launch, with nothing to capture)
    const bool want_graph = pa.use_graph && pa.check_every % 2 == 0 && g.dim > 1;
    PrivateStream own;
    hipStream_t s = s_caller;
    if (want_graph && !pa.own_stream) {
        if ((e = own.create_after(s_caller)) != hipSuccess) return e;
        s = own.s;
    }
    // scalars to the device
    // two versioned state slots (after the step; after the convergence test and the direction);
    // an iteration starts from S_dir
    Scal* S_dir = pa.S + B;
    for (int k = 0; k < 2; ++k)
        if ((e = hipMemcpyAsync(pa.S + k * B, host_S.data(), sizeof(Scal) * B, hipMemcpyHostToDevice, s)) != hipSuccess)
            return e;
    if ((e = normalize_all<T>(f, B, N, S_dir, *pa.red, s)) != hipSuccess) return e;
    if ((e = zero_cg_memory<T>(f, (int64_t)B * N, s)) != hipSuccess) return e;
    for (int b = 0; b < B; ++b) {
        Geo gb = g;
        for (int a = 0; a < 3; ++a) {
            gb.L[a] = host_S[b].L[a];
            gb.h[a] = host_S[b].h[a];
            gb.dk[a] = host_S[b].dk[a];
        }
        gb.cell = host_S[b].cell;
        if ((e = refresh_instance<T>(gb, *pa.tw, f, (int64_t)b * N, S_dir + b, host_S[b].beta, host_S[b].omega,
                                     *pa.red, true, s)) != hipSuccess)
            return e;
    }
    IterCtx<T> c;
    c.g = g;
    c.B = B;
    c.tw = pa.tw;
    c.f = f;
    c.S = pa.S;
    c.parts = (double*)pa.red->parts.ptr;
    c.region_doubles = pa.region_doubles;
    c.precond = pa.precond;
    c.pointwise_blocks = (int)std::max<int64_t>(1, std::min<int64_t>(1024, N / 1024));
    int64_t since_refresh = 0;
    int64_t queued = 0;
    int64_t max_iter = 0;
    for (int b = 0; b < B; ++b) max_iter = std::max<int64_t>(max_iter, host_S[b].max_iter);
    // A chunk of check_every iterations launches the same kernels with the same arguments every
    // time (the r / r_{n-1} roles swap each iteration, so an even chunk ends where it started): the
    // first chunk runs eagerly, is captured into a graph while the device works on it, and every later
    // chunk replays that.
    GraphExec graph;
    // device list of the unfinished instances (used when they are not contiguous), owned by the phase
    struct OwnedBuf : DevBuf {
        ~OwnedBuf() { release(); }
    } imap;
    std::vector<int> imap_host;
    if ((e = imap.ensure(sizeof(int) * (size_t)B)) != hipSuccess) return e;
    // The host polls one chunk behind: while it waits for a chunk's states the next chunk is already
    // queued, so the device does not wait for the poll and the launch (65 us a chunk, against 600 us of
    // work on 256^2).  The chunk after the one that finishes every instance is queued in vain: its
    // kernels return at once.  A chunk's states reach one of two slots of mapped host memory.
    PollSlots poll;
    if ((e = poll.init(*pa.poll, B, s)) != hipSuccess) return e;
    int64_t head = 0, tail = 0;  // chunks queued, chunks polled
    auto queue_chunk = [&]() -> hipError_t {
        // host-side guard: every queued iteration either advances n or finishes the instance
        if (queued > 2 * max_iter + 4 * (int64_t)pa.check_every + 64) return hipErrorUnknown;
        hipError_t ee = hipSuccess;
        if (pa.refresh_every > 0 && since_refresh >= pa.refresh_every) {
            since_refresh = 0;
            for (int b = 0; b < B; ++b) {
                if (host_S[b].done) continue;
                Geo gb = g;
                for (int a = 0; a < 3; ++a) {
                    gb.L[a] = host_S[b].L[a];
                    gb.h[a] = host_S[b].h[a];
                    gb.dk[a] = host_S[b].dk[a];
                }
                gb.cell = host_S[b].cell;
                if ((ee = refresh_instance<T>(gb, *pa.tw, c.f, (int64_t)b * N, S_dir + b, host_S[b].beta,
                                              host_S[b].omega, *pa.red, false, s)) != hipSuccess)
                    return ee;
            }
        }
        int left = pa.check_every;
        const int quarter = pa.check_every / 4;
        // (1-D: a chunk is one launch; no marks either where a second chunk cannot follow)
        if (head == 0 && g.dim > 1 && quarter > 0 && pa.check_every <= max_iter)
            for (int m = 0; m < PollSlots::kMarks; ++m) {
                if ((ee = enqueue_iterations<T>(c, quarter, s)) != hipSuccess) return ee;
                if ((ee = poll.queue(S_dir, 2 + m)) != hipSuccess) return ee;
                left -= quarter;
            }
        ee = graph.exec ? graph.launch(s) : enqueue_iterations<T>(c, left, s);
        if (ee != hipSuccess) return ee;
        queued += pa.check_every;
        since_refresh += pa.check_every;
        if ((ee = poll.queue(S_dir, (int)(head & 1))) != hipSuccess) return ee;
        ++head;
        return ee;
    };
    // A solve from a (nearly) converged start ends in its first chunk.  If that is seen, from the newest state that
    // has arrived, by the time the chunk is queued, no graph is captured; and the second chunk is queued at the
    // first one's last mark, unless it has ended there or is about to.  From the converged field (us; before the
    // chunks overlapped, with both unconditionally behind the first chunk, now): 256^2 FP64 684, 881, 648; 512^2 831,
    // 1250, 755; 64^3 1114, 1790, 883.
    auto first_ended = [&] {
        for (int slot : {0, 4, 3, 2})
            if (poll.ready(slot)) return poll.all_done(slot);
        return false;
    };
    for (;;) {
        if (head == tail && (e = queue_chunk()) != hipSuccess) return e;
        const bool first = head == 1 && tail == 0 && poll.used[4];
        if (queued <= max_iter && !(first && first_ended())) {
            if (!graph.exec && want_graph &&
                (e = graph.capture(s, [&] { return enqueue_iterations<T>(c, pa.check_every, s); })) != hipSuccess)
                return e;
            bool ending = false;
            if (first) {
                if ((e = hipEventSynchronize(poll.ev[4])) != hipSuccess) return e;
                ending = poll.ending(3, 4);
            }
            if (head - tail < 2 && !ending && (e = queue_chunk()) != hipSuccess) return e;
        }
        if ((e = poll.wait((int)(tail & 1), host_S)) != hipSuccess) return e;
        ++tail;
        std::vector<int> run;
        for (int b = 0; b < B; ++b)
            if (!host_S[b].done) run.push_back(b);
        if (run.empty()) break;
        // Converged instances are left out of later launches (a masked instance still costs its
        // workgroups' state and row reads in every pass): a contiguous run of unfinished instances is
        // launched as a range, any other set through the device list of their indices.  Tiles and row
        // layout keep following all B instances.  The chunk in flight still holds the old launches: it
        // is waited for before the list is rewritten and the graph goes.
        auto launched = [&] {
            const int nl = (int)run.size();
            return run.back() - run.front() + 1 == nl
                       ? (!c.g.imap && c.g.b0 == run.front() && (c.g.bl > 0 ? c.g.bl : B) == nl)
                       : (c.g.imap && c.g.bl == nl && run == imap_host);
        };
        if (launched()) continue;
        if (head > tail) {
            if ((e = poll.wait((int)(tail & 1), host_S)) != hipSuccess) return e;
            ++tail;
            run.clear();
            for (int b = 0; b < B; ++b)
                if (!host_S[b].done) run.push_back(b);
            if (run.empty()) break;
        }
        if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
        const int nl = (int)run.size();
        if (run.back() - run.front() + 1 == nl) {
            c.g.imap = nullptr;
            c.g.b0 = run.front();
        } else {
            imap_host = run;
            if ((e = hipMemcpyAsync(imap.ptr, imap_host.data(), sizeof(int) * nl, hipMemcpyHostToDevice, s)) != hipSuccess)
                return e;
            if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
            c.g.imap = (const int*)imap.ptr;
            c.g.b0 = 0;
        }
        c.g.bl = nl;
        graph.reset();
    }
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;  // the chunk queued in vain
    return hipSuccess;
}

// Instrumented iterations: initialise like run_phase, then run exactly `iters` iterations with
// every launch bracketed by events (the solver must not finish meanwhile: tol = 0 is expected).
template <typename T>
hipError_t profile_phase(PhaseArgs& pa, IterFields<T> f, std::vector<Scal>& host_S, int iters, KernelTimer& timer,
                         hipStream_t s) {
    const Geo& g = pa.g;
    const int64_t N = g.N;
    hipError_t e;
    Scal* S_dir = pa.S + pa.B;
    for (int k = 0; k < 2; ++k)
        if ((e = hipMemcpyAsync(pa.S + k * pa.B, host_S.data(), sizeof(Scal) * pa.B, hipMemcpyHostToDevice, s)) !=
            hipSuccess)
            return e;
    if ((e = normalize_all<T>(f, pa.B, N, S_dir, *pa.red, s)) != hipSuccess) return e;
    if ((e = zero_cg_memory<T>(f, (int64_t)pa.B * N, s)) != hipSuccess) return e;
    for (int b = 0; b < pa.B; ++b) {
        if ((e = refresh_instance<T>(g, *pa.tw, f, (int64_t)b * N, S_dir + b, host_S[b].beta, host_S[b].omega,
                                     *pa.red, true, s)) != hipSuccess)
            return e;
    }
    IterCtx<T> c;
    c.g = g;
    c.B = pa.B;
    c.tw = pa.tw;
    c.f = f;
    c.S = pa.S;
    c.parts = (double*)pa.red->parts.ptr;
    c.region_doubles = pa.region_doubles;
    c.precond = pa.precond;
    c.pointwise_blocks = (int)std::max<int64_t>(1, std::min<int64_t>(1024, N / 1024));
    c.timer = &timer;
    for (int k = 0; k < iters; ++k) {
        if ((e = enqueue_iterations<T>(c, 1, s)) != hipSuccess) return e;
        if ((e = timer.collect()) != hipSuccess) return e;
    }
    return hipMemcpy(host_S.data(), S_dir, sizeof(Scal) * pa.B, hipMemcpyDeviceToHost);
}

template hipError_t profile_phase<double>(PhaseArgs&, IterFields<double>, std::vector<Scal>&, int, KernelTimer&,
                                          hipStream_t);
template hipError_t profile_phase<float>(PhaseArgs&, IterFields<float>, std::vector<Scal>&, int, KernelTimer&,
                                         hipStream_t);

template hipError_t run_phase<double>(PhaseArgs&, IterFields<double>, std::vector<Scal>&, hipStream_t);
template hipError_t run_phase<float>(PhaseArgs&, IterFields<float>, std::vector<Scal>&, hipStream_t);

// Fresh FP64 (or FP32 plan) energy parts, lambda and residual of one field, queued into out.
template <typename T>
hipError_t verify_field(const Geo& g, const Twiddles& tw, const void* phi, const void* V, void* hphi, void* tmp,
                        double beta, double omega, Reduce& red, double* out, hipStream_t s) {
    const bool f64 = sizeof(T) == 8;
    hipError_t e;
    if ((e = op_apply(g, f64, 1, tw, phi, V, hphi, tmp, beta, omega, true, s)) != hipSuccess) return e;
    double* parts = (double*)red.parts.ptr;
    const int nb = 256;
    hipLaunchKernelGGL(k_verify_dot<T>, dim3(nb), dim3(256), 0, s, (const C2<T>*)phi, (const C2<T>*)hphi, g.N, parts);
    hipLaunchKernelGGL(k_verify_res<T>, dim3(nb), dim3(256), 0, s, (const C2<T>*)phi, (const C2<T>*)hphi, g.N, parts, nb,
                       parts + 2 * nb, out);
    hipLaunchKernelGGL(k_max_collect, dim3(1), dim3(256), 0, s, parts + 2 * nb, nb, out + 1);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return op_energy(g, f64, tw, phi, V, beta, omega, red, out + 4, s);
}

template hipError_t verify_field<double>(const Geo&, const Twiddles&, const void*, const void*, void*, void*, double,
                                         double, Reduce&, double*, hipStream_t);
template hipError_t verify_field<float>(const Geo&, const Twiddles&, const void*, const void*, void*, void*, double,
                                        double, Reduce&, double*, hipStream_t);

hipError_t convert_complex(bool to64, const void* in, void* out, int64_t n, hipStream_t s) {
    return to64 ? convert<float, double>(in, out, 2 * n, s) : convert<double, float>(in, out, 2 * n, s);
}
hipError_t convert_real(bool to64, const void* in, void* out, int64_t n, hipStream_t s) {
    return to64 ? convert<float, double>(in, out, n, s) : convert<double, float>(in, out, n, s);
}
hipError_t copy_bytes(const void* in, void* out, size_t bytes, hipStream_t s) {
    return hipMemcpyAsync(out, in, bytes, hipMemcpyDeviceToDevice, s);
}

template <typename T>
IterFields<T> carve_fields(DevBuf& buf, int64_t BN, hipError_t* err) {
    return carve<T>(buf, BN, err);
}
template IterFields<double> carve_fields<double>(DevBuf&, int64_t, hipError_t*);
template IterFields<float> carve_fields<float>(DevBuf&, int64_t, hipError_t*);

// Host template of the per-instance scalars.
Scal make_scal(const gpe_problem_t& p, const Geo& g, const gpe_pcg_opts_t& o) {
    Scal s;
    std::memset(&s, 0, sizeof(s));
    s.beta = p.beta;
    s.omega = p.omega;
    s.cell = g.cell;
    s.dim = p.dim;
    for (int a = 0; a < 3; ++a) {
        s.L[a] = g.L[a];
        s.dk[a] = g.dk[a];
        s.h[a] = g.h[a];
    }
    s.tol_res = o.tol_res_inf;
    s.tol_energy = o.tol_energy;
    s.theta_default = o.theta_default;
    s.method = o.method;
    s.beta_rule = o.beta_rule;
    s.line_search = o.line_search;
    s.max_halvings = o.max_halvings;
    s.precond = o.precond;
    s.max_iter = o.max_iter;
    s.switch_res = o.switch_res;
    s.best_res = 1e300;
    s.best_E = 1e300;
    return s;
}

int validate_opts(const gpe_pcg_opts_t* o) {
    if (!o) { set_error("opts is NULL"); return GPE_EINVAL; }
    if (o->method != 0 && o->method != 1) { set_error("method must be 0 (PG) or 1 (PCG)"); return GPE_EINVAL; }
    if (o->precond < GPE_P_NONE || o->precond > GPE_P_C2) { set_error("unknown preconditioner"); return GPE_EINVAL; }
    if (!(o->tol_res_inf >= 0.0) || !(o->tol_energy >= 0.0)) { set_error("tolerances must be >= 0"); return GPE_EINVAL; }
    if (o->max_iter < 0) { set_error("max_iter must be >= 0"); return GPE_EINVAL; }
    if (o->precision != 0 && o->precision != 1) { set_error("precision must be 0 (FP64) or 1 (mixed)"); return GPE_EINVAL; }
    if (o->beta_rule != 0 && o->beta_rule != 1) { set_error("beta_rule must be 0 (PR) or 1 (FR)"); return GPE_EINVAL; }
    if (o->line_search < 0 || o->line_search > 3) {
        set_error("line_search must be 0 (decrease test), 1 (Armijo), 2 (full) or 3 (strong Wolfe)");
        return GPE_EINVAL;
    }
    if (o->max_halvings < 0 || o->max_halvings > 60) { set_error("max_halvings must be in [0, 60]"); return GPE_EINVAL; }
    if (!(o->theta_default > 0.0)) { set_error("theta_default must be positive"); return GPE_EINVAL; }
    if (o->check_every < 1) { set_error("check_every must be >= 1"); return GPE_EINVAL; }
    if (o->refresh_every < 0) { set_error("refresh_every must be >= 0"); return GPE_EINVAL; }
    return GPE_OK;
}

int status_of(int st) {
    switch (st) {
        case ST_OK: return GPE_OK;
        case ST_NOT_CONVERGED: return GPE_NOT_CONVERGED;
        case ST_LINESEARCH: return GPE_ELINESEARCH;
        case ST_NONFINITE: return GPE_ENONFINITE;
        default: return GPE_EHIP;
    }
}

}  // namespace gpe
