// Host-side plan object behind the opaque gpe_plan_t of the C ABI.
#pragma once

#include <atomic>
#include <mutex>

#include "internal.hpp"

constexpr int kHostScalars = 16;

struct gpe_plan {
    gpe_problem_t prob;
    int dtype = GPE_F64;
    int device = 0;
    gpe::Geo g;
    gpe::Twiddles tw;
    gpe::Reduce red;
    gpe::DevBuf tmp;               // scratch field(s) for multi-pass operators
    gpe::DevBuf solver;            // solver fields of the plan's precision (FP64 phase when mixed)
    gpe::DevBuf solver32;          // FP32 solver fields of a mixed-precision solve
    gpe::DevBuf scal;              // per-instance solver scalars
    gpe::DevBuf hist;              // per-iteration history rows
    gpe::HostBuf poll;             // solver states as the host polls them
    int64_t hist_rows = 0;
    // mapped host memory for the scalars a call returns (kHostScalars) and its device address: kernels write
    // them there, no copy is queued.  Made by the first call that returns scalars: the allocation took 60-130 us
    // of every plan's creation.
    std::atomic<double*> host{nullptr};
    double* host_dev = nullptr;
    hipError_t ensure_host() {
        if (host.load(std::memory_order_acquire)) return hipSuccess;
        std::lock_guard<std::mutex> lock(gpe::capture_mutex());
        if (host.load(std::memory_order_relaxed)) return hipSuccess;
        double* p = nullptr;
        hipError_t e = hipHostMalloc((void**)&p, sizeof(double) * kHostScalars, hipHostMallocMapped);
        if (e != hipSuccess) return e;
        if ((e = hipHostGetDevicePointer((void**)&host_dev, p, 0)) != hipSuccess) {
            (void)hipHostFree(p);
            return e;
        }
        host.store(p, std::memory_order_release);
        return hipSuccess;
    }
    bool f64() const { return dtype == GPE_F64; }
    void release() {
        tw.release();
        red.parts.release();
        red.scalars.release();
        tmp.release();
        solver.release();
        solver32.release();
        scal.release();
        hist.release();
        poll.release();
        if (double* const p = host.exchange(nullptr)) {
            std::lock_guard<std::mutex> lock(gpe::capture_mutex());
            (void)hipHostFree(p);
        }
        host_dev = nullptr;
    }
};
