// Host-side plan object behind the opaque gpe_plan_t of the C ABI.
#pragma once

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
    int64_t hist_rows = 0;
    double* host = nullptr;        // mapped host memory for the scalars a call returns (kHostScalars), and
    double* host_dev = nullptr;    // its device address: kernels write them there, no copy is queued
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
        if (host) {
            std::lock_guard<std::mutex> lock(gpe::capture_mutex());
            (void)hipHostFree(host);
        }
        host = host_dev = nullptr;
    }
};
