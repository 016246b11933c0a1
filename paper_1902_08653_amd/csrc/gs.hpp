// gs.hpp -- launch descriptors of the Gauss-Seidel operator engine (k_gs.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cdm.h"
#include "launch.hpp"

namespace cdm {

// Tiling of one instance: panels of k users, Up = npan * k, P workgroups of R rows each in
// the sweep (one workgroup for a single panel of 128), nblk 64 x 64 blocks of the lower
// triangle over nwork workgroups in the Gram pass.
struct GsShape {
    int k = 0, npan = 0, Up = 0, R = 0, P = 0, nblk = 0, nwork = 0;
    bool one = false;
};
GsShape gs_shape(int B, int U);

constexpr int GS_CTR_WORDS = 16;   // uint32: [2] abort, [3] status, [4] done, [6] arrivals
// 64-bit exchange words after the control words, cleared with them per solve
size_t gs_exchange_words(const GsShape& s);

struct GsSweepArgs {
    const double2* W;
    const double2* M;
    const double2* b;
    double2* x;
    uint64_t* xch;
    uint32_t* abort_flag;
    uint32_t* done;
    cdm_info* info;
    double tol;
    uint64_t timeout_ticks;
    int npan, Up;
    // what the single-panel sweep forms b anew from (dense channels)
    const void* H;
    const void* y;
    double2* r;
    uint32_t* arrived;
    int64_t ld;
    int B, U;
    double lambda;
};

struct GsLaunch {
    bool c128;
    GsShape s;
    int B, U;
    const void* H;
    int64_t ld;
    const void* y;
    const void* x0;       // optional
    void* x;
    cdm_info* info;
    double lambda, tol;
    int T_max;
    uint64_t timeout_ticks;
    uint32_t* ctr;        // GS_CTR_WORDS words, then the exchange words
    void* gpart;          // (nwork + nblk) x 4096 complex128
    void* A;              // Up x Up
    void* W;              // Up x Up
    void* M;              // npan x k x k
    void* Mt;             // and transposed
    void* r;              // B
    void* b;              // Up
    void* xw;             // Up
    const SparseLaunch* sp = nullptr;   // CSR input: its column-compressed copy (H is not used)
    int32_t* kexp = nullptr;            // U: column scales
    void* vs = nullptr;                 // nnz: scaled values, complex128
    hipEvent_t ev_pre, ev_init, ev_sweep;   // optional stage marks
};
hipError_t gs_setup(const GsShape& s);   // LDS limits of the kernels, at plan creation
hipError_t launch_gs(const GsLaunch& L, hipStream_t st);
// CSR input (k_gs_sparse.hip): G into L.A, and b (with rows: from x, else from r = y)
hipError_t gs_sparse_setup(int U);
hipError_t gs_sparse_matrix(const GsLaunch& L, hipStream_t st);
hipError_t gs_sparse_refresh(const GsLaunch& L, bool rows, hipStream_t st);

}  // namespace cdm
