// k_gs_sparse.hip -- the Gauss-Seidel operator (k_gs.hip) of a sparse channel: its matrix
// G = H^H H from the CSR rows and the column-compressed copy, and the two products with H
// that form b anew.
//
// G is nearly full (1 % density and 16384 rows leave 1.6 common rows per pair of users), but
// the work in it is small: each entry of column u meets the entries of its row, nnz^2 / B
// products in all.  A workgroup forms one row of G: it scatters those products into the
// row's U sums in LDS.  The order in which waves reach a sum is not fixed, so the sums are
// 64-bit integers, which add up the same in every order: the columns are first scaled by
// powers of two to norms in [1/2, 1), so that every partial sum is at most 1 in magnitude
// (Cauchy-Schwarz), and the products are rounded to multiples of 2^-61.  That error, at most
// sqrt(n) 2^-62 of ||h_u|| ||h_v||, is below the rounding of the products themselves.
// Bound: LDS atomics and the L2 reads of the rows; 16384 x 8192 at 1 % (1.1e8 products) 565 us.
#include "gs.hpp"
#include "la_common.hpp"

namespace cdm {

namespace {
constexpr int GSP_BAD = -100000;   // exponent of a column whose energy is not finite
template <typename V> __device__ __forceinline__ double2 to_d(V v) {
    return make_double2((double)v.x, (double)v.y);
}
__device__ __forceinline__ bool bad_csr(const uint32_t* status) {
    return (__atomic_load_n(status, __ATOMIC_RELAXED) & (uint32_t)CDM_INFO_BAD_INPUT) != 0u;
}
}  // namespace

// kexp[u]: 2^kexp >= ||h_u||, one wave per column
template <typename T>
__global__ __launch_bounds__(256) void k_gsp_scale(const int32_t* __restrict__ colptr, const cv<T>* __restrict__ cval,
                                                   int U, int32_t* __restrict__ kexp) {
    const int u = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (u >= U) return;
    double e = 0.0;
    for (int k = colptr[u] + lane; k < colptr[u + 1]; k += 64) e += cabs2d(cval[k]);
    e = group_sum<1>(e);
    if (lane == 0) {
        int ex = 0;
        if (!isfinite(e))
            ex = GSP_BAD;
        else if (e > 0.0)
            (void)frexp(sqrt(e), &ex);
        kexp[u] = ex;
    }
}

// the CSR values over their columns' scales, in FP64
template <typename T>
__global__ __launch_bounds__(256) void k_gsp_values(const cv<T>* __restrict__ val, const int32_t* __restrict__ colidx,
                                                    int64_t nnz, const int32_t* __restrict__ kexp,
                                                    double2* __restrict__ vs, const uint32_t* __restrict__ status) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= nnz || bad_csr(status)) return;
    const int ex = kexp[colidx[i]];
    const double2 v = to_d(val[i]);
    vs[i] = ex == GSP_BAD ? make_double2(0.0, 0.0) : make_double2(ldexp(v.x, -ex), ldexp(v.y, -ex));
}

// Row u of G into A (Up x Up, zero past U).  16 waves: each takes every 16th entry of column
// u and goes through that entry's row, the first 128 entries of the next RING rows in flight (with one
// row of 64 in flight the round trips took 849 us at 16384 x 8192, 1 %).
__global__ __launch_bounds__(1024) void k_gsp_matrix(const int32_t* __restrict__ colptr,
                                                     const int32_t* __restrict__ rowidx,
                                                     const int32_t* __restrict__ rowptr,
                                                     const int32_t* __restrict__ colidx,
                                                     const double2* __restrict__ vs, const int32_t* __restrict__ kexp,
                                                     int U, int Up, double2* __restrict__ A) {
    constexpr int RING = 3;
    extern __shared__ __attribute__((aligned(16))) longlong2 acc[];
    const int u = blockIdx.x, lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    double2* out = A + (int64_t)u * Up;
    if (u >= U) {
        for (int v = threadIdx.x; v < Up; v += 1024) out[v] = make_double2(0.0, 0.0);
        return;
    }
    const int e0 = colptr[u], e1 = colptr[u + 1];
    for (int v = threadIdx.x; v < U; v += 1024) acc[v] = longlong2{0, 0};
    __syncthreads();
    auto add = [&](int v, const double2& hu, const double2& h) __attribute__((always_inline)) {
        // conj(h_u) h_v as multiples of 2^-61
        const double re = fma(hu.x, h.x, hu.y * h.y), im = fma(hu.x, h.y, -(hu.y * h.x));
        atomicAdd((unsigned long long*)&acc[v].x, (unsigned long long)llrint(re * 0x1p61));
        atomicAdd((unsigned long long*)&acc[v].y, (unsigned long long)llrint(im * 0x1p61));
    };
    auto from_lane = [&](const double2& h, uint64_t mine) __attribute__((always_inline)) -> double2 {
        const int at = __ffsll((unsigned long long)mine) - 1;
        return make_double2(lane_value(h.x, at), lane_value(h.y, at));
    };
    // this wave's entries, a lane each: the row's bounds
    for (int base = e0 + wid; base < e1; base += 16 * 64) {
        const int e = base + 16 * lane;
        const int row = e < e1 ? rowidx[e] : 0;
        const int a0 = e < e1 ? rowptr[row] : 0, a1 = e < e1 ? rowptr[row + 1] : 0;
        const int cnt = min(64, (e1 - base + 15) / 16);
        int v[RING][2];
        double2 h[RING][2];
        auto fetch = [&](int d, int j) __attribute__((always_inline)) {
            if (j >= cnt) return;
            const int b0 = __builtin_amdgcn_readlane(a0, j), b1 = __builtin_amdgcn_readlane(a1, j);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int k = b0 + lane + 64 * c;
                v[d][c] = -1;
                h[d][c] = make_double2(0.0, 0.0);
                if (k < b1) {
                    v[d][c] = colidx[k];
                    h[d][c] = vs[k];
                }
            }
        };
#pragma unroll
        for (int d = 0; d < RING; ++d) fetch(d, d);
        for (int j0 = 0; j0 < cnt; j0 += RING) {
#pragma unroll
            for (int d = 0; d < RING; ++d) {
                if (j0 + d >= cnt) continue;
                const int b0 = __builtin_amdgcn_readlane(a0, j0 + d), b1 = __builtin_amdgcn_readlane(a1, j0 + d);
                // column u's own (scaled) entry of this row
                double2 hu = make_double2(0.0, 0.0);
                const uint64_t m0 = __ballot(v[d][0] == u), m1 = __ballot(v[d][1] == u);
                if (m0)
                    hu = from_lane(h[d][0], m0);
                else if (m1)
                    hu = from_lane(h[d][1], m1);
                else
                    for (int k = b0 + 128; k < b1; k += 64) {
                        const bool in = k + lane < b1;
                        const uint64_t m = __ballot(in && colidx[in ? k + lane : k] == u);
                        if (m) {
                            hu = from_lane(vs[in ? k + lane : k], m);
                            break;
                        }
                    }
                if (v[d][0] >= 0) add(v[d][0], hu, h[d][0]);
                if (v[d][1] >= 0) add(v[d][1], hu, h[d][1]);
                for (int k = b0 + 128 + lane; k < b1; k += 64) add(colidx[k], hu, vs[k]);
                fetch(d, j0 + d + RING);
            }
        }
    }
    __syncthreads();
    const int ku = kexp[u];
    for (int v = threadIdx.x; v < Up; v += 1024) {
        double2 z = make_double2(0.0, 0.0);
        if (v < U) {
            const int kv = kexp[v];
            if (ku == GSP_BAD && v == u)
                z = make_double2(__builtin_nan(""), 0.0);   // reaches every x through this panel
            else if (ku != GSP_BAD && kv != GSP_BAD)
                z = make_double2(ldexp((double)acc[v].x, ku + kv - 61), ldexp((double)acc[v].y, ku + kv - 61));
        }
        out[v] = z;
    }
}

// r = y - H x, one wave per row (r = y where the CSR arrays are malformed: H = 0)
template <typename T>
__global__ __launch_bounds__(256) void k_gsp_rows(const int32_t* __restrict__ rowptr,
                                                  const int32_t* __restrict__ colidx,
                                                  const cv<T>* __restrict__ val, int B, const cv<T>* __restrict__ y,
                                                  const double2* __restrict__ x, double2* __restrict__ r,
                                                  const uint32_t* __restrict__ status,
                                                  const uint32_t* __restrict__ done) {
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (i >= B || *done) return;
    double2 s = make_double2(0.0, 0.0);
    if (!bad_csr(status))
        for (int k = rowptr[i] + lane; k < rowptr[i + 1]; k += 64) cfma(s, to_d(val[k]), x[colidx[k]]);
    s.x = group_sum<1>(s.x);
    s.y = group_sum<1>(s.y);
    if (lane == 0) {
        const double2 z = to_d(y[i]);
        r[i] = make_double2(z.x - s.x, z.y - s.y);
    }
}

// b_u = h_u^H r - lambda x_u, one wave per user (zero past U)
template <typename T>
__global__ __launch_bounds__(256) void k_gsp_grad(const int32_t* __restrict__ colptr,
                                                  const int32_t* __restrict__ rowidx,
                                                  const cv<T>* __restrict__ cval, int U, int Up,
                                                  const double2* __restrict__ r, const double2* __restrict__ x,
                                                  double lambda, double2* __restrict__ b,
                                                  const uint32_t* __restrict__ done) {
    const int u = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (u >= Up || *done) return;
    double2 s = make_double2(0.0, 0.0);
    if (u < U)
        for (int k = colptr[u] + lane; k < colptr[u + 1]; k += 64) cfma_conj(s, to_d(cval[k]), r[rowidx[k]]);
    s.x = group_sum<1>(s.x);
    s.y = group_sum<1>(s.y);
    if (lane == 0) b[u] = make_double2(s.x - lambda * x[u].x, s.y - lambda * x[u].y);
}

size_t gs_sparse_lds(int U) { return 16 * (size_t)U; }

hipError_t gs_sparse_setup(int U) {
    return hipFuncSetAttribute((const void*)k_gsp_matrix, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)gs_sparse_lds(U));
}

template <typename T> static hipError_t matrix_t(const GsLaunch& L, hipStream_t st) {
    const SparseLaunch& S = *L.sp;
    const hipError_t e = launch_sparse(S, st);   // the column-compressed copy
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_gsp_scale<T>, dim3((L.U + 3) / 4), dim3(256), 0, st, S.colptr, (const cv<T>*)S.cval, L.U,
                       L.kexp);
    if (S.nnz > 0)
        hipLaunchKernelGGL(k_gsp_values<T>, dim3((unsigned)((S.nnz + 255) / 256)), dim3(256), 0, st,
                           (const cv<T>*)S.val, S.colidx, S.nnz, L.kexp, (double2*)L.vs, S.status);
    hipLaunchKernelGGL(k_gsp_matrix, dim3(L.s.Up), dim3(1024), gs_sparse_lds(L.U), st, S.colptr, S.rowidx, S.rowptr,
                       S.colidx, (const double2*)L.vs, L.kexp, L.U, L.s.Up, (double2*)L.A);
    return hipGetLastError();
}
template <typename T> static hipError_t refresh_t(const GsLaunch& L, bool rows, hipStream_t st) {
    const SparseLaunch& S = *L.sp;
    const uint32_t* done = L.ctr + 4;
    if (rows)
        hipLaunchKernelGGL(k_gsp_rows<T>, dim3((L.B + 3) / 4), dim3(256), 0, st, S.rowptr, S.colidx,
                           (const cv<T>*)S.val, L.B, (const cv<T>*)L.y, (const double2*)L.xw, (double2*)L.r, S.status,
                           done);
    hipLaunchKernelGGL(k_gsp_grad<T>, dim3((L.s.Up + 3) / 4), dim3(256), 0, st, S.colptr, S.rowidx,
                       (const cv<T>*)S.cval, L.U, L.s.Up, (const double2*)L.r, (const double2*)L.xw, L.lambda,
                       (double2*)L.b, done);
    return hipGetLastError();
}

hipError_t gs_sparse_matrix(const GsLaunch& L, hipStream_t st) {
    return L.c128 ? matrix_t<double>(L, st) : matrix_t<float>(L, st);
}
hipError_t gs_sparse_refresh(const GsLaunch& L, bool rows, hipStream_t st) {
    return L.c128 ? refresh_t<double>(L, rows, st) : refresh_t<float>(L, rows, st);
}

}  // namespace cdm
