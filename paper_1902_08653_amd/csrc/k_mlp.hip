// k_mlp.hip -- the small per-coordinate MLP of the learned warm start.
//
// Three weight layers F -> H1 -> H2 -> 2 with ReLU between them; BF16 operands on
// gfx950's doubled-K MFMA (v_mfma_f32_16x16x32_bf16: 16 x 16 output, K = 32 per
// instruction, each lane holding 8 consecutive k of its row or column) with FP32
// accumulation; FP32 master weights and Adam state.  The GEMM is generic over strides so that one kernel serves the
// forward products, the weight gradients (A^T B) and the input gradients (A B^T).
#include <algorithm>

#include "common.hpp"
#include "launch.hpp"

namespace cdm {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// the MFMA fragment of 8 consecutive BF16 values at p (16-B aligned)
__device__ __forceinline__ bf16x8_t frag8(const unsigned short* p) { return *reinterpret_cast<const bf16x8_t*>(p); }
__device__ __forceinline__ f32x4_t mfma32(const bf16x8_t& a, const bf16x8_t& b, const f32x4_t& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}


// FP32 -> BF16 bits, round to nearest even, by gfx950's conversion instruction
// (v_cvt_pk_bf16_f32; a NaN stays a NaN)
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{lo, hi}, bf16x2_t));
}
__device__ __forceinline__ unsigned short f32_to_bf16(float f) {
    return __builtin_bit_cast(unsigned short, (__bf16)f);
}

// C[m][n] = sum_k A(m, k) B(k, n) (+ bias[n]); A(m, k) = A[m*sam + k*sak], B(k, n) = B[k*sbk + n*sbn];
// C row-major with leading dimension ldc.  64 x 64 tile per workgroup of 4 waves,
// each wave a 32 x 32 block of 2 x 2 MFMA 16 x 16 x 32 tiles.  beta: 0 overwrite, 1 accumulate.
constexpr int GT = 64;
constexpr int GK = 32;

__global__ __launch_bounds__(256) void k_gemm_bf16(const float* __restrict__ A, int64_t sam, int64_t sak,
                                                   const float* __restrict__ Bm, int64_t sbk, int64_t sbn,
                                                   float* __restrict__ C, int64_t ldc, int M, int N, int K,
                                                   const float* __restrict__ bias, int beta, int kc, int64_t zc,
                                                   int relu, const float* __restrict__ mask) {
    // split along K: workgroup z takes K range [z kc, z kc + kc) into C + z zc
    {
        const int z = blockIdx.z;
        A += (int64_t)z * kc * sak;
        Bm += (int64_t)z * kc * sbk;
        C += (int64_t)z * zc;
        K = min(kc, K - z * kc);
    }
    // both tiles k-fastest (a fragment is 8 consecutive k: one 16-B read); rows padded by
    // 8 values to keep the 16-B reads of a wave on distinct banks
    __shared__ __align__(16) unsigned short As[GT][GK + 8];
    __shared__ __align__(16) unsigned short Bs[GT][GK + 8];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int m0 = blockIdx.y * GT, n0 = blockIdx.x * GT;
    const int wm = (wid >> 1) * 32, wn = (wid & 1) * 32;
    f32x4_t acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < K; k0 += GK) {
        // stage A (64 x 32) and B (32 x 64) as BF16: 2048 elements each, 8 per thread
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int e = tid + 256 * q;
            const int am = e / GK, ak = e % GK;
            const int gm = m0 + am, gk = k0 + ak;
            As[am][ak] = (gm < M && gk < K) ? f32_to_bf16(A[(int64_t)gm * sam + (int64_t)gk * sak]) : (unsigned short)0;
            const int bk = e / GT, bn = e % GT;
            const int hk = k0 + bk, hn = n0 + bn;
            Bs[bn][bk] = (hk < K && hn < N) ? f32_to_bf16(Bm[(int64_t)hk * sbk + (int64_t)hn * sbn]) : (unsigned short)0;
        }
        __syncthreads();
        bf16x8_t a[2], b[2];
        const int kk = 8 * (lane >> 4);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            a[i] = frag8(&As[wm + 16 * i + (lane & 15)][kk]);
            b[i] = frag8(&Bs[wn + 16 * i + (lane & 15)][kk]);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = mfma32(a[i], b[j], acc[i][j]);
        __syncthreads();
    }
    // D layout: lane -> column (lane & 15), rows 4 * (lane >> 4) + r
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int gm = m0 + wm + 16 * i + 4 * (lane >> 4) + r;
                const int gn = n0 + wn + 16 * j + (lane & 15);
                if (gm < M && gn < N) {
                    float v = acc[i][j][r];
                    if (bias) v += bias[gn];
                    if (relu) v = v > 0.f ? v : 0.f;
                    if (mask) v = mask[(int64_t)gm * ldc + gn] > 0.f ? v : 0.f;
                    float* cp = &C[(int64_t)gm * ldc + gn];
                    *cp = beta ? (*cp + v) : v;
                }
            }
}

// Large products (the training GEMMs): 128 x 128 tile per workgroup of 4 waves (each a
// 64 x 64 block of 4 x 4 MFMA tiles), K in chunks of 32 staged as BF16 in LDS with the next
// chunk's FP32 loads in flight during the current chunk's MFMAs.  Operands are read with
// 16-B loads along their contiguous dimension: AK = A contiguous in k (else in m), BN = B
// contiguous in n (else in k).  LDS keeps both tiles k-fastest, so an MFMA fragment (8
// consecutive k) is one 16-B read, and one 16 x 16 x 32 MFMA covers the chunk.
constexpr int G2T = 128, G2K = 32, G2P = G2K + 8;   // tile, K chunk, padded LDS row
template <bool AK, bool BN>
__global__ __launch_bounds__(256) void k_gemm2_bf16(const float* __restrict__ A, int64_t lda,
                                                    const float* __restrict__ Bm, int64_t ldb,
                                                    float* __restrict__ C, int64_t ldc, int M, int N, int K,
                                                    const float* __restrict__ bias, int beta, int kc, int64_t zc,
                                                    int relu, const float* __restrict__ mask) {
    // split along K: workgroup z takes K range [z kc, z kc + kc) into C + z zc
    {
        const int z = blockIdx.z;
        A += (int64_t)z * kc * (AK ? 1 : lda);
        Bm += (int64_t)z * kc * (BN ? ldb : 1);
        C += (int64_t)z * zc;
        K = min(kc, K - z * kc);
    }
    __shared__ __align__(16) unsigned short As[G2T][G2P];
    __shared__ __align__(16) unsigned short Bs[G2T][G2P];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int m0 = blockIdx.y * G2T, n0 = blockIdx.x * G2T;
    const int wm = (wid >> 1) * 64, wn = (wid & 1) * 64;
    // each thread moves 16 floats of A and 16 of B per chunk, as four 16-B loads along
    // the operand's contiguous dimension
    //   contiguous in k: row = tid / 2, k offset = (tid % 2) * 16
    //   contiguous in m or n: k = tid / 8, row offset = (tid % 8) * 16
    float4 ra[4], rb[4];
    auto load = [&](int k0) {
        if (AK) {
            const int r = tid >> 1, kk = k0 + (tid & 1) * 16;
            const int gm = m0 + r;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                ra[q] = (gm < M && kk + 4 * q < K) ? *reinterpret_cast<const float4*>(A + (int64_t)gm * lda + kk + 4 * q)
                                                   : make_float4(0.f, 0.f, 0.f, 0.f);
        } else {
            const int kk = k0 + (tid >> 3), mm = m0 + (tid & 7) * 16;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                ra[q] = (kk < K && mm + 4 * q < M) ? *reinterpret_cast<const float4*>(A + (int64_t)kk * lda + mm + 4 * q)
                                                   : make_float4(0.f, 0.f, 0.f, 0.f);
        }
        if (BN) {
            const int kk = k0 + (tid >> 3), nn = n0 + (tid & 7) * 16;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                rb[q] = (kk < K && nn + 4 * q < N) ? *reinterpret_cast<const float4*>(Bm + (int64_t)kk * ldb + nn + 4 * q)
                                                   : make_float4(0.f, 0.f, 0.f, 0.f);
        } else {
            const int r = tid >> 1, kk = k0 + (tid & 1) * 16;
            const int gn = n0 + r;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                rb[q] = (gn < N && kk + 4 * q < K) ? *reinterpret_cast<const float4*>(Bm + (int64_t)gn * ldb + kk + 4 * q)
                                                   : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    auto store = [&]() {
        if (AK) {   // 4 consecutive k per float4: two packed BF16 pairs, one 8-B store
            const int r = tid >> 1, kk = (tid & 1) * 16;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<uint2*>(&As[r][kk + 4 * q]) =
                    make_uint2(pack_bf16x2(ra[q].x, ra[q].y), pack_bf16x2(ra[q].z, ra[q].w));
        } else {
            const int kk = tid >> 3, mm = (tid & 7) * 16;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                As[mm + 4 * q + 0][kk] = f32_to_bf16(ra[q].x);
                As[mm + 4 * q + 1][kk] = f32_to_bf16(ra[q].y);
                As[mm + 4 * q + 2][kk] = f32_to_bf16(ra[q].z);
                As[mm + 4 * q + 3][kk] = f32_to_bf16(ra[q].w);
            }
        }
        if (BN) {
            const int kk = tid >> 3, nn = (tid & 7) * 16;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                Bs[nn + 4 * q + 0][kk] = f32_to_bf16(rb[q].x);
                Bs[nn + 4 * q + 1][kk] = f32_to_bf16(rb[q].y);
                Bs[nn + 4 * q + 2][kk] = f32_to_bf16(rb[q].z);
                Bs[nn + 4 * q + 3][kk] = f32_to_bf16(rb[q].w);
            }
        } else {    // B contiguous in k: packed like A
            const int r = tid >> 1, kk = (tid & 1) * 16;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<uint2*>(&Bs[r][kk + 4 * q]) =
                    make_uint2(pack_bf16x2(rb[q].x, rb[q].y), pack_bf16x2(rb[q].z, rb[q].w));
        }
    };
    f32x4_t acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int kq = 8 * (lane >> 4);
    load(0);
    for (int k0 = 0; k0 < K; k0 += G2K) {
        __syncthreads();   // the previous chunk's MFMAs are done with the tiles
        store();
        __syncthreads();
        if (k0 + G2K < K) load(k0 + G2K);
        bf16x8_t a[4], b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            a[i] = frag8(&As[wm + 16 * i + (lane & 15)][kq]);
            b[i] = frag8(&Bs[wn + 16 * i + (lane & 15)][kq]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = mfma32(a[i], b[j], acc[i][j]);
    }
    // D layout: lane -> column (lane & 15), rows 4 * (lane >> 4) + r
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int gm = m0 + wm + 16 * i + 4 * (lane >> 4) + r;
                const int gn = n0 + wn + 16 * j + (lane & 15);
                if (gm < M && gn < N) {
                    float v = acc[i][j][r];
                    if (bias) v += bias[gn];
                    if (relu) v = v > 0.f ? v : 0.f;
                    if (mask) v = mask[(int64_t)gm * ldc + gn] > 0.f ? v : 0.f;
                    float* cp = &C[(int64_t)gm * ldc + gn];
                    *cp = beta ? (*cp + v) : v;
                }
            }
}

// S > 1: S splits of K (chunks of kc, a multiple of 32) side by side, split z writing C + z zc
static hipError_t gemm_bf16_one(const float* A, int64_t sam, int64_t sak, const float* B, int64_t sbk, int64_t sbn,
                                float* C, int64_t ldc, int M, int N, int K, const float* bias, int beta, hipStream_t st,
                                int S = 1, int kc = 0, int64_t zc = 0, int relu = 0, const float* mask = nullptr) {
    if (S == 1) kc = K;
    // the tiled kernel: large products whose operands are contiguous along one dimension,
    // with 16-B aligned rows (K, M, N multiples of 4 where they are contiguous)
    const bool big = M >= G2T && N >= G2T && kc >= G2K;
    const bool ak = sak == 1, am = sam == 1, bn = sbn == 1, bk = sbk == 1;
    auto al = [](const void* p, int64_t ld) { return ((uintptr_t)p % 16 == 0) && (ld % 4 == 0); };
    if (big && (ak || am) && (bn || bk) && (K % 4 == 0) && (M % 4 == 0) && (N % 4 == 0)) {
        const int64_t lda = ak ? sam : sak, ldb = bn ? sbk : sbn;
        if (al(A, lda) && al(B, ldb)) {
            const dim3 g((N + G2T - 1) / G2T, (M + G2T - 1) / G2T, S);
            if (ak && bn) hipLaunchKernelGGL((k_gemm2_bf16<true, true>), g, dim3(256), 0, st, A, lda, B, ldb, C, ldc, M, N, K, bias, beta, kc, zc, relu, mask);
            else if (ak) hipLaunchKernelGGL((k_gemm2_bf16<true, false>), g, dim3(256), 0, st, A, lda, B, ldb, C, ldc, M, N, K, bias, beta, kc, zc, relu, mask);
            else if (bn) hipLaunchKernelGGL((k_gemm2_bf16<false, true>), g, dim3(256), 0, st, A, lda, B, ldb, C, ldc, M, N, K, bias, beta, kc, zc, relu, mask);
            else hipLaunchKernelGGL((k_gemm2_bf16<false, false>), g, dim3(256), 0, st, A, lda, B, ldb, C, ldc, M, N, K, bias, beta, kc, zc, relu, mask);
            return hipGetLastError();
        }
    }
    dim3 grid((N + GT - 1) / GT, (M + GT - 1) / GT, S);
    hipLaunchKernelGGL(k_gemm_bf16, grid, dim3(256), 0, st, A, sam, sak, B, sbk, sbn, C, ldc, M, N, K, bias, beta, kc, zc,
                       relu, mask);
    return hipGetLastError();
}

// split-K finish: C = sum_s part[s] (fixed order) (+ bias), then relu or the mask
// [mask > 0] (leading dimension ldc) where given, (+ C if beta)
__global__ void k_splitk_sum(const float* __restrict__ part, int S, int M, int N, float* __restrict__ C, int64_t ldc,
                             const float* __restrict__ bias, int beta, int relu, const float* __restrict__ mask) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)M * N) return;
    const int m = (int)(e / N), n = (int)(e % N);
    float v = 0.f;
    for (int k = 0; k < S; ++k) v += part[(int64_t)k * M * N + e];
    if (bias) v += bias[n];
    if (relu) v = v > 0.f ? v : 0.f;
    if (mask) v = mask[(int64_t)m * ldc + n] > 0.f ? v : 0.f;
    float* cp = &C[(int64_t)m * ldc + n];
    *cp = beta ? (*cp + v) : v;
}

// C = A B (+ bias) (+ C): products with a long K and few output tiles (the weight
// gradients, K = rows) are split along K into S chunks computed side by side into
// `splitk` (S * M * N floats), then summed in chunk order.
hipError_t launch_gemm_bf16(const float* A, int64_t sam, int64_t sak, const float* B, int64_t sbk, int64_t sbn, float* C,
                            int64_t ldc, int M, int N, int K, const float* bias, int beta, hipStream_t st,
                            float* splitk, int64_t splitk_floats, int relu = 0, const float* mask = nullptr) {
    const int64_t tiles = (int64_t)((M + 63) / 64) * ((N + 63) / 64);
    int S = 1;
    if (splitk && K >= 4096 && tiles < 256) {
        S = (int)std::min<int64_t>(std::min<int64_t>(64, K / 256), splitk_floats / ((int64_t)M * N));
        S = std::max(S, 1);
    }
    if (S == 1) return gemm_bf16_one(A, sam, sak, B, sbk, sbn, C, ldc, M, N, K, bias, beta, st, 1, 0, 0, relu, mask);
    const int chunk = ((K + S - 1) / S + 31) / 32 * 32;   // multiple of the tiled kernel's K chunk
    const int s = (K + chunk - 1) / chunk;
    hipError_t e = gemm_bf16_one(A, sam, sak, B, sbk, sbn, splitk, N, M, N, K, nullptr, 0, st, s, chunk, (int64_t)M * N);
    if (e != hipSuccess) return e;
    const int64_t mn = (int64_t)M * N;
    hipLaunchKernelGGL(k_splitk_sum, dim3((unsigned)((mn + 255) / 256)), dim3(256), 0, st, (const float*)splitk, s, M,
                       N, C, ldc, bias, beta, relu, mask);
    return hipGetLastError();
}

// A = relu(Z)
__global__ void k_relu(const float* __restrict__ Z, float* __restrict__ A, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) A[i] = Z[i] > 0.f ? Z[i] : 0.f;
}
// dZ = dA * [Z > 0]
__global__ void k_relu_bwd(const float* __restrict__ Z, const float* __restrict__ dA, float* __restrict__ dZ, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dZ[i] = Z[i] > 0.f ? dA[i] : 0.f;
}
// dO = 2 (O - T) / (N * nout); per-block partial sums of (O - T)^2
__global__ void k_mse(const float* __restrict__ O, const float* __restrict__ Tg, float* __restrict__ dO, int64_t n,
                      float scale, float* __restrict__ part) {
    __shared__ float s[256];
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    float e = 0.f;
    if (i < n) {
        const float d = O[i] - Tg[i];
        dO[i] = 2.f * d * scale;
        e = d * d;
    }
    s[threadIdx.x] = e;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) s[threadIdx.x] += s[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = s[0];
}
// Column sums of an M x N row-major matrix (bias gradients) in two fixed-order stages:
// workgroup (bx, by) sums rows [by R, (by + 1) R) of columns 64 bx .. 64 bx + 63 (four row
// lanes per column, combined in order) into part[by][n]; k_colsum_fin adds the CS_SPLIT
// partials of each column in order.
constexpr int CS_SPLIT = 64;
__global__ __launch_bounds__(256) void k_colsum(const float* __restrict__ X, int M, int N, float* __restrict__ part) {
    __shared__ float s[4][64];
    const int c = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int n = blockIdx.x * 64 + c;
    const int R = (M + CS_SPLIT - 1) / CS_SPLIT;
    const int m0 = blockIdx.y * R, m1 = min(M, m0 + R);
    float acc = 0.f;
    if (n < N)
        for (int m = m0 + q; m < m1; m += 4) acc += X[(int64_t)m * N + n];
    s[q][c] = acc;
    __syncthreads();
    if (q == 0 && n < N) part[(int64_t)blockIdx.y * N + n] = ((s[0][c] + s[1][c]) + s[2][c]) + s[3][c];
}
__global__ void k_colsum_fin(const float* __restrict__ part, int N, float* __restrict__ out) {
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= N) return;
    float acc = 0.f;
    for (int k = 0; k < CS_SPLIT; ++k) acc += part[(int64_t)k * N + n];
    out[n] = acc;
}
// Adam (bias-corrected), FP32 master weights
__global__ void k_adam(float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m1, float* __restrict__ m2,
                       int64_t n, float lr, float b1, float b2, float eps, float c1, float c2) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float a = b1 * m1[i] + (1.f - b1) * gi;
    const float b = b2 * m2[i] + (1.f - b2) * gi * gi;
    m1[i] = a;
    m2[i] = b;
    w[i] -= lr * (a / c1) / (sqrtf(b / c2) + eps);
}

hipError_t launch_relu(const float* Z, float* A, int64_t n, hipStream_t st) {
    hipLaunchKernelGGL(k_relu, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, Z, A, n);
    return hipGetLastError();
}
hipError_t launch_relu_bwd(const float* Z, const float* dA, float* dZ, int64_t n, hipStream_t st) {
    hipLaunchKernelGGL(k_relu_bwd, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, Z, dA, dZ, n);
    return hipGetLastError();
}
hipError_t launch_mse(const float* O, const float* T, float* dO, int64_t n, float scale, float* part, hipStream_t st) {
    hipLaunchKernelGGL(k_mse, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, O, T, dO, n, scale, part);
    return hipGetLastError();
}
// part: CS_SPLIT * N floats of scratch
hipError_t launch_colsum(const float* X, int M, int N, float* out, float* part, hipStream_t st) {
    hipLaunchKernelGGL(k_colsum, dim3((N + 63) / 64, CS_SPLIT), dim3(256), 0, st, X, M, N, part);
    hipLaunchKernelGGL(k_colsum_fin, dim3((N + 255) / 256), dim3(256), 0, st, (const float*)part, N, out);
    return hipGetLastError();
}
hipError_t launch_adam(float* w, const float* g, float* m1, float* m2, int64_t n, float lr, float b1, float b2,
                       float eps, float c1, float c2, hipStream_t st) {
    hipLaunchKernelGGL(k_adam, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, w, g, m1, m2, n, lr, b1, b2, eps,
                       c1, c2);
    return hipGetLastError();
}

// ---- the narrow layers (nin <= 16 inputs, nout <= 4 outputs) on VALU -------------
// A GEMM of inner dimension 8 or output width 2 leaves the matrix cores idle and is
// bound by the activations it reads or writes, so these layers are plain loops with the
// tile GEMMs' arithmetic (BF16 operands, FP32 accumulation), fused with the ReLU, the
// ReLU mask of the backward pass and the bias gradients (FP32, as the column sums).
constexpr int NL_MAXIN = 16, NL_MAXOUT = 4, NL_RB = 32;
// the value of x rounded to BF16 (nearest even, the conversion the tile GEMMs use): every
// product operand is rounded as in the matrix-core layers, and the product of two BF16
// values is exact in FP32
__device__ __forceinline__ float bfr(float x) { return __uint_as_float((uint32_t)f32_to_bf16(x) << 16); }

// A1 = relu(X W1 + b1): workgroup -> 64 columns x NL_RB rows; thread -> column c0 + (tid
// & 63), rows q, q + 4, ... of the block (q = tid >> 6); the block's rows of X in LDS
__global__ __launch_bounds__(256) void k_nl_in_fwd(const float* __restrict__ X, const float* __restrict__ W1,
                                                   const float* __restrict__ b1, float* __restrict__ A1, int rows,
                                                   int nin, int h1) {
    __shared__ float xs[NL_RB][NL_MAXIN];
    const int c = blockIdx.x * 64 + (threadIdx.x & 63), q = threadIdx.x >> 6;
    const int rb = blockIdx.y * NL_RB;
    for (int e = threadIdx.x; e < NL_RB * NL_MAXIN; e += 256) {
        const int r = e / NL_MAXIN, k = e % NL_MAXIN;
        xs[r][k] = (rb + r < rows && k < nin) ? bfr(X[(int64_t)(rb + r) * nin + k]) : 0.f;
    }
    __syncthreads();
    if (c >= h1) return;
    float w[NL_MAXIN];
#pragma unroll
    for (int k = 0; k < NL_MAXIN; ++k) w[k] = k < nin ? bfr(W1[(int64_t)k * h1 + c]) : 0.f;
    const float b = b1[c];
    for (int r = q; r < NL_RB && rb + r < rows; r += 4) {
        float v = b;
#pragma unroll
        for (int k = 0; k < NL_MAXIN; ++k) v += xs[r][k] * w[k];
        A1[(int64_t)(rb + r) * h1 + c] = v > 0.f ? v : 0.f;
    }
}
// O = A2 W3 + b3: one wave per row, lanes striding the hidden units
__global__ __launch_bounds__(256) void k_nl_out_fwd(const float* __restrict__ A2, const float* __restrict__ W3,
                                                    const float* __restrict__ b3, float* __restrict__ O, int rows,
                                                    int h2, int nout) {
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (r >= rows) return;
    float acc[NL_MAXOUT] = {0.f, 0.f, 0.f, 0.f};
    for (int i = lane; i < h2; i += 64) {
        const float a = bfr(A2[(int64_t)r * h2 + i]);
#pragma unroll
        for (int j = 0; j < NL_MAXOUT; ++j)
            if (j < nout) acc[j] += a * bfr(W3[(int64_t)i * nout + j]);
    }
#pragma unroll
    for (int j = 0; j < NL_MAXOUT; ++j) {
        float v = acc[j];
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if (j < nout && lane == 0) O[(int64_t)r * nout + j] = v + b3[j];
    }
}
// Output layer backward: dZ2 = (dO W3^T) * [A2 > 0].  Workgroup (bx, by): hidden units
// 64 bx .. 64 bx + 63 over row split `by`; thread -> unit i = 64 bx + (tid & 63) and rows
// q, q + 4, ... of the split (q = tid >> 6).  The four row groups' sums of A2^T dO are
// combined in order in LDS into part[by][i][j]; the column sums of dO (bias gradient) of
// the split go to part[nsplit * h2 * nout + by * nout + j] from the workgroup bx = 0.
__global__ __launch_bounds__(256) void k_nl_out_bwd(const float* __restrict__ A2, const float* __restrict__ dO,
                                                    const float* __restrict__ W3, float* __restrict__ dZ2,
                                                    float* __restrict__ part, int rows, int h2, int nout, int rps) {
    __shared__ float red[4][64][NL_MAXOUT];
    __shared__ float redb[4][64][NL_MAXOUT];
    const int lc = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + lc, by = blockIdx.y, nsplit = gridDim.y;
    const bool on = i < h2;
    float w[NL_MAXOUT], aw[NL_MAXOUT] = {0.f, 0.f, 0.f, 0.f}, ab[NL_MAXOUT] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NL_MAXOUT; ++j) w[j] = (on && j < nout) ? bfr(W3[(int64_t)i * nout + j]) : 0.f;
    const int r0 = by * rps, r1 = min(rows, r0 + rps);
    for (int r = r0 + q; r < r1; r += 4) {
        const float a = on ? A2[(int64_t)r * h2 + i] : 0.f, a16 = bfr(a);
        float d = 0.f;
#pragma unroll
        for (int j = 0; j < NL_MAXOUT; ++j)
            if (j < nout) {
                const float o = dO[(int64_t)r * nout + j], o16 = bfr(o);
                d += o16 * w[j];
                aw[j] += a16 * o16;
                ab[j] += o;
            }
        if (on) dZ2[(int64_t)r * h2 + i] = a > 0.f ? d : 0.f;
    }
#pragma unroll
    for (int j = 0; j < NL_MAXOUT; ++j) {
        red[q][lc][j] = aw[j];
        redb[q][lc][j] = ab[j];
    }
    __syncthreads();
    if (q == 0 && on) {
#pragma unroll
        for (int j = 0; j < NL_MAXOUT; ++j)
            if (j < nout) {
                part[((int64_t)by * h2 + i) * nout + j] = ((red[0][lc][j] + red[1][lc][j]) + red[2][lc][j]) + red[3][lc][j];
                if (i == 0)
                    part[(int64_t)nsplit * h2 * nout + by * nout + j] =
                        ((redb[0][lc][j] + redb[1][lc][j]) + redb[2][lc][j]) + redb[3][lc][j];
            }
    }
}
// Input layer backward: X^T dZ1 (nin x h1) and the column sums of dZ1, per row split, into
// part[by][k][c] (k = nin: the bias row).  Workgroup (bx, by): hidden units 64 bx .. + 63;
// thread -> unit c and rows q, q + 4, ... of the split, combined in order in LDS.
__global__ __launch_bounds__(256) void k_nl_in_bwd(const float* __restrict__ X, const float* __restrict__ dZ1,
                                                   float* __restrict__ part, int rows, int nin, int h1, int rps) {
    __shared__ float red[4][NL_MAXIN + 1][64];
    const int lc = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int c = blockIdx.x * 64 + lc, by = blockIdx.y;
    const bool on = c < h1;
    float acc[NL_MAXIN + 1];
#pragma unroll
    for (int k = 0; k <= NL_MAXIN; ++k) acc[k] = 0.f;
    const int r0 = by * rps, r1 = min(rows, r0 + rps);
    for (int r = r0 + q; r < r1; r += 4) {
        const float d = on ? dZ1[(int64_t)r * h1 + c] : 0.f, d16 = bfr(d);
#pragma unroll
        for (int k = 0; k < NL_MAXIN; ++k)
            if (k < nin) acc[k] += bfr(X[(int64_t)r * nin + k]) * d16;
        acc[NL_MAXIN] += d;
    }
#pragma unroll
    for (int k = 0; k <= NL_MAXIN; ++k) red[q][k][lc] = acc[k];
    __syncthreads();
    if (q != 0 || !on) return;
    float* pb = part + (int64_t)by * (nin + 1) * h1;
#pragma unroll
    for (int k = 0; k <= NL_MAXIN; ++k) {
        const int kk = k < nin ? k : (k == NL_MAXIN ? nin : -1);
        if (kk >= 0) pb[(int64_t)kk * h1 + c] = ((red[0][k][lc] + red[1][k][lc]) + red[2][k][lc]) + red[3][k][lc];
    }
}
// out[e] = sum over the nsplit partial copies (stride n) of part, in a fixed order: four
// thread groups take copies q, q + 4, ... (q = tid >> 6) of 64 consecutive elements,
// combined in order in LDS
__global__ __launch_bounds__(256) void k_nl_sum(const float* __restrict__ part, int nsplit, int64_t n,
                                                float* __restrict__ out) {
    __shared__ float red[4][64];
    const int lc = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int64_t e = (int64_t)blockIdx.x * 64 + lc;
    float v = 0.f;
    if (e < n) {
#pragma unroll 8
        for (int k = q; k < nsplit; k += 4) v += part[(int64_t)k * n + e];
    }
    red[q][lc] = v;
    __syncthreads();
    if (q == 0 && e < n) out[e] = ((red[0][lc] + red[1][lc]) + red[2][lc]) + red[3][lc];
}

// ---- per-coordinate features of a packed uneven batch --------------------------
// One wave per (instance, user): z = h_u^H y / (||h_u||^2 + lambda) (regularised
// matched filter), e = ||h_u||^2.  Row layout (NF = 8 floats):
//   [Re z, Im z, |z|, e, lambda, m/2048, n/m, 1]
template <typename V>
__global__ __launch_bounds__(256) void k_features(const V* __restrict__ H, const V* __restrict__ Y,
                                                  const WgJob* __restrict__ jobs, const int64_t* __restrict__ row_off,
                                                  int njobs, double lambda, float* __restrict__ F) {
    const int lane = threadIdx.x & 63;
    const int64_t gw = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    // locate (job, user) by a binary search over the row offsets
    int lo = 0, hi = njobs;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (row_off[mid] <= gw) lo = mid;
        else hi = mid;
    }
    const WgJob jb = jobs[lo];
    const int64_t u = gw - row_off[lo];
    if (lo >= njobs || u >= jb.n || u < 0) return;
    const V* h = H + jb.h_off + u * jb.ld;
    const V* y = Y + jb.y_off;
    double gr = 0.0, gi = 0.0, e = 0.0;
    for (int i = lane; i < jb.m; i += 64) {
        const V hv = h[i], yv = y[i];
        gr += (double)hv.x * yv.x + (double)hv.y * yv.y;
        gi += (double)hv.x * yv.y - (double)hv.y * yv.x;
        e += (double)hv.x * hv.x + (double)hv.y * hv.y;
    }
    gr = wave_allsum(gr);
    gi = wave_allsum(gi);
    e = wave_allsum(e);
    if (lane == 0) {
        const double den = e + lambda;
        const double zr = den > 0.0 ? gr / den : 0.0, zi = den > 0.0 ? gi / den : 0.0;
        float* f = F + gw * 8;
        f[0] = (float)zr;
        f[1] = (float)zi;
        f[2] = (float)sqrt(zr * zr + zi * zi);
        f[3] = (float)e;
        f[4] = (float)lambda;
        f[5] = (float)jb.m / 2048.f;
        f[6] = (float)jb.n / (float)jb.m;
        f[7] = 1.f;
    }
}

hipError_t launch_features(bool c128, const void* H, const void* Y, const WgJob* jobs, const int64_t* row_off,
                           int njobs, int64_t nrows, double lambda, float* F, hipStream_t st) {
    if (c128)
        hipLaunchKernelGGL(k_features<double2>, dim3((unsigned)((nrows + 3) / 4)), dim3(256), 0, st,
                           (const double2*)H, (const double2*)Y, jobs, row_off, njobs, lambda, F);
    else
        hipLaunchKernelGGL(k_features<float2>, dim3((unsigned)((nrows + 3) / 4)), dim3(256), 0, st, (const float2*)H,
                           (const float2*)Y, jobs, row_off, njobs, lambda, F);
    return hipGetLastError();
}

// (rows x 2) FP32 network output -> interleaved complex warm start
template <typename V>
__global__ void k_out_complex(const float2* __restrict__ O, V* __restrict__ x, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        const float2 o = O[i];
        V v;
        v.x = o.x;
        v.y = o.y;
        x[i] = v;
    }
}

hipError_t launch_out_complex(const float* O, void* x, int64_t n, bool c128, hipStream_t st) {
    const dim3 grid((unsigned)((n + 255) / 256));
    if (c128)
        hipLaunchKernelGGL(k_out_complex<double2>, grid, dim3(256), 0, st, (const float2*)O, (double2*)x, n);
    else
        hipLaunchKernelGGL(k_out_complex<float2>, grid, dim3(256), 0, st, (const float2*)O, (float2*)x, n);
    return hipGetLastError();
}

// ---- the tile product of the fused kernels ----------------------------------------
// acc[i][q] = sum over k of 64 rows in LDS (i: 16 rows each; BF16, k-fastest, row stride LDA) times
// 64 columns of W2 (q: 16 columns each) in NK steps of 32.  W2 comes from memory in fragment
// order ([step][q][lane][8 k], 4 KiB a step), four steps ahead in a ring of registers: a step's
// loads are issued when its slot has been used, and arrive three steps (about 800 cycles)
// later.  The ring holds the steps 0..3 on entry and the first four of `wnext` on return.  ROWS:
// the rows are operand A, so that a lane ends with four rows of one column; else with four
// columns of one row.
constexpr int MT_LD = 8;                             // BF16 row padding: conflict-free b128 reads
typedef bf16x8_t MtRing[4][4];
__device__ __forceinline__ void mt_fetch(bf16x8_t (&f)[4], const bf16x8_t* step) {
    uint32_t o = (uint32_t)(threadIdx.x & 63) * 16;  // scalar base, one offset register
    asm("" : "+v"(o));
#pragma unroll
    for (int q = 0; q < 4; ++q)
        f[q] = *reinterpret_cast<const bf16x8_t*>(reinterpret_cast<const char*>(step) + o + 1024 * q);
}
template <int NK, int LDA, bool ROWS>
__device__ __forceinline__ void mt_product(f32x4_t (&acc)[4][4], MtRing& f, const bf16x8_t* wf, const bf16x8_t* wnext,
                                           const unsigned short* rows) {
    const int lane = threadIdx.x & 63;
    const unsigned short* const ap = rows + (lane & 15) * LDA + 8 * (lane >> 4);
    bf16x8_t a[2][4];
    auto rows_of = [&](int d, int ks) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) a[d][i] = frag8(ap + 16 * i * LDA + 32 * (ks < NK ? ks : 0));
    };
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[i][q] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    rows_of(0, 0);
#pragma unroll 1
    for (int k0 = 0; k0 < NK; k0 += 4) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            // the compiler would gather the loads at the loop's end: this order stands
            rows_of((k + 1) & 1, k0 + k + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    acc[i][q] = ROWS ? mfma32(a[k & 1][i], f[k][q], acc[i][q]) : mfma32(f[k][q], a[k & 1][i], acc[i][q]);
            __builtin_amdgcn_sched_barrier(0);
            mt_fetch(f[k], k0 + 4 < NK ? wf + (k0 + k + 4) * 256 : wnext + k * 256);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}
// Layer 1 of 16 hidden units and 16 rows by the FP32 matrix instruction (16 x 16 x 4), whose sum is
// the chain of fused multiply-adds over k ascending from c.  w: lane -> unit lane & 15, x: lane ->
// row lane & 15, both k = 4 s + (lane >> 4) of step s.
template <int KS> __device__ __forceinline__ f32x4_t mt_layer1(const float (&a)[KS], const float (&b)[KS], f32x4_t c) {
#pragma unroll
    for (int k = 0; k < KS; ++k) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[k], b[k], c, 0, 0, 0);
    return c;
}
template <int KS>
__device__ __forceinline__ void mt_inputs(float (&xb)[4][KS], const float* X, int64_t r0, int64_t rows, int nin) {
    const int l16 = threadIdx.x & 15, grp = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            const int64_t r = r0 + 16 * i + l16;
            const int kk = 4 * k + grp;
            xb[i][k] = bfr((kk < nin && r < rows) ? X[r * nin + kk] : 0.f);   // rows past the end read as 0
        }
}
__device__ __forceinline__ float relu1(float z) { return z > 0.f ? z : 0.f; }

// ---- fused inference (warm-start prediction) -------------------------------------
// One launch evaluates the whole network for a tile of MI_R rows, with the same
// operand rounding as the layered forward pass (BF16 operands, FP32 accumulation):
//   layer 1 (nin <= 16, FP32 MFMA): A1 = relu(bf16(X) bf16(W1) + b1), kept as BF16 in LDS;
//   layer 2 (MFMA 16x16x32): Z2 = A1 bf16(W2) + b2; a wave takes all 64 rows of the columns
//            64 c + 16 wid + 0..15, four blocks c at a time (4 x 4 tiles: a fragment from LDS or
//            from W2 serves four MFMAs), W2 in the order in which its fragments are asked for;
//   layer 3 in the epilogue of each block: Y += bf16(relu(Z2)) bf16(W3), reduced over the
//            slice's 16 columns; the waves' sums are added in a fixed order at the end and
//            written as the complex warm start.
// Only the activations of one tile ever exist, in LDS: nothing but X and x0 touches HBM.
// Bound: the matrix cores and the epilogue's VALU work; two workgroups per CU, so that one's
// runs beside the other's.  262,001 rows, 512 units: 148 us a call (0.93 PFLOP/s); with layer 1 on the
// VALU, rows along the registers and four shuffles a sum 264 us; 128-row tiles whose waves
// took 16 columns each, one LDS fragment per MFMA, 424 us.
constexpr int MI_R = 64;       // rows per workgroup
constexpr int MI_NT = 256;     // 4 waves

// packed inference weights: W1 and W3 as BF16-rounded FP32; W2 as BF16 bits, fragment by
// fragment: [slice of 16 columns in 64][column blocks by four][32 k][block][lane][8 k]
__global__ void k_mlp_pack(const float* __restrict__ w, int nin, int hid, int64_t oW1, int64_t oW2, int64_t oW3,
                           float* __restrict__ w1r, unsigned short* __restrict__ w2f, float* __restrict__ w3r) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < hid * hid / 8) {
        const int lane = i & 63, q = (i >> 6) & 3, nk = hid / 32, ks = (i >> 8) % nk, p = (i >> 8) / nk;
        const int halves = hid / 256, col = 64 * (4 * (p % halves) + q) + 16 * (p / halves) + (lane & 15);
        const float* src = w + oW2 + (int64_t)(32 * ks + 8 * (lane >> 4)) * hid + col;
        uint32_t v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = pack_bf16x2(src[(int64_t)(2 * k) * hid], src[(int64_t)(2 * k + 1) * hid]);
        reinterpret_cast<uint4*>(w2f)[i] = make_uint4(v[0], v[1], v[2], v[3]);
    }
    if (i < nin * hid) w1r[i] = bfr(w[oW1 + i]);
    if (i < hid * 2) w3r[i] = bfr(w[oW3 + i]);
}

template <int HID, int NIN, typename V>
__global__ __launch_bounds__(MI_NT, 2) void k_mlp_infer(const float* __restrict__ X, int64_t rows, int nin,
                                                        const float* __restrict__ w1r, const float* __restrict__ b1,
                                                        const unsigned short* __restrict__ w2f,
                                                        const float* __restrict__ b2, const float* __restrict__ w3r,
                                                        const float* __restrict__ b3, V* __restrict__ x0) {
    constexpr int LDA = HID + MT_LD, NK = HID / 32, PASS = HID / 256, KS = NIN / 4;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    unsigned short* A1 = reinterpret_cast<unsigned short*>(smem_raw);           // [MI_R][LDA]
    float* yp = reinterpret_cast<float*>(A1 + MI_R * LDA);                      // [4 waves][MI_R][2]
    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, grp = lane >> 4;
    const int64_t r0 = (int64_t)blockIdx.x * MI_R;
    // this wave's fragments of W2: HID / 256 passes of HID / 32 steps of four
    const bf16x8_t* const wf = reinterpret_cast<const bf16x8_t*>(w2f) + (int64_t)wid * PASS * NK * 256;
    MtRing f;
    // ---- layer 1: this wave's HID / 4 hidden units of all 64 rows
    {
        float xb[4][KS];
        mt_inputs<KS>(xb, X, r0, rows, nin);
#pragma unroll 4
        for (int m = 0; m < HID / 64; ++m) {
            const int h0 = wid * (HID / 4) + 16 * m;
            float wa[KS];
#pragma unroll
            for (int k = 0; k < KS; ++k) wa[k] = 4 * k + grp < nin ? w1r[(4 * k + grp) * HID + h0 + l16] : 0.f;
            const float4 b = *reinterpret_cast<const float4*>(b1 + h0 + 4 * grp);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f32x4_t z = mt_layer1<KS>(wa, xb[i], f32x4_t{0.f, 0.f, 0.f, 0.f});
                *reinterpret_cast<uint2*>(&A1[(16 * i + l16) * LDA + h0 + 4 * grp]) =
                    make_uint2(pack_bf16x2(relu1(z[0] + b.x), relu1(z[1] + b.y)),
                               pack_bf16x2(relu1(z[2] + b.z), relu1(z[3] + b.w)));
            }
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) mt_fetch(f[k], wf + k * 256);
    __syncthreads();
    // ---- layers 2 and 3
    float y0[4][4], y1[4][4];                        // layer-3 partials of this lane's row 16 i + l16
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) y0[i][r] = y1[i][r] = 0.f;
#pragma unroll 1
    for (int p = 0; p < PASS; ++p) {
        f32x4_t acc[4][4];
        mt_product<NK, LDA, false>(acc, f, wf + p * NK * 256, wf + (p + 1 < PASS ? p + 1 : 0) * NK * 256, A1);
        // epilogue: lane holds Z2[16 i + l16][col .. col + 3]
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int col = 64 * (4 * p + q) + 16 * wid + 4 * grp;
            const float4 bz = *reinterpret_cast<const float4*>(b2 + col);
            const float4 wa = *reinterpret_cast<const float4*>(w3r + 2 * col);
            const float4 wb = *reinterpret_cast<const float4*>(w3r + 2 * col + 4);
            const float bb[4] = {bz.x, bz.y, bz.z, bz.w}, w0[4] = {wa.x, wa.z, wb.x, wb.z}, w1[4] = {wa.y, wa.w, wb.y, wb.w};
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int r = 0; r < 4; r += 2) {
                    const float za = acc[i][q][r] + bb[r], zb = acc[i][q][r + 1] + bb[r + 1];
                    const uint32_t pk = pack_bf16x2(relu1(za), relu1(zb));
                    const float a2 = __uint_as_float(pk << 16), a3 = __uint_as_float(pk & 0xffff0000u);
                    y0[i][r] += a2 * w0[r];
                    y1[i][r] += a2 * w1[r];
                    y0[i][r + 1] += a3 * w0[r + 1];
                    y1[i][r + 1] += a3 * w1[r + 1];
                }
        }
    }
    // sum over the slice's 16 columns (four in this lane, four lanes), then per wave into LDS
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float s0 = (y0[i][0] + y0[i][1]) + (y0[i][2] + y0[i][3]), s1 = (y1[i][0] + y1[i][1]) + (y1[i][2] + y1[i][3]);
        s0 += __shfl_xor(s0, 16);
        s1 += __shfl_xor(s1, 16);
        s0 += __shfl_xor(s0, 32);
        s1 += __shfl_xor(s1, 32);
        if (grp == 0) *reinterpret_cast<float2*>(&yp[(wid * MI_R + 16 * i + l16) * 2]) = make_float2(s0, s1);
    }
    __syncthreads();
    if (tid < MI_R && r0 + tid < rows) {
        float s0 = 0.f, s1 = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            s0 += yp[(w * MI_R + tid) * 2 + 0];
            s1 += yp[(w * MI_R + tid) * 2 + 1];
        }
        V v;
        v.x = s0 + b3[0];
        v.y = s1 + b3[1];
        x0[r0 + tid] = v;
    }
}

// hid in {256, 512}; nin <= 16; nout = 2
hipError_t launch_mlp_infer(const float* w, int nin, int hid, int64_t oW1, int64_t ob1, int64_t oW2, int64_t ob2,
                            int64_t oW3, int64_t ob3, float* w1r, unsigned short* w2f, float* w3r, const float* X,
                            int64_t rows, void* x0, bool c128, hipStream_t st) {
    const int pk = hid * hid / 8;                    // >= nin hid, 2 hid
    hipLaunchKernelGGL(k_mlp_pack, dim3((unsigned)((pk + 255) / 256)), dim3(256), 0, st, w, nin, hid, oW1, oW2, oW3,
                       w1r, w2f, w3r);
    const size_t lds = (size_t)MI_R * (hid + MT_LD) * 2 + 4 * MI_R * 2 * 4;
    const dim3 grid((unsigned)((rows + MI_R - 1) / MI_R));
#define CDM_MI_LAUNCH(H_, N_, V_)                                                                                    do {                                                                                                                 hipError_t e_ = hipFuncSetAttribute((const void*)k_mlp_infer<H_, N_, V_>,                                                                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);                       if (e_ != hipSuccess) return e_;                                                                                 hipLaunchKernelGGL((k_mlp_infer<H_, N_, V_>), grid, dim3(MI_NT), lds, st, X, rows, nin, w1r, w + ob1,                               w2f, w + ob2, w3r, w + ob3, (V_*)x0);                                                     } while (0)
#define CDM_MI_TYPE(H_, N_)                                                                                          do {                                                                                                                 if (c128) CDM_MI_LAUNCH(H_, N_, double2);                                                                        else CDM_MI_LAUNCH(H_, N_, float2);                                                                          } while (0)
    if (hid == 512 && nin <= 8) CDM_MI_TYPE(512, 8);
    else if (hid == 512) CDM_MI_TYPE(512, 16);
    else if (hid == 256 && nin <= 8) CDM_MI_TYPE(256, 8);
    else if (hid == 256) CDM_MI_TYPE(256, 16);
    else return hipErrorInvalidValue;
#undef CDM_MI_TYPE
#undef CDM_MI_LAUNCH
    return hipGetLastError();
}

// ---- fused training pass ------------------------------------------------------------
// Everything of one step that stays within a row, for a tile of 64 rows and HID / 64 waves: the
// forward pass, the error and its gradient, dZ2, dZ1 and the tile's sums for W1, b1, b2, W3 and b3.
// The operands and sums are those of the layered pass (BF16 operands, FP32 accumulation, each
// layer's chain in the same order); no activation is read back from HBM.  For the one product
// over rows, W2's gradient (k_mlp_dw), the tile leaves A1 and dZ2 as BF16 fragments over 32 rows:
// lane -> unit lane & 15, its 8 values the rows 4 g .. 4 g + 3 of both 16-row halves (g = lane >> 4),
// which is how the matrix instructions leave them; both operands are in this order.
// Layers:
//   1   twice on FP32 MFMA: a lane's four units of a row for LDS, four rows of a unit for the
//       fragments (cheaper than transposing);
//   2   as in k_mlp_infer; W2's columns are dealt to waves and tiles so that a lane meets the
//       columns congruent mod 64 one after the other, the order of the layered output layer;
//   3   the 64 partial sums of a row over LDS, one thread per row and output;
//   dZ2 two columns per thread: LDS (in place of A2), fragments, sums of dZ2 and A2^T dO;
//   dZ1 the second product; its four rows per lane are at once an operand of X^T dZ1
//       (16 x 16 x 16 MFMA).
// LDS (512 units: 140 KB) allows one workgroup per CU: bound by the latency of its phases (28 % of
// its cycles in MFMA).  16,384 rows, 512 units: 33 us, in the place of ten launches of 226 us.
typedef short bf16x4s_t __attribute__((ext_vector_type(4)));
constexpr int MTR_R = 64, MTR_Y = 68;   // rows per tile; row stride of layer 3's partial sums
// offsets in a tile's sums: W1 and b1, b2, W3, b3
__host__ __device__ inline int mtr_sums(int nin, int hid) { return (nin + 1) * hid + hid + 2 * hid + 2; }
// bytes of LDS for A2, which the partial sums of layer 3 use first
template <int HID> constexpr int mtr_a2() { return HID == 512 ? 2 * MTR_R * (HID + MT_LD) : 8 * MTR_R * MTR_Y; }
// first column of pair h (registers 2 h, 2 h + 1) of lane group g, tile q, wave w
template <int HID> __device__ __forceinline__ int mtr_col(int w, int q, int g, int h) {
    return HID == 512 ? 64 * (2 * q + h) + 8 * w + 2 * g : 64 * q + 16 * w + 4 * g + 2 * h;
}

// W1 and W3 rounded; W2 in fragment order of the forward (w2f: A operand, columns of mtr_col) and
// backward (w2b: B operand, units 64 w + 16 q + (lane & 15)) products: [w][step][q][lane][8]
template <int HID>
__global__ __launch_bounds__(256) void k_mlp_pack_train(const float* __restrict__ w, int nin, int64_t oW1, int64_t oW2,
                                                        int64_t oW3, float* __restrict__ w1r,
                                                        unsigned short* __restrict__ w2f,
                                                        unsigned short* __restrict__ w2b, float* __restrict__ w3r) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < HID * HID / 8) {
        const int lane = i & 63, q = (i >> 6) & 3, ks = (i >> 8) % (HID / 32), wv = (i >> 8) / (HID / 32);
        const int m = lane & 15, k = 32 * ks + 8 * (lane >> 4);
        const int col = mtr_col<HID>(wv, q, m >> 2, (m & 3) >> 1) + (m & 1);
        const float* src = w + oW2 + (int64_t)k * HID + col;
        uint32_t v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = pack_bf16x2(src[(2 * j) * HID], src[(2 * j + 1) * HID]);
        reinterpret_cast<uint4*>(w2f)[i] = make_uint4(v[0], v[1], v[2], v[3]);
        const float* row = w + oW2 + (int64_t)(64 * wv + 16 * q + m) * HID + k;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = pack_bf16x2(row[2 * j], row[2 * j + 1]);
        reinterpret_cast<uint4*>(w2b)[i] = make_uint4(v[0], v[1], v[2], v[3]);
    }
    if (i < nin * HID) w1r[i] = bfr(w[oW1 + i]);
    if (i < 2 * HID) w3r[i] = bfr(w[oW3 + i]);
}

template <int HID, int NIN>
__global__ __launch_bounds__(HID, 1) void k_mlp_train(const float* __restrict__ X, const float* __restrict__ Tg, int rows,
                                                      int nin, float scale, const float* __restrict__ w1r,
                                                      const float* __restrict__ b1,
                                                      const unsigned short* __restrict__ w2f,
                                                      const unsigned short* __restrict__ w2b,
                                                      const float* __restrict__ b2, const float* __restrict__ w3r,
                                                      const float* __restrict__ b3, uint4* __restrict__ a1f,
                                                      uint4* __restrict__ dzf, float* __restrict__ sums,
                                                      float* __restrict__ sq) {
    constexpr int LDA = HID + MT_LD, NK = HID / 32, KS = NIN / 4, NT = HID / 16, NY = HID == 512 ? 2 : 4;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    unsigned short* A1 = reinterpret_cast<unsigned short*>(smem_raw);           // [64][LDA]
    unsigned short* A2 = A1 + MTR_R * LDA;                                      // [64][LDA]: A2, then dZ2
    float* ys = reinterpret_cast<float*>(A2);                                   // [2][64][MTR_Y], before A2
    float* o16 = reinterpret_cast<float*>(smem_raw + 2 * MTR_R * LDA + mtr_a2<HID>());   // [64][2] dO as BF16
    float* half = o16 + 2 * MTR_R;                                              // [6][HID / 2]
    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, grp = lane >> 4;
    const int64_t r0 = (int64_t)blockIdx.x * MTR_R;
    float* const my = sums + (int64_t)blockIdx.x * mtr_sums(nin, HID);
    const bf16x8_t* const wf = reinterpret_cast<const bf16x8_t*>(w2f) + wid * NK * 256;
    const bf16x8_t* const wb = reinterpret_cast<const bf16x8_t*>(w2b) + wid * NK * 256;
    MtRing f;
#pragma unroll
    for (int k = 0; k < 4; ++k) mt_fetch(f[k], wf + k * 256);
    // ---- layer 1: units 64 wid .. + 63
    {
        float xb[4][KS];
        mt_inputs<KS>(xb, X, r0, rows, nin);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int h0 = 64 * wid + 16 * m;
            float wa[KS];
#pragma unroll
            for (int k = 0; k < KS; ++k) wa[k] = 4 * k + grp < nin ? w1r[(4 * k + grp) * HID + h0 + l16] : 0.f;
            const float4 b = *reinterpret_cast<const float4*>(b1 + h0 + 4 * grp);
            const float bl = b1[h0 + l16];
            uint32_t fr[4][2];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f32x4_t z = mt_layer1<KS>(wa, xb[i], f32x4_t{b.x, b.y, b.z, b.w});
                *reinterpret_cast<uint2*>(&A1[(16 * i + l16) * LDA + h0 + 4 * grp]) =
                    make_uint2(pack_bf16x2(relu1(z[0]), relu1(z[1])), pack_bf16x2(relu1(z[2]), relu1(z[3])));
                const f32x4_t v = mt_layer1<KS>(xb[i], wa, f32x4_t{bl, bl, bl, bl});
                fr[i][0] = pack_bf16x2(relu1(v[0]), relu1(v[1]));
                fr[i][1] = pack_bf16x2(relu1(v[2]), relu1(v[3]));
            }
#pragma unroll
            for (int I = 0; I < 2; ++I)
                a1f[((int64_t)(2 * blockIdx.x + I) * NT + 4 * wid + m) * 64 + lane] =
                    make_uint4(fr[2 * I][0], fr[2 * I][1], fr[2 * I + 1][0], fr[2 * I + 1][1]);
        }
    }
    __syncthreads();
    // ---- layer 2, and the partial sums of layer 3
    f32x4_t acc[4][4];
    mt_product<NK, LDA, false>(acc, f, wf, wb, A1);
    uint32_t a2[4][4][2];
    {
        float y[2][4][NY];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int r = 0; r < NY; ++r) y[0][i][r] = y[1][i][r] = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int col = mtr_col<HID>(wid, q, grp, h), c = NY == 2 ? 0 : 2 * h;
                const float2 bz = *reinterpret_cast<const float2*>(b2 + col);
                const float4 wo = *reinterpret_cast<const float4*>(w3r + 2 * col);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t pk = pack_bf16x2(relu1(acc[i][q][2 * h] + bz.x), relu1(acc[i][q][2 * h + 1] + bz.y));
                    const float u = __uint_as_float(pk << 16), v = __uint_as_float(pk & 0xffff0000u);
                    y[0][i][c] += u * wo.x;
                    y[1][i][c] += u * wo.y;
                    y[0][i][c + 1] += v * wo.z;
                    y[1][i][c + 1] += v * wo.w;
                    a2[i][q][h] = pk;
                }
            }
        const int res = HID == 512 ? 8 * wid + 2 * grp : 16 * wid + 4 * grp;     // column mod 64
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int r = 0; r < NY; r += 2)
                    *reinterpret_cast<float2*>(&ys[(j * MTR_R + 16 * i + l16) * MTR_Y + res + r]) =
                        make_float2(y[j][i][r], y[j][i][r + 1]);
    }
    __syncthreads();
    // ---- layer 3, the error and its gradient: thread -> row lane, output wid
    if (wid < 2) {
        float v[64];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const float4 t = *reinterpret_cast<const float4*>(&ys[(wid * MTR_R + lane) * MTR_Y + 4 * k]);
            v[4 * k] = t.x;
            v[4 * k + 1] = t.y;
            v[4 * k + 2] = t.z;
            v[4 * k + 3] = t.w;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
#pragma unroll
            for (int k = 0; k < o; ++k) v[k] += v[k + o];
        const int64_t e = (r0 + lane) * 2 + wid;
        const bool in = r0 + lane < rows;
        const float d = in ? (v[0] + b3[wid]) - Tg[e] : 0.f;
        const float g = 2.f * d * scale;
        if (in) sq[e] = d * d;
        o16[2 * lane + wid] = bfr(g);
        const float t = wave_allsum(g);
        if (lane == 0) my[(nin + 1) * HID + 3 * HID + wid] = t;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                *reinterpret_cast<uint32_t*>(&A2[(16 * i + l16) * LDA + mtr_col<HID>(wid, q, grp, h)]) = a2[i][q][h];
    __syncthreads();
    // ---- dZ2 = (dO W3^T) [A2 > 0]: thread -> columns c, c + 1 of the 32 rows of half I
    {
        const int c = 2 * (tid % (HID / 2)), I = tid / (HID / 2);
        const float4 wo = *reinterpret_cast<const float4*>(w3r + 2 * c);
        float cs0 = 0.f, cs1 = 0.f, aw[4] = {0.f, 0.f, 0.f, 0.f};
        uint4* const out = dzf + ((int64_t)(2 * blockIdx.x + I) * NT + c / 16) * 64 + c % 16;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            uint32_t p0[4], p1[4];
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                float d0[2], d1[2];
                const int row = 32 * I + (e < 4 ? 4 * g + e : 12 + 4 * g + e);
                unsigned short* const at = &A2[row * LDA + c];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const uint32_t u = *reinterpret_cast<const uint32_t*>(at + t * LDA);
                    const float a = __uint_as_float(u << 16), b = __uint_as_float(u & 0xffff0000u);
                    const float2 o = *reinterpret_cast<const float2*>(&o16[2 * (row + t)]);
                    const float da = o.x * wo.x + o.y * wo.y, db = o.x * wo.z + o.y * wo.w;
                    d0[t] = a > 0.f ? da : 0.f;
                    d1[t] = b > 0.f ? db : 0.f;
                    cs0 += d0[t];
                    cs1 += d1[t];
                    aw[0] += a * o.x;
                    aw[1] += a * o.y;
                    aw[2] += b * o.x;
                    aw[3] += b * o.y;
                }
                p0[e / 2] = pack_bf16x2(d0[0], d0[1]);
                p1[e / 2] = pack_bf16x2(d1[0], d1[1]);
                *reinterpret_cast<uint32_t*>(at) = (p0[e / 2] & 0xffffu) | (p1[e / 2] << 16);
                *reinterpret_cast<uint32_t*>(at + LDA) = (p0[e / 2] >> 16) | (p1[e / 2] & 0xffff0000u);
            }
            out[16 * g] = make_uint4(p0[0], p0[1], p0[2], p0[3]);
            out[16 * g + 1] = make_uint4(p1[0], p1[1], p1[2], p1[3]);
        }
        float s[6] = {cs0, cs1, aw[0], aw[1], aw[2], aw[3]};
        if (I == 1) {
#pragma unroll
            for (int k = 0; k < 6; ++k) half[k * (HID / 2) + c / 2] = s[k];
        }
        __syncthreads();
        if (I == 0) {
#pragma unroll
            for (int k = 0; k < 6; ++k) s[k] += half[k * (HID / 2) + c / 2];
            float* const p = my + (nin + 1) * HID;
            p[c] = s[0];
            p[c + 1] = s[1];
#pragma unroll
            for (int k = 0; k < 4; ++k) p[HID + 2 * c + k] = s[2 + k];
        }
    }
    // ---- dZ1 = (dZ2 W2^T) [A1 > 0], X^T dZ1 and the column sums
    mt_product<NK, LDA, true>(acc, f, wb, wb, A2);
    bf16x4s_t xt[4];                                 // X^T: input l16, rows 16 i + 4 grp + 0..3
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int64_t r = r0 + 16 * i + 4 * grp + e;
            x[e] = (l16 < nin && r < rows) ? X[r * nin + l16] : 0.f;
        }
        const uint2 u = make_uint2(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]));
        xt[i] = __builtin_bit_cast(bf16x4s_t, u);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int hu = 64 * wid + 16 * q + l16;
        f32x4_t dw = {0.f, 0.f, 0.f, 0.f};
        float cs = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                v[r] = A1[(16 * i + 4 * grp + r) * LDA + hu] ? acc[i][q][r] : 0.f;
                cs += v[r];
            }
            const uint2 u = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
            dw = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(xt[i], __builtin_bit_cast(bf16x4s_t, u), dw, 0, 0, 0);
        }
        cs += __shfl_xor(cs, 16);
        cs += __shfl_xor(cs, 32);
        if (grp == 0) my[nin * HID + hu] = cs;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (4 * grp + r < nin) my[(4 * grp + r) * HID + hu] = dw[r];
    }
}

// W2's gradient A1^T dZ2 from the fragments: 128 x 128 tile per workgroup (four waves of 64 x 64),
// blocks [z per, z per + per) of 32 rows into part + z HID^2.  The fragments are read as they lie,
// without LDS: 8 KiB for 16 MFMAs of a wave, half of them hits of the L1 (its other row or
// column of waves).  Bound by fetching the fragments from the MALL: 16,384 rows, 512 units 16 us
// (20 us with a split's tiles spread over the XCDs; 60 us from FP32 activations through LDS).
template <int HID>
__global__ __launch_bounds__(256, 1) void k_mlp_dw(const bf16x8_t* __restrict__ a1f, const bf16x8_t* __restrict__ dzf,
                                                   int nblk, int per, float* __restrict__ part) {
    constexpr int NT = HID / 16, TW = HID / 128, RING = 4;
    // workgroups go to the 8 XCDs in turn: the tiles of a split stay on one, whose L2 holds its rows
    const int tile = (blockIdx.x / 8) % (TW * TW), z = blockIdx.x % 8 + 8 * (blockIdx.x / (8 * TW * TW));
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m0 = 128 * (tile / TW) + 64 * (wid >> 1), n0 = 128 * (tile % TW) + 64 * (wid & 1);
    const int k0 = z * per, k1 = min(nblk, k0 + per);
    if (k0 >= k1) return;
    bf16x8_t a[RING][4], b[RING][4];
    auto fetch = [&](int s, int k) __attribute__((always_inline)) {
        k = k < k1 ? k : k1 - 1;
        mt_fetch(a[s], a1f + ((int64_t)k * NT + m0 / 16) * 64);
        mt_fetch(b[s], dzf + ((int64_t)k * NT + n0 / 16) * 64);
    };
    f32x4_t acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[i][q] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto mma = [&](int s) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[i][q] = mfma32(a[s][i], b[s][q], acc[i][q]);
    };
#pragma unroll
    for (int s = 0; s < RING; ++s) fetch(s, k0 + s);
    int k = k0;
#pragma unroll 1
    for (; k + RING <= k1; k += RING) {
#pragma unroll
        for (int s = 0; s < RING; ++s) {
            mma(s);
            __builtin_amdgcn_sched_barrier(0);
            fetch(s, k + s + RING);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int s = 0; s < RING; ++s)
        if (k + s < k1) mma(s);
    float* const out = part + (int64_t)z * HID * HID;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                out[(m0 + 16 * i + 4 * (lane >> 4) + r) * HID + n0 + 16 * q + (lane & 15)] = acc[i][q][r];
}

// Finish: the sums over tiles and splits in order into g (and grads), and the squared errors by
// 256 into parts (and loss).  Blocks: hh / 1024 for W2 (four values a thread), then the tiles'
// sums (64 values, four threads each), then the errors.
__global__ __launch_bounds__(256) void k_mlp_finish(const float* __restrict__ part, int nsplit, int hh,
                                                    const float* __restrict__ sums, int ntile, int nsum, int n1,
                                                    const float* __restrict__ sq, int nsq, float* __restrict__ g,
                                                    float* __restrict__ grads, float* __restrict__ parts,
                                                    float* __restrict__ loss) {
    __shared__ float red[256];
    const int tid = threadIdx.x;
    int blk = blockIdx.x;
    if (blk < hh / 1024) {
        const int e = 1024 * blk + 4 * tid;
        float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
        for (int z = 0; z < nsplit; ++z) {
            const float4 v = *reinterpret_cast<const float4*>(part + (int64_t)z * hh + e);
            s.x += v.x;
            s.y += v.y;
            s.z += v.z;
            s.w += v.w;
        }
        const float o[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            g[n1 + e + k] = o[k];
            if (grads) grads[n1 + e + k] = o[k];
        }
        return;
    }
    blk -= hh / 1024;
    if (blk < (nsum + 63) / 64) {
        const int e = 64 * blk + (tid & 63), q = tid >> 6;
        float v = 0.f;
        if (e < nsum) {
#pragma unroll 8
            for (int k = q; k < ntile; k += 4) v += sums[(int64_t)k * nsum + e];
        }
        red[tid] = v;
        __syncthreads();
        if (q == 0 && e < nsum) {
            const float s = ((red[tid] + red[64 + tid]) + red[128 + tid]) + red[192 + tid];
            const int at = e < n1 ? e : e + hh;      // W2 stands between b1 and b2
            g[at] = s;
            if (grads) grads[at] = s;
        }
        return;
    }
    blk -= (nsum + 63) / 64;
    const int e = 256 * blk + tid;
    red[tid] = e < nsq ? sq[e] : 0.f;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (tid < k) red[tid] += red[tid + k];
        __syncthreads();
    }
    if (tid == 0) {
        parts[blk] = red[0];
        if (loss) loss[blk] = red[0];
    }
}

struct MlpTrain {
    const float* w;
    int nin, hid, rows;
    int64_t oW1, ob1, oW2, ob2, oW3, ob3;
    float *w1r, *w3r;
    unsigned short *w2f, *w2b;
    const float *X, *T;
    void *a1f, *dzf;              // rows rounded up to 64, times hid, BF16
    float *sums, *sq;             // tiles x mtr_sums, rows x 2
    float* part;                  // nsplit x hid^2
    int nsplit;
    float *g, *grads, *parts, *loss;
};
// Splits of the rows for W2's gradient: workgroups for all CUs, at least four blocks of 32
// rows each (a split costs hid^2 floats written and read again)
int mlp_train_splits_max(int rows, int hid) {
    const int tiles = (hid / 128) * (hid / 128), nblk = 2 * ((rows + MTR_R - 1) / MTR_R);
    return std::max(1, std::min(256 / tiles, nblk / 4));
}
int mlp_train_splits(int rows, int hid) {
    const int nblk = 2 * ((rows + MTR_R - 1) / MTR_R), s = mlp_train_splits_max(rows, hid);
    const int per = (nblk + s - 1) / s;
    return (nblk + per - 1) / per;
}
template <int HID, int NIN> static hipError_t mlp_train_t(const MlpTrain& t, hipStream_t st) {
    const int nt = (t.rows + MTR_R - 1) / MTR_R, nblk = 2 * nt, per = (nblk + t.nsplit - 1) / t.nsplit;
    const int hh = HID * HID, nsum = mtr_sums(t.nin, HID), nsq = 2 * t.rows;
    const size_t lds = (size_t)MTR_R * (HID + MT_LD) * 2 + mtr_a2<HID>() + 8 * MTR_R + 12 * HID;
    hipError_t e = hipFuncSetAttribute((const void*)k_mlp_train<HID, NIN>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_mlp_pack_train<HID>, dim3(hh / 2048), dim3(256), 0, st, t.w, t.nin, t.oW1, t.oW2, t.oW3, t.w1r,
                       t.w2f, t.w2b, t.w3r);
    hipLaunchKernelGGL((k_mlp_train<HID, NIN>), dim3(nt), dim3(HID), lds, st, t.X, t.T, t.rows, t.nin,
                       1.f / (float)((int64_t)t.rows * 2), (const float*)t.w1r, t.w + t.ob1,
                       (const unsigned short*)t.w2f, (const unsigned short*)t.w2b, t.w + t.ob2, (const float*)t.w3r,
                       t.w + t.ob3, (uint4*)t.a1f, (uint4*)t.dzf, t.sums, t.sq);
    hipLaunchKernelGGL(k_mlp_dw<HID>, dim3((HID / 128) * (HID / 128) * ((t.nsplit + 7) / 8 * 8)), dim3(256), 0,
                       st,
                       (const bf16x8_t*)t.a1f, (const bf16x8_t*)t.dzf, nblk, per, t.part);
    hipLaunchKernelGGL(k_mlp_finish, dim3(hh / 1024 + (nsum + 63) / 64 + (nsq + 255) / 256), dim3(256), 0, st,
                       (const float*)t.part, t.nsplit, hh, (const float*)t.sums, nt, nsum, (t.nin + 1) * HID,
                       (const float*)t.sq, nsq, t.g, t.grads, t.parts, t.loss);
    return hipGetLastError();
}
hipError_t launch_mlp_train(const MlpTrain& t, hipStream_t st) {
    if (t.hid == 512) return t.nin <= 8 ? mlp_train_t<512, 8>(t, st) : mlp_train_t<512, 16>(t, st);
    if (t.hid == 256) return t.nin <= 8 ? mlp_train_t<256, 8>(t, st) : mlp_train_t<256, 16>(t, st);
    return hipErrorInvalidValue;
}

}  // namespace cdm

// ============================================================================
// C ABI of the warm-start MLP (host side)
// ============================================================================
namespace {
struct Mlp {
    int nin, h1, h2, nout, max_rows;
    int64_t nparam;
    float *w = nullptr, *g = nullptr, *m1 = nullptr, *m2 = nullptr;
    float *Z1, *A1, *Z2, *A2, *O, *dO, *dA2, *dZ2, *dA1, *dZ1, *part;
    float* cpart = nullptr;                   // column-sum partials (CS_SPLIT x widest layer)
    float* splitk = nullptr;                  // split-K partial products of the weight gradients
    int64_t splitk_floats = 0;
    float *w1r = nullptr, *w3r = nullptr;     // fused kernels: BF16-rounded W1, W3
    unsigned short *w2f = nullptr, *w2b = nullptr;   // and W2 as BF16 in fragment order
    bool fused = false;                       // shape served by k_mlp_infer and k_mlp_train
    void* ws = nullptr;
    int64_t step = 0;
    // parameter block offsets: W1 b1 W2 b2 W3 b3
    int64_t oW1, ob1, oW2, ob2, oW3, ob3;
};
thread_local char g_mlp_err[256] = "";
}  // namespace

struct cdm_mlp : Mlp {};

using namespace cdm;

#define MLP_TRY(call)                                                                       \
    do {                                                                                    \
        hipError_t e_ = (call);                                                             \
        if (e_ != hipSuccess) {                                                             \
            snprintf(g_mlp_err, sizeof(g_mlp_err), "%s: %s", #call, hipGetErrorString(e_)); \
            return CDM_EHIP;                                                                \
        }                                                                                   \
    } while (0)

// The narrow-layer path (nin <= 16, nout <= 4): the input and output layers on the
// kernels above, the hidden layer's ReLU in its GEMM's epilogue, and the ReLU masks of
// the backward pass taken from the activations (A > 0 exactly where Z > 0), so Z1 and Z2
// are not formed; their buffers hold the split partials of the weight gradients.
static bool mlp_narrow(const cdm_mlp* n) { return n->nin <= NL_MAXIN && n->nout <= NL_MAXOUT; }
static int mlp_splits(int rows, int64_t per_split, int64_t cap) {
    // row splits for the gradient partials (64 rows each, at most 256), within `cap`
    // floats of scratch
    int64_t s = std::min<int64_t>(256, std::max<int64_t>(1, rows / 64));
    s = std::min<int64_t>(s, std::max<int64_t>(1, cap / per_split));
    return (int)s;
}

static hipError_t mlp_forward(cdm_mlp* n, const float* X, int rows, hipStream_t st) {
    hipError_t e;
    float* w = n->w;
    if (mlp_narrow(n)) {
        hipLaunchKernelGGL(k_nl_in_fwd, dim3((n->h1 + 63) / 64, (rows + NL_RB - 1) / NL_RB), dim3(256), 0, st, X,
                           (const float*)(w + n->oW1), (const float*)(w + n->ob1), n->A1, rows, n->nin, n->h1);
        if ((e = hipGetLastError())) return e;
        if ((e = launch_gemm_bf16(n->A1, n->h1, 1, w + n->oW2, n->h2, 1, n->A2, n->h2, rows, n->h2, n->h1, w + n->ob2, 0, st,
                                  n->splitk, n->splitk_floats, 1, nullptr)))
            return e;
        hipLaunchKernelGGL(k_nl_out_fwd, dim3((rows + 3) / 4), dim3(256), 0, st, (const float*)n->A2,
                           (const float*)(w + n->oW3), (const float*)(w + n->ob3), n->O, rows, n->h2, n->nout);
        return hipGetLastError();
    }
    if ((e = launch_gemm_bf16(X, n->nin, 1, w + n->oW1, n->h1, 1, n->Z1, n->h1, rows, n->h1, n->nin, w + n->ob1, 0, st, n->splitk, n->splitk_floats)))
        return e;
    if ((e = launch_relu(n->Z1, n->A1, (int64_t)rows * n->h1, st))) return e;
    if ((e = launch_gemm_bf16(n->A1, n->h1, 1, w + n->oW2, n->h2, 1, n->Z2, n->h2, rows, n->h2, n->h1, w + n->ob2, 0, st, n->splitk, n->splitk_floats)))
        return e;
    if ((e = launch_relu(n->Z2, n->A2, (int64_t)rows * n->h2, st))) return e;
    return launch_gemm_bf16(n->A2, n->h2, 1, w + n->oW3, n->nout, 1, n->O, n->nout, rows, n->nout, n->h2, w + n->ob3,
                            0, st, n->splitk, n->splitk_floats);
}

// gradients of the mean squared error (1 / (rows * nout)) sum (O - T)^2 into n->g
static hipError_t mlp_backward(cdm_mlp* n, const float* X, const float* T, int rows, hipStream_t st) {
    hipError_t e;
    float* w = n->w;
    float* g = n->g;
    const int64_t no = (int64_t)rows * n->nout;
    if ((e = launch_mse(n->O, T, n->dO, no, 1.f / (float)no, n->part, st))) return e;
    if (mlp_narrow(n)) {
        const int64_t cap3 = (int64_t)n->max_rows * n->h2, cap1 = (int64_t)n->max_rows * n->h1;
        // layer 3: dZ2, the weight and bias gradient partials (scratch: Z2)
        const int s3 = mlp_splits(rows, (int64_t)n->h2 * n->nout + n->nout, cap3);
        const int rps3 = (rows + s3 - 1) / s3;
        hipLaunchKernelGGL(k_nl_out_bwd, dim3((n->h2 + 63) / 64, s3), dim3(256), 0, st, (const float*)n->A2,
                           (const float*)n->dO, (const float*)(w + n->oW3), n->dZ2, n->Z2, rows, n->h2, n->nout, rps3);
        if ((e = hipGetLastError())) return e;
        const int64_t n3 = (int64_t)n->h2 * n->nout;
        hipLaunchKernelGGL(k_nl_sum, dim3((unsigned)((n3 + 63) / 64)), dim3(256), 0, st, (const float*)n->Z2, s3, n3,
                           g + n->oW3);
        hipLaunchKernelGGL(k_nl_sum, dim3(1), dim3(256), 0, st, (const float*)(n->Z2 + (int64_t)s3 * n3), s3,
                           (int64_t)n->nout, g + n->ob3);
        if ((e = hipGetLastError())) return e;
        // layer 2 (matrix cores): weight gradient, bias gradient, dZ1 = (dZ2 W2^T) * [A1 > 0]
        if ((e = launch_gemm_bf16(n->A1, 1, n->h1, n->dZ2, n->h2, 1, g + n->oW2, n->h2, n->h1, n->h2, rows, nullptr, 0, st,
                                  n->splitk, n->splitk_floats)))
            return e;
        if ((e = launch_colsum(n->dZ2, rows, n->h2, g + n->ob2, n->cpart, st))) return e;
        if ((e = launch_gemm_bf16(n->dZ2, n->h2, 1, w + n->oW2, 1, n->h2, n->dZ1, n->h1, rows, n->h1, n->h2, nullptr, 0, st,
                                  n->splitk, n->splitk_floats, 0, n->A1)))
            return e;
        // layer 1: weight and bias gradient partials (scratch: Z1)
        const int s1 = mlp_splits(rows, (int64_t)(n->nin + 1) * n->h1, cap1);
        const int rps1 = (rows + s1 - 1) / s1;
        hipLaunchKernelGGL(k_nl_in_bwd, dim3((n->h1 + 63) / 64, s1), dim3(256), 0, st, X, (const float*)n->dZ1, n->Z1,
                           rows, n->nin, n->h1, rps1);
        if ((e = hipGetLastError())) return e;
        const int64_t n1 = (int64_t)(n->nin + 1) * n->h1;   // W1 (nin x h1) then b1 (h1): contiguous in g
        hipLaunchKernelGGL(k_nl_sum, dim3((unsigned)((n1 + 63) / 64)), dim3(256), 0, st, (const float*)n->Z1, s1, n1,
                           g + n->oW1);
        return hipGetLastError();
    }
    // layer 3
    if ((e = launch_gemm_bf16(n->A2, 1, n->h2, n->dO, n->nout, 1, g + n->oW3, n->nout, n->h2, n->nout, rows, nullptr, 0, st, n->splitk, n->splitk_floats)))
        return e;
    if ((e = launch_colsum(n->dO, rows, n->nout, g + n->ob3, n->cpart, st))) return e;
    if ((e = launch_gemm_bf16(n->dO, n->nout, 1, w + n->oW3, 1, n->nout, n->dA2, n->h2, rows, n->h2, n->nout, nullptr, 0, st, n->splitk, n->splitk_floats)))
        return e;
    if ((e = launch_relu_bwd(n->Z2, n->dA2, n->dZ2, (int64_t)rows * n->h2, st))) return e;
    // layer 2
    if ((e = launch_gemm_bf16(n->A1, 1, n->h1, n->dZ2, n->h2, 1, g + n->oW2, n->h2, n->h1, n->h2, rows, nullptr, 0, st, n->splitk, n->splitk_floats)))
        return e;
    if ((e = launch_colsum(n->dZ2, rows, n->h2, g + n->ob2, n->cpart, st))) return e;
    if ((e = launch_gemm_bf16(n->dZ2, n->h2, 1, w + n->oW2, 1, n->h2, n->dA1, n->h1, rows, n->h1, n->h2, nullptr, 0, st, n->splitk, n->splitk_floats)))
        return e;
    if ((e = launch_relu_bwd(n->Z1, n->dA1, n->dZ1, (int64_t)rows * n->h1, st))) return e;
    // layer 1
    if ((e = launch_gemm_bf16(X, 1, n->nin, n->dZ1, n->h1, 1, g + n->oW1, n->h1, n->nin, n->h1, rows, nullptr, 0, st, n->splitk, n->splitk_floats)))
        return e;
    return launch_colsum(n->dZ1, rows, n->h1, g + n->ob1, n->cpart, st);
}

// Forward and backward pass of one step, gradients into n->g (and grads), squared errors by 256
// into n->part (and loss).  Widths 256 and 512 with two outputs and at most 16 inputs take the
// fused pass at every row count; others the layered one.  Layered / fused, us a call: 512 units,
// 1 row 91 / 35, 1000 rows 205 / 42, 3001 rows 560 / 47, 16,384 rows 338 / 56; 256 units, 1 row
// 62 / 24, 16,384 rows 215 / 41.
static hipError_t mlp_gradients(cdm_mlp* n, const float* X, const float* T, int rows, float* grads, float* loss,
                                hipStream_t st) {
    if (n->fused) {
        MlpTrain t;
        t.w = n->w;
        t.nin = n->nin;
        t.hid = n->h1;
        t.rows = rows;
        t.oW1 = n->oW1;
        t.ob1 = n->ob1;
        t.oW2 = n->oW2;
        t.ob2 = n->ob2;
        t.oW3 = n->oW3;
        t.ob3 = n->ob3;
        t.w1r = n->w1r;
        t.w3r = n->w3r;
        t.w2f = n->w2f;
        t.w2b = n->w2b;
        t.X = X;
        t.T = T;
        t.a1f = n->Z1;
        t.dzf = n->Z2;
        t.sums = n->dA2;
        t.sq = n->O;
        t.part = n->splitk;
        t.nsplit = mlp_train_splits(rows, n->h1);
        t.g = n->g;
        t.grads = grads;
        t.parts = n->part;
        t.loss = loss;
        return launch_mlp_train(t, st);
    }
    hipError_t e;
    if ((e = mlp_forward(n, X, rows, st))) return e;
    if ((e = mlp_backward(n, X, T, rows, st))) return e;
    if (grads && (e = hipMemcpyAsync(grads, n->g, sizeof(float) * n->nparam, hipMemcpyDeviceToDevice, st))) return e;
    if (loss)
        return hipMemcpyAsync(loss, n->part, sizeof(float) * (((size_t)rows * n->nout + 255) / 256),
                              hipMemcpyDeviceToDevice, st);
    return hipSuccess;
}

extern "C" {

int32_t cdm_mlp_create(int32_t nin, int32_t h1, int32_t h2, int32_t nout, int32_t max_rows, cdm_mlp** out) {
    if (!out) return CDM_EINVAL;
    *out = nullptr;
    if (nin < 1 || h1 < 1 || h2 < 1 || nout < 1 || max_rows < 1) return CDM_ESHAPE;
    cdm_mlp* n = new cdm_mlp();
    n->nin = nin;
    n->h1 = h1;
    n->h2 = h2;
    n->nout = nout;
    n->max_rows = max_rows;
    n->oW1 = 0;
    n->ob1 = n->oW1 + (int64_t)nin * h1;
    n->oW2 = n->ob1 + h1;
    n->ob2 = n->oW2 + (int64_t)h1 * h2;
    n->oW3 = n->ob2 + h2;
    n->ob3 = n->oW3 + (int64_t)h2 * nout;
    n->nparam = n->ob3 + nout;
    n->fused = nin <= 16 && h1 == h2 && (h1 == 256 || h1 == 512) && nout == 2;
    // the fused training pass keeps BF16 fragments of whole 64-row tiles in Z1 and Z2
    const int64_t R = max_rows, Rz = n->fused ? (R + MTR_R - 1) / MTR_R * MTR_R : R;
    const int64_t wmax = std::max<int64_t>(std::max(h1, h2), nout);
    // split-K scratch: up to 64 partial copies of the largest weight block
    const int64_t wblk = std::max<int64_t>(std::max<int64_t>((int64_t)nin * h1, (int64_t)h1 * h2), (int64_t)h2 * nout);
    int64_t skf = (R >= 4096) ? std::min<int64_t>(64, R / 256) * wblk : 0;
    if (n->fused) skf = std::max<int64_t>(skf, (int64_t)mlp_train_splits_max(max_rows, h1) * h1 * h2);
    int64_t off = 0;
    auto take = [&](int64_t floats) {   // 16-B aligned sections
        const int64_t o = off;
        off += (floats + 3) / 4 * 4;
        return o;
    };
    const int64_t o_w = take(n->nparam), o_g = take(n->nparam), o_m = take(2 * n->nparam);
    const int64_t o_Z1 = take(Rz * h1), o_A1 = take(R * h1), o_dA1 = take(R * h1), o_dZ1 = take(R * h1);
    const int64_t o_Z2 = take(Rz * h2), o_A2 = take(R * h2), o_dA2 = take(Rz * h2), o_dZ2 = take(R * h2);
    const int64_t o_O = take(R * nout), o_dO = take(R * nout), o_part = take((R * nout + 255) / 256);
    const int64_t o_cpart = take(CS_SPLIT * wmax), o_splitk = take(skf);
    // fused kernels: BF16-rounded W1, W3 (FP32) and W2 in fragment order, forward and backward
    const int64_t o_w1r = take(n->fused ? (int64_t)nin * h1 : 0), o_w3r = take(n->fused ? 2 * (int64_t)h2 : 0);
    const int64_t o_w2f = take(n->fused ? (int64_t)h1 * h2 / 2 : 0), o_w2b = take(n->fused ? (int64_t)h1 * h2 / 2 : 0);
    if (hipMalloc(&n->ws, sizeof(float) * off) != hipSuccess) {
        delete n;
        return CDM_ENOMEM;
    }
    float* p = (float*)n->ws;
    n->w = p + o_w;
    n->g = p + o_g;
    n->m1 = p + o_m;
    n->m2 = n->m1 + n->nparam;
    n->Z1 = p + o_Z1;
    n->A1 = p + o_A1;
    n->dA1 = p + o_dA1;
    n->dZ1 = p + o_dZ1;
    n->Z2 = p + o_Z2;
    n->A2 = p + o_A2;
    n->dA2 = p + o_dA2;
    n->dZ2 = p + o_dZ2;
    n->O = p + o_O;
    n->dO = p + o_dO;
    n->part = p + o_part;
    n->cpart = p + o_cpart;
    n->splitk = skf ? p + o_splitk : nullptr;
    n->splitk_floats = skf;
    if (n->fused) {
        n->w1r = p + o_w1r;
        n->w3r = p + o_w3r;
        n->w2f = reinterpret_cast<unsigned short*>(p + o_w2f);
        n->w2b = reinterpret_cast<unsigned short*>(p + o_w2b);
    }
    if (hipMemset(n->m1, 0, sizeof(float) * 2 * n->nparam) != hipSuccess) {
        (void)hipFree(n->ws);
        delete n;
        return CDM_EHIP;
    }
    *out = n;
    return CDM_OK;
}

int64_t cdm_mlp_param_count(const cdm_mlp* n) { return n ? n->nparam : -1; }

int32_t cdm_mlp_set_weights(cdm_mlp* n, const float* host, int64_t count) {
    if (!n || !host || count != n->nparam) return CDM_EINVAL;
    MLP_TRY(hipMemcpy(n->w, host, sizeof(float) * count, hipMemcpyHostToDevice));
    MLP_TRY(hipMemset(n->m1, 0, sizeof(float) * 2 * n->nparam));
    n->step = 0;
    return CDM_OK;
}

int32_t cdm_mlp_get_weights(const cdm_mlp* n, float* host, int64_t count) {
    if (!n || !host || count != n->nparam) return CDM_EINVAL;
    MLP_TRY(hipMemcpy(host, n->w, sizeof(float) * count, hipMemcpyDeviceToHost));
    return CDM_OK;
}

int32_t cdm_mlp_forward(cdm_mlp* n, const float* X, int32_t rows, float* Y, void* stream) {
    if (!n || !X || rows < 1 || rows > n->max_rows) return CDM_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    MLP_TRY(mlp_forward(n, X, rows, st));
    if (Y) MLP_TRY(hipMemcpyAsync(Y, n->O, sizeof(float) * (size_t)rows * n->nout, hipMemcpyDeviceToDevice, st));
    return CDM_OK;
}

int32_t cdm_mlp_gradients(cdm_mlp* n, const float* X, const float* T, int32_t rows, float* grads, float* loss_parts,
                          void* stream) {
    if (!n || !X || !T || rows < 1 || rows > n->max_rows) return CDM_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    MLP_TRY(mlp_gradients(n, X, T, rows, grads, loss_parts, st));
    return CDM_OK;
}

int32_t cdm_mlp_train_step(cdm_mlp* n, const float* X, const float* T, int32_t rows, float lr, void* stream) {
    if (!n || !X || !T || rows < 1 || rows > n->max_rows || !(lr > 0.f)) return CDM_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    MLP_TRY(mlp_gradients(n, X, T, rows, nullptr, nullptr, st));
    n->step += 1;
    const float b1 = 0.9f, b2 = 0.999f;
    const float c1 = 1.f - powf(b1, (float)n->step), c2 = 1.f - powf(b2, (float)n->step);
    MLP_TRY(launch_adam(n->w, n->g, n->m1, n->m2, n->nparam, lr, b1, b2, 1e-8f, c1, c2, st));
    return CDM_OK;
}

int32_t cdm_mlp_predict(cdm_mlp* n, const float* X, int64_t rows, void* x0, int32_t precision, void* stream) {
    if (!n || !X || !x0 || rows < 1 || n->nout != 2) return CDM_EINVAL;
    if (precision != CDM_C128 && precision != CDM_C64) return CDM_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    const bool c128 = precision == CDM_C128;
    const size_t esz = c128 ? 16 : 8;
    if (n->fused) {   // one launch, activations in LDS only
        MLP_TRY(launch_mlp_infer(n->w, n->nin, n->h1, n->oW1, n->ob1, n->oW2, n->ob2, n->oW3, n->ob3, n->w1r, n->w2f,
                                 n->w3r, X, rows, x0, c128, st));
        return CDM_OK;
    }
    for (int64_t r0 = 0; r0 < rows; r0 += n->max_rows) {
        const int cnt = (int)std::min<int64_t>(n->max_rows, rows - r0);
        MLP_TRY(mlp_forward(n, X + r0 * n->nin, cnt, st));
        MLP_TRY(launch_out_complex(n->O, (char*)x0 + r0 * esz, cnt, c128, st));
    }
    return CDM_OK;
}

int32_t cdm_mlp_destroy(cdm_mlp* n) {
    if (!n) return CDM_OK;
    if (n->ws) (void)hipFree(n->ws);
    delete n;
    return CDM_OK;
}

}  // extern "C"
