// k_gs.hip -- the cyclic sweep of Algorithm 1 on the Gauss-Seidel operator (one instance).
//
// For a panel K of k consecutive users let G = H^H H + lambda I, G_KK = D + L + L^H (D the
// diagonal) and b = H^H (y - H x) - lambda x.  The k sequential updates of the sweep are
// exactly  delta_K = (D + L)^-1 b_K,  and they change b by -G_JK delta_K in every panel J.
// With M_K = (D + L)^-1 and W formed once per solve,
//     W_JK = G_JK M_K (J != K),   W_KK = L^H M_K,
// a panel step is
//     b_J <- b_J - W_JK b_K (J != K),   b_K <- -W_KK b_K,   x_K <- x_K + M_K b_K,
// so the step needs the k values of b_K and nothing of length B: the sweep streams U^2
// values instead of B U, and one exchange of k values per panel is all that couples the
// workgroups.  k is 256 or 512 instead of the 64 or 128 columns whose tiles of H fit the
// registers, so a sweep has a quarter of the exchanges.  Up to 1024 users one panel holds
// all, and the deltas follow each other directly, delta <- V delta with V = -M L^H.  In exact
// arithmetic every delta is the sequential sweep's.
//
// Everything here runs in FP64, for complex64 input too: G from FP32 sums would lose
// digits against the residual form of the sweep, and the FP64 vector and matrix rates of
// gfx950 equal the (unpacked) FP32 vector rate.  So that rounding does not accumulate in b,
// it is formed anew from H, y and x (two passes over H) after sweeps 2, 8, 40 and 200: the
// drift of the first, largest steps is gone by then.
//
// Stages: k_gs_init, k_gs_gram (64 x 64 blocks of the lower triangle, on
// v_mfma_f64_16x16x4_f64), k_gs_assemble (sum of their parts, both triangles), k_gs_inv64 and
// k_gs_mm (the inverse of each D + L by halves, then W or V), and per segment of sweeps
// k_gs_rows (r = y - H x), k_gs_grad (b) and the sweep kernel: k_gs_one (one workgroup, up to
// 128 users), k_gs_delta (up to 1024) or k_gs_sweep.
#include "gs.hpp"
#include "la_common.hpp"

#include <type_traits>

namespace cdm {

namespace {

typedef double acc4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ acc4 mma64(double a, double b, acc4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
template <typename V> __device__ __forceinline__ double2 to_d(V v) {
    return make_double2((double)v.x, (double)v.y);
}

// ---- complex product tiles on the FP64 matrix cores -----------------------------------------
// A wave's 32 x 32 tile (2 x 2 MFMA tiles).  The 16 MFMAs of a step (four values of the
// contraction index) take 1024 cycles and need four operand loads of 1 KiB, so the operands
// come straight from memory, D steps ahead in a ring of registers: no LDS, no barrier.
// Measured against tiles staged through LDS (32 values at a time, two barriers): H^H H of 3000 x
// 1000 262 -> 220 us (57 TFLOP/s), W of 8192 users 1690 -> 1290 us (60 TFLOP/s).
typedef double gs_d2 __attribute__((ext_vector_type(2)));
struct MmAcc {
    acc4 r[2][2], i[2][2];
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                r[a][b] = acc4{0.0, 0.0, 0.0, 0.0};
                i[a][b] = acc4{0.0, 0.0, 0.0, 0.0};
            }
    }
    // += op(A) B over one step; CONJ: op(A) = conj(A)
    template <bool CONJ> __device__ __forceinline__ void step(const double2 (&x)[2], const double2 (&y)[2]) {
        // the two products of an accumulator are kept apart: back to back the second waits
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                r[a][b] = mma64(x[a].x, y[b].x, r[a][b]);
                i[a][b] = mma64(x[a].x, y[b].y, i[a][b]);
            }
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                r[a][b] = mma64(CONJ ? x[a].y : -x[a].y, y[b].y, r[a][b]);
                i[a][b] = mma64(CONJ ? -x[a].y : x[a].y, y[b].x, i[a][b]);
            }
    }
    // steps s0 .. s1 - 1; fetch(s, x, y): this lane's operands of step s (values of index 4 s +
    // (lane >> 4): rows lane & 15 of A's two tiles, columns lane & 15 of B's); mask(s, x, y) looks at
    // them when they are used: in fetch it would wait for the loads
    template <bool CONJ, typename V, class F, class G>
    __device__ __forceinline__ void run(int s0, int s1, F fetch, G mask) {
        constexpr int D = 4;
        if (s0 >= s1) return;
        V x[D][2], y[D][2];
        auto use = [&](int d, int s) __attribute__((always_inline)) {
            double2 u[2] = {to_d(x[d][0]), to_d(x[d][1])}, v[2] = {to_d(y[d][0]), to_d(y[d][1])};
            mask(s, u, v);
            step<CONJ>(u, v);
        };
#pragma unroll
        for (int d = 0; d < D; ++d) fetch(min(s0 + d, s1 - 1), x[d], y[d]);
        int s = s0;
#pragma unroll 1
        for (; s + D <= s1; s += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                use(d, s + d);
                __builtin_amdgcn_sched_barrier(0);
                fetch(min(s + d + D, s1 - 1), x[d], y[d]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (s + d < s1) use(d, s + d);
    }
    // f(row, col, value) for this lane's values of the tile
    template <class F> __device__ __forceinline__ void each(int lane, F f) const {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    f(16 * a + (lane >> 4) + 4 * e, 16 * b + (lane & 15), make_double2(r[a][b][e], i[a][b][e]));
    }
};

__device__ __forceinline__ void lower_block(int n, int& bi, int& bj) {   // n -> (bi, bj), bi >= bj, row by row
    bi = (int)((sqrtf(8.f * (float)n + 1.f) - 1.f) * 0.5f);
    while ((bi + 1) * (bi + 2) / 2 <= n) ++bi;
    while (bi * (bi + 1) / 2 > n) --bi;
    bj = n - bi * (bi + 1) / 2;
}

}  // namespace

// r = y, x = x0 or 0 (FP64, zero past U), and the control and exchange words cleared
template <typename T>
__global__ __launch_bounds__(256) void k_gs_init(const cv<T>* __restrict__ y, const cv<T>* __restrict__ x0, int B,
                                                 int U, int Up, double2* __restrict__ r, double2* __restrict__ x,
                                                 uint64_t* __restrict__ clear, int nclear) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < B) r[i] = to_d(y[i]);
    if (i < Up) x[i] = (x0 && i < U) ? to_d(x0[i]) : make_double2(0.0, 0.0);
    for (int k = i; k < nclear; k += gridDim.x * 256) clear[k] = 0;
}

// The 64 x 64 blocks of the lower triangle of H^H H, a quadrant per wave.  The work, nblk blocks of
// upb steps of 32 rows, is dealt out evenly: workgroup w takes steps [w n / nw, (w + 1) n / nw)
// of all n = nblk upb, and leaves its part of block m at place w + m.  Neighbours in this
// order, which share columns of H, go to one XCD (workgroups go to the 8 XCDs in turn).
__host__ __device__ inline int64_t gram_first(int w, int64_t n, int nw) { return w * n / nw; }
__host__ __device__ inline int gram_owner(int64_t step, int64_t n, int nw) {   // the workgroup of a step
    int w = (int)((step * nw) / n);
    while (w + 1 < nw && gram_first(w + 1, n, nw) <= step) ++w;
    while (gram_first(w, n, nw) > step) --w;
    return w;
}
template <typename T>
__global__ __launch_bounds__(256, 2) void k_gs_gram(const cv<T>* __restrict__ H, int64_t ld, int B, int U, int nblk,
                                                    double2* __restrict__ gpart) {
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = gridDim.x, upb = (B + 31) / 32;
    const int64_t n = (int64_t)nblk * upb;
    const int w = nw % 8 == 0 ? (blockIdx.x % 8) * (nw / 8) + blockIdx.x / 8 : blockIdx.x;
    const int64_t last = gram_first(w + 1, n, nw);
    for (int64_t at = gram_first(w, n, nw); at < last;) {
        const int m = (int)(at / upb), u0 = (int)(at % upb), u1 = (int)min((int64_t)upb, u0 + last - at);
        int bi, bj;
        lower_block(m, bi, bj);
        const int ci = bi * 64 + 32 * (wv >> 1) + (lane & 15), cj = bj * 64 + 32 * (wv & 1) + (lane & 15);
        // columns past U read the last one: their sums are not stored
        const cv<T>* const pi[2] = {H + (int64_t)min(ci, U - 1) * ld, H + (int64_t)min(ci + 16, U - 1) * ld};
        const cv<T>* const pj[2] = {H + (int64_t)min(cj, U - 1) * ld, H + (int64_t)min(cj + 16, U - 1) * ld};
        MmAcc acc;
        acc.zero();
        const int whole = min(8 * u1, B / 4), end = min(8 * u1, (B + 3) / 4);
        auto fetch = [&](int s, cv<T>(&x)[2], cv<T>(&y)[2]) __attribute__((always_inline)) {
            const int row = 4 * s + (lane >> 4);
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                x[a] = pi[a][row];
                y[a] = pj[a][row];
            }
        };
        acc.template run<true, cv<T>>(8 * u0, whole, fetch, [](int, double2(&)[2], double2(&)[2]) {});
        if (whole < end) {   // the last rows, fewer than four
            const int row = 4 * whole + (lane >> 4);
            double2 x[2], y[2];
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                x[a] = row < B ? to_d(pi[a][row]) : make_double2(0.0, 0.0);
                y[a] = row < B ? to_d(pj[a][row]) : make_double2(0.0, 0.0);
            }
            acc.template step<true>(x, y);
        }
        double2* out = gpart + ((int64_t)w + m) * 4096 + 32 * (wv >> 1) * 64 + 32 * (wv & 1);
        const int ui = bi * 64 + 32 * (wv >> 1), uj = bj * 64 + 32 * (wv & 1);
        acc.each(lane, [&](int i, int j, double2 z) {
            out[i * 64 + j] = (ui + i < U && uj + j < U) ? z : make_double2(0.0, 0.0);
        });
        at += u1 - u0;
    }
}

// A (Up x Up, row-major) = the sum of a block's parts in a fixed order, both triangles (the
// upper as the conjugate of the lower), zero past U.  A workgroup takes 16 rows of a block,
// a thread four of their elements with the loads of four parts in flight.
__global__ __launch_bounds__(256) void k_gs_assemble(const double2* __restrict__ gpart, int nw, int upb, int nblk,
                                                     int Up, double2* __restrict__ A) {
    __shared__ double2 t[16][65];
    int bi, bj;
    lower_block(blockIdx.x, bi, bj);
    const int i0 = 16 * blockIdx.y;
    double2 s[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) s[m] = make_double2(0.0, 0.0);
    if ((int)blockIdx.x < nblk) {   // blocks past the last one that holds users are zero
        const int64_t n = (int64_t)nblk * upb, first = (int64_t)blockIdx.x * upb;
        const int w0 = gram_owner(first, n, nw), parts = gram_owner(first + upb - 1, n, nw) - w0 + 1;
        const double2* p = gpart + ((int64_t)w0 + blockIdx.x) * 4096 + i0 * 64 + threadIdx.x;
        int k = 0;
        for (; k + 3 < parts; k += 4) {
            double2 v[4][4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int m = 0; m < 4; ++m) v[q][m] = p[(int64_t)(k + q) * 4096 + 256 * m];
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    s[m].x += v[q][m].x;
                    s[m].y += v[q][m].y;
                }
        }
        for (; k < parts; ++k) {
            double2 v[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) v[m] = p[(int64_t)k * 4096 + 256 * m];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                s[m].x += v[m].x;
                s[m].y += v[m].y;
            }
        }
    }
    const int j = threadIdx.x & 63;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const int i = (threadIdx.x >> 6) + 4 * m;
        t[i][j] = s[m];
        // a diagonal block's own upper triangle comes from its lower one
        if (bi != bj || j <= i0 + i) A[(int64_t)(bi * 64 + i0 + i) * Up + bj * 64 + j] = s[m];
    }
    __syncthreads();
    const int i = threadIdx.x & 15;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const int c = (threadIdx.x >> 4) + 16 * m;
        const double2 v = t[i][c];
        if (bi != bj || c < i0 + i) A[(int64_t)(bj * 64 + c) * Up + bi * 64 + i0 + i] = make_double2(v.x, -v.y);
    }
}

// The inverse of one 64 x 64 diagonal block of D + L, into M (panels of k x k, row-major) with the
// zeros right of it, and into Mt, its transpose (no zeros: nothing reads them).  Bound by
// latency (a few workgroups): the four 16 x 16 diagonal blocks by substitution, a wave each and
// a lane per column, then the blocks below them a diagonal at a time, X_ij = -X_ii sum_k L_ik
// X_kj, on the matrix cores.
// Inactive coordinates (||h_u||^2 + lambda == 0) get zero rows.
constexpr int IP = 66;   // pitch of the LDS planes
constexpr size_t GS_INV_LDS = (size_t)4 * 64 * IP * 8;
__global__ __launch_bounds__(256) void k_gs_inv64(const double2* __restrict__ A, int Up, int U, int k, double lambda,
                                                  double2* __restrict__ M, double2* __restrict__ Mt,
                                                  uint32_t* __restrict__ status) {
    extern __shared__ __attribute__((aligned(16))) double inv_s[];
    double* Lr = inv_s;
    double* Li = Lr + 64 * IP;
    double* Xr = Li + 64 * IP;
    double* Xi = Xr + 64 * IP;
    __shared__ double rd[64];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int u0 = blockIdx.x * 64;
    const int K = u0 / k, c0 = u0 % k;
    double2* Mk = M + (int64_t)K * k * k + (int64_t)c0 * k;
    if (blockIdx.y > 0) {   // the zeros right of the block, beside its inverse
        const int rest = k - c0 - 64;
        for (int e = (blockIdx.y - 1) * 256 + tid; e < 64 * rest; e += 256 * (gridDim.y - 1))
            Mk[(int64_t)(e / rest) * k + c0 + 64 + e % rest] = make_double2(0.0, 0.0);
        return;
    }
    double2 av[16];
#pragma unroll
    for (int m = 0; m < 16; ++m) av[m] = A[(int64_t)(u0 + (tid >> 6) + 4 * m) * Up + u0 + (tid & 63)];
#pragma unroll
    for (int m = 0; m < 16; ++m) {
        const int i = (tid >> 6) + 4 * m, j = tid & 63;
        const double2 v = av[m];
        Lr[i * IP + j] = j < i ? v.x : 0.0;
        Li[i * IP + j] = j < i ? v.y : 0.0;
        Xr[i * IP + j] = 0.0;
        Xi[i * IP + j] = 0.0;
        if (i == j) {
            const double d = v.x + lambda;
            const bool live = u0 + i < U && d > 0.0;
            if (u0 + i < U && !live) {
                // a NaN energy is not an inactive coordinate: it goes on as NaN
                if (d == d) atomicOr(status, (uint32_t)CDM_INFO_ZERO_COLUMN);
                rd[i] = d == d ? 0.0 : d;
            } else {
                rd[i] = live ? 1.0 / d : 0.0;
            }
        }
    }
    __syncthreads();
    if (lane < 16) {
        const int o = 16 * wv;
        double xr[16], xi[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            double sr = i == lane ? 1.0 : 0.0, si = 0.0;
#pragma unroll
            for (int q = 0; q < i; ++q) {
                const double lr = Lr[(o + i) * IP + o + q], li = Li[(o + i) * IP + o + q];
                sr -= lr * xr[q] - li * xi[q];
                si -= lr * xi[q] + li * xr[q];
            }
            const double d = rd[o + i];
            xr[i] = i >= lane ? sr * d : 0.0;
            xi[i] = i >= lane ? si * d : 0.0;
            Xr[(o + i) * IP + o + lane] = xr[i];
            Xi[(o + i) * IP + o + lane] = xi[i];
        }
    }
    __syncthreads();
    const int lr_ = lane & 15, lk = lane >> 4;
    for (int dg = 1; dg < 4; ++dg) {
        if (wv < 4 - dg) {
            const int bi = wv + dg, bj = wv;
            acc4 cr = {0, 0, 0, 0}, ci = {0, 0, 0, 0};
            for (int q = 16 * bj; q < 16 * bi; q += 4) {
                const double ar = Lr[(16 * bi + lr_) * IP + q + lk], ai = Li[(16 * bi + lr_) * IP + q + lk];
                const double br = Xr[(q + lk) * IP + 16 * bj + lr_], bm = Xi[(q + lk) * IP + 16 * bj + lr_];
                cr = mma64(ar, br, cr);
                cr = mma64(-ai, bm, cr);
                ci = mma64(ar, bm, ci);
                ci = mma64(ai, br, ci);
            }
            // the sum goes through this block's own place in X to become an operand
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                Xr[(16 * bi + lk + 4 * e) * IP + 16 * bj + lr_] = cr[e];
                Xi[(16 * bi + lk + 4 * e) * IP + 16 * bj + lr_] = ci[e];
            }
            __builtin_amdgcn_wave_barrier();
            acc4 dr = {0, 0, 0, 0}, di = {0, 0, 0, 0};
#pragma unroll
            for (int q = 0; q < 16; q += 4) {
                const double ar = -Xr[(16 * bi + lr_) * IP + 16 * bi + q + lk];
                const double ai = -Xi[(16 * bi + lr_) * IP + 16 * bi + q + lk];
                const double br = Xr[(16 * bi + q + lk) * IP + 16 * bj + lr_];
                const double bm = Xi[(16 * bi + q + lk) * IP + 16 * bj + lr_];
                dr = mma64(ar, br, dr);
                dr = mma64(-ai, bm, dr);
                di = mma64(ar, bm, di);
                di = mma64(ai, br, di);
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                Xr[(16 * bi + lk + 4 * e) * IP + 16 * bj + lr_] = dr[e];
                Xi[(16 * bi + lk + 4 * e) * IP + 16 * bj + lr_] = di[e];
            }
        }
        __syncthreads();
    }
    double2* const Mtk = Mt + (Mk - M);
    for (int e = tid; e < 4096; e += 256) {
        const int i = e >> 6, j = e & 63;
        Mk[(int64_t)i * k + c0 + j] = make_double2(Xr[i * IP + j], Xi[i * IP + j]);
        Mtk[(int64_t)i * k + c0 + j] = make_double2(Xr[j * IP + i], Xi[j * IP + i]);
    }
}

// 32 x 32 tiles of the products around the inverse:
//   MERGE_T  T21 = L21 X11, MERGE_X  X21 = -X22 T21: the lower-left half of a 2s x 2s
//            inverse from its two s x s halves (T in W's space, which is not yet in use);
//   FOLD     W_JK = G_JK M_K, for J in K's panel L^H M_K (strictly upper triangle of G_KK);
//   FOLD_V   V = -M L^H for a single panel (the iteration on delta itself).
// Tiles of users past U are zero.  A workgroup makes one tile, its four waves a quarter of the
// contraction index each: tiles are few, and one alone is bound by its chain of MFMAs.  FOLD has
// enough of them: there a workgroup makes 64 x 64, a tile per wave.
enum { MM_MERGE_T = 0, MM_MERGE_X = 1, MM_FOLD = 2, MM_FOLD_V = 3 };
template <int MODE>
__global__ __launch_bounds__(256, 2) void k_gs_mm(const double2* __restrict__ A, double2* __restrict__ M,
                                                  double2* __restrict__ Mt, double2* __restrict__ W, int Up, int U,
                                                  int k, int s) {
    // the left operand lies with the contraction index outermost too (lanes over rows: 256 B a
    // piece): G is its own conjugate transpose, and M is kept transposed as well
    constexpr bool HERM = MODE == MM_MERGE_T || MODE == MM_FOLD;
    __shared__ double red[MODE == MM_FOLD ? 1 : 3][32][64];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kb = k / 32;
    const int64_t kk = (int64_t)k * k;
    const double2 *a, *b;
    double2 *c, *ct = nullptr;
    int64_t lda, ldb, ldc;
    // contraction range in tiles of 32; diag: values of index <= row (FOLD) or >= column (FOLD_V)
    // relative to these belong to the other triangle and count as zero
    int c_lo, c_hi, diag = -(1 << 30);
    double sign = 1.0;
    if (MODE == MM_MERGE_T || MODE == MM_MERGE_X) {
        const int sb = s / 32;
        int n = blockIdx.x;
        const int j = n % sb;
        n /= sb;
        const int i = n % sb;
        n /= sb;
        const int q = n % (kb / (2 * sb)), p = n / (kb / (2 * sb));
        const int lo = 2 * q * s, hi = lo + s;
        const int64_t pm = p * kk;
        const bool live = p * k + hi + 32 * i < U;
        if (MODE == MM_MERGE_T) {
            a = A + (int64_t)(p * k + lo) * Up + p * k + hi + 32 * i;
            lda = Up;
            b = M + pm + (int64_t)lo * k + lo + 32 * j;
            c = W + pm + (int64_t)(hi + 32 * i) * k + lo + 32 * j;
            c_lo = j;
            c_hi = live ? sb : j;
        } else {
            a = Mt + pm + (int64_t)hi * k + hi + 32 * i;
            lda = k;
            b = W + pm + (int64_t)hi * k + lo + 32 * j;
            c = M + pm + (int64_t)(hi + 32 * i) * k + lo + 32 * j;
            ct = Mt + pm + (int64_t)(lo + 32 * j) * k + hi + 32 * i;
            c_lo = 0;
            c_hi = live ? i + 1 : 0;
            sign = -1.0;
        }
        ldb = ldc = k;
    } else if (MODE == MM_FOLD) {
        // The column blocks of one row block and panel go to one XCD, which reads G_JK once.  Their
        // order rotates from one to the next: workgroups go to an XCD's four shader engines in
        // turn and these wait for each other, so one that always drew the longest sums would hold
        // up all (8192 users: 1860 us, rotated 1290).
        const int nb = Up / 64, x = blockIdx.x % 8, m = blockIdx.x / 8;
        const int jk = (m / (kb / 2)) * 8 + x, jr = (m + m / (kb / 2)) % (kb / 2);
        if (jk >= nb * (Up / k)) return;   // the grid is a multiple of 8
        const int J = 2 * (jk % nb) + (wv >> 1), K = jk / nb, jl = 2 * jr + (wv & 1);
        const int j = K * kb + jl, Jl = J - K * kb;
        a = A + (int64_t)K * k * Up + J * 32;
        lda = Up;
        b = M + K * kk + 32 * jl;
        ldb = k;
        c = W + (int64_t)J * 32 * Up + j * 32;
        ldc = Up;
        c_lo = jl;
        c_hi = kb;
        if (Jl >= 0 && Jl < kb) {
            c_lo = max(jl, Jl);
            diag = 32 * Jl;
        }
    } else {
        // shells of equal min(i, j), the longest sums first; every other 256 (one per CU) backwards
        int n = blockIdx.x;
        if ((n >> 8) & 1) n ^= 255;
        int m = (int)sqrtf((float)n);
        while (m * m > n) --m;
        while ((m + 1) * (m + 1) <= n) ++m;
        const int o = n - m * m, c0 = kb - 1 - m;
        const int i = c0 + max(0, o - m), j = c0 + (o <= m ? o : 0);
        a = Mt + 32 * i;
        lda = k;
        b = A + 32 * j;
        ldb = Up;
        c = W + (int64_t)i * 32 * k + j * 32;
        ldc = k;
        c_lo = 0;
        c_hi = 32 * max(i, j) < U ? min(i, j) + 1 : 0;
        diag = 32 * j;
        sign = -1.0;
    }
    const int n4 = 8 * (c_hi - c_lo);   // steps, a quarter per wave
    const int s0 = 8 * c_lo + (MODE == MM_FOLD ? 0 : n4 * wv / 4);
    const int s1 = MODE == MM_FOLD ? 8 * c_hi : 8 * c_lo + n4 * (wv + 1) / 4;
    const int l16 = lane & 15, g = lane >> 4;
    MmAcc acc;
    acc.zero();
    auto fetch = [&](int st, double2(&x)[2], double2(&y)[2]) __attribute__((always_inline)) {
        const int q = 4 * st + g;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            x[t] = a[(int64_t)q * lda + l16 + 16 * t];
            y[t] = b[(int64_t)q * ldb + l16 + 16 * t];
        }
    };
    auto mask = [&](int st, double2(&x)[2], double2(&y)[2]) __attribute__((always_inline)) {
        const int q = 4 * st + g - diag - l16;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (MODE == MM_FOLD && q <= 16 * t) x[t] = make_double2(0.0, 0.0);
            if (MODE == MM_FOLD_V && q >= 16 * t) y[t] = make_double2(0.0, 0.0);
        }
    };
    acc.template run<HERM, double2>(s0, s1, fetch, mask);
    if (MODE == MM_FOLD) {
        acc.each(lane, [&](int i, int j, double2 z) { c[(int64_t)i * ldc + j] = z; });
        return;
    }
    if (wv > 0) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                red[wv - 1][8 * t + e][lane] = acc.r[t >> 1][t & 1][e];
                red[wv - 1][8 * t + 4 + e][lane] = acc.i[t >> 1][t & 1][e];
            }
    }
    __syncthreads();
    if (wv > 0) return;
#pragma unroll
    for (int w = 0; w < 3; ++w)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc.r[t >> 1][t & 1][e] += red[w][8 * t + e][lane];
                acc.i[t >> 1][t & 1][e] += red[w][8 * t + 4 + e][lane];
            }
    acc.each(lane, [&](int i, int j, double2 z) {
        const double2 v = make_double2(sign * z.x, sign * z.y);
        c[(int64_t)i * ldc + j] = v;
        if (MODE == MM_MERGE_X) ct[(int64_t)j * k + i] = v;
    });
}

// r = y - H x: a workgroup takes 16 rows, 16 threads of them a column group each.
template <typename T>
__global__ __launch_bounds__(256) void k_gs_rows(const cv<T>* __restrict__ H, int64_t ld, int B, int U,
                                                 const cv<T>* __restrict__ y, const double2* __restrict__ x,
                                                 double2* __restrict__ r, const uint32_t* __restrict__ done) {
    if (*done) return;
    __shared__ double2 s[16][17];
    const int i = threadIdx.x & 15, g = threadIdx.x >> 4;
    const int row = blockIdx.x * 16 + i;
    const int rc = min(row, B - 1);
    double2 a0 = make_double2(0.0, 0.0), a1 = a0;
    int u = g;
    for (; u + 48 < U; u += 64) {
        cv<T> h[4];
        double2 xv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) h[q] = H[(int64_t)(u + 16 * q) * ld + rc];
#pragma unroll
        for (int q = 0; q < 4; ++q) xv[q] = x[u + 16 * q];
        cfma(a0, to_d(h[0]), xv[0]);
        cfma(a1, to_d(h[1]), xv[1]);
        cfma(a0, to_d(h[2]), xv[2]);
        cfma(a1, to_d(h[3]), xv[3]);
    }
    for (; u < U; u += 16) cfma(a0, to_d(H[(int64_t)u * ld + rc]), x[u]);
    s[g][i] = make_double2(a0.x + a1.x, a0.y + a1.y);
    __syncthreads();
    if (threadIdx.x < 16 && row < B) {
        double2 z = to_d(y[row]);
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            z.x -= s[q][i].x;
            z.y -= s[q][i].y;
        }
        r[row] = z;
    }
}

// b_u = h_u^H r - lambda x_u, a workgroup per user (zero past U)
template <typename T>
__global__ __launch_bounds__(256) void k_gs_grad(const cv<T>* __restrict__ H, int64_t ld, int B, int U,
                                                 const double2* __restrict__ r, const double2* __restrict__ x,
                                                 double lambda, double2* __restrict__ b,
                                                 const uint32_t* __restrict__ done) {
    if (*done) return;
    __shared__ double2 s[4];
    const int u = blockIdx.x;
    double2 a0 = make_double2(0.0, 0.0), a1 = a0;
    if (u < U) {
        const cv<T>* h = H + (int64_t)u * ld;
        int i = threadIdx.x;
        for (; i + 768 < B; i += 1024) {
            cv<T> hv[4];
            double2 rv[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) hv[q] = h[i + 256 * q];
#pragma unroll
            for (int q = 0; q < 4; ++q) rv[q] = r[i + 256 * q];
            cfma_conj(a0, to_d(hv[0]), rv[0]);
            cfma_conj(a1, to_d(hv[1]), rv[1]);
            cfma_conj(a0, to_d(hv[2]), rv[2]);
            cfma_conj(a1, to_d(hv[3]), rv[3]);
        }
        for (; i < B; i += 256) cfma_conj(a0, to_d(h[i]), r[i]);
    }
    a0.x = group_sum<1>(a0.x + a1.x);
    a0.y = group_sum<1>(a0.y + a1.y);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = a0;
    __syncthreads();
    if (threadIdx.x == 0) {
        const double2 xv = x[u];
        b[u] = make_double2((s[0].x + s[1].x) + (s[2].x + s[3].x) - lambda * xv.x,
                            (s[0].y + s[1].y) + (s[2].y + s[3].y) - lambda * xv.y);
    }
}

__device__ __forceinline__ void gs_info(cdm_info* info, int sweeps, double S, double X, double tol, bool ok) {
    const double rel = X > 0.0 ? sqrt(S / X) : (S > 0.0 ? INFINITY : 0.0);
    int fl = 0;
    if (tol > 0.0 && !(rel <= tol)) fl |= CDM_INFO_NOT_CONVERGED;
    if (!ok) fl |= CDM_INFO_TIMEOUT;
    cdm_info o;
    o.sweeps = sweeps;
    o.flags = fl;
    o.rel_step = rel;
    o.resid = -1.0;
    o.reserved = 0.0;
    *info = o;
}

// Sweeps t0 + 1 .. t1 of a single panel of at most 128 users, in one workgroup: with one
// panel the deltas follow each other by delta <- V delta, V = -M L^H, so V stays in
// registers (128 x 128 complex FP64 = 128 VGPRs of 512 threads) and a sweep is one product and
// one barrier.  Thread: 4 rows x 8 columns, 16 lanes to a row.  The eight sums of 4 rows over
// the 16 lanes are formed by halving: a lane keeps half of its sums in each of three exchanges
// (with lane 15 - i, then 7 - i, then i ^ 2) and ends with one part of one delta, and of x.
// The norms of a sweep are formed while the next product's operands come from LDS, and
// looked at by the last wave during the product after that, so a stop is known two sweeps
// later and x of the last three is kept.
// Bound: the product's 1024 cycles of FP64 FMA per SIMD, its 512 cycles of LDS reads, and the
// chain of sums and barrier.  256 x 128, 60 sweeps, the whole solve: 156 us (1.5 us a sweep); 1024
// threads with two rows each, every sum in every lane and the stop looked at by all of them
// between the sweeps 182 us (1.8).
template <int CTRL> __device__ __forceinline__ void halve(double& a, double b, bool upper) {
    // lanes with `upper` keep b, the others a: + what the partner lane has of the same
    const double mine = upper ? b : a, give = upper ? a : b;
    a = mine + dpp_take<CTRL, 0xf>(give);
}
__global__ __launch_bounds__(512) void k_gs_one(const double2* __restrict__ V, const double2* __restrict__ M,
                                                const double2* __restrict__ b, double2* __restrict__ x, int U,
                                                int t0, int t1, double tol, uint32_t* __restrict__ done,
                                                cdm_info* __restrict__ info) {
    if (*done) return;
    __shared__ double2 ds[2][128];
    __shared__ double st[2][16];
    __shared__ int flag[2];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cl = lane & 15, r0 = wv * 16 + (lane >> 4) * 4;
    const bool b3 = lane & 8, b2 = lane & 4, b1 = lane & 2, b0 = lane & 1;
    const int part = 2 * (r0 + 2 * (int)b3 + (int)b2) + (int)b1;   // this lane's double of x and delta
    double2 w[4][8], d[4];
    // delta of sweep t0 + 1 is M b
    if (tid < 128) ds[1][tid] = b[tid];
    if (tid < 2) flag[tid] = 0;
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = 0; q < 8; ++q) w[p][q] = M[(r0 + p) * 128 + cl + 16 * q];
    double xv = ((const double*)x)[part], xp = xv, xpp = xv;   // x after this sweep and the two before
    __syncthreads();
    double2 v[8];
    auto fetch = [&](const double2* in) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = in[cl + 16 * q];
    };
    auto product = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < 4; ++p) d[p] = make_double2(0.0, 0.0);
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
            for (int p = 0; p < 4; ++p) cfma(d[p], w[p][q], v[q]);
    };
    fetch(ds[1]);
    product();
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = 0; q < 8; ++q) w[p][q] = V[(r0 + p) * 128 + cl + 16 * q];
    double S = 0.0, X = 0.0;
    auto norms = [&](int t, double dv) __attribute__((always_inline)) {   // even lanes |delta|^2, odd lanes |x|^2
        double s = b0 ? xv * xv : dv * dv;
        s += row_ror<8>(s);
        s += row_ror<4>(s);
        s += dpp_take<0x4e, 0xf>(s);
        s = swap_add<32>(swap_add<16>(s));
        if (lane < 2) st[t & 1][2 * wv + lane] = s;
    };
    auto decide = [&](int t) __attribute__((always_inline)) -> bool {   // by the last wave, of sweep t
        double s = st[t & 1][cl];
        s += row_ror<8>(s);
        s += row_ror<4>(s);
        s += row_ror<2>(s);
        S = lane_value(s, 0);
        X = lane_value(s, 1);
        // the two roots only where they can decide: FP64 roots cost as much as the product
        return tol > 0.0 && !(S > 2.0 * tol * tol * X) && sqrt(S) <= tol * sqrt(X);
    };
    int t = t0 + 1, back = 0;   // the sweep that ends it is t - back
    double dv;
    for (;; ++t) {
        // rows (0, 1) | (2, 3), then one row, then its real | imaginary part, then both lanes
        halve<0x140>(d[0].x, d[2].x, b3);
        halve<0x140>(d[0].y, d[2].y, b3);
        halve<0x140>(d[1].x, d[3].x, b3);
        halve<0x140>(d[1].y, d[3].y, b3);
        halve<0x141>(d[0].x, d[1].x, b2);
        halve<0x141>(d[0].y, d[1].y, b2);
        halve<0x4e>(d[0].x, d[0].y, b1);
        dv = d[0].x + dpp_take<0xb1, 0xf>(d[0].x);
        xpp = xp;
        xp = xv;
        xv += dv;
        if (!b0) ((double*)ds[t & 1])[part] = dv;
        __syncthreads();
        if (t == t1) break;
        fetch(ds[t & 1]);
        if (tol > 0.0) {   // while the deltas come from LDS
            if (flag[t & 1]) {
                back = 2;
                break;
            }
            norms(t, dv);
            if (wv == 7 && t - 1 > t0) {
                const bool met = decide(t - 1);
                if (lane == 0) flag[(t - 1) & 1] = met;
            }
        }
        product();
    }
    if (back == 0) {   // t == t1: the decisions of the last three sweeps
        norms(t, dv);
        __syncthreads();
        if (wv == 7) {
            int which = -1;
            if (tol > 0.0 && flag[t & 1])
                which = 2;   // S, X are still that sweep's
            else if (t - 1 > t0 && decide(t - 1))
                which = 1;
            else if (decide(t))
                which = 0;
            if (lane == 0) {
                gs_info(info, t - max(which, 0), S, X, tol, true);
                if (which >= 0) *done = 1;
                flag[(t + 1) & 1] = max(which, 0);
            }
        }
        __syncthreads();
        back = flag[(t + 1) & 1];
    } else if (wv == 7 && lane == 0) {
        gs_info(info, t - 2, S, X, tol, true);
        *done = 1;
    }
    if (!b0) ((double*)x)[part] = back == 2 ? xpp : (back == 1 ? xp : xv);
}

// Sweeps t0 + 1 .. t1 over several workgroups (cooperative launch).  Workgroup w owns R
// consecutive rows of W, b and x (all in one panel); its NW tile waves take RW = R / NW
// rows each, a lane per column modulo 64, the row's values of b and x in every lane.  The
// CW other waves do every exchange: per step they gather the k values of b_K (tagged
// words, one memory round trip, no flag) into LDS behind one barrier.  Each tile wave
// loads its tile of the next step once it is done with this one, so the stream of W
// (U^2 x 16 B per sweep, from L2 or MALL) runs during the exchange.
// Slots: b_K of sweep t in slot t & 1 of panel K.  To publish b_K of sweep t + 2 a
// workgroup has gathered every panel of sweep t + 1, and its owners published that after
// they had gathered b_K of sweep t, so the slot is free.
// Stop: the owners of a panel know the deltas, so each workgroup publishes its part of
// (sum |delta|^2, sum |x|^2) of a sweep; every workgroup adds all parts in the same order
// two sweeps later, at its own panel, and stops with the x of that sweep (the one before
// its current x): the exchange of the statistics is hardly ever waited for.  The
// workgroups that stop have published all that the others need to reach their own panel.
constexpr int GS_CW = 4;
// value i of n in an exchange slot: three planes of n tagged words, so that a wave's loads
// of one word are contiguous
__device__ __forceinline__ void gs_put(uint64_t* p, int n, int i, double2 v, uint32_t tag) {
    const uint64_t a = (uint64_t)__double_as_longlong(v.x), b = (uint64_t)__double_as_longlong(v.y);
    Tagged<double>::st48(p + i, a, tag);
    Tagged<double>::st48(p + n + i, (a >> 48) | (b << 16), tag);
    Tagged<double>::st48(p + 2 * n + i, b >> 32, tag);
}
__device__ __forceinline__ bool gs_get(const uint64_t* p, int n, int i, uint32_t tag, double2& v) {
    const uint64_t w0 = ld_tag(p + i), w1 = ld_tag(p + n + i), w2 = ld_tag(p + 2 * n + i);
    const uint64_t t = (uint64_t)(tag & 0xffffu), m = 0xffffffffffffull;
    v.x = __longlong_as_double((long long)((w0 & m) | ((w1 & 0xffffull) << 48)));
    v.y = __longlong_as_double((long long)(((w1 & m) >> 16) | ((w2 & 0xffffffffull) << 32)));
    return ((w0 >> 48) == t) & ((w1 >> 48) == t) & ((w2 >> 48) == t);
}

using gs_v2d = double __attribute__((ext_vector_type(2)));

template <int R, int NW, int KC>
__global__ __launch_bounds__(64 * (NW + GS_CW), 1) void k_gs_sweep(GsSweepArgs a, int t0, int t1) {
    constexpr int RW = R / NW, k = 64 * KC, GC = KC / GS_CW;
    if (*a.done) return;
    __shared__ double2 bs[2][k];
    __shared__ double2 sacc[2][NW];
    __shared__ double2 xs[R], xps[R];       // x of these rows and of the sweep before, wave by wave
    __shared__ int go[2][GS_CW];
    extern __shared__ __attribute__((aligned(16))) double2 ms[];   // this workgroup's rows of M: R x k
    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int w = blockIdx.x, P = gridDim.x, npan = a.npan, Up = a.Up;
    const int Kw = w * R / k;               // the panel that holds this workgroup's rows
    const bool comm = wid >= NW, lead = wid == NW;
    const int row0 = w * R + (comm ? 0 : wid * RW);
    double2 b[RW];
    double2 tile[RW][KC];
    uint64_t* const xch = a.xch;            // [npan][2] slots of k values
    uint64_t* const sch = a.xch + (int64_t)npan * 2 * k * 3;   // [4] slots of P values
    auto publish = [&](int t) __attribute__((always_inline)) {   // this wave's rows of b for sweep t
#pragma unroll
        for (int r = 0; r < RW; ++r)
            if (lane == r) gs_put(xch + (int64_t)(Kw * 2 + (t & 1)) * k * 3, k, (row0 + r) % k, b[r], (uint32_t)t);
    };
    // W past 192 MB goes by the MALL (256 MB, which a cyclic stream would empty each time), so
    // that the first panels stay in it.  8192 users, 1 GiB: 6 of 32 panels cached 206 us a
    // sweep, all of them 223.
    const int Kc = (int)(((int64_t)192 << 20) / ((int64_t)16 * Up * k));
    auto load = [&](int K) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const double2* const p = a.W + (int64_t)(row0 + r) * Up + K * k;   // scalar base, one offset register
            uint32_t o = (uint32_t)lane;
            asm("" : "+v"(o));
            if (K < Kc) {
#pragma unroll
                for (int q = 0; q < KC; ++q) tile[r][q] = p[o + 64 * q];
            } else {
#pragma unroll
                for (int q = 0; q < KC; ++q) {
                    const gs_v2d z = __builtin_nontemporal_load((const gs_v2d*)(p + o + 64 * q));
                    tile[r][q] = make_double2(z.x, z.y);
                }
            }
        }
    };
    if (!comm) {
#pragma unroll
        for (int r = 0; r < RW; ++r) b[r] = a.b[row0 + r];
        if (Kw == 0) publish(t0 + 1);
        load(0);
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            if (lane == 0) xs[wid * RW + r] = xps[wid * RW + r] = a.x[row0 + r];
#pragma unroll
            for (int q = 0; q < KC; ++q)
                ms[(wid * RW + r) * k + lane + 64 * q] =
                    a.M[(int64_t)Kw * k * k + (int64_t)((row0 + r) % k) * k + lane + 64 * q];
        }
    }
    double S = 0.0, X = 0.0;
    uint64_t tw = 0;
    auto expired = [&]() __attribute__((always_inline)) -> bool {   // bounded waits: true once the wait is given up
        if (ld_relaxed(a.abort_flag)) return true;
        const uint64_t now = wall_clock64();
        if (!tw) tw = now;
        if (now - tw > a.timeout_ticks) {
            if (lane == 0) st_relaxed(a.abort_flag, 1u);
            return true;
        }
        return false;
    };
    // S, X: the parts of sweep t summed in a fixed order (every lane and workgroup alike)
    auto stats = [&](int t) __attribute__((always_inline)) -> bool {
        for (;;) {
            bool ok = true;
            S = X = 0.0;
            for (int p = lane; p < P; p += 64) {
                double2 v;
                ok &= gs_get(sch + (int64_t)(t & 3) * P * 3, P, p, (uint32_t)t, v);
                S += v.x;
                X += v.y;
            }
            if (__all(ok)) break;
            if (expired()) return false;
        }
        S = wave_allsum(S);
        X = wave_allsum(X);
        tw = 0;
        return true;
    };
    auto put_stats = [&](int t, int sp) __attribute__((always_inline)) {
        double s1 = 0.0, s2 = 0.0;
#pragma unroll
        for (int q = 0; q < NW; ++q) {
            s1 += sacc[sp][q].x;
            s2 += sacc[sp][q].y;
        }
        if (lane == 0) gs_put(sch + (int64_t)(t & 3) * P * 3, P, w, make_double2(s1, s2), (uint32_t)t);
    };
    auto met = [&]() { return a.tol > 0.0 && !(S > 2.0 * a.tol * a.tol * X) && sqrt(S) <= a.tol * sqrt(X); };

    int code = 1, t = t0 + 1, K = 0, owed = 0, par = 0;   // code: 1 goes on, 2 x of the sweep before, 3 given up
    for (;; par ^= 1) {
        if (comm) {
            int g = 1;
            const uint64_t* src = xch + (int64_t)(K * 2 + (t & 1)) * k * 3;
            const int i0 = (wid - NW) * 64 * GC + lane;
            double2 v[GC];
            bool ok = false;
            for (;;) {
                if (!ok) {
                    ok = true;
#pragma unroll
                    for (int q = 0; q < GC; ++q) ok &= gs_get(src, k, i0 + 64 * q, (uint32_t)t, v[q]);
                }
                if (__all(ok)) break;
                if (expired()) {
                    g = 3;
                    break;
                }
            }
            tw = 0;
#pragma unroll
            for (int q = 0; q < GC; ++q) bs[par][i0 + 64 * q] = v[q];
            if (lead && g == 1 && a.tol > 0.0 && K == Kw && t - 2 > t0) {
                if (!stats(t - 2))
                    g = 3;
                else if (met()) {
                    g = 2;
                    if (w == 0 && lane == 0) gs_info(a.info, t - 2, S, X, a.tol, true);
                }
            }
            if (lane == 0) go[par][wid - NW] = g;
        }
        __syncthreads();
        code = 1;
#pragma unroll
        for (int q = 0; q < GS_CW; ++q) code = max(code, go[par][q]);
        if (code != 1) break;
        const bool own = K == Kw;
        const int Kn = K + 1 < npan ? K + 1 : 0;
        const bool last = t == t1 && Kn == 0;
        if (comm) {
            if (lead && owed) put_stats(owed, par ^ 1);   // written before this barrier
            owed = own ? t : 0;
        } else {
            double2 v[KC];
#pragma unroll
            for (int q = 0; q < KC; ++q) v[q] = bs[par][lane + 64 * q];
#pragma unroll
            for (int r = 0; r < RW; ++r) {
                double2 s = make_double2(0.0, 0.0);
#pragma unroll
                for (int q = 0; q < KC; ++q) cfma(s, tile[r][q], v[q]);
                s.x = group_sum<1>(s.x);
                s.y = group_sum<1>(s.y);
                b[r].x = own ? -s.x : b[r].x - s.x;
                b[r].y = own ? -s.y : b[r].y - s.y;
            }
            if (Kn == Kw && !last) publish(Kn == 0 ? t + 1 : t);
            if (npan > 1 && !last) load(Kn);
            if (own) {
                double s1 = 0.0, s2 = 0.0;
#pragma unroll
                for (int r = 0; r < RW; ++r) {
                    double2 s = make_double2(0.0, 0.0);
#pragma unroll
                    for (int q = 0; q < KC; ++q) cfma(s, ms[(wid * RW + r) * k + lane + 64 * q], v[q]);
                    s.x = group_sum<1>(s.x);
                    s.y = group_sum<1>(s.y);
                    const double2 xo = xs[wid * RW + r], xn = make_double2(xo.x + s.x, xo.y + s.y);
                    if (lane == 0) {
                        xps[wid * RW + r] = xo;
                        xs[wid * RW + r] = xn;
                    }
                    s1 += cabs2d(s);
                    s2 += cabs2d(xn);
                }
                if (lane == 0) sacc[par][wid] = make_double2(s1, s2);
            }
        }
        if (last) break;
        K = Kn;
        if (Kn == 0) ++t;
    }
    if (code == 1) {   // all sweeps run: the decisions of the last two
        __syncthreads();
        if (lead) {
            int g = 1;
            if (owed) put_stats(owed, par);
            bool ok = true;
            if (a.tol > 0.0 && t1 - 1 > t0) {
                ok = stats(t1 - 1);
                if (ok && met()) {
                    g = 2;
                    if (w == 0 && lane == 0) gs_info(a.info, t1 - 1, S, X, a.tol, true);
                }
            }
            if (ok && g == 1) {
                ok = stats(t1);
                if (ok && met()) g = 4;
                if (ok && w == 0 && lane == 0) gs_info(a.info, t1, S, X, a.tol, true);
            }
            if (lane == 0) go[0][0] = ok ? g : 3;
        }
        __syncthreads();
        code = go[0][0];
    }
    if (!comm && lane == 0) {
#pragma unroll
        for (int r = 0; r < RW; ++r) a.x[row0 + r] = code == 2 ? xps[wid * RW + r] : xs[wid * RW + r];
    }
    if (w == 0 && lead && lane == 0) {
        if (code == 3) gs_info(a.info, t - 1, S, X, a.tol, false);
        if (code != 1) *a.done = 1;
    }
}

// x in the caller's type, and the flags that are known now
template <typename T>
__global__ __launch_bounds__(1024) void k_gs_finish(const double2* __restrict__ xw, int U, cv<T>* __restrict__ x,
                                                    const uint32_t* __restrict__ status, cdm_info* __restrict__ info) {
    __shared__ int bad;
    if (threadIdx.x == 0) bad = 0;
    __syncthreads();
    int mine = 0;
    for (int u = threadIdx.x; u < U; u += 1024) {
        const cv<T> v = cmake<T>((T)xw[u].x, (T)xw[u].y);
        x[u] = v;
        if (!isfinite(v.x) || !isfinite(v.y)) mine = 1;
    }
    if (mine) bad = 1;
    __syncthreads();
    if (threadIdx.x == 0)
        info->flags |= (int)(*status & (CDM_INFO_ZERO_COLUMN | CDM_INFO_BAD_INPUT)) | (bad ? CDM_INFO_NONFINITE : 0);
}

// ---- host side -----------------------------------------------------------------------------

#define GS_TRY(call)                        \
    do {                                    \
        const hipError_t e_ = (call);       \
        if (e_ != hipSuccess) return e_;    \
    } while (0)

// Sweeps t0 + 1 .. t1 of a single panel of 129 to 1024 users over several workgroups
// (cooperative launch): delta <- V delta, V = -M L^H, with V in the registers of the chip (16 MiB at
// 1024 users), so a sweep moves nothing but one exchange of k deltas.  Workgroup w owns R rows of
// V; eight tile waves take R / 8 of them, a lane per column modulo 64.  The other GS_CW waves
// gather every delta (tagged words, one memory round trip) into LDS behind one barrier, and
// each workgroup keeps all of x in theirs: its norms, and with them the decision to stop, are the
// same bits everywhere and need no exchange.  They are formed while the tile waves work and
// looked at a sweep later, before x moves on.  With a dense channel's type T the kernel forms b
// anew itself between the segments of sweeps (r from the workgroups' rows, all wait for all, b from
// the workgroups' users).
// Bound by the exchange: 3000 x 1000 complex128, 39 sweeps, 4.0 us each (two panels of 512 with M and W
// streamed: 8.4), the whole solve 850 -> 700 us.
// after sweep t0 the sweep at which b is formed anew
__host__ __device__ inline int gs_segment_end(int t0, int t_max) {
    const int seg = t0 < 2 ? 2 : (t0 < 8 ? 8 : (t0 < 40 ? 40 : (t0 < 200 ? 200 : t_max)));
    return seg < t_max ? seg : t_max;
}
template <typename T> constexpr int gs_rows_per_block() { return 128 / (int)sizeof(cv<T>); }   // one cache line
template <> constexpr int gs_rows_per_block<void>() { return 1; }
template <int R, int KC, typename T>
__global__ __launch_bounds__(64 * (8 + GS_CW), 1) void k_gs_delta(GsSweepArgs a, int t0, int t_end) {
    constexpr int NW = 8, RW = R / NW, k = 64 * KC, GC = KC / GS_CW, NV = NW + GS_CW, RB = gs_rows_per_block<T>();
    if (*a.done) return;
    __shared__ double2 ds[2][k];
    __shared__ double2 st[2][GS_CW];
    __shared__ double2 red[NV][RB];
    __shared__ int go[2][GS_CW];
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int w = blockIdx.x, P = gridDim.x;
    const bool comm = wid >= NW;
    const int row0 = w * R + (comm ? 0 : wid * RW), i0 = (wid - NW) * 64 * GC + lane;
    double2 V[RW][KC], v[GC], x[GC];
    auto product = [&](const double2* in, double2(&d)[RW]) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < RW; ++r) d[r] = make_double2(0.0, 0.0);
#pragma unroll
        for (int q = 0; q < KC; ++q) {
            const double2 z = in[lane + 64 * q];
#pragma unroll
            for (int r = 0; r < RW; ++r) cfma(d[r], V[r][q], z);
        }
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            d[r].x = group_sum<1>(d[r].x);
            d[r].y = group_sum<1>(d[r].y);
        }
    };
    // these rows of M times b; a few columns at a time, as V lives next to them
    auto m_product = [&](const double2* b, double2(&d)[RW]) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const double2* const m = a.M + (int64_t)(row0 + r) * k;
            d[r] = make_double2(0.0, 0.0);
#pragma unroll 4
            for (int q = 0; q < KC; ++q) cfma(d[r], m[lane + 64 * q], b[lane + 64 * q]);
            d[r].x = group_sum<1>(d[r].x);
            d[r].y = group_sum<1>(d[r].y);
        }
    };
    auto publish = [&](const double2(&d)[RW], int slot, int t) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < RW; ++r)
            if (lane == r) gs_put(a.xch + (int64_t)slot * k * 3, k, row0 + r, d[r], (uint32_t)t);
    };
    // bounded waits: given up after the time limit, or with the others
    uint64_t tw = 0;
    auto expired = [&]() __attribute__((always_inline)) -> bool {
        const uint64_t now = wall_clock64();
        if (!tw) tw = now;
        if (!ld_relaxed(a.abort_flag) && now - tw <= a.timeout_ticks) return false;
        if (lane == 0) st_relaxed(a.abort_flag, 1u);
        return true;
    };
    // the k values of a slot into v and `out`: 1, or 3 when given up (per communicating wave)
    auto gather = [&](int slot, int t, double2* out) __attribute__((always_inline)) -> int {
        bool ok = false;
        int g = 1;
        tw = 0;
        for (;;) {
            if (!ok) {
                ok = true;
#pragma unroll
                for (int q = 0; q < GC; ++q)
                    ok &= gs_get(a.xch + (int64_t)slot * k * 3, k, i0 + 64 * q, (uint32_t)t, v[q]);
            }
            if (__all(ok)) break;
            if (expired()) {
                g = 3;
                break;
            }
        }
#pragma unroll
        for (int q = 0; q < GC; ++q) out[i0 + 64 * q] = v[q];
        return g;
    };
    if (!comm) {
        double2 d[RW];   // the first delta is M b
        m_product(a.b, d);
        publish(d, (t0 + 1) & 1, t0 + 1);
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const double2* const p = a.W + (int64_t)(row0 + r) * k;   // scalar base, one offset register
            uint32_t o = (uint32_t)lane;
            asm("" : "+v"(o));
#pragma unroll
            for (int q = 0; q < KC; ++q) V[r][q] = p[o + 64 * q];
        }
    } else {
#pragma unroll
        for (int q = 0; q < GC; ++q) x[q] = a.x[i0 + 64 * q];
    }
    double S = 0.0, X = 0.0;
    // S, X and the decision of the sweep whose parts lie in st[p]
    auto met = [&](int p) __attribute__((always_inline)) {
        S = X = 0.0;
#pragma unroll
        for (int q = 0; q < GS_CW; ++q) {
            S += st[p][q].x;
            X += st[p][q].y;
        }
        return a.tol > 0.0 && !(S > 2.0 * a.tol * a.tol * X) && sqrt(S) <= a.tol * sqrt(X);
    };
    // b anew from H, y and x, and the first delta of sweep t + 1 from it; false: given up.  Rows
    // and users are dealt to the workgroups; r passes through memory, b through a slot.
    int round = 0;
    auto anew = [&](int t, int par) -> bool {
        if constexpr (!std::is_void_v<T>) {
            double2* const xs = ds[par ^ 1];
            const cv<T>* const H = (const cv<T>*)a.H;
            if (comm) {
#pragma unroll
                for (int q = 0; q < GC; ++q) xs[i0 + 64 * q] = x[q];
            }
            __syncthreads();
            for (int blk = w; blk * RB < a.B; blk += P) {   // r: a lane's row and column group
                const int row = blk * RB + lane % RB, rc = min(row, a.B - 1);
                constexpr int G = 64 / RB;
                double2 s = make_double2(0.0, 0.0);
#pragma unroll 4
                for (int u = wid * G + lane / RB; u < a.U; u += NV * G) cfma(s, to_d(H[(int64_t)u * a.ld + rc]), xs[u]);
#pragma unroll
                for (int m = RB; m < 64; m *= 2) {
                    s.x += __shfl_xor(s.x, m);
                    s.y += __shfl_xor(s.y, m);
                }
                if (lane < RB) red[wid][lane] = s;
                __syncthreads();
                if (wid == 0 && lane < RB && row < a.B) {
                    double2 z = to_d(((const cv<T>*)a.y)[row]);
#pragma unroll
                    for (int p = 0; p < NV; ++p) {
                        z.x -= red[p][lane].x;
                        z.y -= red[p][lane].y;
                    }
                    a.r[row] = z;
                }
                __syncthreads();
            }
            ++round;
            if (wid == 0) {   // this wave wrote the rows of r: out to memory, then all wait for all
                __threadfence();
                if (lane == 0) atomicAdd(a.arrived, 1u);
                int g = 1;
                tw = 0;
                while (ld_relaxed(a.arrived) < (uint32_t)(round * P))
                    if (expired()) {
                        g = 3;
                        break;
                    }
                __threadfence();
                if (lane == 0) go[0][0] = g;
            }
            __syncthreads();
            if (go[0][0] == 3) return false;
            if (!comm) {
                double2 d[RW];
#pragma unroll
                for (int r = 0; r < RW; ++r) {
                    const int u = row0 + r;
                    const cv<T>* const h = H + (int64_t)min(u, a.U - 1) * a.ld;
                    double2 s = make_double2(0.0, 0.0);
#pragma unroll 4
                    for (int i = lane; i < a.B; i += 64) cfma_conj(s, to_d(h[i]), a.r[i]);
                    s.x = group_sum<1>(s.x);
                    s.y = group_sum<1>(s.y);
                    d[r] = u < a.U ? make_double2(s.x - a.lambda * xs[u].x, s.y - a.lambda * xs[u].y)
                                   : make_double2(0.0, 0.0);
                }
                publish(d, 2, t + 1);
            }
            __syncthreads();   // go is free
            if (comm) {
                const int g = gather(2, t + 1, ds[par]);
                if (lane == 0) go[0][wid - NW] = g;
            }
            __syncthreads();
            int c = 1;
#pragma unroll
            for (int q = 0; q < GS_CW; ++q) c = max(c, go[0][q]);
            if (c == 3) return false;
            if (!comm) {
                double2 d[RW];
                m_product(ds[par], d);
                publish(d, (t + 1) & 1, t + 1);
            }
            __syncthreads();   // go and ds are free
        }
        return true;
    };
    bool stop = false;
    int code = 1, t = t0 + 1, par = 0, ts = t0;   // code: 1 goes on, 2 met, 3 given up
    int t1 = gs_segment_end(t0, t_end);
    for (;; ++t, par ^= 1) {
        if (comm) {
            const int g = gather(t & 1, t, ds[par]);
            if (lane == 0) go[par][wid - NW] = g;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < GS_CW; ++q) code = max(code, go[par][q]);
        if (code == 3) break;
        if (!comm && t < t1) {
            double2 d[RW];
            product(ds[par], d);
            publish(d, (t + 1) & 1, t + 1);
        }
        if (a.tol > 0.0 && t - 1 > ts && met(par ^ 1)) {
            code = 2;
            break;
        }
        if (comm) {
            double s1 = 0.0, s2 = 0.0;
#pragma unroll
            for (int q = 0; q < GC; ++q) {
                x[q].x += v[q].x;
                x[q].y += v[q].y;
                s1 += cabs2d(v[q]);
                s2 += cabs2d(x[q]);
            }
            s1 = group_sum<1>(s1);
            s2 = group_sum<1>(s2);
            if (lane == 0) st[par][wid - NW] = make_double2(s1, s2);
        }
        if (t < t1) continue;
        __syncthreads();
        stop = met(par);
        if (stop || t == t_end) break;
        if (!anew(t, par)) {
            code = 3;
            break;
        }
        ts = t;
        t1 = gs_segment_end(t, t_end);
    }
    if (w != 0 || !comm) return;
#pragma unroll
    for (int q = 0; q < GC; ++q) a.x[i0 + 64 * q] = x[q];
    if (wid == NW && lane == 0) {
        gs_info(a.info, code == 1 ? t : t - 1, S, X, a.tol, code != 3);
        if (stop || code != 1) *a.done = 1;
    }
}

constexpr int GS_DELTA_R = 8;   // rows per workgroup of k_gs_delta

GsShape gs_shape(int B, int U) {
    GsShape s;
    // Up to 1024 users one panel, V in registers (R = 8: 16 rows of 1024 spill, 773 against 691 us
    // for 3000 x 1000 and 40 sweeps; up to 512 users both alike).  Above, panels as wide as the
    // LDS holds R rows of M (128 KB): one exchange per panel and sweep; R = 16 rows a workgroup
    // up to 4096 users (fewer workgroups poll fewer copies of the same words: 3000 x 1000 on two
    // panels, 39 sweeps, 16 rows 818 us, 8 rows 905 us; 256-column panels 1031 us), 32 above, so
    // that at most 256 workgroups take part
    s.k = U <= 128 ? 128 : (U <= 256 || U > 4096 ? 256 : (U <= 512 || U > 1024 ? 512 : 1024));
    s.npan = (U + s.k - 1) / s.k;
    s.Up = s.npan * s.k;
    s.one = U <= 128;
    s.R = s.one ? 128 : (s.npan == 1 ? GS_DELTA_R : (U > 4096 ? 32 : 16));
    s.P = s.Up / s.R;
    s.nblk = ((U + 63) / 64) * ((U + 63) / 64 + 1) / 2;
    // workgroups of the Gram pass: two per CU, fewer where the parts of blocks that they leave
    // (64 KiB each) would cost more than the shorter runs of steps gain.  Us: a step 4.4 (two on a
    // CU 7.6), a part 0.045
    const int64_t n = (int64_t)s.nblk * ((B + 31) / 32);
    double best = 0.0;
    s.nwork = 1;
    for (int nw = 1; nw <= 512 && nw <= n; nw += nw < 16 ? 1 : 8) {
        const double cost = (double)((n + nw - 1) / nw) * (nw > 256 ? 7.6 : 4.4) + 0.045 * (nw + s.nblk);
        if (nw == 1 || cost < best) {
            best = cost;
            s.nwork = nw;
        }
    }
    return s;
}

size_t gs_exchange_words(const GsShape& s) {
    return s.npan == 1 ? 9 * (size_t)s.k : 3 * ((size_t)s.npan * 2 * s.k + 4 * (size_t)s.P);
}

// all sweeps of a dense channel in one launch
static bool gs_whole(const GsShape& s, int B, int U) {
    return !s.one && s.k <= 512 && s.npan == 1 && (int64_t)B * U <= (int64_t)12000 * s.P;
}
// the sweep kernel of a tiling: its R and k are the kernel's own (NULL: none is built).  SRC: float
// or double, or void where b is formed anew by launches in between
template <typename SRC> static const void* gs_sweep_fn(const GsShape& s) {
    if (s.npan == 1) {
        if (s.R != GS_DELTA_R) return nullptr;
        if (s.k == 256) return (const void*)k_gs_delta<GS_DELTA_R, 4, SRC>;
        if (s.k == 512) return (const void*)k_gs_delta<GS_DELTA_R, 8, SRC>;
        if (s.k == 1024 && std::is_void_v<SRC>) return (const void*)k_gs_delta<GS_DELTA_R, 16, void>;
        return nullptr;
    }
    if (s.k == 512 && s.R == 16) return (const void*)k_gs_sweep<16, 8, 8>;
    if (s.k == 256 && s.R == 32) return (const void*)k_gs_sweep<32, 8, 4>;
    return nullptr;
}

// dynamic LDS of the sweep kernel: the workgroup's rows of M (several panels)
static size_t gs_sweep_lds(const GsShape& s) { return s.npan == 1 ? 0 : (size_t)16 * s.R * s.k; }

template <typename T> static hipError_t launch_gs_t(const GsLaunch& L, hipStream_t st) {
    const GsShape& s = L.s;
    const cv<T>* H = (const cv<T>*)L.H;
    const cv<T>* y = (const cv<T>*)L.y;
    double2* A = (double2*)L.A;
    double2* M = (double2*)L.M;
    double2* Mt = (double2*)L.Mt;
    double2* W = (double2*)L.W;
    double2* r = (double2*)L.r;
    double2* b = (double2*)L.b;
    double2* x = (double2*)L.xw;
    uint32_t* done = L.ctr + 4;
    const int nmax = L.B > s.Up ? L.B : s.Up;
    hipLaunchKernelGGL(k_gs_init<T>, dim3((nmax + 255) / 256), dim3(256), 0, st, y, (const cv<T>*)L.x0, L.B, L.U, s.Up,
                       r, x, (uint64_t*)L.ctr, (int)(GS_CTR_WORDS / 2 + gs_exchange_words(s)));
    GS_TRY(hipGetLastError());
    const int nb = s.Up / 64;
    if (L.sp) {
        GS_TRY(gs_sparse_matrix(L, st));
    } else {
        hipLaunchKernelGGL(k_gs_gram<T>, dim3(s.nwork), dim3(256), 0, st, H, L.ld, L.B, L.U, s.nblk,
                           (double2*)L.gpart);
        hipLaunchKernelGGL(k_gs_assemble, dim3(nb * (nb + 1) / 2, 4), dim3(256), 0, st, (const double2*)L.gpart,
                           s.nwork, (L.B + 31) / 32, s.nblk, s.Up, A);
    }
    hipLaunchKernelGGL(k_gs_inv64, dim3(nb, 1 + s.k / 128), dim3(256), GS_INV_LDS, st, A, s.Up, L.U, s.k, L.lambda, M,
                       Mt, L.ctr + 3);
    GS_TRY(hipGetLastError());
    for (int h = 64; h < s.k; h *= 2) {
        const int blocks = s.npan * (s.k / (2 * h)) * (h / 32) * (h / 32);
        hipLaunchKernelGGL(k_gs_mm<MM_MERGE_T>, dim3(blocks), dim3(256), 0, st, A, M, Mt, W, s.Up, L.U, s.k, h);
        hipLaunchKernelGGL(k_gs_mm<MM_MERGE_X>, dim3(blocks), dim3(256), 0, st, A, M, Mt, W, s.Up, L.U, s.k, h);
    }
    if (s.npan == 1)
        hipLaunchKernelGGL(k_gs_mm<MM_FOLD_V>, dim3(4 * nb * nb), dim3(256), 0, st, A, M, Mt, W, s.Up, L.U, s.k, 0);
    else
        hipLaunchKernelGGL(k_gs_mm<MM_FOLD>, dim3(8 * ((nb * s.npan + 7) / 8) * (s.k / 64)), dim3(256), 0, st, A, M, Mt,
                           W, s.Up, L.U, s.k, 0);
    GS_TRY(hipGetLastError());
    if (L.ev_pre) GS_TRY(hipEventRecord(L.ev_pre, st));
    auto refresh = [&](bool rows) -> hipError_t {
        if (L.sp) return gs_sparse_refresh(L, rows, st);
        if (rows) {
            hipLaunchKernelGGL(k_gs_rows<T>, dim3((L.B + 15) / 16), dim3(256), 0, st, H, L.ld, L.B, L.U, y, x, r, done);
            GS_TRY(hipGetLastError());
        }
        hipLaunchKernelGGL(k_gs_grad<T>, dim3(s.Up), dim3(256), 0, st, H, L.ld, L.B, L.U, r, x, L.lambda, b, done);
        return hipGetLastError();
    };
    if (L.ev_init) GS_TRY(hipEventRecord(L.ev_init, st));
    GsSweepArgs g;
    g.W = W;
    g.M = M;
    g.b = b;
    g.x = x;
    g.xch = (uint64_t*)L.ctr + GS_CTR_WORDS / 2;
    g.abort_flag = L.ctr + 2;
    g.done = done;
    g.info = L.info;
    g.tol = L.tol;
    g.timeout_ticks = L.timeout_ticks;
    g.npan = s.npan;
    g.Up = s.Up;
    g.H = L.H;
    g.y = L.y;
    g.r = r;
    g.arrived = L.ctr + 6;
    g.ld = L.ld;
    g.B = L.B;
    g.U = L.U;
    g.lambda = L.lambda;
    // A cooperative launch costs 22 us of idle time around it.  Up to 512 users of a dense channel
    // one launch runs all sweeps and forms b anew itself; 40 sweeps, launches / in one: 400 x 150
    // 235 / 199 us, 800 x 300 300 / 271, 1500 x 500 335 / 320.  At 1024 users V leaves no registers
    // for the loads of the two products with H (3000 x 1000: 44 us each time against 32), and tall
    // channels want more workgroups for them than the sweep has.
    const bool whole = gs_whole(s, L.B, L.U) && !L.sp;
    const void* const fn = s.one ? nullptr : (whole ? gs_sweep_fn<T>(s) : gs_sweep_fn<void>(s));
    for (int t0 = 0, t1; t0 < L.T_max; t0 = t1) {
        GS_TRY(refresh(t0 > 0 || L.x0));
        t1 = whole ? L.T_max : gs_segment_end(t0, L.T_max);
        if (s.one) {
            hipLaunchKernelGGL(k_gs_one, dim3(1), dim3(512), 0, st, W, M, b, x, L.U, t0, t1, L.tol, done, L.info);
            GS_TRY(hipGetLastError());
        } else {
            void* args[] = {&g, &t0, &t1};
            GS_TRY(hipLaunchCooperativeKernel(fn, dim3(s.P), dim3(64 * (8 + GS_CW)), args, gs_sweep_lds(s), st));
        }
    }
    if (L.ev_sweep) GS_TRY(hipEventRecord(L.ev_sweep, st));
    hipLaunchKernelGGL(k_gs_finish<T>, dim3(1), dim3(1024), 0, st, x, L.U, (cv<T>*)L.x, L.ctr + 3, L.info);
    return hipGetLastError();
}

hipError_t gs_setup(const GsShape& s) {
    if (!s.one && (!gs_sweep_fn<void>(s) || s.P * s.R != s.Up || s.k % s.R != 0)) return hipErrorInvalidValue;
    auto allow = [](const void* fn, size_t lds) {
        return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    };
    if (!s.one && gs_sweep_lds(s) > 0) GS_TRY(allow(gs_sweep_fn<void>(s), gs_sweep_lds(s)));
    return allow((const void*)k_gs_inv64, GS_INV_LDS);
}

hipError_t launch_gs(const GsLaunch& L, hipStream_t st) {
    return L.c128 ? launch_gs_t<double>(L, st) : launch_gs_t<float>(L, st);
}

}  // namespace cdm
