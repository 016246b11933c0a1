// k_small.hip -- decentralized detection and precoding of many small clustered problems.
//
// The shape of the paper's throughput measurements (Sec. VI): S subcarriers, each with a
// channel H_s (B x U, B = C * B_c antennas in C clusters) shared by V received vectors.
// For every (s, v) each cluster c runs T sweeps of Algorithm 1 on its rows
// (H_{s,c}, y_{s,v,c}) from x = 0, and the C local estimates are fused (Sec. III):
//   x_hat = sum_c lambda_c x_c,  lambda_c = sigma_c^-2 / sum_c' sigma_c'^-2,
//   sigma_c^2 = (N0 / U) sum_u m_{u,c}  (N0/U cancels: lambda_c = s_c^-1 / sum s_c'^-1).
//
// The V vectors of a subcarrier share H_{s,c}, so the sweeps run on b = H^H (y - H x) -
// lambda x (U values) instead of the residual (B_c values): with G = H^H H + lambda I,
//   delta_u = m_u b_u,  x_u += delta_u,  b <- b - G_{:,u} delta_u,
// the same numbers in exact arithmetic, with U instead of 2 B_c complex multiply-adds per
// coordinate and no reduction on the chain.  G and H^H y are one contraction on the matrix
// cores.  The precoder (Algorithm 2) has the same recursion: x_c = H z with
//   delta_u = (s - H^H H z)_u / ||h_u||^2,  z_u += delta_u,
// so b starts as s, lambda is 0, and H z is one more contraction at the end.
// complex64 runs in FP64 throughout (v_mfma_f64_16x16x4_f64; the vector rate equals the
// unpacked FP32 one): in FP32 b would lose twice the digits that the residual form loses.
// Complex FP16: FP16 products (exact in FP32) and FP32 from there on.
//
// Mapping: a wave per (subcarrier, cluster), 16 vectors at a time.
//   Contractions: lane = 16 q + j.  The real and the imaginary parts of eight users are the
//   16 rows of one operand A and, for G, the 16 columns of the other (the same registers),
//   so one pass over the 32 antennas gives all four real products; H^H y has eight vectors'
//   real and imaginary parts as columns.  The operands need no staging: any order of the
//   contraction index serves, so lane group q takes antennas 8 q .. 8 q + 7, which are
//   contiguous in memory.  A pair of lanes (re, im column) adds its products into b and G.
//   Sweeps: lane = 4 v + p holds users p, p + 4, ... of vector v (b, x, and its rows of G;
//   these come through the wave's own LDS), and delta_u goes from lane u mod 4 of the quad
//   to the others by DPP.
// 1200 x 15, U = 8 (a call, launch included; before: quads of lanes on the residual):
//   detection, complex64, C = 4, 3 sweeps 25.3 -> 16.3 us; FP16 22.5 -> 8.4 us;
//   precoding, FP16, C = 8, 2 sweeps 30.2 -> 14.1 us; complex64, C = 4, 3 sweeps 25 -> 18 us.
// Bound in FP64 by the contractions (24 matrix instructions a wave at about 100 cycles each:
// 5.4 of the 14 us that one sweep takes) and by the sweep's vector work (1.5 us a sweep),
// in FP16 by the launch and the one round trip of a wave that does one block.
// Tried in FP64: the coordinates of a vector over four rows of 16 lanes (delta by permlane
// swaps) 24.2 us; a lane per vector, b and x in registers 49 us (spills).
#include <hip/hip_fp16.h>

#include <algorithm>
#include <cmath>

#include "common.hpp"
#include "la_common.hpp"
#include "launch.hpp"

namespace cdm {

constexpr int SM_BMAX = 32;           // antennas per cluster at most
constexpr int SM_UMAX = 16;           // users per cluster at most
constexpr size_t SM_LIMIT = 64 * 1024;

// Largest V of a call: S(C, V, U) <= 64 KB, the limit the interface has for one subcarrier's
// channel, local estimates and weights.
template <int UMAX> static size_t sm_call_bytes(int C, int V, bool f16) {
    const size_t esz = f16 ? 4 : 8, blk = (size_t)UMAX * SM_BMAX + (f16 ? 4 : 2);
    return (size_t)C * blk * esz + (size_t)C * V * UMAX * 8 + (size_t)C * 4;
}

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));

// DPP move of a whole value: quad_perm and row controls
template <int CTRL> __device__ __forceinline__ float dpp_all(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, false));
}
template <int CTRL> __device__ __forceinline__ double dpp_all(double v) {
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, false),
                            __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, false));
}
template <typename T> __device__ __forceinline__ T rows_sum(T v) { return swap_add<32>(swap_add<16>(v)); }

// The two number types.  T: the sweep's type.  E: stored complex value.  Op: eight antennas
// of one column, real or imaginary part.
//   part(i), user(i): what row (or column) i of an operand holds, chosen so that accumulator
//   elements 0, 1 of lane (q, j) are the real rows of users q and q + 4 and elements 2, 3
//   their imaginary rows; PAIR: the DPP move from the column of the other part.
template <bool F16> struct SmNum;
template <> struct SmNum<false> {
    using T = double;
    using T2 = double2;
    using E = float2;
    using acc = d4;
    struct Op {
        float v[8];
    };
    static constexpr int PAIR = 0x128;   // row_ror:8
    __device__ static int part(int i) { return i >> 3; }
    __device__ static int user(int i) { return i & 7; }
    // antennas 0..n-1 (at most 8) of p, zero past them
    __device__ static void load(Op& r, const E* p, int n, bool vec, bool im) {
        float2 w[8];
        if (vec) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float4 t = reinterpret_cast<const float4*>(p)[k];
                w[2 * k] = make_float2(t.x, t.y);
                w[2 * k + 1] = make_float2(t.z, t.w);
            }
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k) w[k] = k < n ? p[k] : make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) r.v[k] = im ? w[k].y : w[k].x;
    }
    __device__ static acc mul(const Op& a, const Op& b) {
        acc c = {0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < 8; ++k)
            c = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a.v[k], (double)b.v[k], c, 0, 0, 0);
        return c;
    }
    __device__ static acc mm4(T a, T b, acc c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
    // antenna (of 16) that operand lane i holds so that lane (q, j) receives antennas 4 q + e
    __device__ static int antenna(int i) { return 4 * (i & 3) + (i >> 2); }
    __device__ static float2 get(E e) { return e; }
    __device__ static E put(T re, T im) { return make_float2((float)re, (float)im); }
};
template <> struct SmNum<true> {
    using T = float;
    using T2 = float2;
    using E = __half2;      // (re, im)
    using acc = f4;
    struct Op {
        h8 v;
    };
    static constexpr int PAIR = 0x4e;    // quad_perm [2,3,0,1]
    __device__ static int part(int i) { return (i & 3) >> 1; }
    __device__ static int user(int i) { return (i >> 2) + 4 * (i & 1); }
    __device__ static void load(Op& r, const E* p, int n, bool vec, bool im) {
        uint32_t w[8];
        if (vec) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const uint4 t = reinterpret_cast<const uint4*>(p)[k];
                w[4 * k] = t.x;
                w[4 * k + 1] = t.y;
                w[4 * k + 2] = t.z;
                w[4 * k + 3] = t.w;
            }
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k) w[k] = k < n ? reinterpret_cast<const uint32_t*>(p)[k] : 0u;
        }
        const int sh = im ? 16 : 0;
        uint32_t a[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) a[k] = ((w[2 * k] >> sh) & 0xffffu) | ((w[2 * k + 1] >> sh) << 16);
        __builtin_memcpy(&r.v, a, 16);
    }
    __device__ static acc mul(const Op& a, const Op& b) {
        const acc c = {0, 0, 0, 0};
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(a.v, b.v, c, 0, 0, 0);
    }
    __device__ static acc mm4(T a, T b, acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    __device__ static int antenna(int i) { return i; }
    __device__ static float2 get(E e) { return __half22float2(e); }
    __device__ static E put(T re, T im) { return __floats2half2_rn(re, im); }
};

// LDS of one wave: G by columns, and b (then x or z) of 16 vectors, the rows padded to 20 so
// that the sixteen lanes of four quads read different banks.
template <bool F16, int UMAX> struct SmBlock {
    using T2 = typename SmNum<F16>::T2;
    T2 g[UMAX * UMAX];
    T2 b[UMAX][20];
    typename SmNum<F16>::T rs;   // 1 / sum_u m_u, 0 without an active coordinate
};

template <int I, int N, class F> __device__ __forceinline__ void unrolled(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        unrolled<I + 1, N>(f);
    }
}

// The wave's cluster: its operands, G and the sweeps.
template <bool F16, int UMAX> struct SmWave {
    using N = SmNum<F16>;
    using T = typename N::T;
    using T2 = typename N::T2;
    using Blk = SmBlock<F16, UMAX>;
    static constexpr int NS = UMAX / 4;      // users per lane in the sweeps: p + 4 s
    static constexpr int NT = UMAX / 8;      // operand tiles of eight users
    // this lane's rows of G: in registers for FP32 and U <= 8 (32 of them), else from LDS in
    // every sweep (in FP64 the 64 registers cost more in waves per SIMD than the reads:
    // 20.9 against 14.0 us at one sweep)
    static constexpr bool GREG = F16 && UMAX == 8;
    typename N::Op a[NT];
    T2 g[GREG ? NS : 1][GREG ? UMAX : 1];
    T m[NS];

    __device__ void load(const typename N::E* h, int B, int U, int n, int j, int vec) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int u = 8 * t + N::user(j);
            N::load(a[t], h + (int64_t)min(u, U - 1) * B, u < U ? n : 0, vec && u < U, N::part(j) != 0);
        }
    }
    // the two parts of A^H B for column j's part: z holds, for its column, the products with
    // the real (0, 1) and the imaginary (2, 3) rows of users q, q + 4
    __device__ static void combine(const typename N::acc& z, bool im, T& v0, T& v1) {
        const T w0 = dpp_all<N::PAIR>(z[2]), w1 = dpp_all<N::PAIR>(z[3]);
        v0 = im ? z[0] - w0 : z[0] + w0;
        v1 = im ? z[1] - w1 : z[1] + w1;
    }
    // G = H^H H into LDS
    __device__ void gram(int lane, Blk& o) const {
        const int j = lane & 15, q = lane >> 4;
        const bool im = N::part(j) != 0;
        T* gf = reinterpret_cast<T*>(o.g) + N::part(j);
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int c = 0; c <= t; ++c) {
                T v0, v1;
                combine(N::mul(a[t], a[c]), im, v0, v1);
                const int col = 8 * c + N::user(j), row = 8 * t + q;
                gf[(col * UMAX + row) * 2] = v0;
                gf[(col * UMAX + row + 4) * 2] = v1;
                if (c < t) {   // the tile above the diagonal is the conjugate
                    gf[(row * UMAX + col) * 2] = im ? -v0 : v0;
                    gf[((row + 4) * UMAX + col) * 2] = im ? -v1 : v1;
                }
            }
    }
    // m_u = 1 / (||h_u||^2 + lambda) (a column with ||h_u||^2 + lambda == 0, or past U, stays
    // inactive: 0), and lambda on the diagonal
    __device__ void coefficients(int lane, int U, T lambda, Blk& o) {
        const int p = lane & 3;
        T ms = T(0);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int u = 4 * s + p;
            const T d = o.g[u * UMAX + u].x + lambda;
            m[s] = u < U && !(d == T(0)) ? T(1) / d : T(0);
            ms += m[s];
        }
        ms += dpp_all<0xb1>(ms);
        ms += dpp_all<0x4e>(ms);
        if (lane == 0) o.rs = ms > T(0) ? T(1) / ms : T(0);
        if constexpr (GREG) {
#pragma unroll
            for (int u = 0; u < UMAX; ++u)
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    g[s][u] = o.g[u * UMAX + 4 * s + p];
                    if (u == 4 * s + p) g[s][u].x += lambda;
                }
        } else if (lane < 4) {
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const int u = 4 * s + p;
                o.g[u * UMAX + u].x += lambda;
            }
        }
    }
    // Tn sweeps from x = 0: b in, x out
    __device__ void sweeps(T2 (&b)[NS], T2 (&x)[NS], const Blk& o, int lane, int U, int Tn) const {
        const int p = lane & 3;
#pragma unroll
        for (int s = 0; s < NS; ++s) x[s].x = x[s].y = T(0);
        for (int it = 0; it < Tn; ++it) {
            unrolled<0, UMAX>([&](auto uc) {
                constexpr int u = decltype(uc)::value, so = u >> 2, po = u & 3;
                if (u < U) {
                    const T mr = m[so] * b[so].x, mi = m[so] * b[so].y;
                    if (p == po) {
                        x[so].x += mr;
                        x[so].y += mi;
                    }
                    const T dr = dpp_all<po * 0x55>(mr), di = dpp_all<po * 0x55>(mi);
#pragma unroll
                    for (int s = 0; s < NS; ++s) {
                        T2 c;
                        if constexpr (GREG)
                            c = g[s][u];
                        else
                            c = o.g[u * UMAX + 4 * s + p];
                        b[s].x -= c.x * dr - c.y * di;
                        b[s].y -= c.x * di + c.y * dr;
                    }
                }
            });
        }
    }
};

}  // namespace

// A wave per (subcarrier, cluster); a workgroup holds whole subcarriers (NW = 4 or 8 waves)
// and fuses the estimates of each through LDS, 16 vectors at a time.
template <bool F16, int UMAX, int NW>
__global__ __launch_bounds__(64 * NW, 16 / NW) void k_detect_small(const typename SmNum<F16>::E* __restrict__ H,
                                                          const typename SmNum<F16>::E* __restrict__ Y,
                                                          typename SmNum<F16>::E* __restrict__ X, int S, int V, int C,
                                                          int Bc, int U, int Tn, double lambda, int vec) {
    using N = SmNum<F16>;
    using T = typename N::T;
    using T2 = typename N::T2;
    using W = SmWave<F16, UMAX>;
    __shared__ SmBlock<F16, UMAX> blk[NW];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int j = lane & 15, q = lane >> 4;
    const int s = blockIdx.x * (NW / C) + wv / C, c = wv % C;
    const bool live = s < S;
    const int B = C * Bc, n = Bc - 8 * q;        // this lane's antennas: 8 q .. 8 q + n - 1 (at most 8)
    const int64_t off = c * Bc + 8 * q;
    SmBlock<F16, UMAX>& o = blk[wv];
    const bool im = N::part(j) != 0;
    W w;
    auto load_y = [&](typename N::Op(&y)[2], int v0) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int v = v0 + 8 * t + N::user(j);
            N::load(y[t], Y + ((int64_t)s * V + min(v, V - 1)) * B + off, v < V ? n : 0, vec && v < V, im);
        }
    };
    typename N::Op y[2];
    if (live) {
        w.load(H + (int64_t)s * U * B + off, B, U, n, j, vec);
        load_y(y, 0);
        w.gram(lane, o);
    }
    for (int v0 = 0; v0 < V; v0 += 16) {
        if (v0) __syncthreads();                 // the last round's estimates have been read
        if (live) {
            T* bf = reinterpret_cast<T*>(o.b) + N::part(j);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                if (v0 + 8 * t >= V) break;      // no vector in this tile of eight
#pragma unroll
                for (int k = 0; k < W::NT; ++k) {
                    T r0, r1;
                    W::combine(N::mul(w.a[k], y[t]), im, r0, r1);
                    const int u = 8 * k + q, v = 8 * t + N::user(j);
                    bf[(u * 20 + v) * 2] = r0;
                    bf[((u + 4) * 20 + v) * 2] = r1;
                }
            }
            __builtin_amdgcn_wave_barrier();
            if (v0 == 0) w.coefficients(lane, U, (T)lambda, o);
            __builtin_amdgcn_wave_barrier();
            T2 b[W::NS], x[W::NS];
#pragma unroll
            for (int k = 0; k < W::NS; ++k) b[k] = o.b[4 * k + (lane & 3)][lane >> 2];
            w.sweeps(b, x, o, lane, U, Tn);
#pragma unroll
            for (int k = 0; k < W::NS; ++k) o.b[4 * k + (lane & 3)][lane >> 2] = x[k];
            if (v0 + 16 < V) load_y(y, v0 + 16);
        }
        __syncthreads();
        // fusion: lambda_c = s_c^-1 / sum_c' s_c'^-1 with s_c = sum_u m_{u,c} (the factor N0/U of
        // sigma_c^2 cancels); a cluster without an active coordinate (s_c = 0) gets 0
        if (live) {
            const SmBlock<F16, UMAX>* f = blk + wv - c;
            T tot = T(0);
            for (int k = 0; k < C; ++k) tot += f[k].rs;
            tot = tot > T(0) ? T(1) / tot : T(0);
            const int nv = min(16, V - v0);
            for (int e = c * 64 + lane; e < nv * U; e += 64 * C) {
                const int v = e / U, u = e - v * U;
                T ar = T(0), ai = T(0);
                for (int k = 0; k < C; ++k) {
                    const T g = f[k].rs * tot;
                    ar += g * f[k].b[u][v].x;
                    ai += g * f[k].b[u][v].y;
                }
                X[((int64_t)s * V + v0) * U + e] = N::put(ar, ai);
            }
        }
    }
}

// ---- downlink: Algorithm 2 on the same shape ---------------------------------------
// For every (s, v) each cluster c runs T sweeps of eq. (4) on its rows from x_c = 0
// with the broadcast symbols s_{s,v} (a zero column stays inactive), then scales x_c to norm
// rho_c = rho / sqrt(C) (Sec. IV-B; rho <= 0: no scaling).  The output of (s, v) is the
// stacked [x_1; ...; x_C] (B entries).  x_c = H z is formed once, after the sweeps on z: two
// tiles of 16 antennas, real and imaginary part.  No wave waits for another.
template <bool F16, int UMAX>
__global__ __launch_bounds__(256, 4) void k_precode_small(const typename SmNum<F16>::E* __restrict__ H,
                                                       const typename SmNum<F16>::E* __restrict__ Sym,
                                                       typename SmNum<F16>::E* __restrict__ X, int S, int V, int C,
                                                       int Bc, int U, int Tn, double rho_c, int vec) {
    using N = SmNum<F16>;
    using E = typename N::E;
    using T = typename N::T;
    using T2 = typename N::T2;
    using W = SmWave<F16, UMAX>;
    constexpr int NS = W::NS;
    __shared__ SmBlock<F16, UMAX> blk[4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int j = lane & 15, q = lane >> 4;
    const int64_t id = (int64_t)blockIdx.x * 4 + wv, s = id / C;
    if (s >= S) return;
    const int c = (int)(id - s * C);
    const int B = C * Bc;
    const E* Hc = H + s * U * B + c * Bc;
    SmBlock<F16, UMAX>& o = blk[wv];
    W w;
    w.load(Hc + 8 * q, B, U, Bc - 8 * q, j, vec);
    float2 hz[2][NS];   // the operands of H z: antennas of this lane, users q + 4 k
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int a = 16 * t + N::antenna(j);
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            const bool in = a < Bc && 4 * k + q < U;
            const float2 h = N::get(Hc[(int64_t)min(4 * k + q, U - 1) * B + min(a, Bc - 1)]);
            hz[t][k] = make_float2(in ? h.x : 0.f, in ? h.y : 0.f);
        }
    }
    auto load_s = [&](T2(&b)[NS], int v0) {
        const int v = v0 + (lane >> 2);
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            const int u = 4 * k + (lane & 3);
            const bool in = v < V && u < U;
            const float2 t = N::get(Sym[(s * V + min(v, V - 1)) * U + min(u, U - 1)]);
            b[k].x = in ? (T)t.x : T(0);
            b[k].y = in ? (T)t.y : T(0);
        }
    };
    T2 b[NS];
    load_s(b, 0);
    w.gram(lane, o);
    __builtin_amdgcn_wave_barrier();
    w.coefficients(lane, U, T(0), o);
    for (int v0 = 0; v0 < V; v0 += 16) {
        T2 x[NS];
        w.sweeps(b, x, o, lane, U, Tn);
#pragma unroll
        for (int k = 0; k < NS; ++k) o.b[4 * k + (lane & 3)][lane >> 2] = x[k];
        if (v0 + 16 < V) load_s(b, v0 + 16);
        __builtin_amdgcn_wave_barrier();
        const int v = v0 + j;
        T2 z[NS];
#pragma unroll
        for (int k = 0; k < NS; ++k) z[k] = o.b[4 * k + q][j];
        __builtin_amdgcn_wave_barrier();
        typename N::acc xr[2], xi[2];
        T nn = T(0);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            typename N::acc r = {0, 0, 0, 0}, i = {0, 0, 0, 0};
#pragma unroll
            for (int k = 0; k < NS; ++k) {
                r = N::mm4((T)hz[t][k].x, z[k].x, r);
                i = N::mm4((T)hz[t][k].y, z[k].x, i);
                r = N::mm4(-(T)hz[t][k].y, z[k].y, r);
                i = N::mm4((T)hz[t][k].x, z[k].y, i);
            }
            xr[t] = r;
            xi[t] = i;
#pragma unroll
            for (int e = 0; e < 4; ++e) nn += r[e] * r[e] + i[e] * i[e];
        }
        nn = rows_sum(nn);
        const T sc = rho_c > 0.0 && nn > T(0) ? (T)rho_c / sqrt(nn) : T(1);
        if (v < V) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int a0 = 16 * t + 4 * q;
                E e4[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) e4[e] = N::put(sc * xr[t][e], sc * xi[t][e]);
                E* xo = X + (s * V + v) * B + c * Bc + a0;
                if (vec) {
                    if constexpr (F16) {
                        uint4 t4;
                        __builtin_memcpy(&t4, e4, 16);
                        *reinterpret_cast<uint4*>(xo) = t4;
                    } else {
                        reinterpret_cast<float4*>(xo)[0] = make_float4(e4[0].x, e4[0].y, e4[1].x, e4[1].y);
                        reinterpret_cast<float4*>(xo)[1] = make_float4(e4[2].x, e4[2].y, e4[3].x, e4[3].y);
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (a0 + e < Bc) xo[e] = e4[e];
                }
            }
        }
    }
}

// 16-byte loads: whole blocks of 32 antennas and aligned buffers
static int sm_vec(const void* a, const void* b, const void* c, int Bc) {
    return Bc == SM_BMAX && (((uintptr_t)a | (uintptr_t)b | (uintptr_t)c) & 15) == 0;
}

template <bool F16, int UMAX>
static hipError_t launch_small(const void* H, const void* Y, void* X, int S, int V, int C, int Bc, int U, int T,
                               double lam, hipStream_t st) {
    using E = typename SmNum<F16>::E;
    const int vec = sm_vec(H, Y, nullptr, Bc);
    if (C == 8)
        hipLaunchKernelGGL((k_detect_small<F16, UMAX, 8>), dim3(S), dim3(512), 0, st, (const E*)H, (const E*)Y, (E*)X,
                           S, V, C, Bc, U, T, lam, vec);
    else
        hipLaunchKernelGGL((k_detect_small<F16, UMAX, 4>), dim3((unsigned)(((int64_t)S * C + 3) / 4)), dim3(256), 0, st, (const E*)H,
                           (const E*)Y, (E*)X, S, V, C, Bc, U, T, lam, vec);
    return hipGetLastError();
}

template <bool F16, int UMAX>
static hipError_t launch_precode(const void* H, const void* Sym, void* X, int S, int V, int C, int Bc, int U, int T,
                                 double rho_c, hipStream_t st) {
    using E = typename SmNum<F16>::E;
    hipLaunchKernelGGL((k_precode_small<F16, UMAX>), dim3((unsigned)(((int64_t)S * C + 3) / 4)), dim3(256), 0, st,
                       (const E*)H, (const E*)Sym, (E*)X, S, V, C, Bc, U, T, rho_c, sm_vec(H, X, nullptr, Bc));
    return hipGetLastError();
}

}  // namespace cdm

using namespace cdm;

extern "C" int32_t cdm_precode_batch(int32_t S, int32_t V, int32_t C, int32_t Bc, int32_t U, int32_t T_max,
                                     int32_t precision, const void* H, const void* Sym, double rho, void* X,
                                     void* stream) {
    if (!H || !Sym || !X) return CDM_EINVAL;
    if (!std::isfinite(rho)) return CDM_EINVAL;
    if (T_max < 1 || T_max > 100000) return CDM_EINVAL;
    if (precision != CDM_C64 && precision != CDM_C16) return CDM_EDTYPE;
    if (S < 1 || V < 1 || U < 1 || U > SM_UMAX || Bc < 1 || Bc > SM_BMAX) return CDM_ESHAPE;
    if (C != 1 && C != 2 && C != 4 && C != 8) return CDM_ESHAPE;
    if (Bc < U) return CDM_EINFEASIBLE;   // local zero-forcing needs Bc >= U
    const bool f16 = precision == CDM_C16;
    const double rho_c = rho > 0.0 ? rho / std::sqrt((double)C) : 0.0;
    hipStream_t st = (hipStream_t)stream;
    hipError_t e;
    if (f16)
        e = U <= 8 ? launch_precode<true, 8>(H, Sym, X, S, V, C, Bc, U, T_max, rho_c, st)
                   : launch_precode<true, 16>(H, Sym, X, S, V, C, Bc, U, T_max, rho_c, st);
    else
        e = U <= 8 ? launch_precode<false, 8>(H, Sym, X, S, V, C, Bc, U, T_max, rho_c, st)
                   : launch_precode<false, 16>(H, Sym, X, S, V, C, Bc, U, T_max, rho_c, st);
    return e == hipSuccess ? CDM_OK : CDM_EHIP;
}

extern "C" int32_t cdm_detect_batch(int32_t S, int32_t V, int32_t C, int32_t Bc, int32_t U, int32_t T_max,
                                    int32_t precision, const void* H, const void* Y, double N0, double Ex, void* X,
                                    void* stream) {
    if (!H || !Y || !X) return CDM_EINVAL;
    if (!(Ex > 0.0) || !(N0 >= 0.0) || !std::isfinite(N0) || !std::isfinite(Ex)) return CDM_EINVAL;
    if (T_max < 1 || T_max > 100000) return CDM_EINVAL;
    if (precision != CDM_C64 && precision != CDM_C16) return CDM_EDTYPE;
    if (S < 1 || V < 1 || U < 1 || U > SM_UMAX || Bc < 1 || Bc > SM_BMAX) return CDM_ESHAPE;
    if (C != 1 && C != 2 && C != 4 && C != 8) return CDM_ESHAPE;
    if (N0 == 0.0 && Bc < U) return CDM_EINFEASIBLE;   // lambda = 0: eq. (1) needs Bc >= U
    const bool f16 = precision == CDM_C16;
    if ((U <= 8 ? sm_call_bytes<8>(C, V, f16) : sm_call_bytes<16>(C, V, f16)) > SM_LIMIT) return CDM_ESHAPE;
    const double lam = N0 / Ex;
    hipStream_t st = (hipStream_t)stream;
    hipError_t e;
    if (f16)
        e = U <= 8 ? launch_small<true, 8>(H, Y, X, S, V, C, Bc, U, T_max, lam, st)
                   : launch_small<true, 16>(H, Y, X, S, V, C, Bc, U, T_max, lam, st);
    else
        e = U <= 8 ? launch_small<false, 8>(H, Y, X, S, V, C, Bc, U, T_max, lam, st)
                   : launch_small<false, 16>(H, Y, X, S, V, C, Bc, U, T_max, lam, st);
    return e == hipSuccess ? CDM_OK : CDM_EHIP;
}
