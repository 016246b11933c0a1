// k_wg.hip -- "one workgroup per instance" engine for Algorithm 1 (uplink CD).
//
// Each workgroup owns one instance (an antenna cluster's local problem, or one
// entry of an uneven batch) and runs the whole local CD of Algorithm 1 on it:
// preprocessing, init, T_max (or tolerance-bounded) cyclic sweeps, output.  The residual r
// stays in VGPRs for the whole solve (thread t owns rows t, t+NT, ...).
//
// Two forms.  Up to four rows per thread the columns are taken in panels of KP = 8 or 4
// (cd_panels): the KP dots of a panel are formed from the same residual, and the coupling
// inside the panel is resolved by the inverse M of its small D + L (the block form of the
// sweep: the same deltas in exact arithmetic), so a panel costs one reduction, one barrier
// and one pass of dependent steps where eight columns cost eight.  M is formed once per
// solve (wg_couplings, one read of H) and lives in LDS next to x.  Taller instances, and
// those whose M does not fit, go column by column (cd_instance).  Measured, column by column / panels: one uneven batch of 512 complex64
// instances (m in 64..2048, n = m / 2, to 1e-6) 40.8 / 18.2 ms; four clusters of 250 x 75
// in complex128, four sweeps, 246 / 67 us.  What bounds it: HBM once the batch fills
// the chip; a single instance by the chain of its panels (about 0.5 us each) and the FMAs
// of one CU.
#include "common.hpp"
#include "la_common.hpp"
#include "launch.hpp"
#include "wg.hpp"

namespace cdm {

// One uplink instance, RPT rows per thread (m <= NT * RPT).
template <typename T, int NT, int RPT>
__device__ __forceinline__ void cd_instance(const WgJob& jb, const cv<T>* __restrict__ H, const cv<T>* __restrict__ Y,
                                            const cv<T>* __restrict__ X0, cv<T>* __restrict__ X,
                                            cdm_info* __restrict__ info, T lambda, int T_max, double tol,
                                            double* __restrict__ msum, int64_t ld_arg, unsigned char* smem_raw,
                                            T (*red_s)[NT / 64][3], int& flag_s, int resid,
                                            double (*red64)[NT / 64][4], double lambda_d) {
    using V = cv<T>;
    constexpr int NW = NT / 64;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wid = tid >> 6;
        // ---------------------------------------------------------------- one instance
        const int m = jb.m, n = jb.n;
        const int64_t ld = jb.ld > 0 ? jb.ld : ld_arg;   // ld <= 0: the solve's leading dimension
        const V* Hj = H + jb.h_off;
        V* x_s = reinterpret_cast<V*>(smem_raw);
        V* cf_s = x_s + n;   // (m_u, n_u) of Algorithm 1

        // rows past m load row m - 1 (in bounds) and are zeroed by a select, so that
        // no load sits behind a branch; column bases stay wave-uniform
        uint32_t rowc[RPT];
        bool live[RPT];
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            const int i = tid + q * NT;
            live[q] = i < m;
            rowc[q] = (uint32_t)(live[q] ? i : m - 1) * (uint32_t)sizeof(V);
        }
        auto col = [&](int u, int q) -> V {
            const V v = *reinterpret_cast<const V*>(reinterpret_cast<const char*>(Hj + (int64_t)u * ld) + rowc[q]);
            return live[q] ? v : czero<T>();
        };
        V r[RPT];
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            const V v = *reinterpret_cast<const V*>(reinterpret_cast<const char*>(Y + jb.y_off) + rowc[q]);
            r[q] = live[q] ? v : czero<T>();
        }
        for (int u = tid; u < n; u += NT) x_s[u] = X0 ? X0[jb.x0_off + u] : czero<T>();
        __syncthreads();
        if (X0) {  // warm start: r = y - H x0
            for (int u = 0; u < n; ++u) {
                const V xu = x_s[u];
#pragma unroll
                for (int q = 0; q < RPT; ++q) cfms(r[q], col(u, q), xu);
            }
        }

        int sweeps = 0;
        double S = 0.0, Xn = 0.0;
        for (int t = 1; t <= T_max; ++t) {
            S = 0.0;
            Xn = 0.0;
            V hc[RPT], hn[RPT];
#pragma unroll
            for (int q = 0; q < RPT; ++q) hc[q] = col(0, q);
            for (int u = 0; u < n; ++u) {
                if (u + 1 < n) {
#pragma unroll
                    for (int q = 0; q < RPT; ++q) hn[q] = col(u + 1, q);
                }
                T gr = 0, gi = 0, ee = 0;
#pragma unroll
                for (int q = 0; q < RPT; ++q) {
                    gr += hc[q].x * r[q].x + hc[q].y * r[q].y;
                    gi += hc[q].x * r[q].y - hc[q].y * r[q].x;
                    if (t == 1) ee += hc[q].x * hc[q].x + hc[q].y * hc[q].y;
                }
                gr = wave_sum_last(gr);
                gi = wave_sum_last(gi);
                if (t == 1) ee = wave_sum_last(ee);
                // read x_u and the scalars before the barrier: thread 0 overwrites them after it
                const V xu = x_s[u];
                V cf = (t > 1) ? cf_s[u] : czero<T>();
                const int par = u & 1;
                if (lane == 63) {
                    red_s[par][wid][0] = gr;
                    red_s[par][wid][1] = gi;
                    red_s[par][wid][2] = ee;
                }
                __syncthreads();
                V g = czero<T>();
                T e = 0;
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    g.x += red_s[par][w][0];
                    g.y += red_s[par][w][1];
                    if (t == 1) e += red_s[par][w][2];
                }
                if (t == 1) {
                    // Algorithm 1 preprocessing: m_u = 1/(||h_u||^2 + lambda), n_u = m_u ||h_u||^2.
                    // A coordinate with ||h_u||^2 + lambda == 0 stays inactive: (m, n) = (0, 1).
                    if (e + lambda > T(0)) {
                        cf.x = T(1) / (e + lambda);
                        cf.y = cf.x * e;
                    } else {
                        cf.x = T(0);
                        cf.y = T(1);
                        if (tid == 0) flag_s |= CDM_INFO_ZERO_COLUMN;
                    }
                }
                // x_u <- m_u h_u^H r + n_u x_u ; delta = x_u(new) - x_u(old)
                V xn;
                xn.x = cf.x * g.x + cf.y * xu.x;
                xn.y = cf.x * g.y + cf.y * xu.y;
                V d;
                d.x = xn.x - xu.x;
                d.y = xn.y - xu.y;
                if (tid == 0) {
                    x_s[u] = xn;
                    if (t == 1) cf_s[u] = cf;
                }
                // r <- r - h_u delta
#pragma unroll
                for (int q = 0; q < RPT; ++q) cfms(r[q], hc[q], d);
                S += cabs2d(d);
                Xn += cabs2d(xn);
#pragma unroll
                for (int q = 0; q < RPT; ++q) hc[q] = hn[q];
            }
            __syncthreads();
            if (t == 1 && msum && tid == 0) {
                // sum_u m_u of this cluster, in index order (feeds the fusion weights)
                double ms = 0.0;
                for (int u = 0; u < n; ++u) ms += (double)cf_s[u].x;
                msum[jb.info_idx] = ms;
            }
            sweeps = t;
            if (tol > 0.0 && sqrt(S) <= tol * sqrt(Xn)) break;
        }
        // ---------------------------------------------------------------- output
        int nf = 0;
        for (int u = tid; u < n; u += NT) {
            const V v = x_s[u];
            if (!isfinite(v.x) || !isfinite(v.y)) nf = 1;
            X[jb.x_off + u] = v;
        }
        if (nf) atomicOr(&flag_s, CDM_INFO_NONFINITE);
        __syncthreads();
        // optional FP64 check of the stationarity of eq. (1)
        const double res = resid ? wg_fp64_resid<T, NT, RPT>(Hj, ld, Y + jb.y_off, x_s, m, n, lambda_d, red64) : -1.0;
        if (tid == 0) {
            const double rel = (Xn > 0.0) ? sqrt(S / Xn) : (S > 0.0 ? INFINITY : 0.0);
            int fl = flag_s;
            if (tol > 0.0 && !(rel <= tol)) fl |= CDM_INFO_NOT_CONVERGED;
            cdm_info o;
            o.sweeps = sweeps;
            o.flags = fl;
            o.rel_step = rel;
            o.resid = res;
            o.reserved = 0.0;
            info[jb.info_idx] = o;
        }
}

// Column by column, up to eight rows per thread.
template <typename T, int NT>
__global__ __launch_bounds__(NT) void k_cd_wg(const WgJob* __restrict__ jobs, int njobs,
                                              const cv<T>* __restrict__ H, const cv<T>* __restrict__ Y,
                                              const cv<T>* __restrict__ X0, cv<T>* __restrict__ X,
                                              cdm_info* __restrict__ info, double lambda_d, int T_max,
                                              double tol, const int* __restrict__ order,
                                              uint32_t* __restrict__ queue, double* __restrict__ msum,
                                              int64_t ld_arg, int resid, WgFuse<T> fuse) {
    constexpr int NW = NT / 64;
    extern __shared__ unsigned char smem_raw[];
    __shared__ T red_s[2][NW][3];
    __shared__ double red64[2][NW][4];
    __shared__ int flag_s;
    __shared__ int job_s;
    const int tid = threadIdx.x;
    const T lambda = (T)lambda_d;
    for (;;) {
        // next job from the shared queue; the queue hands out slots in `order`
        // (largest instances first for uneven batches)
        if (tid == 0) {
            job_s = queue ? (int)atomicAdd(queue, 1u) : (int)blockIdx.x;
            flag_s = 0;
        }
        __syncthreads();
        // wave-uniform job index: the job record and the column bases stay scalar
        const int jslot = __builtin_amdgcn_readfirstlane(job_s);
        if (jslot >= njobs) return;
        const WgJob jb = jobs[order ? __builtin_amdgcn_readfirstlane(order[jslot]) : jslot];
        // row tile of this job, chosen on the host per size bucket
        if (jb.rpt == 1)
            cd_instance<T, NT, 1>(jb, H, Y, X0, X, info, lambda, T_max, tol, msum, ld_arg, smem_raw, red_s, flag_s, resid, red64, lambda_d);
        else if (jb.rpt == 2)
            cd_instance<T, NT, 2>(jb, H, Y, X0, X, info, lambda, T_max, tol, msum, ld_arg, smem_raw, red_s, flag_s, resid, red64, lambda_d);
        else if (jb.rpt == 4)
            cd_instance<T, NT, 4>(jb, H, Y, X0, X, info, lambda, T_max, tol, msum, ld_arg, smem_raw, red_s, flag_s, resid, red64, lambda_d);
        else
            cd_instance<T, NT, 8>(jb, H, Y, X0, X, info, lambda, T_max, tol, msum, ld_arg, smem_raw, red_s, flag_s, resid, red64, lambda_d);
        if (!queue) {   // one job per workgroup
            if (fuse.count) wg_fuse<T>(fuse, &job_s);
            return;
        }
        __syncthreads();
    }
}

// ---- panels of KP columns ---------------------------------------------------------------
// Columns per panel for RPT rows per thread: two panels of columns in registers (this one and
// the next, in flight) within 128 VGPRs.
template <typename T, int RPT> constexpr int wg_kp() { return sizeof(T) * RPT >= 16 && sizeof(T) == 8 ? 4 : 8; }
// LDS values of one instance: x, and the packed lower triangle of M per panel (sized for the
// larger of the two widths' shares per column)
__host__ __device__ constexpr int wg_panel_values(int n) { return n + 8 + 36 * ((n + 7) / 8 + 1); }

// Sum of 16 values per lane over the wave: permlane swaps fold the halves and then the rows
// of 16 lanes (two values per instruction), DPP rotations finish inside the rows.  On return
// v[0..3] of row r hold values 4 r' + i, r' = r: lane (r, i) of the first four of its row
// takes value 4 r + i as the result.
template <typename T> __device__ __forceinline__ void swap2(T& a, T& b, std::integral_constant<int, 32>) {
    // a <- (a.lo, b.lo) + (a.hi, b.hi)
    if constexpr (sizeof(T) == 4) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        a = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    } else {
        const auto l = __builtin_amdgcn_permlane32_swap((uint32_t)__double2loint(a), (uint32_t)__double2loint(b), false, false);
        const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)__double2hiint(a), (uint32_t)__double2hiint(b), false, false);
        a = __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
    }
}
template <typename T> __device__ __forceinline__ void swap2(T& a, T& b, std::integral_constant<int, 16>) {
    if constexpr (sizeof(T) == 4) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        a = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    } else {
        const auto l = __builtin_amdgcn_permlane16_swap((uint32_t)__double2loint(a), (uint32_t)__double2loint(b), false, false);
        const auto h = __builtin_amdgcn_permlane16_swap((uint32_t)__double2hiint(a), (uint32_t)__double2hiint(b), false, false);
        a = __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
    }
}
// N = 8, 16 or 64 values: the lanes with (lane & 15) < N / 4 end with value
// (N / 4) (lane >> 4) + (lane & 15)
template <typename T, int N> __device__ __forceinline__ T wave_sums(T (&v)[N], int lane) {
#pragma unroll
    for (int i = 0; i < N / 2; ++i) swap2(v[i], v[i + N / 2], std::integral_constant<int, 32>{});
#pragma unroll
    for (int i = 0; i < N / 4; ++i) swap2(v[i], v[i + N / 4], std::integral_constant<int, 16>{});
#pragma unroll
    for (int i = 0; i < N / 4; ++i) {
        v[i] += row_ror<8>(v[i]);
        v[i] += row_ror<4>(v[i]);
        v[i] += row_ror<2>(v[i]);
        v[i] += row_ror<1>(v[i]);
    }
    T o = v[0];
#pragma unroll
    for (int i = 1; i < N / 4; ++i) o = (lane & 15) == i ? v[i] : o;
    return o;
}
// acc += conj(h) z
template <typename T, typename V> __device__ __forceinline__ void wg_dot(T& re, T& im, const V& h, const V& z) {
    re = fma(h.y, z.y, fma(h.x, z.x, re));
    im = fma(-h.y, z.x, fma(h.x, z.y, im));
}

// M = (D + L)^-1 of one panel, by one wave alone: the couplings G_vw = h_v^H h_w (w < v) and
// the energies over all rows (a lane per row modulo 64), their sums over the wave through
// `tot` (this wave's 64 values in LDS), then the inverse by substitution, a lane per column.
// One more read of H per solve, but no barrier and every wave busy: formed inside the first
// sweep instead, a panel at a time for the whole workgroup, the same work was a third of a
// solve of four sweeps.  Returns sum_v m_v (Algorithm 1's m_u = 1 / (||h_u||^2 + lambda)).
template <typename T, int KP>
__device__ __forceinline__ double wg_couplings(const cv<T>* __restrict__ Hj, int64_t ld, int m, int n, int p, T lambda,
                                               cv<T>* __restrict__ Mp, T* __restrict__ tot, int lane, int& flag_s) {
    using V = cv<T>;
    constexpr int NG = KP * (KP - 1) / 2, NV = 2 * NG + KP;   // 64 or 16
    T a[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) a[i] = T(0);
    V h[KP], nx[KP];
    auto fetch = [&](V(&o)[KP], int r0) __attribute__((always_inline)) {
        uint32_t off = (uint32_t)min(r0 + lane, m - 1) * (uint32_t)sizeof(V);
        asm("" : "+v"(off));
#pragma unroll
        for (int c = 0; c < KP; ++c)
            o[c] = *reinterpret_cast<const V*>(
                reinterpret_cast<const char*>(Hj + (int64_t)min(p * KP + c, n - 1) * ld) + off);
    };
    fetch(nx, 0);
    for (int r0 = 0; r0 < m; r0 += 64) {
        const bool in = r0 + lane < m;
#pragma unroll
        for (int c = 0; c < KP; ++c) h[c] = in ? nx[c] : czero<T>();
        if (r0 + 64 < m) fetch(nx, r0 + 64);
#pragma unroll
        for (int v = 0; v < KP; ++v) {
#pragma unroll
            for (int w = 0; w < v; ++w) wg_dot(a[v * (v - 1) + 2 * w], a[v * (v - 1) + 2 * w + 1], h[v], h[w]);
            a[2 * NG + v] = fma(h[v].y, h[v].y, fma(h[v].x, h[v].x, a[2 * NG + v]));
        }
    }
    T t = wave_sums<T, NV>(a, lane);
    const int idx = NV / 4 * (lane >> 4) + (lane & 15);
    double ms = 0.0;
    if ((lane & 15) < NV / 4) {
        if (idx >= 2 * NG) {
            // a coordinate with ||h_u||^2 + lambda == 0 stays inactive: m_u = 0
            const T d = t + lambda;
            const bool real = p * KP + idx - 2 * NG < n;
            if (real && d == T(0)) atomicOr(&flag_s, CDM_INFO_ZERO_COLUMN);
            t = real && !(d == T(0)) ? T(1) / d : T(0);
            ms = (double)t;
        }
        tot[idx] = t;
    }
    __builtin_amdgcn_wave_barrier();
    V mc[KP];
#pragma unroll
    for (int v = 0; v < KP; ++v) {
        V z = czero<T>();
        z.x = v == lane ? T(1) : T(0);
#pragma unroll
        for (int w = 0; w < v; ++w) cfms(z, cmake<T>(tot[v * (v - 1) + 2 * w], tot[v * (v - 1) + 2 * w + 1]), mc[w]);
        const T mv = tot[2 * NG + v];
        mc[v].x = v < lane ? T(0) : z.x * mv;
        mc[v].y = v < lane ? T(0) : z.y * mv;
        if (lane <= v) Mp[v * (v + 1) / 2 + lane] = mc[v];
        __builtin_amdgcn_sched_barrier(0);
    }
    return group_sum<1>(ms);
}

template <typename T, int NT, int RPT>
__device__ __forceinline__ void cd_panels(const WgJob& jb, const cv<T>* __restrict__ H, const cv<T>* __restrict__ Y,
                                          const cv<T>* __restrict__ X0, cv<T>* __restrict__ X,
                                          cdm_info* __restrict__ info, T lambda, int T_max, double tol,
                                          double* __restrict__ msum, int64_t ld_arg, unsigned char* smem_raw,
                                          T (*red)[NT / 64][16], T (*tot)[64], double* ms_s, int& flag_s, int resid,
                                          double (*red64)[NT / 64][4], double lambda_d) {
    using V = cv<T>;
    constexpr int NW = NT / 64, KP = wg_kp<T, RPT>(), NE = KP * (KP + 1) / 2;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int m = jb.m, n = jb.n;
    const int64_t ld = jb.ld > 0 ? jb.ld : ld_arg;   // ld <= 0: the solve's leading dimension
    const V* Hj = H + jb.h_off;
    V* x_s = reinterpret_cast<V*>(smem_raw);
    V* M_s = x_s + n + 8;                            // [panel][NE], row v of the lower triangle at v (v + 1) / 2
    // rows past m load row m - 1 and columns past n column n - 1 (in bounds), so that no load sits
    // behind a branch.  r stays 0 in rows past m, and the rows and columns of M past n are 0, so
    // what those loads bring is multiplied by 0 (and left out of the couplings)
    uint32_t rowc[RPT];
    bool live[RPT];
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int i = tid + q * NT;
        live[q] = i < m;
        rowc[q] = (uint32_t)(live[q] ? i : m - 1) * (uint32_t)sizeof(V);
    }
    auto col = [&](int u, int q) __attribute__((always_inline)) -> V {
        // the offset's extension to 64 bits stays next to the load, which then takes the column's
        // base from scalar registers (hoisted, every load in flight holds a 64-bit address)
        uint32_t o = rowc[q];
        asm("" : "+v"(o));
        return *reinterpret_cast<const V*>(reinterpret_cast<const char*>(Hj + (int64_t)u * ld) + o);
    };
    const int np = (n + KP - 1) / KP;
    auto load = [&](V(&h)[KP][RPT], int p) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < KP; ++c)
#pragma unroll
            for (int q = 0; q < RPT; ++q) h[c][q] = col(min(p * KP + c, n - 1), q);
    };
    V r[RPT];
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const V v = *reinterpret_cast<const V*>(reinterpret_cast<const char*>(Y + jb.y_off) + rowc[q]);
        r[q] = live[q] ? v : czero<T>();
    }
    for (int u = tid; u < n + 8; u += NT) x_s[u] = X0 && u < n ? X0[jb.x0_off + u] : czero<T>();
    __syncthreads();
    if (X0) {  // warm start: r = y - H x0
        for (int u = 0; u < n; ++u) {
            const V xu = x_s[u];
#pragma unroll
            for (int q = 0; q < RPT; ++q)
                if (live[q]) cfms(r[q], col(u, q), xu);
        }
    }
    // lane (v, w) of the panel's small products: v = row (delta), w = column (b)
    const int lv = lane & (KP - 1), lw = (lane / KP) & (KP - 1);
    double S = 0.0, Xn = 0.0;
    int par = 0, sweeps = 0;
    {
        double ms = 0.0;
        for (int p = wid; p < np; p += NW) ms += wg_couplings<T, KP>(Hj, ld, m, n, p, lambda, M_s + p * NE, tot[wid], lane, flag_s);
        if (lane == 0) ms_s[wid] = ms;
        __syncthreads();
        if (msum && tid == 0) {   // sum_u m_u of this cluster (feeds the fusion weights)
            double all = 0.0;
            for (int k = 0; k < NW; ++k) all += ms_s[k];
            msum[jb.info_idx] = all;
        }
    }

    auto panel = [&](V(&h)[KP][RPT], int p) __attribute__((always_inline)) {
        const int u0 = p * KP;
        // g_c = h_c^H r over this thread's rows, all columns of the panel at once
        T a[2 * KP];
#pragma unroll
        for (int c = 0; c < KP; ++c) {
            T gr = T(0), gi = T(0);
#pragma unroll
            for (int q = 0; q < RPT; ++q) wg_dot(gr, gi, h[c][q], r[q]);
            a[2 * c] = gr;
            a[2 * c + 1] = gi;
        }
        const T o = wave_sums<T, 2 * KP>(a, lane);
        constexpr int Q = KP / 2;
        if ((lane & 15) < Q) red[par][wid][Q * (lane >> 4) + (lane & 15)] = o;
        V mvw = czero<T>();
        if (lw <= lv) mvw = M_s[p * NE + lv * (lv + 1) / 2 + lw];
        __syncthreads();
        const V* rp = reinterpret_cast<const V*>(&red[par][0][0]);
        V b = czero<T>();
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            const V t = rp[k * 8 + lw];
            b.x += t.x;
            b.y += t.y;
        }
        const V xw = x_s[u0 + lw], xv = x_s[u0 + lv];
        b.x -= lambda * xw.x;
        b.y -= lambda * xw.y;
        // delta_v = sum_w M_vw b_w: every lane of row v ends with it
        V d = cmul(mvw, b);
        if (lw > lv) d = czero<T>();
        if constexpr (KP == 4) {
            d.x += row_ror<4>(d.x);
            d.y += row_ror<4>(d.y);
            d.x += row_ror<8>(d.x);
            d.y += row_ror<8>(d.y);
        } else {
            d.x += row_ror<8>(d.x);
            d.y += row_ror<8>(d.y);
            d.x = swap_add<16>(d.x);
            d.y = swap_add<16>(d.y);
            d.x = swap_add<32>(d.x);
            d.y = swap_add<32>(d.y);
        }
        if (lane < KP) {
            const V xn = cmake<T>(xv.x + d.x, xv.y + d.y);
            S += cabs2d(d);
            Xn += cabs2d(xn);
            if (wid == 0) x_s[u0 + lane] = xn;   // next read behind the barrier of a later panel
        }
        // r <- r - H_p delta: the panel's sum first, so that r is rounded once
        V dc[KP];
#pragma unroll
        for (int c = 0; c < KP; ++c) dc[c] = cmake<T>(lane_value(d.x, c), lane_value(d.y, c));
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            V z = cmul(h[0][q], dc[0]);
#pragma unroll
            for (int c = 1; c < KP; ++c) {
                z.x = fma(-h[c][q].y, dc[c].y, fma(h[c][q].x, dc[c].x, z.x));
                z.y = fma(h[c][q].y, dc[c].x, fma(h[c][q].x, dc[c].y, z.y));
            }
            r[q].x = live[q] ? r[q].x - z.x : T(0);
            r[q].y = live[q] ? r[q].y - z.y : T(0);
        }
        par ^= 1;
    };

    V ha[KP][RPT], hb[KP][RPT];
    for (int t = 1; t <= T_max; ++t) {
        S = Xn = 0.0;
        load(ha, 0);
        for (int p = 0; p < np; p += 2) {
            if (p + 1 < np) load(hb, p + 1);
            panel(ha, p);
            if (p + 1 < np) {
                if (p + 2 < np) load(ha, p + 2);
                panel(hb, p + 1);
            }
        }
        // the panel's sums sit in the first KP lanes, equal in every wave
        S = lane < KP ? S : 0.0;
        Xn = lane < KP ? Xn : 0.0;
        S = group_sum<1>(S);
        Xn = group_sum<1>(Xn);
        sweeps = t;
        if (tol > 0.0 && sqrt(S) <= tol * sqrt(Xn)) break;
    }
    __syncthreads();
    // ---------------------------------------------------------------- output
    int nf = 0;
    for (int u = tid; u < n; u += NT) {
        const V v = x_s[u];
        if (!isfinite(v.x) || !isfinite(v.y)) nf = 1;
        X[jb.x_off + u] = v;
    }
    if (nf) atomicOr(&flag_s, CDM_INFO_NONFINITE);
    __syncthreads();
    // optional FP64 check of the stationarity of eq. (1)
    const double res = resid ? wg_fp64_resid<T, NT, RPT>(Hj, ld, Y + jb.y_off, x_s, m, n, lambda_d, red64) : -1.0;
    if (tid == 0) {
        const double rel = (Xn > 0.0) ? sqrt(S / Xn) : (S > 0.0 ? INFINITY : 0.0);
        int fl = flag_s;
        if (tol > 0.0 && !(rel <= tol)) fl |= CDM_INFO_NOT_CONVERGED;
        cdm_info o;
        o.sweeps = sweeps;
        o.flags = fl;
        o.rel_step = rel;
        o.resid = res;
        o.reserved = 0.0;
        info[jb.info_idx] = o;
    }
}

template <typename T, int NT>
__global__ __launch_bounds__(NT) void k_cd_wgp(const WgJob* __restrict__ jobs, int njobs,
                                               const cv<T>* __restrict__ H, const cv<T>* __restrict__ Y,
                                               const cv<T>* __restrict__ X0, cv<T>* __restrict__ X,
                                               cdm_info* __restrict__ info, double lambda_d, int T_max,
                                               double tol, const int* __restrict__ order,
                                               uint32_t* __restrict__ queue, double* __restrict__ msum,
                                               int64_t ld_arg, int resid, WgFuse<T> fuse) {
    constexpr int NW = NT / 64;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    __shared__ __attribute__((aligned(16))) T red[2][NW][16];
    __shared__ T tot[NW][64];
    __shared__ double ms_s[NW];
    __shared__ double red64[2][NW][4];
    __shared__ int flag_s;
    __shared__ int job_s;
    const T lambda = (T)lambda_d;
    for (;;) {   // jobs from the shared queue, as in k_cd_wg
        if (threadIdx.x == 0) {
            job_s = queue ? (int)atomicAdd(queue, 1u) : (int)blockIdx.x;
            flag_s = 0;
        }
        __syncthreads();
        const int jslot = __builtin_amdgcn_readfirstlane(job_s);
        if (jslot >= njobs) return;
        const WgJob jb = jobs[order ? __builtin_amdgcn_readfirstlane(order[jslot]) : jslot];
        if (jb.rpt == 1)
            cd_panels<T, NT, 1>(jb, H, Y, X0, X, info, lambda, T_max, tol, msum, ld_arg, smem_raw, red, tot, ms_s, flag_s, resid, red64, lambda_d);
        else if (jb.rpt == 2)
            cd_panels<T, NT, 2>(jb, H, Y, X0, X, info, lambda, T_max, tol, msum, ld_arg, smem_raw, red, tot, ms_s, flag_s, resid, red64, lambda_d);
        else
            cd_panels<T, NT, 4>(jb, H, Y, X0, X, info, lambda, T_max, tol, msum, ld_arg, smem_raw, red, tot, ms_s, flag_s, resid, red64, lambda_d);
        if (!queue) {   // one job per workgroup
            if (fuse.count) wg_fuse<T>(fuse, &job_s);
            return;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Algorithm 2 (decentralized ZF precoding by CD, eq. (4)), one workgroup per
// cluster.  The local precoded vector x_c (B_c entries) stays in VGPRs with the
// same row ownership as the uplink residual; per user u:
//   a = h_u^H x (partial, wave butterfly, LDS)      e = p_u a - p_u s_u
//   x <- x - e p_u h_u
// with p_u = 1/||h_u|| computed from the same column load in the first sweep
// (Algorithm 2 preprocessing: hbar_u = p_u h_u, sbar_u = p_u s_u).  After the
// sweeps: x_c <- rho_c x_c / ||x_c|| with rho_c = rho / sqrt(C) (Sec. IV-B).
template <typename T, int NT, int RPT>
__device__ __forceinline__ void zf_instance(const WgJob& jb, const cv<T>* __restrict__ H, const cv<T>* __restrict__ S,
                                            cv<T>* __restrict__ X, cdm_info* __restrict__ info, int T_max,
                                            double tol, double rho_c, int64_t ld_arg, unsigned char* smem_raw,
                                            T (*red_s)[NT / 64][3], double* nrm_s, int& flag_s) {
    using V = cv<T>;
    constexpr int NW = NT / 64;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wid = tid >> 6;
        const int m = jb.m, n = jb.n;
        const int64_t ld = jb.ld > 0 ? jb.ld : ld_arg;
        const V* Hj = H + jb.h_off;
        T* p_s = reinterpret_cast<T*>(smem_raw);   // p_u (0 marks an inactive user)

        V x[RPT];
#pragma unroll
        for (int q = 0; q < RPT; ++q) x[q] = czero<T>();

        int sweeps = 0;
        double Ssum = 0.0, Xn = 0.0;
        for (int t = 1; t <= T_max; ++t) {
            Ssum = 0.0;
            V hc[RPT], hn[RPT];
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                const int i = tid + q * NT;
                hc[q] = (i < m) ? Hj[i] : czero<T>();
            }
            for (int u = 0; u < n; ++u) {
                if (u + 1 < n) {
#pragma unroll
                    for (int q = 0; q < RPT; ++q) {
                        const int i = tid + q * NT;
                        hn[q] = (i < m) ? Hj[(int64_t)(u + 1) * ld + i] : czero<T>();
                    }
                }
                T ar = 0, ai = 0, ee = 0;
#pragma unroll
                for (int q = 0; q < RPT; ++q) {
                    ar += hc[q].x * x[q].x + hc[q].y * x[q].y;
                    ai += hc[q].x * x[q].y - hc[q].y * x[q].x;
                    if (t == 1) ee += hc[q].x * hc[q].x + hc[q].y * hc[q].y;
                }
                ar = wave_allsum(ar);
                ai = wave_allsum(ai);
                if (t == 1) ee = wave_allsum(ee);
                const T pu_old = (t > 1) ? p_s[u] : T(0);
                const V su = S[jb.y_off + u];
                const int par = u & 1;
                if (lane == 0) {
                    red_s[par][wid][0] = ar;
                    red_s[par][wid][1] = ai;
                    red_s[par][wid][2] = ee;
                }
                __syncthreads();
                V a = czero<T>();
                T e = 0;
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    a.x += red_s[par][w][0];
                    a.y += red_s[par][w][1];
                    if (t == 1) e += red_s[par][w][2];
                }
                T pu = pu_old;
                if (t == 1) {
                    pu = (e > T(0)) ? T(1) / sqrt(e) : T(0);
                    if (!(e > T(0)) && tid == 0) flag_s |= CDM_INFO_ZERO_COLUMN;
                    if (tid == 0) p_s[u] = pu;
                }
                // err = hbar_u^H x - sbar_u ;  x <- x - err * hbar_u
                V err;
                err.x = pu * a.x - pu * su.x;
                err.y = pu * a.y - pu * su.y;
                V ep;
                ep.x = err.x * pu;
                ep.y = err.y * pu;
#pragma unroll
                for (int q = 0; q < RPT; ++q) cfms(x[q], hc[q], ep);
                if (pu != T(0)) Ssum += cabs2d(err);
#pragma unroll
                for (int q = 0; q < RPT; ++q) hc[q] = hn[q];
            }
            // ||x||^2 (fixed-order block reduction, identical in every thread)
            double xs = 0.0;
#pragma unroll
            for (int q = 0; q < RPT; ++q) xs += cabs2d(x[q]);
            xs = wave_allsum(xs);
            if (lane == 0) nrm_s[wid] = xs;
            __syncthreads();
            Xn = 0.0;
#pragma unroll
            for (int w = 0; w < NW; ++w) Xn += nrm_s[w];
            __syncthreads();
            sweeps = t;
            if (tol > 0.0 && sqrt(Ssum) <= tol * sqrt(Xn)) break;
        }
        // power scaling x_c <- rho_c x_c / ||x_c|| (rho_c <= 0: none; x_c = 0 stays 0)
        const double nrm = sqrt(Xn);
        const double sc = (rho_c > 0.0 && nrm > 0.0) ? rho_c / nrm : 1.0;
        int nf = 0;
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            const int i = tid + q * NT;
            if (i < m) {
                V v;
                v.x = (T)((double)x[q].x * sc);
                v.y = (T)((double)x[q].y * sc);
                if (!isfinite(v.x) || !isfinite(v.y)) nf = 1;
                X[jb.x_off + i] = v;
            }
        }
        if (nf) atomicOr(&flag_s, CDM_INFO_NONFINITE);
        __syncthreads();
        if (tid == 0) {
            const double rel = (Xn > 0.0) ? sqrt(Ssum / Xn) : (Ssum > 0.0 ? INFINITY : 0.0);
            int fl = flag_s;
            if (tol > 0.0 && !(rel <= tol)) fl |= CDM_INFO_NOT_CONVERGED;
            cdm_info o;
            o.sweeps = sweeps;
            o.flags = fl;
            o.rel_step = rel;
            o.resid = -1.0;
            o.reserved = 0.0;
            info[jb.info_idx] = o;
        }
}

template <typename T, int NT>
__global__ __launch_bounds__(NT) void k_zf_wg(const WgJob* __restrict__ jobs, int njobs,
                                              const cv<T>* __restrict__ H, const cv<T>* __restrict__ S,
                                              cv<T>* __restrict__ X, cdm_info* __restrict__ info, int T_max,
                                              double tol, double rho_c, uint32_t* __restrict__ queue,
                                              int64_t ld_arg) {
    constexpr int NW = NT / 64;
    extern __shared__ unsigned char smem_raw[];
    __shared__ T red_s[2][NW][3];
    __shared__ double nrm_s[NW];
    __shared__ int flag_s;
    __shared__ int job_s;
    const int tid = threadIdx.x;
    for (;;) {
        if (tid == 0) {
            job_s = queue ? (int)atomicAdd(queue, 1u) : (int)blockIdx.x;
            flag_s = 0;
        }
        __syncthreads();
        const int jslot = job_s;
        if (jslot >= njobs) return;
        const WgJob jb = jobs[jslot];
        switch (jb.rpt) {
            case 1: zf_instance<T, NT, 1>(jb, H, S, X, info, T_max, tol, rho_c, ld_arg, smem_raw, red_s, nrm_s, flag_s); break;
            case 2: zf_instance<T, NT, 2>(jb, H, S, X, info, T_max, tol, rho_c, ld_arg, smem_raw, red_s, nrm_s, flag_s); break;
            case 4: zf_instance<T, NT, 4>(jb, H, S, X, info, T_max, tol, rho_c, ld_arg, smem_raw, red_s, nrm_s, flag_s); break;
            default: zf_instance<T, NT, 8>(jb, H, S, X, info, T_max, tol, rho_c, ld_arg, smem_raw, red_s, nrm_s, flag_s); break;
        }
        if (!queue) return;   // one job per workgroup
        __syncthreads();
    }
}

template <typename T, int NT> static hipError_t launch_zf_t(const WgLaunch& L, hipStream_t st) {
    const size_t shm = (size_t)L.n_max * sizeof(T);
    hipLaunchKernelGGL((k_zf_wg<T, NT>), dim3(L.grid), dim3(NT), shm, st, L.jobs, L.njobs, (const cv<T>*)L.H,
                       (const cv<T>*)L.Y, (cv<T>*)L.X, L.info, L.T_max, L.tol, L.rho_c, L.queue, L.ld);
    return hipGetLastError();
}

// the panel form where every job has at most four rows per thread and x and M fit (see
// wg_lds_bytes); a 1024-thread workgroup has 128 VGPRs a thread, too few for its two panels
static bool wg_panels(int n_max, bool c128, int nt, int rmax) {
    return nt <= 512 && rmax <= 4 && (size_t)wg_panel_values(n_max) * (c128 ? 16 : 8) <= 128 * 1024;
}

template <typename T, int NT> static const void* wg_fn(bool panels) {
    if constexpr (NT <= 512)
        if (panels) return (const void*)k_cd_wgp<T, NT>;
    return (const void*)k_cd_wg<T, NT>;
}

template <typename T, int NT> static hipError_t launch_wg_t(const WgLaunch& L, hipStream_t st) {
    const bool pan = wg_panels(L.n_max, L.c128, NT, L.rmax);
    const size_t shm = wg_lds_bytes(L.n_max, L.c128, NT, L.rmax);
    const cv<T>*H = (const cv<T>*)L.H, *Y = (const cv<T>*)L.Y, *X0 = (const cv<T>*)L.X0;
    const WgFuse<T> f{L.fuse_count, (const cv<T>*)L.X, L.msum, L.fuse_lam, (cv<T>*)L.fuse_x, L.njobs, L.n_max};
    if constexpr (NT <= 512) {
        if (pan) {
            hipLaunchKernelGGL((k_cd_wgp<T, NT>), dim3(L.grid), dim3(NT), shm, st, L.jobs, L.njobs, H, Y, X0,
                               (cv<T>*)L.X, L.info, L.lambda, L.T_max, L.tol, L.order, L.queue, L.msum, L.ld, L.resid, f);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((k_cd_wg<T, NT>), dim3(L.grid), dim3(NT), shm, st, L.jobs, L.njobs, H, Y, X0, (cv<T>*)L.X,
                       L.info, L.lambda, L.T_max, L.tol, L.order, L.queue, L.msum, L.ld, L.resid, f);
    return hipGetLastError();
}

template <typename T, int NT> static hipError_t set_lds_t(bool panels, size_t bytes) {
    hipError_t e = hipFuncSetAttribute(wg_fn<T, NT>(panels), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute((const void*)k_zf_wg<T, NT>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}
template <typename T, int NT> static int occ_t(bool panels, size_t bytes) {
    int per = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, wg_fn<T, NT>(panels), NT, bytes) != hipSuccess) return 0;
    return per;
}

// complex128 runs on at most 512 threads (the planner's choice: its 8-rows-per-thread tile
// does not fit the register budget of a 1024-thread workgroup), so no such form is built
#define CDM_WG_DISPATCH(FN, c128, nt, ...)                                   \
    do {                                                                     \
        if (c128) {                                                          \
            if (nt == 128) return FN<double, 128>(__VA_ARGS__);              \
            if (nt == 256) return FN<double, 256>(__VA_ARGS__);              \
            if (nt == 512) return FN<double, 512>(__VA_ARGS__);              \
        } else {                                                             \
            if (nt == 128) return FN<float, 128>(__VA_ARGS__);               \
            if (nt == 256) return FN<float, 256>(__VA_ARGS__);               \
            if (nt == 512) return FN<float, 512>(__VA_ARGS__);               \
            if (nt == 1024) return FN<float, 1024>(__VA_ARGS__);             \
        }                                                                    \
    } while (0)

hipError_t launch_wg(const WgLaunch& L, hipStream_t st) {
    CDM_WG_DISPATCH(launch_wg_t, L.c128, L.nt, L, st);
    return hipErrorInvalidValue;
}
hipError_t launch_zf(const WgLaunch& L, hipStream_t st) {
    CDM_WG_DISPATCH(launch_zf_t, L.c128, L.nt, L, st);
    return hipErrorInvalidValue;
}
hipError_t wg_set_lds_limit(bool c128, int nt, int rmax, int n_max, size_t bytes) {
    CDM_WG_DISPATCH(set_lds_t, c128, nt, wg_panels(n_max, c128, nt, rmax), bytes);
    return hipErrorInvalidValue;
}
int wg_occupancy(bool c128, int nt, int rmax, int n_max, size_t bytes) {
    CDM_WG_DISPATCH(occ_t, c128, nt, wg_panels(n_max, c128, nt, rmax), bytes);
    return 0;
}
size_t wg_lds_bytes(int n_max, bool c128, int nt, int rmax) {
    const size_t e = c128 ? 16 : 8;
    return e * (wg_panels(n_max, c128, nt, rmax) ? (size_t)wg_panel_values(n_max) : (size_t)n_max * 2);
}

}  // namespace cdm
