// LLE weights (Section 4.2, Eq. LinSys), HR synthesis (Eq. HR_Rec) and the
// overlap blend (Section 4: quadratic prior on the overlaps, whose equal-
// weight minimiser is the per-pixel mean of the covering patches).
//
// Weights: Z = y - Y (the K neighbour rows), G = Z Z^T, A = G + lam tr(G) I,
// A w~ = 1 by Cholesky, w = w~ / sum(w~); uniform weights when tr(G) = 0.
// Up to 8 neighbours the packed Gram matrices come from the search or k_gram
// and a thread solves one patch's system; above that (and for every match of
// a patch) a wave forms and solves the system of one patch in registers.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "zh_internal.h"

namespace zh {

// One halving step of a reduce-scatter over the lanes of a half wave: lanes
// whose bit O is clear keep the first half of their N values, the others the
// second half, each adding its partner's partial sums; (base, cnt) track the
// index range the lane holds.
template <typename T, int N, int O, int NMAX>
__device__ __forceinline__ void rs_step(T (&v)[NMAX], int& base, int& cnt) {
    constexpr int NK = (N + 1) / 2;
    const bool hb = (threadIdx.x & O) != 0;
#pragma unroll
    for (int i = 0; i < NK; ++i) {
        const T lo_v = v[i];
        const T hi_v = (NK + i < N) ? v[NK + i] : (T)0;
        const T send = hb ? lo_v : hi_v;
        const T keep = hb ? hi_v : lo_v;
        v[i] = keep + __shfl_xor(send, O);
    }
    if (hb) {
        base += NK;
        cnt -= NK;
    } else {
        cnt = cnt < NK ? cnt : NK;
    }
}

// Packed Gram matrix (lower triangle, p = i(i+1)/2 + j, 36 entries) of the
// m <= 8 neighbours of each patch, Z_r = q - y_r, in T precision. Two patches
// per wave: half h of the wave owns one patch and lane l of the half holds
// coordinates [VEC l, VEC l + VEC); the 8 neighbour rows are loaded before
// use, partial products are reduce-scattered over the half in two groups of
// 18 entries.
template <typename T, int VEC>
__global__ __launch_bounds__(256) void k_gram(LleArgs a, T* __restrict__ gram) {
    typedef typename std::conditional<VEC == 4, uint2, uint32_t>::type raw_t;
    constexpr int PI[36] = {0, 1, 1, 2, 2, 2, 3, 3, 3, 3, 4, 4, 4, 4, 4, 5, 5, 5,
                            5, 5, 5, 6, 6, 6, 6, 6, 6, 6, 7, 7, 7, 7, 7, 7, 7, 7};
    constexpr int PJ[36] = {0, 0, 1, 0, 1, 2, 0, 1, 2, 3, 0, 1, 2, 3, 4, 0, 1, 2,
                            3, 4, 5, 0, 1, 2, 3, 4, 5, 6, 0, 1, 2, 3, 4, 5, 6, 7};
    const int lane = threadIdx.x & 63, hl = lane & 31, half = lane >> 5;
    const int wpb = blockDim.x >> 6;
    const int D = a.D;
    const bool dl = hl * VEC < D;
    for (int pr = xcd_block() * wpb + (threadIdx.x >> 6); 2 * pr < a.Q; pr += gridDim.x * wpb) {
        const int q = 2 * pr + half;
        const bool qv = q < a.Q;
        const int m = qv ? a.m[q] : 0;
        float qf[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) qf[e] = (qv && dl) ? a.qfeat[(int64_t)q * D + hl * VEC + e] : 0.0f;
        T z[8][VEC];
        if (VEC == 4 && a.xf) {
            // the fp32 copy: one 16-byte load of a contiguous 400-byte row
            float4 xr[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                xr[r] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (r < m && dl) {
                    const int64_t id = a.ids[(int64_t)q * a.K + r];
                    xr[r] = *reinterpret_cast<const float4*>(a.xf + id * D + hl * VEC);
                }
            }
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const float xv[4] = {xr[r].x, xr[r].y, xr[r].z, xr[r].w};
#pragma unroll
                for (int e = 0; e < VEC; ++e) z[r][e] = (r < m && dl) ? (T)qf[e] - (T)xv[e % 4] : (T)0;
            }
        } else {
            raw_t hr[8], lr[8];
    #pragma unroll
            for (int r = 0; r < 8; ++r) {
                hr[r] = raw_t{};
                lr[r] = raw_t{};
                if (r < m && dl) {
                    const uint32_t id = (uint32_t)a.ids[(int64_t)q * a.K + r];
                    const uint32_t bo = (id * (uint32_t)D + (uint32_t)(hl * VEC)) * 2u;
                    const uint32_t bh = (id * (uint32_t)a.hs + (uint32_t)(hl * VEC)) * 2u;
                    if constexpr (VEC == 4) {
                        hr[r] = *reinterpret_cast<const uint2*>(reinterpret_cast<const char*>(a.hi) + bh);
                        lr[r] = *reinterpret_cast<const uint2*>(reinterpret_cast<const char*>(a.lo) + bo);
                    } else {
                        hr[r] = *reinterpret_cast<const uint16_t*>(reinterpret_cast<const char*>(a.hi) + bh);
                        lr[r] = *reinterpret_cast<const uint16_t*>(reinterpret_cast<const char*>(a.lo) + bo);
                    }
                }
            }
    #pragma unroll
            for (int r = 0; r < 8; ++r) {
                uint32_t hv[VEC], lv[VEC];
                if constexpr (VEC == 4) {
                    hv[0] = hr[r].x & 0xFFFFu; hv[1] = hr[r].x >> 16; hv[2] = hr[r].y & 0xFFFFu; hv[3] = hr[r].y >> 16;
                    lv[0] = lr[r].x & 0xFFFFu; lv[1] = lr[r].x >> 16; lv[2] = lr[r].y & 0xFFFFu; lv[3] = lr[r].y >> 16;
                } else {
                    hv[0] = hr[r];
                    lv[0] = lr[r];
                }
    #pragma unroll
                for (int e = 0; e < VEC; ++e)
                    z[r][e] = (r < m && dl) ? (T)qf[e] - (T)__uint_as_float((hv[e] << 16) | lv[e]) : (T)0;
            }
        }
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            T v[18];
#pragma unroll
            for (int p = 0; p < 18; ++p) {
                T acc = (T)0;
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc += z[PI[18 * g + p]][e] * z[PJ[18 * g + p]][e];
                v[p] = acc;
            }
            int base = 0, cnt = 18;
            rs_step<T, 18, 16>(v, base, cnt);
            rs_step<T, 9, 8>(v, base, cnt);
            rs_step<T, 5, 4>(v, base, cnt);
            rs_step<T, 3, 2>(v, base, cnt);
            rs_step<T, 2, 1>(v, base, cnt);
            if (m > 0 && cnt >= 1) gram[(int64_t)q * 36 + 18 * g + base] = v[0];
        }
    }
}

hipError_t launch_gram(const LleArgs& a, void* gram, int gram_fp64, hipStream_t st) {
    if (a.Q == 0) return hipSuccess;
    if (a.K > 8 || a.D > 128) return hipErrorInvalidValue;
    const bool v4 = a.D % 4 == 0;
    if (!v4 && a.D > 32) return hipErrorInvalidValue;
    int grid = (a.Q + 7) / 8;
    if (grid > 65536) grid = 65536;
    grid = round_grid8(grid);
    if (gram_fp64) {
        if (v4) hipLaunchKernelGGL((k_gram<double, 4>), dim3(grid), dim3(256), 0, st, a, static_cast<double*>(gram));
        else hipLaunchKernelGGL((k_gram<double, 1>), dim3(grid), dim3(256), 0, st, a, static_cast<double*>(gram));
    } else {
        if (v4) hipLaunchKernelGGL((k_gram<float, 4>), dim3(grid), dim3(256), 0, st, a, static_cast<float*>(gram));
        else hipLaunchKernelGGL((k_gram<float, 1>), dim3(grid), dim3(256), 0, st, a, static_cast<float*>(gram));
    }
    return hipGetLastError();
}

// FP64 Gram of patch q's m neighbours straight from the rows (the slow path of
// the fp32 solve when its condition estimate exceeds 1e6).
__device__ void gram_fp64_rows(const LleArgs& a, int q, int m, double* Gd) {
    const int D = a.D;
    const float* qrow = a.qfeat + (int64_t)q * D;
    for (int i = 0; i < m; ++i)
        for (int j = 0; j <= i; ++j) {
            const int64_t ii = a.ids[(int64_t)q * a.K + i], ij = a.ids[(int64_t)q * a.K + j];
            const int64_t bi = ii * D, bj = ij * D, hi_i = ii * a.hs, hi_j = ij * a.hs;
            double g = 0.0;
            for (int t = 0; t < D; ++t) {
                const double zi = (double)qrow[t] - (double)join_planes(a.hi[hi_i + t], a.lo[bi + t]);
                const double zj = (double)qrow[t] - (double)join_planes(a.hi[hi_j + t], a.lo[bj + t]);
                g += zi * zj;
            }
            Gd[i * (i + 1) / 2 + j] = g;
        }
}

// Solve (G + lam tr(G) I) w~ = 1 on the first m rows (rows m..7 are set to
// the identity with a zero right-hand side), w = w~ / sum(w~). Returns the
// squared ratio of the largest to the smallest Cholesky diagonal, infinite where
// a diagonal is not the root of a positive number.
template <typename T>
__device__ __forceinline__ double solve8(T (&A)[36], int m, double lam, T (&w)[8]) {
    T tau = (T)0;
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if (i < m) tau += A[i * (i + 1) / 2 + i];
    if (tau == (T)0) {
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = i < m ? (T)1 / (T)m : (T)0;
        return 1.0;
    }
    const T reg = (T)lam * tau;
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) {
            T& x = A[i * (i + 1) / 2 + j];
            if (i >= m || j >= m) x = (i == j) ? (T)1 : (T)0;
            else if (i == j) x += reg;
        }
    T dmin = (T)0, dmax = (T)0;
    bool pos = true;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        T s = A[j * (j + 1) / 2 + j];
#pragma unroll
        for (int k = 0; k < j; ++k) s -= A[j * (j + 1) / 2 + k] * A[j * (j + 1) / 2 + k];
        const T d = sqrt(s);
        A[j * (j + 1) / 2 + j] = d;
        if (j < m) {
            pos = pos && s > (T)0;
            dmin = (j == 0 || d < dmin) ? d : dmin;
            dmax = d > dmax ? d : dmax;
        }
        const T inv = (T)1 / d;
#pragma unroll
        for (int i = j + 1; i < 8; ++i) {
            T t = A[i * (i + 1) / 2 + j];
#pragma unroll
            for (int k = 0; k < j; ++k) t -= A[i * (i + 1) / 2 + k] * A[j * (j + 1) / 2 + k];
            A[i * (i + 1) / 2 + j] = t * inv;
        }
    }
    T y[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        T s = i < m ? (T)1 : (T)0;
#pragma unroll
        for (int k = 0; k < i; ++k) s -= A[i * (i + 1) / 2 + k] * y[k];
        y[i] = s / A[i * (i + 1) / 2 + i];
    }
    T sum = (T)0;
#pragma unroll
    for (int i = 7; i >= 0; --i) {
        T s = y[i];
#pragma unroll
        for (int k = i + 1; k < 8; ++k) s -= A[k * (k + 1) / 2 + i] * w[k];
        w[i] = s / A[i * (i + 1) / 2 + i];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if (i < m) sum += w[i];
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = i < m ? w[i] / sum : (T)0;
    const double r = (double)dmax / (double)dmin;
    return pos ? r * r : (double)INFINITY;
}

template <typename T>
__global__ __launch_bounds__(256) void k_lle_solve(LleArgs a, const T* __restrict__ gram) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= a.Q) return;
    const int m = a.m[q];
    float* wout = a.w + (int64_t)q * a.K;
    if (m <= 0) {
        for (int r = 0; r < a.K; ++r) wout[r] = 0.0f;
        return;
    }
    T A[36];
#pragma unroll
    for (int p = 0; p < 36; ++p) A[p] = gram[(int64_t)q * 36 + p];
    T w[8];
    const double cond = solve8<T>(A, m, a.lam, w);
    if (sizeof(T) == 4 && cond > 1e6) {
        if (a.n_fp64) atomicAdd(a.n_fp64, 1u);
        double Ad[36], wd[8];
#pragma unroll
        for (int p = 0; p < 36; ++p) Ad[p] = 0.0;
        gram_fp64_rows(a, q, m, Ad);
        solve8<double>(Ad, m, a.lam, wd);
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = (T)wd[i];
    }
    for (int r = 0; r < a.K; ++r) wout[r] = r < m && r < 8 ? (float)w[r] : 0.0f;
}

hipError_t launch_lle_solve(const LleArgs& a, const void* gram, int gram_fp64, hipStream_t st) {
    if (a.Q == 0) return hipSuccess;
    if (a.K > 8) return hipErrorInvalidValue;
    const int grid = (a.Q + 255) / 256;
    if (gram_fp64)
        hipLaunchKernelGGL(k_lle_solve<double>, dim3(grid), dim3(256), 0, st, a, static_cast<const double*>(gram));
    else
        hipLaunchKernelGGL(k_lle_solve<float>, dim3(grid), dim3(256), 0, st, a, static_cast<const float*>(gram));
    return hipGetLastError();
}

// ---- systems of up to 80 rows, one wave per patch ------------------------------
// The M rows of a patch's system are cut into NB blocks of 16; the upper block
// triangle of A = G + lam tr(G) I sits in the wave's registers as tiles U_bj
// (b <= j) in the layout that the 16x16x4 matrix product leaves its result
// in: lane (g = l / 16, c = l % 16) holds column c of rows row_of(i, g),
// i < 4. In that layout a tile is directly the B operand of a product, its
// transpose directly the A operand (the same register for step i of both), so
// the whole block elimination
//   W_bj = U_bb^-1 U_bj,   U_ij -= U_bi^T W_bj   (b < i <= j)
// runs on the matrix cores without moving data between lanes. The diagonal
// blocks are inverted in place by the symmetric sweep operator, one pivot at
// a time (the pivot's column reaches the lanes of a row of 16 by a DPP
// broadcast, its row the four rows by one shuffle). lam > 0 bounds the
// condition number of A by 1 + 1 / lam, so no pivoting is needed where the
// precision holds lam tr(G); a pivot that rounding leaves at zero or below is told
// to the caller.
//
// Bound: the Gram tiles' FP64 products (64 cycles each; 28 per tile at D = 100)
// and, per block, the chain of 16 sweeps. Measured against one wave that
// summed G entry by entry from LDS and factorised it column by column there
// (50 KB of LDS: three waves per compute unit): 24,236 patches of up to 72
// matches (33 on average) 6.21 -> 0.43 ms; 62,721 patches at K = 12
// 0.81 -> 0.11 ms (both FP64, D = 100).
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

template <typename T> struct Tile;
template <> struct Tile<float> {
    typedef f32x4 vec;
    static __device__ __forceinline__ vec mma(float a, float b, vec c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    // row of register i in lane group g
    static __device__ __host__ constexpr int row_of(int i, int g) { return 4 * g + i; }
    static constexpr int reg_of(int r) { return r & 3; }
    static constexpr int grp_of(int r) { return r >> 2; }
};
template <> struct Tile<double> {
    typedef f64x4 vec;
    static __device__ __forceinline__ vec mma(double a, double b, vec c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __host__ constexpr int row_of(int i, int g) { return 4 * i + g; }
    static constexpr int reg_of(int r) { return r >> 2; }
    static constexpr int grp_of(int r) { return r & 3; }
};

template <int CTRL> __device__ __forceinline__ float dpp_mov(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL> __device__ __forceinline__ double dpp_mov(double v) {
    const int64_t b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xFFFFFFFF), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double(((int64_t)hi << 32) | (int64_t)(uint32_t)lo);
}
constexpr int kDppRowBcast = 0x150;   // row_newbcast:n, lane n of each row of 16 to the row
constexpr int kDppRowRor = 0x120;     // row_ror:n

__device__ __forceinline__ float lane_value(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double lane_value(double v, int l) {
    const int64_t b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xFFFFFFFF), l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((int64_t)hi << 32) | (int64_t)(uint32_t)lo);
}
__device__ __forceinline__ float fma_t(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return fma(a, b, c); }

// One sweep of the symmetric 16x16 tile d on pivot P (skipped past the n used
// rows, whose diagonal is -1 already); pmin, pmax: the pivots' range (a pivot that
// is not a number makes every later one so, and pmin the last of them).
template <typename T, int Pv>
__device__ __forceinline__ void sweep_pivot(typename Tile<T>::vec& d, int n, T& pmin, T& pmax) {
    if (Pv >= n) return;
    const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
    constexpr int ip = Tile<T>::reg_of(Pv), gp = Tile<T>::grp_of(Pv);
    const T piv = lane_value(d[ip], 16 * gp + Pv);
    pmin = piv >= pmin ? pmin : piv;
    pmax = piv > pmax ? piv : pmax;
    const T inv = (T)1 / piv;
    const T row = __shfl(d[ip], 16 * gp + c) * inv;   // a_pc / a_pp
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const T col = dpp_mov<kDppRowBcast + Pv>(d[i]);   // a_rp
        const bool rp = Tile<T>::row_of(i, g) == Pv, cp = c == Pv;
        const T upd = fma_t(-col, row, d[i]);
        d[i] = rp ? (cp ? -inv : row) : (cp ? col * inv : upd);
    }
}
template <typename T, int... Pv>
__device__ __forceinline__ void sweep_tile(typename Tile<T>::vec& d, int n, T& pmin, T& pmax,
                                           std::integer_sequence<int, Pv...>) {
    (sweep_pivot<T, Pv>(d, n, pmin, pmax), ...);
}

// Vectors of 16 entries come in two layouts: by column (lane holds entry c)
// and by row (register i holds entry row_of(i, g)).
template <typename T> __device__ __forceinline__ typename Tile<T>::vec to_rows(T v) {
    const int g = (threadIdx.x & 63) >> 4;
    typename Tile<T>::vec r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = __shfl(v, Tile<T>::row_of(i, g));
    return r;
}
// by column: (X^T r)_c
template <typename T>
__device__ __forceinline__ T mul_t(const typename Tile<T>::vec& X, const typename Tile<T>::vec& r) {
    T s = X[0] * r[0];
#pragma unroll
    for (int i = 1; i < 4; ++i) s = fma_t(X[i], r[i], s);
    s += __shfl_xor(s, 16);
    return s + __shfl_xor(s, 32);
}
template <typename T> __device__ __forceinline__ T row_sum16(T v) {
    v += dpp_mov<kDppRowRor + 8>(v);
    v += dpp_mov<kDppRowRor + 4>(v);
    v += dpp_mov<kDppRowRor + 2>(v);
    return v + dpp_mov<kDppRowRor + 1>(v);
}

// Weights of one patch's M <= 16 NB rows xf[id[0..M)] against the query qf, by
// column into x[b] (entry 16 b + c). Returns the squared ratio of the largest
// to the smallest Cholesky diagonal (the pivots' ratio), infinite unless every
// pivot is positive.
template <typename T, int NB, bool V4>
__device__ __forceinline__ double lle_wave(int D, int M, double lam, const float* __restrict__ qf,
                                           const float* __restrict__ xf, const int32_t* __restrict__ id, T (&x)[NB]) {
    typedef typename Tile<T>::vec vec;
    const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
    const int nb = (M + 15) >> 4;
    const float* row[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) row[b] = 16 * b + c < M ? xf + (int64_t)id[16 * b + c] * D : nullptr;
    // Gram tiles: 16 coordinates a step, lane group g on 16 t + 4 g .. + 3
    vec U[NB * (NB + 1) / 2];
    auto at = [](int b, int j) constexpr { return j * (j + 1) / 2 + b; };   // b <= j
#pragma unroll
    for (int p = 0; p < NB * (NB + 1) / 2; ++p) U[p] = vec{0, 0, 0, 0};
    for (int c0 = 4 * g, t = 0; t < D; t += 16, c0 += 16) {
        float qv[4] = {0.f, 0.f, 0.f, 0.f}, xv[NB][4];
        if (V4) {
            const float4 v = c0 < D ? *reinterpret_cast<const float4*>(qf + c0) : make_float4(0.f, 0.f, 0.f, 0.f);
            qv[0] = v.x, qv[1] = v.y, qv[2] = v.z, qv[3] = v.w;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) qv[e] = c0 + e < D ? qf[c0 + e] : 0.0f;
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            // rows past M equal the query: zero differences
#pragma unroll
            for (int e = 0; e < 4; ++e) xv[b][e] = qv[e];
            if (row[b]) {
                if (V4) {
                    if (c0 < D) {
                        const float4 v = *reinterpret_cast<const float4*>(row[b] + c0);
                        xv[b][0] = v.x, xv[b][1] = v.y, xv[b][2] = v.z, xv[b][3] = v.w;
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (c0 + e < D) xv[b][e] = row[b][c0 + e];
                }
            }
        }
        T z[NB][4];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) z[b][e] = (T)qv[e] - (T)xv[b][e];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            if (j >= nb) break;
#pragma unroll
            for (int b = 0; b <= j; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e) U[at(b, j)] = Tile<T>::mma(z[b][e], z[j][e], U[at(b, j)]);
        }
    }
    // tau = tr G; the diagonal's entries sit where row_of(i, g) = c
    T tau = (T)0;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (Tile<T>::row_of(i, g) == c) tau += U[at(b, b)][i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) tau += __shfl_xor(tau, o);
    if (tau == (T)0) {
#pragma unroll
        for (int b = 0; b < NB; ++b) x[b] = 16 * b + c < M ? (T)1 / (T)M : (T)0;
        return 1.0;
    }
    const T reg = (T)lam * tau;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (Tile<T>::row_of(i, g) == c) U[at(b, b)][i] = 16 * b + c < M ? U[at(b, b)][i] + reg : (T)-1;
    // elimination; U_bb becomes -U_bb^-1, x the forward-substituted right-hand side
    T pmin = (T)INFINITY, pmax = (T)0;
#pragma unroll
    for (int b = 0; b < NB; ++b) x[b] = 16 * b + c < M ? (T)1 : (T)0;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (b >= nb) break;
        vec& S = U[at(b, b)];
        sweep_tile<T>(S, M - 16 * b, pmin, pmax, std::make_integer_sequence<int, 16>{});
        x[b] = -mul_t<T>(S, to_rows(x[b]));
        const vec y = to_rows(x[b]);
#pragma unroll
        for (int j = b + 1; j < NB; ++j) {
            if (j >= nb) break;
            x[j] -= mul_t<T>(U[at(b, j)], y);
            vec W = {0, 0, 0, 0};   // -U_bb^-1 U_bj
#pragma unroll
            for (int i = 0; i < 4; ++i) W = Tile<T>::mma(S[i], U[at(b, j)][i], W);
#pragma unroll
            for (int k = b + 1; k <= j; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i) U[at(k, j)] = Tile<T>::mma(U[at(b, k)][i], W[i], U[at(k, j)]);
        }
    }
    // back substitution: x_b = y_b - U_bb^-1 sum_j U_bj x_j
#pragma unroll
    for (int b = NB - 2; b >= 0; --b) {
        if (b + 1 >= nb) continue;
        vec s = {0, 0, 0, 0};
#pragma unroll
        for (int j = b + 1; j < NB; ++j) {
            if (j >= nb) break;
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] = fma_t(U[at(b, j)][i], x[j], s[i]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) s[i] = row_sum16(s[i]);
        x[b] += mul_t<T>(U[at(b, b)], s);
    }
    T sum = (T)0;
#pragma unroll
    for (int b = 0; b < NB; ++b) sum += 16 * b + c < M ? x[b] : (T)0;
    sum = row_sum16(sum);
#pragma unroll
    for (int b = 0; b < NB; ++b) x[b] = 16 * b + c < M ? x[b] / sum : (T)0;
    return pmin > (T)0 ? (double)pmax / (double)pmin : (double)INFINITY;
}

// K <= 16 neighbours, four patches a workgroup. The fp32 form solves again in
// FP64 when the Cholesky diagonals' squared ratio exceeds 1e6.
template <typename T, bool V4>
__global__ __launch_bounds__(256) void k_lle16(LleArgs a) {
    const int q = (int)block_id() * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (q >= a.Q) return;
    const int M = min(a.m[q], a.K);
    float* wout = a.w + (int64_t)q * a.K;
    if (M <= 0) {
        if (lane < a.K) wout[lane] = 0.0f;
        return;
    }
    const float* qf = a.qfeat + (int64_t)q * a.D;
    const int32_t* id = a.ids + (int64_t)q * a.K;
    T x[1];
    const double cond = lle_wave<T, 1, V4>(a.D, M, a.lam, qf, a.xf, id, x);
    float w = (float)x[0];
    if (sizeof(T) == 4 && cond > 1e6) {
        if (a.n_fp64 && lane == 0) atomicAdd(a.n_fp64, 1u);
        double xd[1];
        lle_wave<double, 1, V4>(a.D, M, a.lam, qf, a.xf, id, xd);
        w = (float)xd[0];
    }
    if (lane < a.K) wout[lane] = w;
}

hipError_t launch_lle(const LleArgs& a, hipStream_t st) {
    if (a.Q == 0) return hipSuccess;
    if (a.D < 1 || a.D > 128 || a.K < 1 || a.K > kMaxK || !a.xf) return hipErrorInvalidValue;
    const dim3 grid = grid_rows((a.Q + 3) / 4);
    const bool v4 = a.D % 4 == 0 && ((reinterpret_cast<uintptr_t>(a.xf) | reinterpret_cast<uintptr_t>(a.qfeat)) & 15) == 0;
    if (a.fp64) {
        if (v4) hipLaunchKernelGGL((k_lle16<double, true>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((k_lle16<double, false>), grid, dim3(256), 0, st, a);
    } else {
        if (v4) hipLaunchKernelGGL((k_lle16<float, true>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((k_lle16<float, false>), grid, dim3(256), 0, st, a);
    }
    return hipGetLastError();
}

// LLE over all M matches of each patch (Section 4.2: Eq. LinSys with m
// running over every match found, M <= kAllMax), FP64 from exact differences:
// w = w~ / sum w~, uniform when tr G = 0 (every candidate equals the query).
// Weights past M are 0 and list entries past M are set to -1.
template <int NB, bool V4>
__global__ __launch_bounds__(64) void k_lle_all(int Q, int D, int cap, double lam, const float* __restrict__ qfeat,
                                                const float* __restrict__ xf, int32_t* __restrict__ cand,
                                                const int32_t* __restrict__ ncand, float* __restrict__ w) {
    const int lane = threadIdx.x;
    const int q = xcd_block();
    if (q >= Q) return;
    const int M = min(ncand[q], cap);
    int32_t* cq = cand + (int64_t)q * cap;
    float* wq = w + (int64_t)q * cap;
    for (int i = M + lane; i < cap; i += 64) {
        cq[i] = -1;
        wq[i] = 0.0f;
    }
    if (M <= 0) return;
    double x[NB];
    lle_wave<double, NB, V4>(D, M, lam, qfeat + (int64_t)q * D, xf, cq, x);
    if (lane < 16) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
            if (16 * b + lane < M) wq[16 * b + lane] = (float)x[b];
    }
}

template <int NB>
static void launch_lle_all_nb(int Q, int D, int cap, double lam, const float* qfeat, const float* xf, int32_t* cand,
                              const int32_t* ncand, float* w, bool v4, hipStream_t st) {
    const dim3 grid(round_grid8(Q));
    if (v4) hipLaunchKernelGGL((k_lle_all<NB, true>), grid, dim3(64), 0, st, Q, D, cap, lam, qfeat, xf, cand, ncand, w);
    else hipLaunchKernelGGL((k_lle_all<NB, false>), grid, dim3(64), 0, st, Q, D, cap, lam, qfeat, xf, cand, ncand, w);
}

hipError_t launch_lle_all(int Q, int D, int cap, double lam, const float* qfeat, const float* xf, int32_t* cand,
                          const int32_t* ncand, float* w, hipStream_t st) {
    if (Q == 0) return hipSuccess;
    if (cap < 1 || cap > kAllMax || D < 1 || D > 128) return hipErrorInvalidValue;
    if (!one_row(round_grid8(Q), 64)) return hipErrorInvalidConfiguration;
    static_assert(kAllMax <= 80, "five blocks of 16 rows");
    const bool v4 = D % 4 == 0 && ((reinterpret_cast<uintptr_t>(xf) | reinterpret_cast<uintptr_t>(qfeat)) & 15) == 0;
    switch ((cap + 15) / 16) {
        case 1: launch_lle_all_nb<1>(Q, D, cap, lam, qfeat, xf, cand, ncand, w, v4, st); break;
        case 2: launch_lle_all_nb<2>(Q, D, cap, lam, qfeat, xf, cand, ncand, w, v4, st); break;
        case 3: launch_lle_all_nb<3>(Q, D, cap, lam, qfeat, xf, cand, ncand, w, v4, st); break;
        case 4: launch_lle_all_nb<4>(Q, D, cap, lam, qfeat, xf, cand, ncand, w, v4, st); break;
        default: launch_lle_all_nb<5>(Q, D, cap, lam, qfeat, xf, cand, ncand, w, v4, st); break;
    }
    return hipGetLastError();
}

// ---- synthesis fused with the blend -------------------------------------------
// The synthesised patches are never written out. The patch origins are cut
// into tiles of TI patch rows x sb_cols(s) patch columns; a workgroup takes a
// tile, forms x_q = mu_q + sum_m w_m r_{n_m} of one patch row at a time in
// LDS (the K residual rows read once, in chunks of eight neighbours; each
// value is a fused multiply-add over the neighbours in order from zero, then
// mu_q is added) and adds each
// pixel's values of the row's patches, in ascending column order, to the
// tile's region: the (TI + 4) s x (TJ + 4) s HR pixels its patches cover,
// together with the count of covering patches of every LR cell. Regions go
// to a partial buffer; k_sb_combine then gives each HR pixel the sum of the
// regions that hold it, in tile order, divided by the summed
// count, or the bicubic of the LR image where no patch covers it. The sum
// of a pixel is therefore taken patch row by patch row in row-major order
// inside a tile and tile by tile across tiles.
//
//
// Bound: the gather of the residual rows. The neighbours of the next row are
// staged while the current row is added (two barriers a row; three, and the
// lists in chunks of eight, before: 1020x1020 patches x2 556 -> 540 us, 3.4 GB
// of rows at 6.3 TB/s; 247x259 x2 60 -> 39; 207x303 x4 at K = 12 157 -> 106).
//
// An image of few tiles leaves most of the chip idle for the chain of a tile's
// rows, so its tiles' regions are cut into their rows of LR cells, a workgroup
// each (k_sb_row): the same sums in the same order into the same regions.
constexpr int kSbThreads = 512;   // 256 take 5-15% longer
template <int s, int TI>
struct SbGeom {
    static constexpr int ps = kPatch * s, ps2 = ps * ps;
    static constexpr int VEC = (ps2 & 3) == 0 ? 4 : 1;    // floats per load
    static constexpr int NCH = ps2 / VEC;                  // loads per residual row
    static constexpr int TJ = sb_cols(s);
    static constexpr int CY = TI + kPatch - 1, CX = TJ + kPatch - 1;   // LR cells of a region
    static constexpr int RY = CY * s, RX = CX * s;                       // HR pixels of a region
    static constexpr int64_t PART = (int64_t)RY * RX + CY * CX;         // floats + counts per tile
    static size_t lds(int K) { return sizeof(float) * (size_t)(TJ * ps2 + PART + 2 * TJ * K + 2 * TJ); }
};

// Chunk c (VEC floats) of the synthesised patch sum_m w_m r_{n_m}, mq rows of
// the lists id and wt, as fused multiply-adds in order from zero. L4: the lists
// start on 16 bytes and hold a multiple of four entries.
template <int ps2, int VEC, bool L4 = false>
__device__ __forceinline__ void synth_chunk(const float* __restrict__ resid, const int* id, const float* wt, int mq,
                                            int c, float (&acc)[VEC]) {
    const char* base = reinterpret_cast<const char*>(resid) + c * (VEC * 4);
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] = 0.0f;
    for (int r0 = 0; r0 < mq; r0 += 8) {
        float v[8][VEC], wr[8];
        [[maybe_unused]] int ir[8];
        if constexpr (L4) {
#pragma unroll
            for (int h = 0; h < 8; h += 4) {
                const bool ok = r0 + h < mq;
                const int4 i4 = ok ? *reinterpret_cast<const int4*>(id + r0 + h) : make_int4(0, 0, 0, 0);
                const float4 w4 = ok ? *reinterpret_cast<const float4*>(wt + r0 + h) : make_float4(0.f, 0.f, 0.f, 0.f);
                ir[h] = i4.x, ir[h + 1] = i4.y, ir[h + 2] = i4.z, ir[h + 3] = i4.w;
                wr[h] = w4.x, wr[h + 1] = w4.y, wr[h + 2] = w4.z, wr[h + 3] = w4.w;
            }
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const bool ok = r0 + r < mq;
            wr[r] = ok ? (L4 ? wr[r] : wt[r0 + r]) : 0.0f;
            const float* x = reinterpret_cast<const float*>(
                base + (uint64_t)(uint32_t)(ok ? (L4 ? ir[r] : id[r0 + r]) : 0) * (uint32_t)(4 * ps2));
            if constexpr (VEC == 4) {
                const float4 t = ok ? *reinterpret_cast<const float4*>(x) : make_float4(0.f, 0.f, 0.f, 0.f);
                v[r][0] = t.x;
                v[r][1] = t.y;
                v[r][2] = t.z;
                v[r][3] = t.w;
            } else {
                v[r][0] = ok ? *x : 0.0f;
            }
        }
#pragma unroll
        for (int r = 0; r < 8; ++r)
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc[e] = fmaf(wr[r], v[r][e], acc[e]);
    }
}

template <int s, int TI>
__device__ __forceinline__ void sb_tile(const int32_t* __restrict__ ids, const int32_t* __restrict__ m,
                                        const float* __restrict__ wt, const double* __restrict__ mu,
                                        const float* __restrict__ resid, int K, int h, int w, int64_t tile,
                                        float* __restrict__ part, float* smem) {
    using G = SbGeom<s, TI>;
    constexpr int ps = G::ps, ps2 = G::ps2, VEC = G::VEC, NCH = G::NCH, TJ = G::TJ;
    constexpr int CX = G::CX, RX = G::RX, CY = G::CY, RY = G::RY, NT = kSbThreads;
    float* sx = smem;                                     // [TJ][ps2] the synthesised patches of one patch row
    float* sacc = sx + TJ * ps2;                          // [RY][RX]
    int* scnt = reinterpret_cast<int*>(sacc + RY * RX);   // [CY][CX]
    int* sid = scnt + CY * CX;                            // [TJ][K] neighbours and weights of one patch row
    float* swt = reinterpret_cast<float*>(sid + TJ * K);
    int* smq = reinterpret_cast<int*>(swt + TJ * K);      // [TJ] neighbours used, patch means
    float* smu = reinterpret_cast<float*>(smq + TJ);
    const int tid = threadIdx.x;
    const int npi = h - kPatch + 1, npj = w - kPatch + 1;
    const int ntj = (npj + TJ - 1) / TJ;
    // the grid is rounded up to a multiple of 8: workgroups past the last
    // tile have no region
    if (npi <= 0 || npj <= 0 || tile >= (int64_t)((npi + TI - 1) / TI) * ntj) return;
    const int ti = (int)(tile / ntj), tj = (int)(tile - (int64_t)ti * ntj);
    const int i0 = ti * TI, j0 = tj * TJ;
    const int nc = min(TJ, npj - j0);
    auto stage = [&](int ii) {
        const int64_t q0 = (int64_t)(i0 + ii) * npj + j0;
        const int32_t* ip = ids + q0 * K;
        const float* wp = wt + q0 * K;
        for (int e = tid; e < nc * K; e += NT) {
            sid[e] = ip[e];
            swt[e] = wp[e];
        }
        for (int jj = NT - 1 - tid; jj < TJ; jj += NT) {
            const int mq = jj < nc ? min(m[q0 + jj], K) : 0;
            smq[jj] = mq;
            smu[jj] = mq > 0 ? (float)mu[q0 + jj] : 0.0f;
        }
    };
    stage(0);
    for (int e = tid; e < RY * RX; e += NT) sacc[e] = 0.0f;
    for (int e = tid; e < CY * CX; e += NT) scnt[e] = 0;
    __syncthreads();
    for (int ii = 0; ii < TI && i0 + ii < npi; ++ii) {
        // ---- the patches of this row
        for (int it = tid; it < TJ * NCH; it += NT) {
            const int jj = it / NCH, c = it - jj * NCH;
            const int mq = smq[jj];
            float acc[VEC];
            synth_chunk<ps2, VEC>(resid, sid + jj * K, swt + jj * K, mq, c, acc);
            float* dst = sx + jj * ps2 + c * VEC;
            const float mf = smu[jj];
            if constexpr (VEC == 4)
                *reinterpret_cast<float4*>(dst) = make_float4(mf + acc[0], mf + acc[1], mf + acc[2], mf + acc[3]);
            else
                dst[0] = mf + acc[0];
        }
        __syncthreads();
        // ---- their values added to the region rows s ii .. s ii + 5 s
        uint64_t has = 0;   // patches of the row that have neighbours
        {
            const int jj = tid & 63;
            has = __ballot(jj < TJ && smq[jj < TJ ? jj : 0] > 0);
        }
        for (int it = tid; it < ps * RX; it += NT) {
            const int u = it / RX, X = it - u * RX;
            const int cl = X / s;
            const int jlo = cl - (kPatch - 1) > 0 ? cl - (kPatch - 1) : 0, jhi = cl < TJ - 1 ? cl : TJ - 1;
            float* a = sacc + (s * ii + u) * RX + X;
            float acc = *a;
            for (int jj = jlo; jj <= jhi; ++jj)
                if ((has >> jj) & 1u) acc += sx[jj * ps2 + u * ps + X - s * jj];
            *a = acc;
        }
        for (int it = tid; it < kPatch * CX; it += NT) {
            const int cu = it / CX, cl = it - cu * CX;
            const int jlo = cl - (kPatch - 1) > 0 ? cl - (kPatch - 1) : 0, jhi = cl < TJ - 1 ? cl : TJ - 1;
            const uint64_t cols = (2ull << jhi) - (1ull << jlo);
            scnt[(ii + cu) * CX + cl] += __popcll(has & cols);
        }
        if (ii + 1 < TI && i0 + ii + 1 < npi) {
            __syncthreads();   // the flags are no longer read
            stage(ii + 1);
        }
        __syncthreads();
    }
    float* pa = part + tile * G::PART;
    int* pc = reinterpret_cast<int*>(pa + RY * RX);
    for (int e = tid; e < RY * RX; e += NT) pa[e] = sacc[e];
    for (int e = tid; e < CY * CX; e += NT) pc[e] = scnt[e];
}

template <int s, int TI>
__device__ __forceinline__ float sb_pixel(const float* __restrict__ part, const float* __restrict__ lr, int h, int w,
                                          int Y, int X) {
    using G = SbGeom<s, TI>;
    constexpr int TJ = G::TJ, CX = G::CX, RX = G::RX, RY = G::RY;
    const int npi = h - kPatch + 1, npj = w - kPatch + 1;
    float acc = 0.0f;
    int cnt = 0;
    if (npi > 0 && npj > 0) {
        const int ntj = (npj + TJ - 1) / TJ, nti = (npi + TI - 1) / TI;
        const int cy = Y / s, cx = X / s;
        // tiles holding a patch origin in [cy - 4, cy] x [cx - 4, cx]
        const int tilo = cy >= kPatch - 1 ? (cy - (kPatch - 1)) / TI : 0, tihi = min(nti - 1, cy / TI);
        const int tjlo = cx >= kPatch - 1 ? (cx - (kPatch - 1)) / TJ : 0, tjhi = min(ntj - 1, cx / TJ);
        for (int ti = tilo; ti <= tihi; ++ti)
            for (int tj = tjlo; tj <= tjhi; ++tj) {
                const float* pa = part + ((int64_t)ti * ntj + tj) * G::PART;
                const int ly = Y - s * TI * ti, lx = X - s * TJ * tj;
                acc += pa[ly * RX + lx];
                cnt += reinterpret_cast<const int*>(pa + RY * RX)[(cy - TI * ti) * CX + (cx - TJ * tj)];
            }
    }
    return cnt > 0 ? acc / (float)cnt : bicubic_at(lr, h, w, s, Y, X);
}

template <int s, int TI>
__global__ __launch_bounds__(kSbThreads) void k_sb_tile(int K, int h, int w, const int32_t* __restrict__ ids,
                                                        const int32_t* __restrict__ m, const float* __restrict__ wt,
                                                        const double* __restrict__ mu,
                                                        const float* __restrict__ resid, float* __restrict__ part) {
    extern __shared__ __align__(16) float smem[];
    sb_tile<s, TI>(ids, m, wt, mu, resid, K, h, w, xcd_block(), part, smem);
}

template <int s, int TI>
__global__ __launch_bounds__(256) void k_sb_combine(const float* __restrict__ part, const float* __restrict__ lr,
                                                    int h, int w, float* __restrict__ hr) {
    const int W = s * w;
    const int64_t total = (int64_t)s * h * W;
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < total; p += (int64_t)gridDim.x * blockDim.x) {
        const int Y = (int)(p / W), X = (int)(p - (int64_t)Y * W);
        hr[p] = sb_pixel<s, TI>(part, lr, h, w, Y, X);
    }
}

// how a workgroup reads the lists of neighbours and weights: entry by entry, in
// 16-byte loads (lists of a multiple of four entries), or staged in LDS
enum SbLists { kSbEntries, kSbWide, kSbStaged };

// Images of few tiles: a workgroup takes one row of LR cells of a tile's region
// (s HR rows) and the up to five patch rows that cover it. A patch gives each row
// of cells s of its own rows and no HR pixel twice, so nothing is formed twice;
// all the patches' values are formed at once (one chain of loads), then added per
// pixel in the tile's order (patch rows, then columns, ascending from zero).
// Bound: that chain on small images; above, lines of the pieces of residual rows and
// of the lists in the vector cache (lists of 72 at 150 tiles x2 entry by entry 145
// us, in 16-byte loads 88). 512 threads: with 256 the smallest images take 2-8 us more,
// with 1024 those of 150 tiles 6 us; two rows of cells a workgroup 2-24 us more.
template <int s, int TI, SbLists LM>
__global__ __launch_bounds__(kSbThreads) void k_sb_row(int K, int h, int w, const int32_t* __restrict__ ids,
                                                       const int32_t* __restrict__ m, const float* __restrict__ wt,
                                                       const double* __restrict__ mu,
                                                       const float* __restrict__ resid, float* __restrict__ part) {
    using G = SbGeom<s, TI>;
    constexpr int ps = G::ps, ps2 = G::ps2, VEC = G::VEC, TJ = G::TJ, CY = G::CY, CX = G::CX, RX = G::RX, RY = G::RY;
    constexpr int SEG = s * ps, NC = SEG / VEC, NT = kSbThreads;   // a patch's values in a row of cells, its loads of them
    static_assert(SEG % VEC == 0 && TJ <= 64, "whole loads; a lane for each column");
    __shared__ __align__(16) float sx[kPatch * TJ * SEG];
    __shared__ int smq[kPatch][64];
    const int npi = h - kPatch + 1, npj = w - kPatch + 1;
    const int ntj = (npj + TJ - 1) / TJ;
    const int64_t b = xcd_block(), tile = b / CY;
    const int cy = (int)(b - tile * CY);
    if (tile >= (int64_t)((npi + TI - 1) / TI) * ntj) return;
    const int i0 = (int)(tile / ntj) * TI, j0 = (int)(tile % ntj) * TJ;
    const int nr = min(TI, npi - i0), nc = min(TJ, npj - j0);
    const int ilo = max(0, cy - (kPatch - 1)), n = min(nr - 1, cy) - ilo + 1;
    if (n <= 0) return;   // past the image
    const int tid = threadIdx.x;
    extern __shared__ int slist[];   // kSbStaged: IDs [5][TJ][K], then weights
    float* swt = reinterpret_cast<float*>(slist + kPatch * TJ * K);
    if (LM == kSbStaged) {
        for (int e = tid; e < n * TJ * K; e += NT) {
            const int r = e / (TJ * K), o = e - r * (TJ * K);
            const int64_t p = ((int64_t)(i0 + ilo + r) * npj + j0) * K + o;
            if (o < nc * K) slist[e] = ids[p], swt[e] = wt[p];
        }
        __syncthreads();
    }
    for (int it = tid; it < n * TJ * NC; it += NT) {
        const int r = it / (TJ * NC), jc = it - r * (TJ * NC), jj = jc / NC, c = jc - jj * NC;
        const int64_t q = (int64_t)(i0 + ilo + r) * npj + j0 + jj;
        const int mq = jj < nc ? min(m[q], K) : 0;
        float acc[VEC];
        const int chunk = (cy - ilo - r) * NC + c;
        if (LM == kSbStaged)
            synth_chunk<ps2, VEC>(resid, slist + (r * TJ + jj) * K, swt + (r * TJ + jj) * K, mq, chunk, acc);
        else
            synth_chunk<ps2, VEC, LM == kSbWide>(resid, ids + q * K, wt + q * K, mq, chunk, acc);
        const float mf = mq > 0 ? (float)mu[q] : 0.0f;
        float* dst = sx + (r * TJ + jj) * SEG + c * VEC;
        if constexpr (VEC == 4)
            *reinterpret_cast<float4*>(dst) = make_float4(mf + acc[0], mf + acc[1], mf + acc[2], mf + acc[3]);
        else
            dst[0] = mf + acc[0];
        if (c == 0) smq[r][jj] = mq;
    }
    __syncthreads();
    uint64_t has[kPatch];   // patches of each row that have neighbours
#pragma unroll
    for (int r = 0; r < kPatch; ++r) {
        const int jj = tid & 63;
        has[r] = __ballot(r < n && jj < TJ && smq[r][jj] > 0);
    }
    float* pa = part + tile * G::PART;
    int* pc = reinterpret_cast<int*>(pa + RY * RX);
    for (int it = tid; it < s * RX; it += NT) {
        const int u = it / RX, X = it - u * RX, cl = X / s;
        const int jlo = cl - (kPatch - 1) > 0 ? cl - (kPatch - 1) : 0, jhi = cl < TJ - 1 ? cl : TJ - 1;
        float acc = 0.0f;
#pragma unroll
        for (int r = 0; r < kPatch; ++r)
            for (int jj = jlo; jj <= jhi; ++jj)
                if ((has[r] >> jj) & 1u) acc += sx[(r * TJ + jj) * SEG + u * ps + X - s * jj];
        pa[(s * cy + u) * RX + X] = acc;
    }
    for (int cl = tid; cl < CX; cl += NT) {
        const int jlo = cl - (kPatch - 1) > 0 ? cl - (kPatch - 1) : 0, jhi = cl < TJ - 1 ? cl : TJ - 1;
        const uint64_t cols = (2ull << jhi) - (1ull << jlo);
        int cnt = 0;
#pragma unroll
        for (int r = 0; r < kPatch; ++r) cnt += __popcll(has[r] & cols);
        pc[cy * CX + cl] = cnt;
    }
}

// Batched: the tiles and HR pixels of every image of the batch, the image
// found from its first tile (sbt_off) or HR pixel (hr_off); partial regions
// at the image's first tile.
template <int s, int TI>
__global__ __launch_bounds__(kSbThreads) void k_b_sb_tile(const BatchImage* __restrict__ im, int n, int64_t tiles,
                                                          int K, const int32_t* __restrict__ ids,
                                                          const int32_t* __restrict__ m, const float* __restrict__ wt,
                                                          const double* __restrict__ mu,
                                                          const float* __restrict__ resid, float* __restrict__ part) {
    extern __shared__ __align__(16) float smem[];
    const int64_t t = xcd_block();
    if (t >= tiles) return;   // the grid is rounded up to a multiple of 8
    const BatchImage& b = im[batch_image_of<&BatchImage::sbt_off>(im, n, t)];
    sb_tile<s, TI>(ids + b.q_off * K, m + b.q_off, wt + b.q_off * K, mu + b.q_off, resid, K, b.h, b.w,
                   t - b.sbt_off, part + b.sbt_off * SbGeom<s, TI>::PART, smem);
}

template <int s, int TI>
__global__ __launch_bounds__(256) void k_b_sb_combine(const BatchImage* __restrict__ im, int n, int64_t total,
                                                      const float* __restrict__ part) {
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < total; p += (int64_t)gridDim.x * blockDim.x) {
        const BatchImage& b = im[batch_image_of<&BatchImage::hr_off>(im, n, p)];
        const int W = s * b.w;
        const int64_t lp = p - b.hr_off;
        const int Y = (int)(lp / W), X = (int)(lp - (int64_t)Y * W);
        b.out[lp] = sb_pixel<s, TI>(part + b.sbt_off * SbGeom<s, TI>::PART, b.lr, b.h, b.w, Y, X);
    }
}

int64_t sb_tiles(int s, int rows, int h, int w) {
    if (h < kPatch || w < kPatch) return 0;
    const int64_t npi = h - kPatch + 1, npj = w - kPatch + 1;
    return ((npi + rows - 1) / rows) * ((npj + sb_cols(s) - 1) / sb_cols(s));
}

int64_t sb_part_floats(int s, int rows) {
    const int64_t cy = rows + kPatch - 1, cx = sb_cols(s) + kPatch - 1;
    return cy * s * cx * s + cy * cx;
}

// Up to 16 neighbours the lists of a workgroup's patches fit beside their values in
// LDS (25.6 KB). us entry by entry, in 16-byte loads and staged, both kernels, 140k
// pairs, caches as the query leaves them: x2, 150 tiles, K = 5 33, -, 30, K = 8 40, 33,
// 33, K = 15 54, -, 44; x3, 220 tiles, K = 5 64, -, 45, K = 8 78, 54, 49.
static SbLists sb_lists(int K, const int32_t* ids, const float* wt) {
    if (K <= kMaxK) return kSbStaged;
    return K % 4 == 0 && ((reinterpret_cast<uintptr_t>(ids) | reinterpret_cast<uintptr_t>(wt)) & 15) == 0 ? kSbWide
                                                                                                          : kSbEntries;
}
// Rows of cells below the line, whole tiles from it on: with few tiles the tiles'
// chains leave the chip idle, with many the pieces of the residual rows cost more.
// us in rows and in tiles, as above: x2, K = 5, 16 tiles 17 and 37, 150 30 and 47, 217 36
// and 48, 333 49 and 53; lists of 72 150 tiles 99 and 192, 333 147 and 193; x3, K = 5,
// 220 tiles 45 and 68, 350 60 and 72; x4 220 40 and 62, 494 74 and 72. x1, K = 5, 100
// tiles 21 and 34, 210 29 and 36, 390 43 and 40; lists of 72 210 tiles 109 and 155, 390
// 175 and 163. Lists past 16 entry by entry (72, caches warm): x2 150 tiles 145 and 155,
// 217 161 and 152. (A form that wrote the patches out took x2, K = 5, 17, 32, 47 and 64,
// and ten times the tiles' scratch.)
static int64_t sb_few_tiles(int s, SbLists lm) { return s > 1 && lm != kSbEntries ? 300 : 200; }

template <int s, int TI>
static hipError_t sb_launch(int K, int h, int w, const int32_t* ids, const int32_t* m, const float* wt,
                            const double* mu, const float* resid, float* part, const float* lr, float* hr,
                            hipStream_t st, int which) {
    using G = SbGeom<s, TI>;
    const int64_t nt = sb_tiles(s, TI, h, w), total = (int64_t)s * h * s * w;
    if (which & 1 && nt > 0) {
        if (nt > 0x7FFFFFFF) return hipErrorInvalidValue;
        const SbLists lm = sb_lists(K, ids, wt);
        if (nt < sb_few_tiles(s, lm)) {
            auto k = lm == kSbStaged ? k_sb_row<s, TI, kSbStaged> : lm == kSbWide ? k_sb_row<s, TI, kSbWide>
                                                                                  : k_sb_row<s, TI, kSbEntries>;
            hipLaunchKernelGGL(k, dim3((unsigned)round_grid8((int)nt * G::CY)), dim3(kSbThreads),
                               lm == kSbStaged ? 8 * (size_t)(kPatch * G::TJ * K) : 0, st, K, h, w, ids, m, wt, mu, resid,
                               part);
        } else
            hipLaunchKernelGGL((k_sb_tile<s, TI>), dim3((unsigned)round_grid8((int)nt)), dim3(kSbThreads), G::lds(K), st,
                               K, h, w, ids, m, wt, mu, resid, part);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (which & 2 && total > 0)
        hipLaunchKernelGGL((k_sb_combine<s, TI>), dim3((unsigned)std::min<int64_t>((total + 255) / 256, 1 << 20)),
                           dim3(256), 0, st, part, lr, h, w, hr);
    return hipGetLastError();
}

hipError_t launch_synth_blend(int scale, int rows, int K, int h, int w, const int32_t* ids, const int32_t* m,
                              const float* wt, const double* mu, const float* resid, float* part, const float* lr,
                              float* hr, hipStream_t st, int which) {
    if (K < 1 || K > kAllMax || (rows != 4 && rows != 8)) return hipErrorInvalidValue;
    switch (scale * 10 + rows) {
        case 14: return sb_launch<1, 4>(K, h, w, ids, m, wt, mu, resid, part, lr, hr, st, which);
        case 18: return sb_launch<1, 8>(K, h, w, ids, m, wt, mu, resid, part, lr, hr, st, which);
        case 24: return sb_launch<2, 4>(K, h, w, ids, m, wt, mu, resid, part, lr, hr, st, which);
        case 28: return sb_launch<2, 8>(K, h, w, ids, m, wt, mu, resid, part, lr, hr, st, which);
        case 34: return sb_launch<3, 4>(K, h, w, ids, m, wt, mu, resid, part, lr, hr, st, which);
        case 38: return sb_launch<3, 8>(K, h, w, ids, m, wt, mu, resid, part, lr, hr, st, which);
        case 44: return sb_launch<4, 4>(K, h, w, ids, m, wt, mu, resid, part, lr, hr, st, which);
        case 48: return sb_launch<4, 8>(K, h, w, ids, m, wt, mu, resid, part, lr, hr, st, which);
        default: return hipErrorInvalidValue;
    }
}

template <int s, int TI>
static hipError_t b_sb_launch(const BatchImage* im, int n, int64_t tiles, int64_t hr_total, int K, const int32_t* ids,
                              const int32_t* m, const float* wt, const double* mu, const float* resid, float* part,
                              hipStream_t st) {
    if (tiles > 0) {
        if (tiles > 0x7FFFFFFF) return hipErrorInvalidValue;
        const size_t lds = SbGeom<s, TI>::lds(K);
        hipLaunchKernelGGL((k_b_sb_tile<s, TI>), dim3((unsigned)round_grid8((int)tiles)), dim3(kSbThreads),
                           lds, st, im, n, tiles, K, ids, m, wt, mu, resid, part);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (hr_total > 0)
        hipLaunchKernelGGL((k_b_sb_combine<s, TI>), dim3((unsigned)std::min<int64_t>((hr_total + 255) / 256, 1 << 20)),
                           dim3(256), 0, st, im, n, hr_total, part);
    return hipGetLastError();
}

hipError_t launch_b_synth_blend(const BatchImage* im, int n, int64_t tiles, int64_t hr_total, int scale, int rows,
                                int K, const int32_t* ids, const int32_t* m, const float* wt, const double* mu,
                                const float* resid, float* part, hipStream_t st) {
    if (K < 1 || K > kMaxK || (rows != 4 && rows != 8)) return hipErrorInvalidValue;
    switch (scale * 10 + rows) {
        case 14: return b_sb_launch<1, 4>(im, n, tiles, hr_total, K, ids, m, wt, mu, resid, part, st);
        case 18: return b_sb_launch<1, 8>(im, n, tiles, hr_total, K, ids, m, wt, mu, resid, part, st);
        case 24: return b_sb_launch<2, 4>(im, n, tiles, hr_total, K, ids, m, wt, mu, resid, part, st);
        case 28: return b_sb_launch<2, 8>(im, n, tiles, hr_total, K, ids, m, wt, mu, resid, part, st);
        case 34: return b_sb_launch<3, 4>(im, n, tiles, hr_total, K, ids, m, wt, mu, resid, part, st);
        case 38: return b_sb_launch<3, 8>(im, n, tiles, hr_total, K, ids, m, wt, mu, resid, part, st);
        case 44: return b_sb_launch<4, 4>(im, n, tiles, hr_total, K, ids, m, wt, mu, resid, part, st);
        case 48: return b_sb_launch<4, 8>(im, n, tiles, hr_total, K, ids, m, wt, mu, resid, part, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace zh
