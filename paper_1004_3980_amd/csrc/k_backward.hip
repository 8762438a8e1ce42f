// Adjoint of the zoom: gradients of a loss on the output image with respect
// to the dictionary's HR residual patches and the LLE regulariser lambda.
// Neighbour indices (hash codes, candidates, top-K) are discrete and stay at
// their forward values.
//
// Back-projection (Section 4, the update after Eq. Err_img; Section 4.3,
// Eq. sx2 and Eq. bl_filter_3), one iteration I' = I + S(I) F(I) with
// F = N Up (I_L - Dec Blur I) and S = exp(-(I - Box I)^2 / (2 sigma_r^2)):
//
//   g <- g - Blur^T Dec^T Up^T N^T (S g) + (Id - Box)^T [-(a / sigma_r^2) S F g],
//
// a = I - Box I. Every operator is separable (a matrix per axis with
// replicate or in-image-normalised borders), so each transpose is two
// one-axis gathers (k_adj_down, k_adj_up) whose weights are rebuilt from the
// forward definitions: normalised Gaussian (taps inside the image, divided by their
// sum), box mean (in-image count), Keys' cubic (a = -0.5, replicate border),
// Gaussian blur with replicate border followed by phase-0 decimation.
//
// Blend (per-pixel mean of the covering patches): each patch pixel receives
// g(X) / cnt(X). Synthesis x_q = mu_q + sum_m w_qm r_{n_qm} (Eq. HR_Rec):
// dL/dr_n = sum over the (q, m) with n_qm = n of w_qm g_q, gathered per
// dictionary row over a stable sort of the neighbour lists (no float
// atomics, fixed order); dL/dw_qm = <g_q, r_{n_qm}>. LLE weights (Eq. LinSys)
// with A = G + lambda tr(G) I: the Gram matrix is recomputed in FP64 and
// factorised again, dw~/dlambda = -tr(G) A^-1 w~, dw/dlambda =
// (dw~/dlambda - w 1^T dw~/dlambda) / 1^T w~; dL/dlambda is a fixed-order
// FP64 reduction over the patches.
#include <cmath>

#include "zh_internal.h"

namespace zh {

// HR patch values per lane, in chunks of 64, at the largest zoom factor
constexpr int kPixChunks = (kMaxPs2 + 63) / 64;

// ---- adjoint of a back-projection iteration ----------------------------------
// Two kernels an iteration, each a chain of one-axis gathers within a tile: the
// gradient down to the LR error (k_adj_down), then back up, with the range term
// (k_adj_up). The weights of an axis are formed once a tile; places outside the
// image carry zero values or weights, which leave every sum as if they were
// skipped, and each sum runs over the axis in ascending order.
// Bound: latency of the tile's stages. A launch per axis and operator, with the
// weights (and their divisions) formed for each output: ten launches and 73 us
// an iteration at 400x432 HR, now two and 27.

// Weights of the transposed normalised Gaussian: w[x][k] = c(k - R) / nrm(x) for
// the places x0 .. x0 + n - 1 of an axis of length len, nrm(x) = sum of the
// taps inside the image at x
template <int RM>
__device__ __forceinline__ void gauss_adj_weights(const float* taps, int R, int x0, int n, int len, float* w) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const int x = x0 + i;
        float nrm = 0.0f;
        for (int d = -R; d <= R; ++d)
            if (x + d >= 0 && x + d < len) nrm += taps[d + R];
        for (int k = 0; k <= 2 * R; ++k) w[i * (2 * RM + 1) + k] = x >= 0 && x < len ? taps[k] / nrm : 0.0f;
    }
}
// Weights of the transposed bicubic upsampling: w[o][k] of HR place S (o - 2) + k
// in LR place o = o0 + i: HR place x reads LR floor(x / S) - 1 + t, t = 0..3,
// clamped
template <int S>
__device__ __forceinline__ void up_adj_weights(int o0, int n, int nlr, float* w) {
    for (int e = threadIdx.x; e < n * 5 * S; e += blockDim.x) {
        const int i = e / (5 * S), k = e - i * 5 * S, o = o0 + i, x = S * (o - 2) + k;
        float wsum = 0.0f;
        if (o < nlr && x >= 0 && x < S * nlr) {
            const int i0 = x / S;
            const float tx = (float)(x - i0 * S) / (float)S;
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (clampi(i0 - 1 + t, 0, nlr - 1) == o) wsum += keys_w(tx - (float)(t - 1));
        }
        w[e] = wsum;
    }
}

// Up^T N^T (S g) at an LR tile of T x T: the product S g under it with the
// Gaussian's halo, the Gaussian's transpose along x and y, the upsampling's.
template <int S, int RM, int T>
__global__ __launch_bounds__(256) void k_adj_down(BpAdjArgs a) {
    constexpr int N = S * (T + 4), M = N + 2 * RM, TP = 2 * RM + 1;
    __shared__ float sIn[M * M], sA[M * N];
    __shared__ float wgx[M * TP], wgy[M * TP], wux[T * 5 * S], wuy[T * 5 * S];
    float* sB = sIn;    // [N][N]: the input is no longer read
    float* sU = sA;     // [N][T]
    const int H = S * a.h, W = S * a.w, R = a.R, m = N + 2 * R;
    const int i0 = blockIdx.y * T, j0 = blockIdx.x * T;
    const int Y0 = S * (i0 - 2), X0 = S * (j0 - 2);      // first HR row and column of the Gaussian's output
    for (int e = threadIdx.x; e < m * m; e += 256) {
        const int r = e / m, c = e - r * m, Y = Y0 - R + r, X = X0 - R + c;
        float v = 0.0f;
        if (Y >= 0 && Y < H && X >= 0 && X < W) {
            const int64_t p = (int64_t)Y * W + X;
            v = a.g[p] * a.FSa[(int64_t)H * W + p];
        }
        sIn[r * M + c] = v;
    }
    gauss_adj_weights<RM>(a.taps, R, X0 - R, m, W, wgx);
    gauss_adj_weights<RM>(a.taps, R, Y0 - R, m, H, wgy);
    up_adj_weights<S>(j0, T, a.w, wux);
    up_adj_weights<S>(i0, T, a.h, wuy);
    __syncthreads();
    // out[o] = sum_x c(o - x) in[x] / nrm(x)
    for (int e = threadIdx.x; e < m * N; e += 256) {
        const int r = e / N, c = e - r * N;
        float acc = 0.0f;
        for (int k = 0; k <= 2 * R; ++k) acc = fmaf(wgx[(c + k) * TP + 2 * R - k], sIn[r * M + c + k], acc);
        sA[r * N + c] = acc;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < N * N; e += 256) {
        const int r = e / N, c = e - r * N;
        float acc = 0.0f;
        for (int k = 0; k <= 2 * R; ++k) acc = fmaf(wgy[(r + k) * TP + 2 * R - k], sA[(r + k) * N + c], acc);
        sB[r * N + c] = acc;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < N * T; e += 256) {
        const int r = e / T, o = e - r * T;
        float acc = 0.0f;
#pragma unroll
        for (int k = 0; k < 5 * S; ++k) acc = fmaf(wux[o * 5 * S + k], sB[r * N + S * o + k], acc);
        sU[r * T + o] = acc;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < T * T; e += 256) {
        const int i = e / T, o = e - i * T;
        float acc = 0.0f;
#pragma unroll
        for (int k = 0; k < 5 * S; ++k) acc = fmaf(wuy[i * 5 * S + k], sU[(S * i + k) * T + o], acc);
        if (i0 + i < a.h && j0 + o < a.w) a.lr[(int64_t)(i0 + i) * a.w + j0 + o] = acc;
    }
}

// First LR place whose blur reads HR place o, and the weights of it and the
// following (LR place i reads HR clamp(S i + t), |t| <= R = 3)
template <int S>
struct DecAdj {
    static constexpr int R = 3, TERMS = 2 * R / S + 3;
    __device__ static int first(int o) { return max(0, (o - R) / S - 1); }
    __device__ static void weights(const float* dec, int o, int nlr, float* w) {
        const int ilo = first(o), ihi = min(nlr - 1, (o + R) / S + 1);
        for (int k = 0; k < TERMS; ++k) {
            float wsum = 0.0f;
            if (ilo + k <= ihi)
                for (int t = -R; t <= R; ++t)
                    if (clampi(S * (ilo + k) + t, 0, S * nlr - 1) == o) wsum += dec[t + R];
            w[k] = wsum;
        }
    }
};

// g' = g - Blur^T Dec^T lr + (Id - Box)^T z at an HR tile of T x T,
// z = -(a / sigma_r^2) S F g (none where the range weight is constant)
template <int S, int RM>
__global__ __launch_bounds__(256) void k_adj_up(BpAdjArgs a) {
    using DA = DecAdj<S>;
    constexpr int T = 32, M = T + 2 * RM, L = (T + 2 * DA::R) / S + 5, TERMS = DA::TERMS;
    __shared__ float sZ[M * M], sBx[M * T], sL[L * L], sX[L * T];
    __shared__ float wdx[T * TERMS], wdy[T * TERMS];
    const int H = S * a.h, W = S * a.w, R = a.R, m = T + 2 * R;
    const int64_t n = (int64_t)H * W;
    const int Y0 = blockIdx.y * T, X0 = blockIdx.x * T;
    const int il = DA::first(Y0), jl = DA::first(X0);
    for (int e = threadIdx.x; e < L * L; e += 256) {
        const int r = e / L, c = e - r * L;
        sL[e] = il + r < a.h && jl + c < a.w ? a.lr[(int64_t)(il + r) * a.w + jl + c] : 0.0f;
    }
    auto zat = [&](int64_t p) { return -(a.FSa[2 * n + p] * a.inv_sr2) * a.FSa[n + p] * a.FSa[p] * a.g[p]; };
    if (a.range) {
        for (int e = threadIdx.x; e < m * m; e += 256) {
            const int r = e / m, c = e - r * m, Y = Y0 - R + r, X = X0 - R + c;
            float v = 0.0f;
            if (Y >= 0 && Y < H && X >= 0 && X < W)
                v = zat((int64_t)Y * W + X) / (float)(min(W - 1, X + R) - max(0, X - R) + 1);
            sZ[r * M + c] = v;
        }
    }
    if (threadIdx.x < T)
        DA::weights(a.dec, X0 + threadIdx.x, a.w, wdx + threadIdx.x * TERMS);
    else if (threadIdx.x < 2 * T)
        DA::weights(a.dec, Y0 + threadIdx.x - T, a.h, wdy + (threadIdx.x - T) * TERMS);
    __syncthreads();
    for (int e = threadIdx.x; e < L * T; e += 256) {
        const int r = e / T, c = e - r * T;
        const float* row = sL + r * L + DA::first(X0 + c) - jl;
        float acc = 0.0f;
#pragma unroll
        for (int k = 0; k < TERMS; ++k) acc = fmaf(wdx[c * TERMS + k], row[k], acc);
        sX[e] = acc;
    }
    if (a.range)
        for (int e = threadIdx.x; e < m * T; e += 256) {
            const int r = e / T, c = e - r * T, Y = Y0 - R + r;
            float acc = 0.0f;
            for (int k = 0; k <= 2 * R; ++k) acc += sZ[r * M + c + k];
            sBx[e] = Y >= 0 && Y < H ? acc / (float)(min(H - 1, Y + R) - max(0, Y - R) + 1) : 0.0f;
        }
    __syncthreads();
    for (int e = threadIdx.x; e < T * T; e += 256) {
        const int r = e / T, c = e - r * T, Y = Y0 + r, X = X0 + c;
        if (Y >= H || X >= W) continue;
        const float* col = sX + (DA::first(Y) - il) * T + c;
        float v = 0.0f;
#pragma unroll
        for (int k = 0; k < TERMS; ++k) v = fmaf(wdy[r * TERMS + k], col[k * T], v);
        const int64_t p = (int64_t)Y * W + X;
        float o = a.g[p] - v;
        if (a.range) {
            float bz = 0.0f;
            for (int k = 0; k <= 2 * R; ++k) bz += sBx[(r + k) * T + c];
            o += zat(p) - bz;
        }
        a.out[p] = o;
    }
}

template <int S, int RM>
static void launch_adj(const BpAdjArgs& a, hipStream_t st) {
    constexpr int T = S <= 2 ? 16 : 8;
    hipLaunchKernelGGL((k_adj_down<S, RM, T>), dim3((a.w + T - 1) / T, (a.h + T - 1) / T), dim3(256), 0, st, a);
    hipLaunchKernelGGL((k_adj_up<S, RM>), dim3((S * a.w + 31) / 32, (S * a.h + 31) / 32), dim3(256), 0, st, a);
}

hipError_t launch_bp_adj(const BpAdjArgs& a, int scale, hipStream_t st) {
    if (a.R < 0 || a.R > kMaxAdjR || scale < 1 || scale > kMaxScale || a.h < 1 || a.w < 1) return hipErrorInvalidValue;
    const bool small = a.R <= 5;
    switch (scale) {
        case 1: small ? launch_adj<1, 5>(a, st) : launch_adj<1, kMaxAdjR>(a, st); break;
        case 2: small ? launch_adj<2, 5>(a, st) : launch_adj<2, kMaxAdjR>(a, st); break;
        case 3: small ? launch_adj<3, 5>(a, st) : launch_adj<3, kMaxAdjR>(a, st); break;
        default: small ? launch_adj<4, 5>(a, st) : launch_adj<4, kMaxAdjR>(a, st);
    }
    return hipGetLastError();
}

static dim3 grid1(int64_t n) {
    int64_t g = (n + 255) / 256;
    return dim3((unsigned)(g > 65536 ? 65536 : (g < 1 ? 1 : g)));
}

// ---- blend adjoint: gradient per covered pixel divided by its count ---------
__global__ void k_blend_adj(const float* __restrict__ g, const int32_t* __restrict__ m, int h, int w, int s,
                            float* __restrict__ gp) {
    const int H = s * h, W = s * w, ps = kPatch * s;
    const int npi = h - kPatch + 1, npj = w - kPatch + 1;
    const int64_t total = (int64_t)H * W;
    for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * blockDim.x) {
        const int Y = (int)(idx / W), X = (int)(idx % W);
        const int ilo = Y - ps + 1 <= 0 ? 0 : (Y - ps + s) / s;
        const int ihi = min(npi - 1, Y / s);
        const int jlo = X - ps + 1 <= 0 ? 0 : (X - ps + s) / s;
        const int jhi = min(npj - 1, X / s);
        int cnt = 0;
        for (int i = ilo; i <= ihi; ++i)
            for (int j = jlo; j <= jhi; ++j) cnt += m[i * npj + j] > 0 ? 1 : 0;
        gp[idx] = cnt > 0 ? g[idx] / (float)cnt : 0.0f;
    }
}

hipError_t launch_blend_adj(const float* g, const int32_t* m, int h, int w, int s, float* gp, hipStream_t st) {
    hipLaunchKernelGGL(k_blend_adj, grid1((int64_t)s * h * s * w), dim3(256), 0, st, g, m, h, w, s, gp);
    return hipGetLastError();
}

// ---- LLE adjoint through lambda: one wave per patch --------------------------
// dL/dw_m = <g_q, r_{n_m}> over the patch's HR pixels; the Gram matrix of
// Z = q - X_N in FP64 (coordinates over the lanes, wave sums), then on lane
// 0: A = G + lambda tau I, Cholesky, w~ = A^-1 1, d = -tau A^-1 w~,
// contribution [g_w . d - (g_w . w)(1 . d)] / (1 . w~).
template <int U>
__global__ __launch_bounds__(256) void k_lle_lambda_adj(BackwardArgs a) {
    const int lane = threadIdx.x & 63;
    const int wpb = blockDim.x >> 6;
    const int D = a.D, K = a.K, s = a.s, ps = kPatch * s, ps2 = ps * ps;
    const int npj = a.w - kPatch + 1;
    const int W = s * a.w;
    for (int q = blockIdx.x * wpb + (threadIdx.x >> 6); q < a.Q; q += gridDim.x * wpb) {
        const int mq = a.m[q];
        if (mq <= 0) {
            if (lane == 0) a.c_lam[q] = 0.0;
            continue;
        }
        const int pi = q / npj, pj = q % npj;
        // patch gradient values of this lane: pixels lane + 64 u
        float gq[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int P = lane + 64 * u;
            gq[u] = 0.0f;
            if (P < ps2) {
                const int py = P / ps, px = P % ps;
                gq[u] = a.gp[(int64_t)(s * pi + py) * W + s * pj + px];
            }
        }
        double gw[kMaxK];
        for (int mi = 0; mi < K; ++mi) {
            double acc = 0.0;
            if (mi < mq) {
                const float* r = a.resid + (int64_t)a.ids[(int64_t)q * K + mi] * ps2;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int P = lane + 64 * u;
                    if (P < ps2) acc += (double)gq[u] * (double)r[P];
                }
            }
            gw[mi] = wave_sum_f64(acc);
        }
        // Gram of Z = q - x_n (FP64), coordinates lane and lane + 64
        double z0[kMaxK], z1[kMaxK];
        const float* qf = a.qfeat + (int64_t)q * D;
        for (int mi = 0; mi < K; ++mi) {
            z0[mi] = z1[mi] = 0.0;
            if (mi < mq) {
                const int64_t id = a.ids[(int64_t)q * K + mi];
                if (lane < D)
                    z0[mi] = (double)qf[lane] - (double)join_planes(a.hi[id * a.hs + lane], a.lo[id * D + lane]);
                if (lane + 64 < D)
                    z1[mi] = (double)qf[lane + 64] -
                             (double)join_planes(a.hi[id * a.hs + lane + 64], a.lo[id * D + lane + 64]);
            }
        }
        double G[kMaxK * (kMaxK + 1) / 2];
        for (int i = 0; i < mq; ++i)
            for (int j = 0; j <= i; ++j) G[i * (i + 1) / 2 + j] = wave_sum_f64(z0[i] * z0[j] + z1[i] * z1[j]);
        if (lane == 0) {
            double tau = 0.0;
            for (int i = 0; i < mq; ++i) tau += G[i * (i + 1) / 2 + i];
            double contrib = 0.0;
            if (tau > 0.0) {
                // Cholesky of A = G + lambda tau I (lower, packed)
                double Lc[kMaxK * (kMaxK + 1) / 2];
                for (int i = 0; i < mq; ++i) {
                    for (int j = 0; j <= i; ++j) {
                        double v = G[i * (i + 1) / 2 + j] + (i == j ? a.lam * tau : 0.0);
                        for (int t = 0; t < j; ++t) v -= Lc[i * (i + 1) / 2 + t] * Lc[j * (j + 1) / 2 + t];
                        Lc[i * (i + 1) / 2 + j] = i == j ? sqrt(v) : v / Lc[j * (j + 1) / 2 + j];
                    }
                }
                auto solve = [&](const double* b, double* x) {
                    for (int i = 0; i < mq; ++i) {
                        double v = b[i];
                        for (int t = 0; t < i; ++t) v -= Lc[i * (i + 1) / 2 + t] * x[t];
                        x[i] = v / Lc[i * (i + 1) / 2 + i];
                    }
                    for (int i = mq - 1; i >= 0; --i) {
                        double v = x[i];
                        for (int t = i + 1; t < mq; ++t) v -= Lc[t * (t + 1) / 2 + i] * x[t];
                        x[i] = v / Lc[i * (i + 1) / 2 + i];
                    }
                };
                double one[kMaxK], wt[kMaxK], d[kMaxK];
                for (int i = 0; i < mq; ++i) one[i] = 1.0;
                solve(one, wt);
                double sig = 0.0;
                for (int i = 0; i < mq; ++i) sig += wt[i];
                solve(wt, d);
                double dsum = 0.0, gd = 0.0, gww = 0.0;
                for (int i = 0; i < mq; ++i) {
                    d[i] *= -tau;
                    dsum += d[i];
                    gd += gw[i] * d[i];
                    gww += gw[i] * wt[i] / sig;
                }
                contrib = (gd - gww * dsum) / sig;
            }
            a.c_lam[q] = contrib;
        }
    }
}

// dL/dw_m = <g_q, r_{n_m}> for K <= 8, one wave per patch (pixels lane + 64 u),
// into gw[q][8] (FP64, zero past m_q).
template <int U>
__global__ __launch_bounds__(256) void k_lam_gw(BackwardArgs a, double* __restrict__ gw) {
    const int lane = threadIdx.x & 63;
    const int wpb = blockDim.x >> 6;
    const int K = a.K, s = a.s, ps = kPatch * s, ps2 = ps * ps;
    const int npj = a.w - kPatch + 1;
    const int W = s * a.w;
    for (int q = blockIdx.x * wpb + (threadIdx.x >> 6); q < a.Q; q += gridDim.x * wpb) {
        const int mq = a.m[q];
        const int pi = q / npj, pj = q - (q / npj) * npj;
        float gq[U];
        int P4[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int P = lane + 64 * u;
            P4[u] = P;
            gq[u] = 0.0f;
            if (P < ps2 && mq > 0) {
                const int py = P / ps, px = P - py * ps;
                gq[u] = a.gp[(int64_t)(s * pi + py) * W + s * pj + px];
            }
        }
#pragma unroll
        for (int mi = 0; mi < 8; ++mi) {
            double acc = 0.0;
            if (mi < mq) {
                const float* r = a.resid + (int64_t)a.ids[(int64_t)q * K + mi] * ps2;
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (P4[u] < ps2) acc += (double)gq[u] * (double)r[P4[u]];
            }
            acc = wave_sum_f64(acc);
            if (lane == mi) gw[(int64_t)q * 8 + mi] = acc;
        }
    }
}

// Contribution of each patch to dL/dlambda (K <= 8), one thread per patch,
// from its packed FP64 Gram matrix G and gw: with tau = tr(G) and
// A = G + lambda tau I factored again here (Cholesky),
//   w~ = A^-1 1, sigma = sum w~, d = -tau A^-1 w~,
//   dL/dlambda_q = (gw.d - (gw.w~ / sigma) sum d) / sigma.
__global__ __launch_bounds__(256) void k_lam_solve(BackwardArgs a, const double* __restrict__ gram,
                                                   const double* __restrict__ gw) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= a.Q) return;
    const int m = a.m[q];
    double A[36], g[8];
#pragma unroll
    for (int p = 0; p < 36; ++p) A[p] = gram[(int64_t)q * 36 + p];
#pragma unroll
    for (int i = 0; i < 8; ++i) g[i] = i < m ? gw[(int64_t)q * 8 + i] : 0.0;
    double tau = 0.0;
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if (i < m) tau += A[i * (i + 1) / 2 + i];
    if (m <= 0 || !(tau > 0.0)) {
        a.c_lam[q] = 0.0;
        return;
    }
    // rows m..7: identity, so that the unrolled factorisation stays valid
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) {
            double& x = A[i * (i + 1) / 2 + j];
            if (i >= m || j >= m) x = i == j ? 1.0 : 0.0;
            else if (i == j) x += a.lam * tau;
        }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        double v = A[j * (j + 1) / 2 + j];
#pragma unroll
        for (int t = 0; t < j; ++t) v -= A[j * (j + 1) / 2 + t] * A[j * (j + 1) / 2 + t];
        A[j * (j + 1) / 2 + j] = sqrt(v);
#pragma unroll
        for (int i = j + 1; i < 8; ++i) {
            double t2 = A[i * (i + 1) / 2 + j];
#pragma unroll
            for (int t = 0; t < j; ++t) t2 -= A[i * (i + 1) / 2 + t] * A[j * (j + 1) / 2 + t];
            A[i * (i + 1) / 2 + j] = t2 / A[j * (j + 1) / 2 + j];
        }
    }
    auto solve = [&](const double (&b)[8], double (&x)[8]) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            double v = b[i];
#pragma unroll
            for (int t = 0; t < i; ++t) v -= A[i * (i + 1) / 2 + t] * x[t];
            x[i] = v / A[i * (i + 1) / 2 + i];
        }
#pragma unroll
        for (int i = 7; i >= 0; --i) {
            double v = x[i];
#pragma unroll
            for (int t = i + 1; t < 8; ++t) v -= A[t * (t + 1) / 2 + i] * x[t];
            x[i] = v / A[i * (i + 1) / 2 + i];
        }
    };
    double one[8], wt[8], d[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) one[i] = i < m ? 1.0 : 0.0;
    solve(one, wt);
    double sig = 0.0;
#pragma unroll
    for (int i = 0; i < 8; ++i) sig += i < m ? wt[i] : 0.0;
    solve(wt, d);
    double dsum = 0.0, gd = 0.0, gww = 0.0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (i < m) {
            const double di = -tau * d[i];
            dsum += di;
            gd += g[i] * di;
            gww += g[i] * wt[i] / sig;
        }
    }
    a.c_lam[q] = (gd - gww * dsum) / sig;
}

hipError_t launch_lam_adj8(const BackwardArgs& a, const double* gram, double* gw, hipStream_t st) {
    if (a.Q == 0) return hipSuccess;
    if (a.K > 8 || a.s < 1 || a.s > kMaxScale) return hipErrorInvalidValue;
    int g = (a.Q + 3) / 4;
    if (g > 65536) g = 65536;
    if (kPatch * a.s * kPatch * a.s <= 256) hipLaunchKernelGGL(k_lam_gw<4>, dim3(g), dim3(256), 0, st, a, gw);
    else hipLaunchKernelGGL(k_lam_gw<kPixChunks>, dim3(g), dim3(256), 0, st, a, gw);
    hipLaunchKernelGGL(k_lam_solve, dim3((a.Q + 255) / 256), dim3(256), 0, st, a, gram, gw);
    return hipGetLastError();
}

hipError_t launch_lle_lambda_adj(const BackwardArgs& a, hipStream_t st) {
    if (a.K > kMaxK || a.D > 128 || a.s < 1 || a.s > kMaxScale) return hipErrorInvalidValue;
    int g = (a.Q + 3) / 4;
    if (g > 65536) g = 65536;
    if (g < 1) g = 1;
    if (kPatch * a.s * kPatch * a.s <= 256) hipLaunchKernelGGL(k_lle_lambda_adj<4>, dim3(g), dim3(256), 0, st, a);
    else hipLaunchKernelGGL(k_lle_lambda_adj<kPixChunks>, dim3(g), dim3(256), 0, st, a);
    return hipGetLastError();
}

// Fixed-order FP64 sum of n values: one workgroup, thread t adds t, t + 1024,
// ... in order, then a tree over the threads; the result is rounded to fp32.
__global__ __launch_bounds__(1024) void k_sum_f64(const double* __restrict__ x, int64_t n, float* __restrict__ out) {
    __shared__ double s[1024];
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 1024) acc += x[i];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = (float)s[0];
}

hipError_t launch_sum_f64(const double* x, int64_t n, float* out, hipStream_t st) {
    hipLaunchKernelGGL(k_sum_f64, dim3(1), dim3(1024), 0, st, x, n, out);
    return hipGetLastError();
}

// ---- dictionary gradient ----------------------------------------------------
// Neighbour list entries e = q K + m as (key = dictionary row, value = e);
// entries past m_q get the key `none` and sort last.
__global__ void k_nbr_pairs(const int32_t* __restrict__ ids, const int32_t* __restrict__ m, int Q, int K,
                            uint32_t none, uint32_t* __restrict__ key, uint32_t* __restrict__ val) {
    const int64_t total = (int64_t)Q * K;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int q = (int)(e / K), mi = (int)(e % K);
        key[e] = mi < m[q] ? (uint32_t)ids[e] : none;
        val[e] = (uint32_t)e;
    }
}

hipError_t launch_nbr_pairs(const int32_t* ids, const int32_t* m, int Q, int K, uint32_t none, uint32_t* key,
                            uint32_t* val, hipStream_t st) {
    hipLaunchKernelGGL(k_nbr_pairs, grid1((int64_t)Q * K), dim3(256), 0, st, ids, m, Q, K, none, key, val);
    return hipGetLastError();
}

// Gradient of each dictionary row that some patch uses: the sum over its
// entries (q, m) of w_qm g_q, with the pairs sorted stably by row. Pass 1:
// a wave per chunk of 64 consecutive entries (one per lane) sums each run of
// equal rows inside the chunk in entry order (lane = pixel); a run that lies
// wholly in the chunk is written, while a run that crosses a chunk border
// leaves its partial sum in the chunk's first or last slot. Pass 2: a wave
// per run that starts in a chunk and continues into the next adds the
// partial sums in chunk order. The result depends only on the sorted pairs:
// equal calls give equal gradients.
struct DictGradChunk {
    uint32_t key_last;   // row of the chunk's last run
    uint8_t nseg;        // runs (of used rows) starting or continuing in the chunk
    uint8_t first_cont;  // the first run continues from the previous chunk
    uint8_t last_cont;   // the last run continues into the next chunk
    uint8_t last_start;  // the last run starts in this chunk
};

template <int U>
__global__ __launch_bounds__(256) void k_dict_grad(const uint32_t* __restrict__ key, const uint32_t* __restrict__ val,
                                                   int64_t n_ent, uint32_t none, const float* __restrict__ wts,
                                                   const float* __restrict__ gp, int w, int s, int K,
                                                   float* __restrict__ g_r, float* __restrict__ part,
                                                   DictGradChunk* __restrict__ info) {
    const int lane = threadIdx.x & 63;
    const int wpb = blockDim.x >> 6;
    const int ps = kPatch * s, ps2 = ps * ps;
    const int npj = w - kPatch + 1, W = s * w;
    int off[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int P = lane + 64 * u;
        off[u] = P < ps2 ? (P / ps) * W + P % ps : 0;
    }
    const int64_t nchunk = (n_ent + 63) / 64;
    for (int64_t c = (int64_t)blockIdx.x * wpb + (threadIdx.x >> 6); c < nchunk; c += (int64_t)gridDim.x * wpb) {
        const int64_t base = c * 64;
        const int64_t e = base + lane;
        const bool in = e < n_ent;
        const uint32_t k = in ? key[e] : none;
        const uint32_t kprev = (in && e > 0) ? key[e - 1] : none;
        const uint32_t knext = (e + 1 < n_ent) ? key[e + 1] : none;
        const uint32_t v = in ? val[e] : 0u;
        const float wv = (in && k != none) ? wts[v] : 0.0f;
        // segment starts inside the chunk: first lane, or a change of row
        const uint64_t seg = __ballot(in && k != none && (lane == 0 || k != kprev));
        const uint64_t ends = __ballot(in && k != none && (lane == 63 || e + 1 == n_ent || knext != k));
        uint64_t todo = seg;
        while (todo) {
            const int src = __builtin_ctzll(todo);
            todo &= todo - 1;
            const int stop = __builtin_ctzll(ends & (~0ull << src));   // last entry of the segment
            const uint32_t kk = __shfl(k, src);
            float acc[U];
#pragma unroll
            for (int u = 0; u < U; ++u) acc[u] = 0.0f;
            for (int j = src; j <= stop; ++j) {
                const uint32_t vv = __shfl(v, j);
                const float ww = __shfl(wv, j);
                const int q = (int)(vv / (uint32_t)K);
                const int pi = q / npj, pj = q - pi * npj;
                const float* g = gp + (int64_t)s * pi * W + (int64_t)s * pj;
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (lane + 64 * u < ps2) acc[u] = fmaf(ww, g[off[u]], acc[u]);
            }
            const bool from_prev = src == 0 && __shfl(kprev, 0) == kk;
            const bool into_next = stop == 63 && __shfl(knext, 63) == kk;
            float* dst = g_r + (int64_t)kk * ps2;
            if (from_prev) dst = part + (c * 2) * ps2;
            else if (into_next) dst = part + (c * 2 + 1) * ps2;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int P = lane + 64 * u;
                if (P < ps2) dst[P] = acc[u];
            }
        }
        const int last = seg ? 63 - __builtin_clzll(seg) : 0;
        const uint32_t kl = __shfl(k, last);
        const uint32_t k0 = __shfl(k, 0), kp0 = __shfl(kprev, 0);
        const uint32_t k63 = __shfl(k, 63), kn63 = __shfl(knext, 63);
        if (lane == 0) {
            DictGradChunk ci;
            ci.key_last = seg ? kl : none;
            ci.nseg = (uint8_t)__popcll(seg);
            ci.first_cont = (uint8_t)(k0 != none && kp0 == k0);
            ci.last_cont = (uint8_t)(seg && k63 == kl && kn63 == kl);
            ci.last_start = (uint8_t)(seg && !(last == 0 && kp0 == kl));
            info[c] = ci;
        }
    }
}

// Pass 2: runs that cross chunk borders, from the chunk where they start.
template <int U>
__global__ __launch_bounds__(256) void k_dict_grad_join(int64_t n_ent, int s, const float* __restrict__ part,
                                                        const DictGradChunk* __restrict__ info, float* __restrict__ g_r) {
    const int lane = threadIdx.x & 63;
    const int wpb = blockDim.x >> 6;
    const int ps = kPatch * s, ps2 = ps * ps;
    const int64_t nchunk = (n_ent + 63) / 64;
    for (int64_t c = (int64_t)blockIdx.x * wpb + (threadIdx.x >> 6); c < nchunk; c += (int64_t)gridDim.x * wpb) {
        const DictGradChunk ci = info[c];
        if (!ci.last_cont || !ci.last_start) continue;
        // the run starts in chunk c and continues: its partial is in slot 1,
        // and in slot 0 of every later chunk it reaches
        const float* p0 = part + (c * 2 + 1) * ps2;
        float acc[U];
#pragma unroll
        for (int u = 0; u < U; ++u) acc[u] = lane + 64 * u < ps2 ? p0[lane + 64 * u] : 0.0f;
        for (int64_t cc = c + 1; cc < nchunk; ++cc) {
            const DictGradChunk cn = info[cc];
            const float* pp = part + (cc * 2) * ps2;
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (lane + 64 * u < ps2) acc[u] += pp[lane + 64 * u];
            if (!(cn.nseg == 1 && cn.last_cont)) break;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int P = lane + 64 * u;
            if (P < ps2) g_r[(int64_t)ci.key_last * ps2 + P] = acc[u];
        }
    }
}

hipError_t launch_dict_grad(const uint32_t* key, const uint32_t* val, int64_t n_ent, uint32_t none, const float* wts,
                            const float* gp, int w, int s, int K, float* g_r, float* part, void* info,
                            hipStream_t st) {
    if (s < 1 || s > kMaxScale) return hipErrorInvalidValue;
    if (n_ent == 0) return hipSuccess;
    const int64_t nchunk = (n_ent + 63) / 64;
    int64_t g = (nchunk + 3) / 4;
    if (g > 65536) g = 65536;
    DictGradChunk* ci = static_cast<DictGradChunk*>(info);
    if (kPatch * s * kPatch * s <= 256) {
        hipLaunchKernelGGL(k_dict_grad<4>, dim3((unsigned)g), dim3(256), 0, st, key, val, n_ent, none, wts, gp, w, s, K,
                           g_r, part, ci);
        hipLaunchKernelGGL(k_dict_grad_join<4>, dim3((unsigned)g), dim3(256), 0, st, n_ent, s, part, ci, g_r);
    } else {
        hipLaunchKernelGGL(k_dict_grad<kPixChunks>, dim3((unsigned)g), dim3(256), 0, st, key, val, n_ent, none, wts, gp,
                           w, s, K, g_r, part, ci);
        hipLaunchKernelGGL(k_dict_grad_join<kPixChunks>, dim3((unsigned)g), dim3(256), 0, st, n_ent, s, part, ci, g_r);
    }
    return hipGetLastError();
}

}  // namespace zh
