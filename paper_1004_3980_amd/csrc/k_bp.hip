// Back-projection update with the approximate cross bilateral filter
// (Section 4, the update after Eq. Err_img; Section 4.3, Eq. sx2 and
// Eq. bl_filter_3):
//
//   E  = bicubic upsampling of the LR error e = I_L - (g * I) decimated
//   F  = C * E, C a Gaussian of sigma_s over (2R+1)^2, R = ceil(3 sigma_s),
//        normalised over the taps inside the image (separable)
//   mu = mean of I over the in-image pixels of the same window
//   S  = exp(-(I - mu)^2 / (2 sigma_r^2))
//   I' = I + S * F
//
// One workgroup per output tile; I and the LR error are staged with their
// halos in LDS and the separable passes run from LDS. The LR error itself comes
// from the FP64 degradation kernel.
#include <algorithm>
#include <cmath>

#include "zh_internal.h"

namespace zh {

constexpr int kBpMaxR = 8;
constexpr int kBpSmallR = 5;   // sigma_s up to 5/3: less halo to stage, fewer taps to unroll

// One T x T output tile with origin (Y0, X0), R <= RM. TERMS: instead of the
// update, write F, S and a = I - mu (the pieces the adjoint of the iteration
// needs) to out, out + H W and out + 2 H W.
//
// E on the staged region comes from the LR error patch under it: the patch
// (clamped indices, so the border replicates) is staged in LDS and upsampled
// along x for each of its rows; the horizontal pass takes kBpOut outputs a
// thread, upsampling its window along y in registers (the same fused
// multiply-adds in the same order as bicubic_at: bitwise its values), and the
// vertical pass T * T / 256. Taps outside the image carry zero weight and zero
// values, which leave every sum as if they were skipped.
//
// Bound: instruction issue and LDS reads (44 + 44 multiply-adds and adds a
// pixel for the two passes; 32 MB of images at 2048^2 would take 7 us).
// An iteration's update before (256 threads, four outputs a thread, E in a
// pass of its own, divisions by a run-time zoom factor) and now: 2048^2 65 ->
// 37 us, 844x1228 x4 25 -> 15.5, 502x526 19.3 -> 9.3, 128^2 18.5 -> 6.9.
constexpr int kBpOut = 8;   // outputs of a thread of the horizontal pass

template <int T, int RM, int S>
struct BpGeom {
    static constexpr int REG = T + 2 * RM;                 // staged rows and columns
    static constexpr int ST = (REG + 3) & ~3;              // LDS row stride
    static constexpr int LR = (REG - 2) / S + 1 + 4;        // LR rows under them, with the taps on both sides
    static constexpr int ES = (LR + 3) & ~3;               // stride of the staged LR error
    static constexpr int SH = 2 * REG * T > LR * ES ? 2 * REG * T : LR * ES;   // the sums, or the LR error
};

template <int T, int RM, int S, bool TERMS>
__device__ __forceinline__ void bp_tile(const float* __restrict__ I, const float* __restrict__ e, int H, int W, int h,
                                        int w, int R, float sigma_s, float inv2sr2, float* __restrict__ out, int Y0,
                                        int X0) {
    using G = BpGeom<T, RM, S>;
    constexpr int s = S;
    constexpr int REG = G::REG, ST = G::ST, LR = G::LR, ES = G::ES, NT = 256;
    constexpr int TAPS = 2 * RM + 1;
    __shared__ __align__(16) float sI[REG * ST];
    __shared__ __align__(16) float xU[LR * ST];       // the LR error upsampled along x
    __shared__ __align__(16) float sH[G::SH];         // the horizontal sums; first the staged LR error [LR][ES]
    __shared__ float sg[TAPS];
    __shared__ __align__(16) float snx[T], sny[T];    // sums of the in-image taps of the tile's columns and rows
    float* sHE = sH;
    float* sHB = sH + REG * T;
    float* eL = sH;
    const int reg = T + 2 * R;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    // the staged region's in-image HR rows [ya, yb] and columns [xa, xb]
    const int ya = max(0, Y0 - R), yb = min(H - 1, Y0 - R + reg - 1);
    const int xa = max(0, X0 - R), xb = min(W - 1, X0 - R + reg - 1);
    const int la = ya / s - 1, lc = xa / s - 1;          // first staged LR row / column
    const int nlr = yb / s + 2 - la + 1, nlc = xb / s + 2 - lc + 1;
    {
        float v[(REG * ST + NT - 1) / NT];
#pragma unroll
        for (int u = 0; u < (REG * ST + NT - 1) / NT; ++u) {
            const int t = tid + NT * u, r = t / ST, c = t - r * ST;
            const int Y = Y0 - R + r, X = X0 - R + c;
            v[u] = (r < reg && c < reg && Y >= 0 && Y < H && X >= 0 && X < W) ? I[(int64_t)Y * W + X] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < (LR * ES + NT - 1) / NT; ++u) {
            const int t = tid + NT * u, r = t / ES, c = t - r * ES;
            if (r < nlr && c < nlc)
                eL[t] = e[(int64_t)clampi(la + r, 0, h - 1) * w + clampi(lc + c, 0, w - 1)];
        }
#pragma unroll
        for (int u = 0; u < (REG * ST + NT - 1) / NT; ++u)
            if (tid + NT * u < REG * ST) sI[tid + NT * u] = v[u];
    }
    if (tid < 2 * R + 1) {
        const float d = (float)(tid - R);
        sg[tid] = expf(-(d * d) / (2.0f * sigma_s * sigma_s));
    }
    __syncthreads();
    // along x: a lane per column (zero outside the image), a wave per LR row
    if (lane < ST) {
        const int X = X0 - R + lane;
        const bool in = lane < reg && X >= xa && X <= xb;
        const int j0 = in ? X / s : 0;
        const float tx = (float)(X - j0 * s) / (float)s;
        float wx[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) wx[b] = keys_w(tx - (float)(b - 1));
        const float* col = eL + (in ? j0 - 1 - lc : 0);
        for (int r = wv; r < nlr; r += 4) {
            float v = 0.0f;
            if (in) {
#pragma unroll
                for (int b = 0; b < 4; ++b) v = fmaf(wx[b], col[r * ES + b], v);
            }
            xU[r * ST + lane] = v;
        }
    } else {
        // the lanes past the columns
        const int t = wv * (64 - ST) + lane - ST;
        static_assert(4 * (64 - ST) >= 2 * T, "a thread for each sum");
        if (t < 2 * T) {
            const int x0 = t < T ? X0 + t : Y0 + t - T, n = t < T ? W : H;
            float gn = 0.0f;
#pragma unroll
            for (int u = 0; u < TAPS; ++u) {
                const int x = x0 + u - R;
                gn += u <= 2 * R && x >= 0 && x < n ? sg[u] : 0.0f;
            }
            (t < T ? snx[t] : sny[t - T]) = gn;
        }
    }
    __syncthreads();
    const int nt = 2 * R + 1;
    // along y in registers, then the horizontal sums (taps d = -R .. R in order)
    for (int t = tid; t < reg * (T / kBpOut); t += NT) {
        const int r = t / (T / kBpOut), c = kBpOut * (t - r * (T / kBpOut));
        constexpr int NV = (TAPS - 1 + kBpOut + 3) & ~3;   // columns past the last tap are read and not used
        float ev[NV];
#pragma unroll
        for (int q = 0; q < NV; ++q) ev[q] = 0.0f;
        const int Y = Y0 - R + r;
        if (Y >= ya && Y <= yb) {
            const int i0 = Y / s;
            const float ty = (float)(Y - i0 * s) / (float)s;
            const float* x0 = xU + (i0 - 1 - la) * ST + c;
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const float wy = keys_w(ty - (float)(a - 1));
#pragma unroll
                for (int q = 0; q < NV / 4; ++q) {
                    const float4 x = *reinterpret_cast<const float4*>(x0 + a * ST + 4 * q);
                    ev[4 * q] = fmaf(wy, x.x, ev[4 * q]);
                    ev[4 * q + 1] = fmaf(wy, x.y, ev[4 * q + 1]);
                    ev[4 * q + 2] = fmaf(wy, x.z, ev[4 * q + 2]);
                    ev[4 * q + 3] = fmaf(wy, x.w, ev[4 * q + 3]);
                }
            }
        }
        float ge[kBpOut], bs[kBpOut];
#pragma unroll
        for (int j = 0; j < kBpOut; ++j) ge[j] = bs[j] = 0.0f;
#pragma unroll
        for (int u = 0; u < TAPS; ++u) {
            if (u >= nt) break;
            const float g = sg[u];
#pragma unroll
            for (int j = 0; j < kBpOut; ++j) ge[j] = fmaf(g, ev[j + u], ge[j]);
        }
        float iv[NV];
#pragma unroll
        for (int q = 0; q < NV / 4; ++q) {
            const float4 y = *reinterpret_cast<const float4*>(&sI[r * ST + c + 4 * q]);
            iv[4 * q] = y.x, iv[4 * q + 1] = y.y, iv[4 * q + 2] = y.z, iv[4 * q + 3] = y.w;
        }
#pragma unroll
        for (int u = 0; u < TAPS; ++u) {
            if (u >= nt) break;
#pragma unroll
            for (int j = 0; j < kBpOut; ++j) bs[j] += iv[j + u];
        }
#pragma unroll
        for (int j = 0; j < kBpOut; ++j) {
            const float gn = snx[c + j];
            ge[j] = gn > 0.0f ? ge[j] / gn : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < kBpOut / 4; ++q) {
            *reinterpret_cast<float4*>(&sHE[r * T + c + 4 * q]) =
                make_float4(ge[4 * q], ge[4 * q + 1], ge[4 * q + 2], ge[4 * q + 3]);
            *reinterpret_cast<float4*>(&sHB[r * T + c + 4 * q]) =
                make_float4(bs[4 * q], bs[4 * q + 1], bs[4 * q + 2], bs[4 * q + 3]);
        }
    }
    __syncthreads();
    // vertical sums and the outputs
    constexpr int NO = T * T / NT;
    const int c = tid % T, r = NO * (tid / T);
    const int X = X0 + c;
    float ge[NO], bs[NO];
#pragma unroll
    for (int j = 0; j < NO; ++j) ge[j] = bs[j] = 0.0f;
    {
        float hv[TAPS - 1 + NO], bv[TAPS - 1 + NO];
        // rows past the last tap are read (inside the sums) and not used
#pragma unroll
        for (int q = 0; q < TAPS - 1 + NO; ++q) {
            hv[q] = sHE[(r + q) * T + c];
            bv[q] = sHB[(r + q) * T + c];
        }
#pragma unroll
        for (int u = 0; u < TAPS; ++u) {
            if (u >= nt) break;
            const float g = sg[u];
#pragma unroll
            for (int j = 0; j < NO; ++j) {
                ge[j] = fmaf(g, hv[j + u], ge[j]);
                bs[j] += bv[j + u];
            }
        }
    }
    if (X >= W) return;
    const int nx = min(W - 1, X + R) - max(0, X - R) + 1;
#pragma unroll
    for (int j = 0; j < NO; ++j) {
        const int Y = Y0 + r + j;
        if (Y >= H) break;
        const float gn = sny[r + j];
        const int ny = min(H - 1, Y + R) - max(0, Y - R) + 1;
        const float Ixy = sI[(r + j + R) * ST + c + R];
        const float mu = bs[j] / (float)(ny * nx);
        const float dd = Ixy - mu;
        const float rw = expf(-dd * dd * inv2sr2);
        if (TERMS) {
            const int64_t hw = (int64_t)H * W, o = (int64_t)Y * W + X;
            out[o] = ge[j] / gn;
            out[hw + o] = rw;
            out[2 * hw + o] = dd;
        } else {
            out[(int64_t)Y * W + X] = fmaf(rw, ge[j] / gn, Ixy);
        }
    }
}

template <int T, int RM, int S, bool TERMS>
__global__ __launch_bounds__(256) void k_bp_update(const float* __restrict__ I, const float* __restrict__ e,
                                                   int H, int W, int h, int w, int R, float sigma_s, float inv2sr2,
                                                   float* __restrict__ out) {
    bp_tile<T, RM, S, TERMS>(I, e, H, W, h, w, R, sigma_s, inv2sr2, out, blockIdx.y * T, blockIdx.x * T);
}

int bp_tiles(int H, int W, int tile) { return ((H + tile - 1) / tile) * ((W + tile - 1) / tile); }

// Batched update: a workgroup per (image, tile) item of the concatenated tile
// lists. (Persistent workgroups that looped over items held loop-invariant
// values in registers, 120 against 72, four waves a SIMD.)
template <int T, int RM, int S>
__global__ __launch_bounds__(256) void k_b_bp_update(const BatchImage* __restrict__ im, int n, int R, float sigma_s,
                                                     float inv2sr2, const float* __restrict__ e, int parity) {
    const int64_t it = blockIdx.x;
    const BatchImage& b = im[batch_image_of<&BatchImage::tile_off>(im, n, it)];
    const int H = S * b.h, W = S * b.w;
    const int tx = (W + T - 1) / T;
    const int local = (int)(it - b.tile_off);
    bp_tile<T, RM, S, false>(parity ? b.scr : b.out, e + b.lr_off, H, W, b.h, b.w, R, sigma_s, inv2sr2,
                             parity ? b.out : b.scr, (local / tx) * T, (local % tx) * T);
}

// K<T, RM, S, ...> for a radius (at most kBpSmallR, or up to kBpMaxR) and a zoom factor
template <int T, int RM, int S> constexpr auto kUpdate = k_bp_update<T, RM, S, false>;
template <int T, int RM, int S> constexpr auto kTerms = k_bp_update<T, RM, S, true>;
template <int T, int RM, int S> constexpr auto kBatch = k_b_bp_update<T, RM, S>;
#define ZH_BP_ZOOM(K, T, RM, s) \
    ((s) == 1 ? K<T, RM, 1> : (s) == 2 ? K<T, RM, 2> : (s) == 3 ? K<T, RM, 3> : K<T, RM, 4>)
#define ZH_BP_PICK(K, T, R, s) ((R) <= kBpSmallR ? ZH_BP_ZOOM(K, T, kBpSmallR, s) : ZH_BP_ZOOM(K, T, kBpMaxR, s))

static float inv_2sr2(float sigma_r) {
    return sigma_r > 0.0f && std::isfinite(sigma_r) ? 1.0f / (2.0f * sigma_r * sigma_r) : 0.0f;
}

template <bool TERMS>
static hipError_t bp_launch(const float* I, const float* e, int H, int W, int h, int w, int scale, float sigma_s,
                            float sigma_r, float* out, hipStream_t st) {
    const int R = (int)std::ceil(3.0 * (double)sigma_s);
    if (R > kBpMaxR || R < 0 || scale < 1 || scale > kMaxScale) return hipErrorInvalidValue;
    // few tiles of 32 leave compute units idle: 16 there (the same bits; us an
    // iteration with 32 and 16: 128^2 9.0 and 6.9, 502x526 10.1 and 9.3,
    // 844x1228 15.5 and 21, 2048^2 37 and 67)
    const int T = bp_tiles(H, W, 32) < 512 ? 16 : 32;
    const dim3 grid((W + T - 1) / T, (H + T - 1) / T);
    auto k = T == 16 ? (TERMS ? ZH_BP_PICK(kTerms, 16, R, scale) : ZH_BP_PICK(kUpdate, 16, R, scale))
                     : (TERMS ? ZH_BP_PICK(kTerms, 32, R, scale) : ZH_BP_PICK(kUpdate, 32, R, scale));
    hipLaunchKernelGGL(k, grid, dim3(256), 0, st, I, e, H, W, h, w, R, sigma_s, inv_2sr2(sigma_r), out);
    return hipGetLastError();
}

hipError_t launch_bp_update(const float* I, const float* e, int H, int W, int h, int w, int scale,
                            float sigma_s, float sigma_r, float* out, hipStream_t st) {
    return bp_launch<false>(I, e, H, W, h, w, scale, sigma_s, sigma_r, out, st);
}

hipError_t launch_bp_terms(const float* I, const float* e, int H, int W, int h, int w, int scale,
                           float sigma_s, float sigma_r, float* FSa, hipStream_t st) {
    return bp_launch<true>(I, e, H, W, h, w, scale, sigma_s, sigma_r, FSa, st);
}

hipError_t launch_b_bp_update(const BatchImage* im, int n, int64_t n_tiles, int tile, int per_cu, int scale,
                              float sigma_s, float sigma_r, const float* e, int parity, hipStream_t st) {
    const int R = (int)std::ceil(3.0 * (double)sigma_s);
    if (R > kBpMaxR || R < 0 || (tile != 16 && tile != 32) || per_cu < 1 || scale < 1 || scale > kMaxScale ||
        n_tiles > 0x7FFFFFFF)
        return hipErrorInvalidValue;
    if (n_tiles == 0) return hipSuccess;
    auto k = tile == 16 ? ZH_BP_PICK(kBatch, 16, R, scale) : ZH_BP_PICK(kBatch, 32, R, scale);
    // at most per_cu workgroups on a compute unit: its 160 KB of LDS shared
    // out (8: what registers and LDS allow)
    size_t lds = 0;
    if (per_cu < 8) {
        hipFuncAttributes fa;
        const hipError_t ea = hipFuncGetAttributes(&fa, reinterpret_cast<const void*>(k));
        if (ea != hipSuccess) return ea;
        const size_t share = std::min<size_t>((size_t)(160 << 10) / (per_cu + 1) + 1024, 60 << 10);
        if (share > fa.sharedSizeBytes) lds = share - fa.sharedSizeBytes;
    }
    hipLaunchKernelGGL(k, dim3((unsigned)n_tiles), dim3(256), lds, st, im, n, R, sigma_s, inv_2sr2(sigma_r), e, parity);
    return hipGetLastError();
}

}  // namespace zh
