// Image-side kernels: degradation (Section 2.1: Gaussian blur then
// decimation), the gradient maps and patch features of Section 4.1, cutting
// of the LR/HR training pairs, and bicubic upsampling.
//
// The degradation and the features are evaluated in FP64 in a fixed order
// and rounded once to fp32, so the stored LR images and features are
// reproducible bit for bit by any implementation that follows the same
// order (the file is compiled without multiply-add contraction).
#include "zh_internal.h"

namespace zh {

// (g * hr)[s i, s j] in FP64: horizontal pass along each needed row, then the
// vertical combination, both accumulating taps in ascending offset order.
__device__ __forceinline__ double blur_at(const float* __restrict__ hr, int H, int W, int y, int x,
                                          const Taps& t) {
    double acc = 0.0;
    for (int a = -t.R; a <= t.R; ++a) {
        const float* row = hr + (int64_t)clampi(y + a, 0, H - 1) * W;
        double hrow = 0.0;
        for (int b = -t.R; b <= t.R; ++b) hrow = hrow + t.g[b + t.R] * (double)row[clampi(x + b, 0, W - 1)];
        acc = acc + t.g[a + t.R] * hrow;
    }
    return acc;
}

__global__ void k_degrade(const float* __restrict__ hr, int n_img, int H, int W, int scale, Taps t,
                          float* __restrict__ lr) {
    const int h = (H + scale - 1) / scale, w = (W + scale - 1) / scale;
    const int64_t total = (int64_t)n_img * h * w;
    for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * blockDim.x) {
        const int64_t im = idx / ((int64_t)h * w);
        const int r = (int)(idx % ((int64_t)h * w));
        const int i = r / w, j = r % w;
        lr[idx] = (float)blur_at(hr + im * (int64_t)H * W, H, W, scale * i, scale * j, t);
    }
}

// LR error of back-projection (blur of sigma 1: kDrR = 3 taps a side) by LR
// tiles of kDrI x kDrJ, image sides S h x S w: the HR rows and columns under a
// tile (clamped indices: replicate border) are staged in LDS, the horizontal
// FP64 sums are formed once per (HR row, LR column) and shared by the LR rows
// that use them, then the vertical sums; each value is the blur_at sum to the
// bit (same products, same order). copy (nullable) receives the HR image, each
// tile its own pixels. Bound: latency on small images, FP64 issue on large ones
// (14 products and sums an HR row and LR column). An iteration's error before
// (zoom factor and radius at run time) and now, the first of three with the
// copy: 128^2 6.1 -> 4.6 us, 502x526 6.2 -> 4.8, 2048^2 16.6 -> 11.4, 844x1228
// x4 11.5 -> 5.6; a copy of its own took 6.6 us at 2048^2.
constexpr int kDrI = 8, kDrJ = 32, kDrR = 3;
template <int S>
__device__ __forceinline__ void degrade_tile(const float* __restrict__ hr, int h, int w, const Taps& t,
                                             const float* __restrict__ lr_ref, float* __restrict__ e, int i0, int j0,
                                             float* __restrict__ copy) {
    constexpr int R = kDrR, NY = S * (kDrI - 1) + 2 * R + 1, NX = S * (kDrJ - 1) + 2 * R + 1, NT = 256;
    __shared__ double hrow[NY * kDrJ];
    __shared__ float sh[NY * NX];
    const int H = S * h, W = S * w;
    const int y0 = S * i0 - R, x0 = S * j0 - R;
    const int ii = threadIdx.x / kDrJ, jj = threadIdx.x % kDrJ;
    const int i = i0 + ii, j = j0 + jj;
    const bool in = i < h && j < w;
    const float ref = in ? lr_ref[(int64_t)i * w + j] : 0.0f;
    {
        constexpr int U = (NY * NX + NT - 1) / NT;
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = threadIdx.x + NT * u, r = q / NX, c = q - r * NX;
            v[u] = hr[(int64_t)clampi(y0 + (r < NY ? r : 0), 0, H - 1) * W + clampi(x0 + c, 0, W - 1)];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = threadIdx.x + NT * u;
            if (q < NY * NX) sh[q] = v[u];
        }
        if (copy) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int q = threadIdx.x + NT * u, r = q / NX, c = q - r * NX;
                const int Y = y0 + r, X = x0 + c;
                if (r >= R && r < R + S * kDrI && c >= R && c < R + S * kDrJ && r < NY && Y < H && X < W)
                    copy[(int64_t)Y * W + X] = v[u];
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < (NY * kDrJ + NT - 1) / NT; ++u) {
        const int q = threadIdx.x + NT * u;
        if (q >= NY * kDrJ) break;
        const float* row = sh + (q / kDrJ) * NX + S * (q % kDrJ);
        double v = 0.0;
#pragma unroll
        for (int b = 0; b <= 2 * R; ++b) v = v + t.g[b] * (double)row[b];
        hrow[q] = v;
    }
    __syncthreads();
    if (!in) return;
    double acc = 0.0;
#pragma unroll
    for (int a = 0; a <= 2 * R; ++a) acc = acc + t.g[a] * hrow[(S * ii + a) * kDrJ + jj];
    e[(int64_t)i * w + j] = (float)((double)ref - acc);
}
static_assert(kDrI * kDrJ == 256, "a thread for each LR pixel of a tile");

template <int S>
__global__ __launch_bounds__(256) void k_degrade_residual(const float* __restrict__ hr, int h, int w, Taps t,
                                                          const float* __restrict__ lr_ref, float* __restrict__ e,
                                                          float* __restrict__ copy) {
    degrade_tile<S>(hr, h, w, t, lr_ref, e, blockIdx.y * kDrI, blockIdx.x * kDrJ, copy);
}

// Batched: workgroup b takes tile b of the concatenated tile lists of the
// images (the current estimate in out for parity 0, scr for parity 1; copy:
// it is in out and copied to scr); image b's error at e + lr_off.
template <int S>
__global__ __launch_bounds__(256) void k_b_degrade_residual(const BatchImage* __restrict__ im, int n, Taps t, int parity,
                                                            int copy, float* __restrict__ e) {
    const int64_t tile = blockIdx.x;
    const BatchImage& b = im[batch_image_of<&BatchImage::dtile_off>(im, n, tile)];
    const int local = (int)(tile - b.dtile_off);
    const int tx = (b.w + kDrJ - 1) / kDrJ;
    degrade_tile<S>(parity ? b.scr : b.out, b.h, b.w, t, b.lr, e + b.lr_off, (local / tx) * kDrI, (local % tx) * kDrJ,
                    copy ? b.scr : nullptr);
}

int64_t degrade_tiles(int h, int w) { return (int64_t)((h + kDrI - 1) / kDrI) * ((w + kDrJ - 1) / kDrJ); }

// Four gradient maps per image, fp32 [n_img, 4, h, w]:
//   dx = I(c+1) - I(c-1), dy likewise along rows,
//   dxx = (2 I(c) - I(c-2)) - I(c+2), dyy likewise; replicate border.
__device__ __forceinline__ void gradient_maps_at(const float* __restrict__ I, int h, int w, int rc,
                                                 float* __restrict__ M) {
    const int r = rc / w, c = rc % w;
    auto at = [&](int rr, int cc) -> double {
        return (double)I[(int64_t)clampi(rr, 0, h - 1) * w + clampi(cc, 0, w - 1)];
    };
    const double x0 = at(r, c);
    const double dx = at(r, c + 1) - at(r, c - 1);
    const double dy = at(r + 1, c) - at(r - 1, c);
    const double dxx = (2.0 * x0 - at(r, c - 2)) - at(r, c + 2);
    const double dyy = (2.0 * x0 - at(r - 2, c)) - at(r + 2, c);
    const int64_t plane = (int64_t)h * w;
    M[rc] = (float)dx;
    M[plane + rc] = (float)dy;
    M[2 * plane + rc] = (float)dxx;
    M[3 * plane + rc] = (float)dyy;
}

__global__ void k_gradient_maps(const float* __restrict__ lr, int n_img, int h, int w,
                                float* __restrict__ maps) {
    const int64_t total = (int64_t)n_img * h * w;
    for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * blockDim.x) {
        const int64_t im = idx / ((int64_t)h * w);
        const int rc = (int)(idx % ((int64_t)h * w));
        gradient_maps_at(lr + im * (int64_t)h * w, h, w, rc, maps + im * 4 * (int64_t)h * w);
    }
}

// Patch mean: FP64 sum over the 25 pixels in row-major order, then / 25.
__device__ __forceinline__ double patch_mean(const float* __restrict__ I, int w, int i, int j) {
    double s = 0.0;
    for (int a = 0; a < kPatch; ++a)
        for (int b = 0; b < kPatch; ++b) s = s + (double)I[(int64_t)(i + a) * w + j + b];
    return s / (double)(kPatch * kPatch);
}

// One workgroup per segment of up to 64 consecutive patches of one patch row:
// the LR rows under the segment (two more on every side for the gradients,
// clamped indices: replicate border) are staged in LDS, the first threads form
// the segment's patch means (the sum of patch_mean), all of them the gradient
// maps under it (the values of gradient_maps_at) in LDS, then the threads write
// the segment's features in memory order (coalesced): the map values (gradient
// mode) or the pixels minus the FP64 mean, rounded to fp32. copy (nullable)
// receives the LR image, each pixel from the segment whose first patch row and
// columns hold it; counters (nullable) are cleared by the first segment. Bound:
// the feature rows' writes (1024^2 at D = 100: 416 MB). Features, maps in a
// kernel of their own, copy and clearing, then this: 1024^2 119 -> 93 us,
// 251x263 24 -> 9.9.
template <int MODE>
__device__ __forceinline__ void query_features_seg(const float* __restrict__ lr, int h, int w, int i, int j0,
                                                   float* __restrict__ feat, double* __restrict__ mu,
                                                   float* __restrict__ copy) {
    constexpr int D = MODE == 0 ? 25 : 100;
    constexpr int SW = kFeatSeg + kPatch - 1;     // columns under a segment of patches
    constexpr int B = MODE == 0 ? 0 : 2;          // border of the staged LR rows
    constexpr int SR = kPatch + 2 * B, SC = SW + 2 * B;
    __shared__ double smu[kFeatSeg];
    __shared__ float slr[SR * SC];
    __shared__ float stile[MODE == 0 ? 1 : 4 * kPatch * SW];   // the 5 rows of each gradient map
    const int nj = w - kPatch + 1;
    const int np = nj - j0 < kFeatSeg ? nj - j0 : kFeatSeg;
    const int64_t q0 = (int64_t)i * nj + j0;
    const int t = threadIdx.x;
    const int ncols = np + kPatch - 1;
    for (int e = t; e < SR * SC; e += 256) {
        const int a = e / SC, c = e - a * SC;
        if (c < ncols + 2 * B) slr[e] = lr[(int64_t)clampi(i - B + a, 0, h - 1) * w + clampi(j0 - B + c, 0, w - 1)];
    }
    __syncthreads();
    if (copy) {
        const bool lastc = j0 + np == nj, lastr = i + kPatch == h;
        const int cols = lastc ? ncols : np, rows = lastr ? kPatch : 1;
        for (int e = t; e < rows * cols; e += 256) {
            const int a = e / cols, c = e - a * cols;
            copy[(int64_t)(i + a) * w + j0 + c] = slr[(B + a) * SC + B + c];
        }
    }
    if (t < np) {
        double s = 0.0;
        for (int a = 0; a < kPatch; ++a)
            for (int b = 0; b < kPatch; ++b) s = s + (double)slr[(B + a) * SC + B + t + b];
        const double m = s / (double)(kPatch * kPatch);
        smu[t] = m;
        mu[q0 + t] = m;
    }
    if (MODE == 1) {
        for (int e = t; e < kPatch * SW; e += 256) {
            const int a = e / SW, c = e - a * SW;
            const float* p = slr + (B + a) * SC + B + c;
            const double x0 = (double)p[0];
            stile[e] = (float)((double)p[1] - (double)p[-1]);
            stile[kPatch * SW + e] = (float)((double)p[SC] - (double)p[-SC]);
            stile[2 * kPatch * SW + e] = (float)((2.0 * x0 - (double)p[-2]) - (double)p[2]);
            stile[3 * kPatch * SW + e] = (float)((2.0 * x0 - (double)p[-2 * SC]) - (double)p[2 * SC]);
        }
    }
    __syncthreads();
    if (MODE == 0) {
#pragma unroll 5
        for (int l = t; l < np * D; l += 256) {
            const int p = l / D, e = l - p * D;
            const int a = e / kPatch, b = e - a * kPatch;
            feat[q0 * D + l] = (float)((double)slr[a * SC + p + b] - smu[p]);
        }
    } else {
        // 16-byte stores: D = 100 keeps a group of four inside one patch row
        float4* f4 = reinterpret_cast<float4*>(feat + q0 * D);
#pragma unroll 2
        for (int l4 = t; l4 < np * (D / 4); l4 += 256) {
            const int p = l4 / (D / 4), e0 = 4 * (l4 - p * (D / 4));
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int e = e0 + u;
                const int ch = e / 25, r = e - ch * 25, a = r / kPatch, b = r - a * kPatch;
                v[u] = stile[(ch * kPatch + a) * SW + p + b];
            }
            f4[l4] = make_float4(v[0], v[1], v[2], v[3]);
        }
    }
}

__device__ __forceinline__ void clear_counters_once(uint32_t* counters) {
    if (counters && blockIdx.x == 0 && threadIdx.x < kNumCounters) counters[threadIdx.x] = 0u;
}

template <int MODE>
__global__ __launch_bounds__(256) void k_query_features(const float* __restrict__ lr, int h, int w,
                                                        float* __restrict__ feat, double* __restrict__ mu,
                                                        float* __restrict__ copy, uint32_t* __restrict__ counters) {
    clear_counters_once(counters);
    const int nseg = (w - kPatch + 1 + kFeatSeg - 1) / kFeatSeg;
    const int i = blockIdx.x / nseg, j0 = (blockIdx.x - i * nseg) * kFeatSeg;
    query_features_seg<MODE>(lr, h, w, i, j0, feat, mu, copy);
}

// Batched: one workgroup per segment of every image (the image from the
// table's segment offsets), the single-image code on the image's arrays.
template <int MODE>
__global__ __launch_bounds__(256) void k_b_query_features(const BatchImage* __restrict__ im, int n,
                                                          float* __restrict__ feat, double* __restrict__ mu,
                                                          uint32_t* __restrict__ counters) {
    constexpr int D = MODE == 0 ? 25 : 100;
    clear_counters_once(counters);
    const BatchImage& b = im[batch_image_of<&BatchImage::fblk_off>(im, n, blockIdx.x)];
    const int64_t lb = blockIdx.x - b.fblk_off;
    const int nseg = (b.w - kPatch + 1 + kFeatSeg - 1) / kFeatSeg;
    const int i = (int)(lb / nseg), j0 = (int)(lb - (int64_t)i * nseg) * kFeatSeg;
    query_features_seg<MODE>(b.lr, b.h, b.w, i, j0, feat + b.q_off * D, mu + b.q_off, nullptr);
}

// Training pairs at positions (image, i, j): features, and the HR patch
// (5s x 5s at (s i, s j)) minus the mean of the LR patch, in FP64 rounded to
// fp32. A workgroup takes kCutPairs pairs: their patch means once, then their
// features and residuals in memory order. Bound: the writes (800 bytes a pair at
// D = 100, x2). 300k pairs: 0.29 -> 0.09 ms (a patch mean per element before).
constexpr int kCutPairs = 64;
template <int MODE>
__global__ __launch_bounds__(256) void k_dict_cut(const float* __restrict__ hr, const float* __restrict__ lr,
                                                  const float* __restrict__ maps, int H, int W, int scale,
                                                  const int32_t* __restrict__ pos, int64_t n, float* __restrict__ feat,
                                                  float* __restrict__ resid) {
    constexpr int D = MODE == 0 ? 25 : 100;
    __shared__ double smean[kCutPairs];
    __shared__ int64_t slr[kCutPairs], smap[kCutPairs], shr[kCutPairs];   // offsets of the patches' first pixels
    const int h = (H + scale - 1) / scale, w = (W + scale - 1) / scale;
    const int ps = kPatch * scale, ps2 = ps * ps;
    const int64_t p0 = block_id() * kCutPairs;
    if (p0 >= n) return;
    const int np = (int)(n - p0 < kCutPairs ? n - p0 : kCutPairs);
    if ((int)threadIdx.x < np) {
        const int64_t p = p0 + threadIdx.x;
        const int im = pos[3 * p], i = pos[3 * p + 1], j = pos[3 * p + 2];
        const int64_t o = (int64_t)im * h * w;
        slr[threadIdx.x] = o + (int64_t)i * w + j;
        smap[threadIdx.x] = 4 * o + (int64_t)i * w + j;
        shr[threadIdx.x] = (int64_t)im * H * W + (int64_t)(scale * i) * W + scale * j;
        smean[threadIdx.x] = patch_mean(lr + o, w, i, j);
    }
    __syncthreads();
    for (int l = threadIdx.x; l < np * D; l += 256) {
        const int p = l / D, e = l - p * D;
        float v;
        if (MODE == 0) {
            v = (float)((double)lr[slr[p] + (int64_t)(e / kPatch) * w + e % kPatch] - smean[p]);
        } else {
            const int ch = e / 25, r = e - ch * 25;
            v = maps[smap[p] + (int64_t)ch * h * w + (int64_t)(r / kPatch) * w + r % kPatch];
        }
        feat[p0 * D + l] = v;
    }
    for (int l = threadIdx.x; l < np * ps2; l += 256) {
        const int p = l / ps2, t = l - p * ps2, a = t / ps, b = t - a * ps;
        resid[p0 * ps2 + l] = (float)((double)hr[shr[p] + (int64_t)a * W + b] - smean[p]);
    }
}

// The library's own copies of the dictionary features, read once: fp32 rows,
// and the split storage (the high plane holds the upper 16 bits of each fp32
// value, a bf16 truncation, in rows of hi_stride(D) halfwords with zero padding,
// the low plane the lower 16 bits in rows of D).
__global__ void k_split_planes(const float* __restrict__ x, int64_t n, int D, uint16_t* __restrict__ hi,
                               uint16_t* __restrict__ lo, float* __restrict__ xf) {
    const int hs = hi_stride(D);
    const int64_t count = n * hs;
    for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < count;
         idx += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = idx / hs;
        const int c = (int)(idx - r * hs);
        uint32_t b = 0;
        if (c < D) {
            const float v = x[r * D + c];
            b = __float_as_uint(v);
            lo[r * D + c] = (uint16_t)(b & 0xFFFFu);
            xf[r * D + c] = v;
        }
        hi[idx] = (uint16_t)(b >> 16);
    }
}


__global__ void k_bicubic(const float* __restrict__ lr, int h, int w, int s, float* __restrict__ out) {
    const int H = s * h, W = s * w;
    const int64_t total = (int64_t)H * W;
    for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * blockDim.x)
        out[idx] = bicubic_at(lr, h, w, s, (int)(idx / W), (int)(idx % W));
}

// The LR image interpolated back to the HR grid (Section 2.1, the paired
// LR images of the training set have the HR images' size): bicubic with
// Keys' weights (a = -0.5) taken from the host table wt[r][tap] for the
// phase r = X mod s, taps floor - 1 .. floor + 2, replicate border; FP64,
// along x first (for each of the four rows), then along y, every sum started
// at 0 and taken in tap order; rounded once to fp32.
struct UpWeights {
    double w[kMaxScale * 2][4];
};
__global__ void k_upsample64(const float* __restrict__ lr, int h, int w, int s, UpWeights uw,
                             float* __restrict__ out) {
    const int H = s * h, W = s * w;
    const int64_t total = (int64_t)H * W;
    for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * blockDim.x) {
        const int Y = (int)(idx / W), X = (int)(idx % W);
        const int i0 = Y / s, j0 = X / s;
        const double* wy = uw.w[Y - i0 * s];
        const double* wx = uw.w[X - j0 * s];
        double acc = 0.0;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const float* row = lr + (int64_t)clampi(i0 - 1 + a, 0, h - 1) * w;
            double r = 0.0;
#pragma unroll
            for (int b = 0; b < 4; ++b) r = r + wx[b] * (double)row[clampi(j0 - 1 + b, 0, w - 1)];
            acc = acc + wy[a] * r;
        }
        out[idx] = (float)acc;
    }
}

static inline int grid_for(int64_t total, int block) {
    int64_t g = (total + block - 1) / block;
    if (g > 65536) g = 65536;
    return (int)(g < 1 ? 1 : g);
}

hipError_t launch_degrade(const float* hr, int n_img, int H, int W, int scale, const Taps& t,
                          float* lr, hipStream_t st) {
    const int64_t total = (int64_t)n_img * ((H + scale - 1) / scale) * ((W + scale - 1) / scale);
    hipLaunchKernelGGL(k_degrade, dim3(grid_for(total, 256)), dim3(256), 0, st, hr, n_img, H, W,
                       scale, t, lr);
    return hipGetLastError();
}

hipError_t launch_degrade_residual(const float* hr, int h, int w, int scale, const Taps& t, const float* lr_ref,
                                   float* e, float* copy, hipStream_t st) {
    if (h < 1 || w < 1 || t.R != kDrR || scale < 1 || scale > kMaxScale) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((w + kDrJ - 1) / kDrJ), (unsigned)((h + kDrI - 1) / kDrI));
    auto k = scale == 1 ? k_degrade_residual<1> : scale == 2 ? k_degrade_residual<2>
             : scale == 3 ? k_degrade_residual<3> : k_degrade_residual<4>;
    hipLaunchKernelGGL(k, grid, dim3(256), 0, st, hr, h, w, t, lr_ref, e, copy);
    return hipGetLastError();
}

hipError_t launch_gradient_maps(const float* lr, int n_img, int h, int w, float* maps,
                                hipStream_t st) {
    hipLaunchKernelGGL(k_gradient_maps, dim3(grid_for((int64_t)n_img * h * w, 256)), dim3(256), 0,
                       st, lr, n_img, h, w, maps);
    return hipGetLastError();
}

hipError_t launch_query_features(const float* lr, int h, int w, int mode, float* feat, double* mu, float* copy,
                                 uint32_t* counters, hipStream_t st) {
    const int ni = h - kPatch + 1, nj = w - kPatch + 1;
    if (ni < 1 || nj < 1) return hipErrorInvalidValue;
    const int64_t blocks = feature_segments(h, w);
    if (!one_row(blocks, 256)) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)blocks);
    if (mode == 0)
        hipLaunchKernelGGL(k_query_features<0>, grid, dim3(256), 0, st, lr, h, w, feat, mu, copy, counters);
    else
        hipLaunchKernelGGL(k_query_features<1>, grid, dim3(256), 0, st, lr, h, w, feat, mu, copy, counters);
    return hipGetLastError();
}

hipError_t launch_b_query_features(const BatchImage* im, int n, int64_t seg_total, int mode, float* feat, double* mu,
                                   uint32_t* counters, hipStream_t st) {
    if (seg_total < 1) return hipErrorInvalidValue;
    if (!one_row(seg_total, 256)) return hipErrorInvalidConfiguration;
    if (mode == 0)
        hipLaunchKernelGGL(k_b_query_features<0>, dim3((unsigned)seg_total), dim3(256), 0, st, im, n, feat, mu, counters);
    else
        hipLaunchKernelGGL(k_b_query_features<1>, dim3((unsigned)seg_total), dim3(256), 0, st, im, n, feat, mu, counters);
    return hipGetLastError();
}

hipError_t launch_b_degrade_residual(const BatchImage* im, int n, int64_t tiles, int scale, const Taps& t, int parity,
                                     bool copy, float* e, hipStream_t st) {
    if (tiles == 0) return hipSuccess;
    if (tiles > 0x7FFFFFFF || t.R != kDrR || scale < 1 || scale > kMaxScale) return hipErrorInvalidValue;
    auto k = scale == 1 ? k_b_degrade_residual<1> : scale == 2 ? k_b_degrade_residual<2>
             : scale == 3 ? k_b_degrade_residual<3> : k_b_degrade_residual<4>;
    hipLaunchKernelGGL(k, dim3((unsigned)tiles), dim3(256), 0, st, im, n, t, parity, copy ? 1 : 0, e);
    return hipGetLastError();
}

// flag[0] = 1 when any training position (image, i, j) lies outside
// [0, n_img) x [0, imax] x [0, jmax]; flag is cleared by the caller
__global__ __launch_bounds__(256) void k_check_positions(const int32_t* __restrict__ pos, int64_t n, int n_img,
                                                         int imax, int jmax, uint32_t* __restrict__ flag) {
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x) {
        const int im = pos[3 * r], i = pos[3 * r + 1], j = pos[3 * r + 2];
        if (im < 0 || im >= n_img || i < 0 || i > imax || j < 0 || j > jmax) flag[0] = 1u;
    }
}

hipError_t launch_check_positions(const int32_t* pos, int64_t n, int n_img, int imax, int jmax, uint32_t* flag,
                                  hipStream_t st) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_check_positions, dim3(grid_for(n, 256)), dim3(256), 0, st, pos, n, n_img, imax, jmax, flag);
    return hipGetLastError();
}

hipError_t launch_dict_cut(const float* hr, const float* lr, const float* maps, int H, int W,
                           int scale, const int32_t* pos, int64_t n, int mode, float* feat,
                           float* resid, hipStream_t st) {
    const dim3 grid = grid_rows((n + kCutPairs - 1) / kCutPairs);
    if (mode == 0)
        hipLaunchKernelGGL(k_dict_cut<0>, grid, dim3(256), 0, st, hr, lr, maps, H, W, scale, pos, n, feat, resid);
    else
        hipLaunchKernelGGL(k_dict_cut<1>, grid, dim3(256), 0, st, hr, lr, maps, H, W, scale, pos, n, feat, resid);
    return hipGetLastError();
}

hipError_t launch_split_planes(const float* x, int64_t n, int D, uint16_t* hi, uint16_t* lo, float* xf,
                               hipStream_t st) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_split_planes, dim3(grid_for(n * hi_stride(D), 256)), dim3(256), 0, st, x, n, D, hi, lo, xf);
    return hipGetLastError();
}


hipError_t launch_upsample64(const float* lr, int h, int w, int scale, const double* wt, float* out, hipStream_t st) {
    if (scale < 1 || scale > 2 * kMaxScale) return hipErrorInvalidValue;
    UpWeights uw{};
    for (int r = 0; r < scale; ++r)
        for (int a = 0; a < 4; ++a) uw.w[r][a] = wt[4 * r + a];
    hipLaunchKernelGGL(k_upsample64, dim3(grid_for((int64_t)scale * h * scale * w, 256)), dim3(256), 0, st, lr, h, w,
                       scale, uw, out);
    return hipGetLastError();
}

hipError_t launch_bicubic(const float* lr, int h, int w, int scale, float* out, hipStream_t st) {
    hipLaunchKernelGGL(k_bicubic, dim3(grid_for((int64_t)scale * h * scale * w, 256)), dim3(256),
                       0, st, lr, h, w, scale, out);
    return hipGetLastError();
}

}  // namespace zh
