// Dictionary-construction tools, off the per-image path.
//
// Training crops (Section 5, training data generation): every pixel of a
// training image weighs its first-order gradient (taps [-1, 0, 1] along each
// axis, replicate border), |dx| + |dy| in FP64 from the fp32 pixels,
// quantised to q = floor(g 2^20) (saturated at 2^32 - 1, also for non-finite
// g), so the cumulative distribution is an exact integer sum in any order.
// A 64-bit draw x picks the first pixel (row-major) whose inclusive
// cumulative weight exceeds x mod T (T the image's total; x mod (H W) when
// T = 0); the crop of side S around it has its top-left corner at the centre
// minus S / 2, clamped inside the image.
//
// Hashing quality (Section 4.1, determining r): the entropy in bits of each
// table's bucket occupancy, -sum_b p_b log2 p_b, p_b = (rows in bucket b) / N,
// read from the bin directory.
#include <cmath>

#include "zh_internal.h"

namespace zh {

constexpr int kCdfBlock = 1024;   // pixels per block of cumulative weights
constexpr int kCdfSub = kCdfBlock / 64;   // sub-blocks of 64 pixels per block

__device__ inline unsigned long long wave_sum_u64(unsigned long long v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

__device__ inline unsigned long long wave_incl_scan_u64(unsigned long long v) {
    const int lane = __lane_id();
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long t = __shfl_up(v, o);
        if (lane >= o) v += t;
    }
    return v;
}

__device__ inline uint32_t grad_weight(const float* __restrict__ img, int H, int W, int r, int c) {
    const double dx = (double)img[(int64_t)r * W + min(c + 1, W - 1)] - (double)img[(int64_t)r * W + max(c - 1, 0)];
    const double dy = (double)img[(int64_t)min(r + 1, H - 1) * W + c] - (double)img[(int64_t)max(r - 1, 0) * W + c];
    const double s = (fabs(dx) + fabs(dy)) * 1048576.0;
    return s < 4294967295.0 ? (uint32_t)floor(s) : 0xFFFFFFFFu;
}

// Sum of the weights of block blockIdx.x of image blockIdx.y (bsum) and of
// each of its 16 sub-blocks of 64 pixels (ssum). The weights themselves are
// not stored: the sampler recomputes the 64 of the sub-block it lands in.
__global__ __launch_bounds__(256) void k_cdf_weights(const float* __restrict__ imgs, int H, int W, int nb,
                                                     unsigned long long* __restrict__ bsum,
                                                     unsigned long long* __restrict__ ssum) {
    __shared__ unsigned long long ws[4];
    const int HW = H * W;
    const float* img = imgs + (int64_t)blockIdx.y * HW;
    const int p0 = blockIdx.x * kCdfBlock;
    unsigned long long acc = 0;
    unsigned long long* sub = ssum + ((int64_t)blockIdx.y * nb + blockIdx.x) * kCdfSub;
#pragma unroll
    for (int u = 0; u < kCdfBlock / 256; ++u) {
        const int p = p0 + (int)threadIdx.x + 256 * u;
        unsigned long long v = 0;
        if (p < HW) {
            const int r = p / W;
            v = grad_weight(img, H, W, r, p - r * W);
        }
        // the wave's 64 lanes hold one sub-block (pixels 256 u + 64 w ..)
        v = wave_sum_u64(v);
        if (__lane_id() == 0) sub[4 * u + (threadIdx.x >> 6)] = v;
        acc += v;
    }
    if (__lane_id() == 0) ws[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) bsum[(int64_t)blockIdx.y * nb + blockIdx.x] = ws[0] + ws[1] + ws[2] + ws[3];
}

// Exclusive prefix of the block sums of image blockIdx.x: bpre[0 .. nb], the
// last entry the image's total. One workgroup per image, 256 sums a pass.
__global__ __launch_bounds__(256) void k_cdf_scan(const unsigned long long* __restrict__ bsum, int nb,
                                                  unsigned long long* __restrict__ bpre) {
    __shared__ unsigned long long wt[4];
    const unsigned long long* in = bsum + (int64_t)blockIdx.x * nb;
    unsigned long long* out = bpre + (int64_t)blockIdx.x * (nb + 1);
    unsigned long long carry = 0;
    for (int b0 = 0; b0 < nb; b0 += 256) {
        const int b = b0 + threadIdx.x;
        const unsigned long long v = b < nb ? in[b] : 0ull;
        const unsigned long long incl = wave_incl_scan_u64(v);
        if (__lane_id() == 63) wt[threadIdx.x >> 6] = incl;
        __syncthreads();
        unsigned long long before = carry;
        for (int w = 0; w < (int)(threadIdx.x >> 6); ++w) before += wt[w];
        if (b < nb) out[b] = before + incl - v;
        carry += wt[0] + wt[1] + wt[2] + wt[3];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[nb] = carry;
}

// One wave per draw: the centre pixel, then the clamped crop corner.
__global__ __launch_bounds__(256) void k_cdf_sample(const float* __restrict__ imgs,
                                                    const unsigned long long* __restrict__ bpre,
                                                    const unsigned long long* __restrict__ ssum, int H, int W, int nb,
                                                    const unsigned long long* __restrict__ draws, int64_t n_draws,
                                                    int m, int side, int32_t* __restrict__ corners) {
    const int lane = __lane_id();
    const int64_t d = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (d >= n_draws) return;
    const int64_t img = d / m;
    const int HW = H * W;
    const unsigned long long* pre = bpre + img * (nb + 1);
    const unsigned long long T = pre[nb], x = draws[d];
    int64_t centre = -1;
    if (T == 0) {
        centre = (int64_t)(x % (unsigned long long)HW);
    } else {
        const unsigned long long t = x % T;
        // last block whose exclusive prefix is <= t (pre[0] = 0)
        int lo = 0, hi = nb - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (pre[mid] <= t) lo = mid;
            else hi = mid - 1;
        }
        unsigned long long tl = t - pre[lo];
        // the sub-block of 64 pixels holding tl, then the pixel inside it
        const unsigned long long sv = lane < kCdfSub ? ssum[(img * nb + lo) * kCdfSub + lane] : 0ull;
        const unsigned long long sincl = wave_incl_scan_u64(sv);
        const uint64_t shit = __ballot(sincl > tl);
        const int sb = shit ? __builtin_ctzll(shit) : kCdfSub - 1;
        tl -= __shfl(sincl - sv, sb);
        const int p = lo * kCdfBlock + sb * 64 + lane;
        const float* im = imgs + img * HW;
        unsigned long long q = 0;
        if (p < HW) {
            const int r = p / W;
            q = grad_weight(im, H, W, r, p - r * W);
        }
        const unsigned long long incl = wave_incl_scan_u64(q);
        const uint64_t hit = __ballot(incl > tl);
        const int src = hit ? __builtin_ctzll(hit) : 63;
        centre = (int64_t)lo * kCdfBlock + sb * 64 + src;
    }
    if (lane == 0) {
        const int r = (int)(centre / W), c = (int)(centre - (int64_t)(centre / W) * W);
        corners[2 * d] = min(max(r - side / 2, 0), H - side);
        corners[2 * d + 1] = min(max(c - side / 2, 0), W - side);
    }
}

// One workgroup per crop.
__global__ __launch_bounds__(256) void k_crop_cut(const float* __restrict__ imgs, int H, int W, int m, int side,
                                                  const int32_t* __restrict__ corners, float* __restrict__ crops) {
    const int64_t d = blockIdx.x;
    const int ss = side * side;
    const float* src = imgs + (d / m) * ((int64_t)H * W) + (int64_t)corners[2 * d] * W + corners[2 * d + 1];
    float* dst = crops + d * ss;
    for (int e = threadIdx.x; e < ss; e += 256) {
        const int r = e / side;
        dst[e] = src[(int64_t)r * W + (e - r * side)];
    }
}

int64_t crop_scratch_bytes(int n_img, int H, int W) {
    const int64_t HW = (int64_t)H * W, nb = (HW + kCdfBlock - 1) / kCdfBlock;
    return (int64_t)n_img * (8 * nb + 8 * (nb + 1) + 8 * kCdfSub * nb);
}

hipError_t launch_sample_crops(const float* imgs, int n_img, int H, int W, const uint64_t* draws, int m, int side,
                               int32_t* corners, float* crops, void* scratch, hipStream_t st) {
    const int64_t HW = (int64_t)H * W;
    const int nb = (int)((HW + kCdfBlock - 1) / kCdfBlock);
    if (n_img < 1 || n_img > 65535 || side < 1 || side > H || side > W || m < 0) return hipErrorInvalidValue;
    unsigned long long* bsum = static_cast<unsigned long long*>(scratch);
    unsigned long long* bpre = bsum + (int64_t)n_img * nb;
    unsigned long long* ssum = bpre + (int64_t)n_img * (nb + 1);
    hipLaunchKernelGGL(k_cdf_weights, dim3(nb, n_img), dim3(256), 0, st, imgs, H, W, nb, bsum, ssum);
    hipLaunchKernelGGL(k_cdf_scan, dim3(n_img), dim3(256), 0, st, bsum, nb, bpre);
    const int64_t nd = (int64_t)n_img * m;
    if (nd == 0) return hipGetLastError();
    hipLaunchKernelGGL(k_cdf_sample, dim3((unsigned)((nd + 3) / 4)), dim3(256), 0, st, imgs, bpre, ssum, H, W, nb,
                       reinterpret_cast<const unsigned long long*>(draws), nd, m, side, corners);
    if (crops)
        hipLaunchKernelGGL(k_crop_cut, dim3((unsigned)nd), dim3(256), 0, st, imgs, H, W, m, side, corners, crops);
    return hipGetLastError();
}

// Entropy partial sums: block blockIdx.x of table blockIdx.y, 256 x 16 slots.
constexpr int kEntSlots = 4096;

__global__ __launch_bounds__(256) void k_dir_entropy(const Slot* __restrict__ dir, uint64_t cap, double n,
                                                     int nblk, double* __restrict__ part) {
    __shared__ double ws[4];
    const Slot* tab = dir + (uint64_t)blockIdx.y * cap;
    const uint64_t s0 = (uint64_t)blockIdx.x * kEntSlots;
    double acc = 0.0;
    for (int u = 0; u < kEntSlots / 256; ++u) {
        const uint64_t s = s0 + threadIdx.x + 256 * u;
        if (s < cap) {
            const Slot e = tab[s];
            if (e.key != kEmptyKey && e.count > 0) {
                const double p = (double)e.count / n;
                acc -= p * log2(p);
            }
        }
    }
    acc = wave_sum_f64(acc);
    if (__lane_id() == 0) ws[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) part[(int64_t)blockIdx.y * nblk + blockIdx.x] = ((ws[0] + ws[1]) + ws[2]) + ws[3];
}

// Table blockIdx.x's partials: lane i adds blocks i, i + 64, ... in order,
// then a fixed-order wave sum.
__global__ __launch_bounds__(64) void k_entropy_sum(const double* __restrict__ part, int nblk,
                                                    double* __restrict__ out) {
    double s = 0.0;
    for (int b = threadIdx.x; b < nblk; b += 64) s += part[(int64_t)blockIdx.x * nblk + b];
    s = wave_sum_f64(s);
    if (threadIdx.x == 0) out[blockIdx.x] = s;
}

int64_t entropy_scratch_bytes(int L, uint64_t cap) {
    const int64_t nblk = (int64_t)((cap + kEntSlots - 1) / kEntSlots);
    return 8 * ((int64_t)L * nblk + L);
}

hipError_t launch_table_entropy(const Slot* dir, int L, uint64_t cap, int64_t n, void* scratch, double* out,
                                hipStream_t st) {
    const int nblk = (int)((cap + kEntSlots - 1) / kEntSlots);
    if (L < 1 || n < 1 || nblk < 1) return hipErrorInvalidValue;
    double* part = static_cast<double*>(scratch);
    hipLaunchKernelGGL(k_dir_entropy, dim3(nblk, L), dim3(256), 0, st, dir, cap, (double)n, nblk, part);
    hipLaunchKernelGGL(k_entropy_sum, dim3(L), dim3(64), 0, st, part, nblk, out);
    return hipGetLastError();
}

}  // namespace zh

namespace zh {

// K nearest candidates under l1 (Section 4.1: the Cauchy hash is sensitive to
// l1 distances) or squared l2 (for candidate sets other than the search's,
// such as the t-of-L sets). One wave (one workgroup) per patch. Candidates go in chunks
// of 16: the wave stages their feature rows in LDS (the chunk's rows
// flattened over the lanes, 16-byte loads when D is a multiple of 4; odd row
// stride in LDS: no bank conflicts), then lane j sums the terms of candidate j
// over the coordinates in index order in FP64, so every distance is the
// oracle's to the bit. Then K rounds of a wave minimum over (distance, ID)
// pick the neighbours in order.
constexpr int kL1Chunk = 16;    // candidates staged at a time (6.5 KB of LDS at D = 100)
constexpr int kL1PerLane = 16;  // chunks: at most 256 candidates a patch
constexpr int kL1MaxD = 128;

// DT: the feature dimension at compile time (0: D at run time, up to 128).
// L1: l1 distances; otherwise squared l2, each term (q_i - x_i)^2 rounded
// before it is added, in index order, as the oracle's FP64 loop does.
template <int DT, bool L1>
__global__ __launch_bounds__(64) void k_knn_rank(int Q, int Drt, int K, int cap, const float* __restrict__ qfeat,
                                               const float* __restrict__ xf, const int32_t* __restrict__ cand,
                                               const int32_t* __restrict__ ncand, int32_t* __restrict__ out_ids,
                                               float* __restrict__ out_d, int32_t* __restrict__ out_m) {
    constexpr int kSt = (DT ? DT : kL1MaxD) | 1;
    __shared__ double sq[DT ? DT : kL1MaxD];
    __shared__ float sx[kL1Chunk * kSt];
    __shared__ int sid[kL1Chunk];
    const int D = DT ? DT : Drt;
    const int lane = threadIdx.x;
    const int q = xcd_block();
    if (q >= Q) return;
    const int M = min(ncand[q], cap);
    const int st = DT ? kSt : (D | 1);
    for (int i = lane; i < D; i += 64) sq[i] = (double)qfeat[(int64_t)q * D + i];
    double d[kL1PerLane];
    int id[kL1PerLane];
#pragma unroll
    for (int u = 0; u < kL1PerLane; ++u) {
        d[u] = INFINITY;
        id[u] = 0x7FFFFFFF;
        const int c0 = kL1Chunk * u;
        if (c0 < M) {
            const int nc = min(kL1Chunk, M - c0);
            const int myid = lane < nc ? cand[(int64_t)q * cap + c0 + lane] : 0;
            __syncthreads();
            if (lane < kL1Chunk) sid[lane] = myid;
            __syncthreads();
            // the chunk's rows, flattened over the wave, eight loads in flight a lane
            if ((D & 3) == 0) {
                const int D4 = D >> 2, n4 = nc * D4;
                const float4* x4 = reinterpret_cast<const float4*>(xf);
                for (int e0 = 0; e0 < n4; e0 += 64 * 8) {
                    float4 v[8];
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        const int e = e0 + lane + 64 * t;
                        if (e < n4) {
                            const int c = e / D4;
                            v[t] = x4[(int64_t)sid[c] * D4 + (e - c * D4)];
                        }
                    }
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        const int e = e0 + lane + 64 * t;
                        if (e < n4) {
                            const int c = e / D4;
                            float* dst = sx + c * st + 4 * (e - c * D4);
                            dst[0] = v[t].x;
                            dst[1] = v[t].y;
                            dst[2] = v[t].z;
                            dst[3] = v[t].w;
                        }
                    }
                }
            } else {
                const int n1 = nc * D;
                for (int e0 = 0; e0 < n1; e0 += 64 * 8) {
                    float v[8];
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        const int e = e0 + lane + 64 * t;
                        if (e < n1) {
                            const int c = e / D;
                            v[t] = xf[(int64_t)sid[c] * D + (e - c * D)];
                        }
                    }
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        const int e = e0 + lane + 64 * t;
                        if (e < n1) {
                            const int c = e / D;
                            sx[c * st + (e - c * D)] = v[t];
                        }
                    }
                }
            }
            __syncthreads();
            if (lane < nc) {
                double acc = 0.0;
#pragma unroll 20
                for (int i = 0; i < D; ++i) {
                    const double t = sq[i] - (double)sx[lane * st + i];
                    acc = acc + (L1 ? fabs(t) : t * t);
                }
                d[u] = acc == acc ? acc : INFINITY;   // not a number: last, by ID
                id[u] = myid;
            }
        }
    }
    const int m = min(K, M);
    for (int k = 0; k < m; ++k) {
        // this lane's smallest (distance, ID), then the wave's
        double bd = d[0];
        int bi = id[0];
#pragma unroll
        for (int u = 1; u < kL1PerLane; ++u)
            if (d[u] < bd || (d[u] == bd && id[u] < bi)) {
                bd = d[u];
                bi = id[u];
            }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double od = __shfl_xor(bd, o);
            const int oi = __shfl_xor(bi, o);
            if (od < bd || (od == bd && oi < bi)) {
                bd = od;
                bi = oi;
            }
        }
#pragma unroll
        for (int u = 0; u < kL1PerLane; ++u)
            if (id[u] == bi) {
                d[u] = INFINITY;
                id[u] = 0x7FFFFFFF;
            }
        if (lane == 0) {
            out_ids[(int64_t)q * K + k] = bi;
            out_d[(int64_t)q * K + k] = (float)bd;
        }
    }
    if (lane >= m && lane < K) {
        out_ids[(int64_t)q * K + lane] = -1;   // past m, as the search leaves them
        out_d[(int64_t)q * K + lane] = 0.0f;
    }
    if (lane == 0) out_m[q] = m;
}

// The same ranking when D is a multiple of 4 (D = 100): lane j takes
// candidate j of each chunk of 64, reads its whole row into registers with
// 16-byte loads (all in flight at once) and sums its terms in index order in
// FP64, the same operations as above; the K rounds of wave minimum follow.
template <int DT, bool L1>
__global__ __launch_bounds__(64) void k_knn_rank_rows(int Q, int K, int cap, const float* __restrict__ qfeat,
                                                    const float* __restrict__ xf, const int32_t* __restrict__ cand,
                                                    const int32_t* __restrict__ ncand, int32_t* __restrict__ out_ids,
                                                    float* __restrict__ out_d, int32_t* __restrict__ out_m) {
    static_assert(DT % 4 == 0 && DT <= kL1MaxD, "rows of whole 16-byte chunks");
    constexpr int D4 = DT / 4;
    constexpr int NCH = kL1Chunk * kL1PerLane / 64;
    __shared__ double sq[DT];
    const int lane = threadIdx.x;
    const int q = xcd_block();
    if (q >= Q) return;
    const int M = min(ncand[q], cap);
    for (int i = lane; i < DT; i += 64) sq[i] = (double)qfeat[(int64_t)q * DT + i];
    __syncthreads();
    double d[NCH];
    int id[NCH];
#pragma unroll
    for (int u = 0; u < NCH; ++u) {
        d[u] = INFINITY;
        id[u] = 0x7FFFFFFF;
        const int c = 64 * u + lane;
        if (c < M) {
            const int myid = cand[(int64_t)q * cap + c];
            const float4* row = reinterpret_cast<const float4*>(xf) + (int64_t)myid * D4;
            float4 x[D4];
#pragma unroll
            for (int t = 0; t < D4; ++t) x[t] = row[t];
            double acc = 0.0;
#pragma unroll
            for (int t = 0; t < D4; ++t) {
                const float xv[4] = {x[t].x, x[t].y, x[t].z, x[t].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double dv = sq[4 * t + e] - (double)xv[e];
                    acc = acc + (L1 ? fabs(dv) : dv * dv);
                }
            }
            d[u] = acc == acc ? acc : INFINITY;   // not a number: last, by ID
            id[u] = myid;
        }
    }
    const int m = min(K, M);
    for (int k = 0; k < m; ++k) {
        double bd = d[0];
        int bi = id[0];
#pragma unroll
        for (int u = 1; u < NCH; ++u)
            if (d[u] < bd || (d[u] == bd && id[u] < bi)) {
                bd = d[u];
                bi = id[u];
            }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double od = __shfl_xor(bd, o);
            const int oi = __shfl_xor(bi, o);
            if (od < bd || (od == bd && oi < bi)) {
                bd = od;
                bi = oi;
            }
        }
#pragma unroll
        for (int u = 0; u < NCH; ++u)
            if (id[u] == bi) {
                d[u] = INFINITY;
                id[u] = 0x7FFFFFFF;
            }
        if (lane == 0) {
            out_ids[(int64_t)q * K + k] = bi;
            out_d[(int64_t)q * K + k] = (float)bd;
        }
    }
    if (lane >= m && lane < K) {
        out_ids[(int64_t)q * K + lane] = -1;
        out_d[(int64_t)q * K + lane] = 0.0f;
    }
    if (lane == 0) out_m[q] = m;
}

// The l1 screen rows, one thread an entry. Any lo and step give valid
// bounds, since eps is measured against the very values fmaf(step, u, lo)
// the ranking forms; the row's minimum and range / 255 keep eps small. eps is
// summed in FP64 and rounded up with a margin of 2^-20 relative, which covers
// that sum's own rounding and the fp32 rounding of the bounds formed from it.
__global__ __launch_bounds__(256) void k_l1_screen_rows(const float* __restrict__ xf, int64_t n,
                                                      uint8_t* __restrict__ l1s) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    const float4* x4 = reinterpret_cast<const float4*>(xf + r * kL1sDim);
    float x[kL1sDim];
#pragma unroll
    for (int t = 0; t < kL1sDim / 4; ++t) {
        const float4 v = x4[t];
        x[4 * t] = v.x;
        x[4 * t + 1] = v.y;
        x[4 * t + 2] = v.z;
        x[4 * t + 3] = v.w;
    }
    float lo = x[0], hi = x[0];
#pragma unroll
    for (int i = 1; i < kL1sDim; ++i) {
        lo = fminf(lo, x[i]);
        hi = fmaxf(hi, x[i]);
    }
    float step = (hi - lo) * (1.0f / 255.0f);
    if (!(step > 0.0f) || !(step < INFINITY)) step = 0.0f;
    uint32_t w[kL1sBytes / 4];
#pragma unroll
    for (int i = 0; i < kL1sBytes / 4; ++i) w[i] = 0u;
    double eps = 0.0;
#pragma unroll
    for (int i = 0; i < kL1sDim; ++i) {
        float u = step > 0.0f ? rintf((x[i] - lo) / step) : 0.0f;
        u = fminf(fmaxf(u, 0.0f), 255.0f);
        eps += fabs((double)x[i] - (double)fmaf(step, u, lo));
        w[i >> 2] |= (uint32_t)u << (8 * (i & 3));
    }
    const double eu = eps * (1.0 + 0x1p-20);
    float ef = (float)eu;
    if ((double)ef < eu) ef = nextafterf(ef, INFINITY);
    if (!(ef >= 0.0f)) ef = INFINITY;   // a non-finite feature: bounds that prune nothing
    constexpr int t0 = kL1sTail / 4;
    w[t0] = __float_as_uint(lo);
    w[t0 + 1] = __float_as_uint(step);
    w[t0 + 2] = __float_as_uint(ef);
    uint4* out = reinterpret_cast<uint4*>(l1s + r * kL1sBytes);
#pragma unroll
    for (int t = 0; t < kL1sBytes / 16; ++t) out[t] = make_uint4(w[4 * t], w[4 * t + 1], w[4 * t + 2], w[4 * t + 3]);
}

__global__ void k_min_i32(int n, const int32_t* __restrict__ in, int cap, int32_t* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = min(in[i], cap);
}

hipError_t launch_min_i32(int n, const int32_t* in, int cap, int32_t* out, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_min_i32, dim3((n + 255) / 256), dim3(256), 0, st, n, in, cap, out);
    return hipGetLastError();
}

hipError_t launch_l1_screen_rows(const float* xf, int64_t n, uint8_t* l1s, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    if ((reinterpret_cast<uintptr_t>(xf) & 15) || (reinterpret_cast<uintptr_t>(l1s) & 15)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_l1_screen_rows, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, xf, n, l1s);
    return hipGetLastError();
}

// K nearest under l1 with the screen (D = 100). One wave a patch:
//  1. A = sum_i |q_i - fmaf(step, u_i, lo)| in fp32 from the candidate's
//     128-byte screen row; with eps = ||x - x~||_1 the triangle inequality
//     puts its l1 distance in [A - eps, A + eps]. An fp32 sum of 100
//     non-negative terms, in any order, is within 101 u A of its exact value,
//     so the bounds widen A by 2^-15 relative: lb = fmaf(A, 1 - 2^-15, -eps),
//     ub = fmaf(A, 1 + 2^-15, eps), each rounded once. Lane j takes candidate
//     j of a chunk of 64; a last chunk of at most 8 candidates is spread over
//     8 lanes each, one 16-byte segment of the row a lane.
//  2. tau = the K-th smallest ub, by binary search over the bit patterns of
//     the (non-negative) bounds with ballot counts: K candidates lie within
//     tau.
//  3. A candidate with lb > tau (1 + 2^-20) is farther than those K even
//     after the FP64 rounding of every distance, so it cannot be among the K
//     nearest in (distance, ID) order; the others survive, compacted in LDS.
//  4. The survivors' exact distances, summed in index order in FP64 as the
//     unscreened kernels do; with at most 64 survivors each one's rank in
//     (distance, ID) order is counted against all the others (IDs are
//     distinct), else K rounds of wave minimum pick them.
// With M <= K candidates nothing is screened.
// Bound: VALU issue and the gathers. 203,636 patches at D = 100, cap 72, K = 8:
// with a lane a survivor (300 FP64 instructions for about nine live lanes, the
// query's values in 200 registers or spilled) 487 us; by quads 447, and held to
// the 102 registers of five waves a SIMD 398 (six spill: 634).
__global__ __launch_bounds__(64, 5) void k_knn_l1_screened(int Q, int K, int cap, const float* __restrict__ qfeat,
                                                      const float* __restrict__ xf, const uint8_t* __restrict__ l1s,
                                                      const int32_t* __restrict__ cand,
                                                      const int32_t* __restrict__ ncand, int32_t* __restrict__ out_ids,
                                                      float* __restrict__ out_d, int32_t* __restrict__ out_m,
                                                      int32_t* __restrict__ out_ns) {
    constexpr int DT = kL1sDim, D4 = DT / 4, NCH = kRankMaxCand / 64;
    constexpr int kSeg = (kL1sTail + 12 + 15) / 16;   // 16-byte loads that hold the codes and the tail
    static_assert(kSeg <= 8 && kL1sTail % 16 == 4, "codes, then lo, step, eps in the last 16-byte load");
    __shared__ double sq[DT];
    __shared__ float4 sqf[D4];
    __shared__ int sid[kRankMaxCand];
    __shared__ double sd[kRankMaxCand];
    const int lane = threadIdx.x;
    const int q = xcd_block();
    if (q >= Q) return;
    const int M = min(ncand[q], cap);
    const int32_t* cq = cand + (int64_t)q * cap;
    for (int i = lane; i < DT; i += 64) {
        const float v = qfeat[(int64_t)q * DT + i];
        sq[i] = (double)v;
        reinterpret_cast<float*>(sqf)[i] = v;
    }
    int ns = 0;
    if (M > K) {
        __syncthreads();
        uint32_t ubb[NCH];   // bit patterns of the upper bounds; 0xFFFFFFFF: no candidate
        float lb[NCH];
        int idc[NCH];
#pragma unroll
        for (int u = 0; u < NCH; ++u) {
            ubb[u] = 0xFFFFFFFFu;
            lb[u] = INFINITY;
            idc[u] = 0;
            const int base = 64 * u;
            if (base >= M) continue;
            const int r = M - base;
            float A = 0.0f, lo = 0.0f, st = 0.0f, e = 0.0f;
            bool own = false;   // this lane reports the chunk's candidate
            int id = 0;
            if (r > 8) {
                if (lane < r) {
                    id = cq[base + lane];
                    own = true;
                    const uint4* row = reinterpret_cast<const uint4*>(l1s + (size_t)id * kL1sBytes);
                    uint4 v[kSeg];
#pragma unroll
                    for (int t = 0; t < kSeg; ++t) v[t] = row[t];
                    const uint32_t* wv = reinterpret_cast<const uint32_t*>(v);
                    lo = __uint_as_float(wv[kL1sTail / 4]);
                    st = __uint_as_float(wv[kL1sTail / 4 + 1]);
                    e = __uint_as_float(wv[kL1sTail / 4 + 2]);
#pragma unroll
                    for (int t = 0; t < D4; ++t) {
                        const float4 qv = sqf[t];
                        const uint32_t cw = wv[t];
                        A += fabsf(qv.x - fmaf(st, (float)(cw & 255u), lo));
                        A += fabsf(qv.y - fmaf(st, (float)((cw >> 8) & 255u), lo));
                        A += fabsf(qv.z - fmaf(st, (float)((cw >> 16) & 255u), lo));
                        A += fabsf(qv.w - fmaf(st, (float)(cw >> 24), lo));
                    }
                }
            } else {
                // 8 lanes a candidate, lane seg of the group on codes 16 seg .. 16 seg + 15
                const int g = lane >> 3, seg = lane & 7;
                if (g < r) {
                    id = cq[base + g];
                    own = seg == 0;
                    const uint4* row = reinterpret_cast<const uint4*>(l1s + (size_t)id * kL1sBytes);
                    const uint4 tl = row[kSeg - 1];
                    lo = __uint_as_float(tl.y);
                    st = __uint_as_float(tl.z);
                    e = __uint_as_float(tl.w);
                    if (seg < kSeg) {
                        const uint4 v = row[seg];
                        const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            if (4 * seg + t >= D4) break;
                            const float4 qv = sqf[4 * seg + t];
                            const uint32_t cw = wv[t];
                            A += fabsf(qv.x - fmaf(st, (float)(cw & 255u), lo));
                            A += fabsf(qv.y - fmaf(st, (float)((cw >> 8) & 255u), lo));
                            A += fabsf(qv.z - fmaf(st, (float)((cw >> 16) & 255u), lo));
                            A += fabsf(qv.w - fmaf(st, (float)(cw >> 24), lo));
                        }
                    }
                }
                A = group8_sum_f32(A);
            }
            if (own) {
                float l = fmaf(A, 1.0f - 0x1p-15f, -e);
                float h = fmaf(A, 1.0f + 0x1p-15f, e);
                if (!(h >= 0.0f)) {   // non-finite: keep the candidate, set no threshold by it
                    l = 0.0f;
                    h = INFINITY;
                }
                lb[u] = l;
                ubb[u] = __float_as_uint(h);
                idc[u] = id;
            }
        }
        // 2. tau: the smallest bit pattern with at least K upper bounds at or below it
        uint32_t blo = 0u, bhi = 0x7F800000u;
        while (blo < bhi) {
            const uint32_t mid = blo + ((bhi - blo) >> 1);
            int cnt = 0;
#pragma unroll
            for (int u = 0; u < NCH; ++u) {
                if (64 * u >= M) break;
                cnt += __popcll(__ballot(ubb[u] <= mid));
            }
            if (cnt >= K) bhi = mid;
            else blo = mid + 1u;
        }
        const float thr = __uint_as_float(blo) * (1.0f + 0x1p-20f);
        // 3. survivors, compacted in candidate order
#pragma unroll
        for (int u = 0; u < NCH; ++u) {
            if (64 * u >= M) break;
            const bool keep = ubb[u] != 0xFFFFFFFFu && !(lb[u] > thr);
            const uint64_t bm = __ballot(keep);
            if (keep) sid[ns + __popcll(bm & ((1ull << lane) - 1ull))] = idc[u];
            ns += __popcll(bm);
        }
    } else {
        for (int j = lane; j < M; j += 64) sid[j] = cq[j];
        ns = M;
    }
    __syncthreads();
    if (out_ns && lane == 0) out_ns[q] = ns;
    // 4. exact distances of the survivors, four lanes each: lane qd of a quad
    // forms the terms of every fourth four coordinates, and the sum goes
    // through the coordinates in order (quad_take)
    const int qd = lane & 3;
    for (int j0 = 0; j0 < ns; j0 += 16) {
        const int j = j0 + (lane >> 2);
        const float4* row = reinterpret_cast<const float4*>(xf) + (int64_t)sid[j < ns ? j : j0] * D4;
        constexpr int T = (D4 + 3) / 4;
        float4 x[T];
#pragma unroll
        for (int t = 0; t < T; ++t) x[t] = row[min(4 * t + qd, D4 - 1)];
        double acc = 0.0;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const double* qv = sq + 4 * min(4 * t + qd, D4 - 1);
            const double p0 = fabs(qv[0] - (double)x[t].x), p1 = fabs(qv[1] - (double)x[t].y);
            const double p2 = fabs(qv[2] - (double)x[t].z), p3 = fabs(qv[3] - (double)x[t].w);
            auto add = [&](double s) { return (((s + p0) + p1) + p2) + p3; };
            acc = quad_take<0>(add(acc));
            if (4 * t + 1 < D4) acc = quad_take<1>(add(acc));
            if (4 * t + 2 < D4) acc = quad_take<2>(add(acc));
            if (4 * t + 3 < D4) acc = quad_take<3>(add(acc));
        }
        if (qd == 0 && j < ns) sd[j] = acc == acc ? acc : INFINITY;   // not a number: last, by ID
    }
    __syncthreads();
    double d[NCH];
    int id[NCH];
#pragma unroll
    for (int u = 0; u < NCH; ++u) {
        const int j = 64 * u + lane;
        d[u] = 64 * u < ns && j < ns ? sd[j] : INFINITY;
        id[u] = 64 * u < ns && j < ns ? sid[j] : 0x7FFFFFFF;
    }
    const int m = min(K, M);
    if (ns <= 64) {
        // rank of survivor lane among all survivors in (distance, ID) order
        const int64_t dbits = __double_as_longlong(d[0]);
        const int dlo = (int)(dbits & 0xFFFFFFFF), dhi = (int)(dbits >> 32);
        int rank = 0;
        for (int t = 0; t < ns; ++t) {
            const int tlo = __builtin_amdgcn_readlane(dlo, t), thi = __builtin_amdgcn_readlane(dhi, t);
            const int tid = __builtin_amdgcn_readlane(id[0], t);
            const double dt = __longlong_as_double(((int64_t)thi << 32) | (int64_t)(uint32_t)tlo);
            rank += (dt < d[0] || (dt == d[0] && tid < id[0])) ? 1 : 0;
        }
        if (lane < ns && rank < m) {
            out_ids[(int64_t)q * K + rank] = id[0];
            out_d[(int64_t)q * K + rank] = (float)d[0];
        }
    } else {
        for (int k = 0; k < m; ++k) {
            double bd = d[0];
            int bi = id[0];
#pragma unroll
            for (int u = 1; u < NCH; ++u)
                if (d[u] < bd || (d[u] == bd && id[u] < bi)) {
                    bd = d[u];
                    bi = id[u];
                }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                const double od = __shfl_xor(bd, o);
                const int oi = __shfl_xor(bi, o);
                if (od < bd || (od == bd && oi < bi)) {
                    bd = od;
                    bi = oi;
                }
            }
#pragma unroll
            for (int u = 0; u < NCH; ++u)
                if (id[u] == bi) {
                    d[u] = INFINITY;
                    id[u] = 0x7FFFFFFF;
                }
            if (lane == 0) {
                out_ids[(int64_t)q * K + k] = bi;
                out_d[(int64_t)q * K + k] = (float)bd;
            }
        }
    }
    if (lane >= m && lane < K) {
        out_ids[(int64_t)q * K + lane] = -1;
        out_d[(int64_t)q * K + lane] = 0.0f;
    }
    if (lane == 0) out_m[q] = m;
}

hipError_t launch_knn_l1_screened(int Q, int K, int cap, const float* qfeat, const float* xf, const uint8_t* l1s,
                                  const int32_t* cand, const int32_t* ncand, int32_t* ids, float* d, int32_t* m,
                                  int32_t* ns, hipStream_t st) {
    if (Q == 0) return hipSuccess;
    if (cap < 1 || cap > kRankMaxCand || K < 1 || K > kMaxK) return hipErrorInvalidValue;
    if (!one_row(round_grid8(Q), 64)) return hipErrorInvalidConfiguration;
    if ((reinterpret_cast<uintptr_t>(xf) & 15) || (reinterpret_cast<uintptr_t>(l1s) & 15)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_knn_l1_screened, dim3(round_grid8(Q)), dim3(64), 0, st, Q, K, cap, qfeat, xf, l1s, cand,
                       ncand, ids, d, m, ns);
    return hipGetLastError();
}

hipError_t launch_knn_rank(int Q, int D, int K, int cap, bool l1, const float* qfeat, const float* xf,
                           const int32_t* cand, const int32_t* ncand, int32_t* ids, float* d, int32_t* m,
                           hipStream_t st) {
    if (Q == 0) return hipSuccess;
    if (cap < 1 || cap > kL1Chunk * kL1PerLane || K < 1 || K > kMaxK || D < 1 || D > kL1MaxD) return hipErrorInvalidValue;
    if (!one_row(round_grid8(Q), 64)) return hipErrorInvalidConfiguration;
    const int grid = round_grid8(Q);   // patches in contiguous runs per XCD: neighbours share candidates in L2
#define ZH_RANK(DT, M1) \
    hipLaunchKernelGGL((k_knn_rank<DT, M1>), dim3(grid), dim3(64), 0, st, Q, D, K, cap, qfeat, xf, cand, ncand, ids, d, m)
    if (D == 100) {
        const bool al = (reinterpret_cast<uintptr_t>(xf) & 15) == 0;
        if (al && l1)
            hipLaunchKernelGGL((k_knn_rank_rows<100, true>), dim3(grid), dim3(64), 0, st, Q, K, cap, qfeat, xf, cand, ncand,
                               ids, d, m);
        else if (al)
            hipLaunchKernelGGL((k_knn_rank_rows<100, false>), dim3(grid), dim3(64), 0, st, Q, K, cap, qfeat, xf, cand,
                               ncand, ids, d, m);
        if (al) return hipGetLastError();
    }
    if (l1) {
        if (D == 100) ZH_RANK(100, true);
        else if (D == 25) ZH_RANK(25, true);
        else ZH_RANK(0, true);
    } else {
        if (D == 100) ZH_RANK(100, false);
        else if (D == 25) ZH_RANK(25, false);
        else ZH_RANK(0, false);
    }
#undef ZH_RANK
    return hipGetLastError();
}

}  // namespace zh

namespace zh {

// t-of-L candidates (Section 4.1: a training patch matches when it shares the
// query's bucket in at least t of the L tables). One wave per patch; the
// patch's L bins (sorted by ID) are walked in table order, 64 entries at a
// time. An entry x of bin l is kept at its first table only (no earlier bin
// holds it) and counted in the later ones, both by binary search; IDs with
// at least t hits are written in walk order (the set is what is defined).
__global__ __launch_bounds__(256) void k_cand_t(int Q, int L, int64_t N, int t, const uint2* __restrict__ bins,
                                                const uint32_t* __restrict__ tids, int cap,
                                                int32_t* __restrict__ counts, int32_t* __restrict__ ids) {
    __shared__ uint32_t s_off[4][64], s_cnt[4][64];
    __shared__ int64_t s_st[4][64];
    const int lane = __lane_id(), wv = threadIdx.x >> 6;
    const int q = blockIdx.x * 4 + wv;
    if (q >= Q) return;
    const uint2 b = lane < L ? bins[(int64_t)lane * Q + q] : make_uint2(0u, 0u);
    int64_t incl = b.y;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t v = __shfl_up(incl, o);
        if (lane >= o) incl += v;
    }
    s_off[wv][lane] = b.x;
    s_cnt[wv][lane] = b.y;
    s_st[wv][lane] = incl - b.y;
    const int64_t S = __shfl(incl, 63);
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    auto in_bin = [&](int l, uint32_t x) {
        const uint32_t* p = tids + (int64_t)l * N + s_off[wv][l];
        uint32_t lo = 0, hi = s_cnt[wv][l];
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (p[mid] < x) lo = mid + 1;
            else hi = mid;
        }
        return lo < s_cnt[wv][l] && p[lo] == x;
    };
    int64_t kept = 0;
    for (int64_t e0 = 0; e0 < S; e0 += 64) {
        const int64_t e = e0 + lane;
        bool keep = false;
        uint32_t x = 0;
        if (e < S) {
            int l = 0;
            while (l + 1 < L && s_st[wv][l + 1] <= e) ++l;
            x = tids[(int64_t)l * N + s_off[wv][l] + (e - s_st[wv][l])];
            bool first = true;
            for (int j = 0; j < l && first; ++j) first = !in_bin(j, x);
            if (first) {
                int hits = 1;
                for (int j = l + 1; j < L && hits < t; ++j) hits += in_bin(j, x) ? 1 : 0;
                keep = hits >= t;
            }
        }
        const uint64_t mask = __ballot(keep);
        const int64_t pos = kept + __popcll(mask & lanemask_lt());
        if (keep && pos < cap) ids[(int64_t)q * cap + pos] = (int32_t)x;
        kept += __popcll(mask);
    }
    if (lane == 0) counts[q] = (int32_t)kept;
}

// K nearest of the IDs that at least t of a patch's L bins hold, however many
// there are (t = 1: of the union). One workgroup per patch.
//
// The bins are sorted by ID, so they are taken together in windows of
// ascending ID ranges of at most kWinMax entries: with more entries left, every
// bin may offer kWinMax / (bins left) of them, the window ends before the
// smallest ID that lies just past such an offer, and each bin takes its IDs
// below that end. A window's entries go into a hash table in LDS (open
// addressing; a byte per slot counts the bins that hold the ID); the entry
// that brings an ID to t bins appends it to the window's list. Each ID of the
// list gets its squared distance as the FP64 sequential sum over the
// coordinates in index order (each term rounded before it is added, the
// definition), a lane per ID, and enters its wave's running K nearest, kept
// sorted in lanes 0 .. K-1, when it beats the K-th; the four waves' lists are
// merged at the end. IDs are distinct across windows.
//
// Bound: latency: the dependent reads and LDS passes of each window in turn (a
// window of 800 entries of 16 bins about 7 us, a third of it the listed rows),
// with as many workgroups on a compute unit as LDS allows (five; a row's reads
// 13 or 9 instead of 5 at a time take the registers of one or two of them: 489
// and 403 against 348 us below). The form before searched every other bin for
// each entry (L - 1 binary searches of dependent loads), and the union without
// a stop was sorted in LDS by one wave: 14,732 patches, L = 16, 100k pairs,
// t = 2: 14.8 -> 0.55 ms, with the long patches first and in shares 0.37; 3,600
// patches, L = 8, 20k pairs at D = 25, t = 1 (unions of up to 1,600 IDs): 2.37
// -> 0.06 ms. Up to 64 IDs, the first wave's alone, need no merge, and from 8192
// patches on those of at most 64 entries take a wave each (rank_few): 207,836 patches,
// L = 8, unions of 0 or 1 ID 676 -> 128 us (the wave a patch before all this 356),
// 44,100 at K = 16 with 8 IDs each 290 -> 92 (3502).
constexpr int kWinMax = 2048;               // entries of a window
constexpr int kWinSlots = 2 * kWinMax;      // largest hash table: load at most 1/2

__device__ __forceinline__ double readlane_f64(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}
// (d, id) of the lanes with `act` into the K smallest held sorted by lanes
// 0 .. K-1 (K <= 16: one row of lanes, shifted within the vector unit)
__device__ __forceinline__ void topk_insert(bool act, double d, int id, int K, double& bd, int& bi) {
    const int lane = __lane_id();
    for (;;) {
        const double kd = readlane_f64(bd, K - 1);
        const int ki = __builtin_amdgcn_readlane(bi, K - 1);
        const uint64_t todo = __ballot(act && (d < kd || (d == kd && id < ki)));
        if (!todo) return;
        const int src = __builtin_ctzll(todo);
        const double nd = readlane_f64(d, src);
        const int ni = __builtin_amdgcn_readlane(id, src);
        const int at = __popcll(__ballot(lane < K && (bd < nd || (bd == nd && bi < ni))));
        // row_shr 1
        const int uh = dpp_or0<0x111>(__double2hiint(bd)), ul = dpp_or0<0x111>(__double2loint(bd));
        const int ui = dpp_or0<0x111>(bi);
        if (lane > at) {
            bd = __hiloint2double(uh, ul);
            bi = ui;
        } else if (lane == at) {
            bd = nd;
            bi = ni;
        }
        if (lane == src) act = false;
    }
}
// The K smallest of the first n lanes' (d, id), sorted, into lanes 0 .. K-1 (the
// rest +inf): every lane counts the lanes before it, and those counted to
// 0 .. K-1 hand theirs over through LDS (K places of the wave's own).
__device__ __forceinline__ void topk_first(int n, double d, int id, int K, double* pd, int* pi, double& bd, int& bi) {
    const int lane = __lane_id();
    int rank = 0;
    for (int j = 0; j < n; ++j) {
        const double nd = readlane_f64(d, j);
        const int ni = __builtin_amdgcn_readlane(id, j);
        // (empty places may be equal: by lane, so that every rank has a lane)
        rank += nd < d || (nd == d && (ni < id || (ni == id && j < lane))) ? 1 : 0;
    }
    if (lane < n && rank < K) {
        pd[rank] = d;
        pi[rank] = id;
    }
    __builtin_amdgcn_wave_barrier();
    if (lane < K && lane < n) {
        bd = pd[lane];
        bi = pi[lane];
    }
}

// a patch's result from its sorted list in lanes 0 .. K-1 of a wave
__device__ __forceinline__ void write_ranked(int q, int K, int kept, double bd, int bi, int32_t* __restrict__ counts,
                                             int32_t* __restrict__ out_ids, float* __restrict__ out_d,
                                             int32_t* __restrict__ out_m) {
    const int lane = __lane_id();
    const int m = kept < K ? kept : K;
    if (lane < K) {
        out_ids[(int64_t)q * K + lane] = lane < m ? bi : -1;
        out_d[(int64_t)q * K + lane] = lane < m ? (float)bd : 0.0f;
    }
    if (lane == 0) {
        counts[q] = kept;
        out_m[q] = m;
    }
}

// Long patches, those with more entries than a window, are listed first, so that
// none begins when all others end, and those of more than kLongShare entries
// in shares by ranges of IDs (at most kLongParts), which a last launch joins. The
// other patches of more than kFewMax entries have a list of their own, which the
// remaining workgroups go through; then each takes four of those with fewer, a wave
// a patch (a workgroup a patch is bound by its launch there: 207,836 patches with at
// most one entry 256 us). mid_blocks: enough for the few, and one a patch of the list
// up to kMidBlocks (the list's last patches end together; more would be launched for
// nothing where it is short). Workgroups of their own for the few, and 8192 for the list:
// 14,732 patches of which most are long 537 us instead of 531 for the whole zoom,
// 207,836 of mixed lengths 484 instead of 523.
constexpr int kLongMax = 8192, kLongParts = 16, kLongShare = 4096, kLongBlocks = 1024;
constexpr int kMidBlocks = 16384, kFewMax = 64;
__host__ __device__ constexpr int mid_blocks(int Q) {
    return Q / 4 + 1 > kMidBlocks ? Q / 4 + 1 : (Q < kMidBlocks ? Q : kMidBlocks);
}
// Patches from which the lists' two more launches (18 us for 14,732 patches) pay:
// there the ranking went from 545 to 348 us; 3,600 patches take 56 us in all, and
// their longest begins early enough.
constexpr int kLongMin = 8192;
struct LongLists {
    unsigned int* n;     // entries of item, and of mid; 0 before the first launch
    int2* item;          // [kLongMax] patch, and share + 32 shares
    double* d;           // [kLongMax, K] nearest of a share
    int32_t* id;
    int32_t* kept;       // [kLongMax] IDs of a share
    int32_t* mid;        // [Q] patches of more than kFewMax entries that are not in item
    uint8_t* listed;     // [Q] whether a patch is in one of the lists
};

__global__ __launch_bounds__(256) void k_bins_long(int Q, int L, const uint2* __restrict__ bins, LongLists ll) {
    const int q = blockIdx.x * 256 + threadIdx.x;
    uint32_t total = 0;
#pragma unroll 8
    for (int l = 0; l < L; ++l) total += q < Q ? min(bins[(int64_t)l * Q + q].y, 1u << 25) : 0u;
    bool listed = false;
    if (total > (uint32_t)kWinMax) {
        const int shares = (int)min((uint32_t)kLongParts, (total + kLongShare - 1) / kLongShare);
        const unsigned at = atomicAdd(ll.n, (unsigned)shares);
        listed = at + shares <= (unsigned)kLongMax;
        for (int p = 0; p < shares && at + p < (unsigned)kLongMax; ++p)
            ll.item[at + p] = make_int2(listed ? q : -1, p + 32 * shares);
    }
    // one atomic a workgroup
    __shared__ unsigned cnt[4], base;
    const bool mid = !listed && total > (uint32_t)kFewMax;
    const uint64_t bal = __ballot(mid);
    const int wv = threadIdx.x >> 6;
    if (__lane_id() == 0) cnt[wv] = (unsigned)__popcll(bal);
    __syncthreads();
    if (threadIdx.x == 0) base = atomicAdd(ll.n + 1, cnt[0] + cnt[1] + cnt[2] + cnt[3]);
    __syncthreads();
    unsigned at = base + (unsigned)__popcll(bal & lanemask_lt());
    for (int v = 0; v < wv; ++v) at += cnt[v];
    if (mid) ll.mid[at] = q;
    if (q < Q) ll.listed[q] = listed || mid ? 1 : 0;
}

// Entries below `end` among the first n of src, ascending: seven probes a step.
__device__ __forceinline__ uint32_t count_below(const uint32_t* __restrict__ src, uint32_t n, uint32_t end) {
    uint32_t lo = 0, hi = n;
    while (lo < hi) {
        const uint32_t step = (hi - lo + 7u) >> 3;
        uint32_t v[7], c = 0;
#pragma unroll
        for (uint32_t j = 0; j < 7; ++j) {
            const uint32_t p = lo + (j + 1u) * step - 1u;
            v[j] = src[p < hi ? p : lo];
            v[j] = p < hi ? v[j] : 0xFFFFFFFFu;
        }
#pragma unroll
        for (uint32_t j = 0; j < 7; ++j) c += v[j] < end ? 1u : 0u;
        hi = c < 7u ? min(hi, lo + (c + 1u) * step - 1u) : hi;
        lo += c * step;
    }
    return lo;
}

// FP64 squared distance of row `row` (the sequential sum over the coordinates in
// index order) from the query q (LDS); not a number: infinite, last by ID.
template <int D>
__device__ __forceinline__ double rank_distance(const float* __restrict__ row, const double* q) {
    double d = 0.0;
    auto term = [&](int i, float x) {
        const double t0 = q[i] - (double)x;
        d = d + t0 * t0;
    };
    if (D == 100) {
        // a fifth of a row on its way at a time
        const float4* r4 = reinterpret_cast<const float4*>(row);
#pragma unroll 1
        for (int h = 0; h < 25; h += 5) {
            float4 v[5];
#pragma unroll
            for (int u = 0; u < 5; ++u)
                if (h + u < 25) v[u] = r4[h + u];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < 5; ++u)
                if (h + u < 25) {
                    term(4 * (h + u), v[u].x);
                    term(4 * (h + u) + 1, v[u].y);
                    term(4 * (h + u) + 2, v[u].z);
                    term(4 * (h + u) + 3, v[u].w);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        float v[D];
#pragma unroll
        for (int i = 0; i < D; ++i) v[i] = row[i];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < D; ++i) term(i, v[i]);
    }
    return d == d ? d : INFINITY;
}

// A patch of at most 64 entries by one wave, an entry a lane: each lane counts the
// lanes with its ID; the first of t or more stands for it.
template <int D>
__device__ __forceinline__ void rank_few(int q, int64_t N, int t, int K, uint2 b, const uint32_t* __restrict__ tids,
                                         const float* __restrict__ qfeat, const float* __restrict__ xf,
                                         int32_t* __restrict__ counts, int32_t* __restrict__ out_ids,
                                         float* __restrict__ out_d, int32_t* __restrict__ out_m, double* sq, double* pd,
                                         int* pi) {
    const int lane = __lane_id();
    for (int i = lane; i < D; i += 64) sq[i] = (double)qfeat[(int64_t)q * D + i];   // the wave's own
    const int incl = wave_incl_scan((int)b.y);
    const int n = __builtin_amdgcn_readlane(incl, 63);
    // the bin of entry `lane`: the number of bins that end at or before it
    int l = 0;
#pragma unroll
    for (int s = 32; s > 0; s >>= 1)
        if (__shfl(incl, l + s - 1) <= lane) l += s;
    const uint32_t off = (uint32_t)__shfl((int)b.x, l) + (uint32_t)(lane - (__shfl(incl, l) - __shfl((int)b.y, l)));
    const int id = lane < n ? (int)tids[(int64_t)l * N + off] : -1;
    int hits = 0;
    bool first = true;
    for (int j = 0; j < n; ++j) {
        const bool same = __builtin_amdgcn_readlane(id, j) == id;
        hits += same ? 1 : 0;
        first = first && !(same && j < lane);
    }
    const bool act = lane < n && first && hits >= t;
    const int kept = __popcll(__ballot(act));
    double d = INFINITY, bd = INFINITY;
    int bi = 0x7FFFFFFF;
    __builtin_amdgcn_wave_barrier();
    if (act) d = rank_distance<D>(xf + (int64_t)id * D, sq);
    if (kept) topk_first(n, d, act ? id : 0x7FFFFFFF, K, pd, pi, bd, bi);
    write_ranked(q, K, kept, bd, bi, counts, out_ids, out_d, out_m);
}

template <int D, bool LISTS>
__global__ __launch_bounds__(256, 5) void k_bins_rank(int Q, int L, int64_t N, int t, int K,
                                                   const uint2* __restrict__ bins, const uint32_t* __restrict__ tids,
                                                   const float* __restrict__ qfeat, const float* __restrict__ xf,
                                                   int32_t* __restrict__ counts, int32_t* __restrict__ out_ids,
                                                   float* __restrict__ out_d, int32_t* __restrict__ out_m,
                                                   unsigned int* __restrict__ counters, LongLists ll) {
    __shared__ __align__(8) uint32_t s_key[kWinSlots];
    static_assert(sizeof(s_key) >= 4 * D * sizeof(double), "the few's queries lie there");
    __shared__ uint32_t s_cnt[kWinSlots / 4];
    __shared__ uint32_t s_list[kWinMax];
    __shared__ double s_q[D];
    __shared__ int64_t s_ofs[64];
    __shared__ int s_start[64];
    __shared__ int s_nk, s_pos;
    __shared__ double s_td[4 * kMaxK];
    __shared__ int s_ti[4 * kMaxK];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int blk = (int)block_id();
    const bool longs = LISTS && blk < kLongBlocks;
    int item = blk, items = blk + 1, step = 1;
    if (!LISTS && blk >= Q) return;
    if (LISTS) {
        const int mids = mid_blocks(Q);
        if (blk - kLongBlocks >= mids) return;
        item = longs ? blk : blk - kLongBlocks;
        step = longs ? kLongBlocks : mids;
        items = longs ? (int)min(ll.n[0], (unsigned)kLongMax) : (int)ll.n[1];
    }
    for (; item < items; item += step) {
        // not in runs per XCD: the patches of a flat region, the longest ones, are
        // neighbours (0.91 against 0.56 ms on the 14,732 patches above)
        const int2 it = longs ? ll.item[item] : make_int2(LISTS ? ll.mid[item] : item, 32);
        const int q = it.x;
        const int part = it.y & 31, shares = it.y >> 5;
        if (LISTS && q < 0) continue;
        // every wave holds the patch's bins in its lanes: the position of the next
        // entry and the entries left
        const uint2 b = lane < L ? bins[(int64_t)lane * Q + q] : make_uint2(0u, 0u);
        if (!LISTS && __ballot(b.y > 0u) == 0) {
            if (wv == 0) write_ranked(q, K, 0, 0.0, 0, counts, out_ids, out_d, out_m);
            return;
        }
        if (LISTS) __syncthreads();   // the last item's arrays are no longer read
        for (int i = tid; i < D; i += 256) s_q[i] = (double)qfeat[(int64_t)q * D + i];
        const uint32_t* src = tids + (int64_t)lane * N + b.x;
        int64_t pos = (int64_t)lane * N + b.x;
        uint32_t left = b.y;
        if (counters && tid < 64 && part == 0) {
            // patches over the limits of the LDS forms of the union search
            const int total = wave_sum_i32((int)min(left, 8193u));
            if (lane == 0 && total > 2048) {
                atomicAdd(&counters[C_OVERFLOW], 1u);
                if (total > 8192) atomicAdd(&counters[C_STREAM], 1u);
            }
        }
        if (LISTS && shares > 1) {
            // the ends of the shares are quantiles of the largest bin
            const uint32_t big = wave_max_u32(left);
            const int bl = __builtin_ctzll(__ballot(left == big));
            const uint32_t* bsrc = tids + (int64_t)bl * N + (uint32_t)__builtin_amdgcn_readlane((int)b.x, bl);
            const uint32_t id0 = part == 0 ? 0u : bsrc[(uint64_t)big * part / shares];
            const uint32_t id1 = part + 1 < shares ? bsrc[(uint64_t)big * (part + 1) / shares] : 0xFFFFFFFFu;
            const uint32_t from = count_below(src, left, id0);
            left = count_below(src, left, id1) - from;
            src += from;
            pos += from;
        }
        double bd = INFINITY;
        int bi = 0x7FFFFFFF;
        int kept = 0;
        bool fresh = true;   // the wave's list is empty
        for (bool more = true; more;) {
            // ---- the window: `take` entries of every bin
            uint32_t take = left;
            more = wave_sum_i32((int)min(left, (uint32_t)kWinMax + 1u)) > kWinMax;
            if (more) {
                const uint32_t quota = (uint32_t)kWinMax / (uint32_t)__popcll(__ballot(left > 0));
                const uint32_t end = wave_min_u32(left > quota ? src[quota] : 0xFFFFFFFFu);
                take = count_below(src, min(left, quota), end);
            }
            const int incl = wave_incl_scan((int)take);
            const int n = __shfl(incl, 63);
            int lg = 6;
            while ((1 << lg) < 2 * n) ++lg;
            __syncthreads();   // the last window's list and table are no longer read
            if (wv == 0) {
                s_start[lane] = incl - (int)take;
                s_ofs[lane] = pos - (incl - (int)take);
            }
            for (int i = tid; i < (1 << lg); i += 256) s_key[i] = 0xFFFFFFFFu;
            if (t > 1)
                for (int i = tid; i < (1 << lg) / 4; i += 256) s_cnt[i] = 0u;
            if (tid == 0) s_nk = 0;
            __syncthreads();
            // ---- its entries into the table
            const uint32_t mask = (1u << lg) - 1u;
            for (int e = tid; e < n; e += 256) {
                int lo = 0, hi = L;   // the last bin that starts at or before e
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (s_start[mid] <= e) lo = mid;
                    else hi = mid;
                }
                const uint32_t id = tids[s_ofs[lo] + e];
                uint32_t slot = (id * 0x9E3779B1u) >> (32 - lg);
                uint32_t old;
                for (;;) {
                    old = atomicCAS(&s_key[slot], 0xFFFFFFFFu, id);
                    if (old == 0xFFFFFFFFu || old == id) break;
                    slot = (slot + 1u) & mask;
                }
                bool list = old == 0xFFFFFFFFu;
                if (t > 1) {
                    const int sh = 8 * (slot & 3u);
                    list = (int)((atomicAdd(&s_cnt[slot >> 2], 1u << sh) >> sh) & 0xFFu) == t - 1;
                }
                if (list) s_list[atomicAdd(&s_nk, 1)] = id;
            }
            __syncthreads();
            // ---- distances of the listed IDs
            const int nk = s_nk;
            kept += nk;
            for (int c0 = 64 * wv; c0 < nk; c0 += 256) {
                const bool act = c0 + lane < nk;
                const int id = act ? (int)s_list[c0 + lane] : 0;
                double d = 0.0;
                if (act) {
                    const float* row = xf + (int64_t)id * D;
                    auto term = [&](int i, float x) {
                        const double t0 = s_q[i] - (double)x;
                        d = d + t0 * t0;
                    };
                    if (D == 100) {
                        // a fifth of a row on its way at a time
                        const float4* r4 = reinterpret_cast<const float4*>(row);
#pragma unroll
                        for (int h = 0; h < 25; h += 5) {
                            float4 v[5];
#pragma unroll
                            for (int u = 0; u < 5; ++u)
                                if (h + u < 25) v[u] = r4[h + u];
                            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                            for (int u = 0; u < 5; ++u)
                                if (h + u < 25) {
                                    term(4 * (h + u), v[u].x);
                                    term(4 * (h + u) + 1, v[u].y);
                                    term(4 * (h + u) + 2, v[u].z);
                                    term(4 * (h + u) + 3, v[u].w);
                                }
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    } else {
                        float v[D];
#pragma unroll
                        for (int i = 0; i < D; ++i) v[i] = row[i];
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int i = 0; i < D; ++i) term(i, v[i]);
                    }
                    if (!(d == d)) d = INFINITY;   // not a number: last, by ID
                }
                if (fresh)
                    topk_first(min(64, nk - c0), d, id, K, s_td + wv * K, s_ti + wv * K, bd, bi);
                else
                    topk_insert(act, d, id, K, bd, bi);
                fresh = false;
            }
            pos += take;
            src += take;
            left -= take;
        }
        // ---- the K nearest of the waves' lists (up to 64 IDs: the first wave's)
        const bool merge = kept > 64;
        if (merge) {
            if (lane < K) {
                s_td[wv * K + lane] = bd;
                s_ti[wv * K + lane] = bi;
            }
            __syncthreads();
        }
        if (wv > 0) continue;
        if (merge) {
            const bool act = lane < 4 * K;
            const double d = act ? s_td[lane] : INFINITY;
            const int id = act ? s_ti[lane] : 0x7FFFFFFF;
            bd = INFINITY;
            bi = 0x7FFFFFFF;
            topk_first(4 * K, d, id, K, s_td, s_ti, bd, bi);
        }
        if (LISTS && shares > 1) {
            if (lane < K) {
                ll.d[(int64_t)item * K + lane] = bd;
                ll.id[(int64_t)item * K + lane] = bi;
            }
            if (lane == 0) ll.kept[item] = kept;
        } else {
            write_ranked(q, K, kept, bd, bi, counts, out_ids, out_d, out_m);
        }
    }
    if (LISTS && !longs) {
        __syncthreads();
        const int64_t q4 = (int64_t)4 * (blk - kLongBlocks) + wv;
        const int q = __builtin_amdgcn_readfirstlane((int)min(q4, (int64_t)Q));
        if (q < Q && !ll.listed[q])
            rank_few<D>(q, N, t, K, lane < L ? bins[(int64_t)lane * Q + q] : make_uint2(0u, 0u), tids, qfeat, xf, counts,
                        out_ids, out_d, out_m, reinterpret_cast<double*>(s_key) + wv * D, s_td + wv * kMaxK,
                        s_ti + wv * kMaxK);
    }
}

// The K nearest of a patch from its shares, a wave a patch (at its first share).
__global__ __launch_bounds__(64) void k_bins_join(int K, LongLists ll, int32_t* __restrict__ counts,
                                                  int32_t* __restrict__ out_ids, float* __restrict__ out_d,
                                                  int32_t* __restrict__ out_m) {
    __shared__ double s_td[kMaxK];
    __shared__ int s_ti[kMaxK];
    const int lane = threadIdx.x;
    const int n = (int)min(*ll.n, (unsigned)kLongMax);
    for (int i = blockIdx.x; i < n; i += gridDim.x) {
        const int2 it = ll.item[i];
        const int shares = it.y >> 5, cand = shares * K;
        if (it.x < 0 || shares == 1 || (it.y & 31)) continue;
        const int kept = wave_sum_i32(lane < shares ? ll.kept[i + lane] : 0);
        double bd = INFINITY;
        int bi = 0x7FFFFFFF;
        for (int c0 = 0; c0 < cand; c0 += 64) {
            const bool act = c0 + lane < cand;
            const double d = act ? ll.d[(int64_t)i * K + c0 + lane] : INFINITY;
            const int id = act ? ll.id[(int64_t)i * K + c0 + lane] : 0x7FFFFFFF;
            if (c0 == 0)
                topk_first(min(64, cand), d, id, K, s_td, s_ti, bd, bi);
            else
                topk_insert(act, d, id, K, bd, bi);
        }
        write_ranked(it.x, K, kept, bd, bi, counts, out_ids, out_d, out_m);
    }
}

// distances, IDs, patches and shares, counts, the other list, flags
size_t bins_rank_scratch(int64_t Q, int K) {
    if (Q < kLongMin) return 0;
    return (size_t)kLongMax * ((sizeof(double) + sizeof(int32_t)) * K + sizeof(int2) + sizeof(int32_t)) +
           (sizeof(int32_t) + 1) * (size_t)Q;
}

hipError_t launch_bins_rank(int Q, int L, int64_t N, int t, int D, int K, const uint2* bins, const uint32_t* tids,
                            const float* qfeat, const float* xf, int32_t* counts, int32_t* ids, float* d, int32_t* m,
                            unsigned int* counters, unsigned int* n_long, void* scratch, hipStream_t st) {
    if (Q == 0) return hipSuccess;
    if (L < 1 || L > 64 || t < 1 || t > L || K < 1 || K > kMaxK || (D != 25 && D != 100) ||
        (reinterpret_cast<uintptr_t>(xf) & 15) || !n_long)
        return hipErrorInvalidValue;
    LongLists ll{n_long, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
    if (!scratch || Q < kLongMin) {
        auto k = D == 100 ? k_bins_rank<100, false> : k_bins_rank<25, false>;
        hipLaunchKernelGGL(k, grid_rows(Q), dim3(256), 0, st, Q, L, N, t, K, bins, tids, qfeat, xf, counts, ids, d, m,
                           counters, ll);
        return hipGetLastError();
    }
    ll.d = static_cast<double*>(scratch);
    ll.item = reinterpret_cast<int2*>(ll.d + (size_t)kLongMax * K);
    ll.id = reinterpret_cast<int32_t*>(ll.item + kLongMax);
    ll.kept = ll.id + (size_t)kLongMax * K;
    ll.mid = ll.kept + kLongMax;
    ll.listed = reinterpret_cast<uint8_t*>(ll.mid + Q);
    hipLaunchKernelGGL(k_bins_long, dim3((Q + 255) / 256), dim3(256), 0, st, Q, L, bins, ll);
    auto k = D == 100 ? k_bins_rank<100, true> : k_bins_rank<25, true>;
    hipLaunchKernelGGL(k, grid_rows((int64_t)kLongBlocks + mid_blocks(Q)), dim3(256), 0, st, Q, L, N, t, K, bins, tids,
                       qfeat, xf, counts, ids, d, m, counters, ll);
    hipLaunchKernelGGL(k_bins_join, dim3(4096), dim3(64), 0, st, K, ll, counts, ids, d, m);
    return hipGetLastError();
}

hipError_t launch_cand_t(int Q, int L, int64_t N, int t, const uint2* bins, const uint32_t* tids, int cap,
                         int32_t* counts, int32_t* ids, hipStream_t st) {
    if (Q == 0) return hipSuccess;
    if (L < 1 || L > 64 || t < 1 || t > L || cap < 1) return hipErrorInvalidValue;
    if (!one_row(((int64_t)Q + 3) / 4, 256)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(k_cand_t, dim3((Q + 3) / 4), dim3(256), 0, st, Q, L, N, t, bins, tids, cap, counts, ids);
    return hipGetLastError();
}

}  // namespace zh
