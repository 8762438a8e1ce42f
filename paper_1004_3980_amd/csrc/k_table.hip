// Hash-table build (Section 3.2 and Section 4.1: the IDs of the training
// patches are stored in the bins of L tables, a bin being one k-tuple of
// codes, identified here by its 64-bit key).
//
// Every key is inserted into its table's open-addressing directory with
// linear probing (64-bit compare-and-swap), which gives each ID the slot of its
// bin. A stable LSD radix sort of (slot, ID) pairs, taken in ID order, lays the
// IDs out bin by bin with IDs ascending inside each bin; each run of a slot in
// the sorted order gives its bin's offset and size. Slot placement depends on
// insertion order, the bins' contents and their order do not. Several tables
// go through every kernel together. 24 tables of 300k rows: insertion 2.88 ->
// 0.60 ms (a counter and a compare-and-swap per row before), sort 2.89 -> 0.41
// ms (table by table, 8-bit digits, one workgroup's scan before), offsets 0.14
// -> 0.10 ms.
#include <algorithm>
#include <utility>

#include "zh_internal.h"

namespace zh {

static inline int grid_for(int64_t total, int block) {
    int64_t g = (total + block - 1) / block;
    if (g > 65536) g = 65536;
    return (int)(g < 1 ? 1 : g);
}

__global__ void k_dir_clear(Slot* __restrict__ dir, uint64_t count) {
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < count;
         i += (uint64_t)gridDim.x * blockDim.x) {
        Slot s;
        s.key = kEmptyKey;
        s.count = 0;
        s.offset = 0;
        dir[i] = s;
    }
}

// Keys of the rows of `tables` tables (blockIdx.y) into their directories. A
// slot is looked at before it is claimed: rows of a large bin (flat patches)
// then read its key from the cache instead of queueing on one address with
// compare-and-swaps (a key, once written, does not change; a stale empty slot
// only leads to the compare-and-swap). The bins' sizes come from the sorted
// slots (k_dir_offsets), not from a counter per slot.
__global__ __launch_bounds__(256) void k_dir_insert(const uint64_t* __restrict__ keys, int64_t n,
                                                    Slot* __restrict__ dir, uint64_t cap,
                                                    uint32_t* __restrict__ filter, uint32_t* __restrict__ slot_of) {
    const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (id >= n) return;
    const int64_t l = blockIdx.y;
    const uint64_t mask = cap - 1;
    Slot* dl = dir + (uint64_t)l * cap;
    const unsigned long long key = keys[l * n + id];
    uint64_t s = key & mask;
    // the directory holds at most n distinct keys in cap >= 2n slots, so
    // the probe ends within cap steps
    for (uint64_t step = 0; step < cap; ++step) {
        unsigned long long cur = dl[s].key;
        if (cur == kEmptyKey) {
            cur = atomicCAS(&dl[s].key, (unsigned long long)kEmptyKey, key);
            if (cur == kEmptyKey) {
                const uint32_t fb = dir_filter_bit(key, cap);
                atomicOr(filter + (uint64_t)l * dir_filter_words(cap) + (fb >> 5), 1u << (fb & 31));
                cur = key;
            }
        }
        if (cur == key) {
            slot_of[l * n + id] = (uint32_t)s;
            return;
        }
        s = (s + 1) & mask;
    }
}

// Offset and size of every bin from the sorted slots of a table (blockIdx.y):
// the first entry of a run finds its end by doubling steps and a binary search.
__global__ __launch_bounds__(256) void k_dir_offsets(const uint32_t* __restrict__ sorted_slot, int64_t n,
                                                     Slot* __restrict__ dir, uint64_t cap) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const uint32_t* v = sorted_slot + (int64_t)blockIdx.y * n;
    const uint32_t s = v[i];
    if (i > 0 && v[i - 1] == s) return;
    int64_t lo = i + 1, hi = n, step = 1;   // the end lies in [lo, hi]
    while (lo < hi) {
        const int64_t j = lo + step - 1;
        if (j >= hi) break;
        if (v[j] != s) {
            hi = j;
            break;
        }
        lo = j + 1;
        step <<= 1;
    }
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (v[mid] == s) lo = mid + 1;
        else hi = mid;
    }
    Slot* d = dir + (uint64_t)blockIdx.y * cap + s;
    d->count = (uint32_t)(lo - i);
    d->offset = (uint32_t)i;
}

hipError_t launch_dir_clear(Slot* dir, uint64_t count, hipStream_t st) {
    hipLaunchKernelGGL(k_dir_clear, dim3(grid_for((int64_t)count, 256)), dim3(256), 0, st, dir, count);
    return hipGetLastError();
}

hipError_t launch_dir_insert(const uint64_t* keys, int64_t n, int tables, Slot* dir, uint64_t cap, uint32_t* filter,
                             uint32_t* slot_of, hipStream_t st) {
    hipLaunchKernelGGL(k_dir_insert, dim3((unsigned)((n + 255) / 256), tables), dim3(256), 0, st, keys, n, dir, cap,
                       filter, slot_of);
    return hipGetLastError();
}

hipError_t launch_dir_offsets(const uint32_t* sorted_slot, int64_t n, int tables, Slot* dir, uint64_t cap,
                              hipStream_t st) {
    hipLaunchKernelGGL(k_dir_offsets, dim3((unsigned)((n + 255) / 256), tables), dim3(256), 0, st, sorted_slot, n, dir,
                       cap);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Stable LSD radix sort of one or several tables of (key, value) pairs at once,
// digits of up to 11 bits (two passes for 22 bits). A tile is 4096
// consecutive elements; each of the 4 waves of a tile owns 1024 consecutive
// elements, walked in 16 chunks of 64 in order, so ranks follow the input
// order (stability); its digit counters are its own, so the waves of a tile
// meet at two barriers only. A pass is a histogram of every tile, an exclusive
// scan over the tiles of each digit (a wave per digit), a scan over the
// digits and the scatter.
// ---------------------------------------------------------------------------
constexpr int kRsTile = 4096;
constexpr int kRsChunks = 16;
constexpr int kRsMaxBits = 11;

static int rs_passes(int bits) { return (bits + kRsMaxBits - 1) / kRsMaxBits; }
static int rs_width(int bits) { return bits < 1 ? 1 : (bits + rs_passes(bits) - 1) / rs_passes(bits); }
int64_t radix_hist_size(int64_t n, int tables, int bits) {
    const int64_t bins = 1ll << rs_width(bits), ntiles = (n + kRsTile - 1) / kRsTile;
    return (int64_t)tables * bins * (ntiles + 1);
}

// lanes of the wave holding the same digit of `width` bits (valid lanes only)
__device__ __forceinline__ uint64_t match_digit(uint32_t d, int width, bool valid) {
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < width; ++b) {
        const bool bit = (d >> b) & 1u;
        const uint64_t m = __ballot(bit);
        peers &= bit ? m : ~m;
    }
    return peers;
}

__global__ __launch_bounds__(256) void k_rs_hist(const uint32_t* __restrict__ key, int64_t n, int shift, int width,
                                                 uint32_t* __restrict__ hist, int ntiles) {
    extern __shared__ uint32_t rs_cnt[];
    const int bins = 1 << width;
    for (int d = threadIdx.x; d < bins; d += 256) rs_cnt[d] = 0;
    __syncthreads();
    key += (int64_t)blockIdx.y * n;
    const int64_t base = (int64_t)blockIdx.x * kRsTile;
#pragma unroll 4
    for (int t = threadIdx.x; t < kRsTile; t += 256) {
        const int64_t i = base + t;
        if (i < n) atomicAdd(&rs_cnt[(key[i] >> shift) & (uint32_t)(bins - 1)], 1u);
    }
    __syncthreads();
    uint32_t* h = hist + (int64_t)blockIdx.y * bins * ntiles;
    for (int d = threadIdx.x; d < bins; d += 256) h[(int64_t)d * ntiles + blockIdx.x] = rs_cnt[d];
}

// exclusive scan over the tiles of each digit in place, and the digit's total
__global__ __launch_bounds__(256) void k_rs_scan_tiles(uint32_t* __restrict__ hist, int64_t rows, int ntiles,
                                                       uint32_t* __restrict__ total) {
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= rows) return;
    uint32_t* v = hist + row * ntiles;
    uint32_t carry = 0;
    for (int t0 = 0; t0 < ntiles; t0 += 64) {
        const uint32_t x = t0 + lane < ntiles ? v[t0 + lane] : 0u;
        const uint32_t incl = (uint32_t)wave_incl_scan((int)x);
        if (t0 + lane < ntiles) v[t0 + lane] = carry + incl - x;
        carry += __shfl(incl, 63);
    }
    if (lane == 0) total[row] = carry;
}

// exclusive scan of a table's digit totals (at most 2048) in place
__global__ __launch_bounds__(256) void k_rs_scan_digits(uint32_t* __restrict__ total, int bins) {
    __shared__ uint32_t wsum[4];
    uint32_t* v = total + (int64_t)blockIdx.x * bins;
    const int t = threadIdx.x, per = (bins + 255) / 256;   // at most 8
    uint32_t x[8], sum = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        x[j] = j < per && t * per + j < bins ? v[t * per + j] : 0u;
        sum += x[j];
    }
    const uint32_t incl = (uint32_t)wave_incl_scan((int)sum);
    if ((t & 63) == 63) wsum[t >> 6] = incl;
    __syncthreads();
    uint32_t run = incl - sum;
    for (int w = 0; w < (t >> 6); ++w) run += wsum[w];
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (j < per && t * per + j < bins) {
            v[t * per + j] = run;
            run += x[j];
        }
}

// vin null: the value of an element is its index in its table
__global__ __launch_bounds__(256) void k_rs_scatter(const uint32_t* __restrict__ kin,
                                                    const uint32_t* __restrict__ vin, int64_t n,
                                                    int shift, int width, int mbits,
                                                    const uint32_t* __restrict__ hist,
                                                    const uint32_t* __restrict__ start, int ntiles,
                                                    uint32_t* __restrict__ kout, uint32_t* __restrict__ vout) {
    extern __shared__ uint32_t rs_cnt[];   // [4][bins]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int bins = 1 << width;
    const uint32_t dm = (1u << mbits) - 1u;
    const int64_t tb = (int64_t)blockIdx.y * n;
    kin += tb;
    kout += tb;
    vout += tb;
    if (vin) vin += tb;
    hist += (int64_t)blockIdx.y * bins * ntiles;
    start += (int64_t)blockIdx.y * bins;
    uint32_t* cnt = rs_cnt + wave * bins;
    for (int d = lane; d < bins; d += 64) cnt[d] = 0;
    const int64_t base = (int64_t)blockIdx.x * kRsTile + (int64_t)wave * (kRsChunks * 64);
    uint32_t k[kRsChunks];
#pragma unroll
    for (int c = 0; c < kRsChunks; ++c) {
        const int64_t i = base + c * 64 + lane;
        k[c] = i < n ? kin[i] : 0u;
    }
    // digit counts of the wave
#pragma unroll
    for (int c = 0; c < kRsChunks; ++c)
        if (base + c * 64 + lane < n) atomicAdd(&cnt[(k[c] >> shift) & dm], 1u);
    __syncthreads();
    // running start of each wave's run of every digit
    for (int d = threadIdx.x; d < bins; d += 256) {
        uint32_t run = hist[(int64_t)d * ntiles + blockIdx.x] + start[d];
        for (int w = 0; w < 4; ++w) {
            const uint32_t c = rs_cnt[w * bins + d];
            rs_cnt[w * bins + d] = run;
            run += c;
        }
    }
    __syncthreads();
    // stable scatter: the wave's LDS operations stay in order
#pragma unroll
    for (int c = 0; c < kRsChunks; ++c) {
        const int64_t i = base + c * 64 + lane;
        const bool valid = i < n;
        const uint32_t d = (k[c] >> shift) & dm;
        const uint64_t peers = match_digit(d, mbits, valid);
        const uint64_t before = peers & lanemask_lt();
        if (valid) {
            const uint32_t at = cnt[d];
            const uint32_t pos = at + (uint32_t)__popcll(before);
            kout[pos] = k[c];
            vout[pos] = vin ? vin[i] : (uint32_t)i;
            if (before == 0) cnt[d] = at + (uint32_t)__popcll(peers);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

hipError_t radix_sort_pairs(uint32_t* k0, uint32_t* k1, uint32_t* v0, uint32_t* v1, bool index_values, int64_t n,
                            int tables, int bits, uint32_t* hist, int64_t hist_cap, hipStream_t st,
                            uint32_t** keys_out, uint32_t** vals_out) {
    const int width = rs_width(bits);
    const int bins = 1 << width;
    const int64_t ntiles = (n + kRsTile - 1) / kRsTile;
    if (bits < 1 || bits > 32 || n < 1 || tables < 1 || ntiles > 0x7FFFFFFF ||
        radix_hist_size(n, tables, bits) > hist_cap)
        return hipErrorInvalidValue;
    const int64_t rows = (int64_t)tables * bins;
    uint32_t* total = hist + rows * ntiles;
    const int passes = (bits + width - 1) / width;
    // the values of the last pass, and of every second before it, go to `last`
    uint32_t* const last = index_values || passes % 2 == 0 ? v0 : v1;
    uint32_t *kin = k0, *kout = k1, *vin = index_values ? nullptr : v0;
    const dim3 grid((unsigned)ntiles, tables);
    for (int p = 0; p < passes; ++p) {
        const int shift = p * width;
        const int wd = bits - shift < width ? bits - shift : width;   // bins past 2^wd stay empty
        uint32_t* vout = (passes - 1 - p) % 2 == 0 ? last : last == v0 ? v1 : v0;
        hipLaunchKernelGGL(k_rs_hist, grid, dim3(256), sizeof(uint32_t) * bins, st, kin, n, shift, width, hist,
                           (int)ntiles);
        hipLaunchKernelGGL(k_rs_scan_tiles, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st, hist, rows, (int)ntiles,
                           total);
        hipLaunchKernelGGL(k_rs_scan_digits, dim3(tables), dim3(256), 0, st, total, bins);
        hipLaunchKernelGGL(k_rs_scatter, grid, dim3(256), sizeof(uint32_t) * 4 * bins, st, kin, vin, n, shift, width, wd,
                           hist, total, (int)ntiles, kout, vout);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        std::swap(kin, kout);
        vin = vout;
    }
    *keys_out = kin;
    *vals_out = vin;
    return hipSuccess;
}

// Content hash of n 32-bit words for the table files: the sum over i of
// fmix64((i G + salt) ^ w_i) mod 2^64, G the SplitMix64 increment. Integer sums do not depend on their
// order, so the value is the same for every launch shape; it changes with any
// word and with its position.
__global__ __launch_bounds__(256) void k_hash_words(const uint32_t* __restrict__ p, int64_t n, uint64_t salt,
                                                    unsigned long long* __restrict__ out) {
    uint64_t acc = 0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        acc += fmix64(((uint64_t)i * kGolden + salt) ^ (uint64_t)p[i]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    __shared__ unsigned long long wsum[4];
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = acc;
    __syncthreads();
    // one atomic a workgroup, few workgroups: they queue on one address (an
    // atomic a wave of 65,536 workgroups took 3.1 ms on 120 MB, 0.05 now)
    if (threadIdx.x == 0) atomicAdd(out, wsum[0] + wsum[1] + wsum[2] + wsum[3]);
}

hipError_t launch_hash_words(const void* p, int64_t n_words, uint64_t salt, unsigned long long* out,
                             hipStream_t st) {
    if (n_words == 0) return hipSuccess;
    hipLaunchKernelGGL(k_hash_words, dim3((unsigned)std::min<int64_t>((n_words + 255) / 256, 2048)), dim3(256), 0, st,
                       static_cast<const uint32_t*>(p), n_words, salt, out);
    return hipGetLastError();
}

}  // namespace zh
