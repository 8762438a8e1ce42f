// Projection, p-stable codes, bucket keys and bin lookup (Section 4.1,
// Eq. hash_fn; Section 3.2: k concatenated hashes per table, L tables).
//
//   code_j(v) = floor((alpha_j . v + beta_j) / w)
//
// A wave owns 16 or 32 feature rows and runs over all tables. The dot
// products of its rows with the k hashes of a table run on the matrix cores,
// either as fp32 MFMA (P = (alpha.v + beta) / w evaluated as written) or as
// three bf16 MFMAs over a high/low split of both operands, with alpha / w
// and beta / w rounded to fp32 beforehand (a' = alpha / w = a_hi + a_lo,
// v = v_hi + v_lo; a_hi v_hi + a_hi v_lo + a_lo v_hi accumulate in fp32 and
// P = S + beta / w); the split of the wave's rows stays in registers for all
// tables. A fourth product of the absolute values bounds
// sum_i |a'_i v_i|, which gives a rigorous bound B on |P_mfma - P_exact|;
// when [P - B, P + B] holds no integer the MFMA floor is the exact code,
// otherwise the code is recomputed by the FP64 sequential dot product that
// defines it (in a second kernel, for the few tables that need it). The
// codes therefore equal the FP64 definition bit for bit.
//
// The k codes of a table become a 64-bit key
//   key = fmix64( M_l63 + sum_j uint32(c_j) * M_lj  mod 2^64 ),
// M_lj = SplitMix64 output 64 l + j + 1 from state 0 (table a.key_mul: k
// multipliers and the start value M_l63 per table), and,
// when a directory is given, a third kernel looks up each key's bin
// (offset, count).
#include <algorithm>
#include <cmath>

#include "zh_internal.h"

namespace zh {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));

constexpr int kRowsPerWave = 16;
constexpr uint32_t kFixDirty = 0x80000000u;   // in a region's entry count: rows with a dirty mask
constexpr int64_t kHashBlocks = 512;          // workgroups of k_hash that keep the chip full: two a compute unit

__device__ __forceinline__ int32_t floor_sat(double t) {
    const double f = floor(t);
    if (f >= 2147483647.0) return 2147483647;
    if (f <= -2147483648.0) return (int32_t)0x80000000;
    return (int32_t)f;
}

// floor(x) as int32 in one instruction (x of magnitude below 2^31)
__device__ __forceinline__ int32_t cvt_floor(float x) {
    int32_t r;
    asm volatile("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

// Walk the directory from slot s on (linear probing) to the key or an empty
// slot; (off, cnt) stay 0 for an absent key.
__device__ __forceinline__ void probe_bin_from(const Slot* __restrict__ dir, uint64_t cap, uint64_t key, uint64_t s,
                                               uint32_t& off, uint32_t& cnt) {
    const uint64_t mask = cap - 1;
    off = 0;
    cnt = 0;
    for (uint64_t step = 0; step < cap; ++step) {
        const uint4 e = *reinterpret_cast<const uint4*>(dir + s);
        const uint64_t k = ((uint64_t)e.y << 32) | e.x;
        if (k == key) {
            cnt = e.z;
            off = e.w;
            return;
        }
        if (k == kEmptyKey) return;
        s = (s + 1) & mask;
    }
}

constexpr int kWaves = 4;         // waves per workgroup

// The hash rows of all tables in MFMA tiles of 16: table l has k4 rows (its k
// hashes, padded to a multiple of four and to at least eight), row r of the
// padded list belongs to hash r % k4 of table r / k4. The four rows that a lane
// holds of a tile's result then belong to one table, and a tile to at most two.
__host__ __device__ inline int padded_hashes(int k) { return k <= 8 ? 8 : (k + 3) & ~3; }
inline int hash_tiles(int L, int k) { return (L * padded_hashes(k) + 15) / 16; }

// A tile as it lies in LDS, and in the dictionary's image of it (laid out once
// with the tables, so that a stage is copied as it is): the operand rows, the
// rows of block norms, then of its 16 rows beta, the constant term of the error
// bound, and the low and high halves of the key multiplier. Operand rows: fp32 path
// the coordinates, padded to whole steps of four and an odd number of words;
// split path the high plane and the low plane, each row a whole number of
// 32-coordinate steps and one 16-byte chunk (an odd number of chunks: the
// 16-byte reads of eight consecutive rows fall on distinct banks).
// Split path, D = 100: the last four coordinates would fill a step of 32 to an
// eighth in each of the three products, so one step takes all three:
// (hi, hi, lo) of the hash row in the high plane against (hi, lo, hi) of the
// feature row.
// Block norms: 32 bf16 values a row, rounded up, the norms of blocks of four of
// its coordinates (D = 25: the absolute values), for the bound's MFMA. The
// eight slots 8 kb .. 8 kb + 7 are blocks of coordinates that lane kb holds of
// a feature row (block_of), so its norms need no exchange.
template <int PREC, int D>
struct HashTile {
    static constexpr int TAIL = PREC == 1 && D % 32 == 4 ? 4 : 0;
    static constexpr int NS = PREC == 1 ? (D + 31) / 32 - (TAIL ? 1 : 0) : (D + 3) / 4;   // full steps
    static constexpr int HS = PREC == 1 ? 32 * (NS + (TAIL ? 1 : 0)) + 8 : 0;             // halfwords of a high row
    static constexpr int LS = PREC == 1 ? 32 * NS + 8 : 0;                                // halfwords of a low row
    static constexpr int FS = PREC == 0 ? (4 * NS) | 1 : 0;                               // words of an fp32 row
    static constexpr int LO = 16 * HS * 2;                  // offset of the low plane
    static constexpr int NORM = PREC == 1 ? LO + 16 * LS * 2 : 16 * FS * 4;    // offset of the block norms
    static constexpr int TERMS = NORM + 16 * 40 * 2;        // offset of the 16-row terms
    static constexpr int BYTES = TERMS + 4 * 64;
    static constexpr int G = D > 32 ? 2 : 4;                // tiles of a stage
    static constexpr int SB = (G * BYTES + 4095) & ~4095;   // bytes of a stage: whole 1 KB wave copies of four waves
    static_assert(BYTES % 16 == 0 && NORM % 16 == 0, "16-byte rows");
    // slot of the block norms that coordinate d belongs to
    __host__ __device__ static constexpr int block_of(int d) {
        return PREC == 0     ? 8 * (d % 4) + (D > 32 ? d / 16 : d / 4)
               : D <= 32     ? d
               : d < 32 * NS ? 8 * (d % 32 / 8) + 2 * (d / 32) + d % 8 / 4
                             : 6;
    }
};
// bf16 of x >= 0, rounded up
__device__ __forceinline__ uint16_t bf16_up(float x) { return (uint16_t)((__float_as_uint(x) + 0xFFFFu) >> 16); }

// The image of every tile, one workgroup a tile.
template <int PREC, int D>
__global__ __launch_bounds__(256) void k_hash_image(const float* __restrict__ alpha, const float* __restrict__ beta,
                                                    const uint16_t* __restrict__ a_hi, const uint16_t* __restrict__ a_lo,
                                                    const float* __restrict__ c0, const uint64_t* __restrict__ key_mul,
                                                    float w, int L, int k, unsigned char* __restrict__ img) {
    using HT = HashTile<PREC, D>;
    constexpr int DP = (D + 31) & ~31;
    const int k4 = padded_hashes(k);
    unsigned char* T = img + (int64_t)(blockIdx.x / HT::G) * HT::SB + (blockIdx.x % HT::G) * HT::BYTES;
    const int r0 = 16 * blockIdx.x;
    // hash row of padded row r, or -1
    auto hash_row = [&](int r) {
        const int l = (r0 + r) / k4, j = (r0 + r) - l * k4;
        return l < L && j < k ? l * k + j : -1;
    };
    if (PREC == 0) {
        float* f = reinterpret_cast<float*>(T);
        for (int e = threadIdx.x; e < 16 * HT::FS; e += 256) {
            const int r = e / HT::FS, c = e - r * HT::FS, hr = hash_row(r);
            f[e] = hr >= 0 && c < D ? alpha[(int64_t)hr * D + c] : 0.0f;
        }
    } else {
        uint16_t* hi = reinterpret_cast<uint16_t*>(T);
        uint16_t* lo = reinterpret_cast<uint16_t*>(T + HT::LO);
        for (int e = threadIdx.x; e < 16 * HT::HS; e += 256) {
            const int r = e / HT::HS, c = e - r * HT::HS, hr = hash_row(r);
            uint16_t v = 0;
            if (hr >= 0) {
                const uint16_t* h = a_hi + (int64_t)hr * DP;
                if (c < 32 * HT::NS)
                    v = h[c];
                else if (HT::TAIL && c < 32 * HT::NS + 12) {
                    const int q = c - 32 * HT::NS, d = 32 * HT::NS + (q & 3);
                    v = q < 8 ? h[d] : a_lo[(int64_t)hr * DP + d];
                }
            }
            hi[e] = v;
        }
        for (int e = threadIdx.x; e < 16 * HT::LS; e += 256) {
            const int r = e / HT::LS, c = e - r * HT::LS, hr = hash_row(r);
            lo[e] = hr >= 0 && c < 32 * HT::NS ? a_lo[(int64_t)hr * DP + c] : (uint16_t)0;
        }
    }
    uint16_t* nb = reinterpret_cast<uint16_t*>(T + HT::NORM);
    __shared__ double sq[16 * D];   // squares of the rows
    for (int e = threadIdx.x; e < 16 * D; e += 256) {
        const int r = e / D, hr = hash_row(r);
        const double v = hr >= 0 ? (double)alpha[(int64_t)hr * D + e - r * D] / (PREC == 1 ? (double)w : 1.0) : 0.0;
        sq[e] = v * v;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 16 * 40; e += 256) {
        const int r = e / 40, c = e - r * 40;
        double ss = 0.0;
        for (int d = 0; d < D; ++d)
            if (HT::block_of(d) == c) ss = ss + sq[r * D + d];
        nb[e] = bf16_up((float)(sqrt(ss) * (1.0 + 1e-6)));
    }
    // A padded row has beta = 1/2 and bound 0 (never uncertain) and multiplier 0.
    if (threadIdx.x < 16) {
        const int r = threadIdx.x, hr = hash_row(r);
        float* f = reinterpret_cast<float*>(T + HT::TERMS);
        uint32_t* u = reinterpret_cast<uint32_t*>(f + 32);
        f[r] = hr < 0 ? 0.5f * (PREC == 1 ? 1.0f : w) : PREC == 1 ? beta[hr] / w : beta[hr];
        f[16 + r] = hr < 0 ? 0.0f : c0[hr];
        const int l = (r0 + r) / k4, j = (r0 + r) - l * k4;
        const uint64_t m = hr < 0 ? 0ull : key_mul[l * (k + 1) + j];
        u[r] = (uint32_t)m;
        u[16 + r] = (uint32_t)(m >> 32);
    }
}

// A wave owns RT tiles of 16 feature rows, held in registers as MFMA operands,
// and runs over the hash tiles of all tables, staged through LDS two stages
// deep by copies that go past the registers and shared by the four waves.
// PREC 0: fp32 MFMA (4 coordinates a step); PREC 1: split bf16 (32 a step).
//
// A code whose interval [P - B, P + B] holds an integer is left to the FP64
// definition: it counts as zero in the key sum here, and the table goes to a
// compact list (row, table, mask of its uncertain codes, key sum of the
// others) for k_hash_fix, or, when the list is full, the table's bit is set in
// the row's dirty mask. The list has a region of fix_cap entries per 16
// feature rows.
//
// The sum of a table's key terms is formed where the codes are, a lane four
// of them, and the lanes' sums of a pair of tables meet in two exchanges, so
// the codes pass through no memory unless they are asked for.
//
// B = c1 S_abs + c0, S_abs >= sum |a_i v_i|: one MFMA of the block norms (Cauchy
// and Schwarz in each block; the whole rows' norms leave four times the codes
// open). A product of all absolute values took four MFMAs and the forming of
// |v| at each step.
//
// Bound: instruction issue: a third MFMA (11 for 16 hashes of 16 rows at D =
// 100), the rest the codes, their bounds and key terms (two 64-bit
// multiply-adds a code at a quarter of the rate). D = 100, L = 24, k = 20
// before (codes through LDS, alpha through registers for a pair of tables at a
// time, the product of the absolute values, an atomic a wave) and now: 1040400
// rows 973 us and 512, 70001 rows with their codes 160 and 61, 24236 rows 45
// (without the atomics' wait 32) and 25.
template <int PREC, int D, int RT, bool CODES>
__global__ __launch_bounds__(256, 3) void k_hash(HashArgs a) {
    using HT = HashTile<PREC, D>;
    constexpr int NS = HT::NS, TAIL = HT::TAIL, RPW = kRowsPerWave * RT;
    const int k = a.k, L = a.L, m = L * k, k4 = padded_hashes(k);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ri = lane & 15, kb = lane >> 4;
    const int64_t r0 = ((int64_t)blockIdx.x * kWaves + wave) * RPW;
    __shared__ __align__(16) unsigned char sA[2 * HT::SB];
    __shared__ uint32_t sUall[kWaves * 4 * RPW];    // per wave: uncertain codes of (table % 4, row)
    uint32_t* sU = sUall + wave * 4 * RPW;
    for (int e = lane; e < 4 * RPW; e += 64) sU[e] = 0;
    __shared__ uint64_t sStart[kMaxL];              // start value of each table's key sum
    if ((int)threadIdx.x < L) sStart[threadIdx.x] = a.key_mul[threadIdx.x * (k + 1) + k];

    // the stages of this part of the tables: a part begins at an even table
    const int ntiles = (L * k4 + 15) / 16, nst = (ntiles + HT::G - 1) / HT::G;
    const int st0 = (int)blockIdx.y * a.part_stages;
    const int st1 = st0 + a.part_stages < nst ? st0 + a.part_stages : nst;
    auto fetch = [&](int st) {
        const unsigned char* src = a.img + (int64_t)st * HT::SB;
        unsigned char* dst = sA + (st & 1) * HT::SB;
#pragma unroll
        for (int c = 0; c < HT::SB / 4096; ++c) {
            const int o = (c * kWaves + wave) * 1024;
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void*)(src + o + 16 * lane),
                (__attribute__((address_space(3))) void*)(dst + o), 16, 0, 0);
        }
    };
    fetch(st0);

    // B operands of the wave's rows, and their block norms
    u16x8 bh[RT][PREC == 1 ? NS : 1], bl[RT][PREC == 1 ? NS : 1], bt[RT], bn[RT];
    float bf[PREC == 0 ? NS : 1];
    bool rowok[RT];
    const bool vec = D % 32 == TAIL && (reinterpret_cast<uintptr_t>(a.feat) & 15) == 0;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const int64_t row = r0 + 16 * rt + ri;
        rowok[rt] = row < a.n;
        // rows past the last take the last's values: their codes go nowhere
        const float* fr = a.feat + (rowok[rt] ? row : a.n - 1) * D;
        // squares of a block, rounded up past the errors of the sum; squares that
        // underflow add up to a norm below 1e-18
        auto norm = [](float ss) { return bf16_up(__builtin_amdgcn_sqrtf(ss) * 1.00001f + 1e-18f); };
        bn[rt] = u16x8{0, 0, 0, 0, 0, 0, 0, 0};
        if (PREC == 1) {
            float x[NS][8], xt[4] = {0.f, 0.f, 0.f, 0.f};
            if (vec) {   // rows on 16-byte boundaries: 16-byte loads
#pragma unroll
                for (int s = 0; s < NS; ++s)
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const float4 v = *reinterpret_cast<const float4*>(fr + 32 * s + 8 * kb + 4 * j);
                        x[s][4 * j] = v.x, x[s][4 * j + 1] = v.y, x[s][4 * j + 2] = v.z, x[s][4 * j + 3] = v.w;
                    }
                if (TAIL) {
                    const float4 v = *reinterpret_cast<const float4*>(fr + 32 * NS);
                    xt[0] = v.x, xt[1] = v.y, xt[2] = v.z, xt[3] = v.w;
                }
            } else {
#pragma unroll
                for (int s = 0; s < NS; ++s)
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int d = 32 * s + 8 * kb + e;
                        const float v = fr[d < D ? d : 0];
                        x[s][e] = d < D ? v : 0.0f;
                    }
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (TAIL) xt[e] = fr[32 * NS + e];
            }
            // high part: x rounded to bf16 (nearest even); low part: the exact
            // remainder rounded likewise
            bf16x8 hv, lv;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    hv[e] = (__bf16)x[s][e];
                    lv[e] = (__bf16)(x[s][e] - (float)hv[e]);
                }
                if (D <= 32) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) bn[rt][e] = bf16_up(fabsf(x[s][e]));
                } else {
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const float* y = x[s] + 4 * j;
                        bn[rt][(2 * s + j) & 7] = norm(fmaf(y[0], y[0], fmaf(y[1], y[1], fmaf(y[2], y[2], y[3] * y[3]))));
                    }
                }
                bh[rt][s] = __builtin_bit_cast(u16x8, hv);
                bl[rt][s] = __builtin_bit_cast(u16x8, lv);
            }
            if (TAIL) {
                // slots 0..3 the high parts, 4..7 the low parts, 8..11 the high parts
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const __bf16 h = (__bf16)xt[e];
                    const __bf16 l = (__bf16)(xt[e] - (float)h);
                    hv[e] = kb < 2 ? h : (__bf16)0.0f;
                    hv[4 + e] = kb == 0 ? l : (__bf16)0.0f;
                }
                if (kb == 0)
                    bn[rt][6] = norm(fmaf(xt[0], xt[0], fmaf(xt[1], xt[1], fmaf(xt[2], xt[2], xt[3] * xt[3]))));
                bt[rt] = __builtin_bit_cast(u16x8, hv);
            }
        } else {
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const int d = 4 * s + kb;
                const float v = fr[d < D ? d : 0];
                bf[s] = d < D ? v : 0.0f;
            }
            constexpr int BS = D > 32 ? 4 : 1;
#pragma unroll
            for (int b = 0; b < (NS + BS - 1) / BS; ++b) {
                float ss = 0.0f;
#pragma unroll
                for (int s = BS * b; s < NS && s < BS * (b + 1); ++s) ss = fmaf(bf[s], bf[s], ss);
                bn[rt][b & 7] = norm(ss);
            }
        }
    }
    const float c1 = a.bound_c1, c2 = a.bound_c2;
    const uint32_t kmask = k < 32 ? (1u << k) - 1u : ~0u;
    const bool cvec = (k & 3) == 0 && (reinterpret_cast<uintptr_t>(a.codes) & 15) == 0;

    // fix-list regions of the wave: one per 16 rows and part
    const int64_t w16 = (int64_t)blockIdx.y * ((a.n + kRowsPerWave - 1) / kRowsPerWave) + r0 / kRowsPerWave;
    uint64_t dirty = 0;
    unsigned nflag = 0, marked = 0;      // marked: tables (mod 4) with a mark in sU
    unsigned wcnt[RT];
    uint64_t h[3][RT];                   // key sums of the tables 2 p, 2 p + 1, 2 p + 2
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        wcnt[rt] = 0;
        h[0][rt] = h[1][rt] = h[2][rt] = 0;
    }
    // Keys of the pair of tables 2 p, 2 p + 1: the sums over the four lanes of
    // a row (kb = 0..3), a lane for each (row tile, table): with two row tiles
    // the lanes kb < 2 end with the first tile and odd kb with the second
    // table, with one the lanes kb >= 2 with the second table (and odd kb idle).
    auto flush = [&](int p) {
        uint64_t sum;
        if (RT == 2) {
            uint64_t s2[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const uint64_t send = kb < 2 ? h[t][RT - 1] : h[t][0];
                s2[t] = (kb < 2 ? h[t][0] : h[t][RT - 1]) + __shfl_xor((unsigned long long)send, 32);
            }
            const uint64_t send = kb & 1 ? s2[0] : s2[1];
            sum = (kb & 1 ? s2[1] : s2[0]) + __shfl_xor((unsigned long long)send, 16);
        } else {
            const uint64_t send = kb < 2 ? h[1][0] : h[0][0];
            sum = (kb < 2 ? h[0][0] : h[1][0]) + __shfl_xor((unsigned long long)send, 32);
            sum += __shfl_xor((unsigned long long)sum, 16);
        }
        const int t = RT == 2 ? kb & 1 : kb >> 1;
        const int rr = RT == 2 ? (kb >> 1) * 16 + ri : ri;
        const int lt = 2 * p + t;
        const int64_t row = r0 + rr;
        const bool act = lt < L && row < a.n && (RT == 2 || !(kb & 1));
        if (act) {
            sum += sStart[lt];
            a.keys[key_pos(a, row, lt)] = key_final(sum);
        }
        const unsigned pm = 3u << (2 * (p & 1));
        if (marked & pm) {
            marked &= ~pm;
            uint32_t* mp = sU + (lt & 3) * RPW + rr;
            const uint32_t um = act ? *mp : 0;
            const uint64_t bal = __ballot(um != 0);
            const uint64_t regmask = RT == 1 ? ~0ull : (kb < 2 ? 0xFFFFFFFFull : 0xFFFFFFFF00000000ull);
            if (um) {
                *mp = 0;
                const int reg = rr >> 4;
                const int idx = (int)wcnt[RT == 1 ? 0 : reg] + __popcll(bal & regmask & lanemask_lt());
                if (idx < a.fix_cap)
                    a.fix_list[(w16 + reg) * a.fix_cap + idx] =
                        make_uint4((uint32_t)lt | ((uint32_t)ri << 8), um, (uint32_t)sum, (uint32_t)(sum >> 32));
                else
                    dirty |= 1ull << lt;
            }
            wcnt[0] += (unsigned)__popcll(RT == 1 ? bal : bal & 0xFFFFFFFFull);
            if (RT == 2) wcnt[RT - 1] += (unsigned)__popcll(bal >> 32);
        }
    };

    // the table of the tile's first row, and that row's place in it
    int tlo = st0 * (16 * HT::G) / k4, rem = 0;
    for (int st = st0; st < st1; ++st) {
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the wave's part of the stage is in LDS
        __syncthreads();                      // everyone's part; the other buffer is no longer read
        const int ng = ntiles - st * HT::G < HT::G ? ntiles - st * HT::G : HT::G;
        for (int tt = 0; tt < ng; ++tt) {
            const unsigned char* T = sA + (st & 1) * HT::SB + tt * HT::BYTES;
            f32x4 cs[RT], cab[RT];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) cs[rt] = f32x4{0.f, 0.f, 0.f, 0.f};
            const bf16x8 an = *reinterpret_cast<const bf16x8*>(T + HT::NORM + 80 * ri + 16 * kb);
            auto norms = [&]() {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                    cab[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(an, __builtin_bit_cast(bf16x8, bn[rt]),
                                                                      f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            };
            if (PREC == 1) {
                // the split products share one fp32 accumulator: the bound
                // covers any order of the additions
                const uint16_t* Ah = reinterpret_cast<const uint16_t*>(T) + ri * HT::HS + 8 * kb;
                const uint16_t* Al = reinterpret_cast<const uint16_t*>(T + HT::LO) + ri * HT::LS + 8 * kb;
                bf16x8 ah[NS], al[NS], at;
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    ah[s] = *reinterpret_cast<const bf16x8*>(Ah + 32 * s);
                    al[s] = *reinterpret_cast<const bf16x8*>(Al + 32 * s);
                }
                if (TAIL) at = *reinterpret_cast<const bf16x8*>(Ah + 32 * NS);
                norms();
#pragma unroll
                for (int s = 0; s < NS; ++s) {
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
                        cs[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            ah[s], __builtin_bit_cast(bf16x8, bh[rt][s]), cs[rt], 0, 0, 0);
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
                        cs[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            ah[s], __builtin_bit_cast(bf16x8, bl[rt][s]), cs[rt], 0, 0, 0);
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
                        cs[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            al[s], __builtin_bit_cast(bf16x8, bh[rt][s]), cs[rt], 0, 0, 0);
                }
                if (TAIL) {
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
                        cs[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(at, __builtin_bit_cast(bf16x8, bt[rt]),
                                                                         cs[rt], 0, 0, 0);
                }
            } else {
                const float* Af = reinterpret_cast<const float*>(T) + ri * HT::FS + kb;
                float af[NS];
#pragma unroll
                for (int s = 0; s < NS; ++s) af[s] = Af[4 * s];
                norms();
#pragma unroll
                for (int s = 0; s < NS; ++s) cs[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[s], bf[s], cs[0], 0, 0, 0);
            }
            // 16x16 tile: lane holds hash rows 4 kb + i of the tile, feature row ri
            const float* tf = reinterpret_cast<const float*>(T + HT::TERMS) + 4 * kb;
            const float4 be = *reinterpret_cast<const float4*>(tf);
            const float4 b0 = *reinterpret_cast<const float4*>(tf + 16);
            const uint4 ml = *reinterpret_cast<const uint4*>(tf + 32);
            const uint4 mh = *reinterpret_cast<const uint4*>(tf + 48);
            const float bev[4] = {be.x, be.y, be.z, be.w}, b0v[4] = {b0.x, b0.y, b0.z, b0.w};
            const uint32_t mlv[4] = {ml.x, ml.y, ml.z, ml.w}, mhv[4] = {mh.x, mh.y, mh.z, mh.w};
            // the next stage is called for after the last reads of this one: a read
            // of LDS waits for every copy into it
            __builtin_amdgcn_sched_barrier(0);
            if (tt == ng - 1 && st + 1 < st1) fetch(st + 1);
            __builtin_amdgcn_sched_barrier(0);
            const int o = rem + 4 * kb;
            const bool first = o < k4;
            const int j0 = first ? o : o - k4;      // first of the lane's four hashes in its table
            uint64_t hs[RT];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                int32_t c[4];
                bool f[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float S = cs[rt][i];
                    // split path: alpha and beta came divided by w
                    const float P = PREC == 1 ? S + bev[i] : (S + bev[i]) * a.inv_w;
                    const float B = PREC == 1 ? fmaf(c1, cab[rt][i], b0v[i])
                                              : fmaf(c1, cab[rt][i], fmaf(c2, fabsf(S), b0v[i]));
                    // uncertain when an integer lies within B of P; every P of
                    // magnitude >= 2^23 is an integer, so each certain code has
                    // |floor(P)| <= 2^23 (a NaN P or B is uncertain as well)
                    f[i] = !(fabsf(P - rintf(P)) > B);
                    c[i] = cvt_floor(P);
                }
                if (__ballot(f[0]) | __ballot(f[1]) | __ballot(f[2]) | __ballot(f[3])) {
                    const int lt = tlo + (first ? 0 : 1);
                    uint32_t um = 0;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        um |= f[i] ? 1u << i : 0u;
                        c[i] = f[i] ? 0 : c[i];
                    }
                    um = (um << j0) & kmask;
                    if (!rowok[rt] || lt >= L) um = 0;
                    if (um) {
                        atomicOr(&sU[(lt & 3) * RPW + 16 * rt + ri], um);
                        nflag += (unsigned)__popc(um);
                    }
                    marked |= (1u << (tlo & 3)) | (1u << ((tlo + 1) & 3));
                }
                uint64_t s1 = 0;
                uint32_t s2 = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    s1 += (uint64_t)(uint32_t)c[i] * mlv[i];
                    s2 += (uint32_t)c[i] * mhv[i];
                }
                hs[rt] = s1 + ((uint64_t)s2 << 32);
                if (CODES && rowok[rt] && tlo + (first ? 0 : 1) < L) {
                    int32_t* cd = a.codes + (r0 + 16 * rt + ri) * m + (tlo + (first ? 0 : 1)) * k + j0;
                    if (cvec) {
                        if (j0 < k) *reinterpret_cast<int4*>(cd) = make_int4(c[0], c[1], c[2], c[3]);
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (j0 + i < k) cd[i] = c[i];
                    }
                }
            }
            // to the tables' sums (tlo is one table for the wave)
            if (rem + 16 <= k4) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    if (tlo & 1)
                        h[1][rt] += hs[rt];
                    else
                        h[0][rt] += hs[rt];
                }
            } else {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    const uint64_t x = first ? hs[rt] : 0, y = first ? 0 : hs[rt];
                    if (tlo & 1) {
                        h[1][rt] += x;
                        h[2][rt] += y;
                    } else {
                        h[0][rt] += x;
                        h[1][rt] += y;
                    }
                }
            }
            rem += 16;
            const int told = tlo;
            while (rem >= k4) {
                rem -= k4;
                ++tlo;
            }
            if ((tlo >> 1) != (told >> 1)) {
                flush(told >> 1);
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    h[0][rt] = h[2][rt];
                    h[1][rt] = h[2][rt] = 0;
                }
            }
        }
    }
    // an odd table count leaves the last table alone in its pair
    if (st1 == nst && (L & 1) && (tlo >> 1) == (L >> 1)) flush(L >> 1);
    // tables that did not fit in the list: the lanes of a row together
    if (RT == 2)
        dirty |= __shfl_xor((unsigned long long)dirty, 16);
    else
        dirty |= __shfl_xor((unsigned long long)dirty, 32);
    const uint64_t db = __ballot(dirty != 0);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const bool any = RT == 1 ? db != 0 : ((db >> (32 * rt)) & 0xFFFFFFFFull) != 0;
        const int64_t row = r0 + 16 * rt + ri;
        if (any && kb == 2 * rt && row < a.n) a.dirty[(int64_t)blockIdx.y * a.n + row] = dirty;
        if (lane == 0 && r0 + 16 * rt < a.n)
            a.fix_count[w16 + rt] =
                (wcnt[rt] < (unsigned)a.fix_cap ? wcnt[rt] : (unsigned)a.fix_cap) | (any ? kFixDirty : 0u);
    }
    // open codes of the workgroup, for k_hash_fix to add up (an atomic of every
    // wave on one counter held the kernel back: 63973 rows 68 us with, 32 without)
    if (a.n_open) {
        const int nf = wave_sum_i32((int)nflag);
        if (lane == 0) sU[0] = (uint32_t)nf;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t t = 0;
            for (int v = 0; v < kWaves; ++v) t += sUall[v * 4 * RPW];
            a.n_open[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = t;
        }
    }
}

// FP64 sequential dot product of an alpha row and a feature row (coordinates
// in index order; each product is exact in FP64).
template <int D>
__device__ __forceinline__ double dot_fp64(const float* __restrict__ ar, const float* __restrict__ vr) {
    double s = 0.0;
#pragma unroll 5
    for (int i = 0; i < D; ++i) s = s + (double)ar[i] * (double)vr[i];
    return s;
}

// The same sum by the four lanes of a quad: lane q reads every fourth piece (16
// bytes where the rows allow it) and forms its products; the sum goes through
// the pieces in order, every lane adding its own to it and all taking the
// owner's result (quad_take).
template <int D, int W>   // W values a piece
__device__ __forceinline__ double quad_dot(const float* __restrict__ ar, const float* __restrict__ vr, int q) {
    constexpr int C = D / W, T = (C + 3) / 4;
    float x[T][W], y[T][W];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int c = 4 * t + q;
#pragma unroll
        for (int u = 0; u < W; ++u) x[t][u] = y[t][u] = 0.0f;
        if (c < C) {
            typedef float piece __attribute__((ext_vector_type(W == 1 ? 2 : W)));
            if constexpr (W == 1) {
                x[t][0] = ar[c], y[t][0] = vr[c];
            } else {
                const piece xv = reinterpret_cast<const piece*>(ar)[c], yv = reinterpret_cast<const piece*>(vr)[c];
#pragma unroll
                for (int u = 0; u < W; ++u) x[t][u] = xv[u], y[t][u] = yv[u];
            }
        }
    }
    double s = 0.0;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        double p[W];
#pragma unroll
        for (int u = 0; u < W; ++u) p[u] = (double)x[t][u] * (double)y[t][u];
        auto add = [&](double s0) {
#pragma unroll
            for (int u = 0; u < W; ++u) s0 = s0 + p[u];
            return s0;
        };
        s = quad_take<0>(add(s));
        if (4 * t + 1 < C) s = quad_take<1>(add(s));
        if (4 * t + 2 < C) s = quad_take<2>(add(s));
        if (4 * t + 3 < C) s = quad_take<3>(add(s));
    }
    return s;
}

// Codes that k_hash left open, by the FP64 sequential dot product that defines
// them. One wave takes the lists of kFixRegions regions, four lanes an entry:
// the entry's uncertain codes, added to the key sum of the others. Then the
// rows of regions whose list ran over: every code of the tables in the row's
// dirty mask, in groups of k lanes (at most four), one (row, table) pair each.
// Bound: the rows' lines (a hash row and a feature row a code; a thread an
// entry read 16 bytes of a line at a time) and the chain of 100 FP64 additions.
// 1040400 rows: 94 + 16 us in two kernels with all k codes in an entry, now 47.
constexpr int kFixRegions = 4;
template <int D>
__global__ __launch_bounds__(64) void k_hash_fix(HashArgs a) {
    const int lane = threadIdx.x;
    const int64_t n16 = (a.n + kRowsPerWave - 1) / kRowsPerWave, nw = n16 * a.parts;
    const int k = a.k, L = a.L, m = L * k;
    const double wd = (double)a.w;
    if (a.n_open && blockIdx.x == gridDim.x - 1) {   // the open codes of all workgroups of k_hash
        uint32_t t = 0;
#pragma unroll 8
        for (int64_t i = lane; i < a.open_blocks; i += 64) t += a.n_open[i];
        const int sum = wave_sum_i32((int)t);
        if (lane == 0) *a.n_fixed = (unsigned)sum;
    }
    // rows on 16-byte boundaries
    const bool vec = D % 4 == 0 && ((reinterpret_cast<uintptr_t>(a.alpha) | reinterpret_cast<uintptr_t>(a.feat)) & 15) == 0;
    for (int64_t base = (int64_t)blockIdx.x * kFixRegions; base < nw; base += (int64_t)gridDim.x * kFixRegions) {
        const unsigned cw = lane < kFixRegions && base + lane < nw ? a.fix_count[base + lane] : 0u;
        const int incl = wave_incl_scan((int)(cw & ~kFixDirty));
        const int total = __shfl(incl, kFixRegions - 1);
        for (int i = lane >> 2; i < total; i += 16) {
            // entry i of the regions' lists one after the other
            int reg = 0, before = 0;
#pragma unroll
            for (int q = 0; q < kFixRegions - 1; ++q) {
                const int end = __builtin_amdgcn_readlane(incl, q);
                if (i >= end) reg = q + 1, before = end;
            }
            const int64_t w = base + reg;
            const uint4 e = a.fix_list[w * a.fix_cap + (i - before)];
            const int64_t row = w % n16 * kRowsPerWave + (e.x >> 8);
            const int l = (int)(e.x & 255u);
            const float* vr = a.feat + row * D;
            uint64_t h = ((uint64_t)e.w << 32) | e.z;
            uint32_t um = e.y;   // the same in the four lanes
            while (um) {
                const int j = __builtin_ctz(um);
                um &= um - 1;
                const int hrow = l * k + j;
                const float* ar = a.alpha + (int64_t)hrow * D;
                const double dot = vec ? quad_dot<D, D % 4 ? 1 : 4>(ar, vr, lane & 3) : quad_dot<D, 1>(ar, vr, lane & 3);
                const int32_t c = floor_sat((dot + (double)a.beta[hrow]) / wd);
                if (a.codes) a.codes[row * m + hrow] = c;
                h += key_term(c, a.key_mul[l * (k + 1) + j]);
            }
            a.keys[key_pos(a, row, l)] = key_final(h);
        }
        uint64_t over = __ballot((cw & kFixDirty) != 0);
        while (over) {
            const int64_t w = base + __builtin_ctzll(over);
            const int64_t r0 = w % n16 * kRowsPerWave;
            over &= over - 1;
            uint64_t mk = lane < kRowsPerWave && r0 + lane < a.n ? a.dirty[w / n16 * a.n + r0 + lane] : 0;
            const int G = 64 / k < 4 ? 64 / k : 4;
            const int grp = lane / k, j = lane - grp * k;
            for (;;) {
                int src = 0, l = 0, got = 0;
                for (int g = 0; g < G; ++g) {
                    const uint64_t any = __ballot(mk != 0);
                    if (!any) break;
                    const int sl = __builtin_ctzll(any);
                    const int tl = __builtin_ctzll(__shfl((unsigned long long)mk, sl));
                    if (lane == sl) mk &= mk - 1;
                    if (grp == g) src = sl, l = tl;
                    ++got;
                }
                if (got == 0) break;
                const bool act = grp < got;
                const int64_t row = r0 + src;
                int32_t c = 0;
                if (act) {
                    const int hrow = l * k + j;
                    c = floor_sat((dot_fp64<D>(a.alpha + (int64_t)hrow * D, a.feat + row * D) + (double)a.beta[hrow]) / wd);
                    if (a.codes) a.codes[row * m + hrow] = c;
                }
                uint64_t h = a.key_mul[l * (k + 1) + k];
                const int first = act ? grp * k : 0;
                for (int jj = 0; jj < k; ++jj) h += key_term(__shfl(c, first + jj), a.key_mul[l * (k + 1) + jj]);
                if (act && j == 0) a.keys[key_pos(a, row, l)] = key_final(h);
            }
        }
    }
}

// Bin (offset, count) of every key, keys and bins table by table: each XCD takes
// an eighth of the tables' blocks in order, so that a table's filter and
// directory come into one L2 (with the blocks dealt out over the XCDs 63973
// rows at L = 16 21.8 us, now 18.2; 3600 rows at L = 8 10.4 and 6.7; 1040400
// rows at L = 24 the same, bound by 42M requests to the L2s in 380 us). A thread
// takes kProbeRows rows of a block's kProbeRows * 256 and keeps their
// lookups in flight together: keys, then filter words, then the first
// directory slot of each key the filter lets through; a key that meets
// neither itself nor an empty slot there walks on alone.
constexpr int kProbeRows = 4;
__global__ __launch_bounds__(256) void k_probe(const uint64_t* __restrict__ keys, int64_t n, int L,
                                               const Slot* __restrict__ dir, uint64_t cap,
                                               const uint32_t* __restrict__ filter, uint2* __restrict__ bins) {
    const uint64_t fw = dir_filter_words(cap);
    const uint64_t mask = cap - 1;
    const int64_t span = 256 * kProbeRows;
    const int64_t bpt = (n + span - 1) / span;   // blocks per table
    for (int64_t b = xcd_block(); b < bpt * L; b += gridDim.x) {
        const int l = (int)(b / bpt);
        const int64_t row0 = (b - l * bpt) * span + threadIdx.x;
        const Slot* dl = dir + (uint64_t)l * cap;
        const uint32_t* fl = filter + (uint64_t)l * fw;
        uint64_t key[kProbeRows];
        uint32_t fword[kProbeRows];
        uint4 e[kProbeRows];
#pragma unroll
        for (int j = 0; j < kProbeRows; ++j) {
            const int64_t row = row0 + 256 * j;
            key[j] = row < n ? keys[(int64_t)l * n + row] : kEmptyKey;
        }
#pragma unroll
        for (int j = 0; j < kProbeRows; ++j) fword[j] = key[j] != kEmptyKey ? fl[dir_filter_bit(key[j], cap) >> 5] : 0u;
#pragma unroll
        for (int j = 0; j < kProbeRows; ++j) {
            e[j] = make_uint4(0u, 0u, 0u, 0u);
            if ((fword[j] >> (dir_filter_bit(key[j], cap) & 31)) & 1u)
                e[j] = *reinterpret_cast<const uint4*>(dl + (key[j] & mask));
        }
#pragma unroll
        for (int j = 0; j < kProbeRows; ++j) {
            const int64_t row = row0 + 256 * j;
            if (row >= n) continue;
            uint32_t off = 0, cnt = 0;
            if ((fword[j] >> (dir_filter_bit(key[j], cap) & 31)) & 1u) {
                const uint64_t k0 = ((uint64_t)e[j].y << 32) | e[j].x;
                if (k0 == key[j]) {
                    cnt = e[j].z;
                    off = e[j].w;
                } else if (k0 != kEmptyKey) {
                    probe_bin_from(dl, cap, key[j], ((key[j] & mask) + 1) & mask, off, cnt);
                }
            }
            bins[(int64_t)l * n + row] = make_uint2(off, cnt);
        }
    }
}

// Error bound of the fp32 code value P against the exact (S + beta) / w,
// S = sum_i alpha_i v_i, from the MFMA sums S~ and S_abs (the MFMA value of
// sum |a_i||v_i| over the operands' high parts). u = 2^-24, n the fp32
// additions of one dot product (counted twice for safety).
//   fp32 path, P = fl(fl(S~ + beta) * fl(1/w)): |S~ - S| <= gamma_n
//     sum|alpha_i v_i|, sum <= S_abs / (1 - gamma); the add, the reciprocal
//     and the multiply add 3.1 u (|S~| + |beta|) / w.
//   split path, P = fl(S~ + beta'), alpha' = fl(alpha / w), beta' =
//     fl(beta / w): |S~ - sum alpha'_i v_i| <= (gamma_n 1.016 + 3.5 2^-16)
//     sum|alpha'_i v_i| (the dropped low x low and rounding-residual
//     products contribute at most 3.1 2^-16), the rounding of alpha / w adds
//     u (1 + u) of the same sum and that of beta / w u / (1 - u) |beta'|;
//     the final add u / (1 - u) |P| with |P| <= (1 + u) ((1 + E) sum + |beta'|);
//     sum|alpha'_i v_i| <= S_abs / ((1 - 2^-8)^2 (1 - gamma)). All of it is
//     c1 S_abs + c0_j (c2 = 0): one fused multiply-add a code.
// Every term is doubled, and the FP64 sequential sum of the definition is
// within ~1e-13 of the exact value, far inside the margin.
void hash_bound_coeffs(int prec, int D, double w, const float* beta, int m, float* c0, float* c1,
                       float* c2) {
    const double u = 1.0 / 16777216.0;
    const int DP = prec == 0 ? ((D + 3) & ~3) : ((D + 31) & ~31);
    const int nadd = prec == 0 ? 2 * DP : 2 * 3 * DP;
    const double g = gamma_n(nadd, u);
    const double up = 1.0 + 1e-6;
    if (prec == 0) {
        const double c_abs = 1.0 / (1.0 - gamma_n(2 * DP, u));
        *c1 = (float)(2.0 * g * c_abs / w * up);
        *c2 = (float)(2.0 * 3.1 * u / w * up);
        for (int j = 0; j < m; ++j) c0[j] = (float)((2.0 * 3.1 * u * std::fabs((double)beta[j]) / w + 1e-30) * up);
        return;
    }
    const double t = 1.0 - 1.0 / 256.0;
    const double c_abs = 1.0 / (t * t * (1.0 - gamma_n(2 * DP, u)));
    const double E = g * 1.016 + 3.5 / 65536.0 + u * (1.0 + u);
    const double e2 = u / (1.0 - u);
    *c1 = (float)(2.0 * c_abs * (E + e2 * (1.0 + u) * (1.0 + E)) * up);
    *c2 = 0.0f;
    for (int j = 0; j < m; ++j) {
        const double bw = std::fabs((double)(beta[j] / (float)w));
        c0[j] = (float)((2.0 * (e2 + e2 * (1.0 + u)) * bw + 1e-30) * up);
    }
}

// c1 of k_hash's bound: as above, but with a sum of block norms rounded up in
// place of the MFMA sum of absolute values, and without the last doubling: gamma_n
// counts every addition twice, which covers additions that truncate; the
// split's own terms are exact arithmetic. Largest |P - exact| / bound measured,
// over features of images, normal, sparse, mixed in size and large, D = 25 and
// 100: 0.40 on the split path, 0.16 on the fp32 path.
float hash_bound_norm_c1(int prec, int D, double w) {
    const double u = 1.0 / 16777216.0, up = 1.0 + 2e-5;   // up: the additions of the block norms' MFMA
    const int DP = prec == 0 ? ((D + 3) & ~3) : ((D + 31) & ~31);
    const double g = gamma_n(prec == 0 ? 2 * DP : 2 * 3 * DP, u);
    if (prec == 0) return (float)(2.0 * g / w * up);
    const double E = g * 1.016 + 3.5 / 65536.0 + u * (1.0 + u);
    const double e2 = u / (1.0 - u);
    return (float)((E + 2.0 * e2 * (1.0 + u) * (1.0 + E)) * up);
}

template <int PREC, int D>
static size_t image_bytes(int L, int k) {
    using HT = HashTile<PREC, D>;
    return (size_t)((hash_tiles(L, k) + HT::G - 1) / HT::G) * HT::SB;
}

size_t hash_image_bytes(int prec, int D, int L, int k) {
    if (D == 25) return prec ? image_bytes<1, 25>(L, k) : image_bytes<0, 25>(L, k);
    return prec ? image_bytes<1, 100>(L, k) : image_bytes<0, 100>(L, k);
}

hipError_t launch_hash_image(int prec, int D, int L, int k, float w, const float* alpha, const float* beta,
                             const uint16_t* a_hi, const uint16_t* a_lo, const float* c0, const uint64_t* key_mul,
                             unsigned char* img, hipStream_t st) {
    if ((D != 25 && D != 100) || k < 1 || k > kMaxKHash || L < 1 || L > kMaxL) return hipErrorInvalidValue;
    auto kern = D == 25 ? (prec ? k_hash_image<1, 25> : k_hash_image<0, 25>)
                        : (prec ? k_hash_image<1, 100> : k_hash_image<0, 100>);
    hipLaunchKernelGGL(kern, dim3((unsigned)hash_tiles(L, k)), dim3(256), 0, st, alpha, beta, a_hi, a_lo, c0, key_mul, w,
                       L, k, img);
    return hipGetLastError();
}

hipError_t launch_hash(const HashArgs& a, hipStream_t st) {
    const hipError_t e = launch_hash_codes(a, st);
    if (e != hipSuccess || !a.bins) return e;
    return launch_probe(a, st);
}

hipError_t launch_probe(const HashArgs& a, hipStream_t st) {
    if (a.n == 0 || !a.bins) return hipSuccess;
    if (!a.keys_tmajor || !a.dir || !a.dir_filter) return hipErrorInvalidValue;
    const int64_t total = a.n * a.L;
    int64_t g = (total + 256 * kProbeRows - 1) / (256 * kProbeRows);
    if (g > 65536) g = 65536;
    g = round_grid8((int)g);
    hipLaunchKernelGGL(k_probe, dim3((unsigned)g), dim3(256), 0, st, a.keys, a.n, a.L, a.dir, a.dir_cap,
                       a.dir_filter, a.bins);
    return hipGetLastError();
}

size_t hash_count_words(const HashArgs& a) {
    const int64_t n16 = (a.n + kRowsPerWave - 1) / kRowsPerWave;
    return (size_t)((n16 + (n16 + kWaves - 1) / kWaves) * a.parts) + 1;
}

// Stages of the hash rows, and the fewest that end at an even table.
static void hash_stages(const HashArgs& a, int& nst, int& unit) {
    const int G = a.D > 32 ? HashTile<1, 100>::G : HashTile<1, 25>::G;
    nst = (hash_tiles(a.L, a.k) + G - 1) / G;
    unit = 1;
    while (unit < nst && unit * 16 * G % (2 * padded_hashes(a.k))) ++unit;
}

// Few rows leave compute units without a workgroup: the tables are then shared
// out over several workgroups a row block, up to about two workgroups a compute
// unit in all (us in one part with one row tile a wave, and in parts: 24236
// rows 31.5 and 24.6, 14732 rows 16.7 and 13.7). Larger grids gain nothing by
// parts (203636 rows 120 and 123).
void hash_parts(HashArgs& a) {
    int nst, unit;
    hash_stages(a, nst, unit);
    const int64_t rows = kWaves * kRowsPerWave * (a.prec == 1 ? 2 : 1);
    const int64_t blocks = (a.n + rows - 1) / rows;
    const int units = (nst + unit - 1) / unit;
    const int64_t want = blocks < 1 || blocks >= kHashBlocks ? 1 : (kHashBlocks + blocks - 1) / blocks;
    const int per = (int)((units + std::min<int64_t>(want, units) - 1) / std::min<int64_t>(want, units));
    a.part_stages = per * unit;
    a.parts = (nst + a.part_stages - 1) / a.part_stages;
}

template <int D>
static hipError_t launch_codes(const HashArgs& a, hipStream_t st) {
    // two row tiles a wave share each operand read of the hash rows (1040400
    // rows with one 760 us, with two 512); one where two would leave compute
    // units without a workgroup
    const bool two = a.prec == 1 && (a.n + 127) / 128 * a.parts >= 512;
    const int rows = kWaves * kRowsPerWave * (two ? 2 : 1);
    const dim3 grid((unsigned)((a.n + rows - 1) / rows), (unsigned)a.parts);
    auto kern = a.prec == 0 ? (a.codes ? k_hash<0, D, 1, true> : k_hash<0, D, 1, false>)
                : two       ? (a.codes ? k_hash<1, D, 2, true> : k_hash<1, D, 2, false>)
                            : (a.codes ? k_hash<1, D, 1, true> : k_hash<1, D, 1, false>);
    HashArgs b = a;
    b.n_open = a.n_fixed ? a.fix_count + (a.n + kRowsPerWave - 1) / kRowsPerWave * a.parts : nullptr;
    b.open_blocks = (int64_t)grid.x * grid.y;
    if (!one_row(grid.x, 256)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, b);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t regions = (a.n + kRowsPerWave - 1) / kRowsPerWave * a.parts, gl = (regions + kFixRegions - 1) / kFixRegions;
    hipLaunchKernelGGL(k_hash_fix<D>, dim3((unsigned)(gl < 65536 ? gl : 65536)), dim3(64), 0, st, b);
    return hipGetLastError();
}

hipError_t launch_hash_codes(const HashArgs& a, hipStream_t st) {
    if (a.n == 0) return hipSuccess;
    if ((a.D != 25 && a.D != 100) || a.k < 1 || a.k > kMaxKHash || a.L < 1 || a.L > kMaxL || !a.img || !a.dirty ||
        !a.fix_count || !a.key_mul || a.parts < 1 || a.part_stages < 1 || a.fix_cap < 0 || a.fix_cap > kFixSlots || (a.fix_cap > 0 && !a.fix_list) ||
        (a.bins && (!a.keys_tmajor || !a.dir || !a.dir_filter)))
        return hipErrorInvalidValue;
    return a.D == 25 ? launch_codes<25>(a, st) : launch_codes<100>(a, st);
}

}  // namespace zh
