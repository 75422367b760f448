// ls_mfma.hip - batched (B >= 4) gate/up and down kernels on the matrix cores of gfx950.
//
// With B tokens the gather GEMVs become small dense contractions: for a group of
// 16 neurons, [16 x d] weight rows times [d x B] activations.  These kernels run them as
// v_mfma_f32_16x16x32_{f16,bf16}: the weights are the A operand, loaded straight from
// their rows (one 16-byte load per lane per step), and the activations are the B operand,
// token columns.  Activations are fp32, so each one enters as the sum of 16-bit parts, with fp32
// accumulation in the matrix cores: two or three (input_parts) in the resident gate/up kernel
// and the down projection beside it, a "hi" part and the 16-bit rounding of the remainder, "lo",
// in the staged gate/up and the ordered down kernel (in bfloat16 these carry 16 bits; the others
// match the VALU kernels to fp32 rounding).  Eq. 1 of the paper, union over tokens as for the VALU path.
//
// Lane layout of v_mfma_f32_16x16x32 (lane l, i < 8 / i < 4):
//   A[l % 16][8 (l / 16) + i],  B[8 (l / 16) + i][l % 16],  C[4 (l / 16) + i][l % 16].
#include <algorithm>

#include "ls_device.h"
#include "ls_internal.h"
#include "ls_split.h"

namespace ls {
namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4v __attribute__((ext_vector_type(4)));

// Split 8 fp32 values into hi and lo 16-bit operands of type T.
template <ls_dtype T>
struct Split;

template <>
struct Split<LS_F16> {
    typedef f16x8 vec;
    __device__ static inline void run(const float* x, vec& hi, vec& lo) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const _Float16 h = (_Float16)x[i];
            hi[i] = h;
            lo[i] = (_Float16)(x[i] - (float)h);
        }
    }
    __device__ static inline vec from_raw(const u32x4& r) {
        vec v;
        __builtin_memcpy(&v, &r, 16);
        return v;
    }
    __device__ static inline f32x4v mfma(const vec& a, const vec& b, const f32x4v& c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
    }
};

template <>
struct Split<LS_BF16> {
    typedef s16x8 vec;
    // (the conversion instruction rounds to nearest even, two values at a time)
    typedef __bf16 b16x2 __attribute__((ext_vector_type(2)));
    __device__ static inline void run(const float* x, vec& hi, vec& lo) {
        u32x4 h4, l4;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const b16x2 h = {(__bf16)x[2 * i], (__bf16)x[2 * i + 1]};
            const uint32_t hw = __builtin_bit_cast(uint32_t, h);
            const b16x2 l = {(__bf16)(x[2 * i] - __uint_as_float(hw << 16)),
                             (__bf16)(x[2 * i + 1] - __uint_as_float(hw & 0xffff0000u))};
            h4[i] = hw;
            l4[i] = __builtin_bit_cast(uint32_t, l);
        }
        hi = from_raw(h4);
        lo = from_raw(l4);
    }
    __device__ static inline vec from_raw(const u32x4& r) {
        vec v;
        __builtin_memcpy(&v, &r, 16);
        return v;
    }
    __device__ static inline f32x4v mfma(const vec& a, const vec& b, const f32x4v& c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
};

__device__ inline int list_end_m(const int32_t* count, int end, int n_blk) {
    int c = *count;
    c = c < 0 ? 0 : (c > n_blk ? n_blk : c);
    return end < c ? end : c;
}

// 16 bytes of the input at a wave-uniform base plus a per-lane byte offset
__device__ __forceinline__ f32x4 gload_x(const float* uniform_base, uint32_t byte_off) {
    typedef const __attribute__((address_space(1))) f32x4* gf4_ptr;
    const uint64_t b = (uint64_t)uniform_base;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return *(gf4_ptr)((const char*)(((uint64_t)hi << 32) | lo) + byte_off);
}

// a barrier that orders LDS only: global loads already issued stay in flight
__device__ __forceinline__ void lds_barrier_m() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---- gate/up, inputs in registers -------------------------------------------------------------------------
// The inputs stay in registers.  A workgroup owns many groups of 8 neurons; its W waves cut the
// d values of a row into W slices of NK (or fewer) steps of 64, and a wave keeps its slice of
// every token, already split into 16-bit parts, in registers for the whole launch, so a compute
// unit reads x once instead of once per 16 rows.  The per-CU memory path is what bounds a
// batched gather (about 7 TB/s over the chip whatever the bytes are): read again for every
// group, x cost 8 d bytes per token beside 64 d bytes of weights.
//
// The weights go from global memory straight into MFMA operands: one load instruction covers 8
// rows x 128 bytes (whole cache lines).  Lane l holds row l % 8, chunk l / 8 of 8 values, so as
// operand A its row index l % 16 means (half h = (l / 8) % 2, row l % 8) and holds the 8 values
// of chunk 2 (l / 16) + h.  Operand B is laid out the same way: column (h, slot).  Of the 16 x 16
// products the two diagonal 8 x 8 blocks (equal halves) are the row's even and odd chunks; the
// rest is not used.  A streaming read in this pattern measured 5.75 TB/s (8 KB rows, 180 MB)
// against 5.99 for 1 KB of one row per instruction, which would need a transpose through LDS,
// and 4.3 - 5.1 for 16 rows x 64 bytes, the plain operand layout.
//
// The 8 slots of a fragment hold P parts x BP tokens (BP: tokens padded to 4 or 8); with more
// than 8 there are NF fragments.  A part is the 16-bit rounding of what the parts before it left,
// so P = 2 float16 parts carry 22 bits of an fp32 value and P = 3 parts of either type all 24
// (input_parts).  float16 parts: the slice is scaled by a power of two to below 2 in magnitude and
// each part by 2^11 against the one before, so that none overflows; the factors are taken out of
// the sums.  The last part of a value far below the slice's largest is subnormal: three parts hold 24
// bits down to 2^-23 of the largest and multiples of 2^-46 of it below (two: 22 bits down to 2^-14,
// multiples of 2^-35).  The third part costs 1.3 to 1.7 us a sparse step (2880 x 7720 at B = 5, 96 blocks
// of 40: 21.1 -> 22.8); its error against 64 bits, activations and output together, is below the
// vector-ALU kernels' at every width measured, two parts' is above it at 512.
//
// Measured against the staged kernel below (which keeps rows longer than the registers hold, and
// the thresholded gates of keeps_order): Mistral-7B shape with a ReLU gate at B = 4 (105 blocks, 220
// MB) 61.7 -> 41.6 us, 13B shape at B = 8 (138
// blocks, 181 MB) 45.0 -> 37.2 us.  From 45 to 180 MB it reads 7.0 TB/s; about 8 us of a launch
// are the list, the input's conversion and the last sums.
constexpr int kGuWaves = kSplitSlices;  // slices, at most

// FULL: every wave has NK steps (d / 64 = W NK); the addresses of a unit's loads then differ only in
// their immediate offsets.  PRE: the fragments (and the slices' scales and sums of squares) were
// prepared by the selection launch (the same bits); the wave then only loads them.
template <ls_dtype T, int P, int NK, int BP, bool FULL, bool PRE>
__global__ __launch_bounds__(64 * kGuWaves) void gateup_mfma_kernel(
    const uint8_t* __restrict__ blocks, size_t block_bytes, const int32_t* __restrict__ slot_table,
    const void* __restrict__ bias, float thresh, const float* __restrict__ x, int B, int d, int blk,
    int n_blk, int F, const int32_t* __restrict__ idx, const int32_t* __restrict__ count, int begin,
    int end, float* __restrict__ a_buf, int reglu, int rms, const u32x4* __restrict__ frag,
    const float* __restrict__ meta) {
    using S = Split<T>;
    typedef typename S::vec vec;
    constexpr int NF = (P * BP + 7) / 8;
    // loads of a unit: one row set's steps, or half of them where two whole ones and the
    // fragments would not fit the 256 registers
    constexpr int UL = NK <= 8 || 8 * NK + 4 * NF * NK <= 160 ? NK : NK / 2;
    constexpr int UM = NK / UL;                // units per row set (gate, up)
    static_assert(NK % UL == 0, "whole units");
    // partial sums of two groups: [wave][gate, up][fragment][half][slot][row]
    __shared__ __attribute__((aligned(16))) float part[2][kGuWaves][2][NF][2][8][8];
    __shared__ float pss[kGuWaves][8];
    const int W = (int)(blockDim.x >> 6);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int gpe = blk / 8;  // groups per entry
    // this wave's steps [s0, s0 + nst) of the row's d / 64
    const int steps = d / 64;
    const int s0 = FULL ? NK * wave : steps * wave / W, nst = FULL ? NK : steps * (wave + 1) / W - s0;
    const size_t row_bytes = (size_t)d * 2;
    const uint32_t lane_off = (uint32_t)(lane & 7) * (uint32_t)row_bytes + (uint32_t)(lane >> 3) * 16u;

    // x, this wave's slice of the lane's token, requested before the list is read.  Every address
    // is in bounds: a token past the batch reads token 0 (its columns are never used), a step
    // past the slice its first
    const int tok = (lane & 7) & (BP - 1);
    const int half = (lane >> 3) & 1;
    f32x4 xv[PRE ? 1 : NK][2];
    u32x4 pre[PRE ? NF : 1][PRE ? NK : 1];
    float pre_unscale = 1.f, pre_ss = 0.f;
    if constexpr (PRE) {
        const u32x4* src = frag + (size_t)wave * NK * NF * 64;
#pragma unroll
        for (int s = 0; s < NK; ++s)
#pragma unroll
            for (int f = 0; f < NF; ++f) pre[f][s] = src[(s * NF + f) * 64 + lane];
        pre_unscale = meta[wave * 8 + (lane & 7)];
        pre_ss = meta[kSplitSlices * 8 + wave * 8 + (lane & 7)];
    } else {
        const uint32_t xo = ((uint32_t)(tok < B ? tok : 0) * (uint32_t)d + 16u * (uint32_t)(lane >> 4) + 8u * (uint32_t)half) * 4u;
        const float* xs = x + (size_t)s0 * 64;
#pragma unroll
        for (int s = 0; s < NK; ++s) {
            const uint32_t o = xo + (uint32_t)(s < nst ? s : 0) * 256u;
            xv[s][0] = gload_x(xs, o);
            xv[s][1] = gload_x(xs, o + 16u);
        }
    }
    const int n_groups = (list_end_m(count, end, n_blk) - begin) * gpe;
    if ((int)blockIdx.x >= n_groups) return;

    // a group's first gate row in this wave's slice (an invalid or absent block reads block 0,
    // whose products are dropped at the end)
    auto slot_of = [&](int b) { return b < 0 || b >= n_blk ? -1 : (slot_table ? slot_table[b] : b); };
    auto group_base = [&](int slot, int gi) {
        return blocks + (size_t)(slot < 0 ? 0 : slot) * block_bytes + (size_t)(gi % gpe) * 8 * row_bytes +
               (size_t)s0 * 128;
    };
    u32x4 buf[2][UL];
    auto load_unit = [&](u32x4 (&u4)[UL], const uint8_t* base, int u) {
        const uint8_t* rows = base + (u / UM ? (size_t)blk * row_bytes : 0);
#pragma unroll
        for (int i = 0; i < UL; ++i) {
            const int s = (u % UM) * UL + i;  // steps past the slice repeat its first one
            u4[i] = gload_u(rows, lane_off + (uint32_t)(s < nst ? s : 0) * 128u);
        }
    };
    int gi = (int)blockIdx.x;
    int b_cur = idx[begin + gi / gpe];
    const int gi2 = gi + (int)gridDim.x;
    int b_nxt = gi2 < n_groups ? idx[begin + gi2 / gpe] : -1;
    int slot = slot_of(b_cur);
    const uint8_t* base = group_base(slot, gi);
    load_unit(buf[0], base, 0);
    load_unit(buf[1], base, 1);

    // x into parts
    vec xf[NF][NK];
    float unscale = 1.f;
    if constexpr (PRE) {
#pragma unroll
        for (int s = 0; s < NK; ++s)
#pragma unroll
            for (int f = 0; f < NF; ++f) xf[f][s] = S::from_raw(pre[f][s]);
        unscale = pre_unscale;
        if (lane < 8) pss[wave][lane] = pre_ss;
    } else {
        float s4[4], mx = 0.f;  // four short chains: the scale's error goes into every sum
#pragma unroll
        for (int i = 0; i < 4; ++i) s4[i] = 0.f;
#pragma unroll
        for (int s = 0; s < NK; ++s)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float v = s < nst ? xv[s][i >> 2][i & 3] : 0.f;
                xv[s][i >> 2][i & 3] = v;
                if (T == LS_F16 && fabsf(v) < INFINITY) mx = fmaxf(mx, fabsf(v));
            }
        // lanes l, l + 8, l + 16, ... hold the same slot
        if (T == LS_F16) {
#pragma unroll
            for (int off = 8; off < 64; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
        }
        const int ex = T == LS_F16 ? split_exponent(mx) : 0;
        unscale = ldexpf(1.f, ex);
#pragma unroll
        for (int s = 0; s < NK; ++s) {
            u32x4 words[NF];
            split_step<T, P, BP>(xv[s], ex, lane, s4, words);
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                asm volatile("" : "+v"(words[f]));
                xf[f][s] = S::from_raw(words[f]);
            }
            // one step at a time: its inputs' registers become its fragments'
            if (s + 1 < NK) asm volatile("" : "+v"(xv[s + 1][0]), "+v"(xv[s + 1][1]));
            __builtin_amdgcn_sched_barrier(0);
        }
        float ss = tree_sum<4>(s4);
#pragma unroll
        for (int off = 8; off < 64; off <<= 1) ss += __shfl_xor(ss, off, 64);
        if (lane < 8) pss[wave][lane] = ss;
    }
    lds_barrier_m();
    // the finishing threads' token and its RMS scale
    const int ft = lane >> 3, fr = lane & 7;
    float sc = 1.f;
    if (rms) {
        float q = 0.f;
        float qw[kGuWaves];
#pragma unroll
        for (int w = 0; w < kGuWaves; ++w) qw[w] = w < W ? pss[w][ft & (BP - 1)] : 0.f;
        q = tree_sum<kGuWaves>(qw);
        sc = rms_scale(q, d);
    }

    for (int it = 0;; ++it) {
        const int gn = gi + (int)gridDim.x;
        const bool more = gn < n_groups;
        const int slot_n = slot_of(b_nxt);
        const uint8_t* base_n = group_base(slot_n, gn);
        const int b_this = b_cur;
        {
            const int g2 = gn + (int)gridDim.x;
            b_cur = b_nxt;
            b_nxt = g2 < n_groups ? idx[begin + g2 / gpe] : -1;
        }
        f32x4v c[2][NF];
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int f = 0; f < NF; ++f) c[m][f] = f32x4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < 2 * UM; ++u) {
#pragma unroll
            for (int i = 0; i < UL; ++i) {
                const int s = (u % UM) * UL + i;
                u32x4 raw = buf[u & 1][i];
                if (s >= nst) raw = u32x4{0u, 0u, 0u, 0u};
                const vec a = S::from_raw(raw);
#pragma unroll
                for (int f = 0; f < NF; ++f) c[u / UM][f] = S::mfma(a, xf[f][s], c[u / UM][f]);
            }
            if (u + 2 < 2 * UM) load_unit(buf[u & 1], base, u + 2);
            else if (more) load_unit(buf[u & 1], base_n, u + 2 - 2 * UM);
        }
        // lane l: rows 4 (l / 16) + i of column l % 16; rows and columns of the same half count
        if ((lane >> 5) == half) {
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    f32x4v v = c[m][f];
                    if (T == LS_F16) {
                        const float k = ldexpf(unscale, -Part<T>::kShift * ((f * 8 + (lane & 7)) / BP));
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] *= k;
                    }
                    *reinterpret_cast<f32x4v*>(&part[it & 1][wave][m][f][half][lane & 7][4 * ((lane >> 4) & 1)]) = v;
                }
        }
        // one barrier a group: a buffer is written again two groups later, past the next barrier,
        // which the finishing wave joins after its reads
        lds_barrier_m();
        if (wave == it % W && ft < B) {
            // the waves' sums pairwise, the smallest part first (a loop: its reads must not take the
            // registers that hold the loads in flight)
            float gu[2] = {0.f, 0.f};
#pragma unroll 1
            for (int pm = 2 * P - 1; pm >= 0; --pm) {
                const int m = pm & 1, q = (pm >> 1) * BP + (ft & (BP - 1));
                float sw[kGuWaves];
#pragma unroll
                for (int w = 0; w < kGuWaves; ++w) {
                    const float s = part[it & 1][w][m][q >> 3][0][q & 7][fr] + part[it & 1][w][m][q >> 3][1][q & 7][fr];
                    sw[w] = w < W ? s : 0.f;  // (a wave that is not there wrote nothing)
                }
                const float t = tree_sum<kGuWaves>(sw);
                if (m) gu[1] += t;
                else gu[0] += t;
            }
            float g = gu[0], uv = gu[1];
            const int e = begin + gi / gpe, r0 = (gi % gpe) * 8;
            float a = 0.f;
            if (slot >= 0) {
                g = sc * g + (bias ? Wt<T>::scalar(bias, (size_t)b_this * blk + r0 + fr) : 0.f);
                uv = sc * uv;
                if (reglu) {
                    a = fmaxf(g, 0.f) * uv;
                } else {
                    const float sg = g / (1.f + expf(-g));
                    a = fabsf(sg) > thresh ? sg * uv : 0.f;
                }
            }
            a_buf[(size_t)ft * F + (size_t)e * blk + r0 + fr] = a;
        }
        if (!more) break;
        gi = gn;
        base = base_n;
        slot = slot_n;
    }
}

// ---- gate/up, any d ---------------------------------------------------------------------------------
constexpr int kWaves = 4;     // gate/up: waves per workgroup
constexpr int kRowsW = 32 / kWaves;  // gate/up: staged rows loaded by each wave per chunk

// One workgroup per group of 16 neurons (rows r0..r0+15 of one list entry).  The gate and up
// rows of the group stream through LDS in chunks of 512 K values: each load instruction reads
// one kilobyte of one row (row-contiguous reads stream far better than the 16-row x 64-byte
// pattern of an MFMA operand), the 4 waves write them to LDS rows padded to 1040 bytes (so
// that the 16 lanes reading one fragment column hit different banks), and each wave then runs
// a quarter of the chunk's K steps from LDS while the next chunk's loads are in flight.
// a_buf[tok * F + e * blk + q] as the VALU kernel writes it.  x is the layer input; with RMS
// each lane also sums the squares of the x values it loads (every (token, k) exactly once per
// workgroup) and the dot products are scaled at the end.
constexpr int kChunkK = 512;                 // K values per chunk (1 KB of a 16-bit row)
constexpr int kLpr = 2 * kChunkK / 1024;     // 1 KB loads per staged row and chunk
constexpr int kRowPitch = 2 * kChunkK + 16;  // LDS bytes per staged row
// three waves per SIMD (at most 168 registers a lane): three workgroups per CU
constexpr int kGuWavesPerEu = 3;
template <ls_dtype T, ls_act A, bool RMS>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(kGuWavesPerEu))) void gateup_staged_kernel(
    const uint8_t* __restrict__ blocks, size_t block_bytes, const int32_t* __restrict__ slot_table,
    const void* __restrict__ bias, float thresh, const float* __restrict__ h, int B, int d, int blk,
    int n_blk, int F, const int32_t* __restrict__ idx, const int32_t* __restrict__ count, int begin,
    int end, float* __restrict__ a_buf) {
    using S = Split<T>;
    __shared__ __attribute__((aligned(16))) uint8_t stage[32 * kRowPitch];  // rows 0-15 gate, 16-31 up
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int groups_per_entry = blk / 16;
    const int e = begin + (int)blockIdx.x / groups_per_entry;
    const int r0 = ((int)blockIdx.x % groups_per_entry) * 16;
    if (e >= list_end_m(count, end, n_blk)) return;
    const int b = idx[e];
    const int slot = (b < 0 || b >= n_blk) ? -1 : (slot_table ? slot_table[b] : b);
    if (slot < 0) {  // invalid id or block not in the cache: the entry contributes nothing
        if (threadIdx.x < 16 * B) {
            const int tok = threadIdx.x / 16, r = threadIdx.x % 16;
            a_buf[(size_t)tok * F + (size_t)e * blk + r0 + r] = 0.f;
        }
        return;
    }
    const size_t row_bytes = (size_t)d * 2;
    const uint8_t* base = blocks + (size_t)slot * block_bytes;
    const int tok = lane & 15;
    const bool tok_ok = tok < B;
    const float* hrow = h + (size_t)(tok_ok ? tok : 0) * d;
    // staged row j of this wave's loads: gate row r0 + j (j < 16) or up row r0 + j - 16
    auto row_ptr = [&](int j) {
        return base + (size_t)(j < 16 ? r0 + j : blk + r0 + j - 16) * row_bytes;
    };
    auto load_chunk = [&](int c0, u32x4 (&rw)[kRowsW * kLpr]) {
        const int bytes = 2 * min(kChunkK, d - c0);
#pragma unroll
        for (int i = 0; i < kRowsW; ++i) {
            const int j = wave + kWaves * i;
#pragma unroll
            for (int h = 0; h < kLpr; ++h) {
                const int off = 1024 * h + lane * 16;
                rw[i * kLpr + h] = off < bytes ? ld_stream(reinterpret_cast<const u32x4*>(row_ptr(j) + (size_t)c0 * 2 + off))
                                               : u32x4{0u, 0u, 0u, 0u};
            }
        }
    };
    // x of this wave's K steps of a chunk (s0 = wave + kWaves j), requested once the wave is
    // done with the previous chunk's (after the next chunk's weights: a wave waits for both
    // at the top of the chunk anyway)
    constexpr int kStepsW = kChunkK / 32 / kWaves;
    auto load_x = [&](int c0, f32x4 (&hx)[kStepsW][2]) {
        const int steps = min(kChunkK, d - c0) / 32;
#pragma unroll
        for (int j = 0; j < kStepsW; ++j) {
            const int s0 = wave + kWaves * j;
            const int kc = 32 * s0 + 8 * (lane >> 4);  // this lane's 8 K values in the chunk
            const f32x4 z = {0.f, 0.f, 0.f, 0.f};
            const bool ok = tok_ok && s0 < steps;
            hx[j][0] = ok ? reinterpret_cast<const f32x4*>(hrow + c0 + kc)[0] : z;
            hx[j][1] = ok ? reinterpret_cast<const f32x4*>(hrow + c0 + kc)[1] : z;
        }
    };
    f32x4v cg = {0.f, 0.f, 0.f, 0.f}, cu = {0.f, 0.f, 0.f, 0.f};
    float ss = 0.f;
    u32x4 rw[kRowsW * kLpr];
    f32x4 hx[kStepsW][2];
    load_chunk(0, rw);
    load_x(0, hx);
    for (int c0 = 0; c0 < d; c0 += kChunkK) {
        const int steps = min(kChunkK, d - c0) / 32;
        const bool more = c0 + kChunkK < d;
#pragma unroll
        for (int i = 0; i < kRowsW; ++i)
#pragma unroll
            for (int h = 0; h < kLpr; ++h)
                *reinterpret_cast<u32x4*>(stage + (wave + kWaves * i) * kRowPitch + 1024 * h + lane * 16) = rw[i * kLpr + h];
        __syncthreads();
        if (more) load_chunk(c0 + kChunkK, rw);  // in flight while this chunk runs
#pragma unroll
        for (int j = 0; j < kStepsW; ++j) {
            const int s0 = wave + kWaves * j;
            if (s0 >= steps) break;
            const int kc = 32 * s0 + 8 * (lane >> 4);
            const f32x4 h0 = hx[j][0], h1 = hx[j][1];
            const float xv[8] = {h0.x, h0.y, h0.z, h0.w, h1.x, h1.y, h1.z, h1.w};
            if (RMS) {
#pragma unroll
                for (int i = 0; i < 8; ++i) ss = fmaf(xv[i], xv[i], ss);
            }
            typename S::vec hi, lo;
            S::run(xv, hi, lo);
            const u32x4 wg4 = *reinterpret_cast<const u32x4*>(stage + (lane & 15) * kRowPitch + kc * 2);
            const u32x4 wu4 = *reinterpret_cast<const u32x4*>(stage + (16 + (lane & 15)) * kRowPitch + kc * 2);
            const typename S::vec wg = S::from_raw(wg4), wu = S::from_raw(wu4);
            cg = S::mfma(wg, hi, cg);
            cg = S::mfma(wg, lo, cg);
            cu = S::mfma(wu, hi, cu);
            cu = S::mfma(wu, lo, cu);
        }
        if (more) load_x(c0 + kChunkK, hx);
        __syncthreads();  // every wave is done with the chunk before it is overwritten
    }
    // lane l holds rows 4 (l / 16) + i, token l % 16 of this wave's partial sums
    // the partial sums reuse the staging buffer (every wave is past the last chunk), so that
    // four workgroups fit in a compute unit's LDS
    static_assert(sizeof(float) * (2 * kWaves * 16 * 16 + kWaves * 16) <= sizeof(stage), "epilogue fits the stage");
    float (&pg)[kWaves][16][16] = *reinterpret_cast<float (*)[kWaves][16][16]>(stage);
    float (&pu)[kWaves][16][16] = *reinterpret_cast<float (*)[kWaves][16][16]>(stage + sizeof(float) * kWaves * 16 * 16);
    float (&pss)[kWaves][16] = *reinterpret_cast<float (*)[kWaves][16]>(stage + 2 * sizeof(float) * kWaves * 16 * 16);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        pg[wave][4 * (lane >> 4) + i][lane & 15] = cg[i];
        pu[wave][4 * (lane >> 4) + i][lane & 15] = cu[i];
    }
    if (RMS) {  // lanes l, l+16, l+32, l+48 hold the same token
        ss += __shfl_xor(ss, 16, 64);
        ss += __shfl_xor(ss, 32, 64);
        if (lane < 16) pss[wave][lane] = ss;
    }
    __syncthreads();
    if (threadIdx.x < 16 * B) {
        const int t = threadIdx.x / 16, r = threadIdx.x % 16;
        float sq = 0.f, gs = 0.f, us = 0.f;  // the waves' partial sums in wave order
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            sq += pss[w][t];
            gs += pg[w][r][t];
            us += pu[w][r][t];
        }
        const float sc = RMS ? rms_scale(sq, d) : 1.f;
        const float g = sc * gs +
                        (bias ? Wt<T>::scalar(bias, (size_t)b * blk + r0 + r) : 0.f);
        const float u = sc * us;
        float a;
        if (A == LS_ACT_REGLU) {
            a = fmaxf(g, 0.f) * u;
        } else {
            const float sg = g / (1.f + expf(-g));
            a = fabsf(sg) > thresh ? sg * u : 0.f;
        }
        a_buf[(size_t)t * F + (size_t)e * blk + r0 + r] = a;
    }
}

// The last of the `splits` workgroups of a column group to store its part adds the parts in order of
// part and writes x_acc, instead of one more launch (13B shape at B = 8, three layers 209 -> 206 us;
// 2880 x 7720 at B = 5, one layer 37.6 -> 35.4).  Parts travel as agent-scope atomic words, coherent across the XCDs' L2s without cache
// maintenance; a workgroup counts itself once its stores are complete, so whoever counts last
// sees every part.  Nothing waits; the count is left at zero for the next call.
// m(q): the index of the workgroup's q-th output in [B, d]; n outputs, B d apart per part.
template <typename Index>
__device__ __forceinline__ void finish_parts(const float* part, int splits, size_t stride, int n, Index m,
                                             const float* __restrict__ x_in, float* x_acc, bool first, uint32_t* cnt) {
    __shared__ uint32_t arrived;
    __builtin_amdgcn_s_waitcnt(0);  // this wave's part words are stored
    __syncthreads();
    if (threadIdx.x == 0) arrived = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (arrived != (uint32_t)splits - 1u) return;
    if (threadIdx.x == 0) __hip_atomic_store(cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int q = (int)threadIdx.x; q < n; q += (int)blockDim.x) {
        const size_t i = m(q);
        const float x = first ? x_in[i] : x_acc[i];
        float v[kDownPartsMax];
#pragma unroll
        for (int p = 0; p < kDownPartsMax; ++p)
            v[p] = p < splits ? __hip_atomic_load(part + (size_t)p * stride + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                              : 0.f;
        float y = 0.f;
#pragma unroll
        for (int p = 0; p < kDownPartsMax; ++p)
            if (p < splits) y += v[p];
        x_acc[i] = x + y;
    }
}

constexpr int kWavesDn = 16;  // down: waves per workgroup
constexpr int kDnTiles = 4;   // down: 16-column tiles per workgroup, at most (d is a multiple of 64)

// ---- down projection ------------------------------------------------------------------------------------
// One workgroup per NT adjacent 16-column tiles of y and part of the list; its waves share
// that part's work items.  The down piece of a block for one tile is [blk/8][16][8]: a chunk
// of 8 neurons is 256 contiguous bytes, 16 columns of 16 bytes, and the pieces of adjacent tiles
// are adjacent.  An item is four consecutive chunks of the part's neurons in list order (a K step
// of 32; lane group l / 16 holds chunk l / 16, so an item may cross from one entry into the next
// and any block size works), for every tile of the workgroup: a wave loads the item's activations
// once for NT weight fragments.  Those reads come from L2 but through the same per-CU path
// as the weights, which bounds these kernels: at 8 tokens they are a quarter of the weights'
// bytes at 4 tiles, and half at 2.  With the sum over parts, 13B shape at B = 8 (138 blocks, 91
// MB) 24.2 -> 20.5 us, Mistral-7B shape at B = 4 with a ReLU gate (105 blocks, 110 MB) 31.8 ->
// 24 us against two tiles and eight parts.
//
// The 16 columns of operand B hold the activations' parts: BP (4 or 8) tokens each, part
// (l % 16) / BP (+ 16 / BP in a second fragment, for three parts of 8 tokens).  float16 parts are
// scaled per token by the largest magnitude the wave has met so far (a power of two; the sums
// are rescaled when it grows), so that they do not overflow, and each part by 2^11 against the one
// before (the bits they hold: as for the gate/up kernel's slices).  Two items are in flight per wave.
//
// With splits > 1 the list range is cut into `splits` equal parts (workgroup group + n_groups *
// part); each part's sum goes to part_out[part][token][column] and finish_parts adds the parts
// in order.  A list of up to one item per wave is not: the host chooses by the list's capacity, and
// there the sum over parts costs 1 to 2 us (a sparse step of 2880 x 7720 in blocks of 40 at B = 4, 9 of
// 193 blocks listed: 16.0 -> 14.9 us; 1984 x 5280 in blocks of 24, 11 of 220: 13.9 -> 12.5).
// Waves a workgroup: 8 where the parts take two fragments of several tiles, whose sums and operands do
// not fit the 128 registers that 16 waves leave a lane (7B shape in bfloat16 at B = 8, 172 blocks: with
// 6 registers spilled 23.8 us, 21.2 on 8 waves).
template <int P, int BP, int NT>
constexpr int kDnWaves = P * BP > 16 && NT > 1 ? 8 : kWavesDn;

template <ls_dtype T, int P, int BP, int NT>
__global__ __launch_bounds__((64 * kDnWaves<P, BP, NT>)) void down_mfma_kernel(
    const uint8_t* __restrict__ blocks, size_t block_bytes, const int32_t* __restrict__ slot_table,
    const float* __restrict__ a_buf, int B, int F, int d, int blk, int n_blk,
    const int32_t* __restrict__ idx, const int32_t* __restrict__ count, int begin, int end,
    const float* __restrict__ x_in, float* __restrict__ x_acc, int splits,
    float* __restrict__ part_out, uint32_t* __restrict__ cnt, uint32_t cpe_magic) {
    using S = Split<T>;
    typedef typename S::vec vec;
    constexpr int PF = 16 / BP;              // parts of one fragment
    constexpr int NF = (P + PF - 1) / PF;
    const int n_groups = d / (kColTile * NT);
    const int grp = (int)blockIdx.x % n_groups, sp = (int)blockIdx.x / n_groups;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    constexpr int n_waves = kDnWaves<P, BP, NT>;
    const int len = max(0, list_end_m(count, end, n_blk) - begin);
    if ((long)len * blk <= 32 * n_waves) {  // every item has a wave: not cut
        if (sp > 0) return;
        splits = 1;
    }
    const int e0 = begin + (int)((long)len * sp / splits);
    const int e1 = begin + (int)((long)len * (sp + 1) / splits);
    const size_t piece = (size_t)blk * kColTile * 2;  // bytes of one tile's piece
    const size_t down_off = (size_t)2 * blk * d * 2 + (size_t)grp * NT * piece + (size_t)(lane & 15) * 16;
    // the cache slot of every entry of the part (-1: invalid id or absent), resolved once
    __shared__ int slots[kMaxBlocks];
    for (int e = e0 + (int)threadIdx.x; e < e1; e += (int)blockDim.x) {
        const int b = idx[e];
        slots[e - e0] = (b < 0 || b >= n_blk) ? -1 : (slot_table ? slot_table[b] : b);
    }
    __syncthreads();
    const int col = lane & 15;
    const int tok = col & (BP - 1), prt = col / BP;
    const uint32_t cpe = (uint32_t)blk / 8u;  // chunks per entry
    const uint32_t chunks = (uint32_t)(e1 - e0) * cpe;
    const int items = (int)((chunks + 3u) / 4u);
    const float* arow = a_buf + (size_t)(tok < B ? tok : 0) * F + (size_t)e0 * blk;

    struct Item {
        u32x4 w[NT];
        f32x4 a[2];
        bool live;
    };
    auto load_item = [&](Item& t, int it) {
        const uint32_t f = 4u * (uint32_t)it + (uint32_t)(lane >> 4);
        t.live = f < chunks;
        const uint32_t fc = t.live ? f : 0u;
        // f / cpe by multiplication (cpe_magic = ceil(2^32 / cpe), exact while chunks cpe < 2^32)
        const uint32_t e = cpe_magic ? __umulhi(fc, cpe_magic) : fc / cpe;
        const int slot = slots[e];
        t.live = t.live && slot >= 0;  // an invalid or absent block contributes nothing
        const uint8_t* src = blocks + (size_t)(slot < 0 ? 0 : slot) * block_bytes + down_off + (size_t)(fc - e * cpe) * 256;
#pragma unroll
        for (int j = 0; j < NT; ++j) t.w[j] = ld_stream(reinterpret_cast<const u32x4*>(src + j * piece));
        const f32x4* ap = reinterpret_cast<const f32x4*>(arow + (size_t)fc * 8);
        t.a[0] = ap[0];
        t.a[1] = ap[1];
    };
    f32x4v c[NT][NF];
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int f = 0; f < NF; ++f) c[j][f] = f32x4v{0.f, 0.f, 0.f, 0.f};
    // float16: exponent of the scale (of the largest magnitude so far, not below 2^-100), the same
    // in a token's lanes, and the magnitude that it holds up to
    int ex = -100;
    float s1 = ldexpf(1.f, -ex), limit = ldexpf(1.f, ex + 1);
    auto run_item = [&](Item& t) {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = t.live ? t.a[i >> 2][i & 3] : 0.f;
        float mx = 0.f;
#pragma unroll
        for (int i = 0; i < 8; i += 2) mx = fmaxf(fmaxf(mx, fabsf(v[i])), fabsf(v[i + 1]));
        bool inf_met = false;
        if (__any(T == LS_F16 ? mx >= limit : mx == INFINITY)) {  // rare
            inf_met = __any(mx == INFINITY);
            mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            if (T == LS_F16) {
                const int eg = max(ex, min(127, (int)((__float_as_uint(mx) >> 23) & 0xffu) - 127));
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int f = 0; f < NF; ++f)
#pragma unroll
                        for (int i = 0; i < 4; ++i) c[j][f][i] = ldexpf(c[j][f][i], ex - eg);
                ex = eg;
                s1 = ldexpf(1.f, -ex);
                limit = ldexpf(1.f, ex + 1);
            }
            if (prt > 0) {  // an infinity is its first part alone
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = fabsf(v[i]) < INFINITY ? v[i] : 0.f;
            }
        }
        // a second fragment holds third parts (its second half is never used) in lanes that keep an
        // infinity for the first: it has none
        auto third_part = [&](u32x4 (&words)[NF]) {
            if constexpr (NF > 1) {
                if (inf_met)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        words[1][q] &= (fabsf(v[2 * q]) < INFINITY ? 0xffffu : 0u) |
                                       (fabsf(v[2 * q + 1]) < INFINITY ? 0xffff0000u : 0u);
            }
        };
        vec pt[NF];
        if constexpr (T == LS_F16) {
            typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
            u32x4 words[NF];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float a0 = v[2 * q], a1 = v[2 * q + 1];
                const f16x2 h = {(_Float16)(a0 * s1), (_Float16)(a1 * s1)};
                const float s2 = s1 * 2048.f;
                const float r0 = fmaf((float)h.x, -2048.f, a0 * s2), r1 = fmaf((float)h.y, -2048.f, a1 * s2);
                const f16x2 m = {(_Float16)r0, (_Float16)r1};
                const uint32_t w0 = __builtin_bit_cast(uint32_t, h), w1 = __builtin_bit_cast(uint32_t, m);
                if constexpr (P == 2) {
                    words[0][q] = prt ? w1 : w0;
                } else {
                    const f16x2 l = {(_Float16)fmaf((float)m.x, -2048.f, r0 * 2048.f),
                                     (_Float16)fmaf((float)m.y, -2048.f, r1 * 2048.f)};
                    const uint32_t w2 = __builtin_bit_cast(uint32_t, l);
                    words[0][q] = prt == 0 ? w0 : (prt == 1 ? w1 : w2);
                    if constexpr (NF > 1) words[1][q] = w2;
                }
            }
            third_part(words);
#pragma unroll
            for (int f = 0; f < NF; ++f) pt[f] = S::from_raw(words[f]);
        } else {
            auto rest = [](float x) { return x - __uint_as_float(__float_as_uint(x) & 0xffff0000u); };
            u32x4 words[NF];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float a0 = v[2 * q], a1 = v[2 * q + 1];
                const float b0 = rest(a0), b1 = rest(a1), d0 = rest(b0), d1 = rest(b1);
                auto pack = [](float lo, float hi) { return (__float_as_uint(lo) >> 16) | (__float_as_uint(hi) & 0xffff0000u); };
                const uint32_t w0 = pack(a0, a1), w1 = pack(b0, b1), w2 = pack(d0, d1);
                words[0][q] = prt == 0 ? w0 : (prt == 1 ? w1 : w2);
                if constexpr (NF > 1) words[1][q] = w2;
            }
            third_part(words);
#pragma unroll
            for (int f = 0; f < NF; ++f) pt[f] = S::from_raw(words[f]);
        }
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            u32x4 raw = t.w[j];
#pragma unroll
            for (int i = 0; i < 4; ++i) raw[i] = t.live ? raw[i] : 0u;
            const vec wv = S::from_raw(raw);
#pragma unroll
            for (int f = 0; f < NF; ++f) c[j][f] = S::mfma(wv, pt[f], c[j][f]);
        }
    };
    Item ta, tb;
    int it = wave;
    if (it < items) load_item(ta, it);
    for (; it < items; it += 2 * n_waves) {
        if (it + n_waves < items) load_item(tb, it + n_waves);
        run_item(ta);
        if (it + n_waves >= items) break;
        if (it + 2 * n_waves < items) load_item(ta, it + 2 * n_waves);
        run_item(tb);
    }
    // lane l: columns 4 (l / 16) + i of tile j, slot l % 16
    __shared__ __attribute__((aligned(16))) float part[n_waves][NT][NF][16][16];
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            f32x4v v = c[j][f];
            if (T == LS_F16) v *= ldexpf(1.f, ex - Part<T>::kShift * (f * PF + prt));
            *reinterpret_cast<f32x4v*>(&part[wave][j][f][col][4 * (lane >> 4)]) = v;
        }
    __syncthreads();
    for (int q = (int)threadIdx.x; q < NT * 16 * B; q += (int)blockDim.x) {
        const int t = q / (16 * NT), j = (q / 16) % NT, m16 = q % 16;
        float yp[P];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            float yw[n_waves];
#pragma unroll
            for (int w = 0; w < n_waves; ++w) yw[w] = part[w][j][p / PF][(p % PF) * BP + t][m16];
            yp[p] = tree_sum<n_waves>(yw);
        }
        float y = yp[P - 1];
#pragma unroll
        for (int p = P - 2; p >= 0; --p) y += yp[p];
        const size_t m = (size_t)t * d + (size_t)(grp * NT + j) * kColTile + m16;
        if (splits == 1)
            x_acc[m] = (begin == 0 ? x_in[m] : x_acc[m]) + y;
        else
            __hip_atomic_store(part_out + (size_t)sp * B * d + m, y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (splits > 1)
        finish_parts(part_out, splits, (size_t)B * d, NT * 16 * B,
                     [&](int q) { return (size_t)(q / (16 * NT)) * d + (size_t)grp * NT * kColTile + q % (16 * NT); },
                     x_in, x_acc, begin == 0, cnt + grp);
}

// The batched down projection of thresholded gates (keeps_order below): one workgroup per NT
// adjacent 16-column tiles of y and part of the list; its waves split that part's entries.  The
// down piece of a block for one 16-column tile is [blk/8][16][8]:
// K step s of an entry is the contiguous kilobyte of chunks 64 s .. 64 s + 63, exactly one A
// fragment, and the pieces of adjacent tiles are adjacent.  A wave loads the activations of
// a work item once for its NT fragments: every workgroup reads the whole part's activations
// (L2 hits, but through the same per-CU memory path as the weights, which bounds these
// kernels), so NT tiles per workgroup divide those reads by NT.
// With splits > 1 the list range is cut into `splits` equal parts (workgroup
// tile + n_tiles * part) so that the workgroup count is a multiple of the CU count even when
// the tile count is not; each part's sum goes to part_out[part][token][column] and
// finish_parts adds the parts in order.  The wave count is blockDim.x / 64 (at most
// kWavesDn, and at most kWavesDn / NT with NT > 1).
template <ls_dtype T, int NT, int KU>
__global__ __launch_bounds__(64 * kWavesDn) void down_ordered_kernel(
    const uint8_t* __restrict__ blocks, size_t block_bytes, const int32_t* __restrict__ slot_table,
    const float* __restrict__ a_buf, int B, int F, int d, int blk, int n_blk,
    const int32_t* __restrict__ idx, const int32_t* __restrict__ count, int begin, int end,
    const float* __restrict__ x_in, float* __restrict__ x_acc, int splits,
    float* __restrict__ part_out, uint32_t* __restrict__ cnt) {
    using S = Split<T>;
    constexpr int kU = KU;
    const int n_tiles = d / (kColTile * NT);
    const int tile = (int)blockIdx.x % n_tiles, sp = (int)blockIdx.x / n_tiles;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int n_waves = (int)(blockDim.x >> 6);
    const int len = max(0, list_end_m(count, end, n_blk) - begin);
    const int e0 = begin + (int)((long)len * sp / splits);
    const int e1 = begin + (int)((long)len * (sp + 1) / splits);
    const size_t down_off = (size_t)2 * blk * d * 2 + (size_t)tile * NT * blk * kColTile * 2;
    const int piece_v = blk * kColTile * 2 / 16;  // 16-byte vectors of one tile's piece
    const int ksteps = blk / 32;
    const int tok = lane & 15;
    const bool tok_ok = tok < B;
    // the cache slot of every entry of the part (-1: invalid id or absent), resolved once so
    // that each work item waits only for its weight load
    __shared__ int slots[kMaxBlocks];
    for (int e = e0 + (int)threadIdx.x; e < e1; e += (int)blockDim.x) {
        const int b = idx[e];
        slots[e - e0] = (b < 0 || b >= n_blk) ? -1 : (slot_table ? slot_table[b] : b);
    }
    __syncthreads();
    f32x4v c[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) c[j] = f32x4v{0.f, 0.f, 0.f, 0.f};
    // work items (entry, K step) of the part, dealt to the waves round-robin; kU items per
    // wave are in flight together
    const long items = (long)(e1 - e0) * ksteps;
    for (long i0 = wave; i0 < items; i0 += (long)n_waves * kU) {
        const u32x4* src[kU];
        const float* arow[kU];
        bool live[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const long it = i0 + (long)n_waves * u;
            const int e = e0 + (int)(it / ksteps), s = (int)(it % ksteps);
            live[u] = it < items;
            const int slot = live[u] ? slots[e - e0] : -1;
            live[u] = live[u] && slot >= 0;  // an invalid or absent block contributes nothing
            src[u] = reinterpret_cast<const u32x4*>(blocks + (size_t)(slot < 0 ? 0 : slot) * block_bytes +
                                                    down_off) + 64 * s + lane;
            arow[u] = a_buf + (size_t)(tok_ok ? tok : 0) * F + (size_t)e * blk + 32 * s + 8 * (lane >> 4);
        }
        u32x4 w[kU][NT];
        f32x4 av[kU][2];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < NT; ++j) w[u][j] = live[u] ? ld_stream(src[u] + j * piece_v) : u32x4{0u, 0u, 0u, 0u};
            av[u][0] = live[u] && tok_ok ? reinterpret_cast<const f32x4*>(arow[u])[0] : z;
            av[u][1] = live[u] && tok_ok ? reinterpret_cast<const f32x4*>(arow[u])[1] : z;
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const float xv[8] = {av[u][0].x, av[u][0].y, av[u][0].z, av[u][0].w,
                                 av[u][1].x, av[u][1].y, av[u][1].z, av[u][1].w};
            typename S::vec hi, lo;
            S::run(xv, hi, lo);
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                const typename S::vec wv = S::from_raw(w[u][j]);
                c[j] = S::mfma(wv, hi, c[j]);
                c[j] = S::mfma(wv, lo, c[j]);
            }
        }
    }
    // lane l holds columns 4 (l / 16) + i of tile j for token l % 16
    __shared__ float part[NT == 1 ? kWavesDn : kWavesDn / NT][NT][16][16];
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) part[wave][j][4 * (lane >> 4) + i][lane & 15] = c[j][i];
    __syncthreads();
    for (int q = (int)threadIdx.x; q < NT * 16 * B; q += (int)blockDim.x) {
        const int j = q / (16 * B), t = (q / 16) % B, col = q % 16;
        float y = 0.f;
        for (int w = 0; w < n_waves; ++w) y += part[w][j][col][t];
        const size_t m = (size_t)t * d + (size_t)(tile * NT + j) * kColTile + col;
        if (splits == 1)
            x_acc[m] = (begin == 0 ? x_in[m] : x_acc[m]) + y;
        else
            __hip_atomic_store(part_out + (size_t)sp * B * d + m, y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (splits > 1)
        finish_parts(part_out, splits, (size_t)B * d, NT * 16 * B,
                     [&](int q) { return (size_t)(q / (16 * NT)) * d + (size_t)tile * NT * kColTile + q % (16 * NT); },
                     x_in, x_acc, begin == 0, cnt + tile);
}

}  // namespace

// The resident kernel's registers hold up to 16 steps of 64 values a wave beside the loads in
// flight, but only 12 where the parts take three fragments (three parts, 5 to 8 tokens).
static bool resident_ok(const Shape& s, int B) {
    const int nk = input_parts(s) == 3 && B > 4 ? 12 : 16;
    return s.d <= 64 * nk * kGuWaves;
}

// A thresholded gate turns the last bit of a sum into a neuron kept or dropped, and in a stack a
// neuron into another block of the next layer's list.  Where such a gate was batched on the
// matrix cores with two-part activations (whole K steps a block), the sums keep the order and
// the parts they have always had, so its decisions stay the same.
static bool keeps_order(const Shape& s) { return s.act == LS_ACT_SWIGLU_THRESH && s.blk % 32 == 0; }

// Whether gate/up and down run here for B tokens and a list of up to n entries.  Two and three stay on
// the vector ALU: there the kernels' start (about 4 us more) pays only for long lists (7B shape in
// float16, 2 tokens: 86 blocks 35.5 us on the vector ALU, 31.2 here; 10 blocks 11.9 and 15.1), and the
// host knows a list's capacity, not its length.  With four and five, blocks that are no multiple of 32
// stay there where the capacity itself is short: 2880 values a row and blocks of 40 in float16, 4 tokens,
// 9 blocks 11.7 us on the vector ALU, 14.0 here, 48 blocks 18.4 and 17.8; 5 tokens, 24 blocks 14.5 and
// 15.2; 1984 and blocks of 24, 5 tokens, 27 blocks 12.1 and 12.5, 55 15.8 and 14.1.  (A threshold's
// capacity is all blocks: those calls take 1 to 3 us more than there with under a sixth of them
// listed, 2.5 less with a quarter, 13 with half.)  At 6 tokens and more every length is faster here.
bool mfma_path(const Shape& s, int B, int n) {
    if (B < kMfmaMinBatch || s.dtype == LS_F32) return false;
    if (s.blk % 32 == 0) return true;
    return resident_ok(s, B) && (B > 5 || (double)n * s.blk * s.d > (B == 4 ? 2.5e6 : 1.5e6));
}

// Steps of the shortest slice that eight waves or fewer cover a row with (0: none does).
static int slice_steps(int d) {
    for (int nk : {4, 6, 8, 10, 12, 16})
        if (d <= 64 * nk * kGuWaves) return nk;
    return 0;
}

template <ls_dtype T, int P, int BP>
static hipError_t gateup_resident_bp(const Shape& s, const LayerDev& L, const int32_t* slot_table, const float* x, int B,
                                     const int32_t* idx, const int32_t* count, int begin, int end, float* a_buf,
                                     const SplitJob* job, hipStream_t st) {
    const size_t bb = s.block_elems * elem_size(s.dtype);
    const int steps = s.d / 64;
    const long groups = (long)(end - begin) * (s.blk / 8);
    const int cus = std::max(1, cu_count());
#define LS_GUR_K(NK, FULL, PRE)                                                                                        \
    hipLaunchKernelGGL((gateup_mfma_kernel<T, P, NK, BP, FULL, PRE>), dim3((unsigned)grid), dim3(64 * W), 0, st, L.blocks,  \
                       bb, slot_table, L.bias, L.threshold, x, B, s.d, s.blk, s.n_blk, s.F, idx, count, begin, end,    \
                       a_buf, s.act == LS_ACT_REGLU ? 1 : 0, s.prenorm, reinterpret_cast<const u32x4*>(job ? job->frag : nullptr),      \
                       job ? job->meta : nullptr)
#define LS_GUR(NK)                                                                                                     \
    do {                                                                                                               \
        const int W = (steps + NK - 1) / NK;                                                                           \
        const long grid = std::min<long>(groups, (long)cus * std::max(1, kGuWaves / W));                               \
        if (steps == W * NK) { if (job) LS_GUR_K(NK, true, true); else LS_GUR_K(NK, true, false); }                    \
        else { if (job) LS_GUR_K(NK, false, true); else LS_GUR_K(NK, false, false); }                                  \
    } while (0)
    switch (slice_steps(s.d)) {
        case 4: LS_GUR(4); break;
        case 6: LS_GUR(6); break;
        case 8: LS_GUR(8); break;
        case 10: LS_GUR(10); break;
        case 12: LS_GUR(12); break;
        case 16:
            if constexpr (P == 2 || BP <= 4) { LS_GUR(16); break; }
            return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
#undef LS_GUR
#undef LS_GUR_K
    return hipGetLastError();
}

template <ls_dtype T, int P>
static hipError_t gateup_resident_t(const Shape& s, const LayerDev& L, const int32_t* slot_table, const float* x, int B,
                                    const int32_t* idx, const int32_t* count, int begin, int end, float* a_buf,
                                    const SplitJob* job, hipStream_t st) {
    if (B <= 4) return gateup_resident_bp<T, P, 4>(s, L, slot_table, x, B, idx, count, begin, end, a_buf, job, st);
    return gateup_resident_bp<T, P, 8>(s, L, slot_table, x, B, idx, count, begin, end, a_buf, job, st);
}

bool split_job(const Shape& s, int B, int n, const float* x, void* buf, SplitJob* job) {
    if (!buf || !s.batch_mfma || s.zero_skip || !mfma_path(s, B, n) || keeps_order(s) || !resident_ok(s, B))
        return false;
    const int NK = slice_steps(s.d), W = (s.d / 64 + NK - 1) / NK;
    job->x = x;
    job->meta = static_cast<float*>(buf);
    job->frag = job->meta + 2 * 8 * kSplitSlices;
    job->B = B;
    job->d = s.d;
    job->NK = NK;
    job->W = W;
    job->bp = B <= 4 ? 4 : 8;
    job->bf16 = s.dtype == LS_BF16;
    job->parts = input_parts(s);
    return true;
}

size_t split_bytes(const Shape& s, int max_batch) {
    if (s.dtype == LS_F32 || max_batch < kMfmaMinBatch) return 0;
    const int NK = slice_steps(s.d);
    if (!NK) return 0;
    const size_t W = (size_t)(s.d / 64 + NK - 1) / NK;
    return 2 * 8 * kSplitSlices * sizeof(float) + W * NK * 3 * 1024;  // up to three fragments
}

hipError_t launch_gateup_mfma(const Shape& s, const LayerDev& L, const int32_t* slot_table,
                              const float* x, int B, const int32_t* idx, const int32_t* count,
                              int begin, int end, float* a_buf, const SplitJob* job, hipStream_t st) {
    if (end <= begin) return hipSuccess;
    if (!keeps_order(s) && resident_ok(s, B)) {
        auto launch = s.dtype == LS_BF16 ? gateup_resident_t<LS_BF16, 3>
                    : input_parts(s) == 3 ? gateup_resident_t<LS_F16, 3>
                                          : gateup_resident_t<LS_F16, 2>;
        return launch(s, L, slot_table, x, B, idx, count, begin, end, a_buf, job, st);
    }
    const long groups = (long)(end - begin) * (s.blk / 16);
    const size_t bb = s.block_elems * elem_size(s.dtype);
    const dim3 grid((unsigned)groups), blk(64 * kWaves);
    const bool relu = s.act == LS_ACT_REGLU;
#define LS_GUM(TT, AA)                                                                            \
    do {                                                                                          \
        if (s.prenorm)                                                                            \
            hipLaunchKernelGGL((gateup_staged_kernel<TT, AA, true>), grid, blk, 0, st, L.blocks, bb, \
                               slot_table, L.bias, L.threshold, x, B, s.d, s.blk, s.n_blk, s.F,   \
                               idx, count, begin, end, a_buf);                                    \
        else                                                                                      \
            hipLaunchKernelGGL((gateup_staged_kernel<TT, AA, false>), grid, blk, 0, st, L.blocks,   \
                               bb, slot_table, L.bias, L.threshold, x, B, s.d, s.blk, s.n_blk,    \
                               s.F, idx, count, begin, end, a_buf);                               \
    } while (0)
    if (s.dtype == LS_F16) {
        if (relu) LS_GUM(LS_F16, LS_ACT_REGLU);
        else LS_GUM(LS_F16, LS_ACT_SWIGLU_THRESH);
    } else if (s.dtype == LS_BF16) {
        if (relu) LS_GUM(LS_BF16, LS_ACT_REGLU);
        else LS_GUM(LS_BF16, LS_ACT_SWIGLU_THRESH);
    } else {
        return hipErrorInvalidValue;
    }
#undef LS_GUM
    return hipGetLastError();
}

// List parts of the down projection: as many as the compute units hold at once, one workgroup of
// 64 columns and one part each.
static int down_splits(const Shape& s) {
    return std::min(kDownPartsMax, std::max(1, cu_count() / (s.d / (kColTile * kDnTiles))));
}

template <ls_dtype T, int P, int BP, int NT>
static void down_mfma_nt(const Shape& s, const LayerDev& L, const int32_t* slot_table, const float* a_buf, int B,
                         const int32_t* idx, const int32_t* count, int begin, int end, const float* x_in, float* x_acc,
                         int splits, float* part, uint32_t* cnt, hipStream_t st) {
    const size_t bb = s.block_elems * elem_size(s.dtype);
    const uint32_t cpe = (uint32_t)s.blk / 8u;
    const bool exact = cpe > 1 && (uint64_t)(s.F / 8) * cpe < (1ull << 32);
    const uint32_t magic = exact ? 0xffffffffu / cpe + 1u : 0u;
    hipLaunchKernelGGL((down_mfma_kernel<T, P, BP, NT>), dim3((unsigned)(s.d / (kColTile * NT) * splits)),
                       dim3(64 * kDnWaves<P, BP, NT>), 0, st, L.blocks, bb, slot_table, a_buf, B, s.F, s.d, s.blk, s.n_blk, idx,
                       count, begin, end, x_in, x_acc, splits, part, cnt, magic);
}

// One tile per workgroup and the whole list needs no sum over parts (2 to 3 us) but reads and
// splits the activations once per 16 columns instead of once per 64, and its 16 waves leave room
// for one workgroup per compute unit.  Measured at the longest list the call allows: d = 4096,
// B = 4: 5 MB of weights 7.4 us against 9.0 with four tiles, 22 MB 12.1 / 12.0, 45 MB 15.1 / 15.4;
// d = 1984, B = 8: 6 MB 9.4 / 10, 17 MB 15.4 / 11.5; d = 5120 (320 tiles, 256 units; with 2 tokens,
// which run on the vector ALU now): 71 MB 32 / 18.  (A longer capacity with a short list: not cut, above.)
static bool down_one_tile(const Shape& s, int B, int n) {
    return s.d / kColTile <= cu_count() && 2.0 * B * n * s.blk * s.d <= 80e6;
}

template <ls_dtype T, int P, int BP>
static void down_mfma_bp(const Shape& s, const LayerDev& L, const int32_t* slot_table, const float* a_buf, int B,
                         const int32_t* idx, const int32_t* count, int begin, int end, const float* x_in, float* x_acc,
                         int splits, float* part, uint32_t* cnt, bool one, hipStream_t st) {
    if (one)
        down_mfma_nt<T, P, BP, 1>(s, L, slot_table, a_buf, B, idx, count, begin, end, x_in, x_acc, 1, part, cnt, st);
    else
        down_mfma_nt<T, P, BP, kDnTiles>(s, L, slot_table, a_buf, B, idx, count, begin, end, x_in, x_acc, splits, part, cnt, st);
}

// The order of a thresholded gate's down projection: list parts and waves by shape (tiles that
// do not fill whole rounds of the CUs and 128-row blocks take 8 parts of 4 waves, 64-row blocks
// at B = 8 2 parts of 8, the rest one part of 16); the tiles per workgroup are free.
template <ls_dtype T>
static void down_ordered_t(const Shape& s, const LayerDev& L, const int32_t* slot_table, const float* a_buf, int B,
                          const int32_t* idx, const int32_t* count, int begin, int end, const float* x_in,
                          float* x_acc, float* part, uint32_t* cnt, hipStream_t st) {
    const size_t bb = s.block_elems * elem_size(s.dtype);
    const int cus = cu_count() > 0 ? cu_count() : 256;
    int splits = 1, waves = kWavesDn;
    if (part) {
        if ((s.d / kColTile) % cus != 0 || s.blk >= 128) splits = 8, waves = 4;
        else if (B >= 8 && (s.d / (2 * kColTile)) * 2 % cus == 0) splits = 2, waves = 8;
    }
#define LS_DNO(NT, KU)                                                                                                 \
    hipLaunchKernelGGL((down_ordered_kernel<T, NT, KU>), dim3((unsigned)(s.d / (kColTile * NT) * splits)),             \
                       dim3(64 * waves), 0, st, L.blocks, bb, slot_table, a_buf, B, s.F, s.d, s.blk, s.n_blk, idx,     \
                       count, begin, end, x_in, x_acc, splits, part, cnt)
    if (splits == 8) LS_DNO(4, 2);
    else if (splits == 2) LS_DNO(2, 4);
    else LS_DNO(1, 2);
#undef LS_DNO
}

hipError_t launch_down_mfma(const Shape& s, const LayerDev& L, const int32_t* slot_table,
                            const float* a_buf, int B, const int32_t* idx, const int32_t* count,
                            int begin, int end, const float* x_in, float* x_acc, float* part,
                            uint32_t* cnt, hipStream_t st) {
    const bool one = down_one_tile(s, B, end - begin);
    const int splits = part && !one ? down_splits(s) : 1;
    if (keeps_order(s) && s.dtype == LS_F16)
        down_ordered_t<LS_F16>(s, L, slot_table, a_buf, B, idx, count, begin, end, x_in, x_acc, part, cnt, st);
    else if (keeps_order(s) && s.dtype == LS_BF16)
        down_ordered_t<LS_BF16>(s, L, slot_table, a_buf, B, idx, count, begin, end, x_in, x_acc, part, cnt, st);
    else if (s.dtype == LS_F16 || s.dtype == LS_BF16) {
        auto launch = s.dtype == LS_BF16      ? (B <= 4 ? down_mfma_bp<LS_BF16, 3, 4> : down_mfma_bp<LS_BF16, 3, 8>)
                      : input_parts(s) == 3 ? (B <= 4 ? down_mfma_bp<LS_F16, 3, 4> : down_mfma_bp<LS_F16, 3, 8>)
                                            : down_mfma_bp<LS_F16, 2, 8>;
        launch(s, L, slot_table, a_buf, B, idx, count, begin, end, x_in, x_acc, splits, part, cnt, one, st);
    } else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace ls
