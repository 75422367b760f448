// ls_split.h - fp32 inputs as 16-bit parts in matrix-core operand order, for the resident
// gate/up kernel (ls_mfma.hip) and for the selection launch that prepares them (ls_kernels.hip).
#pragma once

#include "ls_device.h"
#include "ls_internal.h"

namespace ls {

// sum of N (a power of two) values, pairwise
template <int N>
__device__ __forceinline__ float tree_sum(const float (&v)[N]) {
    float t[N];
#pragma unroll
    for (int i = 0; i < N; ++i) t[i] = v[i];
#pragma unroll
    for (int n = N / 2; n > 0; n /= 2)
#pragma unroll
        for (int i = 0; i < n; ++i) t[i] += t[i + n];
    return t[0];
}

// Parts of values, two at a time (a word holds the pair's 16-bit parts).  pack() takes the
// leading parts, rest() the (scaled) remainder; a value that is not finite leaves none.  How many
// parts P: input_parts (ls_internal.h).
template <ls_dtype T>
struct Part;
template <>
struct Part<LS_F16> {
    static constexpr int kShift = 11;  // each part is scaled by 2^11 against the one before
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    __device__ static inline uint32_t pack(float a, float b) {
        const f16x2 h = {(_Float16)a, (_Float16)b};
        return __builtin_bit_cast(uint32_t, h);
    }
    __device__ static inline float rest(float v) {
        const float r = (v - (float)(_Float16)v) * 2048.f;
        return fabsf(v) < INFINITY ? r : 0.f;
    }
};
template <>
struct Part<LS_BF16> {
    static constexpr int kShift = 0;   // (8 bits each, cut off: three are exact)
    // the upper halves of two values (a NaN stays one: its quiet bit is set)
    __device__ static inline uint32_t pack(float a, float b) {
        const uint32_t ua = __float_as_uint(a) | (a != a ? 0x400000u : 0u);
        const uint32_t ub = __float_as_uint(b) | (b != b ? 0x400000u : 0u);
        return (ua >> 16) | (ub & 0xffff0000u);
    }
    __device__ static inline float rest(float v) {
        const float r = v - __uint_as_float(__float_as_uint(v) & 0xffff0000u);
        return fabsf(v) < INFINITY ? r : 0.f;
    }
};

// One step of 64 values: this lane's 8 values x (chunk 2 (lane / 16) + (lane / 8) % 2 of its token) as
// the words of its operand in each fragment, scaled by 2^-ex first (float16); the values' squares
// go into the four chains s4.
template <ls_dtype T, int P, int BP>
__device__ __forceinline__ void split_step(const f32x4 (&x)[2], int ex, int lane, float (&s4)[4],
                                           u32x4 (&words)[(P * BP + 7) / 8]) {
    constexpr int NF = (P * BP + 7) / 8;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float v0 = x[j >> 1][(2 * j) & 3], v1 = x[j >> 1][(2 * j + 1) & 3];
        s4[(2 * j) & 3] = fmaf(v0, v0, s4[(2 * j) & 3]);
        s4[(2 * j + 1) & 3] = fmaf(v1, v1, s4[(2 * j + 1) & 3]);
        if (T == LS_F16) v0 = ldexpf(v0, -ex), v1 = ldexpf(v1, -ex);
        // slot q of fragment f is part (8 f + q) / BP
        float p0[P], p1[P];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            p0[p] = v0;
            p1[p] = v1;
            if (p + 1 < P) v0 = Part<T>::rest(v0), v1 = Part<T>::rest(v1);
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            float a = p0[f * 8 / BP], b = p1[f * 8 / BP];
#pragma unroll
            for (int p = f * 8 / BP + 1; p < P && p * BP < f * 8 + 8; ++p) {
                const bool mine = (lane & 7) >= p * BP - f * 8;
                a = mine ? p0[p] : a;
                b = mine ? p1[p] : b;
            }
            words[f][j] = Part<T>::pack(a, b);
        }
    }
}

// exponent of the scale for a slice whose largest finite magnitude is mx (a subnormal one: -127)
__device__ __forceinline__ int split_exponent(float mx) {
    return mx > 0.f ? (int)((__float_as_uint(mx) >> 23) & 0xffu) - 127 : 0;
}

// One wave: slice `w` of a job, written where the resident kernel's wave w reads it.  The loads of
// four steps are in flight together.
template <ls_dtype T, int P, int BP>
__device__ __forceinline__ void split_slice(const SplitJob& p, int w, int lane) {
    constexpr int NF = (P * BP + 7) / 8;
    const int steps = p.d / 64;
    const int s0 = steps * w / p.W, nst = steps * (w + 1) / p.W - s0;
    const int tok = (lane & 7) & (BP - 1);
    const float* xr = p.x + (size_t)(tok < p.B ? tok : 0) * p.d + (size_t)s0 * 64 + 16 * (lane >> 4) + 8 * ((lane >> 3) & 1);
    auto load4 = [&](int s, f32x4 (&xv)[4][2]) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const f32x4* src = reinterpret_cast<const f32x4*>(xr + 64 * (s + u < nst ? s + u : 0));
            xv[u][0] = src[0];
            xv[u][1] = src[1];
        }
    };
    float mx = 0.f;
    if (T == LS_F16) {
#pragma unroll 1
        for (int s = 0; s < nst; s += 4) {  // (a step past the slice repeats its first)
            f32x4 xv[4][2];
            load4(s, xv);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float v = fabsf(xv[u][i >> 2][i & 3]);
                    if (v < INFINITY) mx = fmaxf(mx, v);
                }
        }
#pragma unroll
        for (int off = 8; off < 64; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    }
    const int ex = T == LS_F16 ? split_exponent(mx) : 0;
    float s4[4] = {0.f, 0.f, 0.f, 0.f};
    u32x4* out = reinterpret_cast<u32x4*>(p.frag) + (size_t)w * p.NK * NF * 64 + lane;
#pragma unroll 1
    for (int s = 0; s < p.NK; s += 4) {
        f32x4 xv[4][2];
        load4(s, xv);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (s + u >= p.NK) break;
            u32x4 words[NF];
            if (s + u < nst) {
                split_step<T, P, BP>(xv[u], ex, lane, s4, words);
            } else {
#pragma unroll
                for (int f = 0; f < NF; ++f) words[f] = u32x4{0u, 0u, 0u, 0u};
            }
#pragma unroll
            for (int f = 0; f < NF; ++f) out[((s + u) * NF + f) * 64] = words[f];
        }
    }
    float ss = tree_sum<4>(s4);
#pragma unroll
    for (int off = 8; off < 64; off <<= 1) ss += __shfl_xor(ss, off, 64);
    if (lane < 8) {
        p.meta[w * 8 + lane] = ldexpf(1.f, ex);
        p.meta[kSplitSlices * 8 + w * 8 + lane] = ss;
    }
}

}  // namespace ls
