// ls_hash.hip - stacked learnable hashing predictor at inference (Sec. 3.3.1, Eq. hash_layer,
// Eq. hashfunc_layer): an alternative block scorer to the low-rank predictor.
//
// Five hashing layers with 8 hash bits each and 256-wide binary features between them.  Layer
// 1 hashes the real input with 8 real hyperplanes (8 dot products over d); layers 2-5 hash the
// previous table row with binary hyperplanes, the signed products taken as XNOR + bitcount
// (x.w = 256 - 2 popcount(x XOR w)).  A code's bucket is the code read as an 8-bit number, first
// hash bit most significant, +1 -> 1 (the paper's sign-pattern order); sign(0) = +1.  The last
// layer's bucket selects a row of 8-bit block-priority levels, the block scores.
//
// One workgroup per token.  The binary layers' tables and hyperplanes (33 KB) are copied into
// LDS while the first layer runs, so the four dependent lookups after it do not go to memory.
// The dot products are the only floating-point work: 256 partial sums of j = t, t + 256, ... with
// fused multiply-adds in order, then a pairwise halving sum gives each hash bit (a fixed order,
// so the codes are reproducible).  The kernel is bound by latency (161 KB through one compute
// unit), so the 8 hash bits are spread over four groups of 256 threads, two bits each, whose loads
// of eight steps are in flight together, and only the first two halvings cross waves: 8 tokens at
// d = 4096 with the selection after it 9.84 -> 9.34 us (this kernel 5.8 of them, the selection 4.0).
// The four binary layers run in one wave (lane b evaluates hash bit b; a ballot forms the bucket).
#include "ls_internal.h"

namespace ls {
namespace {

constexpr int kTau = 8;                // hash bits per layer
constexpr int kDh = 256;               // binary feature width
constexpr int kDhWords = kDh / 32;
constexpr int kHashLayers = 5;
constexpr int kPart = 256;             // partial sums per hash bit
constexpr int kThreads = 1024;         // kPart per pair of hash bits

// bucket of a code whose bit b (hash bit b, 1 = +1) sits in bit b of `mask`: bit b has weight
// 2^(7 - b)
__device__ __forceinline__ int bucket_of(uint64_t mask) {
    return (int)(__brev((uint32_t)(mask & 0xffu)) >> 24);
}

__global__ __launch_bounds__(kThreads) void hash_predict_kernel(int d, int nblk, const float* __restrict__ x,
                                                               const float* __restrict__ w1,
                                                               const uint32_t* __restrict__ w_bin,
                                                               const uint32_t* __restrict__ tables,
                                                               const uint8_t* __restrict__ head,
                                                               float* __restrict__ scores) {
    __shared__ float part[kTau][kPart];
    __shared__ float dots[kTau];
    __shared__ uint32_t tab[(kHashLayers - 1) * kDh * kDhWords];
    __shared__ uint32_t wb[(kHashLayers - 1) * kTau * kDhWords];
    __shared__ int last_bucket;
    const int t = threadIdx.x;
    static_assert(kThreads == kPart * kTau / 2, "two hash bits per group of threads");
    const int p = t & (kPart - 1), b0 = t / kPart * 2;  // this thread's partial sum and first hash bit
    const float* xt = x + (size_t)blockIdx.x * d;
    float acc0 = 0.f, acc1 = 0.f;
    constexpr int kSteps = 8;  // loads in flight together (16 were no faster)
    // (every thread takes the first round, also past a row shorter than kPart: the copy is its part too)
    for (int base = 0; base < d; base += kPart * kSteps) {
        const int j0 = base + p;
        float xv[kSteps];
        float2 wv[kSteps];
#pragma unroll
        for (int i = 0; i < kSteps; ++i) {
            const int j = min(j0 + kPart * i, d - 1);
            xv[i] = xt[j];
            wv[i] = *reinterpret_cast<const float2*>(w1 + (size_t)j * kTau + b0);
        }
        if (base == 0) {
            // 16-byte copies: tables 2048, hyperplanes 64
            const uint4* src = reinterpret_cast<const uint4*>(tables);
            uint4* dst = reinterpret_cast<uint4*>(tab);
            constexpr int n_tab = (kHashLayers - 1) * kDh * kDhWords / 4;
            static_assert(n_tab % kThreads == 0, "whole copies");
#pragma unroll
            for (int i = 0; i < n_tab / kThreads; ++i) dst[t + kThreads * i] = src[t + kThreads * i];
            constexpr int n_wb = (kHashLayers - 1) * kTau * kDhWords / 4;
            if (t < n_wb) reinterpret_cast<uint4*>(wb)[t] = reinterpret_cast<const uint4*>(w_bin)[t];
        }
#pragma unroll
        for (int i = 0; i < kSteps; ++i) {
            if (j0 + kPart * i < d) {
                acc0 = fmaf(xv[i], wv[i].x, acc0);
                acc1 = fmaf(xv[i], wv[i].y, acc1);
            }
        }
    }
    part[b0][p] = acc0;
    part[b0 + 1][p] = acc1;
    __syncthreads();
    // hash bit b by wave b: the halvings 128 and 64 from LDS, the rest between lanes
    if (t < 64 * kTau) {
        const int b = t >> 6, l = t & 63;
        float v = (part[b][l] + part[b][l + 128]) + (part[b][l + 64] + part[b][l + 192]);
#pragma unroll
        for (int s = 32; s >= 1; s >>= 1) v = v + __shfl_down(v, s, 64);
        if (l == 0) dots[b] = v;
    }
    __syncthreads();
    if (t < 64) {
        int idx = bucket_of(__ballot(t < kTau && dots[t & (kTau - 1)] >= 0.f));
        for (int k = 1; k < kHashLayers; ++k) {
            const uint32_t* y = tab + ((k - 1) * kDh + idx) * kDhWords;  // y_k = T_k[idx]
            int mismatch = 0;
            if (t < kTau) {
                const uint32_t* w = wb + ((k - 1) * kTau + t) * kDhWords;
#pragma unroll
                for (int m = 0; m < kDhWords; ++m) mismatch += __popc(y[m] ^ w[m]);
            }
            idx = bucket_of(__ballot(t < kTau && kDh - 2 * mismatch >= 0));
        }
        if (t == 0) last_bucket = idx;
    }
    __syncthreads();
    const uint8_t* row = head + (size_t)last_bucket * nblk;
    for (int b = t; b < nblk; b += kThreads) scores[(size_t)blockIdx.x * nblk + b] = (float)row[b];
}

}  // namespace

hipError_t launch_hash_predict(int d, int nblk, const float* x, int B, const HashDev& h, float* scores,
                               hipStream_t st) {
    if (B <= 0) return hipSuccess;
    hipLaunchKernelGGL(hash_predict_kernel, dim3(B), dim3(kThreads), 0, st, d, nblk, x, h.w1, h.w_bin,
                       h.tables, h.head, scores);
    return hipGetLastError();
}

}  // namespace ls
