// fp32 values as sums of three bf16 parts for the bf16 matrix instructions (matmul_split.hip says why and how exactly),
// and the LDS layout that both kernels keep them in: rows of 32 values, 64 bytes, one plane per part.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lutnn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kSlice = 32;     // values of a row in LDS
constexpr int kRowBytes = 64;  // of one part

// Where the q-th 16 bytes of a row lie in it: rows of 64 bytes start at every fourth bank, and this spreads the same q
// of eight neighbouring rows over all of them, for the 16-byte reads and for the writes.
__device__ __forceinline__ int unit(int row, int q) { return (q ^ ((row >> 1) & 3)) * 16; }

// The upper halves of two words: two values cut to bf16.
__device__ __forceinline__ uint32_t upper(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

// Operands are scaled up before they are cut, and sums down: the lowest part of a value reaches 2^-16 to 2^-24 of it, and
// bf16 has nothing below 2^-133, so that values under 2^-110 (7e-34) would lose bits that fp32 has.  Values from 2^104 and
// products from 2^80 on leave the range that way; such sums are not finite, and formed again.  One instruction more per
// value: 4096 x 768, M = 3072: 115 -> 119 us; 8192 x 768, M = 768: 60.5 -> 62.8.
constexpr float kScale = 1 << 24, kUnscale = 1.f / kScale / kScale;

// 2 n values into n words of each part: the top eight significant bits, the next eight, the rest.
template <int n>
__device__ __forceinline__ void cut(const uint32_t (&v)[2 * n], uint32_t (&high)[n], uint32_t (&mid)[n], uint32_t (&low)[n]) {
#pragma unroll
    for (int i = 0; i < n; ++i) {
        uint32_t top[2], m[2], l[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const uint32_t x = __float_as_uint(__uint_as_float(v[2 * i + j]) * kScale);
            top[j] = x;
            const float r = __uint_as_float(x) - __uint_as_float(x & 0xffff0000u);
            m[j] = __float_as_uint(r);
            l[j] = __float_as_uint(r - __uint_as_float(m[j] & 0xffff0000u));
        }
        high[i] = upper(top[0], top[1]);
        mid[i] = upper(m[0], m[1]);
        low[i] = upper(l[0], l[1]);
    }
}

// For sums from parts that are not finite: an infinite value has none.  g: consecutive values `step` apart.
__device__ __forceinline__ bool is_finite(float x) { return fabsf(x) <= 3.402823466e38f; }
__device__ __forceinline__ float fp32_chain(const float* __restrict__ g, int64_t step, const float* __restrict__ w, int M) {
    float sum = 0.f;
    int m = 0;
    for (; m + 8 <= M && sum == sum; m += 8) {  // nothing changes a NaN
        float a[8], b[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) a[i] = g[(m + i) * step], b[i] = w[m + i];
#pragma unroll
        for (int i = 0; i < 8; ++i) sum = __fmaf_rn(a[i], b[i], sum);
    }
    for (; m < M && sum == sum; ++m) sum = __fmaf_rn(g[m * step], w[m], sum);
    return sum;
}

}  // namespace lutnn
