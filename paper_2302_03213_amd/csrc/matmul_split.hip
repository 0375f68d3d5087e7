// Z = G . W^T in fp32 for the backward pass of training (arXiv 2302.03213, Sec. 3: the input gradient of the ordinary
// linear layer, which the soft encoding's gradients are formed from), on the bf16 matrix instructions of gfx950.
//
//   Z[n][d] = sum_m G[n][m] * W[d][m]
//
// What bounds it.  The fp32 matrix instructions do 157 TFLOP/s, the bf16 ones sixteen times that.  An fp32 value is
// exactly the sum of three bf16 values (its top eight significant bits, the next eight, the rest; cut off, never
// rounded, and scaled so that the last has its bits), and of the nine products of two such sums six reach 2^-21 of the whole or more:
// six sixteenths of the fp32 instructions' time.
//
// Precision.  The products are exact in the matrix instructions' fp32 sums.  What is left out, middle.low, low.middle
// and low.low, is 2^-24 of a product on average and 2^-21 at most.  The matrix instruction cuts its result where an fp32
// addition rounds, so nothing long is summed in it: each slice of 32 m starts from zero, small products first, and is
// added to the running sum by a vector addition.  Against 64-bit sums the error is below that of the library's fp32
// product, which adds all M in one fp32 chain, from 16 terms on: tests/test_gpu_linear_gradient.py states both.
//
// Sums that are not finite are formed again as one fp32 chain, by the thread that has them: an infinite value has no parts.
//
// Mapping.  A workgroup is two groups of four wavefronts, a wavefront of each per SIMD.  Both own the same tile of Z, 32
// RB rows n by 32 CB columns d, and every other slice of m.  They take turns: while one group reads its slice's parts
// from LDS and multiplies, the other cuts its next slice into parts, writes those to its own LDS, and loads the one after
// into registers; one barrier ends the turn for both.  A wavefront multiplies 16 RB rows by 16 CB columns; d is the
// instruction's row, so that a lane holds four consecutive d and stores them at once.  At the end the second group's sums
// go to the first through LDS.
//
// 4096 x 768, M = 3072 (128 x 96 tiles, one per compute unit): 113-119 us by machine, 162-171 TFLOP/s of fp32 results, the
// matrix cores busy for half of it (128 us under a profiler).  Timed with parts left out, before values were scaled (112
// us): without the matrix instructions 78, without cutting 99, without loads 102, operand reads alone 41 - no single one of
// them bounds it, and the clock is down to 1.8 GHz under the products.  Slower were the 32 x 32 instruction (125), two
// slices in flight per wavefront (123), both groups on halves of one slice with a double buffer (131), rows of 80 instead
// of swizzled 64 bytes (118); wave priorities change nothing.
#include <algorithm>

#include "lutnn_kernels.h"
#include "split_bf16.h"

namespace lutnn {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int64_t kMaxStride = 1 << 20;  // floats: a tile's rows within 32-bit offsets
constexpr uint32_t kNowhere = 0xc0000000u;  // an offset beyond any resource: the load returns zero

__device__ __forceinline__ f32x4 product(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Orders the workgroup's LDS operations only: global loads stay in flight.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// One tile's rows of an operand, addressed from its first element.
struct Rows {
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t stride;  // bytes
};

__device__ __forceinline__ Rows rows_of(const float* A, int64_t ld, int64_t first, int64_t rows, int M) {
    const uint32_t bytes = (uint32_t)(((rows - 1) * ld + M) * 4);
    return {__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(A) + first * ld, 0, bytes, 0x00020000), (uint32_t)(ld * 4)};
}

// Four values at column m of a row, zero past the tile's last row and past M.
template <bool VEC>  // rows are 16-byte aligned and M a multiple of four
__device__ __forceinline__ u32x4 load4(const Rows& a, uint32_t row_off, int m, int M) {
    const uint32_t off = row_off + 4u * (uint32_t)m;
    if constexpr (VEC)
        return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(a.rsrc, m < M ? off : kNowhere, 0, 0));
    u32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = __builtin_amdgcn_raw_buffer_load_b32(a.rsrc, m + i < M ? off + 4u * i : kNowhere, 0, 0);
    return r;
}

template <int PLANE>  // bytes between the parts
__device__ __forceinline__ void store_parts(u32x4 v, char* to) {
    uint32_t high[2], mid[2], low[2];
    cut<2>({v[0], v[1], v[2], v[3]}, high, mid, low);
    *reinterpret_cast<u32x2*>(to) = u32x2{high[0], high[1]};
    *reinterpret_cast<u32x2*>(to + PLANE) = u32x2{mid[0], mid[1]};
    *reinterpret_cast<u32x2*>(to + 2 * PLANE) = u32x2{low[0], low[1]};
}

// grid: tiles of Z, column tile fastest.
template <int RB, int CB, bool VEC>
__global__ __launch_bounds__(512, RB * CB > 4 ? 2 : 4) void matmul_split_kernel(const float* __restrict__ G, int64_t ldg,
                                                              const float* __restrict__ W, int64_t ldw,
                                                              float* __restrict__ Z, int64_t ldz, int64_t N, int D, int M,
                                                              int d_tiles, int blocks, int vec4_z) {
    constexpr int TN = 32 * RB, TD = 32 * CB, ROWS = TN + TD, PLANE = ROWS * kRowBytes, BUF = 3 * PLANE;
    static_assert(2 * BUF >= TN * TD * 4, "the second group's sums go through the operand buffers");
    __shared__ __align__(16) char lds[2 * BUF];

    // neighbouring tiles on one XCD: they read the same rows of G at the same time
    const int block = (int)(blockIdx.x % 8) * (int)(gridDim.x / 8) + (int)(blockIdx.x / 8);
    if (block >= blocks) return;
    const int d0 = block % d_tiles * TD;
    const int64_t n0 = (int64_t)(block / d_tiles) * TN;
    const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, i16 = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int group = w >> 2;
    char* const buf = lds + group * BUF;

    // staging: eight threads of a group per row, 32 rows at a time; G's rows, then W's
    const Rows g = rows_of(G, ldg, n0, std::min<int64_t>(TN, N - n0), M);
    const Rows wt = rows_of(W, ldw, d0, std::min(TD, D - d0), M);
    const int srow = (tid & 255) >> 3, scol = (tid & 7) * 4;
    char* const to = buf + srow * kRowBytes + unit(srow, scol >> 3) + (scol & 4) * 2;
    u32x4 val[RB + CB];
    const auto load = [&](int turn) {
        const int m = (2 * turn + group) * kSlice + scol;
#pragma unroll
        for (int i = 0; i < RB + CB; ++i)
            val[i] = i < RB ? load4<VEC>(g, (uint32_t)(srow + 32 * i) * g.stride, m, M)
                            : load4<VEC>(wt, (uint32_t)(srow + 32 * (i - RB)) * wt.stride, m, M);
    };

    // operands: W's rows d for the instruction's rows, G's rows n for its columns
    const int wd = (w >> 1) & 1, wn = w & 1;
    const char* const from_d = buf + (TN + wd * 16 * CB + i16) * kRowBytes + unit(i16, q);
    const char* const from_n = buf + (wn * 16 * RB + i16) * kRowBytes + unit(i16, q);
    f32x4 sum[CB][RB];
#pragma unroll
    for (int a = 0; a < CB; ++a)
#pragma unroll
        for (int b = 0; b < RB; ++b) sum[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int turns = (M + 2 * kSlice - 1) / (2 * kSlice);  // per group; the last may be all zeros
    load(0);
    if (group == 1) lds_barrier();
    for (int t = 0; t < turns; ++t) {
#pragma unroll
        for (int i = 0; i < RB + CB; ++i) store_parts<PLANE>(val[i], to + i * 32 * kRowBytes);
        if (t + 1 < turns) load(t + 1);
        lds_barrier();
        bf16x8 bn[RB][3];
#pragma unroll
        for (int b = 0; b < RB; ++b)
#pragma unroll
            for (int p = 0; p < 3; ++p)
                bn[b][p] = *reinterpret_cast<const bf16x8*>(from_n + p * PLANE + b * 16 * kRowBytes);
#pragma unroll
        for (int a = 0; a < CB; ++a) {
            bf16x8 ad[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) ad[p] = *reinterpret_cast<const bf16x8*>(from_d + p * PLANE + a * 16 * kRowBytes);
            f32x4 s[RB];
#pragma unroll
            for (int b = 0; b < RB; ++b) s[b] = f32x4{0.f, 0.f, 0.f, 0.f};
            constexpr int kPairs[6][2] = {{2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}, {0, 0}};
#pragma unroll
            for (int i = 0; i < 6; ++i)
#pragma unroll
                for (int b = 0; b < RB; ++b) s[b] = product(ad[kPairs[i][0]], bn[b][kPairs[i][1]], s[b]);
#pragma unroll
            for (int b = 0; b < RB; ++b) sum[a][b] += s[b];
        }
        lds_barrier();
    }
    if (group == 0) lds_barrier();

    // both groups have read their last operands: the buffers hold sums from here on
    f32x4* const other = reinterpret_cast<f32x4*>(lds) + (w & 3) * RB * CB * 64 + lane;
    if (group == 1) {
#pragma unroll
        for (int a = 0; a < CB; ++a)
#pragma unroll
            for (int b = 0; b < RB; ++b) other[(a * RB + b) * 64] = sum[a][b];
    }
    lds_barrier();
    if (group == 1) return;
    float probe = 0.f;  // NaN once a sum is not finite
#pragma unroll
    for (int b = 0; b < RB; ++b) {
        const int64_t n = n0 + wn * 16 * RB + 16 * b + i16;
        if (n >= N) continue;
        float* const z = Z + n * ldz;
#pragma unroll
        for (int a = 0; a < CB; ++a) {
            const f32x4 r = (sum[a][b] + other[(a * RB + b) * 64]) * kUnscale;
            const int d = d0 + wd * 16 * CB + 16 * a + 4 * q;
#pragma unroll
            for (int j = 0; j < 4; ++j) probe = __fmaf_rn(r[j], 0.f, probe);
            if (vec4_z && d + 3 < D) {
                *reinterpret_cast<f32x4*>(z + d) = r;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (d + j < D) z[d + j] = r[j];
            }
        }
    }
    if (probe == 0.f) return;
    for (int i = 0; i < RB * CB * 4; ++i) {
        const int64_t n = n0 + wn * 16 * RB + i / (CB * 4) * 16 + i16;
        const int d = d0 + wd * 16 * CB + i / 4 % CB * 16 + 4 * q + i % 4;
        if (n < N && d < D && !is_finite(Z[n * ldz + d])) Z[n * ldz + d] = fp32_chain(G + n * ldg, 1, W + d * ldw, M);
    }
}

int vec4_ok(const float* A, int64_t ld, int width) {
    return width % 4 == 0 && ld % 4 == 0 && (reinterpret_cast<uintptr_t>(A) & 15) == 0;
}

template <int RB, int CB, bool VEC>
hipError_t launch(const float* G, int64_t N, int64_t ldg, const float* W, int64_t ldw, int D, int M, float* Z, int64_t ldz,
                  hipStream_t s) {
    constexpr int TN = 32 * RB, TD = 32 * CB;
    const int64_t d_tiles = (D + TD - 1) / TD, blocks = d_tiles * ((N + TN - 1) / TN);
    if (blocks > 0x7ffffff0LL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((matmul_split_kernel<RB, CB, VEC>), dim3((unsigned)(blocks + 7) / 8 * 8), dim3(512), 0, s, G, ldg, W, ldw,
                       Z, ldz, N, D, M, (int)d_tiles, (int)blocks, vec4_ok(Z, ldz, 4));
    return hipGetLastError();
}

// Tile sizes in units of 32 and what 64 m of one tile take, in us: alone on a compute unit, and two at once where the
// registers and the LDS allow it.  From 14 shapes; over 80 others a launch takes 0.92 to 1.15 of what they predict.
struct Tile {
    int rb, cb;
    float one, two;
};
constexpr Tile kTiles[] = {{4, 4, 3.00f, 6.00f}, {4, 3, 2.30f, 4.60f}, {3, 2, 1.50f, 2.60f}, {2, 2, 1.10f, 1.63f}};
constexpr int kTileCount = sizeof(kTiles) / sizeof(kTiles[0]);

float predicted_us(const Tile& t, int64_t N, int D, int M) {
    const int64_t tiles = ((N + 32 * t.rb - 1) / (32 * t.rb)) * ((D + 32 * t.cb - 1) / (32 * t.cb));
    const int64_t per_cu = (tiles + compute_units() - 1) / compute_units();
    return ((per_cu / 2) * t.two + (per_cu % 2) * t.one) * ((M + 2 * kSlice - 1) / (2 * kSlice)) + 5.f;
}

int best_tile(int64_t N, int D, int M) {
    int best = 0;
    for (int i = 1; i < kTileCount; ++i)
        if (predicted_us(kTiles[i], N, D, M) < predicted_us(kTiles[best], N, D, M)) best = i;
    return best;
}

}  // namespace

// Where this is the faster one.  The library's fp32 product runs at 115-140 TFLOP/s where it fills the chip and takes 8 us
// at least, and it shares a long sum out over workgroups where there are few tiles, which this does not (256 x 256, M =
// 3072: 23 us against 57).  Measured, library against this: 4096 x 768, M = 3072: 143 -> 113 us; 4096 x 3072, M = 768: 144
// -> 127; 8192 x 768, M = 768: 78 -> 63; 8192 x 2048, M = 1024: 245 -> 206; 4096 x 256, M = 256: 19 -> 10; 5000 x 300, M =
// 700: 30 -> 22.  Of 129 shapes that take it, four are behind the library, by 3-9 % (1000 x 1024 and 512 x 2048, M =
// 1024; 1000 x 2048 and 2048 x 1024, M = 3072).  Rows that are not whole 16-byte vectors load value by value (3000 x 1000,
// M = 1001: 81 -> 73 at best, and behind at others): the library.
// Below 16 terms the parts are less exact than one fp32 chain (7e-8 of the result at any length, against 2.5e-8 at one term,
// 6.4e-8 at 12 and 7.4e-8 at 16): the library.
bool matmul_split_preferred(const float* G, int64_t N, int64_t ldg, const float* W, int64_t ldw, int D, int M) {
    if (N <= 0 || M < 16 || !vec4_ok(G, ldg, M) || !vec4_ok(W, ldw, M) || ldg > kMaxStride || ldw > kMaxStride) return false;
    const float library_us = 2.f * N * D * M / 130e6f + 8.f;
    return predicted_us(kTiles[best_tile(N, D, M)], N, D, M) < library_us;
}

hipError_t launch_matmul_split(const float* G, int64_t N, int64_t ldg, const float* W, int64_t ldw, int D, int M, float* Z,
                               int64_t ldz, hipStream_t s) {
    if (N == 0) return hipSuccess;
    if (!vec4_ok(G, ldg, M) || !vec4_ok(W, ldw, M)) return launch<2, 2, false>(G, N, ldg, W, ldw, D, M, Z, ldz, s);
    switch (best_tile(N, D, M)) {
        case 0: return launch<4, 4, true>(G, N, ldg, W, ldw, D, M, Z, ldz, s);
        case 1: return launch<4, 3, true>(G, N, ldg, W, ldw, D, M, Z, ldz, s);
        case 2: return launch<3, 2, true>(G, N, ldg, W, ldw, D, M, Z, ldz, s);
        default: return launch<2, 2, true>(G, N, ldg, W, ldw, D, M, Z, ldz, s);
    }
}

}  // namespace lutnn
