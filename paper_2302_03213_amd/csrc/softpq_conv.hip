// The two steps around the soft-PQ backward pass of a convolution (arXiv 2302.03213, Sec. 3 and Sec. 4): the im2col
// gradient of the ordinary convolution, Z = W . dL/dY per image, in the [B][D][Ho*Wo] layout that the backward kernel
// reads and overwrites with dL/dX, and that result folded back onto the image.
#include <algorithm>

#include "lutnn_kernels.h"
#include "split_bf16.h"

namespace lutnn {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int kTD = 64, kTN = 256;  // workgroup tile: rows of W, output pixels
constexpr int kPlane = (kTD + kTN) * kRowBytes;

__device__ __forceinline__ f32x16 product(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// 16 bytes of each part of a row, eight values.
__device__ __forceinline__ void store_parts(const uint32_t (&v)[8], char* to) {
    uint32_t high[4], mid[4], low[4];
    cut<4>(v, high, mid, low);
    *reinterpret_cast<u32x4*>(to) = u32x4{high[0], high[1], high[2], high[3]};
    *reinterpret_cast<u32x4*>(to + kPlane) = u32x4{mid[0], mid[1], mid[2], mid[3]};
    *reinterpret_cast<u32x4*>(to + 2 * kPlane) = u32x4{low[0], low[1], low[2], low[3]};
}

// Z[b][d][l] = sum_m W[d][m] * G[b][m][l] from bf16 parts, as matmul_split.hip forms G . W^T (the parts, the six products
// and the sums are described there).  A workgroup owns 64 rows d and 256 columns n = (b, l), a wavefront a 64 x 64 part; a
// thread copies one column of G, so that the column's image is found once and images need not be multiples of anything.
// On the fp32 matrix instructions it was bound by them wherever M is not small; the whole backward pass of a 3x3
// convolution, with those and with this: 16 x 256 channels 14 x 14, M = 512: 171 -> 130 us; 4 x 128, 28 x 28, M = 256: 84
// -> 72; 16 x 64, 56 x 56, M = 64: 228 -> 213, where the write of Z bounds it (53 us for 128 MB, 55 before; a library
// batched product: 99).  With softpq_matrix.hip's shorter sums 135, 75 and 220.
__global__ __launch_bounds__(256, 2) void conv_z_kernel(const float* __restrict__ W, int64_t ldw,
                                                        const float* __restrict__ G, float* __restrict__ Z, int D, int M,
                                                        uint32_t L, uint32_t N, int d_tiles, int blocks) {
    __shared__ __align__(16) char lds[3 * kPlane];
    // row tiles of W fastest, and neighbouring blocks on one XCD: the columns of G are then in its L2
    const int block = (int)(blockIdx.x % 8) * (int)(gridDim.x / 8) + (int)(blockIdx.x / 8);
    if (block >= blocks) return;
    const int d0 = block % d_tiles * kTD;
    const uint32_t n0 = (uint32_t)(block / d_tiles) * kTN;
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, half = lane >> 5, j32 = lane & 31;

    const uint32_t n = n0 + tid;
    const bool n_ok = n < N;
    const uint32_t b = n_ok ? n / L : 0u;
    const float* __restrict__ g = G + (int64_t)b * M * L + (n_ok ? n - b * L : 0u);
    const int ad = tid >> 2, aq = tid & 3;
    const float* __restrict__ wr = W + (int64_t)(d0 + ad < D ? d0 + ad : 0) * ldw;
    uint32_t gv[kSlice], wv[8];
    const auto load = [&](int m0) {
        const float* at = g + (int64_t)m0 * L;
        int64_t step = L;
        asm volatile("" : "+s"(step));  // one pointer that walks: the compiler kept 32 of them across the loop, and spilled
#pragma unroll
        for (int i = 0; i < kSlice; ++i, at += step) gv[i] = __float_as_uint(n_ok && m0 + i < M ? *at : 0.f);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int m = m0 + 8 * aq + i;
            wv[i] = __float_as_uint(d0 + ad < D && m < M ? wr[m] : 0.f);
        }
    };
    char* const to_n = lds + (kTD + tid) * kRowBytes;
    char* const to_d = lds + ad * kRowBytes + unit(ad, aq);
    const char* const from_d = lds + j32 * kRowBytes;
    const char* const from_n = lds + (kTD + 64 * w + j32) * kRowBytes;

    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x16{};

    load(0);
    for (int m0 = 0; m0 < M; m0 += kSlice) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q)
            store_parts({gv[8 * q], gv[8 * q + 1], gv[8 * q + 2], gv[8 * q + 3], gv[8 * q + 4], gv[8 * q + 5], gv[8 * q + 6],
                         gv[8 * q + 7]}, to_n + unit(tid, q));
        store_parts(wv, to_d);
        __syncthreads();
        if (m0 + kSlice < M) load(m0 + kSlice);
#pragma unroll
        for (int j = 0; j < 2; ++j) {  // 32 columns at a time: the registers of both at once are not there
            f32x16 s[2] = {f32x16{}, f32x16{}};
            bf16x8 dh[2][2], nh[2];  // high parts, for the last products of the slice
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int u = unit(j32, 2 * k + half);
                const char* const at_n = from_n + j * 32 * kRowBytes + u;
                nh[k] = *reinterpret_cast<const bf16x8*>(at_n);
                const bf16x8 nm = *reinterpret_cast<const bf16x8*>(at_n + kPlane);
                const bf16x8 nl = *reinterpret_cast<const bf16x8*>(at_n + 2 * kPlane);
                bf16x8 dm[2], dl[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const char* const at = from_d + i * 32 * kRowBytes + u;
                    dh[k][i] = *reinterpret_cast<const bf16x8*>(at);
                    dm[i] = *reinterpret_cast<const bf16x8*>(at + kPlane);
                    dl[i] = *reinterpret_cast<const bf16x8*>(at + 2 * kPlane);
                }
#pragma unroll
                for (int i = 0; i < 2; ++i) s[i] = product(dl[i], nh[k], s[i]);
#pragma unroll
                for (int i = 0; i < 2; ++i) s[i] = product(dh[k][i], nl, s[i]);
#pragma unroll
                for (int i = 0; i < 2; ++i) s[i] = product(dm[i], nm, s[i]);
#pragma unroll
                for (int i = 0; i < 2; ++i) s[i] = product(dm[i], nh[k], s[i]);
#pragma unroll
                for (int i = 0; i < 2; ++i) s[i] = product(dh[k][i], nm, s[i]);
            }
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int i = 0; i < 2; ++i) s[i] = product(dh[k][i], nh[k], s[i]);
#pragma unroll
            for (int i = 0; i < 2; ++i) acc[i][j] += s[i];
        }
    }
    float probe = 0.f;  // NaN once a sum is not finite
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const uint32_t no = n0 + 64 * w + 32 * j + j32;
        if (no >= N) continue;
        const uint32_t bo = no / L;
        float* __restrict__ z = Z + ((int64_t)bo * D + d0) * L + (no - bo * L);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int d = 32 * i + 8 * (r / 4) + 4 * half + r % 4;
                const float sum = acc[i][j][r] * kUnscale;
                probe = __fmaf_rn(sum, 0.f, probe);
                if (d0 + d < D) z[(int64_t)d * L] = sum;
            }
    }
    if (probe == 0.f) return;
    for (int i = 0; i < 64; ++i) {  // as in matmul_split.hip
        const uint32_t no = n0 + 64 * w + i / 32 * 32 + j32;
        const int d = d0 + i / 16 % 2 * 32 + i / 4 % 4 * 8 + 4 * half + i % 4;
        if (no >= N || d >= D) continue;
        const uint32_t bo = no / L, l = no - bo * L;
        float* __restrict__ z = Z + ((int64_t)bo * D + d) * L + l;
        if (!is_finite(*z)) *z = fp32_chain(G + (int64_t)bo * M * L + l, L, W + d * ldw, M);
    }
}

// The same for short sums, one fp32 chain each.  Below 16 terms such a chain is the more exact: 2.5e-8 of the result at one
// term, 6.4e-8 at 12 and 7.4e-8 at 16, where the parts leave 7e-8 whatever the length.  A thread owns a pixel, its values of
// G in registers, and goes through kShortD rows of W, which are scalar operands.  The write of Z bounds both: the whole
// backward pass of 16 x 64 channels 56 x 56, M = 15, 195 us with the parts and 198 with this; M = 8, 204.5 and 204.
constexpr int kShortSum = 16, kShortD = 48;
template <int M>
__global__ __launch_bounds__(256) void conv_z_short_kernel(const float* __restrict__ W, int64_t ldw,
                                                           const float* __restrict__ G, float* __restrict__ Z, int D,
                                                           uint32_t L, uint32_t N, int d_tiles) {
    const int d0 = (int)(blockIdx.x % d_tiles) * kShortD;
    const uint32_t n = blockIdx.x / d_tiles * 256 + threadIdx.x;
    if (n >= N) return;
    const uint32_t b = n / L, l = n - b * L;
    const float* __restrict__ at = G + (int64_t)b * M * L + l;
    float g[M];
#pragma unroll
    for (int m = 0; m < M; ++m) g[m] = at[(int64_t)m * L];
    float* __restrict__ z = Z + ((int64_t)b * D + d0) * L + l;
    const int rows = std::min(kShortD, D - d0);
#pragma unroll 4
    for (int d = 0; d < rows; ++d) {
        const float* __restrict__ w = W + (d0 + d) * ldw;
        float sum = 0.f;
#pragma unroll
        for (int m = 0; m < M; ++m) sum = __fmaf_rn(w[m], g[m], sum);
        z[(int64_t)d * L] = sum;
    }
}

template <int M = kShortSum - 1>
hipError_t launch_conv_z_short(const float* W, int64_t ldw, const float* G, int64_t N, int64_t L, int D, int m, float* Z,
                               hipStream_t s) {
    if constexpr (M > 1)
        if (m < M) return launch_conv_z_short<M - 1>(W, ldw, G, N, L, D, m, Z, s);
    const int64_t d_tiles = (D + kShortD - 1) / kShortD, blocks = d_tiles * ((N + 255) / 256);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((conv_z_short_kernel<M>), dim3((unsigned)blocks), dim3(256), 0, s, W, ldw, G, Z, D, (uint32_t)L, (uint32_t)N,
                       (int)d_tiles);
    return hipGetLastError();
}

// A thread owns one input element and adds the taps that reach it in ascending order (no atomics, nothing to clear).
// Consecutive threads are consecutive columns of the image: for stride 1 every read is a contiguous run.
//   grid: blockIdx.y = (image, channel), blockIdx.x = block of 256 elements of it
__global__ __launch_bounds__(256) void fold_kernel(const float* __restrict__ columns, float* __restrict__ image,
                                                   ConvGeom g) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= g.H * g.W) return;
    const int h = e / g.W + g.ph, wi = e % g.W + g.pw;
    const int64_t pix = (int64_t)g.Ho * g.Wo;
    const float* __restrict__ src = columns + (int64_t)blockIdx.y * (g.kh * g.kw) * pix;
    float sum = 0.f;
    if (g.sh == 1 && g.sw == 1) {
        for (int r = 0; r < g.kh; ++r)
            for (int s = 0; s < g.kw; ++s, src += pix) {
                const int ho = h - r, wo = wi - s;
                if ((unsigned)ho < (unsigned)g.Ho && (unsigned)wo < (unsigned)g.Wo) sum += src[ho * g.Wo + wo];
            }
    } else {
        for (int r = 0; r < g.kh; ++r)
            for (int s = 0; s < g.kw; ++s, src += pix) {
                const int ho = (h - r) / g.sh, wo = (wi - s) / g.sw;
                if (h >= r && wi >= s && ho * g.sh == h - r && wo * g.sw == wi - s && ho < g.Ho && wo < g.Wo)
                    sum += src[ho * g.Wo + wo];
            }
    }
    image[(int64_t)blockIdx.y * g.H * g.W + e] = sum;
}

}  // namespace

hipError_t launch_conv_z(const float* W, int64_t ldw, const float* G, int64_t B, int D, int M, const ConvGeom& g, float* Z,
                         hipStream_t s) {
    const int64_t L = (int64_t)g.Ho * g.Wo, N = B * L;
    if (M < kShortSum) return launch_conv_z_short(W, ldw, G, N, L, D, M, Z, s);
    const int64_t d_tiles = (D + kTD - 1) / kTD, blocks = d_tiles * ((N + kTN - 1) / kTN);
    if (blocks > 0x7ffffff0LL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(conv_z_kernel, dim3((unsigned)(blocks + 7) / 8 * 8), dim3(256), 0, s, W, ldw, G, Z, D, M, (uint32_t)L,
                       (uint32_t)N, (int)d_tiles, (int)blocks);
    return hipGetLastError();
}

hipError_t launch_fold(const float* columns, int64_t B, const ConvGeom& g, float* image, hipStream_t s) {
    const unsigned blocks = (unsigned)(((int64_t)g.H * g.W + 255) / 256);
    const int64_t planes = B * g.Cin;
    // the grid's second dimension stops at 65535
    for (int64_t first = 0; first < planes; first += 65535) {
        const int64_t n = std::min<int64_t>(65535, planes - first);
        hipLaunchKernelGGL(fold_kernel, dim3(blocks, (unsigned)n), dim3(256), 0, s,
                           columns + first * g.kh * g.kw * ((int64_t)g.Ho * g.Wo), image + first * g.H * g.W, g);
        if (hipError_t e = hipGetLastError()) return e;
    }
    return hipSuccess;
}

}  // namespace lutnn
