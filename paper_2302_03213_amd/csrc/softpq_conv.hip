// The two steps around the soft-PQ backward pass of a convolution (arXiv 2302.03213, Sec. 3 and Sec. 4): the im2col
// gradient of the ordinary convolution, Z = W . dL/dY per image, in the [B][D][Ho*Wo] layout that the backward kernel
// reads and overwrites with dL/dX, and that result folded back onto the image.
#include <algorithm>

#include "lutnn_kernels.h"

namespace lutnn {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kTD = 64, kTN = 256, kTM = 16;  // workgroup tile: rows of W, output pixels; m per stage
constexpr int kAS = kTD + 4, kBS = kTN + 4;

// Z[b][d][l] = sum_m W[d][m] * G[b][m][l] on v_mfma_f32_32x32x2_f32 (fp32 products and sums, m ascending in steps of
// two).  A workgroup owns 64 rows d and 256 columns n = (b, l), a wavefront a 64 x 64 part; a thread copies one column of
// G, so that the column's image is found once and images need not be multiples of anything.
// Bound by the write of Z.  50176 columns, D = 576, M = 64: 54 us for 128 MB and 3.7 GFLOP (a library batched product:
// 99 us; the same library's plain product 60 us, but from a transposed copy of G and into rows that then had to be
// transposed back).
__global__ __launch_bounds__(256, 4) void conv_z_kernel(const float* __restrict__ W, int64_t ldw,
                                                        const float* __restrict__ G, float* __restrict__ Z, int D, int M,
                                                        uint32_t L, uint32_t N, int d_tiles, int blocks) {
    __shared__ float as[kTM * kAS];
    __shared__ float bs[kTM * kBS];
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
    const int ad = tid >> 2, am = (tid & 3) * 4;
    const float* __restrict__ wr = W + (int64_t)(d0 + ad < D ? d0 + ad : 0) * ldw;

    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    for (int m0 = 0; m0 < M; m0 += kTM) {
        float gv[kTM], wv[4];
#pragma unroll
        for (int i = 0; i < kTM; ++i) gv[i] = n_ok && m0 + i < M ? g[(int64_t)(m0 + i) * L] : 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) wv[i] = d0 + ad < D && m0 + am + i < M ? wr[m0 + am + i] : 0.f;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kTM; ++i) bs[i * kBS + tid] = gv[i];
#pragma unroll
        for (int i = 0; i < 4; ++i) as[(am + i) * kAS + ad] = wv[i];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kTM; k += 2) {
            float a[2], bb[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                a[i] = as[(k + half) * kAS + 32 * i + j32];
                bb[i] = bs[(k + half) * kBS + 64 * w + 32 * i + j32];
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], bb[j], acc[i][j], 0, 0, 0);
        }
    }
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
                if (d0 + d < D) z[(int64_t)d * L] = acc[i][j][r];
            }
    }
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
