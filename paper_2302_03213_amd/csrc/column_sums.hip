// The bias gradient of a layer (arXiv 2302.03213, Sec. 3: the bias is learned with the centroids): dL/dY summed over its rows,
// out[m] = sum_o sum_i G[o][m][i] - rows of M values (inner = 1), or a convolution's NCHW planes.
//
// What bounds it: reading G once.  A first kernel leaves one partial sum per chunk of rows, or per plane, a second adds them in a
// fixed order; nothing has to be cleared and no chain of additions is long.  4096 x 3072: 24 us (a library's reduction with the
// clearing of its flags) -> 12.5; 16 x 64 planes of 56 x 56: 18 -> 8.
#include <algorithm>

#include "lutnn_kernels.h"

namespace lutnn {
namespace {

constexpr int kThreads = 256, kCols = 256;  // 64 lanes x 4 columns
constexpr int kAhead = 8;                   // loads in flight per lane

// grid: chunks * col_tiles workgroups, column tile fastest; partial [chunks][M].  M >= 4; the last lanes of a row overlap.
__global__ __launch_bounds__(kThreads) void row_chunk_sums_kernel(const float* __restrict__ G, int64_t N, int64_t ldg, int M,
                                                                  int col_tiles, int per_chunk, float* __restrict__ partial) {
    typedef float f32x4 __attribute__((ext_vector_type(4), aligned(4)));
    __shared__ float part[3][64][4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int chunk = blockIdx.x / col_tiles;
    const int first = (int)(blockIdx.x % col_tiles) * kCols + 4 * lane;
    const int m = min(first, M - 4);
    const int64_t begin = (int64_t)chunk * per_chunk, end = min(begin + per_chunk, N);
    const float* __restrict__ at = G + m;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    int64_t n = begin + w;
    for (; n + 4 * (kAhead - 1) < end; n += 4 * kAhead) {
        f32x4 v[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) v[i] = *reinterpret_cast<const f32x4*>(at + (n + 4 * i) * ldg);
#pragma unroll
        for (int i = 0; i < kAhead; i += 2) sum += v[i] + v[i + 1];
    }
    for (; n < end; n += 4) sum += *reinterpret_cast<const f32x4*>(at + n * ldg);
    if (w > 0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) part[w - 1][lane][j] = sum[j];
    }
    __syncthreads();
    if (w > 0 || first >= M) return;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        partial[(int64_t)chunk * M + m + j] = (sum[j] + part[0][lane][j]) + (part[1][lane][j] + part[2][lane][j]);
}

// A wavefront per plane: partial[o * M + m] = sum_i G[o][m][i].
__global__ __launch_bounds__(kThreads) void plane_sums_kernel(const float* __restrict__ G, int64_t planes, int64_t inner,
                                                              float* __restrict__ partial) {
    const int lane = threadIdx.x & 63;
    const int64_t plane = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (plane >= planes) return;
    const float* __restrict__ at = G + plane * inner;
    float sum = 0.f;
    int64_t i = lane;
    for (; i + 64 * (kAhead - 1) < inner; i += 64 * kAhead) {
        float v[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) v[k] = at[i + 64 * k];
        sum += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    }
    for (; i < inner; i += 64) sum += at[i];
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) sum += __shfl_xor(sum, m, 64);
    if (lane == 0) partial[plane] = sum;
}

// out[m] = sum over chunks of partial[chunk][m]: four wavefronts take every fourth chunk each.
__global__ __launch_bounds__(kThreads) void chunk_sums_kernel(const float* __restrict__ partial, int64_t chunks, int M,
                                                              float* __restrict__ out) {
    __shared__ float part[3][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int m = blockIdx.x * 64 + lane;
    float sum = 0.f;
    if (m < M) {
        int64_t c = w;
        for (; c + 4 * (kAhead - 1) < chunks; c += 4 * kAhead) {
            float v[kAhead];
#pragma unroll
            for (int k = 0; k < kAhead; ++k) v[k] = partial[(c + 4 * k) * M + m];
            sum += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
        }
        for (; c < chunks; c += 4) sum += partial[c * M + m];
    }
    if (w > 0) part[w - 1][lane] = sum;
    __syncthreads();
    if (w == 0 && m < M) out[m] = (sum + part[0][lane]) + (part[1][lane] + part[2][lane]);
}

// Rows per chunk: four workgroups per compute unit, and at least 32 rows to read.
int64_t rows_per_chunk(int64_t N, int M) {
    const int64_t col_tiles = (M + kCols - 1) / kCols;
    const int64_t chunks = std::max<int64_t>(4 * compute_units() / col_tiles, 1);
    return std::max<int64_t>((N + chunks - 1) / chunks, 32);
}

}  // namespace

int64_t column_sums_partials(int64_t outer, int M, int64_t inner) {
    if (inner > 1) return outer * M;
    const int64_t per = rows_per_chunk(outer, M);
    return (outer + per - 1) / per * M;
}

hipError_t launch_column_sums(const float* G, int64_t outer, int64_t ldg, int M, int64_t inner, float* partial, float* out,
                              hipStream_t s) {
    int64_t chunks = outer;
    if (inner > 1) {
        const int64_t blocks = (outer * M + kThreads / 64 - 1) / (kThreads / 64);
        if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
        if (blocks > 0)
            hipLaunchKernelGGL(plane_sums_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, s, G, outer * M, inner, partial);
    } else {
        const int64_t per = rows_per_chunk(outer, M), col_tiles = (M + kCols - 1) / kCols;
        chunks = (outer + per - 1) / per;
        if (M < 4 || per > 0x7fffffffLL || chunks * col_tiles > 0x7fffffffLL) return hipErrorInvalidValue;
        if (chunks > 0)
            hipLaunchKernelGGL(row_chunk_sums_kernel, dim3((unsigned)(chunks * col_tiles)), dim3(kThreads), 0, s, G, outer, ldg,
                               M, (int)col_tiles, (int)per, partial);
    }
    if (hipError_t e = hipGetLastError()) return e;
    hipLaunchKernelGGL(chunk_sums_kernel, dim3((unsigned)((M + 63) / 64)), dim3(kThreads), 0, s, partial, chunks, M, out);
    return hipGetLastError();
}

}  // namespace lutnn
