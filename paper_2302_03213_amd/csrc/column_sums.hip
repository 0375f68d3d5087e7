// The bias gradient of a layer (arXiv 2302.03213, Sec. 3: the bias is learned with the centroids): dL/dY summed over its rows,
// out[m] = sum_o sum_i G[o][m][i] - rows of M values (inner = 1), or a convolution's NCHW planes.
//
// A first kernel leaves one partial sum per share of a column's values, a second adds them in a fixed order; nothing has to be
// cleared.  A column of few values is one share, and one launch.  Every sum is a 64-bit one, rounded once at the end: the
// additions hide behind the reads, and no chain of them, whatever its length, costs precision.
//
// What bounds it: reading G once, and the launches.  4096 x 3072 10.5 us; 16 x 64 planes of 56 x 56 7, 21 planes of 512 x 512
// 7.5 (a library's reduction, with the clearing of its flags: 21, 15 and 19); 100 x 12 4.5, one launch.
#include <algorithm>
#include <type_traits>

#include "lutnn_kernels.h"

namespace lutnn {
namespace {

constexpr int kTileCols = 256;  // 64 lanes x 4 columns
constexpr int kAhead = 8;       // loads in flight per lane
constexpr int kPlaneThreads = 256;
typedef double f64 __attribute__((aligned(4)));  // the workspace is 4-byte aligned

// A share's sum: the result itself where there is one share only.
__device__ __forceinline__ void put(double sum, int64_t at, f64* __restrict__ partial, float* __restrict__ out, bool single) {
    if (single)
        out[at] = (float)sum;
    else
        partial[at] = sum;
}

// grid: chunks * col_tiles workgroups, column tile fastest.  M >= 4.  A row of the tile takes lpr lanes, the last of which
// overlaps its neighbour, and a wavefront 64 / lpr rows at a time.  The chunks are interleaved, so that all workgroups read one
// region of G (16384 rows of 4096: 46 us, where chunks of neighbouring rows start in the same memory channels and take 53).
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void row_chunk_sums_kernel(const float* __restrict__ G, int64_t N, int64_t ldg, int M,
                                                                    int col_tiles, int lpr, int chunks,
                                                                    f64* __restrict__ partial, float* __restrict__ out,
                                                                    bool single) {
    typedef float f32x4 __attribute__((ext_vector_type(4), aligned(4)));
    __shared__ double part[WAVES * 64][4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int rows = 64 / lpr, sub = lane / lpr;
    const int chunk = blockIdx.x / col_tiles, first = (int)(blockIdx.x % col_tiles) * kTileCols;
    const float* __restrict__ at = G + min(first + 4 * (lane - sub * lpr), M - 4);
    const int step = chunks * WAVES * rows;
    double sum[4] = {0, 0, 0, 0};
    int64_t n = sub < rows ? (chunk * WAVES + w) * rows + sub : N;
    for (; n + (kAhead - 1) * step < N; n += kAhead * step) {
        f32x4 v[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) v[i] = *reinterpret_cast<const f32x4*>(at + (n + i * step) * ldg);
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) sum[j] += v[i][j];
    }
    {  // the rest, in flight at once too
        f32x4 v[kAhead - 1];
#pragma unroll
        for (int i = 0; i < kAhead - 1; ++i)
            if (n + i * step < N) v[i] = *reinterpret_cast<const f32x4*>(at + (n + i * step) * ldg);
#pragma unroll
        for (int i = 0; i < kAhead - 1; ++i)
            if (n + i * step < N)
#pragma unroll
                for (int j = 0; j < 4; ++j) sum[j] += v[i][j];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) part[threadIdx.x][j] = sum[j];
    __syncthreads();
    // the wavefronts' sums, a thread per lane and column, then the rows of a wavefront
    const int l = threadIdx.x >> 2, j = threadIdx.x & 3;
    double total = 0;
    if (l < 64) {
#pragma unroll
        for (int k = 0; k < WAVES; ++k) total += part[64 * k + l][j];
        part[l][j] = total;
    }
    __syncthreads();
    if (l >= lpr) return;
#pragma unroll 4
    for (int r = 1; r < rows; ++r) total += part[r * lpr + l][j];
    const int m = min(first + 4 * l, M - 4) + j;
    put(total, (int64_t)chunk * M + m, partial, out, single);
}

// A workgroup takes one column and a share of its outer planes: `planes` whole ones, or one part in `parts` of one, `length`
// values of a plane either way.  grid: shares * M workgroups, column fastest.
__global__ __launch_bounds__(kPlaneThreads) void plane_share_sums_kernel(const float* __restrict__ G, int64_t outer, int M,
                                                                         int64_t inner, int64_t planes, int parts,
                                                                         int64_t length, f64* __restrict__ partial,
                                                                         float* __restrict__ out, bool single) {
    constexpr int THREADS = kPlaneThreads;
    __shared__ double part[THREADS / 64];
    const int share = blockIdx.x / M, m = blockIdx.x % M;
    const int64_t o = (int64_t)(share / parts) * planes, i = (share % parts) * length;
    const uint32_t len = (uint32_t)min(length, inner - i);
    const int64_t values = min(planes, outer - o) * len;
    const int64_t stride = (int64_t)M * inner;
    const float* __restrict__ at = G + (o * M + m) * inner + i;
    double sum = 0;
    // BATCH values, one in THREADS of the `left` ones, in flight at once; false where there are fewer
    const auto add = [&](auto batch, int64_t left, auto&& value) {
        constexpr int BATCH = decltype(batch)::value;
        if (left <= (BATCH - 1) * THREADS) return false;
        float x[BATCH];
#pragma unroll
        for (int k = 0; k < BATCH; ++k) x[k] = value(k);
#pragma unroll
        for (int k = 0; k < BATCH; ++k) sum += x[k];
        return true;
    };
    using std::integral_constant;
    if (values == len || len >= 8 * THREADS) {  // plane by plane: the addresses are constant distances apart
        for (int64_t n = 0; n < values; n += len, at += stride) {
            uint32_t v = threadIdx.x;
            const auto value = [&](int k) { return at[v + k * THREADS]; };
            while (add(integral_constant<int, kAhead>{}, (int64_t)len - v, value)) v += kAhead * THREADS;
            if (add(integral_constant<int, 4>{}, (int64_t)len - v, value)) v += 4 * THREADS;
            if (add(integral_constant<int, 2>{}, (int64_t)len - v, value)) v += 2 * THREADS;
            add(integral_constant<int, 1>{}, (int64_t)len - v, value);
        }
    } else {  // value v of the share is v % len of plane v / len
        const uint32_t left = THREADS % len;
        const int64_t step = THREADS / len * stride + left;
        uint32_t in_plane = threadIdx.x % len;
        at += threadIdx.x / len * stride + in_plane;
        const auto value = [&](int) {
            const float x = *at;
            in_plane += left;
            at += step;
            if (in_plane >= len) {
                in_plane -= len;
                at += stride - len;
            }
            return x;
        };
        int64_t v = threadIdx.x;
        while (add(integral_constant<int, kAhead>{}, values - v, value)) v += kAhead * THREADS;
        if (add(integral_constant<int, 4>{}, values - v, value)) v += 4 * THREADS;
        if (add(integral_constant<int, 2>{}, values - v, value)) v += 2 * THREADS;
        add(integral_constant<int, 1>{}, values - v, value);
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) sum += __shfl_xor(sum, d, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x != 0) return;
#pragma unroll
    for (int w = 1; w < THREADS / 64; ++w) sum += part[w];
    put(sum, (int64_t)share * M + m, partial, out, single);
}

// out[m] = sum over shares of partial[share][m]: 32 columns per workgroup, every kGroups-th share per thread.
template <int kGroups>
__global__ __launch_bounds__(32 * kGroups) void share_sums_kernel(const f64* __restrict__ partial, int64_t shares, int M,
                                                                  float* __restrict__ out) {
    constexpr int kCols = 32;
    __shared__ double part[kGroups][kCols];
    const int col = threadIdx.x % kCols, g = threadIdx.x / kCols;
    const int m = blockIdx.x * kCols + col;
    double sum = 0;
    if (m < M) {
        int64_t s = g;
        for (; s + kGroups * (kAhead - 1) < shares; s += kGroups * kAhead) {
            double v[kAhead];
#pragma unroll
            for (int k = 0; k < kAhead; ++k) v[k] = partial[(s + kGroups * k) * M + m];
#pragma unroll
            for (int k = 0; k < kAhead; ++k) sum += v[k];
        }
        double v[kAhead - 1];
#pragma unroll
        for (int k = 0; k < kAhead - 1; ++k) v[k] = s + kGroups * k < shares ? partial[(s + kGroups * k) * M + m] : 0.0;
#pragma unroll
        for (int k = 0; k < kAhead - 1; ++k) sum += v[k];
    }
    part[g][col] = sum;
    __syncthreads();
    if (g != 0 || m >= M) return;
#pragma unroll
    for (int k = 1; k < kGroups; ++k) sum += part[k][col];
    out[m] = (float)sum;
}

struct Shares {
    int64_t count = 1;
    int lpr, col_tiles;           // rows
    int64_t planes, length;       // planes
    int parts = 1;
};

// Up to this many rows a workgroup of sixteen wavefronts adds a column tile in one launch (two take 3 us more).
constexpr int64_t kSingleRows = 256;
// ... and up to this many values a workgroup a column of planes.
constexpr int64_t kSingleValues = 4096;

// Otherwise two (rows) or four (planes) workgroups per compute unit: more of them have a longer second step, fewer leave the
// memory waiting.  At least eight loads per lane of a row's, four of a plane's.
Shares share_out(int64_t outer, int M, int64_t inner) {
    Shares p;
    p.lpr = std::min((M + 3) / 4, 64);
    p.col_tiles = (M + kTileCols - 1) / kTileCols;
    p.planes = outer;
    p.length = inner;
    const auto up = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
    if (inner == 1) {
        if (outer <= kSingleRows) return p;
        const int64_t groups = std::max(2 * compute_units() / p.col_tiles, 1);
        p.count = up(outer, std::max<int64_t>(up(outer, groups), 32 * (64 / p.lpr)));
        return p;
    }
    if (outer * inner <= kSingleValues) return p;
    const int64_t groups = std::max(4 * compute_units() / M, 1);
    const int64_t values = std::max<int64_t>(up(outer * inner, groups), 4 * kPlaneThreads);
    if (values >= inner) {
        p.planes = up(values, inner);
        p.count = up(outer, p.planes);
    } else {
        p.planes = 1;
        p.length = up(inner, up(inner, values));
        p.parts = (int)up(inner, p.length);
        p.count = outer * p.parts;
    }
    return p;
}

}  // namespace

size_t column_sums_workspace(int64_t outer, int M, int64_t inner) {
    const size_t sums = (size_t)share_out(outer, M, inner).count * M * sizeof(double);
    // never less than the float per plane that the first form of these kernels took
    return std::max(sums, inner > 1 ? (size_t)outer * M * sizeof(float) : (size_t)0);
}

hipError_t launch_column_sums(const float* G, int64_t outer, int64_t ldg, int M, int64_t inner, void* workspace, float* out,
                              hipStream_t s) {
    const Shares p = share_out(outer, M, inner);
    f64* partial = static_cast<f64*>(workspace);
    const bool single = p.count == 1;
    if (inner > 1) {
        const int64_t blocks = p.count * M;
        if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
        hipLaunchKernelGGL(plane_share_sums_kernel, dim3((unsigned)blocks), dim3(kPlaneThreads), 0, s, G, outer, M, inner,
                           p.planes, p.parts, p.length, partial, out, single);
    } else {
        const int64_t blocks = p.count * p.col_tiles;
        if (M < 4 || blocks > 0x7fffffffLL) return hipErrorInvalidValue;
        if (single)
            hipLaunchKernelGGL(row_chunk_sums_kernel<16>, dim3((unsigned)blocks), dim3(1024), 0, s, G, outer, ldg, M, p.col_tiles,
                               p.lpr, (int)p.count, partial, out, true);
        else
            hipLaunchKernelGGL(row_chunk_sums_kernel<4>, dim3((unsigned)blocks), dim3(256), 0, s, G, outer, ldg, M, p.col_tiles,
                               p.lpr, (int)p.count, partial, out, false);
    }
    if (hipError_t e = hipGetLastError()) return e;
    if (single) return hipSuccess;
    const dim3 grid((unsigned)((M + 31) / 32));
    if (p.count <= 8 * kAhead)
        hipLaunchKernelGGL(share_sums_kernel<8>, grid, dim3(32 * 8), 0, s, partial, p.count, M, out);
    else
        hipLaunchKernelGGL(share_sums_kernel<32>, grid, dim3(32 * 32), 0, s, partial, p.count, M, out);
    return hipGetLastError();
}

}  // namespace lutnn
