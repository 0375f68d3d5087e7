// Stand-alone lookups that read the table rows straight from global memory (arXiv 2302.03213, Eq. 4), for 8-bit and
// 16-bit indices.
#pragma once
#include "gather_row.h"

namespace lutnn {
namespace {

constexpr int kGatherThreads = 256;
constexpr int kGatherWaves = 4;

// ------------------------------------------------------------------------------- any K: no LDS
// One thread per (row, column); the table is read straight from global memory (L2).  For rows of fewer
// columns than a lane of the gather takes, and codebooks whose K x MT slab does not fit the LDS staging buffer.
template <class Table, class Index>
__global__ __launch_bounds__(kGatherThreads) void lookup_global_kernel(
    const typename Table::Entry* __restrict__ T, const float* __restrict__ scale, const float* __restrict__ bias, int C,
    int K, int M, const Index* __restrict__ idx, int64_t N, float* __restrict__ Y, int64_t ldy) {
    const int64_t i = (int64_t)blockIdx.x * kGatherThreads + threadIdx.x;
    if (i >= N * (int64_t)M) return;
    const int64_t n = i / M;
    const int m = (int)(i % M);
    typename Table::Acc acc = 0;
    const Index* __restrict__ irow = idx + n * C;
    const auto entry = [&](int c, int k) {
        k = k < K ? k : K - 1;
        return T[((size_t)c * K + k) * Table::row_entries(M) + Table::offset(m)];
    };
    const auto add = [&](typename Table::Entry e) {
        if constexpr (std::is_same<Table, TableI4>::value)
            acc += (int32_t)((((m & 1) ? e >> 4 : e & 0xf) ^ 8) - 8);
        else
            acc += (typename Table::Acc)e;
    };
    // eight codebooks' indices in flight, then their entries, added in codebook order
    constexpr int kBatch = 8;
    int c = 0;
    for (; c + kBatch <= C; c += kBatch) {
        int k[kBatch];
        typename Table::Entry e[kBatch];
#pragma unroll
        for (int b = 0; b < kBatch; ++b) k[b] = irow[c + b];
#pragma unroll
        for (int b = 0; b < kBatch; ++b) e[b] = entry(c + b, k[b]);
#pragma unroll
        for (int b = 0; b < kBatch; ++b) add(e[b]);
    }
    for (; c < C; ++c) add(entry(c, irow[c]));
    if constexpr (std::is_same<Table, TableF32>::value)
        Y[n * ldy + m] = bias ? acc + bias[m] : acc;
    else
        Y[n * ldy + m] = bias ? __fmaf_rn((float)acc, *scale, bias[m]) : __fmul_rn((float)acc, *scale);
}

template <class Table, class Index>
hipError_t launch_global(const typename Table::Entry* T, const float* scale, const float* bias, int C, int K, int M,
                         const Index* idx, int64_t N, float* Y, int64_t ldy, hipStream_t s) {
    const int64_t blocks = (N * (int64_t)M + kGatherThreads - 1) / kGatherThreads;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((lookup_global_kernel<Table, Index>), dim3((unsigned)blocks), dim3(kGatherThreads), 0, s, T, scale,
                       bias, C, K, M, idx, N, Y, ldy);
    return hipGetLastError();
}

// ------------------------------------------------------------------------- few rows: no staging
// Staging a K x MT slab per codebook pays off when many rows of a workgroup read it.  With few
// rows (a batch of a few hundred) the staged grid cannot even fill the chip, and the slab is read
// from L2 by every row tile anyway.  Here one wavefront owns one row and a run of 64 * kCols columns,
// and reads the selected table rows straight from global memory (gather_row.h).  The
// index is wave-uniform.  Sums run over the codebooks in order, as in the staged kernels.
//
// UNIFORM: a wavefront works on one row (64 lanes or more per row).  Otherwise rows are
// narrower than a wavefront: `lpr` lanes per row, 64 / lpr rows per wavefront, per-lane index loads.
template <class Table, class Index, bool IDX_DWORD, bool UNIFORM>
__global__ __launch_bounds__(kGatherThreads) void lookup_gather_kernel(
    const typename Table::Entry* __restrict__ T, const float* __restrict__ scale, const float* __restrict__ bias, int C,
    int K, int M, const Index* __restrict__ idx, int64_t N, float* __restrict__ Y, int64_t ldy,
    int col_chunks, int lpr) {
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t gw = (int64_t)blockIdx.x * kGatherWaves + w;
    int64_t row;
    int m;
    if (UNIFORM) {
        row = gw / col_chunks;
        m = ((int)(gw % col_chunks) * 64 + lane) * Table::kCols;
    } else {
        const int sub = lane / lpr;
        if (sub >= 64 / lpr) return;
        row = gw * (64 / lpr) + sub;
        m = (lane - sub * lpr) * Table::kCols;
    }
    if (row >= N) return;
    if (m >= M) return;
    gather_row<Table, Index, IDX_DWORD, UNIFORM>(T, scale, bias, C, K, M, idx + row * C, m, Y + row * ldy);
}

// The same gather for a handful of rows (batch-1 inference, the paper's own setting): with so few
// wavefronts the per-row chain of C loads and additions is pure latency, so the SPLIT wavefronts of
// a workgroup share one (row, 64 * kCols columns) and take a contiguous range of codebooks each.
template <class Table, class Index, bool IDX_DWORD, int SPLIT>
__global__ __launch_bounds__(64 * SPLIT) void lookup_gather_split_kernel(
    const typename Table::Entry* __restrict__ T, const float* __restrict__ scale, const float* __restrict__ bias, int C,
    int K, int M, const Index* __restrict__ idx, float* __restrict__ Y, int64_t ldy, int col_chunks, int per_wave) {
    const int lane = threadIdx.x & 63;
    const int64_t row = blockIdx.x / col_chunks;  // < N by construction of the grid
    const int m = ((int)(blockIdx.x % col_chunks) * 64 + lane) * Table::kCols;
    gather_row_split<Table, Index, IDX_DWORD, SPLIT>(T, scale, bias, C, K, M, idx + row * C, m, Y + row * ldy, per_wave);
}

// Fewer (row, column chunk) pairs than this and at least this many codebooks: the split form
// (measured at C = 1024, M = 4096: faster than one wavefront per pair up to about 160 rows).
constexpr int64_t kSplitMaxWaves = 2049;
constexpr int kSplitMinCodebooks = 64;

template <class Table, class Index>
hipError_t launch_gather(const typename Table::Entry* T, const float* scale, const float* bias, int C, int K, int M,
                         const Index* idx, int64_t N, float* Y, int64_t ldy, hipStream_t s) {
    const bool idx_dword = C % (int)(4 / sizeof(Index)) == 0 && (reinterpret_cast<uintptr_t>(idx) & 3) == 0;
    const int lpr = (M + Table::kCols - 1) / Table::kCols;  // lanes per row when a row is narrower than a wavefront
    if (lpr >= 64) {
        const int col_chunks = (lpr + 63) / 64;
        if (N * col_chunks < kSplitMaxWaves && C >= kSplitMinCodebooks) {
            const dim3 grid((unsigned)(N * col_chunks));
#define LUTNN_LAUNCH_SPLIT(DW, SPLIT)                                                                           \
    hipLaunchKernelGGL((lookup_gather_split_kernel<Table, Index, DW, SPLIT>), grid, dim3(64 * SPLIT), 0, s, T, scale,  \
                       bias, C, K, M, idx, Y, ldy, col_chunks, ((C + SPLIT - 1) / SPLIT + 3) & ~3)
            if (C >= 512) {
                if (idx_dword) LUTNN_LAUNCH_SPLIT(true, 16); else LUTNN_LAUNCH_SPLIT(false, 16);
            } else {
                if (idx_dword) LUTNN_LAUNCH_SPLIT(true, 4); else LUTNN_LAUNCH_SPLIT(false, 4);
            }
#undef LUTNN_LAUNCH_SPLIT
            return hipGetLastError();
        }
        const int64_t blocks = (N * col_chunks + kGatherWaves - 1) / kGatherWaves;
        if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
        if (idx_dword)
            hipLaunchKernelGGL((lookup_gather_kernel<Table, Index, true, true>), dim3((unsigned)blocks),
                               dim3(kGatherThreads), 0, s, T, scale, bias, C, K, M, idx, N, Y, ldy, col_chunks, lpr);
        else
            hipLaunchKernelGGL((lookup_gather_kernel<Table, Index, false, true>), dim3((unsigned)blocks),
                               dim3(kGatherThreads), 0, s, T, scale, bias, C, K, M, idx, N, Y, ldy, col_chunks, lpr);
    } else {
        const int64_t rows_per_block = (int64_t)(64 / lpr) * kGatherWaves;
        const int64_t blocks = (N + rows_per_block - 1) / rows_per_block;
        if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
        if (idx_dword)
            hipLaunchKernelGGL((lookup_gather_kernel<Table, Index, true, false>), dim3((unsigned)blocks),
                               dim3(kGatherThreads), 0, s, T, scale, bias, C, K, M, idx, N, Y, ldy, 1, lpr);
        else
            hipLaunchKernelGGL((lookup_gather_kernel<Table, Index, false, false>), dim3((unsigned)blocks),
                               dim3(kGatherThreads), 0, s, T, scale, bias, C, K, M, idx, N, Y, ldy, 1, lpr);
    }
    return hipGetLastError();
}

}  // namespace
}  // namespace lutnn
