// One output row's share of the table read and accumulation (arXiv 2302.03213, Eq. 4) when the
// table rows are read straight from global memory: a lane owns four consecutive columns (eight of a
// 4-bit table) and adds the selected row of every codebook, in codebook order, sixteen loads in
// flight at a time.  Shared by the stand-alone gather kernels and the one-launch kernel for small problems.
//
// Any width and any alignment: the hardware reads a dword or four from any byte (dword) address, so rows that
// start anywhere are read like aligned ones, and the last lane of a row takes the row's last group of
// columns, which may overlap its neighbour's (both then store the same values).  A wavefront that shares a row
// of indices reads them as dwords too, wherever they start.
//
// What bounds it: the chain of loads where rows are few, the rate of the table's reads where they are many.  Whole calls,
// before (staged through LDS where the width was no multiple of four, one load at a time where the number of codebooks was
// none) and with this: 106 rows x 512 codebooks, M = 157, fp32 1016 -> 27 us; 30 x 413, M = 1146, INT8 89 -> 8; 67 x 17 of
// 64 table rows, M = 148, INT4 88 -> 8; 4096 x 96 of 4096 table rows (16-bit indices, four loads in flight before), M =
// 768, INT8 89 -> 63.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace lutnn {

// What a lane reads of a table row, by the table's type.
struct TableF32 {
    using Entry = float;
    using Acc = float;
    static constexpr int kCols = 4;
    typedef float Vec __attribute__((ext_vector_type(4), aligned(4)));
    __host__ __device__ static int row_entries(int M) { return M; }
    __host__ __device__ static int last_group(int M) { return M - 4; }
    __device__ static int offset(int m) { return m; }
    __device__ __forceinline__ static void add(Acc (&a)[4], Vec v) {
#pragma unroll
        for (int j = 0; j < 4; ++j) a[j] += v[j];
    }
};
struct TableI8 {
    using Entry = int8_t;
    using Acc = int32_t;
    static constexpr int kCols = 4;
    typedef uint32_t Vec __attribute__((aligned(1)));
    __host__ __device__ static int row_entries(int M) { return M; }
    __host__ __device__ static int last_group(int M) { return M - 4; }
    __device__ static int offset(int m) { return m; }
    __device__ __forceinline__ static void add(Acc (&a)[4], uint32_t v) {
        a[0] += (int32_t)(int8_t)(v & 0xffu);
        a[1] += (int32_t)(int8_t)((v >> 8) & 0xffu);
        a[2] += (int32_t)(int8_t)((v >> 16) & 0xffu);
        a[3] += (int32_t)v >> 24;
    }
};
struct TableI4 {  // rows of ceil(M / 2) bytes, even column in the low nibble
    using Entry = uint8_t;
    using Acc = int32_t;
    static constexpr int kCols = 8;
    typedef uint32_t Vec __attribute__((aligned(1)));
    __host__ __device__ static int row_entries(int M) { return (M + 1) / 2; }
    __host__ __device__ static int last_group(int M) { return 2 * ((M + 1) / 2 - 4); }
    __device__ static int offset(int m) { return m / 2; }
    __device__ __forceinline__ static void add(Acc (&a)[8], uint32_t v) {
#pragma unroll
        for (int j = 0; j < 8; ++j) a[j] += (int32_t)(v << (28 - 4 * j)) >> 28;  // nibble j, sign extended
    }
};
// A row has at least one whole group of columns.
template <class Table>
inline bool gather_supported(int M) {
    return Table::last_group(M) >= 0;
}

// Adds the rows that irow[c], c in [c, c_end), select to `a`, in that order.
//   tcol     the lane's columns of table row 0
//   irow     index bytes (or 16-bit indices) in global memory or LDS; DWORD: irow + c is 4-byte aligned
//   UNIFORM  the whole wavefront works on the same row: index words are made wave-uniform
template <class Table, class Index, bool DWORD, bool UNIFORM>
__device__ __forceinline__ void gather_range(const typename Table::Entry* __restrict__ tcol, int C, int K, int M,
                                             const Index* __restrict__ irow, int c, int c_end,
                                             typename Table::Acc (&a)[Table::kCols]) {
    using Vec = typename Table::Vec;
    constexpr int kBatch = 16, kPer = 4 / sizeof(Index), kWords = kBatch / kPer;
    constexpr uint32_t kMask = sizeof(Index) == 1 ? 0xffu : 0xffffu;
    auto uni = [](uint32_t x) { return UNIFORM ? (uint32_t)__builtin_amdgcn_readfirstlane(x) : x; };
    auto word_at = [&](int c0) {
        typedef uint32_t AnyByte __attribute__((aligned(1)));
        if constexpr (DWORD) return *reinterpret_cast<const uint32_t*>(irow + c0);
        return (uint32_t)*reinterpret_cast<const AnyByte*>(irow + c0);
    };
    const uint32_t stride = (uint32_t)Table::row_entries(M);
    auto row = [&](int c0, uint32_t word, int b) -> const Vec& {
        uint32_t k = (word >> (8 * sizeof(Index) * (b % kPer))) & kMask;
        k = k < (uint32_t)K ? k : (uint32_t)(K - 1);
        return *reinterpret_cast<const Vec*>(tcol + ((size_t)(c0 + b) * (size_t)(stride * (uint64_t)K) + (uint64_t)k * stride));
    };
    // sixteen table rows in flight at a time (added in codebook order all the same), and behind them the next
    // sixteen indices: with few wavefronts the loop is a latency chain, and every wait of its own counts
    uint32_t next[kWords];
    if (c + kBatch <= c_end) {
#pragma unroll
        for (int q = 0; q < kWords; ++q) next[q] = word_at(c + q * kPer);
    }
    for (; c + kBatch <= c_end; c += kBatch) {
        uint32_t word[kWords];
#pragma unroll
        for (int q = 0; q < kWords; ++q) word[q] = uni(next[q]);
        Vec v[kBatch];
#pragma unroll
        for (int b = 0; b < kBatch; ++b) v[b] = row(c, word[b / kPer], b);
        if (c + 2 * kBatch <= c_end) {
#pragma unroll
            for (int q = 0; q < kWords; ++q) next[q] = word_at(c + kBatch + q * kPer);
        }
#pragma unroll
        for (int b = 0; b < kBatch; ++b) Table::add(a, v[b]);
    }
    // the rest: eight, four and up to three more, all in flight at once
    const int left = max(c_end - c, 0);  // nothing at all for the last wavefronts of a split row
    Vec v8[8], v4[4], v1[3];
    const int c4 = c + (left & 8), c1 = c4 + (left & 4);
    if (left & 8) {
        uint32_t word[8 / kPer];
#pragma unroll
        for (int q = 0; q < 8 / kPer; ++q) word[q] = uni(word_at(c + q * kPer));
#pragma unroll
        for (int b = 0; b < 8; ++b) v8[b] = row(c, word[b / kPer], b);
    }
    if (left & 4) {
        uint32_t word[4 / kPer];
#pragma unroll
        for (int q = 0; q < 4 / kPer; ++q) word[q] = uni(word_at(c4 + q * kPer));
#pragma unroll
        for (int b = 0; b < 4; ++b) v4[b] = row(c4, word[b / kPer], b);
    }
    uint32_t k1[3];
#pragma unroll
    for (int b = 0; b < 3; ++b)
        if (b < (left & 3)) k1[b] = (uint32_t)irow[c1 + b];
#pragma unroll
    for (int b = 0; b < 3; ++b)
        if (b < (left & 3)) v1[b] = row(c1 + b, uni(k1[b]), 0);
    if (left & 8) {
#pragma unroll
        for (int b = 0; b < 8; ++b) Table::add(a, v8[b]);
    }
    if (left & 4) {
#pragma unroll
        for (int b = 0; b < 4; ++b) Table::add(a, v4[b]);
    }
#pragma unroll
    for (int b = 0; b < 3; ++b)
        if (b < (left & 3)) Table::add(a, v1[b]);
}

// Dequantises (r = s*q, Sec. 3.3), adds the bias and stores the lane's columns m ...  Whole vectors, from any address: a load of
// its own for every column's bias, each waited for, was most of a row of few codebooks (20429 rows x 1 codebook, M = 192
// 7.7 -> 6.3 us; 3039 x 3, M = 1472 8.3 -> 7.5).
template <class Table>
__device__ __forceinline__ void store_columns_of_row(const typename Table::Acc (&a)[Table::kCols],
                                                     const float* __restrict__ scale, const float* __restrict__ bias,
                                                     int m, int M, float* __restrict__ yrow) {
    typedef float Four __attribute__((ext_vector_type(4), aligned(4)));
    constexpr int kFours = Table::kCols / 4;
    float s = 1.f;
    if constexpr (!std::is_same<Table, TableF32>::value) s = *scale;
    if (Table::kCols > 4 && m + Table::kCols > M) {  // an odd M leaves half a byte at the end of a 4-bit row
#pragma unroll
        for (int j = 0; j < Table::kCols; ++j)
            if (m + j < M) yrow[m + j] = bias ? __fmaf_rn((float)a[j], s, bias[m + j]) : __fmul_rn((float)a[j], s);
        return;
    }
    Four out[kFours];
    if (bias) {
        Four b[kFours];
#pragma unroll
        for (int q = 0; q < kFours; ++q) b[q] = *reinterpret_cast<const Four*>(bias + m + 4 * q);
#pragma unroll
        for (int j = 0; j < Table::kCols; ++j) {
            if constexpr (std::is_same<Table, TableF32>::value)
                out[j / 4][j % 4] = a[j] + b[j / 4][j % 4];
            else
                out[j / 4][j % 4] = __fmaf_rn((float)a[j], s, b[j / 4][j % 4]);
        }
    } else {
#pragma unroll
        for (int j = 0; j < Table::kCols; ++j) {
            if constexpr (std::is_same<Table, TableF32>::value)
                out[j / 4][j % 4] = a[j];
            else
                out[j / 4][j % 4] = __fmul_rn((float)a[j], s);
        }
    }
#pragma unroll
    for (int q = 0; q < kFours; ++q) *reinterpret_cast<Four*>(yrow + m + 4 * q) = out[q];
}

// The same for column m alone.
template <class Table>
__device__ __forceinline__ float dequantised(typename Table::Acc sum, const float* __restrict__ scale,
                                             const float* __restrict__ bias, int m) {
    if constexpr (std::is_same<Table, TableF32>::value)
        return bias ? sum + bias[m] : sum;
    else
        return bias ? __fmaf_rn((float)sum, *scale, bias[m]) : __fmul_rn((float)sum, *scale);
}

//   T       table, [C][K] rows; gather_supported(M)
//   irow    this row's C indices; DWORD: 4-byte aligned
//   m       first of the lane's columns (< M, a multiple of kCols)
//   yrow    &Y[row][0]
template <class Table, class Index, bool DWORD, bool UNIFORM>
__device__ __forceinline__ void gather_row(const typename Table::Entry* __restrict__ T, const float* __restrict__ scale,
                                           const float* __restrict__ bias, int C, int K, int M,
                                           const Index* __restrict__ irow, int m, float* __restrict__ yrow) {
    m = min(m, Table::last_group(M));
    typename Table::Acc a[Table::kCols] = {};
    gather_range<Table, Index, DWORD, UNIFORM>(T + Table::offset(m), C, K, M, irow, 0, C, a);
    store_columns_of_row<Table>(a, scale, bias, m, M, yrow);
}

// The same for a handful of rows: the SPLIT wavefronts of a workgroup share one row and 64 * kCols columns
// and take a contiguous range of `per_wave` codebooks each (a multiple of 4); the partial sums meet
// in LDS and are added in range order (exact for integer tables, a fixed order for fp32
// ones): by wavefront 0, or of sixteen wavefronts by one for each column of the lanes.  Every thread of the workgroup must call it (it holds a barrier); m may lie past M.
template <class Table, class Index, bool DWORD, int SPLIT>
__device__ __forceinline__ void gather_row_split(const typename Table::Entry* __restrict__ T,
                                                 const float* __restrict__ scale, const float* __restrict__ bias, int C,
                                                 int K, int M, const Index* __restrict__ irow, int m,
                                                 float* __restrict__ yrow, int per_wave) {
    using Acc = typename Table::Acc;
    constexpr int kCols = Table::kCols;
    __shared__ Acc part[SPLIT][kCols][64];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool col_ok = m < M;
    m = min(m, Table::last_group(M));

    Acc a[kCols] = {};
    gather_range<Table, Index, DWORD, true>(T + Table::offset(m), C, K, M, irow, w * per_wave, min(C, (w + 1) * per_wave), a);
#pragma unroll
    for (int j = 0; j < kCols; ++j) part[w][j][lane] = a[j];
    __syncthreads();
    if (!col_ok) return;
    const auto total = [&](int j) {
        Acc sum = part[0][j][lane];
#pragma unroll
        for (int ww = 1; ww < SPLIT; ++ww) sum += part[ww][j][lane];
        return sum;
    };
    if constexpr (SPLIT <= 4) {
        if (w != 0) return;
#pragma unroll
        for (int j = 0; j < kCols; ++j) a[j] = total(j);
        store_columns_of_row<Table>(a, scale, bias, m, M, yrow);
    } else if (w < kCols && (kCols == 4 || m + w < M)) {
        yrow[m + w] = dequantised<Table>(total(w), scale, bias, m + w);
    }
}

}  // namespace lutnn
