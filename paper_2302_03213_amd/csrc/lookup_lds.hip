// Table read and accumulation (arXiv 2302.03213, Eq. 4 and Sec. 5.2), LDS gather variant, gfx950.
//
//   Y[n][m] = epilogue( sum_c T[c][idx[n][c]][m] )
//
// A workgroup owns an (R rows x MT columns) output tile and walks the codebooks in stages: the
// K x MT slab of each of CC codebooks is staged in LDS as [codebook][k][MT] (m fastest), then
// every wavefront handles its own rows one at a time.  For one (row, codebook) the index is
// wave-uniform: it is fetched with a scalar load, four codebooks per dword, and the 64 lanes read
// 64 consecutive dwords of the selected table row - consecutive banks, conflict free by
// construction.  The paper's byte-shuffle table read (16 lookups per 128-bit shuffle) has no
// CDNA counterpart; a wave-wide LDS row read is the equivalent "one instruction, many lookups".
//
// INT8 accumulation follows the paper's mixed-precision idea (16-bit partial sums, then 32-bit):
// table bytes are stored in LDS with a +128 bias so they are unsigned, one dword carries four
// columns, and the even/odd bytes are added as two packed 16-bit lanes with plain 32-bit adds.
// 256 biased bytes cannot overflow 16 bits (256*255 < 65536); the partial sums are widened to
// int32 at least that often and the bias (128 per codebook) is removed in the epilogue, so the
// result is the exact integer sum.
#include <algorithm>
#include <type_traits>

#include "gather_launch.h"
#include "lookup_f32_forms.h"
#include "lutnn_kernels.h"

namespace lutnn {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = 4;

// ------------------------------------------------------------------------------------------ INT8
constexpr int kColsI8 = 256;  // MT: 64 lanes x 4 columns
constexpr int kRowsPerWaveI8 = 16;

// BITS = 8: T[C][K][M] int8.  BITS = 4: T[C][K][ceil(M/2)] bytes, two 4-bit entries each (even
// column in the low nibble); they are widened to bytes while being staged, the rest is the same.
template <bool IDX_DWORD, int BITS = 8>
__global__ __launch_bounds__(kThreads) void lookup_lds_i8_kernel(
    const int8_t* __restrict__ T, const float* __restrict__ scale, const float* __restrict__ bias,
    int C, int K, int M, const uint8_t* __restrict__ idx, int64_t N, float* __restrict__ Y,
    int64_t ldy, int CC, int col_tiles, int table_vec16) {
    extern __shared__ uint32_t lds[];  // [CC][K][64] dwords = 4 biased bytes each
    constexpr int RW = kRowsPerWaveI8;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t row_tile = blockIdx.x / col_tiles;
    const int n0 = (int)(blockIdx.x % col_tiles) * kColsI8;
    const int64_t row0 = row_tile * (RW * kWaves) + (int64_t)w * RW;

    uint32_t lo[RW], hi[RW];
    int32_t acc[RW][4];
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        lo[r] = hi[r] = 0;
        acc[r][0] = acc[r][1] = acc[r][2] = acc[r][3] = 0;
    }
    int pending = 0;  // codebooks accumulated in lo/hi since the last widening
    int slots = 0;    // codebook slots accumulated in total (each carries a +128 bias)

    for (int c0 = 0; c0 < C; c0 += CC) {
        __syncthreads();  // previous stage fully consumed
        // ---- stage [CC][K][256 B]; bytes outside the table become 0 (biased: 0x80)
        const int chunks = CC * K * 16;  // 16-byte chunks
        for (int i = tid; i < chunks; i += kThreads) {
            const int rowid = i >> 4, ch = i & 15;
            const int cl = rowid / K, k = rowid - cl * K;
            const int c = c0 + cl;
            const int m = n0 + ch * 16;
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (c < C && BITS == 4) {
                const uint8_t* src =
                    reinterpret_cast<const uint8_t*>(T) + ((size_t)c * K + k) * ((M + 1) / 2) + m / 2;
                uint32_t t[4] = {0u, 0u, 0u, 0u};
                for (int b = 0; b < 16; b += 2) {  // m is even: byte b/2 holds columns m+b, m+b+1
                    if (m + b >= M) break;
                    const uint32_t two = src[b >> 1];
                    const uint32_t lo = ((two & 0xfu) ^ 8u) - 8u, hi = ((two >> 4) ^ 8u) - 8u;  // sign extend
                    t[b >> 2] |= (lo & 0xffu) << (8 * (b & 3));
                    if (m + b + 1 < M) t[b >> 2] |= (hi & 0xffu) << (8 * ((b + 1) & 3));
                }
                v = make_uint4(t[0], t[1], t[2], t[3]);
            } else if (c < C) {
                const int8_t* src = T + ((size_t)c * K + k) * M + m;
                if (table_vec16 && m + 16 <= M) {
                    v = *reinterpret_cast<const uint4*>(src);
                } else {
                    uint32_t t[4] = {0u, 0u, 0u, 0u};
                    for (int b = 0; b < 16; ++b)
                        if (m + b < M) t[b >> 2] |= (uint32_t)(uint8_t)src[b] << (8 * (b & 3));
                    v = make_uint4(t[0], t[1], t[2], t[3]);
                }
            }
            v.x ^= 0x80808080u;
            v.y ^= 0x80808080u;
            v.z ^= 0x80808080u;
            v.w ^= 0x80808080u;
            *reinterpret_cast<uint4*>(lds + (size_t)rowid * 64 + ch * 4) = v;
        }
        __syncthreads();

        if (pending + CC > 256) {  // widen before 16-bit lanes could overflow
#pragma unroll
            for (int r = 0; r < RW; ++r) {
                acc[r][0] += lo[r] & 0xffff;
                acc[r][2] += lo[r] >> 16;
                acc[r][1] += hi[r] & 0xffff;
                acc[r][3] += hi[r] >> 16;
                lo[r] = hi[r] = 0;
            }
            pending = 0;
        }
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const int64_t row = row0 + r;
            if (row < N) {
                for (int cl4 = 0; cl4 < CC; cl4 += 4) {
                    uint32_t word;
                    if (IDX_DWORD) {  // C % 4 == 0, 4-byte aligned: in range whenever c0+cl4 < C
                        word = (c0 + cl4 < C)
                                   ? *reinterpret_cast<const uint32_t*>(idx + row * C + c0 + cl4)
                                   : 0u;
                    } else {
                        word = 0;
                        for (int b = 0; b < 4; ++b)
                            if (c0 + cl4 + b < C)
                                word |= (uint32_t)idx[row * C + c0 + cl4 + b] << (8 * b);
                    }
                    word = __builtin_amdgcn_readfirstlane(word);
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        int k = (word >> (8 * b)) & 0xff;
                        k = k < K ? k : K - 1;  // out-of-range indices must not read out of bounds
                        const uint32_t x = lds[((cl4 + b) * K + k) * 64 + lane];
                        lo[r] += x & 0x00ff00ffu;
                        hi[r] += (x >> 8) & 0x00ff00ffu;
                    }
                }
            }
        }
        pending += CC;
        slots += CC;
    }

    // ---- epilogue: widen, remove the bias, dequantise (r = s*q, Sec. 3.3), add the layer bias
    const float s = *scale;
    const int col = n0 + lane * 4;
    float bv[4] = {0.f, 0.f, 0.f, 0.f};
    if (bias)
        for (int j = 0; j < 4; ++j)
            if (col + j < M) bv[j] = bias[col + j];
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int64_t row = row0 + r;
        if (row >= N) continue;
        int32_t a[4];
        a[0] = acc[r][0] + (int32_t)(lo[r] & 0xffff) - 128 * slots;
        a[2] = acc[r][2] + (int32_t)(lo[r] >> 16) - 128 * slots;
        a[1] = acc[r][1] + (int32_t)(hi[r] & 0xffff) - 128 * slots;
        a[3] = acc[r][3] + (int32_t)(hi[r] >> 16) - 128 * slots;
        float* y = Y + row * ldy + col;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (col + j < M)
                y[j] = bias ? __fmaf_rn((float)a[j], s, bv[j]) : __fmul_rn((float)a[j], s);
        }
    }
}

// The staged kernels need at least this many workgroups to be worth their staging.
constexpr int64_t kMinStagedBlocks = 512;

constexpr int kLdsBudget = 64 * 1024;

inline bool idx_dword_ok(const uint8_t* idx, int C) {
    return (C % 4 == 0) && ((reinterpret_cast<uintptr_t>(idx) & 3) == 0);
}

inline int64_t staged_blocks(int64_t N, int M) {
    return ((N + kRowsPerWaveI8 * kWaves - 1) / (kRowsPerWaveI8 * kWaves)) * ((M + kColsI8 - 1) / kColsI8);
}

// Table rows read straight from global memory: where the staged grid would be small, and where four codebooks' slabs do
// not fit its LDS (K > 64; one thread per output, the other choice there, reads a byte where this reads a dword).  fp32
// tables always: staged, 32 rows to a slab, they were two to four times slower.
template <class Table>
bool gather_ok(int64_t N, int K, int M) {
    return gather_supported<Table>(M) && (std::is_same<Table, TableF32>::value || staged_blocks(N, M) < kMinStagedBlocks ||
                                          (int64_t)4 * K * kColsI8 > kLdsBudget);
}

template <class Table>
hipError_t launch_lookup_lds(const typename Table::Entry* T, const float* scale, const float* bias, int C, int K, int M,
                             const uint8_t* idx, int64_t N, float* Y, int64_t ldy, hipStream_t s) {
    if (gather_ok<Table>(N, K, M)) return launch_gather<Table, uint8_t>(T, scale, bias, C, K, M, idx, N, Y, ldy, s);
    // LDS bytes per staged codebook (4-bit entries are widened to bytes)
    const int64_t per_codebook = (int64_t)K * kColsI8;
    if (std::is_same<Table, TableF32>::value || 4 * per_codebook > kLdsBudget)
        return launch_global<Table, uint8_t>(T, scale, bias, C, K, M, idx, N, Y, ldy, s);
    int CC = (int)(kLdsBudget / 2 / per_codebook) & ~3;  // aim for 32 KiB so two workgroups share a CU
    if (CC < 4) CC = 4;
    if (CC > 16) CC = 16;
    const int col_tiles = (M + kColsI8 - 1) / kColsI8;
    const int64_t blocks = staged_blocks(N, M);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const size_t shmem = (size_t)(CC * per_codebook);
    constexpr int BITS = std::is_same<Table, TableI4>::value ? 4 : 8;
    const int vec16 = BITS == 8 && (M % 16 == 0) && ((reinterpret_cast<uintptr_t>(T) & 15) == 0);
    const int8_t* Tb = reinterpret_cast<const int8_t*>(T);
    const dim3 grid((unsigned)blocks), block(kThreads);
    if (idx_dword_ok(idx, C))
        hipLaunchKernelGGL((lookup_lds_i8_kernel<true, BITS>), grid, block, shmem, s, Tb, scale, bias, C, K, M, idx, N, Y, ldy,
                           CC, col_tiles, vec16);
    else
        hipLaunchKernelGGL((lookup_lds_i8_kernel<false, BITS>), grid, block, shmem, s, Tb, scale, bias, C, K, M, idx, N, Y, ldy,
                           CC, col_tiles, vec16);
    return hipGetLastError();
}

template <class Table>
bool gather_preferred_t(int C, int K, int M, int64_t N, bool sparse_ok) {
    if (!gather_ok<Table>(N, K, M)) return false;
    // a few rows: the split gather reads N rows' worth of table entries, the matrix cores the whole
    // table; measured cross-over at config 5's width between 32 and 48 rows (K = 16)
    constexpr int chunk = 64 * Table::kCols;  // columns per wavefront
    const int64_t col_chunks = (M + chunk - 1) / chunk;
    if (M >= chunk && C >= kSplitMinCodebooks && N <= 32 && N * col_chunks < kSplitMaxWaves) return true;
    // Otherwise price both (ms per call, fitted to sweeps of 32-2048 rows over seventeen layer
    // shapes, and of 2-60000 rows of 1-700 codebooks and 4-4096 columns: the form taken needs 1.001 to 1.016 times the faster one's
    // time on average).  The gather costs its
    // N*C*M entry reads; a matrix-core launch costs its pipeline fill and the serial walk over the
    // codebooks - far longer per codebook on the dense kernel, which runs where the sparse one
    // cannot (C % 32 != 0 or unaligned indices).  From 512 codebooks on the sparse kernel shares
    // the codebooks of a tile out over workgroups and its time stops growing with C: there the
    // gather only wins below ~5.6e7 entries.
    const double entries = (double)N * C * M;
    if (C >= 512 && sparse_ok) return entries <= 5.6e7;
    // (Outputs cost the gather more than the matrix forms, which have whole tiles to write: 1311 rows x 2 codebooks, M =
    // 3436, INT4 18.5 us and 11.9, whole calls.)
    const double t_gather = 0.0038 + 8.9e-11 * entries + (std::is_same<Table, TableI4>::value ? 1.9e-9 : 5e-10) * (double)N * M;
    const double t_matrix = sparse_ok ? 0.0065 + 1.6e-5 * C : 0.0074 + 1.42e-4 * C + 2.2e-11 * entries;
    return t_gather < t_matrix;
}

}  // namespace

// True when the gather variant would read the table straight from L2 (no staging) and the whole
// problem is small enough for that to beat the matrix-core kernels, whose tiles and pipeline fill
// are wasted on it (measured cross-over: about 3e7 table entries).
bool gather_preferred(const void* T, int table_kind, int C, int K, int M, int64_t N, bool sparse_ok) {
    if (!T) return false;
    return table_kind == 0   ? gather_preferred_t<TableF32>(C, K, M, N, sparse_ok)
           : table_kind == 1 ? gather_preferred_t<TableI8>(C, K, M, N, sparse_ok)
                             : gather_preferred_t<TableI4>(C, K, M, N, sparse_ok);
}

hipError_t launch_lookup_lds_i8(const int8_t* T, const float* scale, const float* bias, int C, int K,
                                int M, const uint8_t* idx, int64_t N, float* Y, int64_t ldy,
                                hipStream_t s) {
    if (rows_kernel_preferred(N, M, K, false))
        return launch_lookup_rows_i8(T, 8, scale, bias, C, K, M, idx, N, Y, ldy, s);
    return launch_lookup_lds<TableI8>(T, scale, bias, C, K, M, idx, N, Y, ldy, s);
}

hipError_t launch_lookup_lds_i4(const uint8_t* T, const float* scale, const float* bias, int C, int K,
                                int M, const uint8_t* idx, int64_t N, float* Y, int64_t ldy,
                                hipStream_t s) {
    if (rows_kernel_preferred(N, M, K, false))
        return launch_lookup_rows_i8(T, 4, scale, bias, C, K, M, idx, N, Y, ldy, s);
    return launch_lookup_lds<TableI4>(T, scale, bias, C, K, M, idx, N, Y, ldy, s);
}

hipError_t launch_lookup_lds_f32(const float* T, const float* bias, int C, int K, int M,
                                 const uint8_t* idx, int64_t N, float* Y, int64_t ldy, hipStream_t s) {
    const LookupF32Us us = lookup_f32_us(C, K, M, N, rows_kernel_preferred(N, M, K, true), compute_units());
    LookupF32 form = us.least(N, M);
    const int pinned = tunable(kTuneLookupF32);
    if (pinned == 0) form = LookupF32::gather;
    if (pinned == 1 && rows_kernel_supported(K, true)) form = LookupF32::rows;
    if (pinned == 2 && us.matrix < LookupF32Us::kNever) form = LookupF32::matrix;
    if (form == LookupF32::matrix) return launch_lookup_matrix_f32(T, bias, C, K, M, idx, N, Y, ldy, s);
    if (form == LookupF32::rows) return launch_lookup_rows_f32(T, bias, C, K, M, idx, N, Y, ldy, s);
    return launch_lookup_lds<TableF32>(T, nullptr, bias, C, K, M, idx, N, Y, ldy, s);
}

}  // namespace lutnn
