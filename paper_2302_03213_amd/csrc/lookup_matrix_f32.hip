// Table read and accumulation (arXiv 2302.03213, Eq. 4) with an unquantised table on the 2:4 structured-sparse matrix
// instructions (v_smfmac_f32_32x32x32_bf16).
//
// The one-hot contraction of lookup_smfmac.hip with every table entry as the sum of three bf16 parts, which hold all of its
// 24 significant bits (split_bf16.h); the one-hot operand is 1.0 or 0, so that the products are the parts themselves.
// A slice of four codebooks is summed from zero, low parts first, and then added to the running sum in fp32: only the two
// instructions with the high parts round at the size of the sum.  Its error against 64-bit sums is 0.55 to 0.75 of the fp32
// chain's from 16 codebooks on where the entries are of one size, and no larger where they spread over 2^40 (relative to the
// sum of the terms' magnitudes: 0.93 at 16 codebooks, 0.83 at 32).  Of fewer codebooks such entries are summed less exactly
// than by the chain (1.2 times its error at 4, 1.07 at 8), which they are left to.  Sums that are not finite (an infinite or huge entry, which has no parts and
// reaches every row of its column) are formed again as that chain.
//
// What bounds it.  A table value read from LDS serves 64 rows here, where a gather reads it for one; the bound is
// the vector instructions that cut the table and build the one-hot operand (about 300 per wavefront and stage) beside 24
// matrix instructions: 1.4 us a stage and workgroup, which is no less with two workgroups on the compute unit.  Against the
// other forms (rows read from L2 by every row; staged in LDS for 256 rows), lookup alone: 1000 rows x 192 codebooks, M = 3072
// 81 us (253 and 161); 4096 x 192, M = 768 81 (118 and 138); 4096 x 192, M = 3072 172 (1064 and 185); 4096 x 700, M = 768 262
// (622 and 581).  Few columns leave the gather ahead: 14000 x 64, M = 150 34 (30).  The table is cut where it is staged, so no second copy of it exists.
//
// Layout (lane = 32 h + l): A values 0-3 are k 8h .. 8h+7 of the first codebook of a pair, values 4-7 those of the second,
// two stored values to four k, their positions in bits 2t of the index word; B, column l, is all 16 k of codebook h.
// Workgroup = 4 wavefronts stacked over rows, 256 rows x 64 columns, two of them per compute unit: one cuts while the other
// multiplies.
#include <algorithm>

#include "lutnn_kernels.h"
#include "mfma_tile.h"
#include "split_bf16.h"

namespace lutnn {
namespace {

typedef __bf16 bf16x16 __attribute__((ext_vector_type(16)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int kBM = 256, kBN = 64, kCB = 4;  // rows, columns, codebooks of a stage
constexpr int kPerCU = 2;                    // workgroups per compute unit
constexpr int kMinCodebooks = 16;            // precision: see above
constexpr int kPlane = kCB * 2 * kBN;        // 16-byte units (8 k of one column) per part

__global__ __launch_bounds__(kMfmaThreads, kPerCU) void lookup_matrix_f32_kernel(
    const float* __restrict__ T, const float* __restrict__ bias, int C, int K, int M, const uint8_t* __restrict__ idx,
    int64_t N, float* __restrict__ Y, int64_t ldy, int row_tiles, int64_t tiles) {
    __shared__ u32x4 parts[3 * kPlane];  // [high, mid, low][codebook][half of k][column]

    const int64_t t = xcd_tile(tiles);
    if (t < 0) return;
    const int n0 = (int)(t / row_tiles) * kBN;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t row0 = (t % row_tiles) * kBM + w * 64;

    const uint8_t* irow[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int64_t row = row0 + 32 * i + l32;
        irow[i] = idx + (row < N ? row : N - 1) * C;  // rows past N are not stored
    }
    // this wavefront stages half w & 1 of the k of codebooks (w >> 1) and (w >> 1) + 2, lane = column
    const int kh = 8 * (w & 1), cs = w >> 1;
    // Rows past K and codebooks past C are read where the last one is: the one-hot operand has nothing there.
    const uint32_t col = n0 + lane < M ? n0 + lane : M - 1;
    uint32_t value[2][8], word[2];
    const auto load = [&](int c0) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const float* __restrict__ slab = T + (int64_t)min(c0 + cs + 2 * j, C - 1) * K * M;
#pragma unroll
            for (int k = 0; k < 8; ++k) value[j][k] = __float_as_uint((slab + (int64_t)min(kh + k, K - 1) * M)[col]);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {  // the last four where fewer are left
            typedef uint32_t AnyByte __attribute__((aligned(1)));
            word[i] = *reinterpret_cast<const AnyByte*>(irow[i] + min(c0, C - 4));
        }
    };

    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x16{};

    load(0);
    for (int c0 = 0; c0 < C; c0 += kCB) {
        __syncthreads();  // the stage before has been read
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            uint32_t high[4], mid[4], low[4];
            cut<4>(value[j], high, mid, low);
            u32x4* const to = parts + (2 * (cs + 2 * j) + (w & 1)) * kBN + lane;
            to[0] = u32x4{high[0], high[1], high[2], high[3]};
            to[kPlane] = u32x4{mid[0], mid[1], mid[2], mid[3]};
            to[2 * kPlane] = u32x4{low[0], low[1], low[2], low[3]};
        }
        // the one-hot operands of both pairs
        const int shift = 8 * (c0 - min(c0, C - 4));
        bf16x8 a[2][2];
        int pos[2][2];
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                // 64: no k of any lane
                const uint32_t k0 = min((word[i] >> shift >> (16 * p)) & 0xffu, (uint32_t)(K - 1)) | (c0 + 2 * p < C ? 0u : 64u);
                const uint32_t k1 = min((word[i] >> shift >> (16 * p + 8)) & 0xffu, (uint32_t)(K - 1)) | (c0 + 2 * p + 1 < C ? 0u : 64u);
                const uint32_t g0 = (k0 >> 2) - 2 * h, g1 = (k1 >> 2) - 2 * h;
                a[p][i] = __builtin_bit_cast(bf16x8, u32x4{g0 == 0 ? 0x3f80u : 0u, g0 == 1 ? 0x3f80u : 0u,
                                                           g1 == 0 ? 0x3f80u : 0u, g1 == 1 ? 0x3f80u : 0u});
                pos[p][i] = (int)((k0 & 3) * 0x11u | (k1 & 3) * 0x1100u);
            }
        __syncthreads();
        if (c0 + kCB < C) load(c0 + kCB);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            f32x16 s[2] = {f32x16{}, f32x16{}};
#pragma unroll
            for (int q = 2; q >= 0; --q)  // low, mid, high
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const u32x4* const from = parts + q * kPlane + 2 * (2 * p + h) * kBN + 32 * j + l32;
                    struct { u32x4 lo, hi; } pair = {from[0], from[kBN]};
                    const bf16x16 b = __builtin_bit_cast(bf16x16, pair);
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        s[i] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(a[p][i], b, s[i], pos[p][i], 0, 0);
                }
#pragma unroll
            for (int i = 0; i < 2; ++i) acc[i][j] += s[i];
        }
    }

    float probe = 0.f;  // NaN once a sum is not finite
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int m = n0 + 32 * j + l32;
        const float b = bias && m < M ? bias[m] : 0.f;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t row = row0 + 32 * i + 8 * (r / 4) + 4 * h + r % 4;
                const float sum = acc[i][j][r] * (1.f / kScale);
                probe = __fmaf_rn(sum, 0.f, probe);
                if (row < N && m < M) Y[row * ldy + m] = bias ? sum + b : sum;
            }
    }
    if (probe == 0.f) return;
    for (int e = 0; e < 64; ++e) {
        const int m = n0 + e / 32 * 32 + l32;
        const int64_t row = row0 + e / 16 % 2 * 32 + e / 4 % 4 * 8 + 4 * h + e % 4;
        if (row >= N || m >= M || is_finite(Y[row * ldy + m])) continue;
        float sum = 0.f;
        for (int c = 0; c < C; ++c) {
            const int k = min((int)idx[row * C + c], K - 1);
            sum += T[((int64_t)c * K + k) * M + m];
        }
        Y[row * ldy + m] = bias ? sum + bias[m] : sum;
    }
}

}  // namespace

hipError_t launch_lookup_matrix_f32(const float* T, const float* bias, int C, int K, int M, const uint8_t* idx, int64_t N,
                                    float* Y, int64_t ldy, hipStream_t s) {
    const int64_t row_tiles = (N + kBM - 1) / kBM, tiles = row_tiles * ((M + kBN - 1) / kBN);
    const int64_t blocks = (tiles + 7) / 8 * 8;
    if (K > 16 || C < kMinCodebooks || blocks > 0x7fffffffLL || row_tiles > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(lookup_matrix_f32_kernel, dim3((unsigned)blocks), dim3(kMfmaThreads), 0, s, T, bias, C, K, M, idx, N, Y,
                       ldy, (int)row_tiles, tiles);
    return hipGetLastError();
}

}  // namespace lutnn
