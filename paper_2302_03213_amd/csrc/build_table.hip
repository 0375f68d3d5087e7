// Offline table construction (arXiv 2302.03213, Eq. 3) and symmetric INT8 scalar quantisation of the
// table (Sec. 3.3) for gfx950.  Offline for inference, but training rebuilds the table from the
// updated centroids in every forward pass (Sec. 3.1), so it is kept to two passes over the table:
// max |T|, then quantise and write both layouts.  No workspace - each pass recomputes the fp32
// entry (V fused multiply-adds) instead of storing it.  Grids are (column block, codebook x
// centroid) so that no thread divides.
//
//   T[c][k][m] = sum_v P[c][k][v] * W[cV+v][m]          fp32, v ascending, one fma per term
//   s = max|T| / 127 (1 if the table is all zero),  q = clamp(rint(T / s), -127, 127)
//   INT4 (n = 4 in the same formula): 7 in place of 127, two entries per byte.
#include <algorithm>

#include "lutnn_kernels.h"

namespace lutnn {
namespace {

constexpr int kThreads = 256;

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float table_entry(const float* __restrict__ P,
                                             const float* __restrict__ W, int64_t ldw, int K, int V,
                                             int c, int k, int m) {
    const float* p = P + ((size_t)c * K + k) * V;
    const float* w = W + (size_t)c * V * ldw + m;
    float acc = 0.f;
    for (int v = 0; v < V; ++v) acc = __fmaf_rn(p[v], w[(size_t)v * ldw], acc);
    return acc;
}

// qmax = 2^(n-1) - 1: 127 for INT8, 7 for INT4.
__device__ __forceinline__ float quantise(float t, float s, float qmax) {
    float r = rintf(__fdiv_rn(t, s));  // IEEE division, round half to even
    r = fminf(fmaxf(r, -qmax), qmax);
    return r;
}

__device__ __forceinline__ float scale_from_amax(float amax, float qmax) {
    return amax == 0.f ? 1.f : __fdiv_rn(amax, qmax);
}

// *scale holds max|T| with the sign bit set while the table is built and the positive scale afterwards, so that the
// last kernel can replace the one by the other while its other workgroups still read it: either gives them the scale.
constexpr uint32_t kAmaxMark = 0x80000000u;
__device__ __forceinline__ float read_scale(const uint32_t* scale, float qmax) {
    const uint32_t v = __atomic_load_n(scale, __ATOMIC_RELAXED);
    return v & kAmaxMark ? scale_from_amax(__uint_as_float(v & ~kAmaxMark), qmax) : __uint_as_float(v);
}
__device__ __forceinline__ void finish_scale(uint32_t* scale, float s) {
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) __atomic_store_n(scale, __float_as_uint(s), __ATOMIC_RELAXED);
}

__global__ void fill_u32_kernel(uint32_t* p, uint32_t v) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *p = v;
}

// A thread's share of a codebook: CPT neighbouring columns of it, whose V weights it loads once and uses for all K
// centroids (scalar operands).  V_T = 0: V is a run-time value; one column, whose weights come one after another, each for
// all 16 centroids of a block (read again for every centroid, 64 codebooks x 1000 columns of fp32, V = 64, took 103 us;
// this way 17, and 41 with a thread per entry).
template <int V_T, int CPT>
struct Columns {
    float w[V_T ? V_T : 16][CPT];  // V_T = 0: the 16 sums

    __device__ __forceinline__ void load(const float* __restrict__ P, const float* __restrict__ W, int64_t ldw, int K, int V,
                                         int c, int kb, int m, int M) {
        if constexpr (V_T == 0) {
#pragma unroll
            for (int k = 0; k < 16; ++k) w[k][0] = 0.f;
            const float* __restrict__ src = W + (size_t)c * V * ldw + (m < M ? m : 0);  // past the last column the first again
            const float* __restrict__ p = P + (size_t)c * K * V;
#pragma unroll 2
            for (int v = 0; v < V; ++v) {
                const float weight = src[(size_t)v * ldw];
#pragma unroll
                for (int k = 0; k < 16; ++k) w[k][0] = __fmaf_rn(p[(size_t)min(kb * 16 + k, K - 1) * V + v], weight, w[k][0]);
            }
        } else {
            const float* __restrict__ src = W + (size_t)c * V_T * ldw + m;
#pragma unroll
            for (int v = 0; v < V_T; ++v) {
                if constexpr (CPT == 4) {
                    const f32x4 q = m < M ? *reinterpret_cast<const f32x4*>(src + (size_t)v * ldw) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int j = 0; j < 4; ++j) w[v][j] = q[j];
                } else {
                    w[v][0] = m < M ? src[(size_t)v * ldw] : 0.f;
                }
            }
        }
    }
    // T[c][16 kb + kk][m + j] of every column, v ascending, one fma per term
    __device__ __forceinline__ void entries(const float* __restrict__ P, int K, int c, int kb, int kk, float (&t)[CPT]) const {
        if constexpr (V_T != 0) {
            const float* __restrict__ p = P + ((size_t)c * K + kb * 16 + kk) * V_T;
#pragma unroll
            for (int j = 0; j < CPT; ++j) t[j] = 0.f;
#pragma unroll
            for (int v = 0; v < V_T; ++v)
#pragma unroll
                for (int j = 0; j < CPT; ++j) t[j] = __fmaf_rn(p[v], w[v][j], t[j]);
        } else {
            t[0] = w[kk][0];
        }
    }
};

// max |T| over the layer.  Floats without their sign order like their bit patterns, so the running maximum is kept with
// an integer atomicMax on the bits of *amax_bits.  A thread owns (c, block of 16 centroids, CPT columns), like the
// quantising pass below.  A wavefront issues its atomic only when its value exceeds the maximum it can see (a
// stale, smaller reading costs an unnecessary atomic, never a missed one): tens of thousands of atomics on one
// address would take longer than the arithmetic.
// grid: blockIdx.x = c*Kb + kb, blockIdx.y = block of blockDim.x * CPT columns.
template <int V_T, int CPT>
__global__ __launch_bounds__(kThreads) void table_amax_kernel(const float* __restrict__ P,
                                                              const float* __restrict__ W, int64_t ldw, int K,
                                                              int V, int M, int Kb, uint32_t* amax_bits) {
    const int m = (blockIdx.y * blockDim.x + threadIdx.x) * CPT;
    const int c = blockIdx.x / Kb, kb = blockIdx.x % Kb;
    Columns<V_T, CPT> col;
    col.load(P, W, ldw, K, V, c, kb, m, M);
    float a = 0.f;
    const int k_end = min(16, K - kb * 16);
#pragma unroll V_T ? 4 : 16
    for (int kk = 0; kk < (V_T ? k_end : 16); ++kk) {
        if (V_T == 0 && kk >= k_end) continue;
        float t[CPT];
        col.entries(P, K, c, kb, kk, t);
#pragma unroll
        for (int j = 0; j < CPT; ++j) a = fmaxf(a, fabsf(t[j]));
    }
    for (int off = 32; off > 0; off >>= 1) a = fmaxf(a, __shfl_xor(a, off));
    if ((threadIdx.x & 63) == 0) {
        const uint32_t mine = __float_as_uint(a) | kAmaxMark;
        if (mine > __atomic_load_n(amax_bits, __ATOMIC_RELAXED)) atomicMax(amax_bits, mine);
    }
}

// INT8: quantises and writes both layouts in one pass.  The 16 codes of a column are the 16 bytes of
// packed[(c*Kb + kb)][m][0..15] (zero where k >= K or m >= M); CPT neighbouring columns of a centroid are one store
// into row T[c][k] (four bytes with CPT = 4).  The last pass over *scale: it becomes the scale here.
// grid: blockIdx.x = c*Kb + kb, blockIdx.y = block of blockDim.x * CPT columns of the padded width Mp.
template <int V_T, int CPT>
__global__ __launch_bounds__(kThreads) void table_quant_pack_kernel(
    const float* __restrict__ P, const float* __restrict__ W, int64_t ldw, int K, int V, int M, int Mp,
    int Kb, uint32_t* scale, int8_t* __restrict__ T, uint4* __restrict__ packed) {
    const int m = (blockIdx.y * blockDim.x + threadIdx.x) * CPT;
    const int c = blockIdx.x / Kb, kb = blockIdx.x % Kb;
    const float s = read_scale(scale, 127.f);
    finish_scale(scale, s);
    if (m >= Mp) return;
    Columns<V_T, CPT> col;
    col.load(P, W, ldw, K, V, c, kb, m, M);
    uint32_t w[CPT][4];
#pragma unroll
    for (int j = 0; j < CPT; ++j) w[j][0] = w[j][1] = w[j][2] = w[j][3] = 0u;
#pragma unroll
    for (int kq = 0; kq < 4; ++kq) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const int k = kb * 16 + 4 * kq + kk;
            if (k >= K || m >= M) break;
            float t[CPT];
            col.entries(P, K, c, kb, 4 * kq + kk, t);
            uint32_t row = 0;
#pragma unroll
            for (int j = 0; j < CPT; ++j) {
                const uint32_t q = (uint32_t)(int)quantise(t[j], s, 127.f) & 0xffu;
                w[j][kq] |= q << (8 * kk);
                row |= q << (8 * j);
            }
            int8_t* dst = T + ((size_t)c * K + k) * M + m;
            if constexpr (CPT == 4) *reinterpret_cast<uint32_t*>(dst) = row; else *dst = (int8_t)row;
        }
    }
    if (packed) {
#pragma unroll
        for (int j = 0; j < CPT; ++j) packed[(size_t)blockIdx.x * Mp + m + j] = make_uint4(w[j][0], w[j][1], w[j][2], w[j][3]);
    }
}

// fp32 tables: the same shares, stored as they are.  Grid as table_amax_kernel.
template <int V_T, int CPT>
__global__ __launch_bounds__(kThreads) void table_f32_kernel(const float* __restrict__ P,
                                                             const float* __restrict__ W, int64_t ldw, int K,
                                                             int V, int M, int Kb, float* __restrict__ T) {
    const int m = (blockIdx.y * blockDim.x + threadIdx.x) * CPT;
    if (m >= M) return;
    const int c = blockIdx.x / Kb, kb = blockIdx.x % Kb;
    Columns<V_T, CPT> col;
    col.load(P, W, ldw, K, V, c, kb, m, M);
    const int k_end = min(16, K - kb * 16);
#pragma unroll V_T ? 4 : 16
    for (int kk = 0; kk < (V_T ? k_end : 16); ++kk) {
        if (V_T == 0 && kk >= k_end) continue;
        float t[CPT];
        col.entries(P, K, c, kb, kk, t);
        float* dst = T + ((size_t)c * K + kb * 16 + kk) * M + m;
        if constexpr (CPT == 4) *reinterpret_cast<f32x4*>(dst) = f32x4{t[0], t[1], t[2], t[3]}; else *dst = t[0];
    }
}

// INT4 storage: byte j of row (c, k) holds columns 2j (low nibble) and 2j+1 (high nibble, 0 past M).
// grid: blockIdx.x = c*K + k, blockIdx.y = block of 256 bytes.
__global__ __launch_bounds__(kThreads) void table_quant_i4_kernel(
    const float* __restrict__ P, const float* __restrict__ W, int64_t ldw, int K, int V, int M,
    uint32_t* scale, int finish, uint8_t* __restrict__ T) {
    const float s = read_scale(scale, 7.f);
    if (finish) finish_scale(scale, s);
    const int Mb = (M + 1) / 2;
    const int j = blockIdx.y * kThreads + threadIdx.x;
    if (j >= Mb) return;
    const int c = blockIdx.x / K, k = blockIdx.x % K;
    const int lo = (int)quantise(table_entry(P, W, ldw, K, V, c, k, 2 * j), s, 7.f);
    const int hi = 2 * j + 1 < M ? (int)quantise(table_entry(P, W, ldw, K, V, c, k, 2 * j + 1), s, 7.f) : 0;
    T[(size_t)blockIdx.x * Mb + j] = (uint8_t)((lo & 0xf) | ((hi & 0xf) << 4));
}

// MFMA operand copy alone (INT4 tables, whose T has its own layout):
// packed[(c*Kb + kb)][m][kk] = q[c][16*kb + kk][m], zero where k >= K or m >= M.
// grid as table_quant_pack_kernel.
__global__ __launch_bounds__(kThreads) void table_pack_kernel(const float* __restrict__ P,
                                                              const float* __restrict__ W, int64_t ldw, int K,
                                                              int V, int M, int Mp, int Kb,
                                                              uint32_t* scale, float qmax,
                                                              uint4* __restrict__ packed) {
    const float s = read_scale(scale, qmax);
    finish_scale(scale, s);
    const int m = blockIdx.y * kThreads + threadIdx.x;
    if (m >= Mp) return;
    const int c = blockIdx.x / Kb, kb = blockIdx.x % Kb;
    uint32_t w[4] = {0u, 0u, 0u, 0u};
    if (m < M) {
        for (int kk = 0; kk < 16; ++kk) {
            const int k = kb * 16 + kk;
            if (k >= K) break;
            const int q = (int)quantise(table_entry(P, W, ldw, K, V, c, k, m), s, qmax);
            w[kk >> 2] |= (uint32_t)(q & 0xff) << (8 * (kk & 3));
        }
    }
    packed[(size_t)blockIdx.x * Mp + m] = make_uint4(w[0], w[1], w[2], w[3]);
}

inline unsigned col_blocks(int64_t cols) { return (unsigned)((cols + kThreads - 1) / kThreads); }

// What a call builds, for the launchers below.
struct Tables {
    const float *P, *W;
    int64_t ldw;
    int C, K, V, M;
    float* f32;        // the fp32 table, or
    int8_t *T, *packed;
    uint32_t* scale;   // max |T| goes here,
    bool quant;        // ... and the INT8 table and its packed copy to T and packed
};

// Four columns per thread where rows of W (and of an fp32 table) can be moved 16 bytes at a time and there are columns
// enough to fill the chip's workgroups that way (from 1024 on); wavefronts of their own below, so that a narrow layer
// (64 columns) still spreads its codebooks over the CUs.  A call's three launches at 48 codebooks x 3072 columns, V
// = 16: 64.5 -> 26 us (the weights were read once per centroid, a byte stored at a time); 1024 x 4096, V = 4: 221 -> 88;
// 64 x 64, V = 9: 29 -> 18.
template <int V_T, int CPT>
hipError_t launch_columns(const Tables& t, hipStream_t s) {
    const int Kb = kblocks(t.K), Mp = (int)packed_cols(t.M);
    // the grid's second dimension stops at 65535
    const int threads = (CPT == 4 && t.M >= 4096) || Mp > 64 * 65535 ? kThreads : 64;
    const auto grid = [&](int cols) {
        return dim3((unsigned)t.C * Kb, (unsigned)((cols + threads * CPT - 1) / (threads * CPT)));
    };
    if (t.f32) {
        hipLaunchKernelGGL((table_f32_kernel<V_T, CPT>), grid(t.M), dim3(threads), 0, s, t.P, t.W, t.ldw, t.K, t.V, t.M, Kb,
                           t.f32);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((table_amax_kernel<V_T, CPT>), grid(t.M), dim3(threads), 0, s, t.P, t.W, t.ldw, t.K, t.V, t.M, Kb,
                       t.scale);
    if (t.quant)  // without a packed copy only the M real columns need threads
        hipLaunchKernelGGL((table_quant_pack_kernel<V_T, CPT>), grid(t.packed ? Mp : t.M), dim3(threads), 0, s, t.P, t.W,
                           t.ldw, t.K, t.V, t.M, Mp, Kb, t.scale, t.T, reinterpret_cast<uint4*>(t.packed));
    return hipGetLastError();
}

template <int V_T>
hipError_t launch_columns_v(const Tables& t, hipStream_t s) {
    if constexpr (V_T != 0) {
        const bool four = t.M % 4 == 0 && t.M >= 1024 && t.ldw % 4 == 0 && (reinterpret_cast<uintptr_t>(t.W) & 15) == 0 &&
                          (reinterpret_cast<uintptr_t>(t.T) & 3) == 0 && (reinterpret_cast<uintptr_t>(t.f32) & 15) == 0;
        if (four) return launch_columns<V_T, 4>(t, s);
    }
    return launch_columns<V_T, 1>(t, s);
}

hipError_t launch_tables(const Tables& t, hipStream_t s) {
    switch (t.V) {
        case 1: return launch_columns_v<1>(t, s);
        case 2: return launch_columns_v<2>(t, s);
        case 4: return launch_columns_v<4>(t, s);
        case 8: return launch_columns_v<8>(t, s);
        case 9: return launch_columns_v<9>(t, s);
        case 16: return launch_columns_v<16>(t, s);
        case 32: return launch_columns_v<32>(t, s);
        default: return launch_columns_v<0>(t, s);
    }
}

}  // namespace

// Callers guarantee C*K < 2^31 (grid.x) and M <= 2^24 - 512: padded to the packed width, up to 65535 blocks of 256 columns
// (grid.y).
hipError_t launch_build_table_f32(const float* P, const float* W, int64_t ldw, int C, int K, int V,
                                  int M, float* T, hipStream_t s) {
    return launch_tables(Tables{P, W, ldw, C, K, V, M, T, nullptr, nullptr, nullptr, false}, s);
}

hipError_t launch_build_table_i8(const float* P, const float* W, int64_t ldw, int C, int K, int V,
                                 int M, int8_t* T, int8_t* packed, float* scale, int bits,
                                 hipStream_t s) {
    const float qmax = bits == 4 ? 7.f : 127.f;
    const int Kb = kblocks(K);
    const int Mp = (int)packed_cols(M);
    uint32_t* bits_of_scale = reinterpret_cast<uint32_t*>(scale);
    hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(64), 0, s, bits_of_scale, kAmaxMark);
    const bool i8 = bits == 8;
    const hipError_t e = launch_tables(Tables{P, W, ldw, C, K, V, M, nullptr, T, packed, bits_of_scale, i8}, s);
    if (e != hipSuccess || i8) return e;
    hipLaunchKernelGGL(table_quant_i4_kernel, dim3((unsigned)C * K, col_blocks((M + 1) / 2)), dim3(kThreads), 0, s, P, W,
                       ldw, K, V, M, bits_of_scale, packed ? 0 : 1, reinterpret_cast<uint8_t*>(T));
    if (packed)
        hipLaunchKernelGGL(table_pack_kernel, dim3((unsigned)C * Kb, col_blocks(Mp)), dim3(kThreads), 0, s, P, W, ldw, K, V,
                           M, Mp, Kb, bits_of_scale, qmax, reinterpret_cast<uint4*>(packed));
    return hipGetLastError();
}

}  // namespace lutnn
