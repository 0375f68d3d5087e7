// Soft-PQ backward pass (arXiv 2302.03213, Sec. 3.1-3.2, Eq. 5-6) on the fp32 matrix instructions, for sub-vectors
// of eight values and more.  The formulas are those of softpq_backward.hip; per row n and codebook c
//
//   d_k  = sum_v (x_v - P_kv)^2        A_k  = sum_v z_v P'_kv            P' = P - m,  y = x - m
//   s    = softmax_k(-d_k / t)         dz_k = s_k (A_k - sum_j s_j A_j)  e_k = 2 dL/dd_k = -2 dz_k / t
//   dL/dx_v   = -sum_k e_k P'_kv
//   dL/dP_kv  = sum_n (s_k z_v - e_k y_v) + P'_kv sum_n e_k
//
// where m is any vector per codebook: sum_k dz_k = 0, so a common shift of the centroids changes neither dz nor
// dL/dx.  The squared distances stay in the direct form (the expanded one cancels).
//
// Precision.  m is zero, moved into the range of the codebook's centroids coordinate by coordinate: that takes a common
// offset off, and |P'_kv| <= |P_kv| whatever the centroids look like, so that A_k is never rounded more coarsely than
// z . P.  The sums above need sum_k dz_k = 0 exactly: what the rounding of A leaves of it would reach dL/dx times the whole
// of P', which one centroid far from the others makes as large as it likes.  So it is taken off again, s_k of it from
// each dz_k; an error of A_k then reaches dL/dx times (sum_j s_j P_j) - P_k, as it does times x - P_k where the differences
// are formed first.  Against 64-bit gradients that is never worse than such a form, for centroids in one cloud, in
// several, or parked far away, and up to three times better; without either step, m being the centroids' mean, one centroid
// of 16 left 7e-2 of dL/dx wrong at a distance of 1e4.
//
// What bounds it.  Three of the four K x V sums per row are contractions (A over v, dL/dx over k, dL/dP over the
// rows), and done with vector instructions they are seven of the nine operations per (row, k, v) - dL/dP's sum over
// the rows also a 63-step exchange between lanes.  Here they are v_mfma_f32_16x16x4_f32: fp32 products and sums at
// the full fp32 rate, issued beside the vector instructions of another wavefront.  A wavefront owns one codebook for
// a whole chunk of rows and keeps its centroids in registers in the three operand forms; it takes 16 rows at a time
// with lane (q, n) holding centroids 4q .. 4q+3 of row n, which is the layout that the matrix instruction returns A
// in and reads e from; s and e cross the wavefront's private LDS once to become operands of dL/dP.  With K = 8 the
// lanes q = 2, 3 take another 16 rows (H = 2 row blocks at a time): the vector work halves, the matrix work does not.
//
// Measured against the vector form (both with the reduction over the chunks): 8192 rows x 192 codebooks, V = 16: 331 ->
// 102 us (60 us for its bytes at 5 TB/s); 8192 x 96, V = 32: 353 -> 106; 4096 x 48, V = 16: 52 -> 24; 8192 x 384, V = 8:
// 187 -> 136; 50176 x 64, V = 9: 305 -> 155 (of which distances and dL/dP products take about 20 us each when left
// out, staging rows of 36 floats most of the rest).  What precision asks for, the remainder taken off dz and the short
// sums of dL/dP, is 1-7 us of these.  Two steps in flight per wavefront, for latency, cost a
// workgroup of registers and gained nothing.
#include <algorithm>
#include <type_traits>

#include "conv_rows.h"
#include "lutnn_kernels.h"

namespace lutnn {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

constexpr int kCT = 4;  // codebooks per workgroup: one per wavefront

// Workgroups per CU: what the registers (4V of them hold centroids) and the two staged tiles allow.
constexpr int per_cu(int V, int K) { return V <= 9 ? 4 : V == 16 && K == 16 ? 3 : 2; }

// Floats of one codebook's partial sums: K*V, rounded up to whole groups of 64.
constexpr int group_floats(int V, int K) { return (V + 64 / K - 1) / (64 / K) * 64; }

template <int V, int K_T>
struct Soft {
    using E = EncTile<V, kCT>;
    static constexpr int VB = (V + 15) / 16;          // blocks of 16 values
    static constexpr int VQ = (V + 3) / 4;            // blocks of 4 values
    static constexpr int H = 16 / K_T;                // blocks of 16 rows per step
    static constexpr int TS = K_T + 4;                // row stride of the transposition buffers (16-byte aligned)
    static constexpr int TBUF = 16 * H * TS + 16 - K_T;
};

// All-reduce over the lanes that share a row: 16 lanes apart and, with four of them (K = 16), 32 apart.
template <int H, class Op>
__device__ __forceinline__ uint32_t across_q(uint32_t x, Op op) {
    u32x2 r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = op(r.x, r.y);
    if constexpr (H == 2) return x;
    r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return op(r.x, r.y);
}

template <int CTRL>
__device__ __forceinline__ float add_ror(float x) {
    return x + __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), CTRL, 0xf, 0xf, false));
}
// Sum over the 16 lanes of a row, in every lane of it.
__device__ __forceinline__ float sum_row16(float x) {
    x = add_ror<0x128>(x);
    x = add_ror<0x124>(x);
    x = add_ror<0x122>(x);
    return add_ror<0x121>(x);
}

// The wavefront's own LDS operations are performed in order; this keeps the compiler to that order too.
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Copies the tile's 64 rows x 4V columns of A into LDS (zero past N and D).  A thread keeps one column and walks down
// the rows by a constant step, so that one pointer and constant LDS offsets serve all its loads: with an index per
// load the compiler kept dozens of them across the loop over the tiles, and spilled.
template <int V>
__device__ __forceinline__ void stage_rows(const float* __restrict__ A, int64_t ld, int64_t N, int D, int64_t row0,
                                           int c0, float* __restrict__ dst, int vec4, int tid) {
    using E = EncTile<V, kCT>;
    if (vec4) {
        constexpr int Q = E::TW / 4, STEP = kEncThreads / Q, ITER = (kEncRows + STEP - 1) / STEP;
        const int r0 = tid / Q, col = (tid % Q) * 4;
        const bool ok = r0 < STEP && c0 * V + col < D;
        const float* __restrict__ src = A + (row0 + r0) * ld + c0 * V + col;
        float4 val[ITER];
#pragma unroll
        for (int it = 0; it < ITER; ++it) {
            val[it] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (ok && r0 + it * STEP < kEncRows && row0 + r0 + it * STEP < N) val[it] = load_once(src + it * STEP * ld);
        }
        float* __restrict__ to = dst + r0 * E::LS + col;
#pragma unroll
        for (int it = 0; it < ITER; ++it) {
            if (r0 < STEP && r0 + it * STEP < kEncRows) {
                to[it * STEP * E::LS + 0] = val[it].x;
                to[it * STEP * E::LS + 1] = val[it].y;
                to[it * STEP * E::LS + 2] = val[it].z;
                to[it * STEP * E::LS + 3] = val[it].w;
            }
        }
    } else {
        constexpr int STEP = kEncThreads / E::TW;  // 256 / (4V) rows at a time
        const int r0 = tid / E::TW, col = tid % E::TW;
        const bool ok = r0 < STEP && c0 * V + col < D;
#pragma unroll 4
        for (int r = r0; r < kEncRows && r0 < STEP; r += STEP)
            dst[r * E::LS + col] = ok && row0 + r < N ? __builtin_nontemporal_load(A + (row0 + r) * ld + c0 * V + col) : 0.f;
    }
}

// ... and dL/dX back from LDS to memory.
template <int V>
__device__ __forceinline__ void store_rows(const float* __restrict__ src, float* __restrict__ A, int64_t ld, int64_t N,
                                           int D, int64_t row0, int c0, int vec4, int tid) {
    using E = EncTile<V, kCT>;
    if (vec4) {
        constexpr int Q = E::TW / 4, STEP = kEncThreads / Q, ITER = (kEncRows + STEP - 1) / STEP;
        const int r0 = tid / Q, col = (tid % Q) * 4;
        if (r0 >= STEP || c0 * V + col >= D) return;
        float* __restrict__ to = A + (row0 + r0) * ld + c0 * V + col;
        const float* __restrict__ from = src + r0 * E::LS + col;
#pragma unroll
        for (int it = 0; it < ITER; ++it)
            if (r0 + it * STEP < kEncRows && row0 + r0 + it * STEP < N)
                *reinterpret_cast<float4*>(to + it * STEP * ld) =
                    make_float4(from[it * STEP * E::LS], from[it * STEP * E::LS + 1], from[it * STEP * E::LS + 2],
                                from[it * STEP * E::LS + 3]);
    } else {
        constexpr int STEP = kEncThreads / E::TW;
        const int r0 = tid / E::TW, col = tid % E::TW;
        if (r0 >= STEP || c0 * V + col >= D) return;
#pragma unroll 4
        for (int r = r0; r < kEncRows && row0 + r < N; r += STEP) A[(row0 + r) * ld + c0 * V + col] = src[r * E::LS + col];
    }
}

// grid: chunks * col_tiles workgroups, column tile fastest.
//   partial    [chunks][C][group_floats(V, K)], element k*V + v: the sums of the dP contributions over the chunk's rows
//   partial_dt [blocks] one sum of dz_k * d_k per workgroup
//   CONV != 0  X is an NCHW image batch (CONV filter taps, -1 = any filter), Z and dX are [B][D][Ho*Wo] arrays, which
//              may be the same one; a wavefront then stages its own codebook's columns with lane = row
template <int V, int K_T, int CONV>
__global__ __launch_bounds__(kEncThreads, per_cu(V, K_T)) void softpq_matrix_kernel(
    const float* __restrict__ X, int64_t ldx, const float* Z, int64_t ldz, const float* __restrict__ P, float inv_t,
    float* dX, int64_t lddx, float* __restrict__ partial, float* __restrict__ partial_dt, int64_t N, int C,
    int tiles_per_chunk, int blocks, int vec4_x, int vec4_z, int vec4_dx, ConvGeom geom) {
    using S = Soft<V, K_T>;
    using E = typename S::E;
    constexpr int VB = S::VB, VQ = S::VQ, H = S::H, TS = S::TS;
    // the operand reads run up to 15 columns past a codebook's V values
    __shared__ __align__(16) float xs[E::kLdsFloats + 16];
    __shared__ __align__(16) float zs[E::kLdsFloats + 16];
    __shared__ __align__(16) float tr[4][2][S::TBUF];
    __shared__ __align__(16) float shift[4][32];  // m
    __shared__ float dt_s[4];

    // Workgroups go round the eight XCDs; each XCD takes a contiguous run of the work, so that neighbouring column
    // tiles - which share the cache lines at their common edge where 4V floats are no whole number of lines - meet
    // in one L2 (V = 9, 50176 rows x 64 codebooks: 4 % of the time).
    const int block = (int)(blockIdx.x % 8) * (int)(gridDim.x / 8) + (int)(blockIdx.x / 8);
    if (block >= blocks) return;
    const int col_tiles = (C + kCT - 1) / kCT;
    const int chunk = block / col_tiles;
    const int c0 = block % col_tiles * kCT;
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, q = lane >> 4, i16 = lane & 15;
    const int c = c0 + w;  // wave-uniform
    const bool live = c < C;
    const int64_t row_tiles = (N + kEncRows - 1) / kEncRows;
    const int64_t tile_begin = (int64_t)chunk * tiles_per_chunk;
    const int64_t tile_end = std::min<int64_t>(tile_begin + tiles_per_chunk, row_tiles);
    const float inv_t_log2e = inv_t * 1.44269504f;
    const float e_scale = -2.0f * inv_t;

    // ---- this wavefront's centroids, in the form each use wants
    const float* __restrict__ pc = P + (size_t)(live ? c : 0) * K_T * V;
    if (lane < 32) {
        float lo = 0.f, hi = 0.f;
        if (lane < V) {
            lo = hi = pc[lane];
            for (int k = 1; k < K_T; ++k) lo = fminf(lo, pc[k * V + lane]), hi = fmaxf(hi, pc[k * V + lane]);
        }
        shift[w][lane] = lo > 0.f ? lo : hi < 0.f ? hi : 0.f;
    }
    if (tid < 16) xs[E::kLdsFloats + tid] = zs[E::kLdsFloats + tid] = 0.f;
    __syncthreads();
    const int kq = q % (4 / H), hb = q / (4 / H);  // this lane's block of four centroids and of 16 rows
    float p[4][V];        // direct distances: centroids 4kq .. 4kq+3
    float pA[VQ];     // A operand of A_k:   P'[k = i16 % K][4j + q]
    float pT[VB][4];  // A operand of dL/dx: -P'[k = 4kq + j][v = 16b + i16]
    float my[VB];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int v = 0; v < V; ++v) p[r][v] = pc[(4 * kq + r) * V + v];
#pragma unroll
    for (int j = 0; j < VQ; ++j) {
        const int v = 4 * j + q;
        pA[j] = v < V ? pc[i16 % K_T * V + v] - shift[w][v] : 0.f;
    }
#pragma unroll
    for (int b = 0; b < VB; ++b) {
        const int v = 16 * b + i16;
        my[b] = shift[w][v];
#pragma unroll
        for (int j = 0; j < 4; ++j) pT[b][j] = v < V ? my[b] - pc[(4 * kq + j) * V + v] : 0.f;
    }

    f32x4 sum[VB];
#pragma unroll
    for (int b = 0; b < VB; ++b) sum[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    float esum[4] = {0.f, 0.f, 0.f, 0.f};
    float dt_acc = 0.f;
    float* __restrict__ ts = tr[w][0];
    float* __restrict__ te = tr[w][1];

    for (int64_t tile = tile_begin; tile < tile_end; ++tile) {
        const int64_t row0 = tile * kEncRows;
        ConvRow cr;
        if constexpr (CONV != 0) {
            if (live) {
                cr = conv_row(geom, (uint32_t)row0 + lane, (uint32_t)N, C * V);
                float xv[V], zv[V];
                load_patch<V, CONV>(X, geom, cr, c * V, C * V, xv);
                load_columns<V>(Z, geom, cr, c * V, C * V, zv);
#pragma unroll
                for (int v = 0; v < V; ++v) xs[lane * E::LS + w * V + v] = xv[v], zs[lane * E::LS + w * V + v] = zv[v];
                wave_lds_fence();
            }
        } else {
            stage_rows<V>(X, ldx, N, C * V, row0, c0, xs, vec4_x, tid);
            stage_rows<V>(Z, ldz, N, C * V, row0, c0, zs, vec4_z, tid);
            __syncthreads();
        }
        if (live) {
#pragma unroll 1
            for (int g = 0; g < 4; g += H) {
                float* const xg = xs + g * 16 * E::LS + w * V;
                const float* const zg = zs + g * 16 * E::LS + w * V;
                // A_k on the matrix pipe, beside the distances on the vector units.  With K = 8 each row block has a
                // product of its own, so that a value that is not finite stays in its row.
                f32x4 a_of[H];
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    a_of[h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int j = 0; j < VQ; ++j) {
                        float z = zg[(16 * h + i16) * E::LS + 4 * j + q];
                        if (4 * j + 3 >= V && 4 * j + q >= V) z = 0.f;
                        a_of[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(pA[j], z, a_of[h], 0, 0, 0);
                    }
                }
                const f32x4 a = hb == 0 ? a_of[0] : a_of[H - 1];
                const int row = i16 + (H == 1 ? 0 : 16 * hb);  // this lane's row of the step
                float d[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    const float x = xg[row * E::LS + v];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float t = x - p[r][v];
                        d[r] = __fmaf_rn(t, t, d[r]);
                    }
                }
                // distances are not negative: they order like their bit patterns
                const uint32_t m01 = min(__float_as_uint(d[0]), __float_as_uint(d[1]));
                const uint32_t m23 = min(__float_as_uint(d[2]), __float_as_uint(d[3]));
                const float dmin = __uint_as_float(across_q<H>(min(m01, m23), [](uint32_t u, uint32_t v) { return min(u, v); }));
                float s[4], e[4];
                float ssum = 0.f, sa = 0.f;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    s[r] = __builtin_amdgcn_exp2f((dmin - d[r]) * inv_t_log2e);  // exp((dmin - d_k) / t)
                    ssum += s[r];
                    sa = __fmaf_rn(s[r], a[r], sa);
                }
                const auto add = [](uint32_t u, uint32_t v) { return __float_as_uint(__uint_as_float(u) + __uint_as_float(v)); };
                ssum = __uint_as_float(across_q<H>(__float_as_uint(ssum), add));
                sa = __uint_as_float(across_q<H>(__float_as_uint(sa), add));
                float rs = __builtin_amdgcn_rcpf(ssum);  // one Newton step: correct to an ulp or so, a third of a division
                rs = __fmaf_rn(__fmaf_rn(-ssum, rs, 1.0f), rs, rs);
                const float abar = sa * rs;
                float dz[4], dz_sum = 0.f;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    s[r] *= rs;
                    dz[r] = s[r] * (a[r] - abar);
                    dz_sum += dz[r];
                }
                dz_sum = __uint_as_float(across_q<H>(__float_as_uint(dz_sum), add));
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    dz[r] = __fmaf_rn(-s[r], dz_sum, dz[r]);
                    dt_acc = __fmaf_rn(dz[r], d[r], dt_acc);
                    e[r] = dz[r] * e_scale;
                    esum[r] += e[r];
                }
                *reinterpret_cast<f32x4*>(ts + row * TS + 4 * kq) = f32x4{s[0], s[1], s[2], s[3]};
                *reinterpret_cast<f32x4*>(te + row * TS + 4 * kq) = f32x4{e[0], e[1], e[2], e[3]};
                wave_lds_fence();
                // dL/dP: rows 4q + j of a block are contracted in step j (rows K .. of the result are not used).  Each step of
                // 16 rows is summed from zero and added to the running sum, so that no chain is long.
                f32x4 acc_z[VB], acc_y[VB];
#pragma unroll
                for (int b = 0; b < VB; ++b) acc_z[b] = acc_y[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int hj = 0; hj < 4 * H; ++hj) {
                    const int n = hj / 4 * 16 + 4 * q + hj % 4;
                    const float sT = ts[n * TS + i16], eT = te[n * TS + i16];
#pragma unroll
                    for (int b = 0; b < VB; ++b) {
                        const int at = n * E::LS + 16 * b + i16;
                        acc_z[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(sT, zg[at], acc_z[b], 0, 0, 0);
                        acc_y[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(eT, xg[at] - my[b], acc_y[b], 0, 0, 0);
                    }
                }
                if (dX) {
                    wave_lds_fence();
                    // dL/dx takes the place of this wavefront's x values
#pragma unroll
                    for (int hv = 0; hv < H * VB; ++hv) {
                        const int h = hv / VB, b = hv % VB;
                        f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            o = __builtin_amdgcn_mfma_f32_16x16x4f32(pT[b][j], H == 1 || hb == h ? e[j] : 0.f, o, 0, 0, 0);
                        float* const dst = xg + (16 * h + i16) * E::LS + 16 * b + 4 * q;
                        if constexpr (V % 4 == 0) {
                            if (16 * b + 4 * q < V) *reinterpret_cast<f32x4*>(dst) = o;
                        } else {
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                if (16 * b + 4 * q + r < V) dst[r] = o[r];
                        }
                    }
                }
#pragma unroll
                for (int b = 0; b < VB; ++b) sum[b] += acc_z[b] - acc_y[b];
                wave_lds_fence();
            }
        }
        if constexpr (CONV != 0) {
            if (dX && live) store_columns<V>(dX, geom, cr, c * V, C * V, xs + lane * E::LS + w * V);
            wave_lds_fence();
        } else {
            __syncthreads();
            if (dX) store_rows<V>(xs, dX, lddx, N, C * V, row0, c0, vec4_dx, tid);
            __syncthreads();  // the tiles are restaged next
        }
    }

    if (live) {
        float* dst = partial + ((size_t)chunk * C + c) * group_floats(V, K_T);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float es = sum_row16(esum[r]);
            if constexpr (H == 2) es += __shfl_xor(es, 32, 64);
#pragma unroll
            for (int b = 0; b < VB; ++b) {
                const int v = 16 * b + i16;
                if (4 * q + r < K_T && v < V)
                    dst[(4 * q + r) * V + v] = __fmaf_rn(-pT[b][r], es, sum[b][r]);
            }
        }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) dt_acc += __shfl_xor(dt_acc, m, 64);
    if (lane == 0) dt_s[w] = dt_acc;
    __syncthreads();
    if (tid == 0) partial_dt[block] = (dt_s[0] + dt_s[1]) + (dt_s[2] + dt_s[3]);
}

// dP[c][k][v] = sum over chunks of partial[chunk][c][k*V + v]: four wavefronts take a quarter of the chunks each, in
// ascending order, and the quarters are added in ascending order (reproducible run to run; no chain is long).  Block 0 also folds
// the workgroups' temperature sums.
__global__ __launch_bounds__(256) void softpq_chunks_kernel(const float* __restrict__ partial,
                                                            const float* __restrict__ partial_dt, int chunks, int n_dt,
                                                            int C, int KV, int group_floats, float inv_t,
                                                            float* __restrict__ dP, float* __restrict__ dt) {
    __shared__ float part[3][64];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t i = (int64_t)blockIdx.x * 64 + lane;
    const int64_t total = (int64_t)C * KV;
    float sum = 0.f;
    if (i < total) {
        const size_t e = (size_t)(i / KV) * group_floats + i % KV;
        const size_t stride = (size_t)C * group_floats;
        const int per = (chunks + 3) / 4;
        const int end = min(chunks, (w + 1) * per);
        int ch = w * per;
        for (; ch + 8 <= end; ch += 8) {  // eight independent loads, added in pairs
            float t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = partial[(size_t)(ch + u) * stride + e];
            sum += ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
        }
        for (; ch < end; ++ch) sum += partial[(size_t)ch * stride + e];
    }
    if (w > 0) part[w - 1][lane] = sum;
    __syncthreads();
    if (w == 0 && i < total) dP[i] = ((sum + part[0][lane]) + part[1][lane]) + part[2][lane];
    if (dt && blockIdx.x == 0 && w == 0) {
        float ds = 0.f;
        for (int j = lane; j < n_dt; j += 64) ds += partial_dt[j];
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) ds += __shfl_xor(ds, m, 64);
        if (lane == 0) *dt = ds * inv_t * inv_t;
    }
}

struct Plan {
    int chunks, tiles_per_chunk, col_tiles;
};

// As many workgroups as are resident at once, so that no second round runs nearly empty; where the column tiles
// alone nearly fill the chip, four short rounds.  No more chunks than the reduction sums up quickly.
Plan make_plan(int C, int64_t N, int per_cu) {
    Plan p;
    p.col_tiles = (C + kCT - 1) / kCT;
    const int64_t row_tiles = (N + kEncRows - 1) / kEncRows;
    const int64_t resident = (int64_t)256 * per_cu;
    int64_t chunks = p.col_tiles * 4 <= resident ? resident / p.col_tiles : 4 * resident / p.col_tiles;
    chunks = std::max<int64_t>(std::min(std::min<int64_t>(chunks, 256), row_tiles), 1);
    p.tiles_per_chunk = (int)((row_tiles + chunks - 1) / chunks);
    p.chunks = (int)((row_tiles + p.tiles_per_chunk - 1) / p.tiles_per_chunk);
    return p;
}

inline int vec4_ok(const float* A, int64_t ld, int C, int V) {
    return (((int64_t)C * V) % 4 == 0) && (ld % 4 == 0) && ((reinterpret_cast<uintptr_t>(A) & 15) == 0);
}

template <int V, int K_T, int CONV>
hipError_t launch(const SoftPqCall& a, hipStream_t s) {
    const float inv_t = 1.0f / a.t;
    Plan p = {0, 0, 0};
    float *partial = a.workspace, *partial_dt = a.workspace;
    int64_t blocks = 0;
    if (a.N > 0) {
        p = make_plan(a.C, a.N, per_cu(V, K_T));
        blocks = (int64_t)p.chunks * p.col_tiles;
        if (blocks > 0x7ffffff0LL) return hipErrorInvalidValue;
        partial_dt = a.workspace + (size_t)p.chunks * a.C * group_floats(V, K_T);
        hipLaunchKernelGGL((softpq_matrix_kernel<V, K_T, CONV>), dim3((unsigned)(blocks + 7) / 8 * 8), dim3(kEncThreads), 0,
                           s, a.X, a.ldx, a.Z, a.ldz, a.P, inv_t, a.dX, a.lddx, partial, partial_dt, a.N, a.C,
                           p.tiles_per_chunk, (int)blocks, vec4_ok(a.X, a.ldx, a.C, V), vec4_ok(a.Z, a.ldz, a.C, V),
                           a.dX ? vec4_ok(a.dX, a.lddx, a.C, V) : 0, a.geom ? *a.geom : ConvGeom{});
        if (hipError_t e = hipGetLastError()) return e;
    }
    // an empty batch: the reduction over zero chunks writes the zeros
    const int64_t total = (int64_t)a.C * K_T * V;
    hipLaunchKernelGGL(softpq_chunks_kernel, dim3((unsigned)((total + 63) / 64)), dim3(256), 0, s, partial, partial_dt,
                       p.chunks, (int)blocks, a.C, K_T * V, group_floats(V, K_T), inv_t, a.dP, a.dt);
    return hipGetLastError();
}

template <int V, int K_T>
hipError_t launch_source(const SoftPqCall& a, hipStream_t s) {
    if (!a.geom) return launch<V, K_T, 0>(a, s);
    if constexpr (V < 32) {
        const int taps = a.geom->kh * a.geom->kw;
        if (taps == 1) return launch<V, K_T, 1>(a, s);
        if constexpr (V == 9)
            if (taps == 9) return launch<V, K_T, 9>(a, s);
        return launch<V, K_T, -1>(a, s);
    }
    return hipErrorInvalidValue;
}

template <int K_T, class F>
auto by_v(int V, F&& f) {
    if constexpr (K_T == 8) {
        return V == 16 ? f(std::integral_constant<int, 16>{}) : f(std::integral_constant<int, 32>{});
    } else {
        switch (V) {
            case 8: return f(std::integral_constant<int, 8>{});
            case 9: return f(std::integral_constant<int, 9>{});
            case 16: return f(std::integral_constant<int, 16>{});
            default: return f(std::integral_constant<int, 32>{});
        }
    }
}

}  // namespace

// Below eight values a 16-row operand is mostly padding, and with K = 8 half of it is: there the vector form
// (softpq_backward.hip) is as fast or faster (K = 8, V = 9, 50176 rows x 64 codebooks: 129 us against 136).
bool softpq_matrix_preferred(int K, int V) { return V >= 16 || (V >= 8 && K == 16); }

size_t softpq_matrix_workspace_bytes(int C, int K, int V, int64_t N) {
    const Plan p = make_plan(C, N, per_cu(V, K));
    return ((size_t)p.chunks * C * group_floats(V, K) + (size_t)p.chunks * p.col_tiles) * sizeof(float);
}

hipError_t launch_softpq_matrix(const SoftPqCall& a, hipStream_t s) {
    if (a.K == 16) return by_v<16>(a.V, [&](auto v) { return launch_source<decltype(v)::value, 16>(a, s); });
    return by_v<8>(a.V, [&](auto v) { return launch_source<decltype(v)::value, 8>(a, s); });
}

}  // namespace lutnn
