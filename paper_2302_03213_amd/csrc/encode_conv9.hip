// Encoding of a 3x3 convolution (arXiv 2302.03213, Eq. 2 with V = 9, Sec. 6.1) with the matrix cores as a filter, for
// gfx950.  The result is that of encode.hip bit for bit:
//
//   idx[n][c] = argmin_k sum_v (X[n][cV+v] - P[c][k][v])^2      fp32, v ascending, one fma per term, lowest k on ties
//
// but the K distances are computed that way for few rows only.  For all rows the matrix cores give
// score_k = |P_k|^2 - 2 x.P_k, to about 18 bits; where the best score is ahead of the second by more than both forms'
// errors can be, its k is the arg-min of the direct form too, and where it is not (one sub-vector in a few thousand
// on random data) the wavefront searches that row directly - all its rows where they are many, and then without the
// filter for the rest of its chunk.
//
// What bounds it.  A convolution's activations arrive nine times faster than its rows are searched: the direct search is
// 334 vector instructions per 64 sub-vectors, half of them with a scalar operand at twice the price, and all of the
// time.  Here it is about 100, and four matrix instructions.  (For rows read from a matrix the same filter gained
// 10-20 % at V = 8 and 16 and lost at V = 2, 4 and 32: there the read of X bounds the search already, or the
// split into parts and the exchange between lanes are as long as the search.)
//
// Mapping.  v_mfma_f32_16x16x32_f16: 16 centroids x 32 products x 16 rows.  x and -2 P are split into fp16 high and low
// parts; the lane groups q = 0, 1, 2 hold high.high, high.low and low.high of the first eight taps, q = 3 the three
// products of the ninth, so that a lane reads eight consecutive fp16 from LDS.  |P_k|^2 is the accumulator's start.
// Lane (q, n) receives the scores of centroids 4q .. 4q+3 for row n; they carry k in their four lowest bits from there
// on, so that the smallest needs no search for its index, and two exchanges between lanes (v_permlane32_swap,
// v_permlane16_swap) merge the four groups of 16 rows into lane = row.
// A wavefront keeps four codebooks' operands in registers for a chunk of pixel tiles, and loads the next tile's band of
// input rows while it works on this one.
//
// Error bound.  With x = xh + xl + rx (|rx| <= 2^-22 |x| + 2^-25 for values that fp16's range covers), the same for
// -2p, and pn = max |P_k|^2, a score is off by at most
//   products   rx, rp and low.low, which is left out: 3 * 2^-22 * 2 sqrt(pn) |x| + 2^-24 (sum |2p_v| + sum |x_v|)
//   sums       2^-20 of the largest magnitude, pn + 2 sqrt(pn) |x| (32 addends cut at 2^-26 of it, the result at 2^-23)
//   |P_k|^2    itself rounded: (V + 1) 2^-24 pn
//   index bits 2^-19 of the score
// and the direct form by (V + 2) 2^-24 d_k, d_k = score + |x|^2.  Summed for the two scores that are compared, and
// doubled for good measure, this is  tx |x| + t2 |x|^2 + t0 + tm (|m1| + |m2|)  with tx and t0 per codebook.
// Sub-vectors with |x|^2 > 2^28 (the parts may overflow), and codebooks whose largest value lies outside 2^-10 .. 2^12 or
// that hold a value that is not finite, are not filtered.
#include <algorithm>

#include "encode_tile.h"
#include "lutnn_kernels.h"

namespace lutnn {
namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int kRowBytes = 48;  // of a row in the operand buffer: 32 used (48 with V = 9), conflict-free for 16-byte reads

constexpr int kV = 9, kCT = 16, kCPW = 4;
constexpr int kFewRows = 16;

struct Threshold {  // wave-uniform
    float tx, t0;
    bool filter;
};
constexpr float kUnit = 1.f / (1 << 24);
constexpr float kT2 = 4.f * (kV + 2) * 2 * kUnit, kTm = 4.f * (32 + kV + 2) * kUnit;

__device__ __forceinline__ float uniform(float x) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(x)));
}

__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// One codebook's operands: a the centroids' parts, norm the four |P_k|^2 of this lane.
template <int K_T>
__device__ __forceinline__ void load_codebook(const float* __restrict__ pc, int lane, f16x8& a, f32x4& norm, Threshold& t) {
    const int q = lane >> 4, k = lane & 15;
    const bool in_k = k < K_T;
    float p[kV];
    float nn = 0.f, pm = 0.f;
#pragma unroll
    for (int v = 0; v < kV; ++v) {
        p[v] = pc[(in_k ? k : 0) * kV + v];
        nn = __fmaf_rn(p[v], p[v], nn);
        pm = fmaxf(pm, fabsf(p[v]));
    }
    if (!(nn <= 3.0e38f)) pm = __builtin_inff();  // a maximum passes NaN by
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const float x = q == 3 ? (j < 3 ? -2.f * p[8] : 0.f) : -2.f * p[j];  // high, low, high of the ninth
        const _Float16 hi = (_Float16)x;
        const _Float16 lo = (_Float16)(x - (float)hi);
        a[j] = !in_k ? (_Float16)0.f : (q == 1 || (q == 3 && j == 1)) ? lo : hi;
    }
    float pn = nn;
#pragma unroll
    for (int m = 8; m >= 1; m >>= 1) {
        pn = fmaxf(pn, __shfl_xor(pn, m, 64));
        pm = fmaxf(pm, __shfl_xor(pm, m, 64));
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) norm[r] = 4 * q + r < K_T ? __shfl(nn, 4 * q + r, 64) : 3.0e38f;
    pn = uniform(pn);
    pm = uniform(pm);
    const float root = __builtin_sqrtf(pn);
    t.tx = 4.f * ((3.f * 4.f * 2.f + 16.f * 2.f) * kUnit * root + 3.f * kUnit);
    t.t0 = 4.f * ((16.f + kV + 1) * kUnit * pn + 2.f * kV * kUnit * pm);
    t.filter = pm >= 1.f / 1024 && pm <= 4096.f;
}

__device__ __forceinline__ float med3(float a, float b, float c) { return __builtin_amdgcn_fmed3f(a, b, c); }
__device__ __forceinline__ float fmin2(float a, float b) {  // v_min_f32 without the quieting of NaN that fminf asks for
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float fmin3(float a, float b, float c) {
    float r;
    asm("v_min3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

struct Top2 {
    float m1, m2;
};
__device__ __forceinline__ Top2 merge(const Top2& a, const Top2& b) {
    // the second smallest of two sorted pairs: the larger head or one of the tails
    float h;
    asm("v_max_f32 %0, %1, %2" : "=v"(h) : "v"(a.m1), "v"(b.m1));
    return {fmin2(a.m1, b.m1), fmin3(h, a.m2, b.m2)};
}
template <bool By32>
__device__ __forceinline__ Top2 exchange_merge(Top2 a, Top2 b) {
    u32x2 r1, r2;
    if constexpr (By32) {
        r1 = __builtin_amdgcn_permlane32_swap(__float_as_uint(a.m1), __float_as_uint(b.m1), false, false);
        r2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(a.m2), __float_as_uint(b.m2), false, false);
    } else {
        r1 = __builtin_amdgcn_permlane16_swap(__float_as_uint(a.m1), __float_as_uint(b.m1), false, false);
        r2 = __builtin_amdgcn_permlane16_swap(__float_as_uint(a.m2), __float_as_uint(b.m2), false, false);
    }
    return merge({__uint_as_float(r1.x), __uint_as_float(r2.x)}, {__uint_as_float(r1.y), __uint_as_float(r2.y)});
}

// Splits this lane's nine values and puts the parts into the wavefront's operand buffer.
__device__ __forceinline__ void store_parts(const float (&x)[kV], char* __restrict__ row) {
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    uint32_t hi[5], lo[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const f32x2 v = {x[2 * i], i < 4 ? x[2 * i + 1] : 0.f};
        const f16x2 h = __builtin_convertvector(v, f16x2);
        hi[i] = __builtin_bit_cast(uint32_t, h);
        f32x2 r = {0.f, 0.f};  // v - h, the half read where it is
        asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r[0]) : "v"(hi[i]), "v"(v[0]));
        if (i < 4) asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r[1]) : "v"(hi[i]), "v"(v[1]));
        lo[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, f16x2));
    }
    *reinterpret_cast<u32x4*>(row) = u32x4{hi[0], hi[1], hi[2], hi[3]};
    *reinterpret_cast<u32x4*>(row + 16) = u32x4{lo[0], lo[1], lo[2], lo[3]};
    *reinterpret_cast<u32x4*>(row + 32) = u32x4{hi[4] | hi[4] << 16, lo[4], 0u, 0u};
}

// The best centroid of 64 rows (lane = row) from the accumulated scores of their four groups, and whether this lane's
// lead is too small to be sure of.
__device__ __forceinline__ uint32_t best_of(const f32x4 (&d)[4], uint32_t k0, float xx, const Threshold& t, bool& unsure) {
    Top2 top[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        float s[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) s[r] = __uint_as_float((__float_as_uint(d[g][r]) & ~15u) | (k0 + r));
        const float m2 = med3(s[0], s[1], s[2]), m1 = fmin3(s[0], s[1], s[2]);
        top[g] = {fmin2(m1, s[3]), med3(m1, m2, s[3])};
    }
    const Top2 a = exchange_merge<true>(top[0], top[2]), b = exchange_merge<true>(top[1], top[3]);
    const Top2 m = exchange_merge<false>(a, b);
    const float need = __fmaf_rn(kTm, fabsf(m.m1) + fabsf(m.m2),
                                 __fmaf_rn(t.tx, __builtin_amdgcn_sqrtf(xx), __fmaf_rn(kT2, xx, t.t0)));
    unsure = !(m.m2 - m.m1 > need) || !(xx <= 268435456.f);
    return __float_as_uint(m.m1) & 15u;
}

// The band of input rows that 64 consecutive output pixels of one image touch (encode.hip's band kernel).  In LDS a
// channel's band is contiguous; a wavefront moves it 64 floats at a time, element e = 64 i + lane being band row
// e / ncols, column e % ncols.
struct Band {
    int64_t image;  // offset of the image's first channel
    int p0, p1, ho0, h_lo, w_lo, nrows, ncols;
};

__device__ __forceinline__ Band band_of(const ConvGeom& g, int b, int pt) {  // image, pixel tile
    Band t;
    const int pix = g.Ho * g.Wo;
    t.image = (int64_t)b * g.Cin * g.H * g.W;
    t.p0 = pt * kEncRows;
    t.p1 = min(t.p0 + kEncRows - 1, pix - 1);
    t.ho0 = t.p0 / g.Wo;
    const int ho1 = t.p1 / g.Wo;
    t.h_lo = t.ho0 * g.sh - g.ph;
    t.nrows = (ho1 - t.ho0) * g.sh + g.kh;
    const bool one_row = t.ho0 == ho1;
    t.w_lo = one_row ? (t.p0 - t.ho0 * g.Wo) * g.sw - g.pw : -g.pw;
    t.ncols = one_row ? (t.p1 - t.p0) * g.sw + g.kw : (g.Wo - 1) * g.sw + g.kw;
    return t;
}

// e / n for small e: the half keeps the product half a quotient step from any integer, far above its rounding while
// e < 2^20.
__device__ __forceinline__ int small_quotient(int e, float recip_n) { return (int)(((float)e + 0.5f) * recip_n); }

// Where this lane's elements of a band lie: row and column, found again only when the band's width changes.
template <int NI>
struct Elements {
    int ncols;
    int at[NI];  // row << 16 | column
    __device__ __forceinline__ void set(int n, int lane) {
        ncols = n;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int row = small_quotient(64 * i + lane, 1.f / n);
            at[i] = row << 16 | (64 * i + lane - row * n);
        }
    }
};

// A wavefront's four channels of the band into registers, zero outside the image and past C: an offset beyond the
// resource makes the load return zero.
template <int NI>
__device__ __forceinline__ void load_band(const float* __restrict__ input, const ConvGeom& g, const Band& t, int channel,
                                          int C, const Elements<NI>& el, float (&val)[kCPW][NI]) {
    const int HW = g.H * g.W;
    // the resource covers the wavefront's channels (fewer at the end of the layer)
    const int64_t first = t.image + (int64_t)channel * HW;
    const int64_t bytes = (int64_t)max(0, min(kCPW, C - channel)) * HW * 4;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(input) + (bytes ? first : 0), 0,
                                                        (uint32_t)bytes, 0x00020000);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int row = el.at[i] >> 16, hi = t.h_lo + row, wi = t.w_lo + (el.at[i] & 0xffff);
        const bool in = (unsigned)hi < (unsigned)g.H && (unsigned)wi < (unsigned)g.W && row < t.nrows;
        const uint32_t off = in ? 4u * (uint32_t)(hi * g.W + wi) : 0xc0000000u;
#pragma unroll
        for (int j = 0; j < kCPW; ++j)
            val[j][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, off + 4u * (uint32_t)(j * HW), 0, 0));
    }
}

template <int CTRL>
__device__ __forceinline__ uint32_t min_ror(uint32_t x) {
    return min(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, false));
}

// The direct search for the rows of `rows` (lanes), four at a time: 16 lanes take a row, one centroid each.  Up to kFewRows
// rows; more of them cost less in the form of encode.hip, lane = row (all 64 rows this way: 3 to 4.5 times the direct
// kernel's time, for data or centroids that the filter can do nothing with).  `taps`
// points at the codebook's channel in LDS, `base` is each lane's patch in it, toff the taps; returns `best` with
// those lanes' bits replaced.
template <int K_T>
__device__ __forceinline__ uint32_t search_rows(uint64_t rows, uint32_t best, const float* __restrict__ taps, int base,
                                                const int (&toff)[kV], const float* __restrict__ pc, int lane) {
    const int q = lane >> 4, k = lane & 15;
    float p[kV];
#pragma unroll
    for (int v = 0; v < kV; ++v) p[v] = pc[min(k, K_T - 1) * kV + v];
    while (rows) {
        int mine = 0, r[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {  // the next four rows (the last one again where there are fewer)
            r[i] = rows ? __builtin_ctzll(rows) : r[i ? i - 1 : 0];
            rows &= rows - 1;
            if (q == i) mine = r[i];
            if (!rows) rows = 0;
        }
        const int at = __shfl(base, mine, 64);
        float d = 0.f;
#pragma unroll
        for (int v = 0; v < kV; ++v) {
            const float t = taps[at + toff[v]] - p[v];
            d = __fmaf_rn(t, t, d);
        }
        // not negative: ordered like its bits, NaN being the largest - but in centroid 0, where the direct search starts
        // and which nothing is below then
        const uint32_t bits = k >= K_T ? 0xffffffffu : k == 0 && d != d ? 0u : __float_as_uint(d);
        const uint32_t least = min_ror<0x121>(min_ror<0x122>(min_ror<0x124>(min_ror<0x128>(bits))));
        const uint64_t hit = __ballot(bits == least);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t win = (uint32_t)__builtin_ctz((uint32_t)(hit >> (16 * i)) & 0xffffu);
            if (lane == r[i]) best = win;
        }
    }
    return best;
}

// grid: chunks * col_tiles workgroups, column tile fastest; a chunk is a run of pixel tiles.
//   NI  64-float pieces of a channel's largest band
template <int K_T, int NI>
__global__ __launch_bounds__(kEncThreads, NI > 5 ? 3 : 4) void encode_conv9_filter_kernel(const float* __restrict__ input,
                                                                             const float* __restrict__ P,
                                                                             const IndexRows idx, int C, ConvGeom g,
                                                                             int per, int longer,
                                                                             int pix_tiles, int idx_dword_ok) {
    constexpr int BS = 64 * NI;  // floats reserved per channel
    __shared__ __align__(16) float band[kCT * BS];
    __shared__ __align__(16) char parts[4][kEncRows * kRowBytes];

    const int col_tiles = (C + kCT - 1) / kCT;
    const int c0 = (int)(blockIdx.x % col_tiles) * kCT;
    // chunks of `longer` tiles first, then of one tile less: the wavefronts of a SIMD share its time
    const int chunk = (int)(blockIdx.x / col_tiles);
    const int tile_begin = chunk * per - max(chunk - longer, 0), tile_end = tile_begin + per - (chunk >= longer);
    int image = tile_begin / pix_tiles, pt = tile_begin - image * pix_tiles;  // of the tile being loaded
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, q = lane >> 4;
    const int channel = c0 + w * kCPW;
    const uint32_t k0 = 4u * q;
    char* const buf = parts[w];
    // lane groups q = 0, 1 read the high parts, 2 the low ones, 3 the ninth value's
    const char* const from = buf + (lane & 15) * kRowBytes + (q == 0 ? 0 : 16 * (q - 1));
    float* const mine = band + w * kCPW * BS;
    const float recip_wo = 1.f / g.Wo;

    Band t = band_of(g, image, pt);
    Elements<NI> el;
    el.set(t.ncols, lane);
    float val[kCPW][NI];
    load_band<NI>(input, g, t, channel, C, el, val);
    f16x8 a[kCPW];
    f32x4 norm[kCPW];
    Threshold th[kCPW];
#pragma unroll
    for (int j = 0; j < kCPW; ++j) load_codebook<K_T>(P + (size_t)min(channel + j, C - 1) * K_T * kV, lane, a[j], norm[j], th[j]);

    // No barriers: a wavefront stages, searches and stores its own four channels, and one that meets a doubtful row
    // keeps nobody waiting.
    for (int tile = tile_begin; tile < tile_end; ++tile) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < kCPW; ++j) mine[j * BS + 64 * i + lane] = val[j][i];
        wave_lds_order();
        const Band now = t;
        const int64_t n0 = image * ((int64_t)g.Ho * g.Wo) + now.p0;
        if (tile + 1 < tile_end) {
            if (++pt == pix_tiles) {
                pt = 0;
                ++image;
            }
            t = band_of(g, image, pt);
            if (t.ncols != el.ncols) el.set(t.ncols, lane);
            load_band<NI>(input, g, t, channel, C, el, val);
        }

        // this lane's pixel and the offsets of its nine taps within a channel's band
        const int p = min(now.p0 + lane, now.p1);  // lanes past the last pixel repeat it (never stored)
        const int in_rows = p - now.ho0 * g.Wo, down = small_quotient(in_rows, recip_wo);
        const int base = down * g.sh * now.ncols + ((in_rows - down * g.Wo) * g.sw - g.pw - now.w_lo);
        int toff[kV];
        const float* tap[kV];
        {
            int rk = 0, sk = 0;
#pragma unroll
            for (int v = 0; v < kV; ++v) {
                toff[v] = rk * now.ncols + sk;
                tap[v] = mine + base + toff[v];
                if (++sk == g.kw) {
                    sk = 0;
                    ++rk;
                }
            }
        }
        uint32_t packed = 0, direct = 0;  // direct: codebooks whose 64 rows are searched directly
#pragma unroll
        for (int j = 0; j < kCPW; ++j) {
            if (!th[j].filter) {
                direct |= 1u << j;
                continue;
            }
            float x[kV];
#pragma unroll
            for (int v = 0; v < kV; ++v) x[v] = tap[v][j * BS];
            float xx = x[0] * x[0];
#pragma unroll
            for (int v = 1; v < kV; ++v) xx = __fmaf_rn(x[v], x[v], xx);
            store_parts(x, buf + lane * kRowBytes);
            wave_lds_order();
            f32x4 d[4];
#pragma unroll
            for (int gr = 0; gr < 4; ++gr) {
                const f16x8 bo = __builtin_bit_cast(f16x8, *reinterpret_cast<const u32x4*>(from + gr * 16 * kRowBytes));
                d[gr] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[j], bo, norm[j], 0, 0, 0);
            }
            wave_lds_order();
            bool unsure;
            uint32_t best = best_of(d, k0, xx, th[j], unsure);
            const uint64_t rows = __ballot(unsure);
            if (__builtin_popcountll(rows) > kFewRows) {
                direct |= 1u << j;
                th[j].filter = false;  // for the rest of the chunk, which is more of the same image
            } else if (rows)
                best = search_rows<K_T>(rows, best, mine + j * BS, base, toff, P + (size_t)min(channel + j, C - 1) * K_T * kV, lane);
            packed |= index_byte(best, j);
        }
        direct &= (1u << max(0, min(kCPW, C - channel))) - 1;
        while (direct) {  // wave-uniform
            const int j = __builtin_amdgcn_readfirstlane(__builtin_ctz(direct));
            direct &= direct - 1;
            const float* __restrict__ ch = mine + j * BS + base;
            float x[kV];
#pragma unroll
            for (int v = 0; v < kV; ++v) x[v] = ch[toff[v]];
            const uint32_t best = nearest_centroid<kV, K_T>(x, P + (size_t)(channel + j) * K_T * kV, K_T);
            packed = (packed & ~(0xffu << (8 * j))) | best << (8 * j);
        }
        // each lane stores its row's four bytes
        if (now.p0 + lane <= now.p1) {
            uint8_t* dst = idx.rows + (n0 + lane) * (int64_t)idx.ld + channel;
            if (idx_dword_ok) {
                if (channel < C) *reinterpret_cast<uint32_t*>(dst) = packed;
            } else {
#pragma unroll
                for (int b = 0; b < kCPW; ++b)
                    if (channel + b < C) dst[b] = (uint8_t)(packed >> (8 * b));
            }
        }
    }
}

template <int K_T, int NI>
hipError_t launch(const float* P, int C, const float* input, int64_t B, const ConvGeom& g, IndexRows idx, int64_t chunks,
                  hipStream_t s) {
    const int64_t pix_tiles = ((int64_t)g.Ho * g.Wo + kEncRows - 1) / kEncRows, tiles = B * pix_tiles;
    const int64_t blocks = chunks * ((C + kCT - 1) / kCT);
    const int per = (int)((tiles + chunks - 1) / chunks), longer = (int)(tiles - (per - 1) * chunks);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const int idx_dword_ok = idx.dwords(C);
    hipLaunchKernelGGL((encode_conv9_filter_kernel<K_T, NI>), dim3((unsigned)blocks), dim3(kEncThreads), 0, s, input, P, idx,
                       C, g, per, longer, (int)pix_tiles, idx_dword_ok);
    return hipGetLastError();
}

template <int K_T>
hipError_t launch_k(const float* P, int C, const float* input, int64_t B, const ConvGeom& g, IndexRows idx, int64_t chunks,
                    hipStream_t s) {
    const int64_t bs = conv_band_floats(g);
    if (bs <= 192) return launch<K_T, 3>(P, C, input, B, g, idx, chunks, s);
    if (bs <= 320) return launch<K_T, 5>(P, C, input, B, g, idx, chunks, s);
    return launch<K_T, 8>(P, C, input, B, g, idx, chunks, s);
}

}  // namespace

// Pixel tiles are shared out over as many chunks as are resident at once (four workgroups per CU; a chunk of several
// tiles prepares its operands once).  Against the direct search (64 channels, K = 16, 56 x 56, with the launch): 32
// images 59.5 -> 37 us, 16 33.4 -> 23, 8 20.1 -> 15.2, 4 12.9 -> 11.8; 32 x 128 channels 28 x 28 36.5 -> 22.5; 32 x 512, 7
// x 7 17.4 -> 12.  With less than a workgroup per CU a wavefront prepares its operands for one tile and waits for them:
// the direct search with its narrower tiles (one image: 6.3 us against 7.6 for the kernel alone).  With K = 8 the direct
// search is half as long, and the filter pays from four workgroups per CU on: 32 images 47 -> 41, 8 15.7 -> 15, 32 x 512, 7
// x 7 14.6 -> 12; 4 images 10.8 against 12.5.
// Where the filter can do nothing (all codebooks too small for it, or every row a tie between equal centroids): 32 images
// 59.4 -> 59 and 63, 8 20 -> 20.7 and 24, 4 12.6 -> 15.2 and 19.
int64_t encode_conv9_filter_chunks(int C, int K, int64_t B, const ConvGeom& g) {
    if (K != 8 && K != 16) return 0;
    // bands of up to 512 floats, and a wavefront's four channels within a resource's 32-bit offsets
    if (conv_band_floats(g) > 512 || (int64_t)g.H * g.W >= 1 << 26 || g.Wo > 1 << 19) return 0;
    const int64_t tiles = B * (((int64_t)g.Ho * g.Wo + kEncRows - 1) / kEncRows);
    const int64_t resident = (int64_t)compute_units() * 4, col_tiles = (C + kCT - 1) / kCT;
    if (K == 16 ? tiles * col_tiles <= compute_units() : tiles * col_tiles < resident) return 0;
    return std::min(std::max<int64_t>(resident / col_tiles, 1), tiles);
}

hipError_t launch_encode_conv9_filter(const float* P, int C, int K, const float* input, int64_t B, const ConvGeom& g,
                                      IndexRows idx, int64_t chunks, hipStream_t s) {
    if (K == 8) return launch_k<8>(P, C, input, B, g, idx, chunks, s);
    return launch_k<16>(P, C, input, B, g, idx, chunks, s);
}

}  // namespace lutnn
