// The rows of a convolution's im2col matrix (arXiv 2302.03213, Sec. 4) read from the image and from [B][D][Ho*Wo]
// arrays - the layout that a product of the weight matrix with the images' output gradients has by itself, and in
// which 64 consecutive output pixels of a column are 64 consecutive words - for kernels with lane = row.
#pragma once
#include "encode_tile.h"
#include "lutnn_kernels.h"

namespace lutnn {

// One lane's row n = (image b, output pixel p): where its patch starts in the image, which filter taps fall inside
// (filters of up to 32 taps), and where the row starts in a [B][D][Ho*Wo] array.
struct ConvRow {
    bool ok;
    uint32_t taps;
    int hi0, wi0;
    int64_t image, column;
};

__device__ __forceinline__ ConvRow conv_row(const ConvGeom& g, uint32_t n, uint32_t N, int D) {
    const uint32_t pix = (uint32_t)(g.Ho * g.Wo);
    ConvRow r;
    r.ok = n < N;
    const uint32_t m = r.ok ? n : 0u;
    const uint32_t b = m / pix, p = m - b * pix;
    const uint32_t ho = p / (uint32_t)g.Wo;
    r.hi0 = (int)ho * g.sh - g.ph;
    r.wi0 = (int)(p - ho * (uint32_t)g.Wo) * g.sw - g.pw;
    r.image = ((int64_t)b * g.Cin * g.H + r.hi0) * g.W + r.wi0;
    r.column = (int64_t)b * D * pix + p;
    r.taps = 0;
    if (g.kh * g.kw <= 32) {
        int t = 0;
        for (int rk = 0; rk < g.kh; ++rk) {
            const bool h_ok = r.ok && (unsigned)(r.hi0 + rk) < (unsigned)g.H;
            for (int sk = 0; sk < g.kw; ++sk, ++t)
                r.taps |= (uint32_t)(h_ok && (unsigned)(r.wi0 + sk) < (unsigned)g.W) << t;
        }
    }
    return r;
}

// Columns [j0, j0 + COLS) of the lane's row into registers, zero outside the image and past D.  TAPS > 0: the filter
// has that many taps and j0 is the first tap of a channel, so channel and tap of every column are known at compile
// time; TAPS < 0: any filter.
template <int COLS, int TAPS>
__device__ __forceinline__ void load_patch(const float* __restrict__ input, const ConvGeom& g, const ConvRow& r, int j0,
                                           int D, float (&x)[COLS]) {
    const int64_t HW = (int64_t)g.H * g.W;
    if constexpr (TAPS > 0) {
        const int64_t first = (int64_t)(j0 / TAPS) * HW;
        int rk = 0, sk = 0;
        int at[TAPS];
#pragma unroll
        for (int t = 0; t < TAPS; ++t) {
            at[t] = rk * g.W + sk;
            if (++sk == g.kw) {
                sk = 0;
                ++rk;
            }
        }
#pragma unroll
        for (int i = 0; i < COLS; ++i) {
            x[i] = 0.f;
            if (j0 + i < D && (r.taps >> (i % TAPS) & 1u)) x[i] = input[r.image + (first + i / TAPS * HW + at[i % TAPS])];
        }
    } else {
        const int taps = g.kh * g.kw;
        int ci = j0 / taps, rk = (j0 - ci * taps) / g.kw, sk = j0 - ci * taps - rk * g.kw;
#pragma unroll
        for (int i = 0; i < COLS; ++i) {
            const bool inside = r.ok && (unsigned)(r.hi0 + rk) < (unsigned)g.H && (unsigned)(r.wi0 + sk) < (unsigned)g.W;
            x[i] = 0.f;
            if (j0 + i < D && inside) x[i] = input[r.image + ((int64_t)ci * HW + rk * g.W + sk)];
            if (++sk == g.kw) {
                sk = 0;
                if (++rk == g.kh) {
                    rk = 0;
                    ++ci;
                }
            }
        }
    }
}

template <int COLS>
__device__ __forceinline__ void load_columns(const float* __restrict__ A, const ConvGeom& g, const ConvRow& r, int j0,
                                             int D, float (&x)[COLS]) {
    const int64_t pix = (int64_t)g.Ho * g.Wo;
#pragma unroll
    for (int i = 0; i < COLS; ++i) {
        x[i] = 0.f;
        if (r.ok && j0 + i < D) x[i] = A[r.column + (j0 + i) * pix];
    }
}

template <int COLS>
__device__ __forceinline__ void store_columns(float* __restrict__ A, const ConvGeom& g, const ConvRow& r, int j0, int D,
                                              const float* __restrict__ x) {
    const int64_t pix = (int64_t)g.Ho * g.Wo;
#pragma unroll
    for (int i = 0; i < COLS; ++i)
        if (r.ok && j0 + i < D) A[r.column + (j0 + i) * pix] = x[i];
}

}  // namespace lutnn
