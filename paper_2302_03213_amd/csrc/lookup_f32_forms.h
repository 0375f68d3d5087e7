// Which form an unquantised lookup (arXiv 2302.03213, Eq. 4) takes: the one that takes the least.  Host code alone.
//
// Prices in us, fitted to 2490 lookups of 16-60000 rows, 1-700 codebooks of 8-150 table rows and 32-4096 columns, each
// timed in all its forms: the form chosen takes 1.004 times the fastest one's time on average (the rule before, which preferred
// rows to the gather wherever they can run: 1.19, up to 4.5).
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace lutnn {

enum class LookupF32 { gather, rows, matrix };

struct LookupF32Us {
    double gather, rows, matrix;  // kNever: not on this shape
    static constexpr double kNever = 1e30;
    LookupF32 least(int64_t N, int M) const {
        if (matrix < rows && matrix < gather) return LookupF32::matrix;
        // outputs past what the gather's grid counts (2^32 threads, 64 for a row of 132 columns): rows, where it can run
        if (rows < gather || (rows < kNever && (double)N * ((M + 255) / 256) > 6e7)) return LookupF32::rows;
        return LookupF32::gather;
    }
};

// rows_ok: rows_kernel_preferred
inline LookupF32Us lookup_f32_us(int C, int K, int M, int64_t N, bool rows_ok, int compute_units) {
    const auto tiles = [&](int rows, int cols) {  // per compute unit
        return (double)((N + rows - 1) / rows) * ((M + cols - 1) / cols) / compute_units;
    };
    const double outputs = 1e-6 * (double)N * M, entries = outputs * C;
    LookupF32Us us;

    // The gather reads every entry from L2, or from behind it where the table is larger than 4 MB: up to 0.5 ps more per entry.
    // A row of 8, 16 or 32 wavefronts keeps an XCD's workgroups to a half, a quarter or an eighth of the columns, and the
    // misses of its L2 are fewer (300 rows x 512 codebooks, M = 4096 180 us; 400 x 192, M = 3072, twice the time an entry).
    // Rows of fewer than four columns have a thread per output in its place, eight codebooks in flight.
    if (M >= 4) {
        const int across = (M + 255) / 256;
        const bool shared = across == 8 || across == 16 || across == 32;
        const double behind = std::log2(4.0 * C * K * M / 1048576 / (shared ? across / 4 : 1));
        const double per_entry = shared ? 0.115 + 0.052 * std::clamp(behind - 1.5, 0.0, 4.5) : 0.14 + 0.082 * std::clamp(behind - 1.8, 0.0, 4.5);
        us.gather = 5 + per_entry * entries + 0.75 * outputs;
    } else {
        us.gather = 5 + 0.05 * C + 1e-6 * (double)N * C * (0.2 + 0.45 * M);
    }

    // Lane = row: four workgroups of a compute unit stage their slabs side by side, and widths that are no multiple of four
    // are staged value by value.
    us.rows = LookupF32Us::kNever;
    if (rows_ok) {
        const double t = tiles(256, 64);
        us.rows = 11 + C * (0.14 + 0.145 * t + 0.03 * K * std::ceil(t / 4)) * (M % 4 ? 1.5 : 1) + 2 * outputs;
    }

    // The matrix form walks the codebooks once per tile, two tiles of a compute unit side by side.
    us.matrix = LookupF32Us::kNever;
    if (K <= 16 && C >= 16) us.matrix = 10 + C * std::max(0.355, 0.295 * tiles(256, 64)) + outputs;
    return us;
}

}  // namespace lutnn
