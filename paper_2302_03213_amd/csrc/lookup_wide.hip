// Table read and accumulation (arXiv 2302.03213, Eq. 4) with 16-bit indices: the lookup behind the
// hash encoder's deep trees (Sec. 2, Sec. 7: up to 12 levels, K = 4096 buckets per codebook).
//
// With thousands of table rows per codebook nothing of the table can be staged or turned into a
// matrix operand: a (row, codebook) pair selects one of K rows of M entries, which is read straight
// from global memory by the gather that 8-bit indices take for small problems (gather_launch.h).
#include "gather_launch.h"
#include "lutnn_kernels.h"

namespace lutnn {
namespace {

template <class Table>
hipError_t launch_wide(const typename Table::Entry* T, const float* scale, const float* bias, int C, int K, int M,
                       const uint16_t* idx, int64_t N, float* Y, int64_t ldy, hipStream_t s) {
    if (gather_supported<Table>(M)) return launch_gather<Table, uint16_t>(T, scale, bias, C, K, M, idx, N, Y, ldy, s);
    return launch_global<Table, uint16_t>(T, scale, bias, C, K, M, idx, N, Y, ldy, s);
}

}  // namespace

hipError_t launch_lookup_wide_i8(const int8_t* T, const float* scale, const float* bias, int C, int K, int M,
                                 const uint16_t* idx, int64_t N, float* Y, int64_t ldy, hipStream_t s) {
    return launch_wide<TableI8>(T, scale, bias, C, K, M, idx, N, Y, ldy, s);
}

hipError_t launch_lookup_wide_f32(const float* T, const float* bias, int C, int K, int M, const uint16_t* idx,
                                  int64_t N, float* Y, int64_t ldy, hipStream_t s) {
    return launch_wide<TableF32>(T, nullptr, bias, C, K, M, idx, N, Y, ldy, s);
}

}  // namespace lutnn
