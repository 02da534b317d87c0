// Log-sum-exp merge of split partials (the flash-decoding reduction, Sec. 2): for each (sequence,
// query head), M* = max_s m_s, l* = sum_s e^{m_s - M*} l_s, out = sum_s e^{m_s - M*} acc_s / l*,
// lse = M* + ln l*. Splits that kept nothing carry m = -inf and are skipped; a head with no split
// gets out = 0 and lse = -inf.
//
// Partial rows of head bh = b * Hq + h: i * G + bh % G for i = first .. last, (first, last) = table[bh / G]
// (last < first: none), or, without a table, the S rows from S * (bh / G) on.
//
// Mapping: one workgroup per (sequence, query head), running merge_partial_rows.
#include "ffd_device.h"
#include "ffd_kernels.h"

namespace ffd {

__global__ __launch_bounds__(kThreads) void lse_merge_kernel(const float* __restrict__ part_m,
                                                             const float* __restrict__ part_l,
                                                             const float* __restrict__ part_acc, int S,
                                                             const int2* __restrict__ table, int G,
                                                             uint16_t* __restrict__ out, float* __restrict__ lse) {
    const size_t x = blockIdx.x / G;                        // blockIdx.x = b * Hq + h
    size_t first = x * S;
    if (table) {
        const int2 fl = table[x];
        first = fl.x;
        S = fl.y - fl.x + 1;
    }
    merge_partial_rows(part_m, part_l, part_acc, first * G + blockIdx.x % G, G, S, out + (size_t)blockIdx.x * kD,
                       lse ? lse + blockIdx.x : nullptr);
}

}  // namespace ffd
