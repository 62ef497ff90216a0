// Choice of a GEMM kernel by rows and weight form; included by the translation units that hold a kind's kernels.
#pragma once

#include "ee_kernels.hpp"

namespace ee {

// A kernel per 8 rows: the kilobytes of a k-tile of the input are compile-time.  With a kernel per 16 rows the odd classes copy
// one kilobyte per k-tile more: 5 rows 3.01 ms a pass against 2.97, 18 rows 1.091 against 1.060, 40 rows 1.433 against
// 1.383 (7B shape; the latter two with 8 layers).
template <int KIND, bool PK>
static pass_kernel_t kernel_for_rows(int rows)
{
    switch ((rows + 7) / 8) {
    case 1: return ee_gemm_kernel<KIND, 1, PK>;
    case 2: return ee_gemm_kernel<KIND, 2, PK>;
    case 3: return ee_gemm_kernel<KIND, 3, PK>;
    case 4: return ee_gemm_kernel<KIND, 4, PK>;
    case 5: return ee_gemm_kernel<KIND, 5, PK>;
    default: return ee_gemm_kernel<KIND, 6, PK>;
    }
}

// (adapters are never packed)
template <int KIND>
pass_kernel_t gemm_kernel_of(int rows, bool packed)
{
    if constexpr (KIND != G_AD && KIND != G_AU)
        if (packed) return kernel_for_rows<KIND, true>(rows);
    return kernel_for_rows<KIND, false>(rows);
}

}  // namespace ee
