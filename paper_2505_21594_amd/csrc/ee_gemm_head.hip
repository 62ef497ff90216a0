#include "ee_gemm_select.hpp"

namespace ee {
template pass_kernel_t gemm_kernel_of<G_HEAD>(int rows, bool packed);
}  // namespace ee
