#include "ee_gemm_select.hpp"

namespace ee {
template pass_kernel_t gemm_kernel_of<G_AD>(int rows, bool packed);
template pass_kernel_t gemm_kernel_of<G_AU>(int rows, bool packed);
}  // namespace ee
