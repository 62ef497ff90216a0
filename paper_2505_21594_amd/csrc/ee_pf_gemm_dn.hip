#include "ee_prefill.hpp"

namespace ee {
template <int KIND, int WN, int WM, int GRP>
pf_kernel_t pf_gemm_of()
{
    return pf_gemm_kernel<KIND, WN, WM, GRP>;
}
#define EE_ONE(WN, WM, GRP) template pf_kernel_t pf_gemm_of<G_DN, WN, WM, GRP>();
EE_PF_SHAPES(EE_ONE)
}  // namespace ee
