// The direct contraction kernels for FP32.
#include "contract_kernel.h"

namespace ttx {

hipError_t launch_contract_f32(const ContractPlan& p, const float* X, const float* Y, float* C, float* part,
                               float alpha, float beta, hipStream_t stream) {
    return launch_contract_variant<float>(p, X, Y, C, part, alpha, beta, stream);
}

}  // namespace ttx
