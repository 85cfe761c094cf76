// The direct contraction kernels for FP64.
#include "contract_kernel.h"

namespace ttx {

hipError_t launch_contract_f64(const ContractPlan& p, const double* X, const double* Y, double* C, double* part,
                               double alpha, double beta, hipStream_t stream) {
    return launch_contract_variant<double>(p, X, Y, C, part, alpha, beta, stream);
}

}  // namespace ttx
