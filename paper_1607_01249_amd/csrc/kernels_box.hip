// Launch of the box-tile kernels.
#include "box_kernel.h"
#include "ttx_internal.h"

namespace ttx {

template <typename T, typename S>
static hipError_t launch_box_as(const BoxPlan& bp, bool beta0, const void* A, const void* Bsrc, void* Bdst,
                                const Scalar& alpha, const Scalar& beta, hipStream_t stream) {
    BoxArgs<T, S> a;
    static_cast<BoxShape&>(a) = bp.s;
    static_cast<BoxPtrs<T, S>&>(a) = {static_cast<const S*>(A), static_cast<const T*>(Bsrc), static_cast<T*>(Bdst),
                                      scalar_as<T>(alpha), scalar_as<T>(beta)};
    const dim3 g(a.ntiles), b(kThreads);
    const auto kernel = bp.nt && box_on_line(Bdst) ? (bp.units == 2 ? k_box<T, S, true, 2, true> : k_box<T, S, true, 4, true>)
                        : bp.units == 2 ? (beta0 ? k_box<T, S, true, 2, false> : k_box<T, S, false, 2, false>)
                                        : (beta0 ? k_box<T, S, true, 4, false> : k_box<T, S, false, 4, false>);
    hipLaunchKernelGGL(kernel, g, b, 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_box(const Problem& p, const BoxPlan& bp, bool beta0, const void* A, const void* Bsrc, void* Bdst,
                      const Scalar& alpha, const Scalar& beta, hipStream_t stream) {
    switch (p.code) {
        case TTX_F32: return launch_box_as<float, float>(bp, beta0, A, Bsrc, Bdst, alpha, beta, stream);
        case TTX_F64: return launch_box_as<double, double>(bp, beta0, A, Bsrc, Bdst, alpha, beta, stream);
        case TTX_C32: return launch_box_as<cf32, cf32>(bp, beta0, A, Bsrc, Bdst, alpha, beta, stream);
        case TTX_C64: return launch_box_as<cf64, cf64>(bp, beta0, A, Bsrc, Bdst, alpha, beta, stream);
        case TTX_F32_F64: return launch_box_as<double, float>(bp, beta0, A, Bsrc, Bdst, alpha, beta, stream);
        case TTX_F64_F32: return launch_box_as<float, double>(bp, beta0, A, Bsrc, Bdst, alpha, beta, stream);
        case TTX_C32_C64: return launch_box_as<cf64, cf32>(bp, beta0, A, Bsrc, Bdst, alpha, beta, stream);
        case TTX_C64_C32: return launch_box_as<cf32, cf64>(bp, beta0, A, Bsrc, Bdst, alpha, beta, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_box_batch(const BoxBatchDesc* desc, const uint32_t* first, const uint32_t* bucket,
                            const BoxBatchGrid& g, hipStream_t stream) {
    hipLaunchKernelGGL(k_box_batch, dim3(g.grid), dim3(kThreads), 0, stream, desc, first, bucket, g.shift, g.chunk,
                       g.chunks);
    return hipGetLastError();
}

}  // namespace ttx
