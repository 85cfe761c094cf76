// The box kernel of many problems, and launches of the box-tile kernels.
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

// The boxes of many problems in one launch (here and not in the header: a
// specialised kernel is compiled with the header, and every kernel that is no
// template would be compiled along, which doubled the time).
//
// Every problem has whole chunks of 2^chunk boxes; consecutive chunks go round
// the XCDs, a chunk's boxes stay on one.  A table of at most kBoxBuckets
// entries narrows the search for a chunk's problem down to those that start in
// one stretch of chunks (one problem as a rule).  Two units a thread: the four bodies need no more
// registers than 8 wavefronts a SIMD leave.
__global__ __launch_bounds__(kThreads, 8) void k_box_batch(const BoxBatchDesc* __restrict__ desc,
                                                           const uint32_t* __restrict__ first,
                                                           const uint32_t* __restrict__ bucket, int shift, int chunk,
                                                           uint32_t chunks) {
    __shared__ __align__(16) unsigned char lds[box_lds(1, 2)];
    const uint32_t set = blockIdx.x >> (chunk + 3), r = blockIdx.x & ((8u << chunk) - 1);
    const uint32_t c = set * 8 + (r & 7);
    if (c >= chunks) return;
    uint32_t lo = bucket[c >> shift], hi = bucket[(c >> shift) + 1];
    while (lo < hi) {   // the last problem whose first chunk is c or before
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (first[mid] <= c) lo = mid;
        else hi = mid - 1;
    }
    // read through the constant address space: fields live in scalar registers
    typedef __attribute__((address_space(4))) const BoxBatchDesc ConstDesc;
    const BoxBatchDesc& d = *(const BoxBatchDesc*)((ConstDesc*)(desc + lo));
    const uint32_t t = ((c - first[lo]) << chunk) + (r >> 3);
    touch(d);
    if (t >= d.f64.ntiles) return;   // the last chunk's tail (both kinds start with BoxShape)
    switch (d.kind) {
        case 0: return box_body<float, float, false, 2>(reinterpret_cast<float*>(lds), d.f32, d.f32, t);
        case 1: return box_body<float, float, true, 2>(reinterpret_cast<float*>(lds), d.f32, d.f32, t);
        case 2: return box_body<double, double, false, 2>(reinterpret_cast<double*>(lds), d.f64, d.f64, t);
        default: return box_body<double, double, true, 2>(reinterpret_cast<double*>(lds), d.f64, d.f64, t);
    }
}

hipError_t launch_box_batch(const BoxBatchDesc* desc, const uint32_t* first, const uint32_t* bucket,
                            const BoxBatchGrid& g, hipStream_t stream) {
    hipLaunchKernelGGL(k_box_batch, dim3(g.grid), dim3(kThreads), 0, stream, desc, first, bucket, g.shift, g.chunk,
                       g.chunks);
    return hipGetLastError();
}

}  // namespace ttx
