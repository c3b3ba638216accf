// One storage type and head dimension of the builder's SVD kernel (SEKV_ELEM bytes, SEKV_D),
// for its sketch widths and wave counts; the build compiles this file once per pair.
#include "sekv_svd.h"

#if !defined(SEKV_ELEM) || !defined(SEKV_D)
#error "build with -DSEKV_ELEM=2|4 -DSEKV_D=64|128"
#endif

#define SEKV_CAT3(a, b, c) a##_##b##_##c
#define SEKV_NAME(fn, e, d) SEKV_CAT3(fn, e, d)

namespace sekv {

hipError_t SEKV_NAME(launch_svd, SEKV_ELEM, SEKV_D)(const BuildArgs &a, unsigned items, bool wide, hipStream_t s) {
    const dim3 grid(items, 2);
    const bool two = a.l <= 32;
    if (wide) {
        if (two) hipLaunchKernelGGL((svd_kernel<SEKV_ELEM, SEKV_D, 2, 4>), grid, dim3(256), 0, s, a);
        else hipLaunchKernelGGL((svd_kernel<SEKV_ELEM, SEKV_D, 3, 4>), grid, dim3(256), 0, s, a);
    } else {
        if (two) hipLaunchKernelGGL((svd_kernel<SEKV_ELEM, SEKV_D, 2, 1>), grid, dim3(64), 0, s, a);
        else hipLaunchKernelGGL((svd_kernel<SEKV_ELEM, SEKV_D, 3, 1>), grid, dim3(64), 0, s, a);
    }
    return hipGetLastError();
}

}  // namespace sekv
