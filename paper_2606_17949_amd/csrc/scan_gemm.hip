// GEMM-structured bank-scan launcher.
#include "scan_gemm.hpp"

namespace rb {

namespace {

template <int TPQ>
hipError_t launch_gemm(const KnnPlan &p, const ScanArgs &a, hipStream_t s)
{
    auto kern = a.m.folded ? gemm_scan_kernel<TPQ, true> : gemm_scan_kernel<TPQ, false>;
    hipError_t e = hipFuncSetAttribute((const void *)kern,
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)p.lds_bytes);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(kern, dim3(p.grid), dim3(GM_WAVES * WAVE), p.lds_bytes, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_scan_gemm(const KnnPlan &p, const ScanArgs &a, hipStream_t s)
{
    return p.qw == 2 ? launch_gemm<2>(p, a, s) : launch_gemm<4>(p, a, s);
}

}  // namespace rb
