// GEMM-structured bank-scan launcher.
#include "scan_gemm.hpp"

namespace rb {

namespace {

template <int TPQ, int OUT>
hipError_t launch_out(const KnnPlan &p, const ScanArgs &a, hipStream_t s)
{
    auto kern = gemm_scan_kernel<TPQ, OUT>;
    hipError_t e = hipFuncSetAttribute((const void *)kern,
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)p.lds_bytes);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(kern, dim3(p.grid), dim3(GM_WAVES * WAVE), p.lds_bytes, s, a);
    return hipGetLastError();
}

template <int TPQ>
hipError_t launch_gemm(const KnnPlan &p, const ScanArgs &a, hipStream_t s)
{
    return a.acc        ? launch_out<TPQ, GM_VALUES>(p, a, s)
           : a.m.folded ? launch_out<TPQ, GM_FOLDED>(p, a, s)
                        : launch_out<TPQ, GM_ENTRIES>(p, a, s);
}

}  // namespace

hipError_t launch_scan_gemm(const KnnPlan &p, const ScanArgs &a, hipStream_t s)
{
    return p.qw == 2 ? launch_gemm<2>(p, a, s) : launch_gemm<4>(p, a, s);
}

}  // namespace rb
