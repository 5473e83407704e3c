// LDS-resident bank-scan instantiations for bf16 embeddings.
#include "scan_res.hpp"

namespace rb {

hipError_t launch_scan_res_bf16(const KnnPlan &p, const ScanArgs &a, hipStream_t s)
{
    return launch_res<1>(p, a, s);
}

}  // namespace rb
