// LDS-resident bank-scan instantiations for fp32 embeddings.
#include "scan_res.hpp"

namespace rb {

hipError_t launch_scan_res_f32(const KnnPlan &p, const ScanArgs &a, hipStream_t s)
{
    return launch_res<0>(p, a, s);
}

}  // namespace rb
