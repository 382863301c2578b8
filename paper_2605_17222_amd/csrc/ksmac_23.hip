// The fused middle layer with 2 or 3 accumulators.
#include "ksmac.hpp"

namespace ckks {
template hipError_t launch_ksmac_nk<2>(const ckks_params*, const KsMacArgs&, hipStream_t);
template hipError_t launch_ksmac_nk<3>(const ckks_params*, const KsMacArgs&, hipStream_t);
}  // namespace ckks
