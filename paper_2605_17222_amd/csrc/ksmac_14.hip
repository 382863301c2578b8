// The fused middle layer with 1 or 4 accumulators.
#include "ksmac.hpp"

namespace ckks {
template hipError_t launch_ksmac_nk<1>(const ckks_params*, const KsMacArgs&, hipStream_t);
template hipError_t launch_ksmac_nk<4>(const ckks_params*, const KsMacArgs&, hipStream_t);
}  // namespace ckks
