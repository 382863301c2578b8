// The fused middle layer with 5 accumulators.
#include "ksmac.hpp"

namespace ckks {
template hipError_t launch_ksmac_nk<5>(const ckks_params*, const KsMacArgs&, hipStream_t);
}  // namespace ckks
