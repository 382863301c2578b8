// The fused middle layer with 7 accumulators.
#include "ksmac.hpp"

namespace ckks {
template hipError_t launch_ksmac_nk<7>(const ckks_params*, const KsMacArgs&, hipStream_t);
}  // namespace ckks
