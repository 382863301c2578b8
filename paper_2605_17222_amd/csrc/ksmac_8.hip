// The fused middle layer with 8 accumulators.
#include "ksmac.hpp"

namespace ckks {
template hipError_t launch_ksmac_nk<8>(const ckks_params*, const KsMacArgs&, hipStream_t);
}  // namespace ckks
