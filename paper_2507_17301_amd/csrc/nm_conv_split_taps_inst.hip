// Explicit instantiation of the tap-staged three-plane fp32 kernel.  Compiled once per shape
// (-DNM_INST_NBLK=.. -DNM_INST_WP=.. -DNM_INST_NJ=.. -DNM_INST_KG=.. -DNM_INST_SPARSE=0 or 1).
#include "nm_conv_split_taps_kernel.h"

namespace nm {
template int launch_split_taps_t<NM_INST_NBLK, NM_INST_WP, NM_INST_NJ, NM_INST_KG, (NM_INST_SPARSE) != 0>(const ConvParams&, hipStream_t);
}  // namespace nm
