// Explicit instantiations of the tap-staged bf16 kernel.  Compiled once per shape and instruction
// (-DNM_INST_NBLK=.. -DNM_INST_WP=.. -DNM_INST_NJ=.. -DNM_INST_SPARSE=.. -DNM_INST_NW=..).
#include "nm_conv_taps_kernel.h"

namespace nm {
template int launch_taps_t<NM_INST_NBLK, NM_INST_WP, NM_INST_NJ, (NM_INST_SPARSE) != 0, NM_INST_NW>(const ConvParams&, hipStream_t);
}  // namespace nm
