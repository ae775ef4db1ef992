// Explicit instantiations of the channel-walking 1x1 bf16 kernel, all numbers of input channels of one tile height
// (-DNM_INST_NBLK=..).
#include "nm_conv_cols_kernel.h"
#include "nm_variants.h"

namespace nm {
#define NM_INSTCOLS(NB, NCH) template int launch_cols_t<NB, NCH>(const ConvParams&, hipStream_t);
NMCOLS_CHUNKS(NM_INSTCOLS, NM_INST_NBLK)
}  // namespace nm
