// Explicit instantiations of the row-staged kernel for few input channels (-DNM_INST_PL=1 bf16, 3 fp32).
#include "nm_conv_rows_kernel.h"
#include "nm_variants.h"

namespace nm {
#define NM_INSTROWS(NJ, KS) template int launch_rows_t<NM_INST_PL, NJ, KS>(const ConvParams&, hipStream_t);
#if NM_INST_PL == 1
NMROWB_CHUNKS(NM_INSTROWS)
#else
NMROWF_CHUNKS(NM_INSTROWS)
#endif
}  // namespace nm
