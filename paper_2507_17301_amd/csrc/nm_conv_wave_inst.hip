// Explicit instantiations of the kernel for small fp32 layers.  Compiled once per shape
// (-DNM_INST_PB=.. -DNM_INST_NJ=..).
#include "nm_conv_wave_kernel.h"
#include "nm_variants.h"

namespace nm {
#define NM_INST_WAVE(PB, NJ, CK, SPC, NW) template int launch_wave_t<PB, NJ, CK, SPC, NW>(const ConvParams&, hipStream_t);
#define NM_INST_LIST(PB, NJ) NMWAVE_##PB##_##NJ(NM_INST_WAVE)
#define NM_INST_SHAPE(PB, NJ) NM_INST_LIST(PB, NJ)
NM_INST_SHAPE(NM_INST_PB, NM_INST_NJ)
}  // namespace nm
