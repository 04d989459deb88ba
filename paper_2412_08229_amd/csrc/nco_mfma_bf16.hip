// Kernels of the bf16 network (nco_mfma.h).
#include "nco_mfma.h"

namespace nco {

NCO_NET_DEFINE(bf16, MLP_PREC_BF16)

}  // namespace nco
