// Kernels of the float32-class network split over the 16-bit matrix cores
// (nco_mfma.h).
#include "nco_mfma.h"

namespace nco {

NCO_NET_DEFINE(split, MLP_PREC_F32S)

}  // namespace nco
