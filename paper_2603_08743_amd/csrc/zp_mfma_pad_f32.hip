// Instantiations of the matrix-core unit kernel for fp32 pools.
#include "zp_mfma.h"

namespace zp {
hipError_t launch_mfma_pad_f32(const Args &a, int units, int rowb, int NW, hipStream_t s) {
    if (rowb == 256) return launch_pad<0, 256>(a, units, NW, s);
    if (rowb == 512) return launch_pad<0, 512>(a, units, NW, s);
    return launch_pad<0, 1024>(a, units, NW, s);
}
}  // namespace zp
