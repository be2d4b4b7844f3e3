// Instantiations of the matrix-core unit kernel for bf16 rows above 256 bytes.
#include "zp_mfma.h"

namespace zp {
hipError_t launch_mfma_pad_bf16_long(const Args &a, int units, int rowb, int NW, hipStream_t s) {
    if (rowb == 384) return launch_pad<1, 384>(a, units, NW, s);
    if (rowb == 512) return launch_pad<1, 512>(a, units, NW, s);
    return launch_pad<1, 1024>(a, units, NW, s);
}
}  // namespace zp
