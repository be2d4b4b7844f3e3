// Instantiations of the matrix-core unit kernel for bf16 rows of any other size up to 256 bytes, and for windows of more than 32 query blocks.
#include "zp_mfma.h"

namespace zp {
hipError_t launch_mfma_pad_bf16(const Args &a, int units, int rowb, int NW, hipStream_t s) {
    if (rowb == 128) return launch_pad<1, 128>(a, units, NW, s);
    if (rowb == 192) return launch_pad<1, 192>(a, units, NW, s);
    return launch_pad<1, 256>(a, units, NW, s);
}
}  // namespace zp
