// Instantiations of the matrix-core unit kernel for bf16 rows of 256 bytes (head dimension 128), eight waves per workgroup.
#include "zp_mfma.h"

namespace zp {
hipError_t launch_mfma_d128_wide(const Args &a, int units, int NW, int RB, hipStream_t s) { return launch_d<256, 1, false>(a, units, NW, RB, s); }
}  // namespace zp
