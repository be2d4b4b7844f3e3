// Instantiations of the matrix-core unit kernel for bf16 rows of 256 bytes (head dimension 128), eight waves per workgroup, with score refinements.
#include "zp_mfma.h"

namespace zp {
hipError_t launch_mfma_d128_wide_ref(const Args &a, int units, int NW, int RB, hipStream_t s) { return launch_d<256, 1, true>(a, units, NW, RB, s); }
}  // namespace zp
