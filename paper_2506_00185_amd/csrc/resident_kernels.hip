// Instantiations of the resident step loop, one translation unit per (width, precision, prediction network): built with
// -DRB_RES_FULL=0|1 (1: H = P = 640) -DRB_RES_FORM=0|1|2 (see ResForm) -DRB_RES_ST=0|1 (1: stateless).
#include "kernels_resident.h"

namespace rb {

template <bool FULL, int FORM, bool ST>
ResKernel resident_kernel(int K, bool plain) {
  if (K <= 4) return plain ? k_decode_resident<FULL, FORM, ST, 4, 1> : k_decode_resident<FULL, FORM, ST, 4, 0>;
  if (K <= 8) return plain ? k_decode_resident<FULL, FORM, ST, 8, 1> : k_decode_resident<FULL, FORM, ST, 8, 0>;
  return plain ? k_decode_resident<FULL, FORM, ST, 16, 1> : k_decode_resident<FULL, FORM, ST, 16, 0>;
}
template ResKernel resident_kernel<RB_RES_FULL != 0, RB_RES_FORM, RB_RES_ST != 0>(int, bool);

}  // namespace rb
