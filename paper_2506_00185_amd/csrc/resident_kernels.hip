// Instantiations of the resident step loop, one translation unit per (width, precision) pair: built with
// -DRB_RES_FULL=0|1 (1: H = P = 640) -DRB_RES_BF16=0|1.
#include "kernels_resident.h"

namespace rb {

namespace {
constexpr bool kFull = RB_RES_FULL != 0, kBf16 = RB_RES_BF16 != 0;
ResKernel pick(int K, bool plain) {
  if (K <= 4) return plain ? k_decode_resident<kFull, kBf16, 4, 1> : k_decode_resident<kFull, kBf16, 4, 0>;
  if (K <= 8) return plain ? k_decode_resident<kFull, kBf16, 8, 1> : k_decode_resident<kFull, kBf16, 8, 0>;
  return k_decode_resident<kFull, kBf16, 16, 0>;
}
}  // namespace

#if RB_RES_FULL && RB_RES_BF16
ResKernel resident_kernel_640_bf16(int K, bool plain) { return pick(K, plain); }
#elif RB_RES_FULL
ResKernel resident_kernel_640_f32(int K, bool plain) { return pick(K, plain); }
#elif RB_RES_BF16
ResKernel resident_kernel_any_bf16(int K, bool plain) { return pick(K, plain); }
#else
ResKernel resident_kernel_any_f32(int K, bool plain) { return pick(K, plain); }
#endif

}  // namespace rb
