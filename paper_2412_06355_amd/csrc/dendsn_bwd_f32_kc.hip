// Backward-kernel instantiations and dispatch for f32 storage with KC = 2 or 4
// compartments per branch.  V: bit 0 = Mexican-hat
// activation, bit 1 = residual dendrite, bits 2-3 = log2(KC), bit 5 = sigmoid
// surrogate (DENDSN_SG); KS: stash steps.
// Bit 6 of V = Stateless Dendrite (the runtime v passed in: psi | residual << 1 |
// stateless << 2, mapped by variant_bits).
#include "dendsn_kernels.h"

#if !defined(DENDSN_SG) || !defined(DENDSN_SL)
#error "compile once per surrogate, -DDENDSN_SG=0 (atan) or 1 (sigmoid), and dendrite, -DDENDSN_SL=0 or 1 (Stateless)"
#endif

namespace dendsn {

constexpr int kVS = DENDSN_SG << 5;  // surrogate bit of the variant

template <int BL, int L, int KC, int KS>
static hipError_t launch_bwd_kc_v(const Plan& pl, const BwdArgs& ba, int v, hipStream_t stream) {
  constexpr int VK = (KC == 2 ? 1 : 2) << 2;
  switch (v & 7) {
#define DENDSN_V(n) \
    case n: return launch_bwd<float, BL, L, kVS | VK | variant_bits(n), KS>(pl, ba, stream);
    DENDSN_EACH_UNIT_VARIANT(DENDSN_V)
#undef DENDSN_V
  }
  return hipErrorInvalidValue;
}

hipError_t DENDSN_SG_NAME(launch_bwd_f32_kc)(const Plan& pl, const BwdArgs& ba, int v, hipStream_t stream) {
#define DENDSN_CASE(FAST_, BL_, L_, KC_)                                              \
  if (bool(pl.fast) == FAST_ && pl.BL == BL_ && pl.L == L_ && pl.KC == KC_) {         \
    if (pl.KS == 4) return launch_bwd_kc_v<BL_, L_, KC_, 4>(pl, ba, v, stream); \
    if constexpr (long_stash(BL_, L_, KC_, false))                                                     \
      if (pl.KS == 8) return launch_bwd_kc_v<BL_, L_, KC_, 8>(pl, ba, v, stream); \
    return hipErrorInvalidValue;                                                      \
  }
#define DENDSN_FAST_CASE(BL_, L_, KC_) DENDSN_CASE(true, BL_, L_, KC_)
#define DENDSN_GENERIC_CASE(BL_, L_, KC_) DENDSN_CASE(false, BL_, L_, KC_)
  DENDSN_KC_FAST_F32(DENDSN_FAST_CASE)
  DENDSN_KC_GENERIC(DENDSN_GENERIC_CASE)
#undef DENDSN_FAST_CASE
#undef DENDSN_GENERIC_CASE
#undef DENDSN_CASE
  return hipErrorInvalidValue;
}

}  // namespace dendsn
