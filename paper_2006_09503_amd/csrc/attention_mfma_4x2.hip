// The instances of attention_mfma.hpp for one launch shape (see shape_for in attention_mfma.hip); a file each, so that they compile
// side by side.
#include "attention_mfma.hpp"

namespace k2bw {

hipError_t attention_fwd_mfma_4x2(const AttnDesc& d, const void* qkv, void* o, float* lse, hipStream_t st) {
  return by_head<Fwd, 4, 2>(d, qkv, o, lse, st);
}

hipError_t attention_bwd_mfma_4x2(const AttnDesc& d, const void* qkv, const void* o, const float* lse, const void* d_o, void* dqkv,
                                  float* delta, hipStream_t st) {
  return by_head<Bwd, 4, 2>(d, qkv, o, lse, d_o, dqkv, delta, st);
}

}  // namespace k2bw
