// bf16 attention at head dimension 64: dispatch and the register-staged kernels.
#include <cstring>
#include "attn_bf16_launch.h"
namespace seka {
hipError_t launch_attention_bf16_d64(const AttnArgs& a, const SteerArgs* steer, hipStream_t s) {
  return launch_attention_bf16_d<64>(a, steer, s);
}
}  // namespace seka
