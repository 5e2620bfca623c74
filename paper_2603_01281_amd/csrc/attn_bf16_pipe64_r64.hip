// Software-pipelined bf16 attention, head dimension 64: steered kernels for a concatenated rank of at most 64.
#include "attn_bf16_pipe_launch.h"
namespace seka {
hipError_t launch_attention_bf16_pipe64_r64(const AttnArgs& a, const SteerArgs* steer, hipStream_t s) {
  return launch_attention_bf16_pipe_group<64, true, 2>(a, steer, s);
}
}  // namespace seka
