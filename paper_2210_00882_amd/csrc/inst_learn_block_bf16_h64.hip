// bf16 gradient kernel of the learner for hidden size 64
#include "learn_wave_bf16.h"

namespace msrl {

// XT, VEC2 as for the other sizes (learn_block_bf16.h)
hipError_t launch_ppo_block_bf16_h64(int in_dim, const BlockArgsB& a, dim3 grid, hipStream_t s) {
  const bool vec2 = in_dim % 2 == 0 && (uintptr_t)a.obs % 8 == 0;
  const int xt = block_bf16_x_tiles(in_dim);
  const bool wide = a.net[0].out > 8 || a.net[1].out > 8;
  if (in_dim < 1 || xt > 2) return hipErrorInvalidValue;
#define MSRL_WAVE(XT, OT, V) hipLaunchKernelGGL((ppo_wave_bf16_kernel<XT, OT, V>), grid, dim3(WaveShapeB<XT>::THREADS), 0, s, a)
  if (xt == 1 && !wide) {
    if (vec2) MSRL_WAVE(1, 8, true); else MSRL_WAVE(1, 8, false);
  } else if (xt == 1) {
    if (vec2) MSRL_WAVE(1, 16, true); else MSRL_WAVE(1, 16, false);
  } else if (!wide) {
    if (vec2) MSRL_WAVE(2, 8, true); else MSRL_WAVE(2, 8, false);
  } else {
    if (vec2) MSRL_WAVE(2, 16, true); else MSRL_WAVE(2, 16, false);
  }
#undef MSRL_WAVE
  return hipGetLastError();
}

}  // namespace msrl
