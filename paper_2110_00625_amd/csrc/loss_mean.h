// Mean loss of a learner's minibatch, losses[r] = (1/B) sum_m rowloss[r][m], r = k*P + j: one wavefront per r, fixed order.
// Runs as a kernel of its own (sampling_loss.hip) or in workgroups at the end of a round's last update launch
// (gemm_f32.hip, update_bf16.hip), which it does not depend on: a launch is about five microseconds, on small models a tenth
// of a round.
#pragma once
#include "kavg_internal.h"

namespace kavg {

__device__ __forceinline__ void loss_mean_wave(const LossMeans& a, int r, int lane) {
    const float* p = a.rowloss + (long)r * a.B;
    float s = 0.f;
    for (int m = lane; m < a.B; m += 64) s += p[m];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) a.losses[r] = s / (float)a.B;
}

}  // namespace kavg
