// The one-launch decode step of bf16 caches (a translation unit per element type: each takes over a minute
// to compile).
#include "fused_dev.h"

namespace mpc {

hipError_t launch_decode_step_bf16(const FusedArgs& f, const FusedPlan& p, int D, int G, hipStream_t st) {
  return launch_dt<BF16>(f, D, G, p, st);
}

}  // namespace mpc
