// The one-launch decode step of fp32 caches (a translation unit per element type: each takes over a minute
// to compile).
#include "fused_dev.h"

namespace mpc {

hipError_t launch_decode_step_fp32(const FusedArgs& f, const FusedPlan& p, int D, int G, hipStream_t st) {
  return launch_dt<F32>(f, D, G, p, st);
}

}  // namespace mpc
