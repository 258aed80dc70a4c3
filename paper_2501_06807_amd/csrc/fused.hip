// Plan and dispatch of the one-launch decode step (kernels in fused_dev.h).
#include "fused.h"

#include "decode_dev.h"
#include "select_dev.h"

namespace mpc {

FusedPlan fused_plan(const SelectArgs& s, int D, int splits) {
  FusedPlan p{};
  p.units = s.n_layers * s.B * s.Hsel;
  p.smem = dev::select_smem_bytes_dev(D, s.S, s.NC, select_query_rows(s));
  p.self = (int64_t)p.units * splits <= kNumCU;
  return p;
}

bool fused_fits(const FusedPlan& p, int D, int G) {
  // the attention's static LDS: selection ids, per-wave (m, l) and partial outputs, a few words;
  // the self-selecting form holds its selection ids once more
  const size_t att = 4 * dev::kMaxSel * (p.self ? 2 : 1) + (size_t)kFusedWaves * G * (2 + D) * 4 + 64;
  return p.smem + att <= kMaxLds;
}

hipError_t launch_decode_step(const FusedArgs& f, const FusedPlan& p, int dtype, int D, int G,
                              hipStream_t st) {
  switch (dtype) {
    case MPC_FP32: return launch_decode_step_fp32(f, p, D, G, st);
    case MPC_FP16: return launch_decode_step_fp16(f, p, D, G, st);
    case MPC_BF16: return launch_decode_step_bf16(f, p, D, G, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace mpc
