// Sparse decode attention over the selected clusters (gather + online softmax), gfx950.
//
// One work unit = (layer, sequence, kv head). Its token list is the concatenation of the
// selected clusters' rows of the kept cache. A unit may be split over several workgroups
// (split-K); each writes an (m, l, acc) partial and the last one to finish merges them.
//
// Lane layout: a K/V row of d elements is read as 16-byte vectors by LPR consecutive lanes, so a
// wave reads RPW = 64 / LPR rows per load instruction, fully coalesced. The G query heads of the
// group are served from the same loaded rows. Scores are kept in log2 units (q is pre-scaled by
// sm_scale * log2 e) so the softmax uses the hardware exp2. V rows are loaded with the
// non-temporal hint; K rows too when the decode step's working set passes the memory-side cache
// (DecodeArgs::stream_k, a template variant).
#include "decode_dev.h"

namespace mpc {
namespace {

template <class DT, int D, int G, int NW, int U, bool STREAM_K>
__global__ __launch_bounds__(NW* kWave) void k_sparse_decode(DecodeArgs a) {
  dev::attend<DT, D, G, NW, U, false, STREAM_K>(a, blockIdx.x / a.splits, blockIdx.x % a.splits);
}

constexpr int kUnitWaves = 4;  // units (waves) per workgroup of the wave form

// One query head over 16-bit rows fits 64 registers, so that 32 units run on a compute unit at once: 8192 units of 48
// rows are then one round (36.2 us at 70 registers, 34.4 at 64).

template <class DT, int D, int G, int U, bool STREAM_K>
__global__ __launch_bounds__(kUnitWaves* kWave, G == 1 && DT::kElt == 2 ? 8 : 1) void k_sparse_decode_wave(DecodeArgs a, int units) {
  __shared__ int32_t s_sel[kUnitWaves][kMaxWaveList];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int unit = blockIdx.x * kUnitWaves + w;
  if (unit < units) dev::attend_wave<DT, D, G, U, STREAM_K>(a, unit, s_sel[w]);
}

template <class DT, int D, int G>
hipError_t launch_dt_d_g(const DecodeArgs& a, int units, const DecodePlan& p, hipStream_t st) {
  if constexpr (G <= 2) {
    if (p.waves == 1) {
      const dim3 grid((units + kUnitWaves - 1) / kUnitWaves), block(kUnitWaves * kWave);
      if (a.stream_k)
        hipLaunchKernelGGL((k_sparse_decode_wave<DT, D, G, 4, true>), grid, block, 0, st, a, units);
      else
        hipLaunchKernelGGL((k_sparse_decode_wave<DT, D, G, 4, false>), grid, block, 0, st, a, units);
      return hipGetLastError();
    }
  }
  if (a.stream_k)
    hipLaunchKernelGGL((k_sparse_decode<DT, D, G, 8, 4, true>), dim3(units * a.splits), dim3(8 * kWave), 0, st, a);
  else
    hipLaunchKernelGGL((k_sparse_decode<DT, D, G, 8, 4, false>), dim3(units * a.splits), dim3(8 * kWave), 0, st, a);
  return hipGetLastError();
}

template <class DT, int D>
hipError_t launch_dt_d(const DecodeArgs& a, int G, int units, const DecodePlan& p, hipStream_t st) {
  switch (G) {
    case 1: return launch_dt_d_g<DT, D, 1>(a, units, p, st);
    case 2: return launch_dt_d_g<DT, D, 2>(a, units, p, st);
    case 4: return launch_dt_d_g<DT, D, 4>(a, units, p, st);
    case 8: return launch_dt_d_g<DT, D, 8>(a, units, p, st);
  }
  return hipErrorInvalidValue;
}

template <class DT>
hipError_t launch_dt(const DecodeArgs& a, int D, int G, int units, const DecodePlan& p, hipStream_t st) {
  if (D == 64) return launch_dt_d<DT, 64>(a, G, units, p, st);
  if (D == 128) return launch_dt_d<DT, 128>(a, G, units, p, st);
  return hipErrorInvalidValue;
}

}  // namespace

DecodePlan decode_plan(int units, int n_slot, int s, int D, int elt, int G) {
  // One 8-wave workgroup per unit when there are at least as many units as CUs; otherwise the
  // token list of each unit may be split over several workgroups (at most about two per CU).
  DecodePlan p;
  p.waves = 8;
  p.splits = p.most = 1;
  if (units < kNumCU) {
    const int lpr = D * elt / 16;
    const int rows_per_pass = p.waves * (kWave / lpr);
    int max_splits = n_slot / rows_per_pass;
    if (max_splits < 1) max_splits = 1;
    p.most = (2 * kNumCU + units - 1) / units;
    if (p.most > max_splits) p.most = max_splits;
    if (p.most > kMaxSplits) p.most = kMaxSplits;
    // Cost of a split count in twentieths of a step (a workgroup's pass over its rows, about 1.15 us): the steps, dearer
    // where a compute unit holds several workgroups, and for a split its partial's stores, the arrival and the merge
    // (three memory round trips, about two steps). So lists of up to three steps stay whole, longer ones become splits of
    // one step while each has a compute unit to itself. The weights are a fit to 900 measured blocks of 1 to 240 units
    // and 128 to 3200 rows of all types, both head dims and 1 to 8 query heads (attention within 2% of the best count on
    // average). us per launch, splits in parentheses:
    //   32 units of 384 rows of 256 B        8.9 (12)   6.2 (3)   5.7 (1)
    //   32 units of 1600 rows of 256 B       9.5 (16)   8.4 (7)  11.1 (3)  17.9 (1)
    //   128 units of 400 rows of 256 B, G=4 10.0 (4)   12.2 (3)   9.4 (2)  10.0 (1)  (fp32)
    //   144 units of 128 rows of 128 B       7.0 (4)    4.4 (1)
    //   4 units of 1600 rows of 256 B        6.4 (14)   7.9 (6)  13.3 (1)
    //   1 unit of 640 rows of 256 B          6.1 (16)   5.5 (5)   6.9 (1)
    const int64_t step = G == 4 && elt == 2 ? p.waves * 16 : 4 * rows_per_pass;  // rows, as the kernels take them
    int64_t best = 0;
    for (int sp = 1; sp <= p.most; ++sp) {
      const int per_cu = (units * sp + kNumCU - 1) / kNumCU;
      int64_t cost = ((n_slot + sp - 1LL) / sp + step - 1) / step * (20 + 35 * (per_cu - 1));
      if (sp > 1) cost += 37 + sp;
      if (per_cu > 1) cost += 10;
      if (sp == 1 || cost < best) {
        best = cost;
        p.splits = sp;
      }
    }
  }
  // Many units with short lists: a wave each. A workgroup's pass is 32 KiB of K rows (8 waves of 4 loads of
  // 1 KiB); a list of at most half of that leaves half of its lanes without a row, beside its barrier and the
  // merge of its waves. us per launch, workgroup and wave form: 8192 units of 48 rows of 256 B 54.7 and 34.4, of 64
  // rows 54.7 and 44.1, of 96 66.1 and 67.5, of 128 83.3 and 88.5; 4096 of 64 27.4 and 23.1; 8192 of 48 rows of
  // 128 B 46.6 and 19.8, of 128 53.6 and 43.1; 1024 of 48 rows of 256 B 9.3 and 9.3.
  if (G <= 2 && p.splits == 1 && units >= 4 * kNumCU && (int64_t)n_slot * D * elt <= (16 << 10) &&
      n_slot <= (int64_t)kMaxWaveList * s)
    p.waves = 1;
  return p;
}

hipError_t launch_sparse_decode(const DecodeArgs& a, int dtype, int D, int G, int units, const DecodePlan& p,
                                hipStream_t st) {
  switch (dtype) {
    case MPC_FP32: return launch_dt<F32>(a, D, G, units, p, st);
    case MPC_FP16: return launch_dt<F16>(a, D, G, units, p, st);
    case MPC_BF16: return launch_dt<BF16>(a, D, G, units, p, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace mpc
