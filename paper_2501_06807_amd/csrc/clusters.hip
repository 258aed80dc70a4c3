// Cluster representatives of each fine cluster and super-cluster of the kept cache, gfx950:
// per-channel max / min folded into alpha * r^max + (1 - alpha) * r^min (linear form), or the
// two bound rows (max-product bound), or the average (fp64 sums, one rounding to fp32).
//
// One workgroup per (owner layer, sequence, kv head, super-cluster), over all super-clusters or,
// when a decode-time tail is sealed into a new cluster, over the one super-cluster that holds it.
// Each wave streams the rows of one fine cluster at a time with coalesced 16-byte loads (LPR
// lanes per row), reduces max / min over its row groups with cross-lane shuffles, writes the fine
// representative and folds the bounds into its super-cluster bounds; the waves' super bounds meet
// in LDS. In prefill mode a wave first reads the kept positions of up to 64 rows of its cluster
// (one coalesced load) and takes each row's position from its lane; every row it reads from the
// prompt cache is also written, with its value row, to the kept cache. Max / min are exact,
// the linear representative is two fp32 products and one fp32 sum with no contraction, and the
// average's fp64 sums of 16-bit keys are exact, so their order does not matter. Small super-clusters, where there
// are many, take a wave each (k_build_small).
#include "clusters.h"

namespace mpc {
namespace {

// Bounds (or sums) of a wave's row groups: every lane receives those of its columns over all rows. By shuffles, which
// run on the LDS pipe beside the vector work that bounds a build from the kept cache; the lane swaps of gfx950 are vector
// instructions (256 heads of 4096 rows of 256 B in clusters of four: 148 us with swaps, 133 so).
template <int LPR, int EPL, bool MEAN>
__device__ __forceinline__ void meet(float (&mx)[EPL], float (&mn)[EPL], double (&sum)[EPL]) {
#pragma unroll
  for (int o = LPR; o < kWave; o <<= 1) {
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      if constexpr (MEAN) {
        sum[e] += __shfl_xor(sum[e], o);
      } else {
        mx[e] = fmaxf(mx[e], __shfl_xor(mx[e], o));
        mn[e] = fminf(mn[e], __shfl_xor(mn[e], o));
      }
    }
  }
}

// A lane's columns of a representative over n_tok tokens.
template <int D, int EPL, int SIM>
__device__ __forceinline__ void put_rep(float* out, float alpha, float beta, const float (&mx)[EPL], const float (&mn)[EPL],
                                        const double (&sum)[EPL], int n_tok) {
#pragma clang fp contract(off)
#pragma unroll
  for (int e = 0; e < EPL; ++e) {
    if constexpr (SIM == MPC_SIM_LINEAR) {
      out[e] = alpha * mx[e] + beta * mn[e];
    } else if constexpr (SIM == MPC_SIM_MAXPROD) {
      out[e] = mx[e];
      out[D + e] = mn[e];
    } else {
      out[e] = (float)(sum[e] / (double)n_tok);
    }
  }
}

// Small super-clusters (at most four row loads): a wave takes a whole super-cluster, with all its rows
// requested before any is folded and no barrier. With a workgroup per super-cluster, clusters of four tokens in
// pairs left half of the waves idle and each load waiting for its position: 17 owner layers of 256 heads, 512 kept
// rows each, 720 us; 494 us so (2.7 GB moved, 5.5 TB/s).
constexpr int kSmallLoads = 4;

template <class DT, int D, int NW, int SIM, bool GATHER>
__global__ __launch_bounds__(NW* kWave) void k_build_small(BuildArgs a) {
  constexpr int EPL = DT::kVec;
  constexpr int LPR = D / EPL;
  constexpr int RPW = kWave / LPR;
  constexpr int R = SIM == MPC_SIM_MAXPROD ? 2 : 1;  // representative rows
  constexpr bool MEAN = SIM == MPC_SIM_MEAN;
  constexpr int RB = D * DT::kElt;  // bytes per row
  const int groups = (a.n_sup + NW - 1) / NW;
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
  const int sup = blockIdx.x % groups * NW + w;
  if (sup >= a.n_sup) return;
  const int ou = blockIdx.x / groups;  // (owner index * B + b) * Hkv + h
  const int l = a.own.local(ou / (a.B * a.Hkv));
  const size_t unit = (size_t)l * a.B * a.Hkv + ou % (a.B * a.Hkv);
  const int rg = lane / LPR, li = lane % LPR;
  const int r0 = (a.sup0 + sup) * a.f * a.s, n = min(a.Ts, r0 + a.f * a.s) - r0;  // rows of the super-cluster

  uint4 kr[kSmallLoads];
  if constexpr (GATHER) {
    const int o = owner_layer(a.layer0 + l, a.g.period, a.g.start) - a.layer0;
    const int src_l = o >= 0 ? o : l;  // an owner before the block: the set is already in place
    const size_t src_set = (unit - (size_t)(l - src_l) * a.B * a.Hkv) * a.g.keep, dst_set = unit * a.g.keep;
    int pos = 0;
    if (lane < n) {
      pos = a.g.kept[src_set + r0 + lane];
      if (src_set != dst_set) a.g.kept[dst_set + r0 + lane] = pos;
      pos = min(max(pos, 0), a.g.T - 1);  // positions supplied by the caller are clamped
    }
    uint4 vr[kSmallLoads];
#pragma unroll
    for (int i = 0; i < kSmallLoads; ++i) {
      const int j = i * RPW + rg;
      const size_t so = (unit * a.g.T + __shfl(pos, min(j, n - 1))) * RB + li * 16;
      if (j < n) {
        kr[i] = ldg16((const char*)a.g.k_src + so);
        vr[i] = ldg16((const char*)a.g.v_src + so);
      }
    }
#pragma unroll
    for (int i = 0; i < kSmallLoads; ++i) {
      const int j = i * RPW + rg;
      const size_t dof = (unit * a.rows + r0 + j) * RB + li * 16;
      if (j < n) {
        *(uint4*)((char*)a.g.k_dst + dof) = kr[i];
        *(uint4*)((char*)a.g.v_dst + dof) = vr[i];
      }
    }
  } else {
    const char* kh = (const char*)a.k + ((size_t)unit * a.rows + r0) * RB + li * 16;
#pragma unroll
    for (int i = 0; i < kSmallLoads; ++i)
      if (i * RPW + rg < n) kr[i] = ldg16(kh + (size_t)(i * RPW + rg) * RB);
  }

  float smax[EPL], smin[EPL], cmax[EPL], cmin[EPL];
  double ssum[EPL], csum[EPL];
  auto clear = [](float(&mx)[EPL], float(&mn)[EPL], double(&sum)[EPL]) {
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      mx[e] = -INFINITY;
      mn[e] = INFINITY;
      sum[e] = 0.0;
    }
  };
  clear(smax, smin, ssum);
  clear(cmax, cmin, csum);
  const int per = a.s / RPW;  // loads of a cluster
  int c = (a.sup0 + sup) * a.f, left = per;
#pragma unroll
  for (int i = 0; i < kSmallLoads; ++i) {
    if (i * RPW >= n) break;
    if (i * RPW + rg < n) {
      float x[EPL];
      unpack<DT>(kr[i], x);
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        if constexpr (MEAN) {
          csum[e] += (double)x[e];
        } else {
          cmax[e] = fmaxf(cmax[e], x[e]);
          cmin[e] = fminf(cmin[e], x[e]);
        }
      }
    }
    if (--left == 0 || (i + 1) * RPW >= n) {  // the cluster's last load
      meet<LPR, EPL, MEAN>(cmax, cmin, csum);
      if (rg == 0)
        put_rep<D, EPL, SIM>(a.cent + ((size_t)unit * a.cs + c) * R * D + li * EPL, a.alpha, a.beta, cmax, cmin, csum,
                             min(a.Ts, (c + 1) * a.s) - c * a.s);
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        if constexpr (MEAN) {
          ssum[e] += csum[e];
        } else {
          smax[e] = fmaxf(smax[e], cmax[e]);
          smin[e] = fminf(smin[e], cmin[e]);
        }
      }
      clear(cmax, cmin, csum);
      ++c;
      left = per;
    }
  }
  if (rg == 0)
    put_rep<D, EPL, SIM>(a.scent + ((size_t)unit * a.ss + a.sup0 + sup) * R * D + li * EPL, a.alpha, a.beta, smax, smin,
                         ssum, n);
}

template <class DT, int D, int NW, int SIM, bool GATHER>
__global__ __launch_bounds__(NW* kWave) void k_build(BuildArgs a) {
#pragma clang fp contract(off)
  constexpr int EPL = DT::kVec;
  constexpr int LPR = D / EPL;
  constexpr int RPW = kWave / LPR;
  constexpr int R = SIM == MPC_SIM_MAXPROD ? 2 : 1;  // representative rows
  constexpr bool MEAN = SIM == MPC_SIM_MEAN;
  __shared__ float s_max[NW][D], s_min[NW][D];
  __shared__ double s_sum[MEAN ? NW : 1][MEAN ? D : 1];

  const int sup = a.sup0 + blockIdx.x % a.n_sup;
  const int ou = blockIdx.x / a.n_sup;  // (owner index * B + b) * Hkv + h
  const int l = a.own.local(ou / (a.B * a.Hkv));
  const size_t unit = (size_t)l * a.B * a.Hkv + ou % (a.B * a.Hkv);
  const int tid = threadIdx.x, lane = tid % kWave, w = tid / kWave;
  const int rg = lane / LPR, li = lane % LPR;
  constexpr int RB = D * DT::kElt;  // bytes per row
  const char* kh = (const char*)a.k + (size_t)unit * a.rows * RB;
  // prefill mode: the unit's kept set, prompt rows and kept-cache rows
  size_t src_set = 0, dst_set = 0, src_rows = 0, dst_rows = 0;
  if constexpr (GATHER) {
    const int o = owner_layer(a.layer0 + l, a.g.period, a.g.start) - a.layer0;
    const int src_l = o >= 0 ? o : l;  // an owner before the block: the set is already in place
    src_set = (unit - (size_t)(l - src_l) * a.B * a.Hkv) * a.g.keep;
    dst_set = unit * a.g.keep;
    src_rows = unit * a.g.T;
    dst_rows = unit * a.rows;
  }

  float smax[EPL], smin[EPL];
  double ssum[EPL];
#pragma unroll
  for (int e = 0; e < EPL; ++e) {
    smax[e] = -INFINITY;
    smin[e] = INFINITY;
    ssum[e] = 0.0;
  }
  const int c_end = min(a.C, (sup + 1) * a.f);
  for (int c = sup * a.f + w; c < c_end; c += NW) {
    float cmax[EPL], cmin[EPL];
    double csum[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      cmax[e] = -INFINITY;
      cmin[e] = INFINITY;
      csum[e] = 0.0;
    }
    const int r_end = min(a.Ts, (c + 1) * a.s);
    auto fold = [&](const uint4 raw) {
      float x[EPL];
      unpack<DT>(raw, x);
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        if constexpr (MEAN) {
          csum[e] += (double)x[e];
        } else {
          cmax[e] = fmaxf(cmax[e], x[e]);
          cmin[e] = fminf(cmin[e], x[e]);
        }
      }
    };
    if constexpr (GATHER) {
      for (int r0 = c * a.s; r0 < r_end; r0 += kWave) {
        const int n = min(kWave, r_end - r0);
        int pos = 0;
        if (lane < n) {
          pos = a.g.kept[src_set + r0 + lane];
          if (src_set != dst_set) a.g.kept[dst_set + r0 + lane] = pos;
          pos = min(max(pos, 0), a.g.T - 1);  // positions supplied by the caller are clamped
        }
        for (int j0 = 0; j0 < n; j0 += RPW) {  // wave-uniform trip count: every lane shuffles
          const int j = j0 + rg;
          const int p = __shfl(pos, min(j, n - 1));
          if (j < n) {
            const size_t so = (src_rows + p) * RB + li * 16, dof = (dst_rows + r0 + j) * RB + li * 16;
            const uint4 kr = ldg16((const char*)a.g.k_src + so);
            const uint4 vr = ldg16((const char*)a.g.v_src + so);
            *(uint4*)((char*)a.g.k_dst + dof) = kr;
            *(uint4*)((char*)a.g.v_dst + dof) = vr;
            fold(kr);
          }
        }
      }
    } else {
      for (int r = c * a.s + rg; r < r_end; r += RPW) fold(ldg16(kh + (size_t)r * RB + li * 16));
    }
    meet<LPR, EPL, MEAN>(cmax, cmin, csum);
    if (rg == 0)
      put_rep<D, EPL, SIM>(a.cent + ((size_t)unit * a.cs + c) * R * D + li * EPL, a.alpha, a.beta, cmax, cmin, csum,
                           r_end - c * a.s);
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      if constexpr (MEAN) {
        ssum[e] += csum[e];
      } else {
        smax[e] = fmaxf(smax[e], cmax[e]);
        smin[e] = fminf(smin[e], cmin[e]);
      }
    }
  }
  if (rg == 0) {
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      if constexpr (MEAN) {
        s_sum[w][li * EPL + e] = ssum[e];
      } else {
        s_max[w][li * EPL + e] = smax[e];
        s_min[w][li * EPL + e] = smin[e];
      }
    }
  }
  __syncthreads();
  const int n_tok = min(a.Ts, c_end * a.s) - sup * a.f * a.s;  // tokens of the super-cluster
  float* sout = a.scent + ((size_t)unit * a.ss + sup) * R * D;
  for (int i = tid; i < D; i += NW * kWave) {
    if constexpr (MEAN) {
      double sum = 0.0;
#pragma unroll
      for (int j = 0; j < NW; ++j) sum += s_sum[j][i];
      sout[i] = (float)(sum / (double)n_tok);
    } else {
      float mx = -INFINITY, mn = INFINITY;
#pragma unroll
      for (int j = 0; j < NW; ++j) {
        mx = fmaxf(mx, s_max[j][i]);
        mn = fminf(mn, s_min[j][i]);
      }
      if constexpr (SIM == MPC_SIM_LINEAR) {
        sout[i] = a.alpha * mx + a.beta * mn;
      } else {
        sout[i] = mx;
        sout[D + i] = mn;
      }
    }
  }
}

template <class DT, int D, int SIM, bool GATHER>
void launch_shape(const BuildArgs& a, hipStream_t st) {
  constexpr int NW = 4, RPW = kWave * DT::kVec / D;  // rows per load of a wave
  const int heads = a.own.n * a.B * a.Hkv;
  if (small_build(a, RPW))
    hipLaunchKernelGGL((k_build_small<DT, D, NW, SIM, GATHER>), dim3(heads * ((a.n_sup + NW - 1) / NW)), dim3(NW * kWave),
                       0, st, a);
  else
    hipLaunchKernelGGL((k_build<DT, D, NW, SIM, GATHER>), dim3(heads * a.n_sup), dim3(NW * kWave), 0, st, a);
}

template <class DT, int D, bool GATHER>
void launch_sim(const BuildArgs& a, hipStream_t st) {
  if (a.similarity == MPC_SIM_MAXPROD)
    launch_shape<DT, D, MPC_SIM_MAXPROD, GATHER>(a, st);
  else if (a.similarity == MPC_SIM_MEAN)
    launch_shape<DT, D, MPC_SIM_MEAN, GATHER>(a, st);
  else
    launch_shape<DT, D, MPC_SIM_LINEAR, GATHER>(a, st);
}

template <class DT, int D>
void launch_mode(const BuildArgs& a, hipStream_t st) {
  if (a.g.kept)
    launch_sim<DT, D, true>(a, st);
  else
    launch_sim<DT, D, false>(a, st);
}

template <class DT>
hipError_t launch_dt(const BuildArgs& a, int D, hipStream_t st) {
  if (D == 64)
    launch_mode<DT, 64>(a, st);
  else if (D == 128)
    launch_mode<DT, 128>(a, st);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace

// A wave takes its clusters one after the other, which only many super-clusters hide. Up to two clusters leave half of a
// workgroup idle, so from as many super-clusters on as workgroups are resident at once (eight to a compute unit);
// three or four only from the size on where the whole build is bound by its instructions. A sealed tail rebuilds one
// super-cluster per head, which a workgroup of such waves would leave idle. Builds from the kept cache, us, a workgroup
// and a wave per super-cluster: pairs of four tokens of 256 B, 512 super-clusters 3.7 and 4.1, 2048 5.5 and 4.9, 131072
// 187 and 120; fours of eight tokens of 128 B, 4096 13.3 and 13.1 (gathered, with the passes, 49.3 and 53.8), 32768 77.5
// and 70.6 (259 and 248); fours of four of 256 B, 128 3.3 and 5.3, 65536 133 and 116.
bool small_build(const BuildArgs& a, int rpw) {
  return a.f <= kSmallLoads * rpw / a.s && a.s % rpw == 0 && a.n_sup > 1 &&
         (int64_t)a.own.n * a.B * a.Hkv * a.n_sup >= (a.f <= 2 ? 8 : 128) * (int64_t)kNumCU;
}

hipError_t launch_build(const BuildArgs& a, int dtype, int D, hipStream_t st) {
  switch (dtype) {
    case MPC_FP32: return launch_dt<F32>(a, D, st);
    case MPC_FP16: return launch_dt<F16>(a, D, st);
    case MPC_BF16: return launch_dt<BF16>(a, D, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace mpc
