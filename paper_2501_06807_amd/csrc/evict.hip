// Look-once static eviction on gfx950: accumulated window attention, top-k, gather.
//
// The accumulated attention of key j is A[j] = sum over the group's window rows t of
// softmax_j(sm_scale * q_t . k_j). It needs every row's normaliser before any column can be
// summed, so it takes two passes over the scores, both on the matrix cores (16-bit inputs:
// v_mfma_f32_16x16x32_{bf16,f16}; fp32 inputs: v_mfma_f32_32x32x2f32):
//   pass 1 (k_rowstats16 for 16-bit inputs, k_rowstats for fp32): window rows stay in registers as the
//     B operand, key tiles stream through LDS as the A operand; each lane owns one query column of its
//     blocks, so a row's sum needs no exchange until the end. Output per row: a whole-number
//     offset b with every exponent fma(c, s, b) at most 1 (b = -ceil(fp32(c * m)) for fp32 inputs, m the
//     row max), and 1 / sum of exp2(fma(c, s, b)), c = fp32(sm_scale * log2(e)). A row block's keys
//     may be split over several workgroups (row_splits), whose sums k_rowmerge brings together.
//   pass 2 (k_colsum16 for 16-bit inputs, k_colsum for fp32): keys stay in registers as the B
//     operand, window-row tiles (all query heads of the group) stream through LDS as the A
//     operand; each lane owns one key column, so the column sum needs no exchange within a tile.
//     p = exp2(fma(c, s, b)) / sum, summed over a lane's rows of a tile in fp32 and accumulated
//     across tiles in fp64. A key block's window rows may be split over several workgroups (col_splits),
//     whose sums k_colmerge brings together. For 16-bit inputs both passes take 64-row (64-key) tiles, so that a
//     barrier serves 64 rows. Both passes form the exponent with one fused multiply-add
//     against the same offset, so the offset is a common factor of a row's terms and of its sum
//     and cancels in p; it only has to keep the exponents of the large terms small. Being a whole
//     number, a move of the offset rescales pass 1's sums by an exact power of two (ldexp). The
//     exponents of the terms near the max lie in (-1, 1], so their rounding, and that of c
//     (proportional to |c * (s - m)|), stay smallest on the terms that carry the sums.
// The top-k is an 8-bit LDS radix select on the fp32 score bits followed by an ordered block
// compaction, each thread's run of scores held in registers up to 32K older tokens; the
// gather copies kept rows with 16-byte lanes (all layers, or those whose representatives are not
// built in the same pass).
#include "evict.h"

#include <algorithm>
#include <type_traits>

namespace mpc {
namespace {

typedef float f32x16 __attribute__((__vector_size__(16 * sizeof(float))));
typedef __bf16 bf16x8 __attribute__((__vector_size__(8 * sizeof(__bf16))));
typedef _Float16 f16x8 __attribute__((__vector_size__(8 * sizeof(_Float16))));

// 32x32x2 matrix-core operations of fp32 inputs on a 16-byte vector per lane: lane l feeds row (l % 32) of A /
// column (l % 32) of B with the (l / 32)-th half of eight elements, four two-wide steps; any assignment of
// elements to steps works as long as A and B share it.
__device__ __forceinline__ f32x16 mma32(float4 a, float4 b, f32x16 c) {
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b.x, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b.y, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, b.z, c, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, b.w, c, 0, 0, 0);
}

// 16x16x32 matrix-core operation for 16-bit inputs: lane l feeds row (l % 16) of A / column
// (l % 16) of B with the k-slice [(l / 16) * 8, + 8) of each 32-wide step, and receives the output
// rows 4 (l / 16) + r, r = 0..3, of column l % 16.
typedef float f32x4 __attribute__((__vector_size__(4 * sizeof(float))));
template <class DT>
__device__ __forceinline__ f32x4 mma16(uint4 a, uint4 b, f32x4 c);
template <>
__device__ __forceinline__ f32x4 mma16<BF16>(uint4 a, uint4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
template <>
__device__ __forceinline__ f32x4 mma16<F16>(uint4 a, uint4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// Row of the 32x32 output held in accumulator register r of `lane` (the column is lane % 32).
__device__ __forceinline__ int acc_row(int r, int lane) {
  return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
}

// Workgroup ids are dealt round-robin over the dies; renumber them so that each die gets one
// contiguous range of work items (all tiles of a head share that die's L2).
__device__ __forceinline__ int xcd_remap(int bid, int n) {
  const int q = n / kNumXcd, r = n % kNumXcd;
  const int x = bid % kNumXcd, slot = bid / kNumXcd;
  return x < r ? x * (q + 1) + slot : r * (q + 1) + (x - r) * q + slot;
}

// Column-pass workgroup: its unit (owner head and row split) and key block.
struct ColItem {
  int unit, kb;
};

// Item `id` of the 16-bit column pass, n_kb key blocks to each of n units. Units come in groups of a.col_group: the
// blocks that every window row sees, unit by unit, then those that end inside the window (half the work on average),
// block by block over the group. So a die's last workgroups, which run few to a compute unit, are short ones.
// Prefill of one layer of 7177 tokens and 32 heads (928 workgroups, three to a unit at once) 241.2 -> 236.5 us, of
// eight prompts of 1024 tokens and 32 layers 1681 -> 1624 us, of 8192 tokens and 32 layers 2871 us both.
__device__ __forceinline__ ColItem col_item(const EvictArgs& a, int id, int n, int n_kb) {
  if (a.col_group == 1) return {id / n_kb, id % n_kb};
  const int seen = a.causal ? (a.T - a.W + 1) / kColBlockKeys : n_kb;  // blocks that the first window row sees whole
  const int first = id / (a.col_group * n_kb) * a.col_group;
  const int units = min(a.col_group, n - first);
  const int i = id - first * n_kb, tail = i - units * seen;
  if (tail < 0) return {first + i / seen, i % seen};
  return {first + tail % units, seen + tail / units};
}

// Tiles of ROWS rows of a [rows][D] matrix staged through LDS with 16-byte chunks; the row stride
// is padded by 16 bytes to spread the rows of a fragment read over the LDS banks.
template <class DT, int D, int NT = 256, int ROWS = 32>
struct Tile {
  static constexpr int RB = D * DT::kElt;
  static constexpr int RS = RB + 16;
  static constexpr int CH = RB / 16;
  static constexpr int CHUNKS = ROWS * CH;
  static constexpr int PER = (CHUNKS + NT - 1) / NT;  // chunks per thread (NT threads)
  static constexpr int BYTES = ROWS * RS;
};

// The PER 16-byte chunks a thread stages from each tile: chunk i is row row(i) of the tile, at byte
// mem(i) from the tile's first row in memory and byte lds(i) of an LDS buffer. The threads cover whole
// rows, so the chunks of a thread are a fixed number of rows apart: one offset each and constant strides
// (one register instead of one per chunk; the row and column passes hold 168 at most).
template <class TL, int NT>
struct TileChunks {
  static_assert(NT % TL::CH == 0, "the threads cover whole rows");
  static constexpr int STEP = NT / TL::CH;  // rows between a thread's chunks
  int tid;
  unsigned row0, mem0, lds0;
  __device__ explicit TileChunks(int t) : tid(t) {
    row0 = t / TL::CH;
    mem0 = row0 * TL::RB + (t % TL::CH) * 16;
    lds0 = row0 * TL::RS + (t % TL::CH) * 16;
  }
  __device__ int row(int i) const { return row0 + i * STEP; }
  __device__ unsigned mem(int i) const { return mem0 + i * STEP * TL::RB; }
  __device__ unsigned lds(int i) const { return lds0 + i * STEP * TL::RS; }
  // whether chunk i exists (always, when the threads cover the tile's chunks exactly)
  __device__ bool ok(int i) const { return (i + 1) * NT <= TL::CHUNKS || tid + i * NT < TL::CHUNKS; }
};

// Waves of the fp32 passes, one 32-row (32-key) block each: eight (256 rows or keys to a workgroup), or in the column
// pass two when that many workgroups would leave most compute units idle (launch_pass).
constexpr int kWaves32 = 8, kFewWaves32 = 2;
static_assert(kRowBlock == kColBlockKeys && kRowBlock == 32 * kWaves32, "both passes cover 256 rows / keys");

// A row's offset before its first score: every term is then infinite, so that the offset moves, but a score of
// -infinity already adds nothing.
constexpr float kNoOffset = 3.4028234664e38f;

// Part of a row's sum moved to a smaller offset (exact). A part without terms stays zero and NaN, which a NaN score
// leaves, stays NaN, so that a row that sees one is NaN however its keys are divided over lanes and workgroups.
__device__ __forceinline__ double moved(double sum, double from, double to) {
  return sum > 0.0 ? ldexp(sum, (int)(to - from)) : sum;
}

// A window row's statistics: offset o and sum L of exp2(fma(c, s, o)) over its visible keys.
__device__ __forceinline__ void put_stat(const EvictArgs& a, size_t row, double L, float o) {
  a.rowstat[row] = make_float2(o, (float)(1.0 / L));
  // log-sum-exp of the scaled scores: log2 of sum exp2(c * s) = log2(L) - offset
  if (a.row_lse) a.row_lse[row] = (float)((log2(L) - (double)o) * 0.69314718055994531);
}

// The same from one workgroup of owner head ou: final, or the partial of key split sp.
__device__ __forceinline__ void put_row(const EvictArgs& a, int ou, size_t row0, int sp, int t, double L, float o) {
  if (a.splits == 1)
    put_stat(a, row0 + t, L, o);
  else
    a.part[((size_t)ou * a.splits + sp) * a.W + t] = make_double2(L, (double)o);
}

// Key j's accumulated attention from one workgroup of owner head ou: final, or the part of row split sp.
__device__ __forceinline__ void put_score(const EvictArgs& a, int ou, size_t unit, int sp, int j, double sum) {
  if (a.col_splits == 1)
    a.score[unit * a.T + j] = (float)sum;
  else
    a.col_part[((size_t)ou * a.col_splits + sp) * a.T + j] = sum;
}

// Row pass on 32x32 matrix instructions (fp32 inputs; 16-bit inputs take k_rowstats16 below):
// the offset follows the running max, so every exponent is at most 0.
template <class DT, int D>
__global__ __launch_bounds__(kWaves32* kWave) void k_rowstats(EvictArgs a) {
  constexpr int NT = kWaves32 * kWave;
  using TL = Tile<DT, D, NT>;
  constexpr int KS = D / 8;
  static_assert(DT::kElt == 4, "16-bit inputs take k_rowstats16");
  __shared__ __align__(16) unsigned char s_k[2][TL::BYTES];

  const int n_rb = (a.W + kRowBlock - 1) / kRowBlock;
  const int id = xcd_remap(blockIdx.x, gridDim.x);
  const int rb = id % n_rb, sp = id / n_rb % a.splits;
  const int ou = id / n_rb / a.splits;  // (owner index * B + b) * Hq + hq
  const int l = a.own.local(ou / (a.B * a.Hq));
  const int b = (ou / a.Hq) % a.B, hq = ou % a.Hq;
  const size_t qunit = ((size_t)l * a.B + b) * a.Hq + hq;
  const int G = a.Hq / a.Hkv;
  const size_t kvunit = ((size_t)l * a.B + b) * a.Hkv + hq / G;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, c32 = lane & 31, hl = lane >> 5;

  // this wave holds window rows row0 .. + 31; lane column c32 is row t
  const int row0 = rb * kRowBlock + w * 32, t = row0 + c32;
  const int tcl = t < a.W ? t : a.W - 1, pos = a.T - a.W + tcl;
  float4 qf[KS];
  const char* qrow = (const char*)a.q_win + ((size_t)qunit * a.W + tcl) * TL::RB;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) qf[ks] = *(const float4*)(qrow + ks * 32 + hl * 16);

  const char* kh = (const char*)a.k + kvunit * a.T * TL::RB;
  const int last_row = min(a.W - 1, rb * kRowBlock + kRowBlock - 1);
  const int jend = a.causal ? min(a.T, a.T - a.W + last_row + 1) : a.T;
  const int ntile = (jend + 31) / 32, per = (ntile + a.splits - 1) / a.splits;
  const int it0 = min(sp * per, ntile), it1 = min(it0 + per, ntile);  // this split's tiles

  const TileChunks<TL, NT> tc(tid);
  uint4 pre[TL::PER];
  // key tiles lying wholly inside the cache load without per-chunk row tests or zero fills
  auto fetch = [&](int tile) {
    const char* tb = kh + (size_t)tile * (32 * TL::RB);
    if (tile * 32 + 32 <= a.T) {
#pragma unroll
      for (int i = 0; i < TL::PER; ++i)
        if (tc.ok(i)) pre[i] = ldg16(tb + tc.mem(i));
    } else {
#pragma unroll
      for (int i = 0; i < TL::PER; ++i)
        pre[i] = tc.ok(i) && tile * 32 + tc.row(i) < a.T ? ldg16(tb + tc.mem(i)) : make_uint4(0, 0, 0, 0);
    }
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int i = 0; i < TL::PER; ++i)
      if (tc.ok(i)) *(uint4*)&s_k[buf][tc.lds(i)] = pre[i];
  };
  if (it0 < it1) {
    fetch(it0);
    stash(0);
  }
  // the row operands are in registers before the loop, so that no wait for them lands inside it
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  const float cf = a.c32;
  float m = -INFINITY, nb = kNoOffset;  // running max and its whole-number offset -ceil(c * m)
  double ell = 0.0;                    // sum of exp2(fma(c, s, nb)) so far
  for (int it = it0; it < it1; ++it) {
    const int buf = (it - it0) & 1;
    if (it + 1 < it1) fetch(it + 1);
    f32x16 acc = {};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      acc = mma32(*(const float4*)&s_k[buf][c32 * TL::RS + ks * 32 + hl * 16], qf[ks], acc);
    const int j0 = it * 32;
    // a tile wholly inside the causal triangle and the key range needs no per-element mask
    // (uniform over the wave: the block's smallest row bounds every row's last visible key)
    const bool full = j0 + 31 < a.T && (!a.causal || j0 + 31 <= a.T - a.W + row0);
    float tmax = -INFINITY;
    if (full) {
#pragma unroll
      for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, acc[r]);
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int j = j0 + acc_row(r, lane);
        if (j < a.T && (!a.causal || j <= pos)) tmax = fmaxf(tmax, acc[r]);
      }
    }
    if (tmax > m) {
      // offsets are whole numbers, so moving one rescales the sum by a power of two (exact)
      const float nb_new = -ceilf(cf * tmax);
      if (ell > 0.0 && nb_new != nb) ell = ldexp(ell, (int)(nb_new - nb));
      m = tmax;
      nb = nb_new;
    }
    float ps = 0.f;
    if (full) {
#pragma unroll
      for (int r = 0; r < 16; ++r) ps += fast_exp2(fmaf(cf, acc[r], nb));
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int j = j0 + acc_row(r, lane);
        if (j < a.T && (!a.causal || j <= pos)) ps += fast_exp2(fmaf(cf, acc[r], nb));
      }
    }
    ell += (double)ps;
    if (it + 1 < it1) stash(buf ^ 1);
    __syncthreads();
  }
  // the two half-waves' sums meet at the offset of the larger max (the smaller offset)
  const double eo = __shfl_xor(ell, 32);
  const float nbo = __shfl_xor(nb, 32);
  const float nbx = fminf(nb, nbo);
  const double L = moved(ell, nb, nbx) + moved(eo, nbo, nbx);
  if (hl == 0 && t < a.W) put_row(a, ou, (size_t)qunit * a.W, sp, t, L, nbx);
}

// Column pass on 32x32 matrix instructions (fp32 inputs; 16-bit inputs take k_colsum16 below).
template <class DT, int D, int WAVES>
__global__ __launch_bounds__(WAVES* kWave) void k_colsum(EvictArgs a) {
  constexpr int NT = WAVES * kWave, KEYS = 32 * WAVES;
  using TL = Tile<DT, D, NT>;
  constexpr int KS = D / 8;
  static_assert(DT::kElt == 4, "16-bit inputs take k_colsum16");
  __shared__ __align__(16) unsigned char s_q[2][TL::BYTES];
  __shared__ __align__(16) float s_nb[2][32], s_il[2][32];  // offset and 1 / sum of the staged rows

  const int n_kb = (a.T + KEYS - 1) / KEYS;
  const int id = xcd_remap(blockIdx.x, gridDim.x);
  const int kb = id % n_kb, sp = id / n_kb % a.col_splits;
  const int ou = id / n_kb / a.col_splits;  // (owner index * B + b) * Hkv + h
  const int l = a.own.local(ou / (a.B * a.Hkv));
  const int b = (ou / a.Hkv) % a.B, h = ou % a.Hkv;
  const size_t kvunit = ((size_t)l * a.B + b) * a.Hkv + h;
  const int G = a.Hq / a.Hkv;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, c32 = lane & 31, hl = lane >> 5;

  // this wave holds keys jw .. + 31; lane column c32 is key jw + c32
  const int jw = kb * KEYS + w * 32, j = jw + c32;
  const float cf = a.c32;
  const char* krow = (const char*)a.k + ((size_t)kvunit * a.T + min(j, a.T - 1)) * TL::RB;
  float4 kf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) kf[ks] = *(const float4*)(krow + ks * 32 + hl * 16);

  const int j_lo = kb * KEYS;
  const int t_start = a.causal ? (max(0, j_lo - (a.T - a.W)) & ~31) : 0;
  const int n_t = (a.W - t_start + 31) / 32;
  const int ntile = G * n_t, per = (ntile + a.col_splits - 1) / a.col_splits;
  const int it0 = min(sp * per, ntile), it1 = min(it0 + per, ntile);  // this split's tiles
  const size_t qunit0 = ((size_t)l * a.B + b) * a.Hq + (size_t)h * G;

  const TileChunks<TL, NT> tc(tid);
  uint4 pre[TL::PER];
  float2 pre_b = make_float2(0.f, 0.f);
  // tiles run through the group's heads, each from row t_start to t_end; the next one to fetch is
  // head fg's rows ft0 .. ft0 + 31 (a counter, not a division per tile)
  const int t_end = t_start + n_t * 32;
  int fg = it0 / n_t, ft0 = t_start + it0 % n_t * 32;
  int t0 = ft0;  // first window row of the tile being scored
  auto fetch = [&]() {
    const size_t r0 = (qunit0 + fg) * a.W + ft0;
    const char* tb = (const char*)a.q_win + r0 * TL::RB;
    if (ft0 + 32 <= a.W) {
#pragma unroll
      for (int i = 0; i < TL::PER; ++i)
        if (tc.ok(i)) pre[i] = ldg16(tb + tc.mem(i));
    } else {
#pragma unroll
      for (int i = 0; i < TL::PER; ++i)
        pre[i] = tc.ok(i) && ft0 + tc.row(i) < a.W ? ldg16(tb + tc.mem(i)) : make_uint4(0, 0, 0, 0);
    }
    if (tid < 32) pre_b = ft0 + tid < a.W ? a.rowstat[r0 + tid] : make_float2(0.f, 0.f);
    ft0 += 32;
    if (ft0 == t_end) {
      ft0 = t_start;
      ++fg;
    }
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int i = 0; i < TL::PER; ++i)
      if (tc.ok(i)) *(uint4*)&s_q[buf][tc.lds(i)] = pre[i];
    if (tid < 32) {
      s_nb[buf][tid] = pre_b.x;
      s_il[buf][tid] = pre_b.y;
    }
  };
  if (it0 < it1) {
    fetch();
    stash(0);
  }
  // the key operands are in registers before the loop, so that no wait for them lands inside it
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  double cacc = 0.0;
  for (int it = it0; it < it1; ++it) {
    const int buf = (it - it0) & 1;
    if (it + 1 < it1) fetch();
    f32x16 acc = {};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      acc = mma32(*(const float4*)&s_q[buf][c32 * TL::RS + ks * 32 + hl * 16], kf[ks], acc);
    // every row of the tile valid and every key of the wave visible to its first row
    const bool full = t0 + 31 < a.W && (!a.causal || jw + 31 <= a.T - a.W + t0);
    float ps = 0.f;
    if (full) {
      // the tile's rows of this lane: 8 g + 4 hl + (0..3), g = 0..3, read four at a time
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const float4 nb4 = *(const float4*)&s_nb[buf][8 * g4 + 4 * hl];
        const float4 il4 = *(const float4*)&s_il[buf][8 * g4 + 4 * hl];
        const float nbv[4] = {nb4.x, nb4.y, nb4.z, nb4.w}, ilv[4] = {il4.x, il4.y, il4.z, il4.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) ps = fmaf(fast_exp2(fmaf(cf, acc[4 * g4 + q], nbv[q])), ilv[q], ps);
      }
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int rr = acc_row(r, lane);
        const int trow = t0 + rr;
        if (trow < a.W && (!a.causal || j <= a.T - a.W + trow))
          ps = fmaf(fast_exp2(fmaf(cf, acc[r], s_nb[buf][rr])), s_il[buf][rr], ps);
      }
    }
    cacc += (double)ps;
    if (it + 1 < it1) stash(buf ^ 1);
    t0 = t0 + 32 == t_end ? t_start : t0 + 32;
    __syncthreads();
  }
  const double tot = cacc + __shfl_xor(cacc, 32);
  if (hl == 0 && j < a.T) put_score(a, ou, kvunit, sp, j, tot);
}

// Row pass for 16-bit inputs on 16x16x32 matrix instructions. A wave holds 64 window rows in
// registers as four 16-row B operands (query groups) and takes each 64-key tile from LDS as four
// 16-key A operands, so a tile is sixteen 16x16 blocks; a lane holds keys 4 (lane / 16) + r of one
// row per block. Each block's exponentials are taken against the row's current offset, with no
// running max, beside the next block's matrix chain (one basic block, so the two interleave). A
// block whose four terms sum to at most 2 has every exponent at most 1, as accurate as an offset
// at the max; a larger sum takes the slow path: the offset moves to the block's max if that is
// higher (the running sums rescaled by an exact power of two) and the block is summed again. The
// four lanes of a row meet once at the end at the smallest offset, so no exponent of pass 2 exceeds 1.
//
// 32x32x16 blocks in a written-out order, with their offsets checked once per tile of 64 keys, were faster (a prefill of
// 32 x 8192 keys by 5%, of 12 layers of 2048 keys of 64 channels by a fifth) only while exponents up to 5 were let
// through, which doubled the largest error of a score on peaked rows. Held to exponents of at most 1 they were no
// faster (eviction of eight layers of 8192 keys and 32 heads: 1880 us here, 1898 us so; with scores of three times the
// spread 1944 and 2104 us).
//
// What bounds it beside the column pass's causes: the slow path. The four lanes of a row keep offsets of their own, and in
// the first tiles of a row or split a wave often holds a lane whose block exceeds its own: 84 heads of 2048 keys of
// 64 channels in three splits run it in about a quarter of the blocks, at twice the column pass's vector
// instructions (44 and 27 us).
template <class DT, int D>
__global__ __launch_bounds__(kRowThreads16, 3) void k_rowstats16(EvictArgs a) {
  constexpr int NT = kRowThreads16;
  constexpr int KT = 64;  // keys per staged tile
  using TL = Tile<DT, D, NT, KT>;
  constexpr int KS = D / 32;
  static_assert(DT::kElt == 2, "16-bit inputs");
  static_assert(NT / kWave * 64 == kRowBlock, "four waves of 64 rows");
  __shared__ __align__(16) unsigned char s_k[2][TL::BYTES];

  const int n_rb = (a.W + kRowBlock - 1) / kRowBlock;
  const int id = xcd_remap(blockIdx.x, gridDim.x);
  const int rb = id % n_rb, sp = id / n_rb % a.splits;
  const int ou = id / n_rb / a.splits;  // (owner index * B + b) * Hq + hq
  const int l = a.own.local(ou / (a.B * a.Hq));
  const int b = (ou / a.Hq) % a.B, hq = ou % a.Hq;
  const size_t qunit = ((size_t)l * a.B + b) * a.Hq + hq;
  const int G = a.Hq / a.Hkv;
  const size_t kvunit = ((size_t)l * a.B + b) * a.Hkv + hq / G;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, c16 = lane & 15, q4 = lane >> 4;

  // query group g of this wave holds window rows row0 + 16 g + lane % 16
  const int row0 = rb * kRowBlock + w * 64;
  int t[4], pos[4];
  uint4 qf[4][KS];
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    t[g] = row0 + 16 * g + c16;
    const int tc = t[g] < a.W ? t[g] : a.W - 1;
    pos[g] = a.T - a.W + tc;
    const char* qrow = (const char*)a.q_win + ((size_t)qunit * a.W + tc) * TL::RB;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[g][ks] = ldg16(qrow + (ks * 32 + q4 * 8) * DT::kElt);
  }

  const char* kh = (const char*)a.k + kvunit * a.T * TL::RB;
  const int last_row = min(a.W - 1, rb * kRowBlock + kRowBlock - 1);
  const int jend = a.causal ? min(a.T, a.T - a.W + last_row + 1) : a.T;
  const int ntile = (jend + KT - 1) / KT, per = (ntile + a.splits - 1) / a.splits;
  const int it0 = min(sp * per, ntile), it1 = min(it0 + per, ntile);  // this split's tiles

  const TileChunks<TL, NT> tc(tid);
  uint4 pre[TL::PER];
  // key tiles lying wholly inside the cache load without per-chunk row tests or zero fills
  auto fetch = [&](int tile) {
    const char* tb = kh + (size_t)tile * (KT * TL::RB);
    if (tile * KT + KT <= a.T) {
#pragma unroll
      for (int i = 0; i < TL::PER; ++i)
        if (tc.ok(i)) pre[i] = ldg16(tb + tc.mem(i));
    } else {
#pragma unroll
      for (int i = 0; i < TL::PER; ++i)
        pre[i] = tc.ok(i) && tile * KT + tc.row(i) < a.T ? ldg16(tb + tc.mem(i)) : make_uint4(0, 0, 0, 0);
    }
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int i = 0; i < TL::PER; ++i)
      if (tc.ok(i)) *(uint4*)&s_k[buf][tc.lds(i)] = pre[i];
  };
  if (it0 < it1) {
    fetch(it0);
    stash(0);
  }
  // the row operands are in registers before the loop, so that no wait for them lands inside it
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  const float cf = a.c32;
  float nb[4];    // whole-number offset of each query group's row (this lane's keys)
  double ell[4];  // sum of exp2(fma(c, s, nb)) so far
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    nb[g] = kNoOffset;
    ell[g] = 0.0;
  }
  // one tile; block b = (key quarter b / 4, query group b % 4). FULL: every key of the tile visible
  // to every row of the wave
  auto tile = [&](auto full_tag, int buf, int j0) {
    constexpr bool FULL = decltype(full_tag)::value;
    float psg[4] = {0.f, 0.f, 0.f, 0.f};
    uint4 af[KS];
    auto load_af = [&](int kq) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        af[ks] = *(const uint4*)&s_k[buf][(16 * kq + c16) * TL::RS + (ks * 32 + q4 * 8) * DT::kElt];
    };
    auto chain = [&](int g) {
      f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) c = mma16<DT>(af[ks], qf[g][ks], c);
      return c;
    };
    auto visible = [&](int kq, int g, int r) {
      if constexpr (FULL) return true;
      const int j = j0 + 16 * kq + 4 * q4 + r;
      return j < a.T && (!a.causal || j <= pos[g]);
    };
    auto sum4 = [&](const f32x4& c, int kq, int g) {
      float ps = 0.f;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (visible(kq, g, r)) ps += fast_exp2(fmaf(cf, c[r], nb[g]));
      return ps;
    };
    auto finish = [&](const f32x4& c, int kq, int g, float ps) {
      if (ps > 2.f) {  // an exponent may exceed 1 (or the row's first terms): offset at the max
        float tmax = -INFINITY;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (visible(kq, g, r)) tmax = fmaxf(tmax, c[r]);
        const float nb_new = -ceilf(cf * tmax);
        if (nb_new < nb[g]) {
          const int d = (int)(nb_new - nb[g]);
          if (ell[g] > 0.0) ell[g] = ldexp(ell[g], d);
          if (psg[g] > 0.f) psg[g] = ldexpf(psg[g], d);
          nb[g] = nb_new;
        }
        ps = sum4(c, kq, g);
      }
      psg[g] += ps;
    };
    load_af(0);
    f32x4 cp = chain(0);
#pragma unroll
    for (int bb = 1; bb < 4 * (KT / 16); ++bb) {
      if ((bb & 3) == 0) load_af(bb >> 2);
      const f32x4 cc = chain(bb & 3);
      const int kp = (bb - 1) >> 2, gp = (bb - 1) & 3;
      finish(cp, kp, gp, sum4(cp, kp, gp));
      cp = cc;
    }
    finish(cp, KT / 16 - 1, 3, sum4(cp, KT / 16 - 1, 3));
#pragma unroll
    for (int g = 0; g < 4; ++g) ell[g] += (double)psg[g];
  };
  for (int it = it0; it < it1; ++it) {
    const int buf = (it - it0) & 1;
    if (it + 1 < it1) fetch(it + 1);
    const int j0 = it * KT;
    // a wave none of whose rows sees the tile (rows past a ragged window, keys after its last row) only
    // helps stage it
    if (row0 < a.W && (!a.causal || j0 <= a.T - a.W + row0 + 63)) {
      if (j0 + KT - 1 < a.T && (!a.causal || j0 + KT - 1 <= a.T - a.W + row0))
        tile(std::true_type{}, buf, j0);
      else
        tile(std::false_type{}, buf, j0);
    }
    if (it + 1 < it1) stash(buf ^ 1);
    __syncthreads();
  }
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    // the four lanes of a row (lane % 16 equal) meet at the smallest offset, in two pairwise steps
    double e = ell[g];
    float o = nb[g];
#pragma unroll
    for (int x = 16; x <= 32; x <<= 1) {
      const double eo = __shfl_xor(e, x);
      const float oo = __shfl_xor(o, x);
      const float ox = fminf(o, oo);
      e = moved(e, o, ox) + moved(eo, oo, ox);
      o = ox;
    }
    if (q4 == 0 && t[g] < a.W) put_row(a, ou, (size_t)qunit * a.W, sp, t[g], e, o);
  }
}

constexpr int kMergeThreads = 64;

// Statistics of the window rows whose keys were split over several workgroups: the splits' sums meet at the
// smallest offset. A split none of whose keys the row sees holds a zero sum at kNoOffset. Bound by
// latency: one memory round trip for all splits (12 heads of 102 rows in eight splits: 5.7 -> 4.5 us).
__global__ __launch_bounds__(kMergeThreads) void k_rowmerge(EvictArgs a) {
  const int64_t n = (int64_t)a.own.n * a.B * a.Hq * a.W, i = (int64_t)blockIdx.x * kMergeThreads + threadIdx.x;
  if (i >= n) return;
  const int ou = (int)(i / a.W), t = (int)(i % a.W);
  const double2* p = a.part + (size_t)ou * a.splits * a.W + t;
  double2 x[kMaxRowSplits];  // every split's partial is requested before any is used
#pragma unroll
  for (int s = 0; s < kMaxRowSplits; ++s) x[s] = s < a.splits ? p[(size_t)s * a.W] : make_double2(0.0, INFINITY);
  double o = INFINITY, L = 0.0;
#pragma unroll
  for (int s = 0; s < kMaxRowSplits; ++s) o = fmin(o, x[s].y);
#pragma unroll
  for (int s = 0; s < kMaxRowSplits; ++s) L += moved(x[s].x, x[s].y, o);
  const size_t unit = (size_t)a.own.local(ou / (a.B * a.Hq)) * a.B * a.Hq + ou % (a.B * a.Hq);
  put_stat(a, unit * a.W + t, L, (float)o);
}

// Column pass for 16-bit inputs on 16x16x32 matrix instructions. A wave holds 64 keys in
// registers as four 16-key B operands and takes each 64-row window tile from LDS as four 16-row A
// operands, so a tile is sixteen 16x16 blocks of four accumulators each; every block's
// exponentials and sums run while the next block's four matrix instructions execute (a block's
// vector work, twelve instructions, matches its matrix work), with no second accumulator set, and
// a barrier, a tile load and a row-statistics stash serve 64 rows. A lane holds rows
// 4 (lane / 16) + r of one key per block; its fp32 sum over a tile's sixteen rows goes into an fp64
// total, and the four lanes of a key meet once at the end.
// What bounds it: matrix and vector work that overlap only in part, at the 1.9 GHz that the chip keeps under this load
// (4 x 32768 keys, 32 heads: 3.3 ms, the matrix cores busy 51% of the cycles; 45% in the row pass, 3.7 ms). A written-out
// order of the blocks changes nothing (fewer cycles at a lower clock; 8192 keys to 131072 within 0.3%), and 32x32x16
// blocks, which need 222 registers with the row statistics of their sixteen rows a lane, are slower (two waves per
// SIMD: 3.7 against 3.3 ms). Quarters of a
// masked tile that no key of the wave is seen by, or past the window, are left out: of a window of 204 rows
// the last tile holds 12 (8 x 1024 keys, 17 owner layers: 490 -> 467 us).
template <class DT, int D>
__global__ __launch_bounds__(kColThreads16, 3) void k_colsum16(EvictArgs a) {
  constexpr int NT = kColThreads16;
  constexpr int RT = 64;  // window rows per staged tile
  using TL = Tile<DT, D, NT, RT>;
  constexpr int KS = D / 32;
  static_assert(DT::kElt == 2, "16-bit inputs");
  static_assert(NT / kWave * 64 == kColBlockKeys, "four waves of 64 keys");
  __shared__ __align__(16) unsigned char s_q[2][TL::BYTES];
  __shared__ __align__(16) float s_nb[2][RT], s_il[2][RT];  // offset and 1 / sum of the staged rows

  const int n_kb = (a.T + kColBlockKeys - 1) / kColBlockKeys;
  const int id = xcd_remap(blockIdx.x, gridDim.x);
  const ColItem item = col_item(a, id, gridDim.x / n_kb, n_kb);
  const int kb = item.kb, sp = item.unit % a.col_splits;
  const int ou = item.unit / a.col_splits;  // (owner index * B + b) * Hkv + h
  const int l = a.own.local(ou / (a.B * a.Hkv));
  const int b = (ou / a.Hkv) % a.B, h = ou % a.Hkv;
  const size_t kvunit = ((size_t)l * a.B + b) * a.Hkv + h;
  const int G = a.Hq / a.Hkv;
  const int tid = threadIdx.x, lane = tid & 63, c16 = lane & 15, q4 = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform over the wave

  // key group g of this wave holds keys jw + 16 g + lane % 16
  const int jw = kb * kColBlockKeys + w * 64;
  const float cf = a.c32;
  const char* kh = (const char*)a.k + (size_t)kvunit * a.T * TL::RB;
  uint4 kf[4][KS];
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int j = min(jw + 16 * g + c16, a.T - 1);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kf[g][ks] = ldg16(kh + (size_t)j * TL::RB + (ks * 32 + q4 * 8) * DT::kElt);
  }

  const int j_lo = kb * kColBlockKeys;
  const int t_start = a.causal ? (max(0, j_lo - (a.T - a.W)) & ~31) : 0;
  const int n_t = (a.W - t_start + RT - 1) / RT;
  const int ntile = G * n_t, per = (ntile + a.col_splits - 1) / a.col_splits;
  const int it0 = min(sp * per, ntile), it1 = min(it0 + per, ntile);  // this split's tiles
  const size_t qunit0 = ((size_t)l * a.B + b) * a.Hq + (size_t)h * G;

  const TileChunks<TL, NT> tc(tid);
  uint4 pre[TL::PER];
  float2 pre_b = make_float2(0.f, 0.f);
  // tiles run through the group's heads, each from row t_start to t_end; the next one to fetch is
  // head fg's rows ft0 .. ft0 + RT - 1
  const int t_end = t_start + n_t * RT;
  int fg = it0 / n_t, ft0 = t_start + it0 % n_t * RT;
  int t0 = ft0;  // first window row of the tile being scored
  auto fetch = [&]() {
    const size_t r0 = (qunit0 + fg) * a.W + ft0;
    const char* tb = (const char*)a.q_win + r0 * TL::RB;
    if (ft0 + RT <= a.W) {
#pragma unroll
      for (int i = 0; i < TL::PER; ++i)
        if (tc.ok(i)) pre[i] = ldg16(tb + tc.mem(i));
    } else {
#pragma unroll
      for (int i = 0; i < TL::PER; ++i)
        pre[i] = tc.ok(i) && ft0 + tc.row(i) < a.W ? ldg16(tb + tc.mem(i)) : make_uint4(0, 0, 0, 0);
    }
    if (tid < RT) pre_b = ft0 + tid < a.W ? a.rowstat[r0 + tid] : make_float2(0.f, 0.f);
    ft0 += RT;
    if (ft0 == t_end) {
      ft0 = t_start;
      ++fg;
    }
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int i = 0; i < TL::PER; ++i)
      if (tc.ok(i)) *(uint4*)&s_q[buf][tc.lds(i)] = pre[i];
    if (tid < RT) {
      s_nb[buf][tid] = pre_b.x;
      s_il[buf][tid] = pre_b.y;
    }
  };
  if (it0 < it1) {
    fetch();
    stash(0);
  }
  // the key operands are in registers before the loop, so that no wait for them lands inside it
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  double cacc[4] = {0.0, 0.0, 0.0, 0.0};
  // one tile; FULL: every row valid and every key of the wave visible to the tile's first row
  auto tile = [&](auto full_tag, int buf) {
    constexpr bool FULL = decltype(full_tag)::value;
    float ps[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int rh = 0; rh < RT / 16; ++rh) {
      // a quarter of rows past the window, or none of which sees a key of the wave
      if constexpr (!FULL)
        if (t0 + 16 * rh >= a.W || (a.causal && jw > a.T - a.W + t0 + 16 * rh + 15)) continue;
      // this lane's rows of the quarter: t0 + 16 rh + 4 (lane / 16) + r
      const float4 nb4 = *(const float4*)&s_nb[buf][16 * rh + 4 * q4];
      const float4 il4 = *(const float4*)&s_il[buf][16 * rh + 4 * q4];
      const float nbv[4] = {nb4.x, nb4.y, nb4.z, nb4.w}, ilv[4] = {il4.x, il4.y, il4.z, il4.w};
      uint4 af[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        af[ks] = *(const uint4*)&s_q[buf][(16 * rh + c16) * TL::RS + (ks * 32 + q4 * 8) * DT::kElt];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) c = mma16<DT>(af[ks], kf[g][ks], c);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if constexpr (FULL) {
            ps[g] = fmaf(fast_exp2(fmaf(cf, c[r], nbv[r])), ilv[r], ps[g]);
          } else {
            const int t = t0 + 16 * rh + 4 * q4 + r, j = jw + 16 * g + c16;
            if (t < a.W && (!a.causal || j <= a.T - a.W + t))
              ps[g] = fmaf(fast_exp2(fmaf(cf, c[r], nbv[r])), ilv[r], ps[g]);
          }
        }
      }
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) cacc[g] += (double)ps[g];
  };
  for (int it = it0; it < it1; ++it) {
    const int buf = (it - it0) & 1;
    if (it + 1 < it1) fetch();
    // keys past the prompt, or past what the tile's last row sees: the wave only helps stage the tile
    if (jw < a.T && (!a.causal || jw <= a.T - a.W + t0 + RT - 1)) {
      if (t0 + RT - 1 < a.W && (!a.causal || jw + 63 <= a.T - a.W + t0))
        tile(std::true_type{}, buf);
      else
        tile(std::false_type{}, buf);
    }
    if (it + 1 < it1) stash(buf ^ 1);
    t0 = t0 + RT == t_end ? t_start : t0 + RT;
    __syncthreads();
  }
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    double tot = cacc[g] + __shfl_xor(cacc[g], 16);
    tot += __shfl_xor(tot, 32);
    const int j = jw + 16 * g + c16;
    if (q4 == 0 && j < a.T) put_score(a, ou, kvunit, sp, j, tot);
  }
}

// ---------------------------------------------------------------------------------------------
// Top-k: the n_sel best-scored older tokens of an owner head, in ascending order, by one workgroup.
// Scores are non-negative, so their bits order like their values. A radix select finds the threshold: it
// starts at the highest bit in which the largest and the smallest score differ (below it the bins spread,
// above it every score would count into one bin), and ends as soon as a bin is taken whole, which for
// distinct scores happens after about two digits. Then an ordered compaction: the scores above the
// threshold bin, and as many of the bin (all, or of equal scores the lowest positions) as are wanted.
constexpr int kHistCopies = 4;  // histograms of a workgroup, one per wave modulo this

template <int NT>
struct TopkLds {
  uint32_t hist[kHistCopies][256];
  uint32_t tot[256];
  uint32_t red[2][NT / kWave];
  uint32_t prefix;
  int rem, done;
  uint32_t wsum[NT / kWave], wbin[NT / kWave];
};

// Exclusive prefix sum over the NT threads of a workgroup.
template <int NT>
__device__ uint32_t block_excl_scan(uint32_t v, uint32_t* wsum) {
  constexpr int NW = NT / kWave;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  uint32_t before = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) before += i < w ? wsum[i] : 0;
  return before + x - v;
}

// The digit (bins in descending order) at which the running count of tot[] reaches rem, by the 64 lanes of
// wave 0 (four bins each, a wave prefix sum): writes prefix | digit << shift, rem minus the count of the
// higher bins, and whether the bin is taken whole. Requires sum(tot) >= rem >= 1.
__device__ __forceinline__ void pick_digit(const uint32_t* tot, int rem, uint32_t prefix, int shift,
                                           uint32_t* s_prefix, int* s_rem, int* s_done) {
  const int lane = threadIdx.x & 63;
  uint32_t c[4], sum = 0;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    c[u] = tot[255 - 4 * lane - u];
    sum += c[u];
  }
  uint32_t x = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  uint32_t cum = x - sum;  // count of the bins above this lane's first
  const uint32_t r = (uint32_t)rem;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    if (cum < r && r <= cum + c[u]) {
      *s_prefix = prefix | ((uint32_t)(255 - 4 * lane - u) << shift);
      *s_rem = (int)(r - cum);
      *s_done = r == cum + c[u];
    }
    cum += c[u];
  }
}

// The threshold bin of the rem best of a head's scores: scores with (u & mask) > prefix are in, and `rem`
// of those with (u & mask) == prefix. each(f) calls f(u) for every score of the calling thread.
template <int NT, class Each>
__device__ void radix_threshold(TopkLds<NT>& s, Each each, int& rem, uint32_t& prefix, uint32_t& mask) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  uint32_t hi = 0u, lo = ~0u;
  each([&](uint32_t u) {
    hi = max(hi, u);
    lo = min(lo, u);
  });
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, o));
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, o));
  }
  if (lane == 0) {
    s.red[0][w] = hi;
    s.red[1][w] = lo;
  }
  for (int i = tid; i < kHistCopies * 256; i += NT) s.hist[i / 256][i % 256] = 0;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NT / kWave; ++i) {
    hi = max(hi, s.red[0][i]);
    lo = min(lo, s.red[1][i]);
  }
  int top = hi == lo ? 0 : 32 - __clz((int)(hi ^ lo));  // bits still undecided
  mask = top >= 32 ? 0u : ~0u << top;
  prefix = hi & mask;
  while (top > 0) {
    const int shift = max(0, top - 8);
    each([&](uint32_t u) {
      if ((u & mask) == prefix) atomicAdd(&s.hist[w % kHistCopies][(u >> shift) & 255u & ~(~0u << (top - shift))], 1u);
    });
    __syncthreads();
    if (tid < 256) {
      uint32_t sum = 0;
#pragma unroll
      for (int i = 0; i < kHistCopies; ++i) {
        sum += s.hist[i][tid];
        s.hist[i][tid] = 0;
      }
      s.tot[tid] = sum;
    }
    __syncthreads();
    if (tid < 64) pick_digit(s.tot, rem, prefix, shift, &s.prefix, &s.rem, &s.done);
    __syncthreads();
    prefix = s.prefix;
    rem = s.rem;
    top = s.done ? 0 : shift;
    mask = ~0u << shift;
  }
}

// Each thread holds a run of KPT scores in registers from one read on. NT follows the prompt (launch_topk):
// a thread per 4 to 32 scores, and no more threads than scores, which is what short prompts of many heads
// need. 4352 heads of 992 older tokens: 76 us with 1024 threads and four full digits, 17 us so; 32
// heads of 7145: 13.5 and 12.5 us.
template <int NT, int KPT>
__global__ __launch_bounds__(NT) void k_topk_reg(EvictArgs a) {
  __shared__ TopkLds<NT> s;
  const int ou = blockIdx.x;  // (owner index * B + b) * Hkv + h
  const int l = a.own.local(ou / (a.B * a.Hkv));
  const size_t unit = (size_t)l * a.B * a.Hkv + ou % (a.B * a.Hkv);
  const int tid = threadIdx.x;
  const int loc = min(a.local_keep, a.keep);
  const int n_old = a.T - loc, n_sel = a.keep - loc;
  const uint32_t* key = (const uint32_t*)(a.score + (size_t)unit * a.T);
  int32_t* out = a.kept + (size_t)unit * a.keep;
  for (int i = tid; i < loc; i += NT) out[n_sel + i] = n_old + i;
  if (n_sel <= 0) return;

  // this thread's run [j0, j0 + nv) of the older tokens' scores
  const int j0 = tid * KPT;
  const int nv = max(0, min(KPT, n_old - j0));
  uint32_t kv[KPT];
  if (nv == KPT && (((uintptr_t)(key + j0)) & 15) == 0) {
#pragma unroll
    for (int i = 0; i < KPT; i += 4) {
      const uint4 v = *(const uint4*)(key + j0 + i);
      kv[i] = v.x;
      kv[i + 1] = v.y;
      kv[i + 2] = v.z;
      kv[i + 3] = v.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < KPT; ++i) kv[i] = i < nv ? key[j0 + i] : 0u;
  }
  int rem = n_sel;
  uint32_t prefix, mask;
  radix_threshold<NT>(s,
                      [&](auto f) {
#pragma unroll
                        for (int i = 0; i < KPT; ++i)
                          if (i < nv) f(kv[i]);
                      },
                      rem, prefix, mask);
  static_assert(NT * KPT <= 1 << 15, "counts fit 16 bits");
  uint32_t cnt = 0;  // scores of the bin, then (upper half) scores above it
#pragma unroll
  for (int i = 0; i < KPT; ++i)
    if (i < nv) cnt += (kv[i] & mask) > prefix ? 1u << 16 : (kv[i] & mask) == prefix;
  const uint32_t before = block_excl_scan<NT>(cnt, s.wsum);
  int eq = (int)(before & 0xFFFFu), off = (int)(before >> 16) + min(eq, rem);
#pragma unroll
  for (int i = 0; i < KPT; ++i) {
    if (i >= nv) break;
    const uint32_t u = kv[i] & mask;
    if (u > prefix || (u == prefix && eq < rem)) out[off++] = j0 + i;
    eq += u == prefix;
  }
}

// Longer prompts: each wave streams a contiguous share of the scores, 256 at a time (four per lane), and
// places its own by wave prefix sums. 8 heads of 131040 older tokens: 277 us with one score per thread and
// step and four full digits, 119 us so.
constexpr int kTopkThreads = 1024;

__global__ __launch_bounds__(kTopkThreads) void k_topk(EvictArgs a) {
  constexpr int NT = kTopkThreads, NW = NT / kWave, STEP = 4 * kWave;
  __shared__ TopkLds<NT> s;
  const int ou = blockIdx.x;  // (owner index * B + b) * Hkv + h
  const int l = a.own.local(ou / (a.B * a.Hkv));
  const size_t unit = (size_t)l * a.B * a.Hkv + ou % (a.B * a.Hkv);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int loc = min(a.local_keep, a.keep);
  const int n_old = a.T - loc, n_sel = a.keep - loc;
  const uint32_t* key = (const uint32_t*)(a.score + (size_t)unit * a.T);
  int32_t* out = a.kept + (size_t)unit * a.keep;
  for (int i = tid; i < loc; i += NT) out[n_sel + i] = n_old + i;
  if (n_sel <= 0) return;

  const int share = (n_old + NW * STEP - 1) / (NW * STEP) * STEP;
  const int lo = min(n_old, w * share), hi = min(n_old, lo + share);  // this wave's scores
  const bool wide = ((uintptr_t)key & 15) == 0;
  // scores j .. j + 3 (those below hi)
  auto four = [&](int j, uint32_t (&v)[4]) {
    if (wide && j + 4 <= hi) {
      const uint4 q = *(const uint4*)(key + j);
      v[0] = q.x;
      v[1] = q.y;
      v[2] = q.z;
      v[3] = q.w;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = j + i < hi ? key[j + i] : 0u;
    }
  };
  int rem = n_sel;
  uint32_t prefix, mask;
  radix_threshold<NT>(s,
                      [&](auto f) {
#pragma unroll 4
                        for (int b = lo; b < hi; b += STEP) {
                          const int j = b + 4 * lane;
                          uint32_t v[4];
                          four(j, v);
#pragma unroll
                          for (int i = 0; i < 4; ++i)
                            if (j + i < hi) f(v[i]);
                        }
                      },
                      rem, prefix, mask);
  auto tally = [&](int j, const uint32_t (&v)[4]) {
    uint32_t c = 0;  // scores of the bin, then (upper half) scores above it: at most 256 in a step
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (j + i < hi) c += (v[i] & mask) > prefix ? 1u << 16 : (v[i] & mask) == prefix;
    return c;
  };
  uint32_t above = 0, bin = 0;
#pragma unroll 4
  for (int b = lo; b < hi; b += STEP) {
    uint32_t v[4];
    four(b + 4 * lane, v);
    const uint32_t c = tally(b + 4 * lane, v);
    above += c >> 16;
    bin += c & 0xFFFFu;
  }
  above = wave_sum(above);
  bin = wave_sum(bin);
  if (lane == 0) {
    s.wsum[w] = above;
    s.wbin[w] = bin;
  }
  __syncthreads();
  above = bin = 0;  // of the scores before this wave's, then before its next step's
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    above += i < w ? s.wsum[i] : 0;
    bin += i < w ? s.wbin[i] : 0;
  }
#pragma unroll 4
  for (int b = lo; b < hi; b += STEP) {
    const int j = b + 4 * lane;
    uint32_t v[4];
    four(j, v);
    const uint32_t c = tally(j, v);
    uint32_t x = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(x, o);
      if (lane >= o) x += y;
    }
    int eq = (int)(bin + ((x - c) & 0xFFFFu)), off = (int)(above + ((x - c) >> 16)) + min(eq, rem);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (j + i >= hi) break;
      const uint32_t u = v[i] & mask;
      if (u > prefix || (u == prefix && eq < rem)) out[off++] = j + i;
      eq += u == prefix;
    }
    const uint32_t all = __shfl(x, 63);
    above += all >> 16;
    bin += all & 0xFFFFu;
  }
}

template <int RB>
__global__ __launch_bounds__(256) void k_gather(EvictArgs a) {
  constexpr int CH = RB / 16;
  constexpr int RPP = 256 / CH;
  constexpr int ROWS = 64;
  const int n_chunks = (a.keep + ROWS - 1) / ROWS;
  const int chunk = blockIdx.x % n_chunks;
  const size_t unit = blockIdx.x / n_chunks;
  const int l = (int)(unit / ((size_t)a.B * a.Hkv));
  if ((a.skip[l >> 6] >> (l & 63)) & 1) return;
  const int o = owner_layer(a.layer0 + l, a.period, a.start) - a.layer0;
  const int src_l = o >= 0 ? o : l;
  const size_t src_unit = unit - (size_t)(l - src_l) * a.B * a.Hkv;
  const int r_in = threadIdx.x / CH, c16 = threadIdx.x % CH;
  const int end = min(a.keep, chunk * ROWS + ROWS);
  for (int i = chunk * ROWS + r_in; i < end; i += RPP) {
    int idx = a.kept[src_unit * a.keep + i];
    if (src_l != l && c16 == 0) a.kept[unit * a.keep + i] = idx;
    idx = min(max(idx, 0), a.T - 1);  // indices supplied by the caller are clamped into the cache
    const size_t so = (unit * a.T + idx) * RB + c16 * 16;
    const size_t dst = (unit * a.out_rows + i) * RB + c16 * 16;
    *(uint4*)((char*)a.k_out + dst) = ldg16((const char*)a.k + so);
    *(uint4*)((char*)a.v_out + dst) = ldg16((const char*)a.v + so);
  }
}

// Scores of keys whose window rows were split over several workgroups.
__global__ __launch_bounds__(256) void k_colmerge(EvictArgs a) {
  const int64_t n = (int64_t)a.own.n * a.B * a.Hkv * a.T, i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int ou = (int)(i / a.T), j = (int)(i % a.T);
  const double* p = a.col_part + (size_t)ou * a.col_splits * a.T + j;
  double x[kMaxColSplits], sum = 0.0;  // every split's part is requested before any is used
#pragma unroll
  for (int s = 0; s < kMaxColSplits; ++s) x[s] = s < a.col_splits ? p[(size_t)s * a.T] : 0.0;
#pragma unroll
  for (int s = 0; s < kMaxColSplits; ++s) sum += x[s];
  const size_t unit = (size_t)a.own.local(ou / (a.B * a.Hkv)) * a.B * a.Hkv + ou % (a.B * a.Hkv);
  a.score[unit * a.T + j] = (float)sum;
}

template <class DT, int D>
hipError_t launch_pass(const EvictArgs& a, bool rows, hipStream_t st) {
  if (rows) {
    const int n_rb = (a.W + kRowBlock - 1) / kRowBlock;
    if constexpr (DT::kElt == 2)
      hipLaunchKernelGGL((k_rowstats16<DT, D>), dim3(a.own.n * a.B * a.Hq * n_rb * a.splits), dim3(kRowThreads16), 0, st, a);
    else
      hipLaunchKernelGGL((k_rowstats<DT, D>), dim3(a.own.n * a.B * a.Hq * n_rb * a.splits), dim3(kWaves32 * kWave), 0, st,
                         a);
  } else {
    const int n_kb = (a.T + kColBlockKeys - 1) / kColBlockKeys;
    const int heads = a.own.n * a.B * a.Hkv * a.col_splits;
    if constexpr (DT::kElt == 2) {
      hipLaunchKernelGGL((k_colsum16<DT, D>), dim3(heads * n_kb), dim3(kColThreads16), 0, st, a);
    } else if (heads * n_kb <= kNumCU / 4) {
      // few workgroups: a quarter of the keys each (12 heads of 512 keys, 24 workgroups of eight waves: prefill
      // 46.9 us; 96 of two, with operands read four elements at a time in both passes: 34.7)
      const int n_few = (a.T + 32 * kFewWaves32 - 1) / (32 * kFewWaves32);
      hipLaunchKernelGGL((k_colsum<DT, D, kFewWaves32>), dim3(heads * n_few), dim3(kFewWaves32 * kWave), 0, st, a);
    } else {
      hipLaunchKernelGGL((k_colsum<DT, D, kWaves32>), dim3(heads * n_kb), dim3(kWaves32 * kWave), 0, st, a);
    }
  }
  return hipGetLastError();
}

template <class DT>
hipError_t launch_pass_dt(const EvictArgs& a, int D, bool rows, hipStream_t st) {
  if (D == 64) return launch_pass<DT, 64>(a, rows, st);
  if (D == 128) return launch_pass<DT, 128>(a, rows, st);
  return hipErrorInvalidValue;
}

hipError_t launch_pass_any(const EvictArgs& a, int dtype, int D, bool rows, hipStream_t st) {
  switch (dtype) {
    case MPC_FP32: return launch_pass_dt<F32>(a, D, rows, st);
    case MPC_FP16: return launch_pass_dt<F16>(a, D, rows, st);
    case MPC_BF16: return launch_pass_dt<BF16>(a, D, rows, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_rowstats(const EvictArgs& a, int dtype, int D, hipStream_t st) {
  const hipError_t e = launch_pass_any(a, dtype, D, true, st);
  if (e != hipSuccess || a.splits == 1) return e;
  const int64_t rows = (int64_t)a.own.n * a.B * a.Hq * a.W;
  hipLaunchKernelGGL(k_rowmerge, dim3((unsigned)((rows + kMergeThreads - 1) / kMergeThreads)), dim3(kMergeThreads), 0, st, a);
  return hipGetLastError();
}

// A split is taken where it evens out the work: the launch ends with the compute unit that holds the most
// workgroups (one alone on its unit runs at about 1.4 times the time of one among several), and each split
// costs about two tiles beside its own: its rows' loads, and the first tile's slow path to its offsets. Unsplit
// and split, the merge (4.8 us) not counted: 32 heads of 7177 keys (192 row blocks) 218 and 126 us, in four; 84 heads
// of 2048 keys (168) 75 and 50 us, in three; 144 heads of 2048 keys of 64 channels 87 and 67 us; 12 heads of 512 fp32
// keys 25 and 11 us; 128 heads of 32768 keys (1664 = 6.5 a unit) 4.04 and 3.66 ms, in two. 320 heads of 8192 keys (8.75
// a unit) stay whole.
int row_splits(int heads, int T, int W, int causal) {
  const int64_t base = (int64_t)heads * ((W + kRowBlock - 1) / kRowBlock);
  const int ntile = ((causal ? T - W / 2 : T) + 63) / 64;
  int best = 1;
  double cost = INFINITY;
  for (int s = 1; s <= kMaxRowSplits && s <= ntile; ++s) {
    const int64_t per_cu = (base * s + kNumCU - 1) / kNumCU;
    const double len = (double)((ntile + s - 1) / s) + kSplitTiles;
    const double c = per_cu == 1 ? 1.4 * len : per_cu * len;
    if (c < 0.97 * cost) {
      cost = c;
      best = s;
    }
  }
  return best;
}

hipError_t launch_colsum(const EvictArgs& a, int dtype, int D, hipStream_t st) {
  const hipError_t e = launch_pass_any(a, dtype, D, false, st);
  if (e != hipSuccess || a.col_splits == 1) return e;
  const int64_t keys = (int64_t)a.own.n * a.B * a.Hkv * a.T;
  hipLaunchKernelGGL(k_colmerge, dim3((unsigned)((keys + 255) / 256)), dim3(256), 0, st, a);
  return hipGetLastError();
}

// A split is taken where the key blocks leave compute units idle or with one workgroup: it costs three tiles beside
// its own (key loads, first tile) and, all together, a merge of about five tiles' time. Prefill of one layer with
// eight kv heads of four query heads: 1023 keys 81.9 -> 42.1 us, 8191 keys 365 -> 308 us; two kv heads of 700 keys 64.8
// -> 35.8 us; eight heads of 3000 keys (fp32) 302 -> 191 us. 32 heads of 7177 keys and more stay whole.
int col_splits(int heads, int T, int W, int group) {
  const int64_t base = (int64_t)heads * ((T + kColBlockKeys - 1) / kColBlockKeys);
  const int ntile = group * ((W + 63) / 64);
  int best = 1;
  double cost = INFINITY;
  for (int s = 1; s <= kMaxColSplits && s <= ntile; ++s) {
    const int64_t per_cu = (base * s + kNumCU - 1) / kNumCU;
    if (s > 1 && per_cu > 3) break;
    const double len = (double)((ntile + s - 1) / s) + 3.0;
    const double c = (per_cu == 1 ? 1.4 * len : per_cu * len) + (s > 1 ? 5.0 : 0.0);
    if (c < 0.95 * cost) {
      cost = c;
      best = s;
    }
  }
  return best;
}

// Units whose key blocks are dealt together (col_item): as many as a die holds, and no more than have their window
// rows in half of its 4 MiB L2 while the group's last blocks are scored. One where all workgroups are resident at
// once (three to a compute unit) and none is last: the order then only costs its arithmetic (12 layers of 2048 tokens,
// 672 workgroups: 80.2 us in groups of one, 81.1 in larger ones).
int col_group(int units, int T, int64_t unit_bytes) {
  if ((int64_t)units * ((T + kColBlockKeys - 1) / kColBlockKeys) <= 3 * kNumCU) return 1;
  const int64_t fit = (2 << 20) / unit_bytes;
  return std::max(1, (int)std::min<int64_t>(units / kNumXcd, fit));
}

template <int NT, int KPT>
static void launch_topk_reg(const EvictArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((k_topk_reg<NT, KPT>), dim3(a.own.n * a.B * a.Hkv), dim3(NT), 0, st, a);
}

hipError_t launch_topk(const EvictArgs& a, hipStream_t st) {
  // a run of up to 32 scores per thread stays in registers; longer prompts stream the scores
  const int n_old = a.T - min(a.local_keep, a.keep);
  if (n_old <= 1024)
    launch_topk_reg<256, 4>(a, st);
  else if (n_old <= 2048)
    launch_topk_reg<512, 4>(a, st);
  else if (n_old <= 4096)
    launch_topk_reg<1024, 4>(a, st);
  else if (n_old <= 8192)
    launch_topk_reg<1024, 8>(a, st);
  else if (n_old <= 16384)
    launch_topk_reg<1024, 16>(a, st);
  else if (n_old <= 32768)
    launch_topk_reg<1024, 32>(a, st);
  else
    hipLaunchKernelGGL(k_topk, dim3(a.own.n * a.B * a.Hkv), dim3(kTopkThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_gather(const EvictArgs& a, int dtype, int D, hipStream_t st) {
  const int rb = D * (dtype == MPC_FP32 ? 4 : 2);
  const int blocks = a.n_layers * a.B * a.Hkv * ((a.keep + 63) / 64);
  switch (rb) {
    case 128: hipLaunchKernelGGL(k_gather<128>, dim3(blocks), dim3(256), 0, st, a); break;
    case 256: hipLaunchKernelGGL(k_gather<256>, dim3(blocks), dim3(256), 0, st, a); break;
    case 512: hipLaunchKernelGGL(k_gather<512>, dim3(blocks), dim3(256), 0, st, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace mpc
