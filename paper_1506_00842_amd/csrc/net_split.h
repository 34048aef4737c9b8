// fp32 networks (TUNER_ALGO_AUTO) whose second hidden layer runs on the 16-bit matrix cores
// with every operand split into two f16 planes, and whose first layer is, where the space
// allows it, a product of two tabulated exponentials.  Paper: Section 4.2 (neuron), Section
// 5.2 (sigmoid hidden layers), Section 5.1 (the space is a Cartesian product).
//
// Layer 2.  v_mfma_f32_32x32x2_f32 runs on the SIMD's own FMA lanes: 64 cycles for 2,048
// multiply-adds, added to the sigmoids' vector cycles.  v_mfma_f32_32x32x16_f16 does 16,384 in
// 32 cycles beside them.  x = x_hi + x_lo with x_hi = f16(x), x_lo = f16(x - x_hi) keeps 22
// significant bits, and a_hi b_hi + a_hi b_lo + a_lo b_hi in fp32 accumulators costs 96 cycles
// per 16,384 products instead of 512.  Against 64-bit results the error is that of the fp32
// instructions or less (their 32 roundings per unit of a 64-wide layer are 12 here): over spaces
// of 256 to 2^27 configurations and layers of 8 to 128 units the relative 2-norm is 0.98 times
// theirs in the geometric mean.  That holds while the weights are not large against the sums: a
// 32-row tile with a weight beyond 64 (times log2 e), where sums cancel and 22 bits would show,
// or with one that is not finite keeps its fp32 weights and the fp32 instructions (flag 1 + u).
//
// Layer 1 ("factored").  Let `span` be the number of configurations the parameters p0 .. P-1 run
// through (the stride of parameter p0 - 1): configuration i lies in row i / span at place
// i % span.  The pre-activation splits as z[u](i) = z_row[u] + z_low[u][i % span], and the
// sigmoid needs only 2^z = 2^z_row[u] * 2^z_low[u][place].  The second factor is a table per
// member made when the weights are packed (rounded once from double); the first is computed
// once per row, one unit per lane, and passed through a per-wave LDS scratch.  A unit then
// costs one fma and one reciprocal instead of its share of the matrix work, an exponential, an
// add and a reciprocal (14 vector cycles instead of 24 and 8 matrix cycles).
// The products of exponentials cannot leave the fp32 range while every unit's
// |b| + sum |w| (features are in [0, 1]), scaled by log2 e, is at most 120; a member beyond that
// has the exponents themselves in its tables (flag word 0) and pays the exponential.
//
// Packed member (32-bit words), hidden-layer weights and biases times -log2(e):
//   factored:  TB  [span][8 NT1 float4]   unit 32 t + 4 e + j (e = 0..7) of place l at float4
//                                         8 t + (e ^ (l & 7)), so that the lanes of a wave, which
//                                         read different places, spread over the LDS banks
//              WH  [ceil((p0 + 1) / 4)][units][4]   W1[u][p], b1[u] at p = p0, 0 beyond
//   otherwise: the first layer's tables of net_f32.h or net_f32h.h
//   W2A [2][NT2][2 NT1][64 lanes][4]      f16 planes, as in net_lp.h
//              a tile in fp32: its [NT1][4][64][4] words of net_f32.h, the first half in place of
//              the tile's first plane, the second half in place of its second
//   b2A [NT2][4][2][4], woA [NTlast][4][2][4]
//   flags [8]  0: exponents instead of exponentials; 1 + u: tile u of layer 2 is in fp32
#pragma once
#include "../../include/tuner.h"
#include "net_f32.h"
#include "net_f32h.h"
#include "net_lp.h"

namespace tuner {

constexpr int kSplitFlagWords = 8;
constexpr float kFactoredMaxExponent = 120.0f;
constexpr float kSplitMaxWeight = 64.0f;

// x_lo of a pair: f16(a - hi.x), f16(b - hi.y), each one fused multiply-add that reads the f16
// half directly and rounds its fp32 result into one half of the word (the compiler forms them
// for some pairs only and spends a third instruction on the others).
__device__ __forceinline__ uint32_t split_remainders(float a, float b, uint32_t hi) {
  uint32_t lo;
  asm("v_fma_mixlo_f16 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(lo) : "v"(hi), "v"(a));
  asm("v_fma_mixhi_f16 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(lo) : "v"(hi), "v"(b));
  return lo;
}
// pair jj of block b of a tile's sigmoid values
__device__ __forceinline__ void split_pair(const floatx16& a, int b, int jj, B4& hi, B4& lo) {
  const float2v ab = {a[8 * b + 2 * jj], a[8 * b + 2 * jj + 1]};
  hi.w[jj] = __builtin_bit_cast(uint32_t, __builtin_convertvector(ab, f16x2));
  lo.w[jj] = split_remainders(ab.x, ab.y, hi.w[jj]);
}
__device__ __forceinline__ void split_block(const floatx16& a, int b, B4& hi, B4& lo) {
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) split_pair(a, b, jj, hi, lo);
}

// Layer 2 and the output from the sigmoid values of layer 1, which `tile` produces for the
// 32-unit tiles t = 0 .. NT1 - 1: one tile at a time (sigmoid, split, matrix steps), so that a
// wave holds one layer-1 tile and the matrix steps of one wave run beside the vector work of the
// others.  tile.load(t) issues the LDS reads of a tile, tile.finish(a) turns them into sigmoid
// values.  Every LDS read is issued a phase ahead of its use: with a read and its use back to
// back the 2^27-configuration sweep of the 4 x 14-64-64-1 ensemble took 8.3 ms.
// (The empty asm statements pin what they name to its phase: a scheduling barrier alone does not
// keep plain arithmetic from being moved past it, and registers run out.)
// FP32_TILES: tiles of layer 2 may be in fp32 (flags); a version of its own, since tests inside
// the fast one would cut it into blocks, between which the compiler moves work and spills.
// Returns the lane's share of the output.
template <int NT1, int NT2, bool FP32_TILES, class Tile>
__device__ __forceinline__ float split_layers(const uint32_t* wm, int lane, const NetOffsets& o, Tile& tile) {
  const int h = lane >> 5;
  const float4* wo = reinterpret_cast<const float4*>(wm + o.wo);
  float part = 0.0f;
  // The two tiles of a wave read the same weights one after the other; without the fence the
  // compiler keeps what it has read for the first in registers for the second, and spills.
  asm volatile("" ::: "memory");
  tile.load(0);
  if constexpr (NT2 == 0) {
#pragma unroll
    for (int t = 0; t < NT1; ++t) {
      floatx16 a;
      float4 q[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) q[g] = wo[(t * 4 + g) * 2 + h];
      tile.finish(a);
      if (t + 1 < NT1) tile.load(t + 1);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        part = fmaf(q[g].x, a[4 * g + 0], part);
        part = fmaf(q[g].y, a[4 * g + 1], part);
        part = fmaf(q[g].z, a[4 * g + 2], part);
        part = fmaf(q[g].w, a[4 * g + 3], part);
      }
      asm volatile("" : "+v"(part));
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
    typedef LpNet<_Float16, 2, 1, NT1, NT2, true> Lp;
    typedef typename Lp::Tr Tr;
    const float4* b2 = reinterpret_cast<const float4*>(wm + o.b2);
    const uint4* w2 = reinterpret_cast<const uint4*>(wm + o.w2);
    floatx16 a2[NT2];
#pragma unroll
    for (int u = 0; u < NT2; ++u) Lp::init_bias(b2, u, h, a2[u]);
    // one block of 16 inputs: the three products, each over all output tiles so that
    // consecutive matrix instructions do not wait for each other
    auto block = [&](const typename Lp::A4 (&w)[NT2], const B4& hi, const B4& lo) {
#pragma unroll
      for (int u = 0; u < NT2; ++u) a2[u] = Tr::mfma(B4{{w[u].p[0].x, w[u].p[0].y, w[u].p[0].z, w[u].p[0].w}}, hi, a2[u]);
#pragma unroll
      for (int u = 0; u < NT2; ++u) a2[u] = Tr::mfma(B4{{w[u].p[0].x, w[u].p[0].y, w[u].p[0].z, w[u].p[0].w}}, lo, a2[u]);
#pragma unroll
      for (int u = 0; u < NT2; ++u) a2[u] = Tr::mfma(B4{{w[u].p[1].x, w[u].p[1].y, w[u].p[1].z, w[u].p[1].w}}, hi, a2[u]);
    };
#pragma unroll
    for (int t = 0; t < NT1; ++t) {
      floatx16 a1;
      B4 hi[2], lo[2];
      if constexpr (FP32_TILES) {
        tile.finish(a1);
        split_block(a1, 0, hi[0], lo[0]);
        split_block(a1, 1, hi[1], lo[1]);
#pragma unroll
        for (int u = 0; u < NT2; ++u) {
          if (__builtin_amdgcn_readfirstlane(wm[o.flags + 1 + u])) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
              const int q = 4 * t + g, plane = q / (2 * NT1);
              const float4 w = reinterpret_cast<const float4*>(w2)[(plane * NT2 * 2 * NT1 + u * 2 * NT1 + q % (2 * NT1)) * 64 + lane];
              a2[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(w.x, a1[4 * g + 0], a2[u], 0, 0, 0);
              a2[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(w.y, a1[4 * g + 1], a2[u], 0, 0, 0);
              a2[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(w.z, a1[4 * g + 2], a2[u], 0, 0, 0);
              a2[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(w.w, a1[4 * g + 3], a2[u], 0, 0, 0);
            }
          } else {
#pragma unroll
            for (int b = 0; b < 2; ++b) a2[u] = Lp::mma(Lp::load_w2(w2, t, b, u, lane), hi[b], lo[b], a2[u]);
          }
        }
        if (t + 1 < NT1) tile.load(t + 1);
        continue;
      }
      typename Lp::A4 w_a[NT2], w_b[NT2];
#pragma unroll
      for (int u = 0; u < NT2; ++u) w_a[u] = Lp::load_w2(w2, t, 0, u, lane);
      __builtin_amdgcn_sched_barrier(0);
      tile.finish(a1);
      split_block(a1, 0, hi[0], lo[0]);
      split_block(a1, 1, hi[1], lo[1]);
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) asm volatile("" : "+v"(lo[b].w[jj]));
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < NT2; ++u) w_b[u] = Lp::load_w2(w2, t, 1, u, lane);
      block(w_a, hi[0], lo[0]);
      __builtin_amdgcn_sched_barrier(0);
      if (t + 1 < NT1) tile.load(t + 1);
      block(w_b, hi[1], lo[1]);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int u = 0; u < NT2; ++u) {
      float4 q[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) q[g] = wo[(u * 4 + g) * 2 + h];
      sigmoid16(a2[u]);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        part = fmaf(q[g].x, a2[u][4 * g + 0], part);
        part = fmaf(q[g].y, a2[u][4 * g + 1], part);
        part = fmaf(q[g].z, a2[u][4 * g + 2], part);
        part = fmaf(q[g].w, a2[u][4 * g + 3], part);
      }
      asm volatile("" : "+v"(part));
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  return part;
}

// The same for two tiles of 32 configurations at once: for second layers of three or four tiles of
// units, whose accumulators leave room for two waves per SIMD only.  Two waves do not keep the
// matrix cores and the vector ALU busy side by side by themselves (MFMA 0.40 and VALU 0.52 of the
// cycles, in turn), so the order inside the wave does: while the matrix instructions of one tile
// of configurations and 32 inputs run, the sigmoids of the other tile's (or the next) 32 inputs are
// formed and split, a few vector instructions behind each matrix instruction.
template <int NT1, int NT2, class Tile>
__device__ __forceinline__ void split_layers_pair(const uint32_t* wm, int lane, const NetOffsets& o, Tile (&tile)[2],
                                                  float (&out)[2]) {
  typedef LpNet<_Float16, 2, 1, NT1, NT2, true> Lp;
  typedef typename Lp::Tr Tr;
  const int h = lane >> 5;
  const float4* wo = reinterpret_cast<const float4*>(wm + o.wo);
  const float4* b2 = reinterpret_cast<const float4*>(wm + o.b2);
  const uint4* w2 = reinterpret_cast<const uint4*>(wm + o.w2);
  asm volatile("" ::: "memory");
  tile[0].load(0);
  floatx16 a2[2][NT2];
#pragma unroll
  for (int u = 0; u < NT2; ++u) {
    Lp::init_bias(b2, u, h, a2[0][u]);
    a2[1][u] = a2[0][u];
  }
  B4 hi[2][2], lo[2][2];                   // [tile of configurations][block of 16 inputs]
  floatx16 a1;
  // piece k = 0 .. 19 of forming and splitting 32 sigmoid values of tile c
  auto piece = [&](int k, int c) {
    if (k < 4) {
      tile[c].sums(a1, k);
#pragma unroll
      for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(a1[4 * k + j]));
    } else if (k < 12) {
      const int v = 2 * (k - 4);
      a1[v] = __builtin_amdgcn_rcpf(a1[v]);
      a1[v + 1] = __builtin_amdgcn_rcpf(a1[v + 1]);
      asm volatile("" : "+v"(a1[v]), "+v"(a1[v + 1]));
    } else {
      const int b = (k - 12) / 4, jj = (k - 12) % 4;
      split_pair(a1, b, jj, hi[c][b], lo[c][b]);
      asm volatile("" : "+v"(lo[c][b].w[jj]));
    }
  };
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < 20; ++k) piece(k, 0);
  __builtin_amdgcn_sched_barrier(0);
  constexpr int kSteps = 2 * NT1, kMatrix = 6 * NT2;
#pragma unroll
  for (int s = 0; s < kSteps; ++s) {
    const int c = s & 1, t = s >> 1, cn = 1 - c, tn = (s + 1) >> 1;
    // first the next step's table reads, then this step's first weights
    if (s + 1 < kSteps) tile[cn].load(tn);
    typename Lp::A4 w[2], w_next[2];
    w_next[0] = Lp::load_w2(w2, t, 0, 0, lane);
    w_next[1] = Lp::load_w2(w2, t, 0, 1, lane);
    __builtin_amdgcn_sched_barrier(0);
    int i = 0;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int u0 = 0; u0 < NT2; u0 += 2) {
        w[0] = w_next[0];
        w[1] = w_next[1];
        const int un = u0 + 2 < NT2 ? u0 + 2 : 0, bn = un ? b : b + 1;
        if (bn < 2) {
          w_next[0] = Lp::load_w2(w2, t, bn, un, lane);
          if (un + 1 < NT2) w_next[1] = Lp::load_w2(w2, t, bn, un + 1, lane);
        }
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
          for (int d = 0; d < 2; ++d) {
            if (u0 + d >= NT2) continue;
            const uint4 q = w[d].p[p < 2 ? 0 : 1];
            a2[c][u0 + d] = Tr::mfma(B4{{q.x, q.y, q.z, q.w}}, p == 1 ? lo[c][b] : hi[c][b], a2[c][u0 + d]);
            // pieces from the third instruction on: the table reads have arrived by then
            if (s + 1 < kSteps) {
#pragma unroll
              for (int k = 0; k < 20; ++k)
                if (2 + k * (kMatrix - 2) / 20 == i) piece(k, cn);
            }
            ++i;
            __builtin_amdgcn_sched_barrier(0);
          }
      }
  }
  float part[2] = {0.0f, 0.0f};
#pragma unroll
  for (int u = 0; u < NT2; ++u) {
    float4 q[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) q[g] = wo[(u * 4 + g) * 2 + h];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      sigmoid16(a2[c][u]);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        part[c] = fmaf(q[g].x, a2[c][u][4 * g + 0], part[c]);
        part[c] = fmaf(q[g].y, a2[c][u][4 * g + 1], part[c]);
        part[c] = fmaf(q[g].z, a2[c][u][4 * g + 2], part[c]);
        part[c] = fmaf(q[g].w, a2[c][u][4 * g + 3], part[c]);
      }
      asm volatile("" : "+v"(part[c]));
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  out[0] += part[0];
  out[1] += part[1];
}

// flag 0 and those of layer 2's tiles
template <int NT2>
__device__ __forceinline__ bool split_flags(const uint32_t* wm, const NetOffsets& o) {
  uint32_t any = 0u;
#pragma unroll
  for (int u = 0; u <= NT2; ++u) any |= wm[o.flags + u];
  return __builtin_amdgcn_readfirstlane(any) != 0u;
}

// First layer of net_f32.h or net_f32h.h (fp32 matrix instructions), two-plane second layer: for
// lists of configurations and for spaces without a suitable span.
template <class L1, int NT1, int NT2>
struct SplitNet : L1 {
  typedef typename L1::Feat Feat;
  static __device__ __forceinline__ float forward(const uint32_t* wm, const Feat& f, int lane,
                                                  const NetOffsets& o, const float* xs = nullptr, float* zs = nullptr) {
    struct Tile {
      floatx16 a1[NT1];
      int next = 0;
      __device__ __forceinline__ void load(int) {}
      __device__ __forceinline__ void finish(floatx16& a) {
        a = a1[next++];
        sigmoid16(a);
      }
    } tile;
    L1::layer1(reinterpret_cast<const float*>(wm), f, lane, o, xs, zs, tile.a1);
    if (split_flags<NT2>(wm, o)) return split_layers<NT1, NT2, true>(wm, lane, o, tile);
    return split_layers<NT1, NT2, false>(wm, lane, o, tile);
  }
};

// ROWS_SHARED (one hidden layer, resident ensemble): the rows of a whole chunk are computed by the
// workgroup for all members before the chunk is evaluated, instead of by every wave for its own
// tiles, member by member.  A wave's pass over its rows is a chain of LDS reads, sums, an
// exponential and a write before the member can begin; with one tile per wave it cost more than
// the member (655,360 configurations, 11 x 10-30-1, all predictions: 72 us, shared 57; with two
// tiles per wave a pass serves both: 2,359,296 x 11-30-1 155 us, shared 162).
// TABLES_IN_MEMORY: TB and WH stay in memory (a member's are 22 KB and serve from the L1) where the
// second layer's weights alone fill the two stage buffers: [(t, g)][span][2][4] instead of the
// swizzled rows, so that the lanes of a wave read side by side.
template <int NT1, int NT2, bool TABLES_IN_MEMORY = false, bool ROWS_SHARED = false>
struct FactoredNet {
  static constexpr int kTile = 32;
  static constexpr bool kHoist = false;
  static constexpr bool kRows = true;
  static constexpr bool kRowsShared = ROWS_SHARED;
  static constexpr bool kPair = NT2 >= 3;
  static constexpr bool kTablesInMemory = TABLES_IN_MEMORY;
  static constexpr int kUnits = NT1 * 32;
  static constexpr int kRowFloats = kUnits + 4;   // scratch row (rows are read side by side: 4 floats apart in the banks)
  struct Feat { uint32_t tb, zs; };               // byte offsets of the lane's place in TB and of its row in the scratch

  // whether any of the nm members of a stage has a flag set (uniform)
  static __device__ __forceinline__ bool any_flags(const uint32_t* stage, int nm, int member_words, int lane, const NetOffsets& o) {
    bool any = false;
    for (int m = lane; m < nm; m += 64)
#pragma unroll
      for (int u = 0; u <= NT2; ++u) any = any || stage[(size_t)m * member_words + o.flags + u] != 0u;
    return __ballot(any) != 0ull;
  }

  // `at` = the lane's configuration counted from the start of the wave's (the chunk's) first row
  static __device__ __forceinline__ void place(uint32_t at, int lane, const NetOffsets& o, Feat& f) {
    const uint32_t h = (uint32_t)lane >> 5;
    const uint32_t row = (at * o.span_magic) >> 20, lo = at - row * o.span;
    f.tb = TABLES_IN_MEMORY ? lo * 32u + (h << 4) : lo * (kUnits * 4u) + ((h ^ (lo & 7u)) << 4);
    f.zs = row * (kRowFloats * 4u) + (h << 4);
  }

  // xs[row][p]: feature of high parameter p in a row, 1 at p = p0 (the bias), 0 beyond; by the
  // wave (tid = lane, threads = 64) or the workgroup
  static __device__ __forceinline__ void load_rows(const DevSpace& sp, uint32_t row0, uint32_t n_rows, uint32_t tid,
                                                   uint32_t threads, bool pow2, const NetOffsets& o, float* xs) {
    const int p = (int)(tid & 31u);
    for (uint32_t r = tid >> 5; r < n_rows; r += threads / 32u) {
      const float x = feature_at(sp, p, (row0 + r) * o.span, pow2);
      xs[r * 32 + p] = p < o.p0 ? x : (p == o.p0 ? 1.0f : 0.0f);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }

  // Once per member: 2^z_row[u] (or z_row[u], flag 0) of every unit for the wave's rows
  // (`tables`: the member's TB and WH, in memory or in LDS like the rest of it)
  static __device__ __forceinline__ void rows(const uint32_t* wm, const uint32_t* tables, uint32_t n_rows, bool flagged,
                                              int lane, const NetOffsets& o, const float* xs, float* zs) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const float4* wh = reinterpret_cast<const float4*>(tables + o.wh);
    const float4* x4 = reinterpret_cast<const float4*>(xs);
    const bool plain = flagged && __builtin_amdgcn_readfirstlane(wm[o.flags]) != 0u;
    for (uint32_t r0 = 0; r0 < n_rows; r0 += kRowsPerPass) row_pass(wh, x4, r0, plain, lane, o, zs);
    // a wave's LDS instructions execute in program order; the fences keep the compiler from
    // moving the reads of forward() above these writes, or the next member's writes above them
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }

  // The rows of a chunk for all members, by the workgroup's waves in turn (ROWS_SHARED); the
  // caller puts barriers around it.
  static __device__ __forceinline__ void rows_of_chunk(const uint32_t* wts, int n_members, int member_words, uint32_t n_rows,
                                                       uint32_t wave, uint32_t waves, bool flagged, int lane,
                                                       const NetOffsets& o, const float* xs, float* zs) {
    const uint32_t passes = (n_rows + kRowsPerPass - 1) / kRowsPerPass, tasks = passes * (uint32_t)n_members;
    for (uint32_t task = wave; task < tasks; task += waves) {
      const uint32_t m = task / passes, r0 = (task - m * passes) * kRowsPerPass;
      const uint32_t* wm = wts + (size_t)m * member_words;
      const bool plain = flagged && __builtin_amdgcn_readfirstlane(wm[o.flags]) != 0u;
      row_pass(reinterpret_cast<const float4*>(wm + o.wh), reinterpret_cast<const float4*>(xs), r0, plain, lane, o,
               zs + (size_t)m * o.rows * kRowFloats);
    }
  }

  static constexpr uint32_t kRowsPerPass = kUnits == 32 ? 2u : 1u;
  static __device__ __forceinline__ void row_pass(const float4* wh, const float4* x4, uint32_t r0, bool plain, int lane,
                                                  const NetOffsets& o, float* zs) {
    const int groups = (o.p0 + 4) >> 2;
    constexpr int kPer = (kUnits + 63) / 64;                  // units per lane
    const int u = kUnits == 32 ? (lane & 31) : lane;
    {
      const uint32_t r = r0 + (kUnits == 32 ? (uint32_t)lane >> 5 : 0u);
      float z[kPer];
#pragma unroll
      for (int q = 0; q < kPer; ++q) z[q] = 0.0f;
      for (int g = 0; g < groups; ++g) {
        const float4 x = x4[r * 8 + g];
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
          const float4 w = wh[g * kUnits + (kUnits == 96 && q ? 64 + (u & 31) : u + 64 * q)];
          z[q] = fmaf(w.x, x.x, z[q]);
          z[q] = fmaf(w.y, x.y, z[q]);
          z[q] = fmaf(w.z, x.z, z[q]);
          z[q] = fmaf(w.w, x.w, z[q]);
        }
      }
#pragma unroll
      for (int q = 0; q < kPer; ++q)
        zs[r * kRowFloats + (kUnits == 96 && q ? 64 + (u & 31) : u + 64 * q)] = plain ? z[q] : __builtin_amdgcn_exp2f(z[q]);
    }
  }

  // flagged: some member of the stage has a flag set
  static __device__ __forceinline__ float forward(const uint32_t* wm, const uint32_t* tables, bool flagged, const Feat& f,
                                                  int lane, const NetOffsets& o, const float* zs) {
    if (flagged) return forward_t<true>(wm, tables, f, lane, o, zs);
    return forward_t<false>(wm, tables, f, lane, o, zs);
  }
  // two tiles at once (kPair): the sums are added to y
  static __device__ __forceinline__ void forward_pair(const uint32_t* wm, const uint32_t* tables, bool flagged,
                                                      const Feat (&f)[2], int lane, const NetOffsets& o, const float* zs,
                                                      float (&y)[2]) {
    if (flagged) {
      for (int c = 0; c < 2; ++c) y[c] += forward_t<true>(wm, tables, c ? f[1] : f[0], lane, o, zs);
      return;
    }
    Tile<false> tile[2];
    tile[0].init(wm, tables, f[0], o, zs);
    tile[1].init(wm, tables, f[1], o, zs);
    split_layers_pair<NT1, NT2>(wm, lane, o, tile, y);
  }
  // FLAGS: exponents in the tables or fp32 tiles in layer 2, as the member's flags say
  template <bool FLAGS>
  static __device__ __forceinline__ float forward_t(const uint32_t* wm, const uint32_t* tables, const Feat& f, int lane,
                                                    const NetOffsets& o, const float* zs) {
    Tile<FLAGS> tile;
    tile.init(wm, tables, f, o, zs);
    return split_layers<NT1, NT2, FLAGS>(wm, lane, o, tile);
  }

  template <bool FLAGS>
  struct Tile {
    const char *tb, *zb;
    uint32_t at, exponents, step;
    float4 eh[4], el[4];
    __device__ __forceinline__ void init(const uint32_t* wm, const uint32_t* tables, const Feat& f, const NetOffsets& o,
                                         const float* zs) {
      tb = reinterpret_cast<const char*>(tables + o.w1);
      zb = reinterpret_cast<const char*>(zs) + f.zs;
      at = f.tb;
      step = o.span * 32u;
      exponents = FLAGS ? (uint32_t)__builtin_amdgcn_readfirstlane(wm[o.flags]) : 0u;
    }
    __device__ __forceinline__ void load(int t) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        if constexpr (TABLES_IN_MEMORY) el[g] = *reinterpret_cast<const float4*>(tb + (uint32_t)(t * 4 + g) * step + at);
        else el[g] = *reinterpret_cast<const float4*>(tb + (at ^ (uint32_t)(g << 5)) + t * 128);
        eh[g] = *reinterpret_cast<const float4*>(zb + t * 128 + g * 32);
      }
    }
    // 1 + 2^z of units 4 g + j
    __device__ __forceinline__ void sums(floatx16& a, int g) {
      a[4 * g + 0] = fmaf(eh[g].x, el[g].x, 1.0f);
      a[4 * g + 1] = fmaf(eh[g].y, el[g].y, 1.0f);
      a[4 * g + 2] = fmaf(eh[g].z, el[g].z, 1.0f);
      a[4 * g + 3] = fmaf(eh[g].w, el[g].w, 1.0f);
    }
    __device__ __forceinline__ void finish(floatx16& a) {
      if (FLAGS && exponents) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          a[4 * g + 0] = 1.0f + __builtin_amdgcn_exp2f(eh[g].x + el[g].x);
          a[4 * g + 1] = 1.0f + __builtin_amdgcn_exp2f(eh[g].y + el[g].y);
          a[4 * g + 2] = 1.0f + __builtin_amdgcn_exp2f(eh[g].z + el[g].z);
          a[4 * g + 3] = 1.0f + __builtin_amdgcn_exp2f(eh[g].w + el[g].w);
        }
      } else {
#pragma unroll
        for (int g = 0; g < 4; ++g) sums(a, g);
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) a[v] = __builtin_amdgcn_rcpf(a[v]);
    }
  };
};

// ---- packing --------------------------------------------------------------------------------
// Weights enter the products as w' = -log2(e) w, formed in double and rounded where they are
// stored.
constexpr double kNegLog2eD = -1.4426950408889634073599246810019;

// 2^z to 0.6 ulp for |z| <= 120: the Taylor polynomial of 2^f on [-1/2, 1/2] (its remainder is
// 5e-9), whose last step rounds once; a dozen fp32 operations where exp2(double) takes a hundred
// double ones.
__device__ __forceinline__ float exp2_of(double z) {
  const double n = rint(z);
  const float f = (float)(z - n);
  float q = 1.525273380e-05f;
  q = fmaf(q, f, 1.540353039e-04f);
  q = fmaf(q, f, 1.333355815e-03f);
  q = fmaf(q, f, 9.618129108e-03f);
  q = fmaf(q, f, 5.550410866e-02f);
  q = fmaf(q, f, 2.402265070e-01f);
  q = fmaf(q, f, 6.931471806e-01f);
  return ldexpf(fmaf(q, f, 1.0f), (int)n);
}

// The words of one member that stand for themselves (fp32 first layers): everything but W2A and
// the flags, which the workgroups below write.
__device__ inline bool split_word_is_plain(const Shape& sh, int q) {
  return q < sh.o_flags && !(q >= sh.o_w2 && q < sh.o_b2);
}
__device__ inline float split_plain_word(const Shape& sh, const float* raw, int q) {
  if (sh.hoist) return pack_word_f32h(sh, raw, q);
  return pack_word_f32(sh, raw, q);
}

// LDS of the packing workgroups: the raw weights they work on, and the features of the low
// parameters at every place of a row.
struct PackScratch {
  float w[(TUNER_MAX_PARAMS + 1) * TUNER_MAX_WIDTH];
  float x[128 * TUNER_MAX_PARAMS];
  uint32_t any;
};
constexpr int kMaxSpan = 128;
// Words of TB one workgroup writes: the more workgroups the shorter the chain, until the members
// alone fill the chip (500 members of 64 units, 100 configurations: 745 us with 512, 730 with 2048).
__host__ __device__ inline int split_table_slice(const Shape& sh) { return sh.E >= 128 ? 2048 : 512; }
// Workgroups that pack a member's factored first layer: one per slice of TB, and one for the rest.
__host__ __device__ inline int split_table_jobs(const Shape& sh) {
  return sh.span ? (sh.span * sh.NT1 * 32 + split_table_slice(sh) - 1) / split_table_slice(sh) + 1 : 0;
}

// put(x, src[x]) for x = 0 .. n - 1 by 256 threads, eight loads of a thread in flight.
template <class Put>
__device__ __forceinline__ void stage_words(const float* src, int n, Put put) {
  for (int x0 = (int)threadIdx.x; x0 < n; x0 += 8 * 256) {
    float v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = src[min(x0 + 256 * q, n - 1)];
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (x0 + 256 * q < n) put(x0 + 256 * q, v[q]);
  }
}

// A workgroup of 256 threads writes one slice of TB of one member (factored layout), the last
// one WH, b2A, woA and flag 0 instead.  Everything is read into LDS first, in one trip to memory.
// What bounds it is the chain of one thread (a double-precision sum and exp2 per word), so the
// slices are short: with 512 words instead of 2048 the packing of 11 x (11-30-1) takes 5.5 us
// instead of 8.1.
// `tables`: where the member's TB and WH go (the member itself, or its place behind all members).
__device__ inline void pack_factored(const Shape& sh, const float* raw, uint32_t* member, uint32_t* tables, const DevSpace& sp,
                                     int slice, PackScratch& s) {
  const int tid = threadIdx.x, units = sh.NT1 * 32, n_low = sh.P - sh.p0;
  const bool pow2 = sp.all_pow2 != 0;
  if (tid == 0) s.any = 0u;
  stage_words(raw, sh.H1 * (sh.P + 1), [&](int x, float v) { s.w[x] = v; });       // W1, then b1
  const bool rest = slice == split_table_jobs(sh) - 1;
  const int begin = slice * split_table_slice(sh);
  const int end = rest ? begin : min(begin + split_table_slice(sh), sh.span * units);
  const int l0 = begin / units, n_x = rest ? 0 : ((end - 1) / units - l0 + 1) * n_low;   // the slice's places
  for (int x = tid; x < n_x; x += 256) {
    const int l = x / n_low;
    s.x[x] = feature_at(sp, sh.p0 + (x - l * n_low), (uint32_t)(l0 + l), pow2);
  }
  const float* b1 = s.w + sh.H1 * sh.P;
  __syncthreads();
  if (tid < sh.H1) {
    float sum = fabsf(b1[tid]);
    for (int p = 0; p < sh.P; ++p) sum += fabsf(s.w[tid * sh.P + p]);
    if (!(sum * -kNegLog2e <= kFactoredMaxExponent)) atomicOr(&s.any, 1u);     // infinities and NaN too
  }
  __syncthreads();
  const bool plain = s.any != 0u;
  for (int x = begin + tid; x < end; x += 256) {
    const int l = x / units, u = x - l * units;
    double z = 0.0;
    if (u < sh.H1)
      for (int p = 0; p < n_low; ++p) z = fma((double)s.w[u * sh.P + sh.p0 + p], (double)s.x[(l - l0) * n_low + p], z);
    z *= kNegLog2eD;
    const int t = u >> 5, e = (u >> 2) & 7, j = u & 3;
    const int at = sh.table_words ? ((t * 4 + (e >> 1)) * sh.span + l) * 8 + (e & 1) * 4 + j
                                  : l * units + 32 * t + 4 * (e ^ (l & 7)) + j;
    tables[at] = __float_as_uint(plain ? (float)z : exp2_of(z));
  }
  if (!rest) return;
  if (tid == 0) member[sh.o_flags] = plain ? 1u : 0u;
  const int groups = (sh.p0 + 4) / 4;
  for (int x = tid; x < groups * units * 4; x += 256) {
    const int j = x & 3, u = (x >> 2) % units, p = 4 * ((x >> 2) / units) + j;
    float v = 0.0f;
    if (u < sh.H1 && p <= sh.p0) v = (float)((double)(p < sh.p0 ? s.w[u * sh.P + p] : b1[u]) * kNegLog2eD);
    tables[sh.o_wh + x] = __float_as_uint(v);
  }
  for (int x = tid; x < sh.NT2 * 32; x += 256) {
    // accumulator order [4][2][4]: word 8 g + 4 h + j of a tile is its unit 8 g + 4 h + j
    const float b = x < sh.H2 ? raw[sh.H1 * sh.P + sh.H1 + sh.H2 * sh.H1 + x] : 0.0f;
    member[sh.o_b2 + x] = __float_as_uint(b * kNegLog2e);
  }
  const int ntl = sh.NT2 ? sh.NT2 : sh.NT1, HL = sh.H2 ? sh.H2 : sh.H1;
  const float* wo = raw + sh.raw_member_floats - 1 - HL;
  for (int x = tid; x < ntl * 32; x += 256) member[sh.o_wo + x] = __float_as_uint(x < HL ? wo[x] : 0.0f);
}

// A workgroup of 256 threads writes the 32 rows (output units) of tile u of layer 2, both f16
// planes or fp32, and flag 1 + u.  Bound by the trips to memory of its first loop and by LDS: with
// eight loads in flight and an odd row pitch 16 members of 14-128-128-1 take 10.9 us instead of
// 13.1, 4 of 14-64-64-1 6.7 instead of 8.3.
__device__ inline void pack_split_w2(const Shape& sh, const float* raw, uint32_t* member, int u, PackScratch& s) {
  const int tid = threadIdx.x;
  const int r_w2 = sh.H1 * sh.P + sh.H1;
  const int n_rows = min(32, sh.H2 - 32 * u);                   // may be <= 0: a tile of padding
  if (tid == 0) s.any = 0u;
  __syncthreads();
  bool fits = true;
  const int pitch = sh.H1 | 1;                                  // odd: the lanes of a wave read 32 rows at once
  stage_words(raw + r_w2 + 32 * u * sh.H1, n_rows * sh.H1, [&](int x, float w) {
    const int n = x / sh.H1;
    s.w[n * pitch + (x - n * sh.H1)] = w;
    fits = fits && fabsf(w) * -kNegLog2e <= kSplitMaxWeight;    // false for NaN
  });
  if (!fits) atomicOr(&s.any, 1u);
  __syncthreads();
  const bool fp32 = s.any != 0u;
  const int half = 2 * sh.NT1 * 256, plane_words = sh.NT2 * half;
  uint32_t* out = member + sh.o_w2 + u * half;
  for (int x = tid; x < half; x += 256) {
    uint32_t hi = 0u, lo = 0u;
    if (!fp32) {
      const int jj = x & 3, lane = (x >> 2) & 63, kbg = x >> 8;
      const int n = lane & 31, h = lane >> 5;
      for (int k = 0; k < 2; ++k) {
        const int j = 2 * jj + k, in = 16 * kbg + 8 * (j >> 2) + 4 * h + (j & 3);
        if (n < n_rows && in < sh.H1) {
          const double v = (double)s.w[n * pitch + in] * kNegLog2eD;
          const _Float16 a = (_Float16)(float)v;
          const _Float16 r = (_Float16)(float)(v - (double)(float)a);
          hi |= (uint32_t)__builtin_bit_cast(uint16_t, a) << (16 * k);
          lo |= (uint32_t)__builtin_bit_cast(uint16_t, r) << (16 * k);
        }
      }
    } else {
      // words x and half + x of the tile's [NT1][4][64 lanes][4]
      for (int k = 0; k < 2; ++k) {
        const int q = x + k * half, j = q & 3, lane = (q >> 2) & 63, g = (q >> 8) & 3, t = q >> 10;
        const int n = lane & 31, in = 32 * t + 8 * g + 4 * (lane >> 5) + j;
        const float v = n < n_rows && in < sh.H1 ? s.w[n * pitch + in] * kNegLog2e : 0.0f;
        (k ? lo : hi) = __float_as_uint(v);
      }
    }
    out[x] = hi;
    out[plane_words + x] = lo;
  }
  if (tid == 0) member[sh.o_flags + 1 + u] = fp32 ? 1u : 0u;
}

}  // namespace tuner
