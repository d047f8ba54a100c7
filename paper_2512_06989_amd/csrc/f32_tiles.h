// Shared pieces of the fp32 kernels (fwd_f32.hip, bwd_f32.hip): fp32 products on
// v_mfma_f32_16x16x4_f32, 16 rows x 16 columns x 4 contraction slots per instruction.
//
// Lane l of a wave: i = l % 16, gq = l / 16.
//   A operand: row i, slot gq;  B operand: column i, slot gq  (one float each)
//   D / C    : column i, register v (0..3) is row 4 gq + v
//
// Which index a slot stands for is free as long as both operands agree, and so is which
// matrix row an operand row stands for.  Both freedoms turn the operand reads into 16-byte
// LDS reads of tiles kept in their natural row-major layout:
//   * contraction along a row: chunk kk covers 16 columns and four products; in product n the
//     slot gq is column 16 kk + 4 gq + n, so one 16-byte read per lane feeds all four;
//   * contraction over rows ("transposed"): the slot gq of product v is row 4 gq + v (which is
//     how a D register of the previous product lies, so chained products stay in registers),
//     and one 16-byte read at column 64 J + 4 i feeds four output tiles: row i of tile (J, n)
//     is column 64 J + 4 i + n, and a lane's D registers of the four tiles are four
//     consecutive columns of an output row.
// A product takes 32 cycles for 2048 flop, so a CU consumes one operand read of 1 KB per
// 64 .. 128 cycles and SIMD: LDS bandwidth (128 B per cycle) is at most a quarter used.
#pragma once

#include "mhffn_device.h"

#include <type_traits>

namespace mhffn {

__device__ __forceinline__ f32x4 mfma16_f32(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float sigmoid_f32(float x) {
  // exact division, branch on sign so exp never overflows
  if (x >= 0.f) return 1.0f / (1.0f + __expf(-x));
  const float t = __expf(x);
  return t / (1.0f + t);
}

// sum over the four lane groups that share a D column (fixed order, same result in all)
__device__ __forceinline__ float sum_lane_groups(float v) {
  v += __shfl_xor(v, 16);
  v += __shfl_xor(v, 32);
  return v;
}

// Head width rounded up to the compiled widths (contraction along a row); outputs come in
// groups of 64 columns.
constexpr int f32_padded_width(int dh) { return dh <= 64 ? 64 : dh <= 96 ? 96 : dh <= 128 ? 128 : dh <= 192 ? 192 : 256; }
constexpr int f32_col_groups(int dhp) { return (dhp + 63) / 64; }
// Tiles hold 16 rows.  Row stride in floats: four words past a multiple of the 64 banks
// spread the 16 rows of an operand read over all banks.
constexpr int kF32Rows = 16;
constexpr int f32_ld(int dhp) { return 64 * f32_col_groups(dhp) + 4; }

// Runs use(n, load(n)) for n = 0 .. NI-1, each load issued one item ahead and not earlier: the
// operands of one item are all that is in flight, which is what keeps the register count
// within two to four waves per SIMD.
template <int NI, int N = 0, typename Op, typename L, typename U>
__device__ __forceinline__ void f32_stream_from(const Op& cur, const L& load, const U& use) {
  if constexpr (N < NI) {
    Op nxt;
    if constexpr (N + 1 < NI) nxt = load(std::integral_constant<int, N + 1>{});
    __builtin_amdgcn_sched_barrier(0);
    use(std::integral_constant<int, N>{}, cur);
    __builtin_amdgcn_sched_barrier(0);
    f32_stream_from<NI, N + 1>(nxt, load, use);
  }
}
template <int NI, typename L, typename U>
__device__ __forceinline__ void f32_stream(const L& load, const U& use) {
  f32_stream_from<NI>(load(std::integral_constant<int, 0>{}), load, use);
}
// Waits for loads into resident operands here.  Left to itself the compiler puts that wait at
// their first use, inside the tile loop, where it would hold every pass until the tile just
// requested has arrived.
template <int N>
__device__ __forceinline__ void f32_settle(f32x4 (&x)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(x[i]));
}
struct F32Op1 { f32x4 a; };
struct F32Op2 { f32x4 a, b; };
struct F32Op3 { f32x4 a, b, c; };
__device__ __forceinline__ f32x4 lds_f32x4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }

// How many workgroups share one unit of work (the tiles of a token block, the tokens of a
// neuron group) so that the chip is evenly loaded.  The time is taken as that of the CU with the
// most workgroups, ceil(items * s / 256), times the steps of one, plus what a split costs
// (partials written and read back), `step_cost` and `split_cost` (per split) in the same unit.
// How many of a CU's workgroups run at once is not in the rule: by registers (head width 64 / 96,
// 128 / 192, 256) five / three / two of the forward's, four / two / one of the token-major
// sweep's, three / two / one of the weight-major sweep's.
inline int f32_plan_splits(int64_t items, int64_t steps, double step_cost, double split_cost, double fixed_cost,
                           int max_splits) {
  int best = 1;
  double best_cost = 0;
  for (int s = 1; s <= max_splits && s <= steps; ++s) {
    const int64_t per = (steps + s - 1) / s;
    if (s > 1 && (steps + per - 1) / per != s) continue;   // s workgroups would not all have work
    const double cost = (double)((items * s + 255) / 256) * per * step_cost + (s > 1 ? fixed_cost + s * split_cost : 0);
    if (s == 1 || cost < best_cost) { best = s; best_cost = cost; }
  }
  return best;
}

}  // namespace mhffn
