// Last step of the token-major backward when its sub-networks were shared out over several
// workgroups (few tokens: bwd.hip, bwd_f32.hip).  Every share left dr_e of its own
// sub-networks and an fp32 partial of dX; here, per token and head,
//   ds_e = (dr_e - sum_e' dr_e' r_e') / (Z + eps),  dp_e = ds_e s_e (1 - s_e)   (params mode)
//   dX   = sum_shares partial + dp W_r^T
// A wave takes 16 tokens of one head.  The lane group gq of a token walks the sub-networks
// 4 k + gq, which is how the fp32 product dp W_r^T (f32_tiles.h) wants its operand, so nothing
// passes through LDS.  Bound: reading the partials, by few waves that wait for memory, so all quads of a
// share are in flight at once.  bf16 partials lie as the token-major kernel's registers held them
// (256 bytes a load, not 64 bytes of each of 16 rows): three shares of 1536 x 2048, 384 workgroups,
// weights given, 9.7 us; two took 10.6 as rows.
#include "f32_tiles.h"
#include "mhffn_internal.h"

namespace mhffn {
namespace {

__device__ __forceinline__ float wide(float v) { return v; }
__device__ __forceinline__ float wide(uint16_t v) { return bf16_bits_to_f32(v); }
__device__ __forceinline__ void store4(float* p, f32x4 v) { *reinterpret_cast<f32x4*>(p) = v; }
__device__ __forceinline__ void store8(uint16_t* p, f32x4 v, f32x4 w) {
  *reinterpret_cast<u32x4*>(p) = u32x4{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(w[0], w[1]), pack_bf16(w[2], w[3])};
}

template <typename T, int DHP>
__global__ __launch_bounds__(256) void bwd_tok_finish_kernel(BwdFinish a) {
  constexpr int JG = f32_col_groups(DHP);
  const int lane = threadIdx.x & 63;
  const int i16 = lane & 15, gq = lane >> 4;
  const uint32_t waves = (uint32_t)a.block_tokens / 16, per_head = (uint32_t)((a.N + a.block_tokens - 1) / a.block_tokens);
  const uint32_t item = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (item >= a.n_units * waves) return;
  const uint32_t unit = item / waves, block = a.first_unit + unit;
  const int h = (int)(block / per_head);
  const int64_t tok0 = (int64_t)(block % per_head) * a.block_tokens + 16 * (item % waves), tok = tok0 + i16;
  if (tok0 >= a.N) return;
  const bool ok = tok < a.N;
  const int64_t t = ok ? tok : a.N - 1;
  const int dh = a.dh, E = a.E;

  f32x4 acc[JG][4];
  if (a.dX) {
    // (all quads of a share in flight at once: there are few waves, and this is what they wait for)
    // bf16: columns 64 J + 16 gq + 4 v .. of token t are quad 8 J + 4 (gq / 2) + 2 (gq % 2) + v / 2,
    // lane half v % 2, of the [quad][lane] tile of its 32 tokens
    constexpr bool kTiles = sizeof(T) == 2;
    constexpr int kStepJ = kTiles ? 8 * 256 : 64;
    const size_t stride = kTiles ? (size_t)a.n_units * a.block_tokens * DHP : (size_t)a.N * a.H * dh;
    const float* src = kTiles ? a.P + ((size_t)item / 2) * 32 * DHP + (4 * (gq >> 1) + 2 * (gq & 1)) * 256 + (16 * (item & 1) + i16) * 4
                              : a.P + ((size_t)t * a.H + h) * dh + 16 * gq;
    f32x4 sum[JG][4];   // [J][v]
#pragma unroll
    for (int J = 0; J < JG; ++J)
#pragma unroll
      for (int v = 0; v < 4; ++v) sum[J][v] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
    for (int s = 0; s < a.shares; ++s, src += stride) {
#pragma unroll
      for (int J = 0; J < JG; ++J)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (kTiles || 64 * J + 16 * gq + 4 * v < dh)
            sum[J][v] += *reinterpret_cast<const f32x4*>(src + kStepJ * J + (kTiles ? (v >> 1) * 256 + (v & 1) * 128 : 4 * v));
    }
#pragma unroll
    for (int J = 0; J < JG; ++J)
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int n = 0; n < 4; ++n) acc[J][n][v] = sum[J][v][n];
  }
  if (a.params) {
    const float* R = a.R + (size_t)h * E * a.N + t;
    float* DP = a.DP + (size_t)h * E * a.N + t;
    float dot = 0.f;
#pragma unroll 4
    for (int e = gq; e < E; e += 4) dot = fmaf(DP[(size_t)e * a.N], R[(size_t)e * a.N], dot);
    dot = sum_lane_groups(dot);
    const float zinv = a.Zinv[(size_t)h * a.N + t], zpe = 1.0f / zinv;
    const T* Wr = static_cast<const T*>(a.Wr) + (size_t)h * dh * E;
    for (int eb = 0; eb < E; eb += 4) {
      const int e = eb + gq;
      const bool in = e < E;
      float dp = 0.f;
      if (in) {
        const float s = R[(size_t)e * a.N] * zpe;
        dp = (DP[(size_t)e * a.N] - dot) * zinv * s * (1.0f - s);
        if (ok) DP[(size_t)e * a.N] = dp;
      }
      if (a.dX) {
#pragma unroll
        for (int J = 0; J < JG; ++J)
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            const int j = 64 * J + 4 * i16 + n;
            const float w = (in && j < dh) ? wide(Wr[(size_t)j * E + e]) : 0.f;
            acc[J][n] = mfma16_f32(w, dp, acc[J][n]);
          }
      }
    }
  }
  if (a.dX && ok) {
    T* dst = static_cast<T*>(a.dX) + tok * a.ldx + (size_t)h * dh;
#pragma unroll
    for (int J = 0; J < JG; ++J)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int col = 64 * J + 16 * gq + 4 * v;
        auto quad = [&](int k) { return f32x4{acc[J][0][k], acc[J][1][k], acc[J][2][k], acc[J][3][k]}; };
        if constexpr (sizeof(T) == 2) {
          if (v % 2 == 0) store8(dst + col, quad(v), quad(v | 1));
        } else {
          if (col < dh) store4(dst + col, quad(v));
        }
      }
  }
}

template <typename T>
int launch(const BwdFinish& a, hipStream_t stream) {
  const dim3 grid((a.n_units * (uint32_t)(a.block_tokens / 16) + 3) / 4), block(256);
  switch (64 * ((a.dh + 63) / 64)) {
    case 64: hipLaunchKernelGGL((bwd_tok_finish_kernel<T, 64>), grid, block, 0, stream, a); break;
    case 128: hipLaunchKernelGGL((bwd_tok_finish_kernel<T, 128>), grid, block, 0, stream, a); break;
    case 192: hipLaunchKernelGGL((bwd_tok_finish_kernel<T, 192>), grid, block, 0, stream, a); break;
    default: hipLaunchKernelGGL((bwd_tok_finish_kernel<T, 256>), grid, block, 0, stream, a); break;
  }
  return (int)hipGetLastError();
}

}  // namespace

int launch_bwd_tok_finish(int dtype, const BwdFinish& a, void* stream) {
  if (!a.dX && !a.params) return 0;
  hipStream_t st = static_cast<hipStream_t>(stream);
  return dtype == 1 ? launch<uint16_t>(a, st) : launch<float>(a, st);
}

}  // namespace mhffn
