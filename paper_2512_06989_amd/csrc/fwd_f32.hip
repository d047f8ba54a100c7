// Fused Multi-Head FFN forward in fp32 (storage and arithmetic), gfx950.
//
// Shape-generic companion of the bf16 kernels: any E, any d_e, d_h a multiple of 4 up to 256.
// Same structure as eq:flash-ffn-loop / appendix algorithm "SRAMFFN-Forward": a wave owns 16
// tokens of one head (q as operands in registers), a workgroup of NW waves walks the
// intermediate dimension in tiles of 16 neurons whose K, U, V rows are staged in LDS (one
// tile in LDS, the next one in registers); M, N, A and the output accumulator never leave the
// chip.  All three contractions run on v_mfma_f32_16x16x4_f32, transposed (neurons or output
// columns on the MFMA rows, tokens on the columns) as in the bf16 kernels: the accumulator of
// the gate/up products is, register for register, the operand of the down projection.
//
// Bound: the fp32 matrix rate (157 TFLOP/s; one product per 32 cycles and SIMD).  Several
// small workgroups per CU (64 tokens, 29 KB of LDS at E = 16) hide each other's staging and
// activation.  When token blocks x heads cannot load the 256 CUs evenly the tiles of a block
// are shared out over several workgroups whose fp32 partial outputs a second kernel adds up
// in fixed order.  2000 tokens, H = 6, E = 16, d_e = 128: 0.191 ms with the sum over the
// shares (99 TFLOP/s, MFMA busy 67 %), against 1.50 ms of the plain-FMA kernel it replaces
// (32 tokens per workgroup, operands read from LDS one float at a time).
#include "f32_tiles.h"
#include "mhffn_internal.h"

namespace mhffn {
namespace {

constexpr int kMaxDh = 256;

struct F32Args {
  const float* X;
  const float* Wg;
  const float* Wu;
  const float* Wd;
  const void* route;
  float* Y;
  float* P;     // [n_split][N][H*dh] partial outputs (only when n_split > 1 and there is scratch)
  int64_t N, ldx, ldy, n_tiles, n_items;
  int H, dh, E, de, route_mode;
  int n_split, tiles_per_split;
  float eps;
};

// SERIAL: the shares of a token block run one after the other (no scratch); a workgroup then adds
// them up in Y as the reduce kernel adds their partials, so the result does not depend on the
// scratch.  (An instantiation of its own: as a branch it cost the other one 3 %.)  What it costs,
// with scratch | without: 2000 tokens, H = 6, E = 16, d_e = 128 181 | 274 us (1448 of the
// plain-FMA kernel, which took none), 4200 tokens, H = 8 505 | 647 (3834), 16 tokens, H = 6, where
// six workgroups are all there is, 21 | 311 (1147).
template <int DHP, int NW, bool SERIAL>
__global__ __launch_bounds__(64 * NW, DHP <= 64 ? 4 : DHP <= 128 ? 3 : 2) void fwd_f32_kernel(F32Args a) {
  constexpr int THREADS = 64 * NW, BT = 16 * NW;
  constexpr int KC = DHP / 16, JG = f32_col_groups(DHP), LD = f32_ld(DHP), TILE = kF32Rows * LD;
  constexpr int CPT = (kF32Rows * DHP / 4 + THREADS - 1) / THREADS;   // 16-byte chunks of a tile per thread
  extern __shared__ __attribute__((aligned(16))) float smem_f[];
  float* Ks = smem_f;                     // [16][LD]
  float* Us = Ks + TILE;
  float* Vs = Us + TILE;
  float* Rs = Vs + TILE;                  // [E][BT]

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i16 = lane & 15, gq = lane >> 4;
  const int dh = a.dh, E = a.E, de = a.de;
  const int cpr = dh >> 2;                            // 16-byte chunks per row
  const int64_t item = xcd_work_item(blockIdx.x, a.n_items);
  if (item >= a.n_items) return;  // whole workgroup leaves together
  const int split = SERIAL ? 0 : (int)(item % a.n_split);
  const int64_t ht = SERIAL ? item : item / a.n_split;
  const int h = (int)(ht / a.n_tiles);
  const int64_t tok0 = (ht % a.n_tiles) * BT;
  const int wtok = 16 * wave + i16;                   // token of this lane inside the block
  const int64_t tok = tok0 + wtok;
  const bool active = tok0 + 16 * wave < a.N;

  // ---- weight-tile stream: global -> registers -> LDS --------------------------
  // (rows of a tile are contiguous in memory; rows past the sub-network's width are zero)
  const int cps = (de + kF32Rows - 1) / kF32Rows;     // tiles per sub-network
  const int t_begin = split * a.tiles_per_split;
  const int t_end = SERIAL ? E * cps : min(E * cps, t_begin + a.tiles_per_split);
  const size_t head_off = (size_t)h * E * de * dh;
  int loff[CPT];
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int idx = tid + THREADS * c;
    loff[c] = idx < kF32Rows * cpr ? (idx / cpr) * LD + 4 * (idx % cpr) : -1;
  }
  f32x4 kreg[CPT], ureg[CPT], vreg[CPT];
  auto gload = [&](int t) {
    const int e = t / cps, cb = (t - e * cps) * kF32Rows;
    const int n4 = min(kF32Rows, de - cb) * cpr;      // valid 16-byte chunks
    const size_t base = head_off + ((size_t)e * de + cb) * dh;
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      const int idx = tid + THREADS * c;
      kreg[c] = ureg[c] = vreg[c] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (idx < n4) {
        kreg[c] = *reinterpret_cast<const f32x4*>(a.Wg + base + 4 * idx);
        ureg[c] = *reinterpret_cast<const f32x4*>(a.Wu + base + 4 * idx);
        vreg[c] = *reinterpret_cast<const f32x4*>(a.Wd + base + 4 * idx);
      }
    }
  };
  gload(t_begin);

  // ---- q operands: slot (kk, n) of lane group gq is column 16 kk + 4 gq + n -----------
  f32x4 q[KC];
  {
    const float* src = a.X + (tok < a.N ? tok : 0) * a.ldx + (size_t)h * dh;
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
      const int col = 16 * kk + 4 * gq;
      q[kk] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (tok < a.N && col < dh) q[kk] = *reinterpret_cast<const f32x4*>(src + col);
    }
  }
  // columns dh.. of the tiles are read as operands and never staged
  const int pad = 64 * JG - dh;
  for (int idx = tid; idx < 3 * kF32Rows * pad; idx += THREADS) Ks[(idx / pad) * LD + dh + idx % pad] = 0.f;

  // ---- gating weights: eq:routing (every lane writes and later reads its own token) ----
  if (a.route_mode == 0) {
    const float* Wr = reinterpret_cast<const float*>(a.route) + (size_t)h * dh * E;
    float z = 0.f;
    if (active) {
      for (int eb = 0; eb < E; eb += 16) {
        const bool ok = eb + i16 < E;
        f32x4 p = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < KC; ++kk)
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            const int j = 16 * kk + 4 * gq + n;
            const float w = (ok && j < dh) ? Wr[(size_t)j * E + eb + i16] : 0.f;
            p = mfma16_f32(w, q[kk][n], p);
          }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int e = eb + 4 * gq + v;
          if (e < E) {
            const float s = sigmoid_f32(p[v]);
            z += s;
            Rs[e * BT + wtok] = s;
          }
        }
      }
      const float inv = 1.0f / (sum_lane_groups(z) + a.eps);
      for (int eb = 0; eb < E; eb += 16)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int e = eb + 4 * gq + v;
          if (e < E) Rs[e * BT + wtok] *= inv;
        }
    }
  } else {
    const float* R = reinterpret_cast<const float*>(a.route);
    for (int idx = tid; idx < BT * E; idx += THREADS) {
      const int t = idx / E, e = idx - t * E;
      Rs[e * BT + t] = (tok0 + t < a.N) ? R[((size_t)(tok0 + t) * a.H + h) * E + e] : 0.f;
    }
  }

  f32x4 O[JG][4];
#pragma unroll
  for (int J = 0; J < JG; ++J)
#pragma unroll
    for (int n = 0; n < 4; ++n) O[J][n] = f32x4{0.f, 0.f, 0.f, 0.f};

  const float* krow = Ks + i16 * LD + 4 * gq;
  const float* urow = Us + i16 * LD + 4 * gq;
  const float* vcol = Vs + 4 * gq * LD + 4 * i16;
  f32_settle(q);
  // ---- store: lane = token, register v of the four tiles = columns 64 J + 16 gq + 4 v .. +3 ----
  auto store = [&](bool first) __attribute__((always_inline)) {
    if (tok >= a.N) return;
    float* dst = !SERIAL && a.n_split > 1 ? a.P + (((size_t)split * a.N + tok) * a.H + h) * dh
                                          : a.Y + tok * a.ldy + (size_t)h * dh;
#pragma unroll
    for (int J = 0; J < JG; ++J)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int col = 64 * J + 16 * gq + 4 * v;
        if (col < dh) {
          f32x4 o = {O[J][0][v], O[J][1][v], O[J][2][v], O[J][3][v]};
          if constexpr (SERIAL) {
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            o = (first ? zero : *reinterpret_cast<const f32x4*>(dst + col)) + o;
          }
          *reinterpret_cast<f32x4*>(dst + col) = o;
        }
      }
  };
  int left = a.tiles_per_split;   // tiles of the share that are left
  for (int t = t_begin; t < t_end; ++t) {
    if constexpr (SERIAL) {
      if (left == 0) {
        store(t == a.tiles_per_split);
#pragma unroll
        for (int J = 0; J < JG; ++J)
#pragma unroll
          for (int n = 0; n < 4; ++n) O[J][n] = f32x4{0.f, 0.f, 0.f, 0.f};
        left = a.tiles_per_split;
      }
      --left;
    }
    __syncthreads();   // everyone is done with the previous tile (first pass: R and the padding are written)
#pragma unroll
    for (int c = 0; c < CPT; ++c)
      if (loff[c] >= 0) {
        *reinterpret_cast<f32x4*>(Ks + loff[c]) = kreg[c];
        *reinterpret_cast<f32x4*>(Us + loff[c]) = ureg[c];
        *reinterpret_cast<f32x4*>(Vs + loff[c]) = vreg[c];
      }
    __syncthreads();
    if (t + 1 < t_end) gload(t + 1);
    if (!active) continue;
    const float rw = Rs[(t / cps) * BT + wtok];
    f32x4 m = {0.f, 0.f, 0.f, 0.f}, nn = {0.f, 0.f, 0.f, 0.f};
    f32_stream<KC>(
        [&](auto K_) { return F32Op2{lds_f32x4(krow + 16 * K_.value), lds_f32x4(urow + 16 * K_.value)}; },
        [&](auto K_, const F32Op2& o) {
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            m = mfma16_f32(o.a[n], q[K_.value][n], m);
            nn = mfma16_f32(o.b[n], q[K_.value][n], nn);
          }
        });
    f32x4 act;
#pragma unroll
    for (int v = 0; v < 4; ++v) act[v] = m[v] * sigmoid_f32(m[v]) * nn[v] * rw;
    f32_stream<4 * JG>(
        [&](auto S_) { return F32Op1{lds_f32x4(vcol + (S_.value / JG) * LD + 64 * (S_.value % JG))}; },
        [&](auto S_, const F32Op1& o) {
          constexpr int v = S_.value / JG, J = S_.value % JG;
#pragma unroll
          for (int n = 0; n < 4; ++n) O[J][n] = mfma16_f32(o.a[n], act[v], O[J][n]);
        });
  }

  store(false);
}

// Y[tok][col] = sum_s P[s][tok][col], fixed order
__global__ void fwd_f32_reduce_kernel(F32Args a) {
  const int64_t dm = (int64_t)a.H * a.dh;
  const int64_t idx = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (idx >= a.N * dm) return;
  const size_t stride = (size_t)a.N * dm;
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int s = 0; s < a.n_split; ++s) sum += *reinterpret_cast<const f32x4*>(a.P + (size_t)s * stride + idx);
  const int64_t tok = idx / dm, col = idx % dm;
  *reinterpret_cast<f32x4*>(a.Y + tok * a.ldy + col) = sum;
}

size_t lds_bytes(const Problem& p, int nw) {
  return sizeof(float) * (3 * (size_t)kF32Rows * f32_ld(f32_padded_width(p.dh)) + (size_t)p.E * 16 * nw);
}
// four waves (64 tokens) per workgroup; two, or one, where the gating weights of more tokens do not fit
int block_waves(const Problem& p) {
  return lds_bytes(p, 4) <= kLdsBytesPerWorkgroup ? 4 : lds_bytes(p, 2) <= kLdsBytesPerWorkgroup ? 2 : 1;
}

int64_t tiles_of(const Problem& p) { return (int64_t)p.E * ((p.de + kF32Rows - 1) / kF32Rows); }

size_t output_bytes(const Problem& p) { return (size_t)p.N * p.H * p.dh * sizeof(float); }
int plan_splits(const Problem& p) {
  const int nw = block_waves(p);
  const int64_t items = ((p.N + 16 * nw - 1) / (16 * nw)) * p.H;
  // microseconds: a tile of 16 neurons takes 32 cycles for each of its 3 DHP / 4 products and
  // wave of a SIMD; a split's partials are written and read at about 4 TB/s, and the second
  // launch costs about 4
  const double tile_us = 0.0100 * f32_padded_width(p.dh) * nw / 4;
  return f32_plan_splits(items, tiles_of(p), tile_us, 2.0 * output_bytes(p) / 4e6, 4.0, 32);
}

template <int DHP, int NW, bool SERIAL>
int launch(const Problem& p, F32Args a, hipStream_t stream) {
  a.n_tiles = (p.N + 16 * NW - 1) / (16 * NW);
  a.n_items = a.n_tiles * p.H * (SERIAL ? 1 : a.n_split);
  if (hipError_t e0 = LdsLimit<&fwd_f32_kernel<DHP, NW, SERIAL>, (int)kLdsBytesPerWorkgroup>::ensure(); e0 != hipSuccess)
    return (int)e0;
  hipLaunchKernelGGL((fwd_f32_kernel<DHP, NW, SERIAL>), dim3((unsigned)xcd_grid_size(a.n_items)), dim3(64 * NW),
                     lds_bytes(p, NW), stream, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || SERIAL || a.n_split == 1) return (int)e;
  const int64_t n4 = p.N * p.H * p.dh / 4;
  hipLaunchKernelGGL(fwd_f32_reduce_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, stream, a);
  return (int)hipGetLastError();
}

template <int NW, bool SERIAL>
int launch_width(const Problem& p, const F32Args& a, hipStream_t stream) {
  switch (f32_padded_width(p.dh)) {
    case 64: return launch<64, NW, SERIAL>(p, a, stream);
    case 96: return launch<96, NW, SERIAL>(p, a, stream);
    case 128: return launch<128, NW, SERIAL>(p, a, stream);
    case 192: return launch<192, NW, SERIAL>(p, a, stream);
    default: return launch<256, NW, SERIAL>(p, a, stream);
  }
}

template <bool SERIAL>
int launch_block(const Problem& p, const F32Args& a, hipStream_t stream) {
  switch (block_waves(p)) {
    case 4: return launch_width<4, SERIAL>(p, a, stream);
    case 2: return launch_width<2, SERIAL>(p, a, stream);
    default: return launch<64, 1, SERIAL>(p, a, stream);   // d_h <= 16 is all that the entry point's limit lets through
  }
}

}  // namespace

// What the entry point takes: the tiles of a 32-token block, or, at d_h = 4 .. 16, unpadded rows of
// 32 neurons and of 32 tokens beside the gating weights of 32 tokens (up to 1229 sub-networks
// where the padded tiles leave room for 1178; those run as 16-token blocks).  The limit is part
// of the interface and stays where it is.
size_t fwd_f32_lds_bytes(const Problem& p) {
  const size_t dh = p.dh;
  const size_t narrow = sizeof(float) * (2 * 32 * dh + 2 * 32 * (dh + 1) + 32 * 33 + 32 * (size_t)p.E);
  const size_t tiles = lds_bytes(p, 2);
  return tiles < narrow ? tiles : narrow;
}

std::string fwd_f32_plan(const Problem& p) {
  return "f32 width=" + std::to_string(f32_padded_width(p.dh)) + " waves=" + std::to_string(block_waves(p)) +
         " shares=" + std::to_string(p.N ? plan_splits(p) : 1);
}

size_t fwd_f32_workspace_bytes(const Problem& p) {
  if (p.N == 0) return 0;
  const int s = plan_splits(p);
  return s > 1 ? s * output_bytes(p) : 0;
}

int launch_fwd_f32(const Problem& p, const void* X, const void* Wg, const void* Wu,
                   const void* Wd, const void* route, void* Y, void* ws, size_t ws_bytes, void* stream) {
  if (p.dh > kMaxDh) return (int)hipErrorInvalidValue;
  F32Args a;
  a.X = static_cast<const float*>(X);
  a.Wg = static_cast<const float*>(Wg);
  a.Wu = static_cast<const float*>(Wu);
  a.Wd = static_cast<const float*>(Wd);
  a.route = route;
  a.Y = static_cast<float*>(Y);
  a.P = static_cast<float*>(ws);
  a.N = p.N; a.ldx = p.ldx; a.ldy = p.ldy;
  a.H = p.H; a.dh = p.dh; a.E = p.E; a.de = p.de; a.route_mode = p.route_mode; a.eps = p.eps;
  a.n_split = plan_splits(p);
  a.tiles_per_split = (int)((tiles_of(p) + a.n_split - 1) / a.n_split);
  a.n_tiles = 0; a.n_items = 0;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const bool serial = a.n_split > 1 && !(ws && ws_bytes >= a.n_split * output_bytes(p));
  return serial ? launch_block<true>(p, a, st) : launch_block<false>(p, a, st);
}

}  // namespace mhffn
