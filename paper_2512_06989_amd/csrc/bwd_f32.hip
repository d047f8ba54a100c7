// Fused, recompute-based backward of the Multi-Head FFN in fp32 (storage and
// arithmetic), gfx950.  Shape-generic companion of the bf16 MFMA kernels: any E,
// any d_e, d_h a multiple of 4 up to 256.  Same two sweeps as the bf16 path (appendix
// algorithms "Backward (dQ,dR)" and "Backward (dK,dU,dV)", plus the derivative through
// eq:routing); nothing of the [N][H][d_ff] intermediate is saved or written.  All
// contractions run on v_mfma_f32_16x16x4_f32 with the operand layouts of f32_tiles.h.
//
//   bwd_f32_tok_kernel   wave = 16 tokens x one head, all neurons: R, dX, dr_e -> dp_e (or dR)
//   bwd_f32_wgt_kernel   wave = 16 neurons of one sub-network, a segment of the tokens: dK, dU, dV
//   bwd_f32_route_kernel dW_r[h][j][e] = sum_tok q[tok][j] dp[tok][e], a segment of the tokens
// Segments leave fp32 partials that bwd_f32_reduce_kernel adds up in order.
// Every sum runs in a fixed order: results are bit-identical run to run.
//
// When token blocks x heads cannot load the CUs evenly, the sub-networks of a block are shared
// out over several workgroups, which leave partial dX and their own dr_e for bwd_finish.hip.
//
// Bound: the fp32 matrix rate (157 TFLOP/s) in the two sweeps.  2000 tokens, H = 6, E = 16,
// d_e = 128: token-major 0.293 + 0.016 ms (0.426 ms as 192 workgroups that are not shared out),
// weight-major 0.345 + 0.015 ms (110 TFLOP/s executed, MFMA busy 71 %), dW_r 0.011 ms, against
// 4.02, 7.12 and 0.52 ms of the plain-FMA kernels they replace.
#include "f32_tiles.h"
#include "mhffn_internal.h"

namespace mhffn {
namespace {

struct BwdF32Args {
  const float* X;
  const float* Wg;
  const float* Wu;
  const float* Wd;
  const void* route;
  const float* dY;
  float* dX;
  float* dWg;
  float* dWu;
  float* dWd;
  float* d_route;
  float* Rws;   // [H][E][N]
  float* DPws;  // [H][E][N]  dp (params mode)
  float* Zws;   // [H][N]  1 / (Z + eps) (params mode, shares > 1)
  float* XPws;  // [shares][N][H*dh] partial dX (shares > 1)
  float* WPws;  // [segs][K | U | V][H*E*de*dh] partial weight gradients (segs > 1)
  float* WRws;  // [route_parts][H*dh*E] partial dW_r
  int64_t N, ldx, ldy, n_tiles, n_items;
  int H, dh, E, de, route_mode, chunks_per_sub;
  int shares, subs_per_share;    // token-major: sub-networks shared out over workgroups
  int segs, blocks_per_seg;      // weight-major: token segments and 16-token blocks of one
  int route_parts, route_steps;  // dW_r: token parts and 16-token steps of one
  float eps;
};

// ---------------------------------------------------------------------------
// token-major: R (to the workspace), dX, dp or dR
// ---------------------------------------------------------------------------
template <int DHP, int NW>
__global__ __launch_bounds__(64 * NW, DHP <= 64 ? 3 : DHP <= 128 ? 2 : 1) void bwd_f32_tok_kernel(BwdF32Args a) {
  constexpr int THREADS = 64 * NW, BT = 16 * NW;
  constexpr int KC = DHP / 16, JG = f32_col_groups(DHP), LD = f32_ld(DHP), TILE = kF32Rows * LD;
  constexpr int CPT = (kF32Rows * DHP / 4 + THREADS - 1) / THREADS;
  extern __shared__ __attribute__((aligned(16))) float smem_f[];
  float* Ks = smem_f;                     // [16][LD]
  float* Us = Ks + TILE;
  float* Vs = Us + TILE;
  float* Rs = Vs + TILE;                  // [E][BT]
  float* DRs = Rs + a.E * BT;             // [E][BT]  dr_e, later dp_e

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i16 = lane & 15, gq = lane >> 4;
  const int dh = a.dh, E = a.E, de = a.de;
  const int cpr = dh >> 2;
  const int64_t N = a.N;
  const int64_t item = xcd_work_item(blockIdx.x, a.n_items);
  if (item >= a.n_items) return;
  const int share = (int)(item % a.shares);
  const int64_t ht = item / a.shares;
  const int h = (int)(ht / a.n_tiles);
  const int64_t tok0 = (ht % a.n_tiles) * BT;
  const int wtok = 16 * wave + i16;
  const int64_t tok = tok0 + wtok;
  const bool active = tok0 + 16 * wave < N;
  const int e_begin = share * a.subs_per_share, e_end = min(E, e_begin + a.subs_per_share);

  // weight-tile stream, as in the forward kernel
  const int cps = a.chunks_per_sub;
  const int t_begin = e_begin * cps, t_end = e_end * cps;
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
    const int n4 = min(kF32Rows, de - cb) * cpr;
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

  f32x4 q[KC], y[KC];   // q and dY operands of this lane's token
  {
    const float* xs = a.X + (tok < N ? tok : 0) * a.ldx + (size_t)h * dh;
    const float* ys = a.dY + (tok < N ? tok : 0) * a.ldy + (size_t)h * dh;
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
      const int col = 16 * kk + 4 * gq;
      q[kk] = y[kk] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (tok < N && col < dh) {
        q[kk] = *reinterpret_cast<const f32x4*>(xs + col);
        y[kk] = *reinterpret_cast<const f32x4*>(ys + col);
      }
    }
  }
  const int pad = 64 * JG - dh;
  for (int idx = tid; idx < 3 * kF32Rows * pad; idx += THREADS) Ks[(idx / pad) * LD + dh + idx % pad] = 0.f;

  // gating weights: eq:routing (every lane writes and later reads its own token)
  float zinv = 0.f;   // 1 / (Z + eps) of this lane's token
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
      zinv = 1.0f / (sum_lane_groups(z) + a.eps);
      for (int eb = 0; eb < E; eb += 16)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int e = eb + 4 * gq + v;
          if (e < E) Rs[e * BT + wtok] *= zinv;
        }
    }
  } else {
    const float* R = reinterpret_cast<const float*>(a.route);
    for (int idx = tid; idx < BT * E; idx += THREADS) {
      const int t = idx / E, e = idx - t * E;
      Rs[e * BT + t] = (tok0 + t < N) ? R[((size_t)(tok0 + t) * a.H + h) * E + e] : 0.f;
    }
  }
  __syncthreads();
  // R for the weight-major kernel
  for (int idx = tid; idx < BT * (e_end - e_begin); idx += THREADS) {
    const int e = e_begin + idx / BT, t = idx % BT;
    if (tok0 + t < N) a.Rws[((size_t)h * E + e) * N + tok0 + t] = Rs[e * BT + t];
  }

  f32x4 acc[JG][4];   // dX of this lane's token
#pragma unroll
  for (int J = 0; J < JG; ++J)
#pragma unroll
    for (int n = 0; n < 4; ++n) acc[J][n] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int row_off = i16 * LD + 4 * gq, col_off = 4 * gq * LD + 4 * i16;
  float dr = 0.f;
  int left = cps, e = e_begin;     // tiles left of sub-network e
  f32_settle(q);
  f32_settle(y);
  for (int t = t_begin; t < t_end; ++t) {
    __syncthreads();
#pragma unroll
    for (int c = 0; c < CPT; ++c)
      if (loff[c] >= 0) {
        *reinterpret_cast<f32x4*>(Ks + loff[c]) = kreg[c];
        *reinterpret_cast<f32x4*>(Us + loff[c]) = ureg[c];
        *reinterpret_cast<f32x4*>(Vs + loff[c]) = vreg[c];
      }
    __syncthreads();
    if (t + 1 < t_end) gload(t + 1);
    if (active) {
      const float rw = Rs[e * BT + wtok];
      f32x4 m = {0.f, 0.f, 0.f, 0.f}, nn = {0.f, 0.f, 0.f, 0.f}, da = {0.f, 0.f, 0.f, 0.f};
      f32_stream<KC>(
          [&](auto K_) {
            return F32Op3{lds_f32x4(Ks + row_off + 16 * K_.value), lds_f32x4(Us + row_off + 16 * K_.value),
                          lds_f32x4(Vs + row_off + 16 * K_.value)};
          },
          [&](auto K_, const F32Op3& o) {
#pragma unroll
            for (int n = 0; n < 4; ++n) {
              m = mfma16_f32(o.a[n], q[K_.value][n], m);
              nn = mfma16_f32(o.b[n], q[K_.value][n], nn);
              da = mfma16_f32(o.c[n], y[K_.value][n], da);
            }
          });
      f32x4 dm, dn;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float sg = sigmoid_f32(m[v]);
        const float silu = m[v] * sg;
        const float rda = rw * da[v];
        dr = fmaf(da[v] * silu, nn[v], dr);     // dr_e += dA SiLU(M) N, this lane's neurons
        dn[v] = rda * silu;
        dm[v] = rda * nn[v] * fmaf(silu, 1.0f - sg, sg);   // SiLU'(m)
      }
      // dX += dM K + dN U
      f32_stream<4 * JG>(
          [&](auto S_) {
            constexpr int off = (S_.value / JG) * LD + 64 * (S_.value % JG);
            return F32Op2{lds_f32x4(Ks + col_off + off), lds_f32x4(Us + col_off + off)};
          },
          [&](auto S_, const F32Op2& o) {
            constexpr int v = S_.value / JG, J = S_.value % JG;
#pragma unroll
            for (int n = 0; n < 4; ++n) acc[J][n] = mfma16_f32(o.a[n], dm[v], acc[J][n]);
#pragma unroll
            for (int n = 0; n < 4; ++n) acc[J][n] = mfma16_f32(o.b[n], dn[v], acc[J][n]);
          });
    }
    if (--left == 0) {
      const float sum = sum_lane_groups(dr);
      if (gq == 0) DRs[e * BT + wtok] = active ? sum : 0.f;
      dr = 0.f;
      left = cps;
      ++e;
    }
  }
  __syncthreads();

  // a share leaves its dr_e and its partial dX; bwd_finish.hip does what follows here
  const bool whole = a.shares == 1;
  if (!whole && a.route_mode == 0) {
    for (int idx = tid; idx < BT * (e_end - e_begin); idx += THREADS) {
      const int ee = e_begin + idx / BT, t = idx % BT;
      if (tok0 + t < N) a.DPws[((size_t)h * E + ee) * N + tok0 + t] = DRs[ee * BT + t];
    }
    if (share == 0 && gq == 0 && tok < N) a.Zws[(size_t)h * N + tok] = zinv;
  } else if (a.route_mode == 0) {
    // through r = s / (Z + eps), s = sigmoid(p):
    //   ds_e = (dr_e - sum_e' dr_e' r_e') / (Z + eps),  dp_e = ds_e s_e (1 - s_e)
    float dot = 0.f;
    for (int ee = gq; ee < E; ee += 4) dot = fmaf(DRs[ee * BT + wtok], Rs[ee * BT + wtok], dot);
    dot = sum_lane_groups(dot);
    if (active) {
      const float zpe = 1.0f / zinv;
      for (int ee = gq; ee < E; ee += 4) {
        const float s = Rs[ee * BT + wtok] * zpe;
        const float dp = (DRs[ee * BT + wtok] - dot) * zinv * s * (1.0f - s);
        DRs[ee * BT + wtok] = dp;
        if (tok < N) a.DPws[((size_t)h * E + ee) * N + tok] = dp;
      }
      // dX += dp W_r^T: the lane group gq holds the dp of sub-networks 4 s + gq, as the
      // operand wants them
      const float* Wr = reinterpret_cast<const float*>(a.route) + (size_t)h * dh * E;
      for (int eb = 0; eb < E; eb += 4) {
        const bool ok = eb + gq < E;
        const float dp = ok ? DRs[(eb + gq) * BT + wtok] : 0.f;
#pragma unroll
        for (int J = 0; J < JG; ++J)
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            const int j = 64 * J + 4 * i16 + n;
            const float w = (ok && j < dh) ? Wr[(size_t)j * E + eb + gq] : 0.f;
            acc[J][n] = mfma16_f32(w, dp, acc[J][n]);
          }
      }
    }
  } else if (a.d_route) {
    const int ne = e_end - e_begin;
    for (int idx = tid; idx < BT * ne; idx += THREADS) {
      const int t = idx / ne, ee = e_begin + idx % ne;
      if (tok0 + t < N) a.d_route[((size_t)(tok0 + t) * a.H + h) * E + ee] = DRs[ee * BT + t];
    }
  }

  if (a.dX && tok < N) {
    float* dst = whole ? a.dX + tok * a.ldx + (size_t)h * dh
                       : a.XPws + (((size_t)share * N + tok) * a.H + h) * dh;
#pragma unroll
    for (int J = 0; J < JG; ++J)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int col = 64 * J + 16 * gq + 4 * v;
        if (col < dh) {
          const f32x4 o = {acc[J][0][v], acc[J][1][v], acc[J][2][v], acc[J][3][v]};
          *reinterpret_cast<f32x4*>(dst + col) = o;
        }
      }
  }
}

// ---------------------------------------------------------------------------
// weight-major: dK, dU, dV of 16 neurons per wave, summed over a segment of the tokens.
// The K, U, V rows are resident as operands (tokens on the MFMA rows here, neurons on the
// columns); blocks of 16 tokens of q and dY pass through two LDS buffers.  From d_h = 192 on
// the V rows lie in LDS instead: operands and accumulators of three matrices would take 384 of
// a lane's 512 registers at d_h = 256.  With V in LDS 428 bytes per lane still spill there, 25
// reloads beside the 384 products of a block; at 192 nothing does.
// ---------------------------------------------------------------------------
constexpr int kWgtWaves = 4;
constexpr bool wgt_v_in_lds(int dhp) { return dhp >= 192; }
constexpr size_t wgt_lds_bytes(int dhp) {
  return (4 + (wgt_v_in_lds(dhp) ? kWgtWaves : 0)) * (size_t)kF32Rows * f32_ld(dhp) * sizeof(float);
}

template <int DHP>
__global__ __launch_bounds__(64 * kWgtWaves, DHP <= 128 ? 2 : 1) void bwd_f32_wgt_kernel(BwdF32Args a) {
  constexpr int THREADS = 64 * kWgtWaves;
  constexpr int KC = DHP / 16, JG = f32_col_groups(DHP), LD = f32_ld(DHP), TILE = kF32Rows * LD;
  constexpr int CPT = (kF32Rows * DHP / 4 + THREADS - 1) / THREADS;
  extern __shared__ __attribute__((aligned(16))) float smem_f[];   // [2 buffers][q | dY][16][LD], V [4 waves][16][LD]
  constexpr bool VLDS = wgt_v_in_lds(DHP);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i16 = lane & 15, gq = lane >> 4;
  const int dh = a.dh, E = a.E, de = a.de;
  const int cpr = dh >> 2;
  const int64_t N = a.N;
  const int64_t item = xcd_work_item(blockIdx.x, a.n_items);
  if (item >= a.n_items) return;
  const int seg = (int)(item % a.segs);
  const int64_t grp = item / a.segs;
  const int per_head = E * a.chunks_per_sub;                        // waves' worth of neurons
  const int groups = (per_head + kWgtWaves - 1) / kWgtWaves;
  const int h = (int)(grp / groups);
  const int ec = (int)(grp % groups) * kWgtWaves + wave;
  const bool active = ec < per_head;
  const int e = active ? ec / a.chunks_per_sub : 0;
  const int cb = active ? (ec % a.chunks_per_sub) * kF32Rows : 0;
  const int64_t row = ((int64_t)h * E + e) * de + cb + i16;         // this lane's neuron
  const bool row_ok = active && cb + i16 < de;

  const int64_t b0 = (int64_t)seg * a.blocks_per_seg;
  const int64_t nb = (N + kF32Rows - 1) / kF32Rows;
  const int64_t b1 = b0 + a.blocks_per_seg < nb ? b0 + a.blocks_per_seg : nb;

  // q and dY rows of a block: global -> registers -> LDS
  int loff[CPT], grow[CPT], gcol[CPT];
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int idx = tid + THREADS * c;
    const bool ok = idx < kF32Rows * cpr;
    grow[c] = ok ? idx / cpr : 0;
    gcol[c] = ok ? 4 * (idx % cpr) : 0;
    loff[c] = ok ? grow[c] * LD + gcol[c] : -1;
  }
  const float* Xh = a.X + (size_t)h * dh;
  const float* Yh = a.dY + (size_t)h * dh;
  const float* Rrow = a.Rws + ((size_t)h * E + e) * N;
  // (no read-ahead: the resident operands and accumulators fill the registers.  Up to d_h = 128
  // the other workgroups of the CU compute meanwhile; at 192 and 256 there is none, and every
  // block waits for its loads)
  auto stage = [&](int64_t b, float* buf) {
    const int64_t t0 = b * kF32Rows;
    f32x4 xreg[CPT], yreg[CPT];
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      xreg[c] = yreg[c] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (loff[c] >= 0 && t0 + grow[c] < N) {
        xreg[c] = *reinterpret_cast<const f32x4*>(Xh + (t0 + grow[c]) * a.ldx + gcol[c]);
        yreg[c] = *reinterpret_cast<const f32x4*>(Yh + (t0 + grow[c]) * a.ldy + gcol[c]);
      }
    }
#pragma unroll
    for (int c = 0; c < CPT; ++c)
      if (loff[c] >= 0) {
        *reinterpret_cast<f32x4*>(buf + loff[c]) = xreg[c];
        *reinterpret_cast<f32x4*>(buf + TILE + loff[c]) = yreg[c];
      }
  };

  const int row_off = i16 * LD + 4 * gq, col_off = 4 * gq * LD + 4 * i16;
  f32x4 kw[KC], uw[KC], vw[VLDS ? 1 : KC];
  float* Vw = smem_f + (4 + wave) * TILE + row_off;   // this lane's own V operands
#pragma unroll
  for (int kk = 0; kk < KC; ++kk) {
    const int col = 16 * kk + 4 * gq;
    f32x4 v4 = {0.f, 0.f, 0.f, 0.f};
    kw[kk] = uw[kk] = v4;
    if (row_ok && col < dh) {
      kw[kk] = *reinterpret_cast<const f32x4*>(a.Wg + row * dh + col);
      uw[kk] = *reinterpret_cast<const f32x4*>(a.Wu + row * dh + col);
      v4 = *reinterpret_cast<const f32x4*>(a.Wd + row * dh + col);
    }
    if constexpr (VLDS) *reinterpret_cast<f32x4*>(Vw + 16 * kk) = v4;
    else vw[kk] = v4;
  }
  const int pad = 64 * JG - dh;
  for (int idx = tid; idx < 4 * kF32Rows * pad; idx += THREADS) smem_f[(idx / pad) * LD + dh + idx % pad] = 0.f;

  f32x4 gk[JG][4], gu[JG][4], gv[JG][4];
#pragma unroll
  for (int J = 0; J < JG; ++J)
#pragma unroll
    for (int n = 0; n < 4; ++n) gk[J][n] = gu[J][n] = gv[J][n] = f32x4{0.f, 0.f, 0.f, 0.f};

  f32_settle(kw);
  f32_settle(uw);
  if constexpr (!VLDS) f32_settle(vw);
  for (int64_t b = b0; b < b1; ++b) {
    float* Qs = smem_f + (b & 1) * 2 * TILE;
    const float* Ys = Qs + TILE;
    f32x4 r;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t t = b * kF32Rows + 4 * gq + v;
      r[v] = t < N ? Rrow[t] : 0.f;
    }
    stage(b, Qs);
    __syncthreads();   // block b is staged, and everyone is done with block b - 1
    if (!active) continue;
    f32x4 m = {0.f, 0.f, 0.f, 0.f}, nn = {0.f, 0.f, 0.f, 0.f}, da = {0.f, 0.f, 0.f, 0.f};
    f32_stream<KC>(
        [&](auto K_) {
          F32Op3 o{lds_f32x4(Qs + row_off + 16 * K_.value), lds_f32x4(Ys + row_off + 16 * K_.value), f32x4{}};
          if constexpr (VLDS) o.c = lds_f32x4(Vw + 16 * K_.value);
          return o;
        },
        [&](auto K_, const F32Op3& o) {
          f32x4 v4;
          if constexpr (VLDS) v4 = o.c;
          else v4 = vw[K_.value];
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            m = mfma16_f32(o.a[n], kw[K_.value][n], m);
            nn = mfma16_f32(o.a[n], uw[K_.value][n], nn);
            da = mfma16_f32(o.b[n], v4[n], da);
          }
        });
    f32x4 ag, dm, dn;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float sg = sigmoid_f32(m[v]);
      const float silu = m[v] * sg;
      ag[v] = r[v] * silu * nn[v];
      const float rda = r[v] * da[v];
      dn[v] = rda * silu;
      dm[v] = rda * nn[v] * fmaf(silu, 1.0f - sg, sg);
    }
    // dK[c][j] += dM[tok][c] q[tok][j]; dU likewise; dV[c][j] += A_gated[tok][c] dY[tok][j]
    f32_stream<4 * JG>(
        [&](auto S_) {
          constexpr int off = (S_.value / JG) * LD + 64 * (S_.value % JG);
          return F32Op2{lds_f32x4(Qs + col_off + off), lds_f32x4(Ys + col_off + off)};
        },
        [&](auto S_, const F32Op2& o) {
          constexpr int v = S_.value / JG, J = S_.value % JG;
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            gk[J][n] = mfma16_f32(o.a[n], dm[v], gk[J][n]);
            gu[J][n] = mfma16_f32(o.a[n], dn[v], gu[J][n]);
            gv[J][n] = mfma16_f32(o.b[n], ag[v], gv[J][n]);
          }
        });
  }
  if (!row_ok) return;
  // lane = neuron, register v of the four tiles = columns 64 J + 16 gq + 4 v .. +3
  const size_t count = (size_t)a.H * E * de * dh;
  float* outs[3] = {a.dWg, a.dWu, a.dWd};
  if (a.segs > 1)
    for (int i = 0; i < 3; ++i) outs[i] = a.WPws + ((size_t)seg * 3 + i) * count;
#pragma unroll
  for (int J = 0; J < JG; ++J)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int col = 64 * J + 16 * gq + 4 * v;
      if (col >= dh) continue;
      const size_t o = (size_t)row * dh + col;
      if (outs[0]) *reinterpret_cast<f32x4*>(outs[0] + o) = f32x4{gk[J][0][v], gk[J][1][v], gk[J][2][v], gk[J][3][v]};
      if (outs[1]) *reinterpret_cast<f32x4*>(outs[1] + o) = f32x4{gu[J][0][v], gu[J][1][v], gu[J][2][v], gu[J][3][v]};
      if (outs[2]) *reinterpret_cast<f32x4*>(outs[2] + o) = f32x4{gv[J][0][v], gv[J][1][v], gv[J][2][v], gv[J][3][v]};
    }
}

// out_i[x] = sum_s P[s][i][x] for up to three outputs of `count` values (count % 4 == 0), in order
struct ReduceF32Args {
  const float* P;
  float* out[3];
  int64_t count;
  int n_out, parts;
};
__global__ void bwd_f32_reduce_kernel(ReduceF32Args a) {
  const int64_t idx = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  const int i = blockIdx.y;
  if (idx >= a.count || !a.out[i]) return;
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int s = 0; s < a.parts; ++s)
    sum += *reinterpret_cast<const f32x4*>(a.P + ((size_t)s * a.n_out + i) * a.count + idx);
  *reinterpret_cast<f32x4*>(a.out[i] + idx) = sum;
}

// dW_r[h][j][e] = sum_tok q[tok][j] dp[tok][e]: one wave per (head, 16 columns j, 16
// sub-networks, token part); rows of the product are j, columns e, and the slot gq of product
// n is token 4 gq + n of a 16-token step
__global__ __launch_bounds__(256) void bwd_f32_route_kernel(BwdF32Args a) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i16 = lane & 15, gq = lane >> 4;
  const int jblocks = (a.dh + 15) >> 4;
  const int h = blockIdx.x / jblocks, j0 = 16 * (blockIdx.x % jblocks);
  const int e = 16 * blockIdx.y + i16;
  const int part = blockIdx.z * 4 + wave;
  if (part >= a.route_parts) return;
  const int64_t N = a.N;
  const int64_t t_begin = (int64_t)part * a.route_steps * 16;
  const int64_t t_end = min(N, t_begin + (int64_t)a.route_steps * 16);
  const bool j_ok = j0 + i16 < a.dh, e_ok = e < a.E;
  const float* x = a.X + (size_t)h * a.dh + (j_ok ? j0 + i16 : 0);
  const float* dp = a.DPws + ((size_t)h * a.E + (e_ok ? e : 0)) * N;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int64_t t0 = t_begin; t0 < t_end; t0 += 16) {
    float xv[4], dv[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const int64_t t = t0 + 4 * gq + n;
      const bool ok = t < t_end;
      xv[n] = (ok && j_ok) ? x[t * a.ldx] : 0.f;
      dv[n] = (ok && e_ok) ? dp[t] : 0.f;
    }
#pragma unroll
    for (int n = 0; n < 4; ++n) acc = mfma16_f32(xv[n], dv[n], acc);
  }
  float* out = a.WRws + (size_t)part * a.H * a.dh * a.E + (size_t)h * a.dh * a.E;
  if (e_ok)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int j = j0 + 4 * gq + v;
      if (j < a.dh) out[(size_t)j * a.E + e] = acc[v];
    }
}

__global__ void fill_zero_f32_kernel(float* p, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.f;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

size_t tok_lds_bytes(const Problem& p, int nw) {
  return sizeof(float) * (3 * (size_t)kF32Rows * f32_ld(f32_padded_width(p.dh)) + 2 * (size_t)p.E * 16 * nw);
}
// four waves (64 tokens) per workgroup; two, or one, where the gating rows of more tokens do not fit
int tok_block_waves(const Problem& p) {
  return tok_lds_bytes(p, 4) <= kLdsBytesPerWorkgroup ? 4 : tok_lds_bytes(p, 2) <= kLdsBytesPerWorkgroup ? 2 : 1;
}

size_t weight_count(const Problem& p) { return (size_t)p.H * p.E * p.de * p.dh; }

// Token segments of the weight-major kernel.  In microseconds: a 16-token block takes 32
// cycles for each of its 6 DHP / 4 products; partials pass through memory at about 4 TB/s.
int plan_wgt_segs(const Problem& p) {
  const int cps = (p.de + kF32Rows - 1) / kF32Rows;
  const int64_t items = (int64_t)p.H * ((p.E * cps + kWgtWaves - 1) / kWgtWaves);
  return f32_plan_splits(items, (p.N + kF32Rows - 1) / kF32Rows, 0.0200 * f32_padded_width(p.dh),
                         2.0 * 3 * weight_count(p) * sizeof(float) / 4e6, 4.0, 16);
}
// Shares of the sub-networks per token block of the token-major kernel
int plan_tok_shares(const Problem& p) {
  const int nw = tok_block_waves(p);
  const int64_t items = ((p.N + 16 * nw - 1) / (16 * nw)) * p.H;
  const int cps = (p.de + kF32Rows - 1) / kF32Rows;
  return f32_plan_splits(items, p.E, 0.0167 * f32_padded_width(p.dh) * nw / 4 * cps,
                         2.0 * p.N * p.H * p.dh * sizeof(float) / 4e6, 8.0, 16);
}
// Token parts of dW_r: at least four 16-token steps each, at most 64 parts
int plan_route_parts(const Problem& p) {
  const int64_t parts = (p.N + 63) / 64;
  return parts < 1 ? 1 : parts > 64 ? 64 : (int)parts;
}

template <int DHP, int NW>
int launch_tok(const Problem& p, BwdF32Args a, hipStream_t stream) {
  if (hipError_t e0 = LdsLimit<&bwd_f32_tok_kernel<DHP, NW>, (int)kLdsBytesPerWorkgroup>::ensure(); e0 != hipSuccess)
    return (int)e0;
  a.n_tiles = (p.N + 16 * NW - 1) / (16 * NW);
  a.n_items = a.n_tiles * p.H * a.shares;
  hipLaunchKernelGGL((bwd_f32_tok_kernel<DHP, NW>), dim3((unsigned)xcd_grid_size(a.n_items)), dim3(64 * NW),
                     tok_lds_bytes(p, NW), stream, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.shares == 1) return (int)e;
  const BwdFinish f{a.XPws, a.Rws, a.DPws, a.Zws, a.route, a.dX, p.N, p.ldx, p.H, p.dh, p.E, a.shares, p.route_mode == 0, 16,
                    0, (uint32_t)((p.N + 15) / 16 * p.H)};
  return launch_bwd_tok_finish(0, f, stream);
}

template <int DHP>
int launch_width(const Problem& p, BwdF32Args a, bool weights, hipStream_t stream) {
  // token-major kernel (always: it also produces R for the weight-major kernel)
  int rc;
  switch (tok_block_waves(p)) {
    case 4: rc = launch_tok<DHP, 4>(p, a, stream); break;
    case 2: rc = launch_tok<DHP, 2>(p, a, stream); break;
    default:   // d_h below 30 with about 600 sub-networks: all that the entry point's limit lets through
      if constexpr (DHP == 64) rc = launch_tok<DHP, 1>(p, a, stream);
      else rc = (int)hipErrorInvalidValue;
  }
  if (rc || !weights) return rc;
  if (hipError_t e0 = LdsLimit<&bwd_f32_wgt_kernel<DHP>, (int)kLdsBytesPerWorkgroup>::ensure(); e0 != hipSuccess)
    return (int)e0;
  a.n_items = (int64_t)p.H * ((p.E * a.chunks_per_sub + kWgtWaves - 1) / kWgtWaves) * a.segs;
  hipLaunchKernelGGL(bwd_f32_wgt_kernel<DHP>, dim3((unsigned)xcd_grid_size(a.n_items)), dim3(64 * kWgtWaves),
                     wgt_lds_bytes(DHP), stream, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.segs == 1) return (int)e;
  ReduceF32Args r{a.WPws, {a.dWg, a.dWu, a.dWd}, (int64_t)weight_count(p), 3, a.segs};
  hipLaunchKernelGGL(bwd_f32_reduce_kernel, dim3((unsigned)((r.count / 4 + 255) / 256), 3), dim3(256), 0, stream, r);
  return (int)hipGetLastError();
}

}  // namespace

// What the entry point takes: whole d_h-wide rows of a 32-token block and of 16 neurons and
// two n_sub-wide rows per token within one workgroup's LDS.  (The kernels here need less; the
// limit is part of the interface and stays where it is.)
size_t bwd_f32_lds_bytes(const Problem& p) {
  const size_t dh = p.dh;
  return sizeof(float) * (2 * 32 * dh + 3 * 16 * (dh + 1) + 2 * 32 * 17 + 2 * 32 * (size_t)p.E + 32);
}

std::string bwd_f32_plan(const Problem& p) {
  return "tok waves=" + std::to_string(tok_block_waves(p)) + " shares=" + std::to_string(plan_tok_shares(p)) +
         "; wgt segs=" + std::to_string(plan_wgt_segs(p)) + "; route parts=" + std::to_string(plan_route_parts(p));
}

size_t bwd_f32_workspace_bytes(const Problem& p) {
  if (p.N == 0) return 0;
  const int segs = plan_wgt_segs(p), shares = plan_tok_shares(p);
  const size_t wp = segs > 1 ? (size_t)segs * 3 * weight_count(p) * sizeof(float) : 0;
  const size_t xp = shares > 1 ? (size_t)shares * p.N * p.H * p.dh * sizeof(float) : 0;
  return align256((size_t)p.N * p.H * sizeof(float)) + 2 * align256((size_t)p.N * p.H * p.E * sizeof(float)) +
         align256((size_t)plan_route_parts(p) * p.H * p.dh * p.E * sizeof(float)) +
         (wp > xp ? wp : xp);   // the token-major kernel's partials are used up before the weight-major one starts
}

int launch_bwd_f32(const Problem& p, const void* X, const void* Wg, const void* Wu,
                   const void* Wd, const void* route, const void* dY, void* dX, void* dWg,
                   void* dWu, void* dWd, void* d_route, void* ws, void* stream_) {
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  const size_t wcount = weight_count(p);
  if (p.N == 0) {   // no tokens: the weight gradients are zero, there is nothing else
    float* outs[4] = {static_cast<float*>(dWg), static_cast<float*>(dWu), static_cast<float*>(dWd),
                      p.route_mode == 0 ? static_cast<float*>(d_route) : nullptr};
    const size_t counts[4] = {wcount, wcount, wcount, (size_t)p.H * p.dh * p.E};
    for (int i = 0; i < 4; ++i) {
      if (!outs[i] || !counts[i]) continue;
      hipLaunchKernelGGL(fill_zero_f32_kernel, dim3((unsigned)((counts[i] + 255) / 256)), dim3(256),
                         0, stream, outs[i], counts[i]);
    }
    return (int)hipGetLastError();
  }
  BwdF32Args a;
  a.X = static_cast<const float*>(X);
  a.Wg = static_cast<const float*>(Wg);
  a.Wu = static_cast<const float*>(Wu);
  a.Wd = static_cast<const float*>(Wd);
  a.route = route;
  a.dY = static_cast<const float*>(dY);
  a.dX = static_cast<float*>(dX);
  a.dWg = static_cast<float*>(dWg);
  a.dWu = static_cast<float*>(dWu);
  a.dWd = static_cast<float*>(dWd);
  a.d_route = static_cast<float*>(d_route);
  a.route_parts = plan_route_parts(p);
  a.route_steps = (int)(((p.N + 15) / 16 + a.route_parts - 1) / a.route_parts);
  a.segs = plan_wgt_segs(p);
  a.blocks_per_seg = (int)(((p.N + kF32Rows - 1) / kF32Rows + a.segs - 1) / a.segs);
  const size_t nhe = align256((size_t)p.N * p.H * p.E * sizeof(float));
  unsigned char* w = static_cast<unsigned char*>(ws);
  a.Rws = reinterpret_cast<float*>(w);
  a.DPws = reinterpret_cast<float*>(w + nhe);
  a.WRws = reinterpret_cast<float*>(w + 2 * nhe);
  w += 2 * nhe + align256((size_t)a.route_parts * p.H * p.dh * p.E * sizeof(float));
  a.Zws = reinterpret_cast<float*>(w);
  a.WPws = a.XPws = reinterpret_cast<float*>(w + align256((size_t)p.N * p.H * sizeof(float)));
  a.shares = plan_tok_shares(p);
  a.subs_per_share = (p.E + a.shares - 1) / a.shares;
  a.N = p.N; a.ldx = p.ldx; a.ldy = p.ldy;
  a.H = p.H; a.dh = p.dh; a.E = p.E; a.de = p.de; a.route_mode = p.route_mode; a.eps = p.eps;
  a.chunks_per_sub = (p.de + kF32Rows - 1) / kF32Rows;
  a.n_tiles = 0; a.n_items = 0;

  const bool weights = dWg || dWu || dWd;
  int rc;
  switch (f32_padded_width(p.dh)) {
    case 64: rc = launch_width<64>(p, a, weights, stream); break;
    case 96: rc = launch_width<96>(p, a, weights, stream); break;
    case 128: rc = launch_width<128>(p, a, weights, stream); break;
    case 192: rc = launch_width<192>(p, a, weights, stream); break;
    default: rc = launch_width<256>(p, a, weights, stream); break;
  }
  if (rc != 0) return rc;
  if (d_route && p.route_mode == 0) {
    const dim3 grid((unsigned)(p.H * ((p.dh + 15) / 16)), (unsigned)((p.E + 15) / 16),
                    (unsigned)((a.route_parts + 3) / 4));
    hipLaunchKernelGGL(bwd_f32_route_kernel, grid, dim3(256), 0, stream, a);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return (int)e;
    ReduceF32Args r{a.WRws, {a.d_route, nullptr, nullptr}, (int64_t)p.H * p.dh * p.E, 1, a.route_parts};
    hipLaunchKernelGGL(bwd_f32_reduce_kernel, dim3((unsigned)((r.count / 4 + 255) / 256), 1), dim3(256), 0, stream, r);
    return (int)hipGetLastError();
  }
  return 0;
}

}  // namespace mhffn
