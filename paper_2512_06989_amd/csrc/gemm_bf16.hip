// bf16 matrix product for the module's d_model x d_model projections (Methodology:
// Q = split_H(X W_in), O = concat_H(S) W_out, and the four products of their backward).
//
//   C[m][n] = sum_k A(m,k) B(n,k),   C row-major bf16, fp32 accumulation on the MFMA,
//
// each operand given either with k contiguous ("row form": [rows][K]) or with its row
// index contiguous ("transposed form": [K][rows]), so all three products of a linear
// layer read their operands where they lie:
//   Y = X W      A = X row form,   B = W transposed form
//   dX = dY W^T  A = dY row form,  B = W row form
//   dW = X^T dY  A = X transposed, B = dY transposed
//
// A workgroup owns a BM x BN tile of C (256 x 256 where there are enough of them, smaller
// ones otherwise: plan_tiles), its waves take TM x TN pieces as products of 32 x 32, and k
// runs in slices of 32.  What bounds it:
//   * the global -> LDS rate: measured, a CU takes about 27 bytes per clock through direct
//     loads (14 TB/s over the chip), so a slice of 256 + 256 rows (32 KB) costs 1200 clocks
//     against 1024 of products;
//   * their latency, about 2 us when all CUs load: the slices go into a ring of up to five
//     stages, requested as many slices ahead, with counted waits (two stages of 64, waited for
//     with one slice of look-ahead, made every 64 of k cost 4600 clocks);
//   * LDS reads: a wave of 128 x 64 reads six operands for eight products (of 64 x 64: eight
//     for eight).
// The n side sits on the MFMA row axis and the m side on the column axis, so a lane ends up
// with four consecutive n of one row m; the tile goes out through LDS as whole rows.
// LDS images: row form [rows][32 k], 64-byte rows whose four 16-byte chunks are permuted by
// (row / 4) % 4; transposed form the swizzled [32 k][128] tile of the fused kernels; both are
// free of bank conflicts for their reads.  Operand reads are issued untracked, six to eight
// instructions ahead and across slice boundaries, and waited for by count.
// Rates (row x transposed form): 16384 x 2048 x 2048 126 us (1090 TFLOP/s; 16 waves of 64 x 64
// on two stages of 64: 136 .. 162), 16384 x 1024 x 1024 42 us (54), 4000 x 2048 x 2048 41 us
// (62 with its partials), 1000 x 2048 x 2048 19 us (33); weight gradient of 16384 rows,
// 1024 x 1024: 60 us (71).
#include "mhffn_device.h"
#include "mhffn_internal.h"

#include <type_traits>

namespace mhffn {
namespace {

constexpr int kGBK = 32;   // k per slice

struct TunedGemmArgs {
  const uint16_t* A;   // m side
  const uint16_t* B;   // n side
  uint16_t* C;
  int64_t M, N, K, lda, ldb, ldc;
  int64_t n_items, tiles_n;
  // split-k: each output tile is shared out over `splits` workgroups, slices_per_split
  // slices of k each; they leave fp32 partial tiles in P [splits][M][N]
  int splits;
  int64_t slices_per_split;
  float* P;
  int accumulate;   // add to what C holds (one more rounding to bf16)
};

template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// Tile shapes: output tile, waves along m and n, stages of the ring
template <int BM_, int BN_, int WM_, int WN_, int S_>
struct GemmTile {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, S = S_;
  static constexpr int NW = WM * WN, TM = BM / WM, TN = BN / WN, IM = TM / 32, IN = TN / 32;
  static constexpr int kMBytes = BM * kGBK * 2, kNBytes = BN * kGBK * 2, kStage = kMBytes + kNBytes;
  static constexpr int kLoads = kStage / 1024 / NW;      // wave-wide 1 KB loads per wave and slice
  static constexpr int kLds = S * kStage > NW * TM * TN * 2 ? S * kStage : NW * TM * TN * 2;
  static_assert(kLoads * 1024 * NW == kStage && kMBytes / 1024 % NW == 0 && BN % 128 == 0, "whole loads per wave");
  static_assert(kLds <= (int)kLdsBytesPerWorkgroup, "stages and the output tile must fit in LDS");
};
using Tile256x256 = GemmTile<256, 256, 2, 4, 5>;
using Tile256x128 = GemmTile<256, 128, 4, 2, 6>;
using Tile128x128 = GemmTile<128, 128, 2, 4, 4>;
using Tile64x128 = GemmTile<64, 128, 2, 2, 5>;   // (m side in row form: a transposed image is 128 wide)

// byte offset of 16-byte chunk `chunk` of `row` in a row-form image
__device__ __forceinline__ int row_image_off(int row, int chunk) { return row * 64 + ((chunk ^ ((row >> 2) & 3)) << 4); }

template <bool A_TR, bool B_TR, typename G>
__global__ __launch_bounds__(64 * G::NW, G::BM == 256 ? 2 : 4) void gemm_bf16_kernel(TunedGemmArgs a) {
  constexpr int IM = G::IM, IN = G::IN, S = G::S, NW = G::NW;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 31, g = lane >> 5;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const int wm = wave_u / G::WN, wn = wave_u % G::WN;
  const int64_t item = xcd_work_item(blockIdx.x, a.n_items);
  if (item >= a.n_items) return;
  const int split = (int)(item % a.splits);
  const int64_t tile = item / a.splits;
  const int64_t m0 = (tile / a.tiles_n) * G::BM, n0 = (tile % a.tiles_n) * G::BN;
  const int64_t K = a.K;
  const int64_t KT_all = (K + kGBK - 1) / kGBK;
  const int64_t kbase = split * a.slices_per_split;           // first slice of this workgroup
  const int64_t kend = kbase + a.slices_per_split < KT_all ? kbase + a.slices_per_split : KT_all;
  const int KT = (int)(kend - kbase);                         // its number of slices (>= 1)

  // ---- staging: wave-wide 1 KB loads, kLoads per wave and slice ---------------------------
  // Load q of wave w is image q NW + w of the stage: first the m side's, then the n side's.
  // Row form: image i = rows 16 i .. + 15, lane l -> row + l / 4, physical chunk l % 4.
  // Transposed form: image i = k rows 4 (i % 8) .. + 3 of the 128-wide tile i / 8, lane l -> k
  // row + l / 16, physical chunk l % 16.  Rows / columns past the edge are clamped (their
  // products are never stored); k rows past K are clamped too and their slots cleared before use.
  // A request is a wave-uniform base (advanced with the slice) plus a 32-bit byte offset per lane.
  constexpr bool kRagged = A_TR && B_TR;   // only then may K end inside a slice (gemm_bf16_supported)
  unsigned goff[G::kLoads], glast[G::kLoads];   // glast: for the last slice, k rows past K repeat row K - 1
  const int k_left = (int)(K - (KT_all - 1) * kGBK);
#pragma unroll
  for (int q = 0; q < G::kLoads; ++q) {
    const bool m_side = q < G::kMBytes / 1024 / NW;           // (a compile-time fact)
    const int img = q * NW + wave_u - (m_side ? 0 : G::kMBytes / 1024);
    const int64_t ld = m_side ? a.lda : a.ldb, row0 = m_side ? m0 : n0, rows = m_side ? a.M : a.N;
    if (!(m_side ? A_TR : B_TR)) {
      const int row = 16 * img + (lane >> 2);
      const int64_t gr = row0 + row < rows ? row : rows - 1 - row0;
      goff[q] = glast[q] = (unsigned)(gr * ld * 2 + (((lane & 3) ^ ((row >> 2) & 3)) << 4));
    } else {
      const int kr = 4 * (img & 7) + (lane >> 4);
      int64_t gc = row0 + 128 * (img >> 3) + (((lane & 15) ^ swz(kr)) << 3);
      gc = (gc + 8 <= rows ? gc : rows - 8) - row0;
      goff[q] = (unsigned)((kr * ld + gc) * 2);
      glast[q] = (unsigned)(((kr < k_left ? kr : k_left - 1) * ld + gc) * 2);
    }
  }
  const unsigned char* const abase =
      reinterpret_cast<const unsigned char*>(a.A + (A_TR ? m0 + kbase * kGBK * a.lda : m0 * a.lda + kbase * kGBK));
  const unsigned char* const bbase =
      reinterpret_cast<const unsigned char*>(a.B + (B_TR ? n0 + kbase * kGBK * a.ldb : n0 * a.ldb + kbase * kGBK));
  const int64_t astep = (A_TR ? a.lda : 1) * (kGBK * 2), bstep = (B_TR ? a.ldb : 1) * (kGBK * 2);
  auto request = [&](int kt, int stage) {
    const bool last = kRagged && kbase + kt == KT_all - 1;
    const unsigned char* const pa = abase + kt * astep;
    const unsigned char* const pb = bbase + kt * bstep;
#pragma unroll
    for (int q = 0; q < G::kLoads; ++q) {
      const unsigned off = last ? glast[q] : goff[q];
      global_to_lds_16B((q < G::kMBytes / 1024 / NW ? pa : pb) + off, smem + stage * G::kStage + (q * NW + wave_u) * 1024);
    }
  };

  // ---- operand addresses inside a stage ----------------------------------------------------
  // operand (side, idx, t2): 32-row block idx of the wave's piece, 16-wide contraction step t2.
  //   row form:        one 16-byte read; register per t2 (the chunk permutation is an XOR), + 2048 per idx
  //   transposed form: two transposing reads of four k rows each, register per idx, + 4096 per t2;
  //                    slots 8 g .. 8 g + 7 are k rows 16 t2 + 8 g .. as in the row form
  const unsigned lbase = lds_addr_of(smem);
  unsigned arow[2][2];                              // row form [side][t2]
  unsigned atr[2][IM > IN ? IM : IN][2];            // transposed form [side][idx]: k rows .. and .. + 4
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    const bool tr = side ? A_TR : B_TR;
    const int wrow = side ? G::TM * wm : G::TN * wn;
    const unsigned sbase = lbase + (side ? 0 : G::kMBytes);
    if (!tr) {
#pragma unroll
      for (int t2 = 0; t2 < 2; ++t2) arow[side][t2] = sbase + row_image_off(wrow + r, 2 * t2 + g);
    } else {
#pragma unroll
      for (int idx = 0; idx < (side ? IM : IN); ++idx) {
        const int li = lane & 15, kr = 8 * g + (li >> 2);
        const int col = wrow + 32 * idx + 16 * ((lane >> 4) & 1) + 4 * (li & 3);
        atr[side][idx][0] = sbase + (col >> 7) * 8192 + tile_off8(kr, col & 127);
        atr[side][idx][1] = sbase + (col >> 7) * 8192 + tile_off8(kr + 4, col & 127);
      }
    }
  }

  f32x16 acc[IN][IM];
#pragma unroll
  for (int i = 0; i < IN; ++i)
#pragma unroll
    for (int j = 0; j < IM; ++j) acc[i][j] = f32x16{0};

  // ---- main loop ------------------------------------------------------------------------------
  // Top of slice kt: wait for this wave's part of slice kt + 1 (the requests behind it stay in
  // flight), barrier (slices kt and kt + 1 have landed everywhere, everyone is done with slice
  // kt - 1), request slice kt + S - 1 into the stage of slice kt - 1.  Items c of a slice:
  // contraction step t2 = c / (IN + IM), first the n operands, then the m operands; an m operand
  // is followed by its IN products.  Reads run kWin items ahead and across the slice boundary,
  // so that no wave starts a slice by waiting for LDS.
  constexpr int OPS = IN + IM, NOP = 2 * OPS, kWin = OPS;
  constexpr int kNInstr = B_TR ? 2 : 1, kMInstr = A_TR ? 2 : 1;   // LDS instructions per operand
  constexpr int kPending = IN * kNInstr + IM * kMInstr;           // of the OPS items behind any item
  static_assert(kPending <= 15, "lgkmcnt holds four bits");
  s16x4 lo[NOP], hi[NOP];
  bf16x8 full[NOP], nf[IN];
  auto issue = [&](auto C_, unsigned so) {
    constexpr int c = decltype(C_)::value, t2 = c / OPS, o = c % OPS;
    constexpr int side = o < IN ? 0 : 1, idx = side ? o - IN : o;
    if constexpr (side ? A_TR : B_TR) {
      lo[c] = lds_read_tr16_untracked<t2 * 4096>(atr[side][idx][0] + so);
      hi[c] = lds_read_tr16_untracked<t2 * 4096>(atr[side][idx][1] + so);
    } else {
      full[c] = lds_read_b128_untracked<2048 * idx>(arow[side][t2] + so);
    }
  };
  auto slice = [&](int kt, unsigned so, unsigned so_next) {
    const bool ragged_last = (A_TR && B_TR) && (kbase + kt == KT_all - 1) && (K % kGBK) != 0;
    static_for<0, NOP>([&](auto C_) {
      constexpr int c = decltype(C_)::value, t2 = c / OPS, o = c % OPS;
      constexpr int side = o < IN ? 0 : 1;
      if constexpr (c + kWin < NOP) issue(std::integral_constant<int, c + kWin>{}, so);
      else issue(std::integral_constant<int, c + kWin - NOP>{}, so_next);   // (past the last slice: never used)
      bf16x8 v;
      if constexpr (side ? A_TR : B_TR) {
        lds_wait<kPending>(lo[c], hi[c]);
        v = join_tr(lo[c], hi[c]);
      } else {
        lds_wait<kPending>(full[c]);
        v = full[c];
      }
      if constexpr (side == 0) {
        if (ragged_last) {   // k rows past K were clamped: clear their slots on the n side
#pragma unroll
          for (int sl = 0; sl < 8; ++sl)
            if ((kbase + kt) * kGBK + 16 * t2 + 8 * g + sl >= K) v[sl] = (__bf16)0.0f;
        }
        nf[o] = v;
      } else {
#pragma unroll
        for (int jn = 0; jn < IN; ++jn) acc[jn][o - IN] = mfma32(nf[jn], v, acc[jn][o - IN]);
      }
    });
  };

  for (int i = 0; i < S - 1 && i < KT; ++i) request(i, i);
  constexpr int kAhead = G::kLoads * (S - 3);   // this wave's loads behind slice kt + 1
  static_assert(S >= 3 && kAhead < 64, "vmcnt holds six bits");
  int stage = 0;
  for (int kt = 0; kt < KT; ++kt) {
    asm volatile("" ::: "memory");
    if (kt + S - 2 < KT) __builtin_amdgcn_s_waitcnt(0x0F70 | (kAhead & 15) | ((kAhead >> 4) << 14));   // vmcnt(kAhead)
    else __builtin_amdgcn_s_waitcnt(0x0F70);                                                          // vmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (kt == 0) static_for<0, kWin>([&](auto C_) { issue(C_, 0u); });
    if (kt + S - 1 < KT) request(kt + S - 1, stage == 0 ? S - 1 : stage - 1);
    const int next = stage + 1 == S ? 0 : stage + 1;
    slice(kt, stage * G::kStage, next * G::kStage);
    stage = next;
  }
  // the reads issued for a slice that never comes: their registers stay taken until they have landed
  static_for<0, kWin>([&](auto C_) {
    constexpr int c = decltype(C_)::value;
    if constexpr ((c % OPS < IN) ? B_TR : A_TR) lds_wait<0>(lo[c], hi[c]);
    else lds_wait<0>(full[c]);
  });

  // ---- store: lane = row m, registers = four consecutive n per group ----------------------
  if (a.splits > 1 || a.accumulate) {
#pragma unroll
    for (int im = 0; im < IM; ++im) {
      const int64_t m = m0 + G::TM * wm + 32 * im + r;
      if (m >= a.M) continue;
#pragma unroll
      for (int jn = 0; jn < IN; ++jn) {
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
          const int64_t n = n0 + G::TN * wn + 32 * jn + 8 * vq + 4 * g;
          if (n + 4 > a.N) continue;
          float o[4] = {acc[jn][im][4 * vq], acc[jn][im][4 * vq + 1], acc[jn][im][4 * vq + 2],
                        acc[jn][im][4 * vq + 3]};
          if (a.splits > 1) {
            *reinterpret_cast<f32x4*>(a.P + ((size_t)split * a.M + m) * a.N + n) = f32x4{o[0], o[1], o[2], o[3]};
            continue;
          }
          u32x2* dst = reinterpret_cast<u32x2*>(a.C + m * a.ldc + n);
          const u32x2 old = *dst;
          o[0] += __builtin_bit_cast(float, old[0] << 16);
          o[1] += __builtin_bit_cast(float, old[0] & 0xFFFF0000u);
          o[2] += __builtin_bit_cast(float, old[1] << 16);
          o[3] += __builtin_bit_cast(float, old[1] & 0xFFFF0000u);
          *dst = u32x2{pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3])};
        }
      }
    }
    return;
  }
  // whole rows: the wave's piece passes through LDS ([TM][TN] bf16, the 16-byte chunks of a row
  // permuted by the row so that neither side meets more than two lanes per bank)
  constexpr int CR = G::TN / 8;                        // chunks per row
  __syncthreads();                                     // the stages are done with
  unsigned char* piece = smem + wave * (G::TM * G::TN * 2);
#pragma unroll
  for (int im = 0; im < IM; ++im)
#pragma unroll
    for (int jn = 0; jn < IN; ++jn)
#pragma unroll
      for (int vq = 0; vq < 4; ++vq) {
        const int row = 32 * im + r, chunk = (4 * jn + vq) ^ (row & (CR - 1));
        const u32x2 pk = {pack_bf16(acc[jn][im][4 * vq], acc[jn][im][4 * vq + 1]),
                          pack_bf16(acc[jn][im][4 * vq + 2], acc[jn][im][4 * vq + 3])};
        *reinterpret_cast<u32x2*>(piece + row * (G::TN * 2) + chunk * 16 + 8 * g) = pk;
      }
  // (the piece is this wave's own: its reads follow its writes in the same queue)
#pragma unroll 4
  for (int i = lane; i < G::TM * CR; i += 64) {
    const int row = i / CR, chunk = i % CR;
    const int64_t m = m0 + G::TM * wm + row, n = n0 + G::TN * wn + 8 * chunk;
    const u32x4 v = *reinterpret_cast<const u32x4*>(piece + row * (G::TN * 2) + ((chunk ^ (row & (CR - 1))) << 4));
    if (m < a.M && n + 8 <= a.N) {
      u32x2* dst = reinterpret_cast<u32x2*>(a.C + m * a.ldc + n);   // (ldc is a multiple of four)
      if ((a.ldc & 7) == 0) *reinterpret_cast<u32x4*>(dst) = v;
      else { dst[0] = u32x2{v[0], v[1]}; dst[1] = u32x2{v[2], v[3]}; }
    }
  }
}

// C[m][n] = bf16(sum_s P[s][m][n]), fixed order
__global__ void gemm_bf16_reduce_kernel(TunedGemmArgs a) {
  const int64_t idx = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (idx >= a.M * a.N) return;
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < a.splits; ++s)
    sum += *reinterpret_cast<const f32x4*>(a.P + (size_t)s * a.M * a.N + idx);
  const int64_t m = idx / a.N, n = idx % a.N;
  u32x2* dst = reinterpret_cast<u32x2*>(a.C + m * a.ldc + n);
  if (a.accumulate) {
    const u32x2 old = *dst;
    sum[0] += __builtin_bit_cast(float, old[0] << 16);
    sum[1] += __builtin_bit_cast(float, old[0] & 0xFFFF0000u);
    sum[2] += __builtin_bit_cast(float, old[1] << 16);
    sum[3] += __builtin_bit_cast(float, old[1] & 0xFFFF0000u);
  }
  u32x2 pk;
  pk[0] = pack_bf16(sum[0], sum[1]);
  pk[1] = pack_bf16(sum[2], sum[3]);
  *dst = pk;
}

// ---------------------------------------------------------------------------
// Few rows (decoding): C[M][N] = A[M][K] B, A row form, B in either form.  The weights are read
// once and the rest is latency, so: one launch, no partials in memory, every load of a wave in
// flight before the first is waited for.  A workgroup owns 32 rows x 32 columns of C over all
// of K; wave w takes the 64-wide k slices w, w + 16, ...; MFMA rows are the columns of C, MFMA
// columns the rows of A.  The waves' partial tiles are added up through LDS in wave order.
// Both operands pass through a private LDS slice per wave, so that the loads are whole
// 128-byte (transposed weights: 64-byte) pieces of rows: fetched in operand layout, 8 bytes
// per lane from 32 rows, A held the address unit for 64 cycles a load.  What a CU then takes
// is the 27 bytes per clock it can load (128 rows in one workgroup: 30 us, in four: 8.4).
// 16 x 2048 x 2048: 7.8 us against 9.9 of the tiled kernel (64 x 128 tiles, the contraction
// split and summed by a second launch); 128 rows: 8.7 against 15.1.
// ---------------------------------------------------------------------------
constexpr int kSkinnyWaves = 16, kSkinnyRows = 32, kSkinnyCols = 32;
constexpr int kSkinnyWaveLds = 2 * 4096;   // a slice of B and one of A
constexpr int kSkinnyLds = kSkinnyWaves * kSkinnyWaveLds;
constexpr int kSkinnyK = 64;               // k per slice of this kernel
constexpr int kSkinnySlices = 2;           // k slices in flight per wave (registers)

template <bool B_TR>
__global__ __launch_bounds__(64 * kSkinnyWaves) void gemm_bf16_skinny_kernel(TunedGemmArgs a) {
  constexpr int NW = kSkinnyWaves, SL = kSkinnySlices;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 31, g = lane >> 5;
  const int64_t n0 = (int64_t)blockIdx.x * kSkinnyCols, m0 = (int64_t)blockIdx.y * kSkinnyRows;
  const int KT = (int)(a.K / kSkinnyK);
  unsigned char* btile = smem + wave * kSkinnyWaveLds;   // [64 k][32 n], or [32 n][64 k] swizzled
  unsigned char* atile = btile + 4096;                   // [32 m][64 k], swizzled
  // row-form pieces: load i takes rows 8 i + lane / 8, 16-byte chunk lane % 8
  const int lrow = lane >> 3, lchunk = lane & 7;
  const uint16_t* asrc = a.A + (m0 + lrow) * a.lda + 8 * lchunk;
  const uint16_t* bsrc = B_TR ? a.B + (int64_t)(lane >> 2) * a.ldb + n0 + 8 * (lane & 3)
                              : a.B + (n0 + lrow) * a.ldb + 8 * lchunk;
  f32x16 acc = f32x16{0};

  for (int s0 = wave; s0 < KT; s0 += NW * SL) {
    u32x4 w[SL][4], x[SL][4];
#pragma unroll
    for (int s = 0; s < SL; ++s) {
      const int sl = s0 + NW * s;
      if (sl >= KT) continue;
      const int64_t k0 = (int64_t)sl * kSkinnyK;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        w[s][i] = *reinterpret_cast<const u32x4*>(B_TR ? bsrc + (k0 + 16 * i) * a.ldb : bsrc + 8 * i * a.ldb + k0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        x[s][i] = u32x4{0, 0, 0, 0};
        if (m0 + 8 * i + lrow < a.M) x[s][i] = *reinterpret_cast<const u32x4*>(asrc + 8 * i * a.lda + k0);
      }
    }
#pragma unroll
    for (int s = 0; s < SL; ++s) {
      if (s0 + NW * s >= KT) continue;
      // (the wave's own LDS slice: its reads of the slice before are ahead of these stores in
      // the same queue)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<u32x4*>(btile + (B_TR ? i * 1024 + lane * 16 : tile_off_dh<64>(8 * i + lrow, lchunk))) = w[s][i];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<u32x4*>(atile + tile_off_dh<64>(8 * i + lrow, lchunk)) = x[s][i];
#pragma unroll
      for (int t2 = 0; t2 < 4; ++t2) {
        bf16x8 wf, xf;
        if constexpr (B_TR) {   // contraction slots follow the transposing read
          const int li = lane & 15;
          const unsigned char* p = btile + (16 * t2 + 4 * g + (li >> 2)) * 64 + (16 * ((lane >> 4) & 1) + 4 * (li & 3)) * 2;
          wf = join_tr(lds_read_tr16(p), lds_read_tr16(p + 8 * 64));
          const unsigned char* q = atile + 8 * g;
          xf = join_tr(*reinterpret_cast<const s16x4*>(q + tile_off_dh<64>(r, 2 * t2)),
                       *reinterpret_cast<const s16x4*>(q + tile_off_dh<64>(r, 2 * t2 + 1)));
        } else {
          wf = *reinterpret_cast<const bf16x8*>(btile + tile_off_dh<64>(r, 2 * t2 + g));
          xf = *reinterpret_cast<const bf16x8*>(atile + tile_off_dh<64>(r, 2 * t2 + g));
        }
        acc = mfma32(wf, xf, acc);
      }
    }
  }
  __syncthreads();
  f32x4* red = reinterpret_cast<f32x4*>(smem);   // [wave][4 quads][lane]
#pragma unroll
  for (int vq = 0; vq < 4; ++vq)
    red[(wave * 4 + vq) * 64 + lane] = f32x4{acc[4 * vq], acc[4 * vq + 1], acc[4 * vq + 2], acc[4 * vq + 3]};
  __syncthreads();
  if (tid >= 256) return;
  f32x4 sum = red[tid];
#pragma unroll
  for (int w = 1; w < NW; ++w) sum += red[w * 256 + tid];
  const int64_t m = m0 + (tid & 31), n = n0 + 8 * (tid >> 6) + 4 * ((tid >> 5) & 1);
  if (m < a.M) {
    u32x2 pk;
    pk[0] = pack_bf16(sum[0], sum[1]);
    pk[1] = pack_bf16(sum[2], sum[3]);
    *reinterpret_cast<u32x2*>(a.C + m * a.ldc + n) = pk;
  }
}

template <bool B_TR>
int launch_skinny(const TunedGemmArgs& a, hipStream_t stream) {
  if (hipError_t e0 = LdsLimit<&gemm_bf16_skinny_kernel<B_TR>, kSkinnyLds>::ensure(); e0 != hipSuccess)
    return (int)e0;
  hipLaunchKernelGGL(gemm_bf16_skinny_kernel<B_TR>,
                     dim3((unsigned)(a.N / kSkinnyCols), (unsigned)((a.M + kSkinnyRows - 1) / kSkinnyRows)),
                     dim3(64 * kSkinnyWaves), kSkinnyLds, stream, a);
  return (int)hipGetLastError();
}

// ---------------------------------------------------------------------------
// Up to 16 rows: a workgroup owns 16 columns of C, so that d_model = 2048 fills 128 CUs and not
// 64.  Same idea otherwise: wave w takes the 64-wide k slices w, w + 16, .., every load in flight
// before the first is waited for, the waves' partial tiles added up through LDS in wave order.
// 16x16x32 products: MFMA rows are the columns of C, MFMA columns the rows of A, whose operand
// is 16 bytes per lane of 16 rows as it lies in memory (no LDS); so is the weights' in row form.
// Transposed weights pass through the wave's LDS slice ([32 k][16 n] per product) for the
// transposing read.  Bound: one memory latency, and the 128-byte lines of the transposed weights,
// of which a workgroup uses a quarter (neighbours share them in one L2; read past the L1 they
// cost 3 us more).  Kernel above | this one: 1 x 1024 x 1024 4.9 | 4.0 us a product, 1 x 2048 x
// 2048 7.3 | 6.3, 16 x 2048 x 2048 7.6 | 7.0; row form 1 x 2048 x 2048 0.7 less, 16 rows 0.2 more.
// ---------------------------------------------------------------------------
constexpr int kFewCols = 16, kFewTile = 1024;   // LDS of one product's transposed weights
// rows up to which it is the faster one, by the weights' form
bool few_takes(bool b_tr, int64_t M) { return M <= (b_tr ? 16 : 8); }
template <bool B_TR>
__global__ __launch_bounds__(64 * kSkinnyWaves) void gemm_bf16_few_kernel(TunedGemmArgs a) {
  constexpr int NW = kSkinnyWaves, SL = kSkinnySlices;
  __shared__ __attribute__((aligned(16))) unsigned char smem[NW * SL * 2 * kFewTile];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i16 = lane & 15, gq = lane >> 4;
  const int64_t item = xcd_work_item(blockIdx.x, a.n_items);
  if (item >= a.n_items) return;
  const int64_t n0 = item * kFewCols;
  const int KT = (int)(a.K / kSkinnyK);
  unsigned char* btile = smem + wave * (SL * 2 * kFewTile);
  const uint16_t* bsrc = B_TR ? a.B + (int64_t)(lane >> 1) * a.ldb + n0 + 8 * (lane & 1) : a.B + (n0 + i16) * a.ldb + 8 * gq;
  const uint16_t* asrc = a.A + i16 * a.lda + 8 * gq;
  f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int s0 = wave; s0 < KT; s0 += NW * SL) {
    u32x4 w[SL][2], x[SL][2];
#pragma unroll
    for (int s = 0; s < SL; ++s) {
      const int sl = s0 + NW * s;
      if (sl >= KT) continue;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int64_t k0 = (int64_t)sl * kSkinnyK + 32 * t;
        w[s][t] = *reinterpret_cast<const u32x4*>(B_TR ? bsrc + k0 * a.ldb : bsrc + k0);
        x[s][t] = u32x4{0, 0, 0, 0};
        if (i16 < a.M) x[s][t] = *reinterpret_cast<const u32x4*>(asrc + k0);
      }
    }
#pragma unroll
    for (int s = 0; s < SL; ++s) {
      if (s0 + NW * s >= KT) continue;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        bf16x8 wf;
        if constexpr (B_TR) {   // (the wave's own slice: its reads follow its stores in the same queue)
          unsigned char* tile = btile + (2 * s + t) * kFewTile;
          *reinterpret_cast<u32x4*>(tile + lane * 16) = w[s][t];
          const unsigned char* p = tile + (8 * gq + (i16 >> 2)) * 32 + (i16 & 3) * 8;
          wf = join_tr(lds_read_tr16(p), lds_read_tr16(p + 4 * 32));
        } else {
          wf = __builtin_bit_cast(bf16x8, w[s][t]);
        }
        acc = mfma16(wf, __builtin_bit_cast(bf16x8, x[s][t]), acc);
      }
    }
  }
  __syncthreads();
  f32x4* red = reinterpret_cast<f32x4*>(smem);   // [wave][lane]
  red[tid] = acc;
  __syncthreads();
  if (tid >= 64) return;
  f32x4 sum = red[lane];
#pragma unroll
  for (int w = 1; w < NW; ++w) sum += red[w * 64 + lane];
  if (i16 < a.M)
    *reinterpret_cast<u32x2*>(a.C + i16 * a.ldc + n0 + 4 * gq) = u32x2{pack_bf16(sum[0], sum[1]), pack_bf16(sum[2], sum[3])};
}

template <bool B_TR>
int launch_few(TunedGemmArgs a, hipStream_t stream) {
  a.n_items = a.N / kFewCols;
  hipLaunchKernelGGL(gemm_bf16_few_kernel<B_TR>, dim3((unsigned)xcd_grid_size(a.n_items)), dim3(64 * kSkinnyWaves), 0, stream, a);
  return (int)hipGetLastError();
}

// Tile shape and split of the contraction, from what was measured (clocks of a CU at 2.2 GHz):
// a slice of k costs a workgroup kSliceClocks (the smaller shapes share the CU, so two of them
// take as long as one after the other); a workgroup starts in about 4000 and stores its tile at
// 9 bytes per clock (all CUs do so at the same time: 5 TB/s); the sum of the partials is a launch
// of about 9000 and reads 2600 bytes per clock.
struct GemmPlan { int shape, splits; int64_t slices_per_split; double clocks; };
constexpr int kShapeM[4] = {256, 256, 128, 64}, kShapeN[4] = {256, 128, 128, 128};
constexpr double kSliceClocks[2][4] = {{1900, 1220, 770, 550}, {1980, 1300, 850, 0}};   // [A transposed]
GemmPlan plan_tiles(bool a_tr, int64_t M, int64_t N, int64_t K) {
  const int64_t KT = (K + kGBK - 1) / kGBK;
  GemmPlan best{0, 1, KT, 0.0};
  for (int sh = 0; sh < (a_tr ? 3 : 4); ++sh) {
    const int64_t tiles = ((M + kShapeM[sh] - 1) / kShapeM[sh]) * ((N + kShapeN[sh] - 1) / kShapeN[sh]);
    for (int want = 1; want <= 16; ++want) {
      const int64_t per = (KT + want - 1) / want;
      if (want > 1 && (per < 8 || (KT + per - 1) / per != want)) continue;   // at least eight slices per workgroup
      const double out = kShapeM[sh] * kShapeN[sh] * (want > 1 ? 4 : 2) / 9.0;
      double cost = (double)((tiles * want + 255) / 256) * (per * kSliceClocks[a_tr][sh] + 4000 + out);
      if (want > 1) cost += 9000 + (double)want * M * N * 4 / 2600;
      if (best.clocks == 0.0 || cost < best.clocks) best = {sh, want, per, cost};
    }
  }
  return best;
}

template <bool A_TR, bool B_TR, typename G>
int launch_shape(TunedGemmArgs a, hipStream_t stream) {
  a.tiles_n = (a.N + G::BN - 1) / G::BN;
  a.n_items = ((a.M + G::BM - 1) / G::BM) * a.tiles_n * a.splits;
  if (hipError_t e0 = LdsLimit<&gemm_bf16_kernel<A_TR, B_TR, G>, G::kLds>::ensure(); e0 != hipSuccess) return (int)e0;
  hipLaunchKernelGGL((gemm_bf16_kernel<A_TR, B_TR, G>), dim3((unsigned)xcd_grid_size(a.n_items)), dim3(64 * G::NW),
                     G::kLds, stream, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.splits == 1) return (int)e;
  const int64_t n4 = a.M * a.N / 4;
  hipLaunchKernelGGL(gemm_bf16_reduce_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0,
                     stream, a);
  return (int)hipGetLastError();
}
template <bool A_TR, bool B_TR>
int launch_form(const TunedGemmArgs& a, int shape, hipStream_t stream) {
  switch (shape) {
    case 0: return launch_shape<A_TR, B_TR, Tile256x256>(a, stream);
    case 1: return launch_shape<A_TR, B_TR, Tile256x128>(a, stream);
    case 2: return launch_shape<A_TR, B_TR, Tile128x128>(a, stream);
    default: break;
  }
  if constexpr (A_TR) return -1;
  else return launch_shape<A_TR, B_TR, Tile64x128>(a, stream);
}

}  // namespace

// Where a few-rows kernel is the faster one: a round of the 32-column kernel's workgroups (one per
// CU) takes about 520 clocks per 64-wide slice of k and 2000 around them.  It is chosen for up to 512
// rows at d_model = 1024, 160 at 1536, 128 at 2048, 45 .. 96 at 2560 and not at all from 3072 on.
// Microseconds, few rows | tiled with its sum: d_model = 1024, 128 rows 5.0 | 9.1, 512 9.1 | 10.1,
// 513 11.5 | 10.0; 1536, 160 rows 6.5 | 13.0; 2048, 128 rows 8.7 | 15.1, 320 18.8 | 15.5; 2560, 64 rows
// 10.7 | 12.9, 128 16.9 | 14.6.  The tiled kernel gets some sizes too early: 2048, 129 .. 256 rows
// 12.4 .. 13.8 | 14.6 .. 15.2; 1536, 192 .. 320 rows 10.0 .. 11.2 | 13.7 .. 14.8; 3072 and 4096, 64 rows
// 12.6 | 14.7 and 15.2 | 17.1.  For 1 .. 16 rows the 16-column kernel lies on the same side of the
// tiled one: 2.7 .. 3.1 us less a product at 512, 3.4 .. 3.8 at 1024, 2.5 .. 2.9 at 2048; 1.1 .. 1.6
// more at 2560, 2.4 .. 2.9 at 3072, 2.0 .. 4.0 at 4096, 23 .. 28 at 5120.
bool skinny_takes(int64_t M, int64_t N, int64_t K) {
  if (N % kSkinnyCols != 0 || K % kSkinnyK != 0) return false;
  const int64_t wgs = ((M + kSkinnyRows - 1) / kSkinnyRows) * (N / kSkinnyCols);
  return (double)((wgs + 255) / 256) * (520.0 * (K / kSkinnyK) + 2000) < plan_tiles(false, M, N, K).clocks;
}

bool gemm_bf16_supported(bool a_tr, bool b_tr, const void* A, int64_t lda, const void* B,
                         int64_t ldb, const void* C, int64_t ldc, int64_t M, int64_t N, int64_t K) {
  auto al16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
  if (M < 1 || N < 8 || K < 1 || N % 8 != 0) return false;
  if (!al16(A) || !al16(B) || !al16(C) || lda % 8 != 0 || ldb % 8 != 0 || ldc % 4 != 0) return false;
  // a row-form operand is read in whole slices of k; a transposed one in whole
  // 8-wide groups of its row index
  if ((!a_tr || !b_tr) && K % kGBK != 0) return false;
  if (lda > (1 << 22) || ldb > (1 << 22)) return false;   // lane offsets inside a tile are 32-bit
  if (a_tr && (M < 8 || M % 8 != 0)) return false;
  if (b_tr && N % 8 != 0) return false;
  return true;
}

std::string gemm_bf16_plan(bool a_tr, int64_t M, int64_t N, int64_t K) {
  if (!a_tr && skinny_takes(M, N, K)) return "few rows";
  const GemmPlan plan = plan_tiles(a_tr, M, N, K);
  return std::to_string(kShapeM[plan.shape]) + "x" + std::to_string(kShapeN[plan.shape]) + " splits=" +
         std::to_string(plan.splits);
}

int gemm_bf16_few_columns(bool b_tr, int64_t M, int64_t N, int64_t K) {
  return !skinny_takes(M, N, K) ? 0 : few_takes(b_tr, M) ? kFewCols : kSkinnyCols;
}

size_t gemm_bf16_workspace_bytes(int64_t M, int64_t N, int64_t K) {
  const int s0 = plan_tiles(false, M, N, K).splits, s1 = plan_tiles(true, M, N, K).splits;
  const int splits = s0 > s1 ? s0 : s1;
  return splits > 1 ? (size_t)splits * M * N * sizeof(float) : 0;
}

int launch_gemm_bf16(bool a_tr, bool b_tr, const void* A, int64_t lda, const void* B, int64_t ldb,
                     void* C, int64_t ldc, int64_t M, int64_t N, int64_t K, void* ws, void* stream,
                     bool accumulate) {
  TunedGemmArgs a;
  a.accumulate = accumulate ? 1 : 0;
  a.A = static_cast<const uint16_t*>(A);
  a.B = static_cast<const uint16_t*>(B);
  a.C = static_cast<uint16_t*>(C);
  a.M = M; a.N = N; a.K = K; a.lda = lda; a.ldb = ldb; a.ldc = ldc;
  const GemmPlan plan = plan_tiles(a_tr, M, N, K);
  a.tiles_n = 0; a.n_items = 0;
  a.splits = plan.splits;
  a.slices_per_split = plan.slices_per_split;
  a.P = static_cast<float*>(ws);
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (!a_tr && skinny_takes(M, N, K) && !accumulate) {
    if (few_takes(b_tr, M)) return b_tr ? launch_few<true>(a, st) : launch_few<false>(a, st);
    return b_tr ? launch_skinny<true>(a, st) : launch_skinny<false>(a, st);
  }
  if (a.splits > 1 && !ws) return -1;
  if (!a_tr && b_tr) return launch_form<false, true>(a, plan.shape, st);
  if (!a_tr && !b_tr) return launch_form<false, false>(a, plan.shape, st);
  if (a_tr && b_tr) return launch_form<true, true>(a, plan.shape, st);
  return -1;   // transposed A with row-form B: no caller
}

}  // namespace mhffn
