// Projection of long segments through local moments (used by fa_compress, fa_compress_kv and
// fa_select_dims when the M kept harmonics vary slowly over a block of tokens).
//
// With the block's centre c and x = (j - c) / (U / 2) in [-1, 1] the Jacobi-Anger expansion is
//   exp(i w_n j) = exp(i w_n c) * sum_p (2 - [p = 0]) i^p J_p(theta_n) T_p(x),  theta_n = w_n U / 2,
// and J_p falls off like (theta/2)^p / p! once p > theta: P = 16 Chebyshev polynomials carry every
// harmonic of a block with theta <= kThetaBf16 to 2e-6 (kThetaF32: 1e-8).  Hence
//   mu[p, i] = sum_{j in block} T_p(x_j) X[j, i]                          (fa_moments: one pass over X)
//   C[n, i]  = sum_blocks Rot(w_n c) * (2 - [p = 0]) i^p J_p(theta_n) mu  (fa_expand)
// so a token costs 16 matrix rows instead of M, and the M-row contraction runs once per block.
// Measured, direct projection -> moments: K and V of 8 heads x 129020 tokens, M = 512, 252 -> 145 us
// (fa_moments moves 0.62 GB in 112 us = 5.5 TB/s); 8 x 31740 tokens, M = 256, 47.1 -> 46.3 us; a 2 K
// piece at an offset that is no multiple of 8, 94.6 -> 27.1 us (K and V, four launches); fa_select_dims on
// 8 x 31740 tokens 294 -> 37 us.
#pragma once

#include "fa_common.hpp"

namespace fa {

constexpr int kMomP = 16;             // Chebyshev polynomials per block
constexpr double kThetaBf16 = 6.0;    // 2 J_16(6.0) = 2.4e-6, far below the 2^-9 of bf16 data
constexpr double kThetaF32 = 4.2;     // 2 J_16(4.2) = 1.0e-8, below fp32 rounding
constexpr int kMomMinU = 64;
constexpr int kMomMaxU = 1024;        // tokens per block (the Chebyshev table lives in LDS)

struct MomentPlan {
  bool use;
  int umax;            // longest block the expansion allows (a measure of T / M: about 3.8 T / M)
  int U, S;            // tokens per block, 32-token steps per block
  int lead;            // zero tokens put in front, so that groups of 8 kept tokens are aligned
  int blocks, bpc;     // blocks per (sequence, head), blocks per workgroup
  int chunks;          // workgroups per (sequence, head)
  int parts;           // bf16 terms of a Chebyshev value (2: 2^-17, 3: fp32)
  unsigned lds;
  size_t mom_bytes;    // workspace of one tensor
  size_t op_bytes;     // workspace of the call: A operands of fa_expand16
};

// the plan for `tensors` tensors of one shape that share a launch; keep_offset only matters mod 8
MomentPlan make_moment_plan(int dtype, int B, int H, int N, int D, int Dc, int M, int T, int keep_offset,
                            int tensors, bool exact);

struct MomentTensor {
  const void* x;
  const uint8_t* mask;   // null: every dim is compressed
  float* mom;            // [B*H][blocks][Dc][16]
  void* keep;            // null: nothing kept is written
  float* coeffs;         // [B*H][M][Dc]
  float* epart;          // fa_select_dims: per-chunk sums of squares [chunks][B*H][D]
  double* ecoef;         // fa_select_dims: weighted squares [row tiles][B*H][D] instead of coefficients
  int64_t keep_stride;
  int Dc, Du, keep_layout, keep_pitch;
};

struct MomentParams {
  MomentTensor t[2];
  int64_t sx_b, sx_h, sx_n;
  int B, H, N, D, M, T, t0, accumulate, keep_offset;
  int U, S, lead, blocks, bpc, nmax, tiles;
  void* op;              // A operands of fa_expand16 [16-harmonic tile][2-block step][4 KB]
};

int launch_moments(const MomentParams& p, const MomentPlan& pl, int tensors, hipStream_t st, KernelTimers* tm);
int launch_expand(const MomentParams& p, int tensors, hipStream_t st, KernelTimers* tm);

constexpr int kExpandRows = 16;       // harmonics per workgroup of fa_expand
// 16-column tiles a workgroup of fa_expand16 takes out of ct: all share the operands; with fewer workgroups than units two groups of columns.
// At exactly one workgroup per unit (tiles x pairs = 256: numbers of heads and states that are powers of two) and many blocks, two groups
// of two tiles each are as many workgroups and read less (16 pairs, M = 512, 112 dims: 128 K tokens, the call 144.6 -> 140.7 us, 32 K
// tokens 64.9 -> 62.1; few blocks lose, 72 of 32 pairs, M = 256: 83.3 -> 85.2; the line between them is not measured closer than that)
inline int expand_columns(int ct, int tiles, double pairs, int blocks) {
  int ctw = ct < 8 ? ct : 8;
  const bool one_round = ct > 4 && tiles > 1 && blocks >= 128 && tiles * pairs <= 256.0;
  if (ct > 2 && ct <= 8 && (tiles * pairs < 256.0 || one_round)) ctw = (ct + 1) / 2;
  return ctw < 2 ? 2 : ctw;
}
inline int expand_tiles_per_wg(int ct, int tiles, double pairs, int blocks) {
  const int ctw = expand_columns(ct, tiles, pairs, blocks);
  return tiles > 1 && pairs * tiles * ((ct + ctw - 1) / ctw) > 256.0 ? 2 : 1;
}
inline int expand_tiles(int M) { return M / 2 > 0 ? (M / 2 + kExpandRows - 1) / kExpandRows : 1; }

}  // namespace fa
