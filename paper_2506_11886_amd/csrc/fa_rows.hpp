// Projection row by row onto a basis of fp32 precision (used by fa_compress, fa_compress_kv and fa_select_dims for fp32 segments,
// where the harmonics vary too fast for moments, or where a segment is too short to be worth two launches).
#pragma once

#include "fa_common.hpp"
#include "fa_moments.hpp"

namespace fa {

struct RowsParams {
  MomentTensor t[2];   // (mom is not used)
  int64_t sx_b, sx_h, sx_n;
  int B, H, N, M, T, t0, accumulate, keep_offset;
  int lead;            // zero tokens put in front, so that groups of 8 kept tokens are aligned
  int hw;              // 16-harmonic tiles per workgroup
  int steps;           // 32-token steps per wave
  int spc;             // steps of a chunk (grid z)
  float* part;         // partial sums of the chunks, [chunk][B*H][M][Dc] per tensor, or null: one chunk
  size_t part_z, part_stride[2];   // second tensor's place in it, floats from chunk to chunk
  int nmax;
};

// A wave adds up at most this many steps of 32 tokens in fp32 (2048 tokens; a workgroup's waves have eight such shares, D = 256
// four).  fa_select_dims, whose errors are differences of sums: half of them, the fp32 projection it would take else adds up 512
// tokens at a quarter of the tokens a product.
constexpr int kRowsLongest = 64;
constexpr int kRowsLongestSelect = 32;
constexpr int kRowsLongestF32 = 16;   // (fp32 rows: 512 tokens, as in the fp32 projection)

struct RowsPlan {
  bool use;
  int hw, groups, steps, spc, chunks, lead;
  double us;           // estimated time
};

struct RowsShape {
  int dtype, B, H, N, D, M;
  int64_t sx_n;
  int keep_offset, tensors;
  double Du;           // kept dims written, over the tensors
  bool stats;          // fa_select_dims: energies and weighted squares
};
// terms: bf16 terms of a basis value (2: 2^-17, 3: fp32)
RowsPlan make_rows_plan(const RowsShape& c, int terms, int longest, int most);
int launch_rows(const RowsParams& p, const RowsPlan& pl, int dtype, int D, int tensors, int terms, hipStream_t st, KernelTimers* tm);

}  // namespace fa
