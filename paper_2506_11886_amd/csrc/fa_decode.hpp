// Shared pieces of the decode kernels: launch parameters, sequence views, small device helpers.
#pragma once

#include "fa_common.hpp"
#include "fa_mma.hpp"

namespace fa {

constexpr int kBlock = 256;
constexpr int kWaves = 4;
constexpr int kWaves8 = 8;         // of the kernels for long series
constexpr int kMaxG = FA_MAX_GROUP;
constexpr int kTJ = 64;            // tokens per tile (rows of the E table)
constexpr int kRB = kTJ / 16;      // 16-row blocks per tile
constexpr int kXN = kTJ / 32;      // 32-token contraction steps per tile on the V side
constexpr int kMaxKT = 4;          // tiles per wave step
constexpr int kWChunk = 256;       // full-width rows per workgroup
constexpr int kMaxDvTiles = 8;     // kept V dims handled per middle row: 8 * 16
constexpr int kMaxPartials = 1024; // partial records per query head
constexpr unsigned kMaxDynLds = 160 * 1024 - 4096;   // dynamic LDS a workgroup may ask for
constexpr int kFinBlock = 256;     // threads of decode_finish

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2d __attribute__((ext_vector_type(2)));


struct DecodeParams {
  const void* q;
  const float* ck;
  const float* cv;
  const uint8_t* kmask;
  const uint8_t* vmask;
  const void* k_keep;
  const void* v_keep;
  const void* k_full;
  const void* v_full;
  int64_t kk_stride, vk_stride, full_stride;
  int B, Hq, Hkv, G, D, Dkc, Dvc, Dku, Dvu, M, T, t0, N, W;
  int Tq, Gq;       // query tokens per sequence (1: plain decode) and query heads per KV head and token
  int Gp, KT;       // group size padded to a power of two, tiles per wave step
  int Mint;         // series length: 2 * (M/2) padded to a compiled size
  int Sw, Sm;       // chunks of full-width rows / of middle rows (middle chunks come first)
  int nprep, Swp;   // workgroups per head of the series-coefficient part when the full-width rows share its launch;
                    // chunks of full-width rows inside the middle-row launch (0 when they ran with the coefficients)
  int chunk_m;      // middle rows per chunk (multiple of the workgroup step)
  int recm, recw;   // floats per partial record: 4 + 16 ceil(Dvu/16) + Mint (middle), 4 + D (full rows)
  unsigned lds_tab; // bytes of the exchange / reduction region of a middle-row workgroup
  float scale;
  double ph_scale;  // 2^32 / T
  float* gs;        // [B,Hq,Mint] series coefficients, K-side order
  float* g0;        // [B,Hq]      constant-term coefficient
  void* qkeep;      // [B,Hq,Dkq]  q at the kept K dims, zero padded to Dkq = 32 ceil(Dku/32)
  float* part_m;    // [B,Hq,Sm,recm]
  float* part_w;    // [B,Hq,Sw,recw]
  float* out;       // [B,Hq,D]
  const int32_t* seq_n;   // [B] middle rows of each sequence (<= N), or null: N for all
  const int32_t* seq_w;   // [B] full-width rows of each sequence (<= W), or null: W for all
  int Sw_rec;       // full-row records reserved per query head (= Sw of the longest sequence)
  int wrb;          // 16-row blocks per wave of a full-width-row workgroup: 4 (256 rows per workgroup) or 1 (64)
  // (what only decode_local reads comes last: in the middle it moved the kernel arguments of the others, whose scalar loads and
  // spills then fell out worse: fp32, 14 sequences of 2 heads x 4613 rows, M = 92, middle rows 38.1 -> 38.9 us, 6 - 12 more spills)
  int U, ni;        // local Chebyshev form of the middle rows: tokens per block, steps per wave
  uint64_t ph64;    // 2^63 / T
};

// What a workgroup uses of one sequence: its row counts, the chunking that follows from them and
// where its records go.  The three-launch kernels take the call's own values; the one-launch form
// resolves them per sequence.
struct SeqView {
  int N, W, Sm, Sw, chunk_m;
  float* part_m;
  float* part_w;
};
// rows of sequence b: the call's counts, or the sequence's own (clamped into them) when the caller gave lists
__device__ __forceinline__ int seq_middle_rows(const DecodeParams& p, int b) {
  return p.seq_n ? min(max(p.seq_n[b], 0), p.N) : p.N;
}
__device__ __forceinline__ int seq_full_rows(const DecodeParams& p, int b) {
  return p.seq_w ? min(max(p.seq_w[b], 0), p.W) : p.W;
}
__device__ __forceinline__ SeqView call_view(const DecodeParams& p, int b) {
  return SeqView{seq_middle_rows(p, b), seq_full_rows(p, b), p.Sm, p.Sw, p.chunk_m, p.part_m, p.part_w};
}

// Middle-row chunks [chunk_lo, chunk_hi) of a (sequence, KV head) that lie past the sequence's rows:
// records that say "nothing here" (maximum -inf, everything else zero), for every query head.
__device__ __forceinline__ void write_empty_middle(const DecodeParams& p, size_t hq0, int chunk_lo, int chunk_hi,
                                                   int nthreads) {
  const int recm = p.recm, G = p.G;
  const int per = (chunk_hi - chunk_lo) * recm;
  for (int it = threadIdx.x; it < G * per; it += nthreads) {
    const int h = it / per, x = it - h * per;
    p.part_m[((hq0 + h) * p.Sm + chunk_lo) * recm + x] = (x % recm == 0) ? -INFINITY : 0.0f;
  }
}

// LDS of a workgroup of the one-launch form, after the exchange region of the middle-row phase:
// series coefficients [G][Mint + 32] | packed kept q [G][32] | constant-term coefficients | the
// middle-row record [G][recm] | the full-row record [G][recw] | C_v of the pair [M][Dvc] (1 KB aligned)
struct FusedLds {
  unsigned gs, qk, g0, recm, recw, cv, total;
};
__host__ __device__ __forceinline__ FusedLds fused_lds(unsigned lds_tab, int G, int Mint, int recm, int recw, int M,
                                                       int Dvc) {
  FusedLds L;
  L.gs = lds_tab;
  L.qk = L.gs + G * (Mint + 32) * 4;
  L.g0 = L.qk + G * 32 * 2;
  L.recm = L.g0 + 64;
  L.recw = L.recm + G * recm * 4;
  L.cv = (L.recw + G * recw * 4 + 1023u) & ~1023u;
  L.total = L.cv + ((static_cast<unsigned>(M) * Dvc * 4 + 1023u) & ~1023u);
  return L;
}

// ---------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------
template <typename T> struct SeriesType;
template <> struct SeriesType<bf16_t> { using type = f16_t; };   // E, g', p on the series side
template <> struct SeriesType<float> { using type = float; };

__device__ __forceinline__ void pack8(Frag<f16_t>& f, const float* v) {
#pragma unroll
  for (int e = 0; e < 4; ++e)
    f.v[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{v[2 * e], v[2 * e + 1]}, f16x2));
}
__device__ __forceinline__ void pack8(Frag<bf16_t>& f, const float* v) {
#pragma unroll
  for (int e = 0; e < 4; ++e)
    f.v[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{v[2 * e], v[2 * e + 1]}, bf16x2));
}
__device__ __forceinline__ void pack8(Frag<float>& f, const float* v) {
#pragma unroll
  for (int e = 0; e < 8; ++e) f.v[e] = v[e];
}

__device__ __forceinline__ void unpack8(const Frag<bf16_t>& f, float* v) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[2 * e] = __uint_as_float(f.v[e] << 16);
    v[2 * e + 1] = __uint_as_float(f.v[e] & 0xffff0000u);
  }
}
__device__ __forceinline__ void unpack8(const Frag<float>& f, float* v) {
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = f.v[e];
}
// element e of a fragment, as stored
__device__ __forceinline__ bf16_t frag_elem(const Frag<bf16_t>& f, int e) {
  return bf16_t{static_cast<uint16_t>((f.v[e >> 1] >> (16 * (e & 1))) & 0xffffu)};
}
__device__ __forceinline__ float frag_elem(const Frag<float>& f, int e) { return f.v[e]; }
__device__ __forceinline__ float to_f32(bf16_t x) { return bf16_to_f32(x.bits); }
__device__ __forceinline__ float to_f32(float x) { return x; }

// keep the first `nvalid` (<= 8, may be <= 0) elements, zero the rest
__device__ __forceinline__ void mask_tail(Frag<bf16_t>& f, int nvalid) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t lo = (2 * e < nvalid) ? 0x0000ffffu : 0u;
    const uint32_t hi = (2 * e + 1 < nvalid) ? 0xffff0000u : 0u;
    f.v[e] &= (lo | hi);
  }
}
__device__ __forceinline__ void mask_tail(Frag<float>& f, int nvalid) {
#pragma unroll
  for (int e = 0; e < 8; ++e)
    if (e >= nvalid) f.v[e] = 0.0f;
}

// cos / sin of a 32-bit fixed-point phase (2^32 = one turn)
template <typename T>
__device__ __forceinline__ void phase_cs(uint32_t ph, float* c, float* s) {
  const float x = static_cast<float>(static_cast<int32_t>(ph)) * 2.3283064365386963e-10f;  // turns in [-0.5, 0.5)
  if constexpr (sizeof(T) == 4) {
    sincospif(2.0f * x, s, c);          // fp32 inputs: full-accuracy evaluation
  } else {
    *s = __builtin_amdgcn_sinf(x);      // hardware sin/cos take turns
    *c = __builtin_amdgcn_cosf(x);
  }
}

// fixed-point phase of position pos: frac(pos / T) * 2^32 (wraps for pos >= T)
__device__ __forceinline__ uint32_t phase_of(int pos, double ph_scale) {
  return static_cast<uint32_t>(static_cast<uint64_t>(static_cast<double>(pos) * ph_scale));
}

// value held by lane i of the caller's quad (4 consecutive lanes)
__device__ __forceinline__ float quad_bcast(float v, int i) {
  const int x = __float_as_int(v);
  int r;
  switch (i) {
    case 0: r = __builtin_amdgcn_mov_dpp(x, 0x00, 0xf, 0xf, true); break;
    case 1: r = __builtin_amdgcn_mov_dpp(x, 0x55, 0xf, 0xf, true); break;
    case 2: r = __builtin_amdgcn_mov_dpp(x, 0xaa, 0xf, 0xf, true); break;
    default: r = __builtin_amdgcn_mov_dpp(x, 0xff, 0xf, 0xf, true); break;
  }
  return __int_as_float(r);
}

// rotation by N lanes within each row of 16 lanes (lane i receives lane (i + N) % 16 of its row)
template <int N>
__device__ __forceinline__ float row_ror(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + N, 0xf, 0xf, false));
}
// sum / max over the lanes of a row whose indices differ by a multiple of `stride` (a power of two)
__device__ __forceinline__ float row_stride_sum(float v, int stride) {
  if (stride <= 8) v += row_ror<8>(v);
  if (stride <= 4) v += row_ror<4>(v);
  if (stride <= 2) v += row_ror<2>(v);
  if (stride <= 1) v += row_ror<1>(v);
  return v;
}
__device__ __forceinline__ float row_stride_max(float v, int stride) {
  if (stride <= 8) v = fmaxf(v, row_ror<8>(v));
  if (stride <= 4) v = fmaxf(v, row_ror<4>(v));
  if (stride <= 2) v = fmaxf(v, row_ror<2>(v));
  if (stride <= 1) v = fmaxf(v, row_ror<1>(v));
  return v;
}

// value of lane `src` (compile-time) broadcast to the wave
template <int SRC>
__device__ __forceinline__ float lane_value(float v) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), SRC));
}
// wave-wide sum / max, result in every lane: rotations inside the rows, then the four row totals
__device__ __forceinline__ float wave_sum_fast(float v) {
  v = row_stride_sum(v, 1);
  return (lane_value<0>(v) + lane_value<16>(v)) + (lane_value<32>(v) + lane_value<48>(v));
}
__device__ __forceinline__ float wave_max_fast(float v) {
  v = row_stride_max(v, 1);
  return fmaxf(fmaxf(lane_value<0>(v), lane_value<16>(v)), fmaxf(lane_value<32>(v), lane_value<48>(v)));
}

// every wave reads the whole mask row (D <= 256) and keeps it as 4 ballot words
__device__ __forceinline__ void mask_ballots(const uint8_t* mask, int D, int lane, uint64_t* bal) {
  uint8_t b[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) b[j] = mask[min(lane + 64 * j, D - 1)];
#pragma unroll
  for (int j = 0; j < 4; ++j) bal[j] = __ballot(b[j] != 0 && lane + 64 * j < D);
}

// rank of dimension d among the kept dims (>= 0) or -(1 + rank among the
// compressed dims), from the ballot words of the mask
__device__ __forceinline__ int dim_rank(const uint64_t* bal, int d) {
  const int w = d >> 6;
  const uint64_t bit = 1ull << (d & 63);
  int nc = 0;
  uint64_t hit = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {   // static indices only: the words stay in registers
    const uint64_t below = (j < w) ? ~0ull : ((j == w) ? (bit - 1ull) : 0ull);
    nc += __popcll(bal[j] & below);
    hit |= bal[j] & ((j == w) ? bit : 0ull);
  }
  return hit ? -(1 + nc) : d - nc;
}

constexpr float kSoftmaxSlack = 8.0f;   // how far a score may exceed its column's reference before the reference moves

// max over the four 16-lane rows of a wave, per lane position, result in every lane
__device__ __forceinline__ float cross_row_max(float v) {
  auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float cross_row_sum(float v) {
  auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

}  // namespace fa
