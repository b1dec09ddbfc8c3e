// Projection of rows onto the M basis functions, the basis formed on the fly in fp32 and split into bf16 terms (fp32 rows are, too):
//   C[m,i] = sum_j phi_m(t0+j) X[j,i]
// A workgroup owns (sequence, head), `hw` tiles of 16 harmonics and a chunk of the tokens; its waves take the 32-token steps in turn
// and their shares meet in LDS.  One chunk: one launch and no partial sums in memory; more leave theirs to a reduction.

#include "fa_rows.hpp"

#include "fa_mma.hpp"

namespace fa {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

template <typename T, int D>
struct RowsTile {
  static constexpr bool kF32 = sizeof(T) == 4;
  static constexpr int kCols = D == 64 || kF32 ? 4 : 8;        // 16-column tiles per wave
  static constexpr int kHalves = D / 16 / kCols;               // waves side by side over the columns
  static constexpr int kSlots = 8 / kHalves;                   // waves along tokens and harmonics
  static constexpr bool kOwn = kF32 || kHalves == 1;           // every wave fills a tile of its own (else the two of a slot one together)
  static constexpr int kRow = kF32 ? 64 : D;                   // columns of a tile
  static constexpr int kPitch = 2 * kRow + 32;                 // bytes of a tile row
  static constexpr int kVec = 16 / sizeof(T);                  // elements of a 128-bit vector
  static constexpr int kLoads = 32 * (kRow / kVec) / (kOwn ? 64 : 64 * kHalves);   // vectors per thread and step of 32 tokens
  // fp32: a tile for each of the three terms of a value; two waves to a tile: two tiles in turn
  static constexpr unsigned kTiles = (kF32 ? 3u * 8 : kOwn ? 8u : 2u * kSlots) * 32 * kPitch;
  static constexpr unsigned kSums = 8u * 2 * kCols * 1024 + kSlots * D * 4;   // the epilogue's
  static constexpr unsigned kExtra = kTiles > kSums ? kTiles : kSums;         // offset of fa_select_dims' energies
  static constexpr unsigned kLds = kExtra + kSlots * D * 8;
};

// cosine and sine of 2 pi n pos / T; the product is exact, its fraction is taken in fp64
__device__ __forceinline__ void turn(int64_t npos, double inv_t, float* c, float* s) {
  double f = static_cast<double>(npos) * inv_t;
  f -= rint(f);
  sincospif(2.0f * static_cast<float>(f), s, c);
}

// eight values as NT bf16 terms, rounded two at a time
template <int NT>
__device__ __forceinline__ void split_terms(const float (&v)[8], Frag<bf16_t> (&t)[NT]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    f32x2 r = f32x2{v[2 * e], v[2 * e + 1]};
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, bf16x2));
      t[k].v[e] = w;
      if (k + 1 < NT) {
        r[0] -= __builtin_bit_cast(float, w << 16);
        r[1] -= __builtin_bit_cast(float, w & 0xffff0000u);
      }
    }
  }
}

constexpr bool rows_stats_tile(int D) { return D > 64; }
constexpr int kReseed = 8;   // steps between exact phases

// NT: bf16 terms of a basis value; kEnergy (fa_select_dims): sums of squares, and weighted squares of the states instead of them.
// grid (tensors * B * H, groups of hw 16-harmonic tiles): the workgroups of a pair share an XCD's L2 when the pairs are a
// multiple of eight.  Wave (column half, tile, share of the steps).  A wave stages its 32 rows in an LDS tile of its own and
// reads them back transposed (ds_read_b64_tr_b16) as the B operand; its A operands are one harmonic's cosines and sines per
// lane, at the eight tokens of the lane's k slots, rotated by a step's angle and split anew each step.  All D columns are
// multiplied (the kept ones' sums are dropped), so that nothing is gathered.  No barrier in the loop but at D = 256, where the
// two waves of a slot fill a tile together: with one per 256 tokens and tiles shared by all waves, 8 x 2048 tokens, M = 256, took
// 23.5 us a call against 16.5.
// Bound: instruction issue; see make_rows_plan for the rate.
template <typename T, int D, int NT, bool kEnergy>
__global__ __launch_bounds__(512, 2) void project_rows(RowsParams p) {
  using L = RowsTile<T, D>;
  constexpr bool kF32 = L::kF32;
  constexpr int NV = L::kRow / L::kVec, PB = L::kPitch, CW = L::kCols, NL = L::kLoads, RPL = (L::kOwn ? 64 : 64 * L::kHalves) / NV;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ __attribute__((aligned(16))) uint16_t kdim[D + 8];
  __shared__ int16_t cidx[D], crank[D];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, r16 = lane & 15;
  const int BH = p.B * p.H;
  const int z = blockIdx.x >= BH;
  const int bh = blockIdx.x - (z ? BH : 0), b = bh / p.H, h = bh - b * p.H;
  const uint8_t* mask = z ? p.t[1].mask : p.t[0].mask;
  const int Dc = z ? p.t[1].Dc : p.t[0].Dc, Du = D - Dc;
  const T* xb = static_cast<const T*>(z ? p.t[1].x : p.t[0].x) + b * p.sx_b + h * p.sx_h;
  const int N = p.N, lead = p.lead, hw = p.hw;

  // ---- this wave's harmonics, and its share of the 32-token steps: every shares-th
  const int half = wave % L::kHalves, slot = wave / L::kHalves;
  const int ht = slot % hw, share = slot / hw, shares = L::kSlots / hw;
  const int htile = blockIdx.y * hw + ht;
  // the wave that takes the constant function, too, and the energies of fa_select_dims: that of the first tile; above D = 64, where
  // both would not leave it the registers (59 spilled), fa_select_dims has a tile of its own for them behind the last one, in
  // the accumulators that hold cosines and sines elsewhere (2 pairs x 2531, M = 316: 34.5 -> 23.8 us)
  constexpr bool kStats = kEnergy && rows_stats_tile(D);
  const int stile = kStats ? (p.nmax + 15) / 16 : 0;
  const bool first = htile == stile;
  const bool live = first || htile * 16 < p.nmax;

  const int wl = L::kOwn ? lane : lane + 64 * half, ch = wl % NV, row0 = wl / NV;
  const int st0 = kEnergy ? 0 : blockIdx.z * p.spc, st1 = kEnergy ? p.steps : min(p.steps, st0 + p.spc);   // this chunk's steps
  const uint32_t lane_bytes = (kF32 ? half * 256u : 0u) + ch * 16u;
  // Rows are requested through a buffer descriptor that begins at the step's first row: a lane's offsets are the same in every
  // step, and rows past the segment come back as zeros.  Only the first step may have rows in front of it (made zero below).
  const uint32_t row_bytes = static_cast<uint32_t>(p.sx_n) * static_cast<uint32_t>(sizeof(T));
  const int64_t total = static_cast<int64_t>(N - 1) * row_bytes + static_cast<int>(sizeof(T)) * D;
  uint32_t voff[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) voff[i] = (row0 + i * RPL) * row_bytes + lane_bytes;
  auto load = [&](u32x4 (&x)[NL], int st) {
    const int64_t first = static_cast<int64_t>((st * shares + share) * 32 - lead) * row_bytes;
    const int64_t left = total - first;
    const uint32_t bytes = left <= 0 ? 0u : left > 0xffffffffll ? 0xffffffffu : static_cast<uint32_t>(left);
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(reinterpret_cast<const char*>(xb)) + (left <= 0 ? 0 : first), 0, bytes, 0x00027000);
#pragma unroll
    for (int i = 0; i < NL; ++i) x[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff[i], 0, 0));
  };
  uint8_t mb[D / 64];
#pragma unroll
  for (int j = 0; j < D / 64; ++j) mb[j] = mask ? mask[static_cast<size_t>(bh) * D + lane + 64 * j] : uint8_t{1};
  u32x4 x[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {                                // (the first step: clamped)
    const int j = min(max((st0 * shares + share) * 32 - lead + row0 + i * RPL, 0), N - 1);
    x[i] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(xb) + static_cast<uint64_t>(j) * row_bytes + lane_bytes);
  }

  // ---- compressed ranks, kept dims in order (pad entries point at the zero column of a tile row)
  {
    uint64_t bal[D / 64];
#pragma unroll
    for (int j = 0; j < D / 64; ++j) bal[j] = __ballot(mb[j] != 0);
    if (tid < D) {
      const int w = tid >> 6;
      const uint64_t bit = 1ull << (tid & 63);
      int nc = 0;
      bool hit = false;
#pragma unroll
      for (int j = 0; j < D / 64; ++j) {
        nc += __popcll(bal[j] & ((j < w) ? ~0ull : ((j == w) ? (bit - 1ull) : 0ull)));
        hit = hit || (j == w && (bal[j] & bit) != 0);
      }
      cidx[tid] = hit && nc < Dc ? static_cast<int16_t>(nc) : static_cast<int16_t>(-1);   // (nothing past column Dc)
      crank[tid] = hit ? static_cast<int16_t>(-1) : static_cast<int16_t>(tid - nc);
      if (!hit) kdim[tid - nc] = static_cast<uint16_t>(tid);
    }
    if (tid < 8) kdim[Du + tid] = D;
  }
  if constexpr (!kF32)
    for (int r = tid; r < static_cast<int>(L::kTiles / PB); r += 512) *reinterpret_cast<u32x4*>(smem + r * PB + 2 * D) = u32x4{0u, 0u, 0u, 0u};

  const int n = htile * 16 + 1 + r16;
  const double inv_t = 1.0 / static_cast<double>(p.T);
  float c1, s1, c16, s16, cj, sj;
  turn(n, inv_t, &c1, &s1);
  turn(static_cast<int64_t>(n) * 16, inv_t, &c16, &s16);
  turn(static_cast<int64_t>(n) * (32 * shares), inv_t, &cj, &sj);
  float bc[8], bs[8];                                           // basis of slot e: token 4 g + e, or 16 + 4 g + e - 4
  auto seed = [&](int st) {
    const int64_t pos = static_cast<int64_t>(p.t0) - lead + (static_cast<int64_t>(st) * shares + share) * 32 + 4 * g;
    turn(pos * n, inv_t, &bc[0], &bs[0]);
    bc[4] = bc[0] * c16 - bs[0] * s16;
    bs[4] = bs[0] * c16 + bc[0] * s16;
#pragma unroll
    for (int e = 0; e < 8; e += 4)
#pragma unroll
      for (int i = 1; i < 4; ++i) {
        bc[e + i] = bc[e + i - 1] * c1 - bs[e + i - 1] * s1;
        bs[e + i] = bs[e + i - 1] * c1 + bc[e + i - 1] * s1;
      }
  };

  const bool keep_rows = (z ? p.t[1].keep_layout : p.t[0].keep_layout) == FA_KEEP_ROWS;
  T* keep = static_cast<T*>(z ? p.t[1].keep : p.t[0].keep);
  const bool write_keep = keep != nullptr && Du > 0;
  const int kp = z ? p.t[1].keep_pitch : p.t[0].keep_pitch;
  if (write_keep) keep += static_cast<int64_t>(bh) * (z ? p.t[1].keep_stride : p.t[0].keep_stride);
  const int kdiv = max(1, keep_rows ? kp >> 3 : Du);               // kept vectors per token / per 8-token group
  const uint32_t kmagic = ((1u << 21) + kdiv - 1) / kdiv;         // it / kdiv exactly: it * kdiv < 2^21

  // (acc0: column sums, the constant function; fp32: of the lane's own rows and columns)
  constexpr int N0 = kF32 || kStats ? 1 : CW;
  f32x4 acc[2][CW], acc0[N0], ene[CW];
  acc0[0] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < CW; ++w) acc[0][w] = acc[1][w] = acc0[N0 == 1 ? 0 : w] = ene[w] = f32x4{0.f, 0.f, 0.f, 0.f};
  // Sums of squares only grow, and an fp32 sum over all steps would round one way: they go to fp64, in LDS, every kReseed steps.
  // (They are the diagonal of X^T X: column r16 in lane group r16 >> 2, element r16 & 3.)
  double* enr = reinterpret_cast<double*>(smem + L::kExtra);
  auto flush_energy = [&]() {
#pragma unroll
    for (int w = 0; w < CW; ++w) {
      f32x4& sq = kStats ? acc[1][w] : ene[w];
      const float lo = (r16 & 1) ? sq[1] : sq[0], hi = (r16 & 1) ? sq[3] : sq[2];
      if (g == (r16 >> 2)) {
        double* e = enr + share * D + (half * CW + w) * 16 + r16;
        *e += (r16 & 2) ? hi : lo;
      }
      sq = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };
  Frag<bf16_t> ones;
  ones.v = u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};

  if constexpr (kEnergy) {
    for (int i = tid; i < L::kSlots * D; i += 512) enr[i] = 0.0;
  }
  __syncthreads();                                              // kdim, cidx, zero columns
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int j = (st0 * shares + share) * 32 - lead + row0 + i * RPL;
    if (j < 0 || j >= N) x[i] = u32x4{0u, 0u, 0u, 0u};
  }
  int krank[4];                                                 // fp32: ranks of the lane's columns among the kept dims, or -1
  if constexpr (kF32) {
    const int c0 = half * 64 + 4 * ch;
#pragma unroll
    for (int e = 0; e < 4; ++e) krank[e] = crank[c0 + e];
  }
  // kept dims: the workgroups of a pair take the steps in turn, and the waves of a share theirs
  const int turns = static_cast<int>(gridDim.y) * hw;
  int my_turn = static_cast<int>(blockIdx.y) * hw + ht;
  for (int st = st0; st < st1; ++st) {
    const int v = (st * shares + share) * 32;                   // first (virtual) token: token j is virtual j + lead
    unsigned char* tile = smem + (kF32 ? 3 * wave : L::kOwn ? wave : (st & 1) * L::kSlots + slot) * (32 * PB);
    if constexpr (kF32) {
      if (first) {
#pragma unroll
        for (int i = 0; i < NL; ++i) acc0[0] += __builtin_bit_cast(f32x4, x[i]);
      }
      // three bf16 terms, cut off (a value of 24 bits is their sum exactly, and the largest stay finite)
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        f32x4 r = __builtin_bit_cast(f32x4, x[i]);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          u32x2 w;
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const uint32_t lo = __float_as_uint(r[2 * e]), hi = __float_as_uint(r[2 * e + 1]);
            w[e] = __builtin_amdgcn_perm(hi, lo, 0x07060302u);   // the upper halves
            if (k < 2) {
              r[2 * e] -= __uint_as_float(lo & 0xffff0000u);
              r[2 * e + 1] -= __uint_as_float(hi & 0xffff0000u);
            }
          }
          *reinterpret_cast<u32x2*>(tile + k * (32 * PB) + (row0 + i * RPL) * PB + ch * 8) = w;
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < NL; ++i) *reinterpret_cast<u32x4*>(tile + (row0 + i * RPL) * PB + ch * 16) = x[i];
    }
    // kept dims of fp32 rows: element by element, while they are in registers
    if constexpr (kF32) {
      if (write_keep && my_turn-- == 0 && v < N + lead) {
        my_turn = turns - 1;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
          const int j = v + row0 + i * RPL - lead;
          if (j >= 0 && j < N) {
            const int64_t tok = static_cast<int64_t>(p.keep_offset) + j;
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (krank[e] >= 0)
                keep[keep_rows ? tok * kp + krank[e] : ((tok >> 3) * Du + krank[e]) * 8 + (tok & 7)] = __uint_as_float(x[i][e]);
            if (keep_rows && half == 0 && ch < kp - Du) keep[tok * kp + Du + ch] = 0.0f;   // (pad columns)
          }
        }
      }
    }
    load(x, st + 1);
    if constexpr (!L::kOwn) {
      lds_barrier();
    } else {                                                    // a wave's own LDS operations take place in order
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
      __builtin_amdgcn_wave_barrier();
    }
    if (live && v < N + lead) {
      const unsigned char* trp = tile + (4 * g + (r16 >> 2)) * PB + (r16 & 3) * 8 + (L::kOwn ? 0 : half * CW * 32);
      constexpr int NX = kF32 ? 3 : 1;                            // terms of a value
      Frag<bf16_t> bx[NX][CW];
#pragma unroll
      for (int t = 0; t < NX; ++t)
#pragma unroll
      for (int w = 0; w < CW; ++w) {
        const unsigned char* tp = trp + t * (32 * PB) + w * 32;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)tp);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(tp + 16 * PB));
        const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
        bx[t][w].v = u32x4{l2[0], l2[1], h2[0], h2[1]};
      }
      if constexpr (kStats) {
        if (first) {
          if (st % kReseed == 0) flush_energy();
#pragma unroll
          for (int w = 0; w < CW; ++w) {
            mma_k32(acc[0][w], ones, bx[0][w]);
            mma_k32(acc[1][w], bx[0][w], bx[0][w]);
          }
          continue;                                             // (no kept dims here, and no barrier behind)
        }
      }
      if ((st - st0) % kReseed == 0) {
        seed(st);
        if constexpr (kEnergy && !kStats) {
          if (first) flush_energy();
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float c = bc[e] * cj - bs[e] * sj;
          bs[e] = bs[e] * cj + bc[e] * sj;
          bc[e] = c;
        }
      }
      Frag<bf16_t> ac[NT], as[NT];
      split_terms<NT>(bc, ac);
      split_terms<NT>(bs, as);
#pragma unroll
      for (int k = NX + NT - 2; k >= 0; --k)                      // (products of terms below 2^-24 of the first are left out)
#pragma unroll
        for (int t = 0; t < NX; ++t)
          if (k - t >= 0 && k - t < NT && k < 3)
#pragma unroll
            for (int w = 0; w < CW; ++w) {
              mma_k32(acc[0][w], ac[k - t], bx[t][w]);
              mma_k32(acc[1][w], as[k - t], bx[t][w]);
            }
      if constexpr (!kF32) {
        if (first) {
#pragma unroll
          for (int w = 0; w < CW; ++w) {
            mma_k32(acc0[N0 == 1 ? 0 : w], ones, bx[0][w]);
            if constexpr (kEnergy && !kStats) mma_k32(ene[w], bx[0][w], bx[0][w]);
          }
        }
      }
    }
    if constexpr (!kF32) if (write_keep && my_turn-- == 0 && v < N + lead) {
      my_turn = turns - 1;
      const int rows = min(32, (N + lead - v + 7) & ~7);
      const int kvec = keep_rows ? rows * kdiv : (rows >> 3) * kdiv;
      for (int it = wl; it < kvec; it += L::kOwn ? 64 : 64 * L::kHalves) {
        const int q = static_cast<int>((static_cast<uint32_t>(it) * kmagic) >> 21);
        const int c = it - q * kdiv;
        uint32_t w[4];
        if (keep_rows) {           // token q of the tile, kept dims 8 c ..
          const u32x4 kd = *reinterpret_cast<const u32x4*>(kdim + c * 8);
          const unsigned char* rp = tile + q * PB;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t lo = *reinterpret_cast<const uint16_t*>(rp + 2 * (kd[e] & 0xffffu));
            const uint32_t hi = *reinterpret_cast<const uint16_t*>(rp + 2 * (kd[e] >> 16));
            w[e] = lo | (hi << 16);
          }
          const int j = v + q - lead;
          if (j >= 0 && j < N)
            *reinterpret_cast<u32x4*>(keep + static_cast<int64_t>(p.keep_offset + j) * kp + c * 8) =
                u32x4{w[0], w[1], w[2], w[3]};
        } else {                   // tokens 8 q .. 8 q + 7 of the tile, kept dim c
          const unsigned char* rp = tile + q * 8 * PB + 2 * kdim[c];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t lo = *reinterpret_cast<const uint16_t*>(rp + (2 * e) * PB);
            const uint32_t hi = *reinterpret_cast<const uint16_t*>(rp + (2 * e + 1) * PB);
            w[e] = lo | (hi << 16);
          }
          const int j = v + q * 8 - lead;
          bf16_t* o = keep + (static_cast<int64_t>((p.keep_offset + j) >> 3) * Du + c) * 8;
          if (j >= 0 && j + 8 <= N) {
            *reinterpret_cast<u32x4*>(o) = u32x4{w[0], w[1], w[2], w[3]};
          } else {                 // a group shared with tokens outside this call
#pragma unroll
            for (int e = 0; e < 8; ++e)
              if (j + e >= 0 && j + e < N) o[e].bits = static_cast<uint16_t>(w[e >> 1] >> (16 * (e & 1)));
          }
        }
      }
    }
  }

  // ---- the shares of a tile meet in LDS: [wave][cos | sin][column tile][lane], then constants and energies per share
  __syncthreads();
  f32x4* red = reinterpret_cast<f32x4*>(smem);
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int w = 0; w < CW; ++w) red[((wave * 2 + q) * CW + w) * 64 + lane] = acc[q][w];
  float* cst = reinterpret_cast<float*>(smem + 8 * 2 * CW * 1024);
  float* dst = (p.part ? p.part + z * p.part_z + blockIdx.z * (z ? p.part_stride[1] : p.part_stride[0])
                       : z ? p.t[1].coeffs : p.t[0].coeffs) + static_cast<size_t>(bh) * p.M * Dc;
  if (first) {
    if constexpr (kEnergy) flush_energy();
    if constexpr (kF32) {                                       // (lanes of a column are NV apart)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float v = acc0[0][e];
        v += __shfl_xor(v, 16, 64);
        v += __shfl_xor(v, 32, 64);
        if (lane < 16) cst[share * D + half * 64 + 4 * ch + e] = v;
      }
    } else {
#pragma unroll
      for (int w = 0; w < CW; ++w) {
        const int col = (half * CW + w) * 16 + r16;
        if (g == 0) cst[share * D + col] = kStats ? acc[0][w][0] : acc0[N0 == 1 ? 0 : w][0];
      }
    }
  }
  __syncthreads();
  if (static_cast<int>(blockIdx.y) == stile / hw && tid < D) {
    double c0 = 0.0;
    for (int q = 0; q < shares; ++q) c0 += cst[q * D + tid];
    if constexpr (kEnergy) {
      double e = 0.0;
      for (int q = 0; q < shares; ++q) e += enr[q * D + tid];
      p.t[0].epart[static_cast<size_t>(bh) * D + tid] = static_cast<float>(e);
      // the constant's weighted square takes a row of its own behind the tiles'
      p.t[0].ecoef[(static_cast<size_t>((p.nmax + 15) / 16) * BH + bh) * D + tid] = static_cast<double>(basis_weight(0, p.T)) * c0 * c0;
    } else if (cidx[tid] >= 0) {
      float* C = dst + cidx[tid];
      C[0] = static_cast<float>(p.accumulate ? C[0] + c0 : c0);
    }
  }
  if (!live || (kStats && first)) return;
  if constexpr (kEnergy) {
    // weighted squares over the 16 harmonics of a tile: share `share` of the tile's waves takes every shares-th column tile
    for (int w = share; w < CW; w += shares) {
      double e = 0.0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int hn = htile * 16 + 1 + 4 * g + i;
        double cc = 0.0, cs = 0.0;
        for (int q = 0; q < shares; ++q) {
          const int wv = (q * hw + ht) * L::kHalves + half;
          cc += red[((wv * 2 + 0) * CW + w) * 64 + lane][i];
          cs += red[((wv * 2 + 1) * CW + w) * 64 + lane][i];
        }
        if (hn <= p.nmax) {
          const double wt = basis_weight(hn, p.T);
          e += wt * cc * cc;
          if (2 * hn < p.M) e += wt * cs * cs;
        }
      }
      e += __shfl_xor(e, 16, 64);
      e += __shfl_xor(e, 32, 64);
      if (g == 0 && htile * 16 < p.nmax)
        p.t[0].ecoef[(static_cast<size_t>(htile) * BH + bh) * D + (half * CW + w) * 16 + r16] = e;
    }
  } else {
    for (int w = share; w < CW; w += shares) {
      f32x4 sum[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        double d[4] = {0.0, 0.0, 0.0, 0.0};
        for (int q = 0; q < shares; ++q) {
          const f32x4 a = red[(((q * hw + ht) * L::kHalves + half) * 2 + k) * CW * 64 + w * 64 + lane];
#pragma unroll
          for (int i = 0; i < 4; ++i) d[i] += a[i];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) sum[k][i] = static_cast<float>(d[i]);
      }
      const int rank = cidx[(half * CW + w) * 16 + r16];
      if (rank >= 0) {
        float* C = dst + rank;
        const int m0 = 2 * (htile * 16 + 4 * g) + 1;               // cosine row of harmonic n = htile * 16 + 1 + 4 g
        float old[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) old[i] = 0.f;
        if (p.accumulate) {
#pragma unroll
          for (int i = 0; i < 8; ++i)
            if (m0 + i < p.M) old[i] = C[static_cast<size_t>(m0 + i) * Dc];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (m0 + i < p.M) C[static_cast<size_t>(m0 + i) * Dc] = old[i] + sum[i & 1][i >> 1];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// host
// ---------------------------------------------------------------------------
// Time: a step of 32 tokens per wave is bound by instruction issue (rotating and splitting the basis, 80 to 112 vector
// instructions, and 32 to 48 products, which two waves per SIMD hardly overlap; fp32 rows are split, too).  Measured, us a step:
// 0.75 / 0.95 / 1.4 (two terms; D = 64 / 128 / 256), 0.9 / 1.15 / 1.65 (three; with clamped addresses per row and step instead of a
// buffer descriptor a tenth more), 1.6 fp32; a round of workgroups, one per compute unit, takes 4 us and its states besides, a launch 5,
// the reduction of chunks another.  Many rows are bound by their bytes at 3 TB/s (rounds of workgroups in step), read once per workgroup of a pair where they exceed the caches
// (352 pairs x 5881 tokens, M = 50, two workgroups each: 253 us).  More tiles per workgroup mean fewer workgroups, each with a longer
// walk; more chunks the reverse.  longest: 32-token steps per fp32 sum; most: chunks there is room for; Du: kept dims.
RowsPlan make_rows_plan(const RowsShape& c, int terms, int longest, int most) {
  RowsPlan pl{};
  const bool f32 = c.dtype == FA_F32;
  if ((c.D != 64 && c.D != 128 && c.D != 256) || c.N <= 0) return pl;
  if (static_cast<long>(c.tensors) * c.B * c.H > 65535 || c.sx_n >= (f32 ? 1 << 24 : 1 << 25)) return pl;   // (32 rows within 4 GB)
  pl.lead = c.keep_offset & 7;
  const int slots = f32 ? 512 / c.D : c.D == 256 ? 4 : 8;
  const int64_t blocks = (static_cast<int64_t>(c.N) + pl.lead + 31) / 32;
  const int tiles = c.stats && rows_stats_tile(c.D) ? (c.M / 2 + 15) / 16 + 1 : expand_tiles(c.M);
  const double pairs = static_cast<double>(c.tensors) * c.B * c.H, es = f32 ? 4.0 : 2.0;
  const double step = f32 ? 1.6 : terms == 2 ? (c.D == 64 ? 0.75 : c.D == 128 ? 0.95 : 1.4) : (c.D == 64 ? 0.9 : c.D == 128 ? 1.15 : 1.65);
  const double x_bytes = pairs * c.N * es * c.D, keep_us = pairs * c.N * es * c.Du / 3.0e6;
  for (int hw = 1; hw <= slots; hw *= 2) {
    const int64_t steps = (blocks * hw + slots - 1) / slots;
    const int groups = (tiles + hw - 1) / hw;
    const double again = x_bytes > 256e6 ? 1.0 : x_bytes > 128e6 ? 0.6 : 0.0;
    const double mem = 8.0 + keep_us + x_bytes * (1.0 + again * (groups - 1)) / 3.0e6;
    const double alike = 1.0 + (f32 ? 0.2 : 0.5) * (hw - 1) / (slots > 1 ? slots - 1 : 1);   // (waves that ask for the same rows at once)
    const double fixed = 4.0 + hw * (c.D - c.Du) / 200.0;   // (the states a workgroup writes, too)
    for (int want = 1; want <= most; want = want < 4 ? want + 1 : want + want / 2) {
      const int64_t spc = (steps + want - 1) / want;
      const int chunks = static_cast<int>((steps + spc - 1) / spc);
      if (spc > longest) continue;
      const double work = 5.0 + ceil(pairs * groups * chunks / 256.0) * (fixed + spc * step * alike);
      const double us = (work > mem ? work : mem) + (chunks > 1 ? 6.0 + 2.0 * chunks * pairs * c.M * (c.D - c.Du) * 4.0 / 8.0e6 : 0.0);
      if (!pl.use || us < pl.us) {
        pl.use = true;
        pl.us = us;
        pl.hw = hw;
        pl.groups = groups;
        pl.steps = static_cast<int>(steps);
        pl.spc = static_cast<int>(spc);
        pl.chunks = chunks;
      }
    }
  }
  return pl;
}

template <typename T, int D, int NT, bool kEnergy>
static int launch_rows_t(const RowsParams& p, const RowsPlan& pl, int tensors, hipStream_t st, KernelTimers* tm) {
  using L = RowsTile<T, D>;
  auto kern = project_rows<T, D, NT, kEnergy>;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                          static_cast<int>(L::kLds)) != hipSuccess)
    return FA_ERR_HIP;
  FA_LAUNCH_TIMED(tm, 0, kern, dim3(tensors * p.B * p.H, pl.groups, pl.chunks), dim3(512), L::kLds, st, p);
  return FA_OK;
}

int launch_rows(const RowsParams& p, const RowsPlan& pl, int dtype, int D, int tensors, int terms, hipStream_t st, KernelTimers* tm) {
#define FA_ROWS(T_, NT_, E_)                                                                                              \
  return D == 64 ? launch_rows_t<T_, 64, NT_, E_>(p, pl, tensors, st, tm)                                                 \
       : D == 128 ? launch_rows_t<T_, 128, NT_, E_>(p, pl, tensors, st, tm) : launch_rows_t<T_, 256, NT_, E_>(p, pl, tensors, st, tm)
  if (dtype == FA_F32) FA_ROWS(float, 3, false);
  if (p.t[0].ecoef) FA_ROWS(bf16_t, 3, true);
  if (terms == 3) FA_ROWS(bf16_t, 3, false);
  FA_ROWS(bf16_t, 2, false);
#undef FA_ROWS
}

}  // namespace fa
