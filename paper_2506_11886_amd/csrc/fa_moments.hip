// Long-segment projection through local Chebyshev moments: see fa_moments.hpp for the expansion.
//
//   fa_moments : one streaming pass over X.  Rows go registers -> an LDS tile and come back
//                transposed (ds_read_b64_tr_b16) as the B operand of v_mfma_f32_16x16x32_bf16 against
//                the Chebyshev table (A operand, 2 or 3 bf16 terms); the kept dims of the same tile
//                leave as 128-bit vectors.
//   fa_expand16: coefficients from the moments, a product of split bf16 terms (fa_compress)
//   fa_expand  : the same in fp32 for fa_select_dims: 16 harmonics x 16 columns per wave, four
//                v_mfma_f32_16x16x4_f32 per block (even and odd polynomials apart), then one
//                rotation by the block centre's exact phase.

#include "fa_moments.hpp"

#include <math.h>

#include "fa_mma.hpp"

namespace fa {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// a[p] = (2 - [p = 0]) i^p J_p(theta) without the i of odd p (even p belong to the cosine, odd p to the
// sine of the block centre).  Miller's backward recurrence J_{p-1} = (2p / theta) J_p - J_{p+1} from
// p = 34, normalised by J_0 + 2 sum J_{2k} = 1; below theta = 0.05, where 2 / theta grows without bound, the
// leading terms of the power series (relative error 1e-11).
__device__ __forceinline__ void bessel_coeffs(double theta, float (&a)[kMomP]) {
  double j[kMomP];
  const bool tiny = theta < 0.05;
  {
    const double inv = 2.0 / (tiny ? 0.05 : theta);
    double jp1 = 0.0, jp = 1e-30, norm = 0.0;
#pragma unroll
    for (int q = 34; q > 0; --q) {      // jp = J_q on entry
      const double jm = inv * q * jp - jp1;
      jp1 = jp;
      jp = jm;
      if (q - 1 < kMomP) j[q - 1] = jp;
      if (((q - 1) & 1) == 0) norm += (q == 1 ? 1.0 : 2.0) * jp;
    }
    const double sc = 1.0 / norm;
#pragma unroll
    for (int q = 0; q < kMomP; ++q) j[q] *= sc;
  }
  if (__any(tiny)) {
    const double hx = 0.5 * theta, y = hx * hx;
    double t = 1.0;                    // (theta/2)^p / p!
#pragma unroll
    for (int q = 0; q < kMomP; ++q) {
      const double v = t * (1.0 - y * (1.0 / (q + 1)) + y * y * (0.5 / ((q + 1) * (q + 2))));
      if (tiny) j[q] = v;
      t *= hx * (1.0 / (q + 1));
    }
  }
#pragma unroll
  for (int q = 0; q < kMomP; ++q) a[q] = static_cast<float>((q == 0 ? 1.0 : ((q >> 1) & 1) ? -2.0 : 2.0) * j[q]);
}

template <int D>
struct MomTile {
  static constexpr int kTokens = D == 256 ? 64 : 128;              // tokens of a tile
  static constexpr int kWaves = D == 64 ? 4 : 8;
  static constexpr int kColTiles = D / 16 / kWaves;                // 16-column tiles per wave
  static constexpr int kPitch = 2 * D + 32;                        // bytes of a tile row
  static constexpr int kLoads = kTokens * (D / 8) / (64 * kWaves); // 128-bit vectors per thread and tile
};

// A operand of fa_expand16 for one 16-harmonic tile and two blocks: 4 x 1 KB in lane order (cosine
// rows head / remainder, sine rows head / remainder).  Lane (r16, g): harmonic r16 of the tile, block
// g >> 1, polynomials 8 (g & 1) ..; the block's rotation is multiplied in, so that nothing is left to
// do per block outside the matrix cores.  Formed once per call (it does not depend on the head).
__device__ void form_expand_operand(const MomentParams& p, int item, int nstep) {
  const int lane = threadIdx.x & 63, g = lane >> 4, r16 = lane & 15;
  const int tile = item / nstep, st = item - tile * nstep;
  const int n = tile * kExpandRows + 1 + r16;
  float a[kMomP];
  bessel_coeffs(3.14159265358979323846 * n * p.U / p.T, a);
  const int blk = 2 * st + (g >> 1);
  // 2^-32-turn phase of the block's centre, rounded to nearest: half a unit times n <= 512 is 6e-8 turns, without a bias
  const double c2 = static_cast<double>(2ll * (p.t0 - p.lead) + p.U - 1) + 2.0 * p.U * blk;
  const uint32_t ph = static_cast<uint32_t>(static_cast<uint64_t>(c2 * (2147483648.0 / p.T) + 0.5));
  const float x = static_cast<float>(static_cast<int32_t>(ph * static_cast<uint32_t>(n))) * 2.3283064365386963e-10f;
  float sn = __builtin_amdgcn_sinf(x), c = __builtin_amdgcn_cosf(x);
  if (blk >= p.blocks) sn = c = 0.0f;
  bf16x8 ch, cl, sh, sl;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float lo = a[e], hi = a[8 + e], ae = (g & 1) ? hi : lo;
    const float vc = (e & 1) ? -sn * ae : c * ae;
    const float vs = (e & 1) ? c * ae : sn * ae;
    ch[e] = static_cast<__bf16>(vc);
    cl[e] = static_cast<__bf16>(vc - static_cast<float>(ch[e]));
    sh[e] = static_cast<__bf16>(vs);
    sl[e] = static_cast<__bf16>(vs - static_cast<float>(sh[e]));
  }
  bf16x8* o = reinterpret_cast<bf16x8*>(p.op) + static_cast<size_t>(item) * 256 + lane;
  o[0] = ch; o[64] = cl; o[128] = sh; o[192] = sl;
}

// Sums of squares: fp32 over this many tiles per thread (32 squares at most), fp64 from there on.  The error of a
// dim is the difference of its energy and of what the states hold, so a sum over a workgroup's whole share (all tokens of a
// pair when there are many pairs) in fp32 would decide the order of well-compressed dims: 6e-5 of the energy of a
// constant dim at 131072 tokens.
constexpr int kEnergyTiles = 8;

// D: head dim; NT: bf16 terms of a table value; kEnergy: also per-dim sums of squares (fa_select_dims).
// grid (chunks, tensors * B * H).  LDS: table [S][NT][64 lanes][8] | two tiles.
// Bound: HBM.  Three tiles of a workgroup are in flight in registers; a tile goes to LDS, one barrier
// later every wave multiplies its own 16-column tiles of it (so a block's sums are complete in one
// wave's registers and leave from there) and all waves pack the kept dims.  A row pitch of 2 D + 32
// bytes puts the 8 rows x 32 bytes that half a wave reads transposed on distinct banks; the table is
// stored in lane order.
// At most 256 registers (two waves per SIMD), also where a workgroup has four waves only: with more the
// compiler keeps acc in accumulation registers, and at D = 64 with three terms it read them back one to
// five instructions behind the last product of a tile, across a branch, where the hardware needs eight
// (sums of blocks longer than a tile then lacked the smaller terms' products: selection errors of 1e-3).
template <int D, int NT, bool kEnergy>
__global__ __launch_bounds__(64 * MomTile<D>::kWaves, 2) void fa_moments(MomentParams p) {
  using L = MomTile<D>;
  constexpr int NV = D / 8, PB = L::kPitch, NTH = 64 * L::kWaves, TT = L::kTokens, NL = L::kLoads;
  constexpr int RPL = NTH / NV, CW = L::kColTiles, NST = TT / 32;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ __attribute__((aligned(16))) uint16_t kdim[D + 8];
  __shared__ int16_t cidx[D];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, r16 = lane & 15;
  const int BH = p.B * p.H;
  const int z = blockIdx.y >= BH;
  const int bh = blockIdx.y - (z ? BH : 0), b = bh / p.H, h = bh - b * p.H;
  const uint8_t* mask = z ? p.t[1].mask : p.t[0].mask;
  const int Dc = z ? p.t[1].Dc : p.t[0].Dc, Du = D - Dc;
  const bf16_t* xb = static_cast<const bf16_t*>(z ? p.t[1].x : p.t[0].x) + b * p.sx_b + h * p.sx_h;
  const int S = p.S, U = p.U, N = p.N, lead = p.lead;
  const int blk0 = blockIdx.x * p.bpc, nblk = min(p.bpc, p.blocks - blk0);
  const int ntok = nblk * U;                        // tokens of this workgroup, a multiple of 32
  const int vbase = blk0 * U;                       // first (virtual) token: token j is virtual j + lead
  const int ntile = (ntok + TT - 1) / TT;
  const int jlast = min(N, vbase + ntok - lead) - 1; // requests past the workgroup's tokens repeat its last row

  unsigned char* table = smem;
  unsigned char* tiles = smem + S * NT * 1024;

  const int ch = tid % NV, row0 = tid / NV;
  auto load = [&](u32x4 (&x)[NL], int t) {
    const int v = vbase + t * TT - lead + row0;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int j = min(max(v + i * RPL, 0), jlast);
      x[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(xb + (static_cast<int64_t>(j) * p.sx_n + ch * 8)));
    }
  };
  // (the mask is requested before the rows: answers arrive in order)
  uint8_t mb[D / 64];
#pragma unroll
  for (int j = 0; j < D / 64; ++j) mb[j] = mask ? mask[static_cast<size_t>(bh) * D + lane + 64 * j] : uint8_t{1};
  u32x4 xa[NL], xc[NL], xd[NL];
  load(xa, 0);
  load(xc, 1);
  load(xd, 2);

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
      if (!hit) kdim[tid - nc] = static_cast<uint16_t>(tid);
    }
    if (tid < 8) kdim[Du + tid] = D;
  }
  if (tid < 2 * TT) *reinterpret_cast<u32x4*>(tiles + tid * PB + 2 * D) = u32x4{0u, 0u, 0u, 0u};

  // ---- Chebyshev table: all T_p of one token by the three-term recurrence in fp64, split into bf16
  // terms.  Slot e of lane group q holds token 4 q + e (e < 4) or 16 + 4 q + e - 4 of its step.
  for (int u = tid; u < U; u += NTH) {
    const double x = static_cast<double>(2 * u + 1 - U) / static_cast<double>(U);
    const int s = u >> 5, t = u & 31;
    unsigned char* dst = table + s * NT * 1024 + ((t & 15) >> 2) * 256 + ((t & 3) + ((t >> 4) << 2)) * 2;
    double a = 1.0, c = x;
#pragma unroll
    for (int q = 0; q < kMomP; ++q) {
      double rem = a;
#pragma unroll
      for (int k = 0; k < NT; ++k) {
        const __bf16 hb = static_cast<__bf16>(static_cast<float>(rem));
        *reinterpret_cast<__bf16*>(dst + k * 1024 + q * 16) = hb;
        if (k + 1 < NT) rem -= static_cast<double>(static_cast<float>(hb));
      }
      const double nx = 2.0 * x * c - a;
      a = c;
      c = nx;
    }
  }
  // operands of fa_expand16: the last waves first, they have least of the table to build
  if constexpr (NT == 2) {
    const int nstep = (p.blocks + 1) / 2, items = nstep * p.tiles, wgs = gridDim.x * gridDim.y;
    for (int it = (L::kWaves - 1 - wave) * wgs + blockIdx.y * gridDim.x + blockIdx.x; it < items; it += wgs * L::kWaves)
      form_expand_operand(p, it, nstep);
  }
  __syncthreads();

  const bool keep_rows = (z ? p.t[1].keep_layout : p.t[0].keep_layout) == FA_KEEP_ROWS;
  bf16_t* keep = static_cast<bf16_t*>(z ? p.t[1].keep : p.t[0].keep);
  const bool write_keep = keep != nullptr && Du > 0;
  const int kp = z ? p.t[1].keep_pitch : p.t[0].keep_pitch;
  if (write_keep) keep += static_cast<int64_t>(bh) * (z ? p.t[1].keep_stride : p.t[0].keep_stride);
  const int kdiv = max(1, keep_rows ? kp >> 3 : Du);               // kept vectors per token / per 8-token group
  const uint32_t kmagic = ((1u << 21) + kdiv - 1) / kdiv;         // it / kdiv exactly: it * kdiv < 2^21
  int cpos[CW];                                                    // compressed rank of this lane's columns
#pragma unroll
  for (int w = 0; w < CW; ++w) cpos[w] = cidx[(wave * CW + w) * 16 + r16];

  f32x4 acc[CW];
#pragma unroll
  for (int i = 0; i < CW; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float e2[8];                                                     // at most kEnergyTiles * NL squares each, then
  double energy[8];                                                // added up here
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    e2[i] = 0.f;
    energy[i] = 0.0;
  }
  float* const mom_t = z ? p.t[1].mom : p.t[0].mom;
  const size_t mblk = static_cast<size_t>(bh) * p.blocks + blk0;
  float* mom = mom_t + mblk * (kMomP * Dc);
  int s = 0;                                                       // step inside the current block

  auto one_tile = [&](u32x4 (&x)[NL], int t) {
    const int v = vbase + t * TT;
    unsigned char* tile = tiles + (t & 1) * (TT * PB);
    if (v < lead || v + TT > N + lead) {
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int j = v + row0 + i * RPL - lead;
        if (j < 0 || j >= N) x[i] = u32x4{0u, 0u, 0u, 0u};
      }
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) *reinterpret_cast<u32x4*>(tile + (row0 + i * RPL) * PB + ch * 16) = x[i];
    if constexpr (kEnergy) {
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const bool mine = t * TT + row0 + i * RPL < ntok;          // the tile may reach into the next workgroup's tokens
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float lo = mine ? __builtin_bit_cast(float, x[i][e] << 16) : 0.0f;
          const float hi = mine ? __builtin_bit_cast(float, x[i][e] & 0xffff0000u) : 0.0f;
          e2[2 * e] += lo * lo;
          e2[2 * e + 1] += hi * hi;
        }
      }
      if ((t + 1) % kEnergyTiles == 0 || t + 1 == ntile) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          energy[e] += e2[e];
          e2[e] = 0.f;
        }
      }
    }
    load(x, t + 3);
    lds_barrier();
    const unsigned char* trp = tile + (4 * g + (r16 >> 2)) * PB + (r16 & 3) * 8 + wave * CW * 32;
#pragma unroll
    for (int st = 0; st < NST; ++st) {
      if (t * TT + st * 32 < ntok) {
        Frag<bf16_t> a[NT];
#pragma unroll
        for (int k = 0; k < NT; ++k)
          a[k].v = *reinterpret_cast<const u32x4*>(table + (s * NT + k) * 1024 + lane * 16);
#pragma unroll
        for (int w = 0; w < CW; ++w) {
          const unsigned char* tp = trp + st * 32 * PB + w * 32;
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)tp);
          const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(tp + 16 * PB));
          const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
          Frag<bf16_t> bx;
          bx.v = u32x4{l2[0], l2[1], h2[0], h2[1]};
#pragma unroll
          for (int k = 0; k < NT; ++k) mma_k32(acc[w], a[k], bx);
        }
        if (++s == S) {               // the block is complete: [Dc][16] moments
          s = 0;
#pragma unroll
          for (int w = 0; w < CW; ++w) {
            const int c = cpos[w];
            if (c >= 0) *reinterpret_cast<f32x4*>(mom + c * kMomP + g * 4) = acc[w];
            acc[w] = f32x4{0.f, 0.f, 0.f, 0.f};
          }
          mom += kMomP * Dc;
        }
      }
    }
    if (write_keep) {
      const int rows = min(TT, ntok - t * TT);                     // a multiple of 32
      const int kvec = keep_rows ? rows * kdiv : (rows >> 3) * kdiv;
      for (int it = tid; it < kvec; it += NTH) {
        const int q = static_cast<int>((static_cast<uint32_t>(it) * kmagic) >> 21);
        const int c = it - q * kdiv;
        uint32_t w[4];
        if (keep_rows) {           // token q of the tile, kept dims 8 c ..
          const u32x4 kd = *reinterpret_cast<const u32x4*>(kdim + c * 8);
          const unsigned char* r = tile + q * PB;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t lo = *reinterpret_cast<const uint16_t*>(r + 2 * (kd[e] & 0xffffu));
            const uint32_t hi = *reinterpret_cast<const uint16_t*>(r + 2 * (kd[e] >> 16));
            w[e] = lo | (hi << 16);
          }
          const int j = v + q - lead;
          if (j >= 0 && j < N)
            *reinterpret_cast<u32x4*>(keep + static_cast<int64_t>(p.keep_offset + j) * kp + c * 8) =
                u32x4{w[0], w[1], w[2], w[3]};
        } else {                   // tokens 8 q .. 8 q + 7 of the tile, kept dim c
          const unsigned char* r = tile + q * 8 * PB + 2 * kdim[c];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t lo = *reinterpret_cast<const uint16_t*>(r + (2 * e) * PB);
            const uint32_t hi = *reinterpret_cast<const uint16_t*>(r + (2 * e + 1) * PB);
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
  };
  for (int t = 0; t < ntile; t += 3) {
    one_tile(xa, t);
    if (t + 1 >= ntile) break;
    one_tile(xc, t + 1);
    if (t + 2 >= ntile) break;
    one_tile(xd, t + 2);
  }
  if constexpr (kEnergy) {
    double* red = reinterpret_cast<double*>(tiles);                // [rows of a vector pass][D]
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 8; ++e) red[row0 * D + ch * 8 + e] = energy[e];
    __syncthreads();
    if (tid < D) {
      double v = 0.0;
      for (int r = 0; r < RPL; ++r) v += red[r * D + tid];
      p.t[0].epart[(static_cast<size_t>(blockIdx.x) * BH + bh) * D + tid] = static_cast<float>(v);
    }
  }
}

// grid (16-harmonic tiles, column groups, tensors * B * H), ctw * ks waves: wave (column tile, share of
// the blocks).  The block centres' phases (exact: the product is formed in fp64) are shared through
// LDS, kPhBlocks blocks at a time.  Bound: the fp32 matrix rate on long segments, latency else.
constexpr int kPhBlocks = 128;
constexpr int kExpandBatch = 4;
constexpr int kExpandRun = 4;
constexpr int kExpandWaves = 12;
__global__ __launch_bounds__(64 * kExpandWaves) void fa_expand(MomentParams p, int ctw, int ks) {
  __shared__ __attribute__((aligned(16))) float2 ph[kPhBlocks][kExpandRows];
  __shared__ float red[9 * 64 * 9];                             // (ks - 1) * ctw <= 9 waves hand their sums over
  const int tid = threadIdx.x, lane = tid & 63, nt = blockDim.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, r16 = lane & 15;
  const int BH = p.B * p.H;
  const int z = blockIdx.z >= BH;
  const int bh = blockIdx.z - (z ? BH : 0);
  const int Dc = z ? p.t[1].Dc : p.t[0].Dc;
  const int tile = blockIdx.x, n0 = tile * kExpandRows + 1;      // first harmonic of the tile
  const int ctl = wave % ctw, part = wave / ctw;
  const int col = (blockIdx.y * ctw + ctl) * 16 + r16;
  const bool live = (blockIdx.y * ctw + ctl) * 16 < Dc;          // (wave-uniform)
  const float* mom = (z ? p.t[1].mom : p.t[0].mom) + static_cast<size_t>(bh) * p.blocks * kMomP * Dc + min(col, Dc - 1) * kMomP + 2 * g;
  const int nblk = p.blocks;

  float bm[kExpandBatch][4];
  auto load = [&](int b0) {
#pragma unroll
    for (int i = 0; i < kExpandBatch; ++i) {
      const float* m = mom + static_cast<size_t>(min(b0 + i * ks, nblk - 1)) * (kMomP * Dc);
      const float2 lo = *reinterpret_cast<const float2*>(m), hi = *reinterpret_cast<const float2*>(m + 8);
      bm[i][0] = lo.x; bm[i][1] = hi.x;
      bm[i][2] = lo.y; bm[i][3] = hi.y;
    }
  };
  load(part);
  const double theta = 3.14159265358979323846 * (n0 + r16) * p.U / p.T;
  float aE1, aE2, aO1, aO2;           // polynomials 2 g, 2 g + 8 / 2 g + 1, 2 g + 9
  {
    float a[kMomP];
    bessel_coeffs(theta, a);
    auto pick = [&](int o) { return g == 0 ? a[o] : g == 1 ? a[o + 2] : g == 2 ? a[o + 4] : a[o + 6]; };
    aE1 = pick(0); aE2 = pick(8); aO1 = pick(1); aO2 = pick(9);
  }

  // kExpandRun batches are summed in fp32, those sums in fp64: an out-of-band dim's blocks are individually
  // large and cancel, and the error of a dim is a small difference of sums
  double cc[4] = {0.0, 0.0, 0.0, 0.0}, cs[4] = {0.0, 0.0, 0.0, 0.0}, c0 = 0.0;
  float bc[4] = {0.f, 0.f, 0.f, 0.f}, bs[4] = {0.f, 0.f, 0.f, 0.f}, b00 = 0.f;
  int run = 0;
  const double inv2t = 0.5 / p.T;
  for (int seg = 0; seg < nblk; seg += kPhBlocks) {
    const int nseg = min(kPhBlocks, nblk - seg);
    if (seg > 0) __syncthreads();
    for (int it = tid; it < nseg * kExpandRows; it += nt) {
      const int bb = it / kExpandRows, n = n0 + it % kExpandRows;
      // twice the centre of block seg + bb, counted from the period's origin
      const int64_t c2 = 2ll * (p.t0 - p.lead) + 2ll * (seg + bb) * p.U + p.U - 1;
      double f = static_cast<double>(c2 * n) * inv2t;
      f -= floor(f);
      float sn, c;
      sincospif(2.0f * static_cast<float>(f), &sn, &c);
      ph[bb][it % kExpandRows] = float2{c, sn};
    }
    __syncthreads();
    if (live) {
      for (int b0 = part; b0 < nseg; b0 += ks * kExpandBatch) {
        float cur[kExpandBatch][4];
#pragma unroll
        for (int i = 0; i < kExpandBatch; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) cur[i][e] = b0 + i * ks < nseg ? bm[i][e] : 0.0f;
        const int nb = b0 + ks * kExpandBatch;
        load(nb < nseg ? seg + nb : seg + kPhBlocks + part);
#pragma unroll
        for (int i = 0; i < kExpandBatch; ++i) {
          f32x4 E = f32x4{0.f, 0.f, 0.f, 0.f}, O = f32x4{0.f, 0.f, 0.f, 0.f};
          E = __builtin_amdgcn_mfma_f32_16x16x4f32(aE1, cur[i][0], E, 0, 0, 0);
          O = __builtin_amdgcn_mfma_f32_16x16x4f32(aO1, cur[i][2], O, 0, 0, 0);
          E = __builtin_amdgcn_mfma_f32_16x16x4f32(aE2, cur[i][1], E, 0, 0, 0);
          O = __builtin_amdgcn_mfma_f32_16x16x4f32(aO2, cur[i][3], O, 0, 0, 0);
          const f32x4* pp = reinterpret_cast<const f32x4*>(&ph[min(b0 + i * ks, nseg - 1)][4 * g]);
          const f32x4 pa = pp[0], pb = pp[1];
          const float c[4] = {pa[0], pa[2], pb[0], pb[2]}, sn[4] = {pa[1], pa[3], pb[1], pb[3]};
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            bc[r] += c[r] * E[r] - sn[r] * O[r];
            bs[r] += sn[r] * E[r] + c[r] * O[r];
          }
          b00 += cur[i][0];    // lane group 0: moment 0, the constant function
        }
        if (++run == kExpandRun || nb >= nseg) {
          run = 0;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            cc[r] += bc[r];
            cs[r] += bs[r];
            bc[r] = bs[r] = 0.f;
          }
          c0 += b00;
          b00 = 0.f;
        }
      }
    }
  }
  // ---- shares of the blocks meet in a fixed order
  if (ks > 1) {
    if (part > 0 && live) {
      float* r = red + ((part - 1) * ctw + ctl) * (64 * 9) + lane;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        r[64 * i] = static_cast<float>(cc[i]);
        r[64 * (4 + i)] = static_cast<float>(cs[i]);
      }
      r[64 * 8] = static_cast<float>(c0);
    }
    __syncthreads();
    if (part == 0 && live)
      for (int q = 1; q < ks; ++q) {
        const float* r = red + ((q - 1) * ctw + ctl) * (64 * 9) + lane;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          cc[i] += r[64 * i];
          cs[i] += r[64 * (4 + i)];
        }
        c0 += r[64 * 8];
      }
  }
  if (part > 0 || !live) return;
  double* ecoef = z ? p.t[1].ecoef : p.t[0].ecoef;
  double e = 0.0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int n = n0 + 4 * g + i;
    if (n <= p.nmax) {
      const double w = basis_weight(n, p.T);
      e += w * cc[i] * cc[i];
      if (2 * n < p.M) e += w * cs[i] * cs[i];
    }
  }
  if (tile == 0 && g == 0) e += static_cast<double>(basis_weight(0, p.T)) * c0 * c0;
  e += __shfl_xor(e, 16, 64);
  e += __shfl_xor(e, 32, 64);
  if (g == 0 && col < Dc) ecoef[(static_cast<size_t>(tile) * BH + bh) * Dc + col] = e;
}

// The same contraction for fa_compress on the bf16 matrix rate: a plain product
// A[(n, cos | sin), (block, p)] x mu[(block, p), column].  A is formed by fa_moments as head + remainder, the fp32
// moments are split here into three terms: four products a value, 2^-17 relative (A's own rounding).  The split, 44 vector
// instructions, is the longest part of a step.  HT 16-harmonic tiles per workgroup share it: two where one would take more
// workgroups than there are compute units (K and V of 128 x 8 K, head dim 256, M = 256: 710 -> 598 us the call; head dim 64: 180
// -> 149), else one (8 x 4 K, head dim 128, M = 64: 16.6 us against 19.4).
// grid (tensors * B * H, column groups, groups of harmonic tiles): the workgroups of one head
// are eight apart and share an XCD's L2 when the heads are a multiple of eight.  ctw * ks waves: wave
// (column tile, share of the 2-block steps).  A batch is kExpSteps / HT steps per wave; its A operands are
// shared through LDS.  Bound: latency of the moments, which other XCDs wrote (two batches in flight).
constexpr int kExpSteps = 4;
// NOPS: A operands (one tile and 2-block step each) a wave copies per batch
template <int kSteps, int NOPS>
struct ExpBatch {
  f32x4 m[kSteps][2];
  u32x4 a[NOPS][4];
};
// Eight moments as three bf16 terms, which hold all their bits; pairs are rounded by one instruction.
__device__ __forceinline__ void split3(const f32x4 (&m)[2], Frag<bf16_t> (&t)[3]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    f32x2 r = f32x2{m[e >> 1][2 * (e & 1)], m[e >> 1][2 * (e & 1) + 1]};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, bf16x2));
      t[k].v[e] = w;
      r[0] -= __builtin_bit_cast(float, w << 16);
      r[1] -= __builtin_bit_cast(float, w & 0xffff0000u);
    }
  }
}
template <int HT, int NOPS>
__global__ __launch_bounds__(512) void fa_expand16(MomentParams p, int ctw, int ks) {
  constexpr int kSteps = kExpSteps / HT;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, r16 = lane & 15;
  const int ctl = wave % ctw, part = wave / ctw, nw = ctw * ks, batch = ks * kSteps;
  const int BH = p.B * p.H;
  const int z = blockIdx.x >= BH;
  const int bh = blockIdx.x - (z ? BH : 0);
  const int Dc = z ? p.t[1].Dc : p.t[0].Dc;
  const int tile0 = blockIdx.z * HT;
  const int col = (blockIdx.y * ctw + ctl) * 16 + r16;
  const int nblk = p.blocks, nstep = (nblk + 1) / 2;
  const uint32_t bstride = kMomP * Dc;
  const float* mom = (z ? p.t[1].mom : p.t[0].mom) + static_cast<size_t>(bh) * nblk * bstride +
                     min(col, Dc - 1) * kMomP + (g & 1) * 8;
  const u32x4* op = reinterpret_cast<const u32x4*>(p.op) + lane;
  const bool with_dc = tile0 == 0;

  // operand u of a batch: tile u % HT (past the last: the last, its sums are dropped), step u / HT
  auto load = [&](ExpBatch<kSteps, NOPS>& x, int st0) {
#pragma unroll
    for (int i = 0; i < NOPS; ++i) {
      const int u = min(wave + i * nw, batch * HT - 1);
      const size_t st = static_cast<size_t>(min(tile0 + u % HT, p.tiles - 1)) * nstep + min(st0 + u / HT, nstep - 1);
#pragma unroll
      for (int k = 0; k < 4; ++k) x.a[i][k] = op[st * 256 + k * 64];
    }
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
      const uint32_t blk = min(2 * (st0 + i * ks + part) + (g >> 1), nblk - 1);
      const f32x4* m = reinterpret_cast<const f32x4*>(mom + static_cast<size_t>(blk) * bstride);
      x.m[i][0] = m[0];
      x.m[i][1] = m[1];
    }
  };
  ExpBatch<kSteps, NOPS> xa, xb;
  load(xa, 0);
  load(xb, batch);

  // a batch (2 kSteps blocks per wave) is summed in fp32, the batches in fp64: the blocks of a slow out-of-band
  // tone are individually large and cancel
  double sc[HT][4], ss[HT][4], s0 = 0.0;
#pragma unroll
  for (int q = 0; q < HT; ++q)
#pragma unroll
    for (int i = 0; i < 4; ++i) sc[q][i] = ss[q][i] = 0.0;
  auto one_batch = [&](ExpBatch<kSteps, NOPS>& x, int st0, int buf) {
    unsigned char* base = smem + buf * (batch * HT * 4096);
#pragma unroll
    for (int i = 0; i < NOPS; ++i) {
      if (wave + i * nw < batch * HT) {
        u32x4* o = reinterpret_cast<u32x4*>(base + (wave + i * nw) * 4096) + lane;
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k * 64] = x.a[i][k];
      }
    }
    lds_barrier();
    f32x4 cc[HT], cs[HT], cc1[HT], cs1[HT];   // (1: the remainders' products)
#pragma unroll
    for (int q = 0; q < HT; ++q) cc[q] = cs[q] = cc1[q] = cs1[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    float c0 = 0.0f;
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
      const int si = i * ks + part;
      if (st0 + si < nstep) {
        Frag<bf16_t> f[HT][4], t[3];
#pragma unroll
        for (int q = 0; q < HT; ++q) {
          const u32x4* o = reinterpret_cast<const u32x4*>(base + (si * HT + q) * 4096) + lane;
#pragma unroll
          for (int k = 0; k < 4; ++k) f[q][k].v = o[k * 64];
        }
        split3(x.m[i], t);
#pragma unroll
        for (int q = 0; q < HT; ++q) {
          mma_k32(cc[q], f[q][0], t[0]);
          mma_k32(cs[q], f[q][2], t[0]);
          mma_k32(cc1[q], f[q][1], t[0]);
          mma_k32(cs1[q], f[q][3], t[0]);
        }
#pragma unroll
        for (int k = 1; k < 3; ++k)
#pragma unroll
          for (int q = 0; q < HT; ++q) {
            mma_k32(cc1[q], f[q][0], t[k]);
            mma_k32(cs1[q], f[q][2], t[k]);
          }
        if (2 * (st0 + si) + (g >> 1) < nblk) c0 += x.m[i][0][0];   // (even g: moment 0)
      }
    }
    load(x, st0 + 2 * batch);
#pragma unroll
    for (int q = 0; q < HT; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        sc[q][i] += cc[q][i] + cc1[q][i];
        ss[q][i] += cs[q][i] + cs1[q][i];
      }
    s0 += c0;
  };
  for (int st0 = 0; st0 < nstep; st0 += 2 * batch) {
    one_batch(xa, st0, 0);
    if (st0 + batch >= nstep) break;
    one_batch(xb, st0 + batch, 1);
  }
  s0 += __shfl_xor(s0, 32, 64);        // even and odd blocks
  if (ks > 1) {                        // the shares meet in a fixed order
    __syncthreads();
    double* red = reinterpret_cast<double*>(smem);
    if (part > 0) {
      double* r = red + ((part - 1) * ctw + ctl) * ((8 * HT + 1) * 64) + lane;
#pragma unroll
      for (int q = 0; q < HT; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          r[64 * (8 * q + i)] = sc[q][i];
          r[64 * (8 * q + 4 + i)] = ss[q][i];
        }
      r[64 * ((8 * HT + 1) - 1)] = s0;
    }
    __syncthreads();
    if (part > 0) return;
    for (int w = 1; w < ks; ++w) {
      const double* r = red + ((w - 1) * ctw + ctl) * ((8 * HT + 1) * 64) + lane;
#pragma unroll
      for (int q = 0; q < HT; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          sc[q][i] += r[64 * (8 * q + i)];
          ss[q][i] += r[64 * (8 * q + 4 + i)];
        }
      s0 += r[64 * ((8 * HT + 1) - 1)];
    }
  }
  if (col >= Dc) return;
  float* C = (z ? p.t[1].coeffs : p.t[0].coeffs) + static_cast<size_t>(bh) * p.M * Dc + col;
  // the old state is read as a whole before any of it is written (row by row, each would wait for memory: a 2 K piece in two
  // calls 28.4 us against 27.1), and the sum rounded once behind it
  float old[HT][8], old0 = 0.f;
#pragma unroll
  for (int q = 0; q < HT; ++q)
#pragma unroll
    for (int i = 0; i < 8; ++i) old[q][i] = 0.f;
  if (p.accumulate) {
#pragma unroll
    for (int q = 0; q < HT; ++q)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int m = 2 * ((tile0 + q) * kExpandRows + 4 * g) + 1 + i;
        if (m < p.M) old[q][i] = C[static_cast<size_t>(m) * Dc];
      }
    if (with_dc) old0 = C[0];
  }
  if (with_dc && g == 0) C[0] = static_cast<float>(old0 + s0);
#pragma unroll
  for (int q = 0; q < HT; ++q)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      // harmonic n = 1 + 16 tile + 4 g + i / 2: row 2 n - 1 its cosine, row 2 n its sine
      const int m = 2 * ((tile0 + q) * kExpandRows + 4 * g) + 1 + i;
      const double v = (i & 1) ? ss[q][i >> 1] : sc[q][i >> 1];
      if (m < p.M) C[static_cast<size_t>(m) * Dc] = static_cast<float>(old[q][i] + v);
    }
}

// ---------------------------------------------------------------------------
// host
// ---------------------------------------------------------------------------
static int moment_max_u(int M, int T, bool exact) {
  const int nmax = M / 2;
  const int cap = exact ? 512 : kMomMaxU;
  if (nmax == 0) return cap;
  const double u = (exact ? kThetaF32 : kThetaBf16) * T / (3.14159265358979323846 * nmax);
  return u >= cap ? cap : static_cast<int>(u) / 32 * 32;
}

MomentPlan make_moment_plan(int dtype, int B, int H, int N, int D, int Dc, int M, int T, int keep_offset,
                            int tensors, bool exact) {
  MomentPlan pl{};
  if (dtype != FA_BF16 || (D != 64 && D != 128 && D != 256) || Dc <= 0 || N <= 0) return pl;
  if (static_cast<long>(tensors) * B * H > 65535) return pl;
  const int umax = moment_max_u(M, T, exact);
  if (umax < kMomMinU) return pl;
  pl.use = true;
  pl.umax = umax;
  pl.parts = exact ? 3 : 2;
  pl.lead = keep_offset & 7;
  const long nv = static_cast<long>(N) + pl.lead;
  const long steps = (nv + 31) / 32;
  const long groups = static_cast<long>(B) * H * tensors;
  // one round of workgroups, a compute unit each, but at least a tile of tokens per workgroup
  const long want = groups < 256 ? 256 / groups : 1;
  long per = (steps + want - 1) / want;
  if (per < 4) per = 4;
  if (per > steps) per = steps;
  pl.bpc = static_cast<int>((per * 32 + umax - 1) / umax);
  pl.S = static_cast<int>((per + pl.bpc - 1) / pl.bpc);
  pl.U = 32 * pl.S;
  pl.blocks = static_cast<int>((nv + pl.U - 1) / pl.U);
  pl.chunks = (pl.blocks + pl.bpc - 1) / pl.bpc;
  const unsigned tile_tokens = D == 256 ? 64 : 128;
  pl.lds = static_cast<unsigned>(pl.S) * pl.parts * 1024u + 2u * tile_tokens * (2u * D + 32u);
  pl.op_bytes = exact ? 0 : static_cast<size_t>(expand_tiles(M)) * ((pl.blocks + 1) / 2) * 4096;
  pl.mom_bytes = align_up(static_cast<size_t>(B) * H * pl.blocks * kMomP * Dc * sizeof(float), 256);
  return pl;
}

template <int D, int NT, bool kEnergy>
static int launch_moments_t(const MomentParams& p, const MomentPlan& pl, int tensors, hipStream_t st, KernelTimers* tm) {
  auto kern = fa_moments<D, NT, kEnergy>;
  if (pl.lds > 48u * 1024u &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                          158 * 1024) != hipSuccess)
    return FA_ERR_HIP;
  FA_LAUNCH_TIMED(tm, 0, kern, dim3(pl.chunks, tensors * p.B * p.H), dim3(64 * MomTile<D>::kWaves), pl.lds, st, p);
  return FA_OK;
}

int launch_moments(const MomentParams& p, const MomentPlan& pl, int tensors, hipStream_t st, KernelTimers* tm) {
  const bool energy = p.t[0].epart != nullptr;
  if (p.D == 64) return energy ? launch_moments_t<64, 3, true>(p, pl, tensors, st, tm) : launch_moments_t<64, 2, false>(p, pl, tensors, st, tm);
  if (p.D == 128) return energy ? launch_moments_t<128, 3, true>(p, pl, tensors, st, tm) : launch_moments_t<128, 2, false>(p, pl, tensors, st, tm);
  return energy ? launch_moments_t<256, 3, true>(p, pl, tensors, st, tm) : launch_moments_t<256, 2, false>(p, pl, tensors, st, tm);
}

int launch_expand(const MomentParams& p, int tensors, hipStream_t st, KernelTimers* tm) {
  const int dmax = tensors == 2 && p.t[1].Dc > p.t[0].Dc ? p.t[1].Dc : p.t[0].Dc;
  const int ct = (dmax + 15) / 16, tiles = expand_tiles(p.M);
  if (!p.t[0].ecoef) {
    const int ht = expand_tiles_per_wg(ct, tiles, static_cast<double>(tensors) * p.B * p.H, p.blocks);
    const int ctw = expand_columns(ct, tiles, static_cast<double>(tensors) * p.B * p.H, p.blocks);
    const int ks = ctw <= 4 ? 2 : 1;
    const unsigned lds = 2u * ks * kExpSteps * 4096u;            // (kExpSteps / ht steps of ht operands; the shares' sums fit in)
    auto kern = ht == 2 ? (ctw >= kExpSteps ? fa_expand16<2, 1> : fa_expand16<2, 2>) : (ctw >= kExpSteps ? fa_expand16<1, 1> : fa_expand16<1, 2>);
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                            2 * 2 * kExpSteps * 4096) != hipSuccess)
      return FA_ERR_HIP;
    FA_LAUNCH_TIMED(tm, 1, kern, dim3(tensors * p.B * p.H, (ct + ctw - 1) / ctw, (tiles + ht - 1) / ht), dim3(64 * ctw * ks), lds, st, p, ctw, ks);
    return FA_OK;
  }
  // split the columns while that leaves fewer than a workgroup per compute unit, then share the blocks
  int ctw = ct < 8 ? ct : 8;
  while (ctw > 1 && static_cast<long>(tiles) * ((ct + ctw - 1) / ctw) * tensors * p.B * p.H < 256) ctw = (ctw + 1) / 2;
  // Fewer workgroups than compute units (of a column each, then) and 64 blocks or more: eight shares of the blocks (2 heads x 8171 tokens,
  // D = 64, the call 21.9 -> 19.9 us; 4 x 39062, 31.3 -> 27.0; over 7000 calls, against four, 8 - 15 blocks 1.06 of the time, 32 - 63 1.007,
  // 64 - 95 0.99, 192 - 255 0.95); else four (256 workgroups: 13.8 us against 15.0 with eight, the matrix rate bounds both)
  // and at most twelve waves (with sixteen 22 heads x 17644 tokens, M = 172: 60.5 -> 64.2 the call; 45 x 3326, D = 256, M = 102:
  // 68.4 -> 73.6).
  int ks = kExpandWaves / ctw;
  const int shares = p.blocks >= 64 && static_cast<long>(tiles) * ((ct + ctw - 1) / ctw) * tensors * p.B * p.H < 256 ? 8 : 4;
  if (ks > shares) ks = shares;
  if (ks > p.blocks) ks = p.blocks;
  if (ks < 1) ks = 1;
  const dim3 grid(tiles, (ct + ctw - 1) / ctw, tensors * p.B * p.H);
  FA_LAUNCH_TIMED(tm, 1, fa_expand, grid, dim3(64 * ctw * ks), 0, st, p, ctw, ks);
  return FA_OK;
}

}  // namespace fa
