// Last launch of fa_decode: merges the partial records of a query head, applies diag(w) C_v, normalises.
//
// A query head is shared by NS workgroups that divide the output dims by RANK (compressed dims cb0 .. cb0 + cbw - 1 and
// kept dims kb0 .. kb0 + kbw - 1 in mask order), so the band of C_v columns and the kept-dim columns of the records are
// known before the mask row arrives.  The launch is a chain of latencies (a few tens of KB per workgroup), so everything
// is requested at the start: the statistics by every wave for itself (no barrier until the sums meet), the series sums, the
// band of C_v, and the full-row records at all dims instead of the slice's own, which only the mask tells.  Further
// batches only where a list is longer than WR requests a thread (series sums) or WC (C_v).  The workgroups of one KV head
// are numbered so that they run on one XCD and share its L2 (workgroup ids go round the eight XCDs); fewer than eight heads
// of more workgroups than an XCD has compute units are spread over all of them (one KV head, eight query heads, D = 256,
// M = 800: 17.7 -> 13.3 us; with few workgroups the shared L2 is worth 0.3 us).
#include <type_traits>

#include "fa_finish.hpp"

namespace fa {

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
template <int VEC> struct FinVec { using type = f32x4; using load = f32x4; };
template <> struct FinVec<3> { using type = f32x4; using load = f32x4u; };
template <> struct FinVec<1> { using type = float; using load = float; };

__host__ __device__ __forceinline__ bool spread_finish(int pairs, int per_kv) { return pairs < 8 && per_kv > 32; }

// VEC: 4 floats of a C_v row read at once; 3: the same for counts that are no multiple of 4, whose rows lie at any 4-byte
// boundary (the last vector of a row ends with the row; what it holds twice is not used); 1: one by one, for fewer than 4
template <int VEC, int WR, int WC>
__global__ __launch_bounds__(kFinBlock, WR > 16 ? 1 : WR > 8 ? 2 : 4) void decode_finish(DecodeParams p, int NS) {
  using V = typename FinVec<VEC>::type;
  using VL = typename FinVec<VEC>::load;
  constexpr int kV = VEC == 1 ? 1 : 4;
  constexpr int kNW = kFinBlock / 64;
  constexpr int kSL = 4;                            // statistics per lane requested at the start (longer lists: read again)
  constexpr int kWB = WR > 8 ? 4 : 2;               // independent requests per batch: full-row records, kept dims
  __shared__ float es_s[kNW][kMaxPartials];         // e^{m_s - m} per record, a copy per wave
  __shared__ f32x4 red4[kFinBlock];                 // series sums per record group, then C_v partial sums per row group
  __shared__ f32x4 redw[kFinBlock];                 // full-row records per record group
  __shared__ float redk[kFinBlock];                 // kept dims per record group
  __shared__ float rr[FA_MAX_DECODE_STATES + 4];
  __shared__ int dim_of[FA_MAX_HEAD_DIM + 8];       // output dim of each rank of this slice

  // workgroup -> (KV head, query head of the group, slice)
  const int per_kv = p.G * NS, sh = spread_finish(p.B * p.Hkv, per_kv) ? 0 : 3, slot = blockIdx.x >> sh;
  const int bh = ((slot / per_kv) << sh) + (blockIdx.x & ((1 << sh) - 1));
  if (bh >= p.B * p.Hkv) return;
  const int g = (slot % per_kv) / NS, sl = slot % NS;
  const int b = bh / p.Hkv, hkv = bh % p.Hkv, hq = b * p.Hq + hkv * p.G + g;
  const int D = p.D, M = p.M, Sm = p.Sm, Sw = p.Sw, S = Sm + Sw, Dvc = p.Dvc, Dvu = p.Dvu, Mint = p.Mint;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int Dva = 16 * ((Dvu + 15) / 16), recm = p.recm, recw = p.recw;
  const float* pm = p.part_m + static_cast<size_t>(hq) * Sm * recm;
  const float* pw = p.part_w + static_cast<size_t>(hq) * Sw * recw;
  const bool do_cv = Sm > 0 && Dvc > 0;
  const int cbw = ((Dvc + NS - 1) / NS + kV - 1) / kV * kV, cb0 = sl * cbw, cbn = max(0, min(cbw, Dvc - cb0));
  const int kbw = (Dvu + NS - 1) / NS, kb0 = sl * kbw, kbn = max(0, min(kbw, Dvu - kb0));

  // ---- every request that depends on nothing (clamped, never predicated) ------------------------
  auto stat = [&](int i) {
    const int s = min(lane + 64 * i, S - 1);
    return *reinterpret_cast<const float2*>(s < Sm ? pm + static_cast<size_t>(s) * recm : pw + static_cast<size_t>(s - Sm) * recw);
  };
  float2 st[kSL];
#pragma unroll
  for (int i = 0; i < kSL; ++i)
    if (i * 64 < S) st[i] = stat(i);
  uint8_t vmb[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) vmb[i] = p.vmask[static_cast<size_t>(bh) * D + min(lane + 64 * i, D - 1)];
  // series sums: thread (4 slots c4r, record group gr)
  const int lgr = 29 - __clz(Mint), ngr = kFinBlock >> lgr, c4r = tid & ((1 << lgr) - 1), gr = tid >> lgr;   // (Mint is 128, 256, 512 or 1024)
  const float* pr = pm + 4 + Dva + 4 * c4r;
  f32x4 rv[WR];
  if (do_cv) {
#pragma unroll
    for (int u = 0; u < WR; ++u)
      if (u * ngr < Sm) rv[u] = *reinterpret_cast<const f32x4*>(pr + static_cast<size_t>(min(gr + u * ngr, Sm - 1)) * recm);
  }
  // C_v band: thread (column vector cqv, row group rgv)
  const int nq = max((cbn + kV - 1) / kV, 1), ngrp = kFinBlock / nq, cqv = tid % nq, rgv = tid / nq;
  const bool cv_on = do_cv && cbn > 0 && tid < nq * ngrp;
  const int back = VEC == 3 ? 4 * nq - cbn : 0;    // (not 0 in the slice that ends with the row)
  const float* cvb = p.cv + static_cast<size_t>(bh) * M * Dvc + cb0 + kV * cqv - (cqv == nq - 1 ? back : 0);
  V cvv[WC];
  if (do_cv && cbn > 0) {
#pragma unroll
    for (int u = 0; u < WC; ++u)
      if (u * ngrp < M) cvv[u] = *reinterpret_cast<const VL*>(cvb + static_cast<size_t>(min(rgv + u * ngrp, M - 1)) * Dvc);
  }
  // full-row records: thread (4 dims d4, record group wg)
  const int nd4 = D / 4, nwg = kFinBlock / nd4, d4 = tid % nd4, wg = tid / nd4;
  const float* pwd = pw + 4 + 4 * d4;
  f32x4 wv[kWB];
  if (Sw > 0) {
#pragma unroll
    for (int u = 0; u < kWB; ++u)
      if (u * nwg < Sw) wv[u] = *reinterpret_cast<const f32x4*>(pwd + static_cast<size_t>(min(wg + u * nwg, Sw - 1)) * recw);
  }
  // kept dims of the middle records: thread (kept rank kc, record group kg)
  const int kcn = max(kbn, 1), nkg = kFinBlock / kcn, kc = tid % kcn, kg = tid / kcn;
  const bool k_on = Sm > 0 && kbn > 0 && tid < kcn * nkg;
  const float* pk = pm + 4 + kb0 + kc;
  float kv[kWB];
  if (Sm > 0 && kbn > 0) {
#pragma unroll
    for (int u = 0; u < kWB; ++u)
      if (u * nkg < Sm) kv[u] = pk[static_cast<size_t>(min(kg + u * nkg, Sm - 1)) * recm];
  }

  // which dims this slice writes (the mask row arrives before the long lists)
  {
    uint64_t vbal[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) vbal[i] = __ballot(vmb[i] != 0 && lane + 64 * i < D);
    if (tid < D) {
      const int rk = dim_rank(vbal, tid);
      const int c = rk < 0 ? -rk - 1 - cb0 : rk - kb0;
      if (c >= 0 && c < (rk < 0 ? cbn : kbn)) dim_of[rk < 0 ? c : cbw + c] = tid;
    }
  }
  // ---- maximum, factors and normaliser, by every wave for itself ---------------------------------
  float* es = es_s[wave];
  float m = -INFINITY, L = 0.0f, Lm = 0.0f;
#pragma unroll
  for (int i = 0; i < kSL; ++i)
    if (i * 64 < S) m = fmaxf(m, st[i].x);          // (clamped repeats do not matter here)
  for (int i = kSL; i * 64 < S; ++i) m = fmaxf(m, stat(i).x);
  m = wave_max_fast(m);
  auto take = [&](int i, const float2& x) {
    const int s = lane + 64 * i;
    const float e = x.x == -INFINITY ? 0.0f : __expf(x.x - m);
    if (s < S) {
      es[s] = e;
      L += e * x.y;
      if (s < Sm) Lm += e * x.y;                    // the middle rows' share: r of the constant basis function
    }
  };
#pragma unroll
  for (int i = 0; i < kSL; ++i)
    if (i * 64 < S) take(i, st[i]);
  for (int i = kSL; i * 64 < S; ++i) take(i, stat(i));
  L = wave_sum_fast(L);
  Lm = wave_sum_fast(Lm);
  // the factors were written by this wave and are read by this wave: its LDS operations complete in order
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

  // ---- per-thread sums over the records -----------------------------------------------------------
  if (do_cv) {
    f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < WR; ++u) {
      const int s = gr + u * ngr;
      if (s < Sm) a += es[s] * rv[u];
    }
    for (int s0 = WR * ngr; s0 < Sm; s0 += WR * ngr) {   // further batches: requests first, sums after
#pragma unroll
      for (int u = 0; u < WR; ++u) rv[u] = *reinterpret_cast<const f32x4*>(pr + static_cast<size_t>(min(s0 + gr + u * ngr, Sm - 1)) * recm);
#pragma unroll
      for (int u = 0; u < WR; ++u) {
        const int s = s0 + gr + u * ngr;
        if (s < Sm) a += es[s] * rv[u];
      }
    }
    red4[tid] = a;
  }
  if (Sw > 0) {
    f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < kWB; ++u) {
      const int s = wg + u * nwg;
      if (s < Sw) a += es[Sm + s] * wv[u];
    }
    for (int s = wg + kWB * nwg; s < Sw; s += nwg) a += es[Sm + s] * *reinterpret_cast<const f32x4*>(pwd + static_cast<size_t>(s) * recw);
    if (wg < nwg) redw[tid] = a;
  }
  {
    float o = 0.0f;
    if (k_on) {
#pragma unroll
      for (int u = 0; u < kWB; ++u) {
        const int s = kg + u * nkg;
        if (s < Sm) o += es[s] * kv[u];
      }
      for (int s = kg + kWB * nkg; s < Sm; s += nkg) o += es[s] * pk[static_cast<size_t>(s) * recm];
    }
    redk[tid] = o;
  }
  __syncthreads();
  // ---- r in basis order, weighted by the inverse squared norms ------------------------------------
  if (do_cv) {
    for (int ig = tid; ig < Mint; ig += kFinBlock) {   // record order: 32 * chunk + 16 * (cos | sin) + order
      const float* src = reinterpret_cast<const float*>(red4) + ig;
      auto sum = [&](auto n) {
        float v = 0.0f;
#pragma unroll
        for (int gi = 0; gi < decltype(n)::value; ++gi) v += src[gi * Mint];
        return v;
      };
      const float v = ngr == 8 ? sum(std::integral_constant<int, 8>{}) : ngr == 4 ? sum(std::integral_constant<int, 4>{})
                      : ngr == 2 ? sum(std::integral_constant<int, 2>{}) : src[0];
      const int n = 16 * (ig >> 5) + (ig & 15) + 1, mm = 2 * n - 1 + ((ig >> 4) & 1);
      if (mm < M) rr[mm] = v * basis_weight(n, p.T);
    }
    if (tid == kFinBlock - 1) rr[0] = Lm * basis_weight(0, p.T);
  }
  __syncthreads();
  // ---- compressed dims of the slice: sum_m rr[m] C_v[m, rank] -------------------------------------
  {
    V o{};
    if (cv_on) {
#pragma unroll
      for (int u = 0; u < WC; ++u) {
        const int mm = rgv + u * ngrp;
        if (mm < M) o += rr[mm] * cvv[u];
      }
      for (int m0 = WC * ngrp; m0 < M; m0 += WC * ngrp) {
#pragma unroll
        for (int u = 0; u < WC; ++u) cvv[u] = *reinterpret_cast<const VL*>(cvb + static_cast<size_t>(min(m0 + rgv + u * ngrp, M - 1)) * Dvc);
#pragma unroll
        for (int u = 0; u < WC; ++u) {
          const int mm = m0 + rgv + u * ngrp;
          if (mm < M) o += rr[mm] * cvv[u];
        }
      }
    }
    reinterpret_cast<V*>(red4)[tid] = o;   // [row group][column vector]
  }
  __syncthreads();
  // ---- a power of two of lanes per output dim adds the shares up -----------------------------------
  // (of the groups that had a row or record: a slice with one kept dim has 256 groups for it, odd counts 8.1 -> 9.4 us with all)
  const int nj = cbw + kbw, ncv = min(ngrp, M), nkm = min(nkg, Sm), nwr = min(nwg, Sw);
  int lper = 0;
  while (lper < 4 && (nj << (lper + 1)) <= kFinBlock) ++lper;
  const int per = 1 << lper, part = tid & (per - 1);
  for (int j0 = 0; j0 < nj; j0 += kFinBlock >> lper) {
    const int j = j0 + (tid >> lper);
    const bool cdim = j < cbn, kdim = j >= cbw && j < cbw + kbn;
    float v = 0.0f;
    if (cdim || kdim) {
      const int d = dim_of[j];
      if (do_cv && cdim) {
        const float* src = reinterpret_cast<const float*>(red4) + j + (j >= kV * (nq - 1) ? back : 0);
        for (int gi = part; gi < ncv; gi += per) v += src[kV * gi * nq];
      }
      if (kdim)
        for (int gi = part; gi < nkm; gi += per) v += redk[gi * kcn + (j - cbw)];
      const float* src = reinterpret_cast<const float*>(redw) + d;
      for (int gi = part; gi < nwr; gi += per) v += src[gi * 4 * nd4];
    }
    for (int o = per >> 1; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    if (part == 0 && (cdim || kdim)) p.out[static_cast<size_t>(hq) * D + dim_of[j]] = L > 0.0f ? v / L : 0.0f;   // (a sequence without rows)
  }
}

// Slices per query head: as many as keep the launch within one round of resident workgroups; up to 128 slots and head dim 128,
// counts in fours, half of that (the chain is then longer than what a slice reads: 512 heads, M = 128, 9.0 -> 8.3 us; odd counts
// lose by it, 10.9 -> 12.7, and so does head dim 256, 12.8 -> 14.1; at M = 556, 9 of 60).  Long lists of requests where the
// XCD with most workgroups holds them at once: one of the longest per compute unit, two of the next.  Odd counts by vectors instead
// of floats: 224 pairs of six heads, M = 585, 102 dims, the call 171 -> 138 us; 256 of twelve, D = 64, M = 341, 47 dims, 110 -> 97;
// 24 of eight, M = 130, 101 dims, 26.5 -> 25.  This launch against the two
// kernels it replaced: 32 heads, M = 256, 7.9 -> 7.0 us, M = 1023 13.2 -> 11.8; odd counts, 192 heads, M = 130, 15.5 -> 7.2; 128 heads of
// eight KV heads, M = 256, 8.5 -> 7.9; over 430 record lists of 4 - 3072 heads, both types, 0.77 of the time, four of them 3 - 6 % slower
// (thousands of heads with one or two records each).
int launch_finish(const DecodeParams& p, hipStream_t st, KernelTimers* tm) {
  const int BH = p.B * p.Hkv;
  const long heads = static_cast<long>(p.B) * p.Hq;
  const bool v4 = (p.Dvc & 3) == 0, v3 = p.Dvc >= 4;
  int NS = p.D <= 32 ? 1 : (p.D <= 64 ? 2 : (p.D <= 128 ? 4 : 8));
  while (NS > 1 && heads * NS > (v4 && p.D <= 128 && p.Mint <= 128 ? 512 : 1024)) NS /= 2;
  const long wgs = static_cast<long>(spread_finish(BH, p.G * NS) ? BH : (BH + 7) / 8 * 8) * p.G * NS, xcd = (wgs + 7) / 8;
  const dim3 grid(static_cast<unsigned>(wgs));
  if (xcd <= 32 && p.Mint > 512) {
    if (v4) FA_LAUNCH_TIMED(tm, 2, (decode_finish<4, 32, 28>), grid, dim3(kFinBlock), 0, st, p, NS);
    else if (v3) FA_LAUNCH_TIMED(tm, 2, (decode_finish<3, 32, 28>), grid, dim3(kFinBlock), 0, st, p, NS);
    else FA_LAUNCH_TIMED(tm, 2, (decode_finish<1, 32, 32>), grid, dim3(kFinBlock), 0, st, p, NS);
  } else if (xcd <= 64) {
    if (v4) FA_LAUNCH_TIMED(tm, 2, (decode_finish<4, 16, 16>), grid, dim3(kFinBlock), 0, st, p, NS);
    else if (v3) FA_LAUNCH_TIMED(tm, 2, (decode_finish<3, 16, 16>), grid, dim3(kFinBlock), 0, st, p, NS);
    else FA_LAUNCH_TIMED(tm, 2, (decode_finish<1, 16, 32>), grid, dim3(kFinBlock), 0, st, p, NS);
  } else {
    if (v4) FA_LAUNCH_TIMED(tm, 2, (decode_finish<4, 8, 8>), grid, dim3(kFinBlock), 0, st, p, NS);
    else if (v3) FA_LAUNCH_TIMED(tm, 2, (decode_finish<3, 8, 8>), grid, dim3(kFinBlock), 0, st, p, NS);
    else FA_LAUNCH_TIMED(tm, 2, (decode_finish<1, 8, 16>), grid, dim3(kFinBlock), 0, st, p, NS);
  }
  return FA_OK;
}

}  // namespace fa
