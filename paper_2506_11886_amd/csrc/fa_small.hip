// Small calls of fa_decode in one launch, one workgroup per (sequence, KV head), plain fp32 arithmetic.
//
// Three launches of a few microseconds' work are mostly launch ramps, table builds and round trips.  Here everything a
// call reads is requested at once into registers; cos / sin come from a table of one period in LDS, indexed by n j mod T
// (exact phases); then rows are scored (a thread per middle row, 8 dims of a full-width row per thread), normalised over the
// workgroup, and the series sums, kept dims and full-width rows are summed by (harmonic | dim, row group) and meet in LDS.
#include "fa_small.hpp"

namespace fa {

constexpr int kSmThreads = 512;
constexpr int kSmWaves = kSmThreads / 64;
constexpr int kSmG = 4;                // query heads per KV head, at most
constexpr int kSmMaxT = 4096;          // period (the table is 8 T bytes of LDS)
constexpr int kSmMaxM = 128, kSmMaxD = 128, kSmMaxRows = 2048;
constexpr int kSmC = 24;               // elements of C_k (C_v) a thread holds
constexpr int kSmKV = 4;               // 8-dim vectors of a kept K row requested at the start
constexpr int kSmKF = 4, kSmVF = 4, kSmVK = 4;   // items of full-width K, full-width V and kept V requested at the start

__host__ __device__ __forceinline__ int pow2_at_least(int x) {
  int p = 1;
  while (p < x) p *= 2;
  return p;
}

// LDS: table | queries | coefficients | scores | series sums, weighted sums | partial sums (full-width rows; series; kept dims)
struct SmallLds {
  unsigned q, qk, g, sc, rr, fp, rp, kp, total;
};
__host__ __device__ __forceinline__ SmallLds small_layout(int D, int Dup, int M, int T, int rows) {
  SmallLds L;
  L.q = (T * 8 + 15u) & ~15u;
  L.qk = L.q + D * 16;
  L.g = L.qk + Dup * 16;
  L.sc = L.g + (M / 2 + 1) * 32;
  L.rr = L.sc + rows * 16;
  L.fp = L.rr + M * 16;
  const int segs = kSmThreads / pow2_at_least(D / 8);
  L.rp = L.fp + segs * D * 16;
  L.kp = L.rp + kSmThreads * 32;
  L.total = L.kp + kSmThreads * 16;
  return L;
}

// sum over the lanes whose index differs in bits below `n` (a power of two)
__device__ __forceinline__ float lanes_sum(float v, int n) {
  for (int o = n >> 1; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

template <typename T>
__global__ __launch_bounds__(kSmThreads, 2) void decode_small(DecodeParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ float wred[2][kSmWaves][kSmG];
  __shared__ float lmid[kSmWaves][kSmG];
  const int bh = blockIdx.x, b = bh / p.Hkv, hkv = bh % p.Hkv;
  const int G = p.G, D = p.D, M = p.M, per = p.T, Dkc = p.Dkc, Dvc = p.Dvc, Dku = p.Dku, Dvu = p.Dvu;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int Nb = seq_middle_rows(p, b), Wb = seq_full_rows(p, b), R = Nb + Wb;
  const int Dup = (Dku + 7) & ~7, nmax = M / 2;
  const SmallLds L = small_layout(D, Dup, M, per, p.N + p.W);
  float2* tab = reinterpret_cast<float2*>(smem);
  f32x4* q_s = reinterpret_cast<f32x4*>(smem + L.q);      // [D] queries of the group
  f32x4* qk_s = reinterpret_cast<f32x4*>(smem + L.qk);    // [Dup] at the kept K dims, zero padded
  f32x4* g_s = reinterpret_cast<f32x4*>(smem + L.g);      // [0]: constant; [2 n - 1], [2 n]: cosine, sine of order n
  f32x4* sc = reinterpret_cast<f32x4*>(smem + L.sc);      // [row] scores, then probabilities (middle rows first)
  f32x4* rr = reinterpret_cast<f32x4*>(smem + L.rr);      // [M] weighted series sums
  float* fp = reinterpret_cast<float*>(smem + L.fp);      // [segment][4][D] full-width rows
  float* rp = reinterpret_cast<float*>(smem + L.rp);      // [thread][cosine 4 | sine 4]; then the shares of C_v
  f32x4* kp = reinterpret_cast<f32x4*>(smem + L.kp);      // [thread] kept dims
  const size_t hq0 = static_cast<size_t>(b) * p.Hq + hkv * G;

  // ---- requests (clamped, never predicated; lists longer than this are finished where they are used) -----------
  uint8_t kmb[2], vmb[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    kmb[i] = p.kmask[static_cast<size_t>(bh) * D + min(lane + 64 * i, D - 1)];
    vmb[i] = p.vmask[static_cast<size_t>(bh) * D + min(lane + 64 * i, D - 1)];
  }
  const T* q = static_cast<const T*>(p.q) + hq0 * D;
  const T qe = q[min(tid, G * D - 1)];                     // (G D <= 512)
  // C_k: thread (row, part of its columns); C_v: thread (column, part of its rows)
  const int kparts = min(kSmThreads / pow2_at_least(M), 64), km = tid / kparts, kpart = tid % kparts;
  const int vcp = pow2_at_least(max(Dvc, 1)), vparts = kSmThreads / vcp, vc = tid % vcp, vpart = tid / vcp;
  const float* ck = p.ck + (static_cast<size_t>(bh) * M + min(km, M - 1)) * Dkc;
  const float* cv = p.cv + static_cast<size_t>(bh) * M * Dvc + min(vc, max(Dvc - 1, 0));
  float cke[kSmC], cve[kSmC];
  if (Nb > 0) {
#pragma unroll
    for (int i = 0; i < kSmC; ++i)
      if (i * kparts < Dkc) cke[i] = ck[min(kpart + i * kparts, Dkc - 1)];
#pragma unroll
    for (int i = 0; i < kSmC; ++i)
      if (Dvc > 0 && i * vparts < M) cve[i] = cv[static_cast<size_t>(min(vpart + i * vparts, M - 1)) * Dvc];
  }
  // kept K dims: a thread per middle row; full-width rows: thread (row, 8 dims)
  const T* kk = static_cast<const T*>(p.k_keep) + bh * p.kk_stride;
  const T* vk = static_cast<const T*>(p.v_keep) + bh * p.vk_stride;
  const T* kf = static_cast<const T*>(p.k_full) + bh * p.full_stride;
  const T* vf = static_cast<const T*>(p.v_full) + bh * p.full_stride;
  const int nd8 = D / 8, PP = pow2_at_least(nd8), segs = kSmThreads / PP, part8 = tid % PP, seg = tid / PP;
  const int pc = min(part8, nd8 - 1) * 8;
  Frag<T> xk[kSmKV], xf[kSmKF], yf[kSmVF];
  if (Nb > 0) {
#pragma unroll
    for (int i = 0; i < kSmKV; ++i)
      if (i * 8 < Dup) xk[i].load(kk + static_cast<size_t>(min(tid, Nb - 1)) * Dup + 8 * i);
  }
  if (Wb > 0) {
#pragma unroll
    for (int i = 0; i < kSmKF; ++i)
      if (i * segs < Wb) xf[i].load(kf + static_cast<size_t>(min(seg + i * segs, Wb - 1)) * D + pc);
#pragma unroll
    for (int i = 0; i < kSmVF; ++i)
      if (i * segs < Wb) yf[i].load(vf + static_cast<size_t>(min(seg + i * segs, Wb - 1)) * D + pc);
  }
  // kept V dims: thread (dim, group of 8 tokens)
  const int UP = pow2_at_least(max(Dvu, 1)), usegs = kSmThreads / UP, uu = tid % UP, useg = tid / UP, ngrp = (Nb + 7) / 8;
  Frag<T> yk[kSmVK];
  if (Nb > 0 && Dvu > 0) {
#pragma unroll
    for (int i = 0; i < kSmVK; ++i)
      if (i * usegs < ngrp)
        yk[i].load(vk + (static_cast<size_t>(min(useg + i * usegs, ngrp - 1)) * Dvu + min(uu, Dvu - 1)) * 8);
  }

  // ---- table of one period; ranks and queries --------------------------------------------------------
  if (Nb > 0)
    for (int r = tid; r < per; r += kSmThreads) {
      float2 e;
      sincospif(2.0f * (static_cast<float>(r) / static_cast<float>(per)), &e.y, &e.x);
      tab[r] = e;
    }
  uint64_t kb[4] = {0, 0, 0, 0}, vb[4] = {0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    kb[i] = __ballot(kmb[i] != 0 && lane + 64 * i < D);
    vb[i] = __ballot(vmb[i] != 0 && lane + 64 * i < D);
  }
  __shared__ int16_t kcdim[kSmMaxD];                       // compressed K dims in order
  for (int i = tid; i < (D + Dup) * kSmG; i += kSmThreads) {   // heads past the group, pad columns
    const int d = i / kSmG, h = i % kSmG;
    if (d < D ? h >= G : (d - D >= Dku || h >= G)) reinterpret_cast<float*>(d < D ? q_s + d : qk_s + (d - D))[h] = 0.0f;
  }
  if (tid < G * D) {
    const int h = tid / D, d = tid % D;
    const float x = to_f32(qe);
    const int rk = dim_rank(kb, d);
    reinterpret_cast<float*>(q_s + d)[h] = x;
    if (rk >= 0) reinterpret_cast<float*>(qk_s + rk)[h] = x;
    else if (h == 0) kcdim[-rk - 1] = static_cast<int16_t>(d);
  }
  __syncthreads();

  // ---- g = diag(w) C_k q at the compressed dims ---------------------------------------------------------
  if (Nb > 0) {
    f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < kSmC; ++i) {
      const int c = kpart + i * kparts;
      if (c < Dkc && km < M) a += cke[i] * q_s[kcdim[c]];
    }
    const float w = km < M ? basis_weight((km + 1) / 2, per) : 0.0f;
#pragma unroll
    for (int h = 0; h < kSmG; ++h) a[h] = lanes_sum(a[h], kparts) * w;
    if (kpart == 0 && km < M) g_s[km] = a;
    if (tid == 0 && (M & 1) == 0) g_s[M] = f32x4{0.f, 0.f, 0.f, 0.f};   // (the unpaired cosine has no sine)
  }
  __syncthreads();

  // ---- scores -----------------------------------------------------------------------------------------
  for (int j = tid; j < Nb; j += kSmThreads) {
    f32x4 s = g_s[0];
    const int pos = p.t0 + j;                              // (< T)
    int r = 0;
    for (int n = 1; n <= nmax; ++n) {
      r += pos;
      if (r >= per) r -= per;
      const float2 e = tab[r];
      s += e.x * g_s[2 * n - 1] + e.y * g_s[2 * n];
    }
    for (int i = 0; 8 * i < Dup; ++i) {
      Frag<T> x;
      if (j == tid && i < kSmKV) {
#pragma unroll
        for (int k = 0; k < kSmKV; ++k)
          if (k == i) x = xk[k];
      } else {
        x.load(kk + static_cast<size_t>(j) * Dup + 8 * i);
      }
      float v[8];
      unpack8(x, v);
#pragma unroll
      for (int e = 0; e < 8; ++e) s += v[e] * qk_s[8 * i + e];
    }
    sc[j] = p.scale * s;
  }
  const int pass_f = (Wb + segs - 1) / segs;
#pragma unroll 1
  for (int i = 0; i < pass_f; ++i) {
    const int j = seg + i * segs;
    Frag<T> x;
    if (i < kSmKF) {
#pragma unroll
      for (int k = 0; k < kSmKF; ++k)
        if (k == i) x = xf[k];
    } else {
      x.load(kf + static_cast<size_t>(min(j, Wb - 1)) * D + pc);
    }
    float v[8];
    unpack8(x, v);
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    if (part8 < nd8) {
#pragma unroll
      for (int e = 0; e < 8; ++e) s += v[e] * q_s[pc + e];
    }
#pragma unroll
    for (int h = 0; h < kSmG; ++h) s[h] = lanes_sum(s[h], PP);
    if (part8 == 0 && j < Wb) {
#pragma unroll
      for (int h = 0; h < kSmG; ++h)   // (the last Tq rows are the new tokens: query token h / Gq sees those up to its own)
        s[h] = j <= Wb - p.Tq + h / p.Gq ? s[h] * p.scale : -INFINITY;
      sc[Nb + j] = s;
    }
  }
  __syncthreads();

  // ---- softmax over all rows, per head --------------------------------------------------------------------
  f32x4 m = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
  for (int r = tid; r < R; r += kSmThreads) {
    const f32x4 s = sc[r];
#pragma unroll
    for (int h = 0; h < kSmG; ++h) m[h] = fmaxf(m[h], s[h]);
  }
#pragma unroll
  for (int h = 0; h < kSmG; ++h) {
    m[h] = wave_max_fast(m[h]);
    if (lane == 0) wred[0][wave][h] = m[h];
  }
  __syncthreads();
  f32x4 l = {0.f, 0.f, 0.f, 0.f}, lm = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int h = 0; h < kSmG; ++h) {
    m[h] = wred[0][0][h];
#pragma unroll
    for (int w = 1; w < kSmWaves; ++w) m[h] = fmaxf(m[h], wred[0][w][h]);
    if (m[h] == -INFINITY) m[h] = 0.0f;
  }
  for (int r = tid; r < R; r += kSmThreads) {
    f32x4 s = sc[r];
#pragma unroll
    for (int h = 0; h < kSmG; ++h) {
      s[h] = __expf(s[h] - m[h]);
      l[h] += s[h];
      if (r < Nb) lm[h] += s[h];
    }
    sc[r] = s;
  }
#pragma unroll
  for (int h = 0; h < kSmG; ++h) {
    const float a = wave_sum_fast(l[h]), c = wave_sum_fast(lm[h]);
    if (lane == 0) {
      wred[1][wave][h] = a;
      lmid[wave][h] = c;
    }
  }
  __syncthreads();

  // ---- weighted sums --------------------------------------------------------------------------------------
  const int nP = pow2_at_least(max(nmax, 1)), rsegs = kSmThreads / nP, rn = tid % nP, rseg = tid / nP;
  if (Nb > 0 && nmax > 0) {   // r: thread (order rn + 1, rows rseg, rseg + rsegs, ...)
    f32x4 c = {0.f, 0.f, 0.f, 0.f}, s = {0.f, 0.f, 0.f, 0.f};
    if (rn < nmax) {
      const unsigned n = rn + 1, T_ = per;
      int r = static_cast<int>(n * static_cast<unsigned>(p.t0 + rseg) % T_);
      const int d = static_cast<int>(n * static_cast<unsigned>(rsegs) % T_);
      for (int j = rseg; j < Nb; j += rsegs) {
        const float2 e = tab[r];
        const f32x4 w = sc[j];
        c += e.x * w;
        s += e.y * w;
        r += d;
        if (r >= per) r -= per;
      }
    }
    *reinterpret_cast<f32x4*>(rp + 8 * tid) = c;
    *reinterpret_cast<f32x4*>(rp + 8 * tid + 4) = s;
  }
  {   // full-width rows
    float acc[kSmG][8];
#pragma unroll
    for (int h = 0; h < kSmG; ++h)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[h][e] = 0.0f;
#pragma unroll 1
    for (int i = 0; i < pass_f; ++i) {
      const int j = seg + i * segs;
      Frag<T> x;
      if (i < kSmVF) {
#pragma unroll
        for (int k = 0; k < kSmVF; ++k)
          if (k == i) x = yf[k];
      } else {
        x.load(vf + static_cast<size_t>(min(j, Wb - 1)) * D + pc);
      }
      if (j < Wb) {
        const f32x4 w = sc[Nb + j];
        float v[8];
        unpack8(x, v);
#pragma unroll
        for (int h = 0; h < kSmG; ++h)
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[h][e] += w[h] * v[e];
      }
    }
    if (part8 < nd8) {
#pragma unroll
      for (int h = 0; h < kSmG; ++h) {
        float* o = fp + (seg * kSmG + h) * D + pc;
        *reinterpret_cast<f32x4*>(o) = f32x4{acc[h][0], acc[h][1], acc[h][2], acc[h][3]};
        *reinterpret_cast<f32x4*>(o + 4) = f32x4{acc[h][4], acc[h][5], acc[h][6], acc[h][7]};
      }
    }
  }
  if (Nb > 0 && Dvu > 0) {   // kept dims
    f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int i = 0; i * usegs < ngrp; ++i) {
      const int g = useg + i * usegs;
      Frag<T> x;
      if (i < kSmVK) {
#pragma unroll
        for (int k = 0; k < kSmVK; ++k)
          if (k == i) x = yk[k];
      } else {
        x.load(vk + (static_cast<size_t>(min(g, ngrp - 1)) * Dvu + min(uu, Dvu - 1)) * 8);
      }
      float v[8];
      unpack8(x, v);
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (g < ngrp && 8 * g + e < Nb) a += v[e] * sc[8 * g + e];   // (past the rows the slab holds anything)
    }
    kp[tid] = a;
  }
  __syncthreads();
  // ---- r in basis order, weighted by the inverse squared norms --------------------------------------------------
  if (Nb > 0)
    for (int i = tid; i < M * kSmG; i += kSmThreads) {
      const int mm = i / kSmG, h = i % kSmG, n = (mm + 1) / 2;
      float v = 0.0f;
      if (mm == 0) {
#pragma unroll
        for (int w = 0; w < kSmWaves; ++w) v += lmid[w][h];
      } else {
        const float* src = rp + 8 * (n - 1) + ((mm & 1) ? 0 : 4) + h;
        for (int s = 0; s < rsegs; ++s) v += src[8 * s * nP];
      }
      reinterpret_cast<float*>(rr + mm)[h] = v * basis_weight(n, per);
    }
  __syncthreads();
  // ---- C_v: thread (column, rows vpart, vpart + vparts, ...) --------------------------------------------------
  f32x4* cp = reinterpret_cast<f32x4*>(rp);
  if (Nb > 0 && Dvc > 0) {
    f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < kSmC; ++i) {
      const int mm = vpart + i * vparts;
      if (mm < M) a += cve[i] * rr[mm];
    }
    cp[tid] = a;
  }
  __syncthreads();
  if (tid < G * D) {
    const int h = tid / D, d = tid % D, rk = dim_rank(vb, d);
    float v = 0.0f, lsum = 0.0f;
    if (Wb > 0)
      for (int s = 0; s < segs; ++s) v += fp[(s * kSmG + h) * D + d];
    if (Nb > 0) {
      const float* src = reinterpret_cast<const float*>(rk < 0 ? cp + (-rk - 1) : kp + rk) + h;
      const int np = rk < 0 ? vparts : usegs, step = 4 * (rk < 0 ? vcp : UP);
      for (int s = 0; s < np; ++s) v += src[s * step];
    }
#pragma unroll
    for (int w = 0; w < kSmWaves; ++w) lsum += wred[1][w][h];
    p.out[(hq0 + h) * D + d] = lsum > 0.0f ? v / lsum : 0.0f;   // (a sequence without rows)
  }
}

// ---------------------------------------------------------------------------
// host
// ---------------------------------------------------------------------------
unsigned small_lds(int dtype, int B, int Hkv, int G, int D, int Dkc, int Dvc, int M, int T, int N, int W) {
  const int Dup = (D - Dkc + 7) & ~7, rows = N + W;
  if (static_cast<long>(B) * Hkv > 256 || G > kSmG || D > kSmMaxD || G * D > kSmThreads || M > kSmMaxM || T > kSmMaxT || rows > kSmMaxRows) return 0;
  // a thread holds its share of both states
  const int kparts = kSmThreads / pow2_at_least(M) < 64 ? kSmThreads / pow2_at_least(M) : 64;
  if (kparts * kSmC < Dkc || kSmThreads / pow2_at_least(Dvc > 0 ? Dvc : 1) * kSmC < M) return 0;
  // one compute unit does all of a pair's work: series terms and full-width products, at about 10^4 a microsecond each
  if (static_cast<long>(N) * M + static_cast<long>(W) * D > (dtype == FA_F32 ? 60000 : 30000)) return 0;
  const unsigned lds = small_layout(D, Dup, M, T, rows).total;
  return lds <= kMaxDynLds - 1024 ? lds : 0;
}

template <typename T>
static int launch_small_t(const DecodeParams& p, unsigned lds, hipStream_t st, KernelTimers* tm) {
  auto kern = decode_small<T>;
  if (lds > 48u * 1024u &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)) != hipSuccess)
    return FA_ERR_HIP;
  FA_LAUNCH_TIMED(tm, 1, kern, dim3(p.B * p.Hkv), dim3(kSmThreads), lds, st, p);
  return FA_OK;
}

int launch_small(const DecodeParams& p, int dtype, unsigned lds, hipStream_t st, KernelTimers* tm) {
  return dtype == FA_F32 ? launch_small_t<float>(p, lds, st, tm) : launch_small_t<bf16_t>(p, lds, st, tm);
}

}  // namespace fa
