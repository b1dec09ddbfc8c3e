// fa_append: per-token cache maintenance during decoding (Eq. 5 and the window of Eq. 1).
//
// The recent window is a ring inside the full-width row buffers.  When it is full, the row that
// holds its oldest token is folded into the compressed state before the new token takes it:
//   C[m,i] += phi_m(n_mid) * x[idx_c[i]]     (Eq. 5: one basis column times the evicted row)
//   X_keep[n_mid, :] = x[idx_u]              (kept dims appended at middle position n_mid)
// for K and for V, in one launch on the caller's stream.

#include "fa_common.hpp"

namespace fa {

constexpr int kABlock = 256;
constexpr int kAFly = 16;    // rows of C in flight per thread

struct AppendParams {
  const void* k_new;
  const void* v_new;
  void* k_full;
  void* v_full;
  int64_t full_stride;
  const uint8_t* kmask;
  const uint8_t* vmask;
  float* ck;
  float* cv;
  void* k_keep;
  void* v_keep;
  int64_t kk_stride, vk_stride;
  int B, Hkv, D, W, slot, Dkc, Dvc, M, T, n_mid;
  // per-sequence lists (fa_append_varlen), or null: `slot` / `n_mid` for all
  const int32_t* seq_slot;   // [B] ring row of each sequence; out of [0, W): the sequence is left alone
  const int32_t* seq_nmid;   // [B] middle position of the evicted token; < 0 or >= n_cap: nothing is folded
  int n_cap;                 // tokens the middle slabs have room for
};

// this sequence's ring row and fold position (-1: no fold; slot -1: nothing at all)
__device__ __forceinline__ void seq_append(const AppendParams& p, int b, int* slot, int* n_mid) {
  int s = p.slot, n = p.n_mid;
  if (p.seq_slot) {
    s = p.seq_slot[b];
    if (s < 0 || s >= p.W) s = -1;
  }
  if (p.seq_nmid) {
    n = p.seq_nmid[b];
    if (n < 0 || n >= p.n_cap || n >= p.T || s < 0) n = -1;
  }
  *slot = s;
  *n_mid = n;
}

// One launch: the fold reads the old row and the new token overwrites it, so a workgroup takes a slice of
// head dims for ALL basis rows - nobody else reads or writes its part of the row, and its columns of C are
// one contiguous band.  grid (sequences x heads, K | V, slices of kADims dims: a divisor of 64, see the ballot words): with the pair index fastest
// the slices of a pair land on one XCD whenever the pairs are a multiple of four, and the cache lines of C
// they share meet in one L2.  Bound: the round trips row/mask -> C -> store; the rows of C are requested
// kAFly at a time before the basis column is evaluated.
// Against a split by basis rows, which took a second launch for the overwrite and one round trip per 256
// elements: a step (append + decode) of 8 heads x 32 K tokens, M = 256, 34.1 -> 29.5 us; 16 sequences of
// up to 8 K tokens, M = 128, 62.6 -> 57.7 us.
template <typename T, int kADims>
__global__ __launch_bounds__(kABlock) void append_token(AppendParams p) {
  __shared__ float xc[kADims];              // the evicted row at this slice's compressed dims
  __shared__ float phi[FA_MAX_STATES + 2];  // basis column at n_mid
  const int tid = threadIdx.x, lane = tid & 63;
  const int bh = blockIdx.x, is_v = blockIdx.y, d0 = blockIdx.z * kADims;
  int slot, n_mid;
  seq_append(p, bh / p.Hkv, &slot, &n_mid);
  if (slot < 0) return;   // (only with per-sequence lists) this sequence is left alone
  const int D = p.D;
  const bool mine = tid < kADims && d0 + tid < D;
  T* ring = static_cast<T*>(is_v ? p.v_full : p.k_full) + bh * p.full_stride + static_cast<int64_t>(slot) * D + d0;
  const T* src = static_cast<const T*>(is_v ? p.v_new : p.k_new) + static_cast<size_t>(bh) * D + d0;
  T fresh{}, old{};
  if (mine) {
    fresh = src[tid];
    old = ring[tid];
  }
  if (n_mid < 0) {   // the window is still filling: nothing leaves it
    if (mine) ring[tid] = fresh;
    return;
  }

  const int Dc = is_v ? p.Dvc : p.Dkc, Du = D - Dc, M = p.M;
  const uint8_t* mask = (is_v ? p.vmask : p.kmask) + static_cast<size_t>(bh) * D;
  float* C = (is_v ? p.cv : p.ck) + static_cast<size_t>(bh) * M * Dc;

  // ranks of the dims: every wave reads the whole mask row
  uint8_t mb[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) mb[j] = mask[min(lane + 64 * j, D - 1)];
  uint64_t bal[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) bal[j] = __ballot(mb[j] != 0 && lane + 64 * j < D);
  // compressed dims in front of the slice, and the slice's own bits (a slice never straddles a ballot word)
  const int w0 = d0 >> 6, o0 = d0 & 63;
  int cb = 0;
  uint64_t bits = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {   // static indices only: the words stay in registers
    cb += __popcll(bal[j] & ((j < w0) ? ~0ull : ((j == w0) ? ((1ull << o0) - 1ull) : 0ull)));
    if (j == w0) bits = (bal[j] >> o0) & (~0ull >> (64 - kADims));
  }
  const int nc = min(__popcll(bits), max(Dc - cb, 0));   // (nothing past column Dc, whatever the mask holds)

  // columns [cb, cb + nc) of C: kADims lanes a row
  const int col = tid & (kADims - 1), r0 = tid / kADims;
  constexpr int kRowsPass = kABlock / kADims;
  const bool live = col < nc;
  float* dst = C + cb + min(col, max(nc - 1, 0));
  float cv[kAFly];
  auto load = [&](int m0) {
#pragma unroll
    for (int i = 0; i < kAFly; ++i)
      cv[i] = dst[static_cast<size_t>(min(m0 + r0 + i * kRowsPass, M - 1)) * Dc];
  };
  if (nc > 0) load(0);

  if (mine) {
    ring[tid] = fresh;
    const int below = __popcll(bits & ((1ull << tid) - 1ull));
    if ((bits >> tid) & 1u) {
      xc[below] = Elem<T>::load(&old);
    } else {   // kept dims: appended at middle position n_mid
      const int cp = d0 + tid - cb - below;
      if (is_v) {   // [ceil(n/8), Du, 8]
        T* keep = static_cast<T*>(p.v_keep) + bh * p.vk_stride;
        keep[(static_cast<int64_t>(n_mid >> 3) * Du + cp) * 8 + (n_mid & 7)] = old;
      } else {      // [n, Du rounded up to 8]
        T* keep = static_cast<T*>(p.k_keep) + bh * p.kk_stride;
        keep[static_cast<int64_t>(n_mid) * ((Du + 7) & ~7) + cp] = old;
      }
    }
  }
  if (d0 == 0 && !is_v && Du > 0) {   // zero pad columns of the new K^mu row
    const int kp = (Du + 7) & ~7;
    T* keep = static_cast<T*>(p.k_keep) + bh * p.kk_stride;
    if (tid < kp - Du) keep[static_cast<int64_t>(n_mid) * kp + Du + tid] = T{};
  }
  if (nc == 0) return;   // (uniform over the workgroup)
  for (int n = tid; n <= M / 2; n += kABlock) {   // row 0: the constant; rows 2n - 1, 2n: cosine, sine of order n
    float c = 1.0f, s = 0.0f;
    if (n > 0) {
      unit_phase(n, n_mid, p.T, &c, &s);
      phi[2 * n - 1] = c;
      phi[2 * n] = s;
    } else {
      phi[0] = 1.0f;
    }
  }
  __syncthreads();
  const float x = live ? xc[col] : 0.0f;
  for (int m0 = 0; m0 < M; m0 += kAFly * kRowsPass) {
    if (m0 > 0) load(m0);
#pragma unroll
    for (int i = 0; i < kAFly; ++i) {
      const int m = m0 + r0 + i * kRowsPass;
      if (live && m < M) dst[static_cast<size_t>(m) * Dc] = cv[i] + phi[m] * x;
    }
  }
}

// Head dims per workgroup.  Narrow slices are more workgroups, which few pairs need; wide ones read whole lines of C and evaluate
// the basis column fewer times, and are no better where the head does not fill them.  By the number of narrow ones, over 2700 drawn calls
// and a sweep (head dims 8 - 256, 1 - 2048 pairs, M up to 1023), time against slices of 16: 32 dims 1.1 at 768 workgroups, 0.95 (0.8 - 1.18)
// at 1024 - 1400, 0.83 at 1400 - 1700; 64 dims 0.95 at 2048 (32 there: 0.77), 0.71 at 2560 - 3072 (0.72), 0.48 at 4096 (0.63).  Head dim 8
// in slices of 32 or 64: 1.3 and 1.9 throughout.
// 224 pairs, D = 256, M = 292: 95 / 66 / 59 us; 128, D = 128, M = 128: 11.2 / 9.9 / 10.0; 8, D = 128, M = 1023: 10.8 / 15 / 26.
static int append_dims(int pairs, int D) {
  const long narrow = 2l * pairs * ((D + 15) / 16);
  return D > 32 && narrow >= 2560 ? 64 : D > 16 && narrow >= 1400 ? 32 : 16;
}

}  // namespace fa

static int append_impl(const void* k_new, const void* v_new, int dtype, int B, int Hkv, int D,
                       void* k_full, void* v_full, int W, int64_t full_stride_bh, int slot, int evict,
                       const uint8_t* kmask, int Dkc, const uint8_t* vmask, int Dvc, int M, int T,
                       int n_mid, float* ck, float* cv, void* k_keep, int64_t kk_stride_bh,
                       void* v_keep, int64_t vk_stride_bh, void* hip_stream, const int32_t* seq_slot,
                       const int32_t* seq_nmid, int n_cap) {
  using namespace fa;
  if (dtype != FA_F32 && dtype != FA_BF16) return FA_ERR_UNSUPPORTED;
  if (B <= 0 || Hkv <= 0 || D <= 0 || W <= 0 || slot < 0 || slot >= W) return FA_ERR_SHAPE;
  if (D % 8 != 0 || D > FA_MAX_HEAD_DIM || static_cast<long>(B) * Hkv > 65535) return FA_ERR_UNSUPPORTED;
  if (!k_new || !v_new || !k_full || !v_full) return FA_ERR_NULL;
  if (full_stride_bh == 0) full_stride_bh = static_cast<int64_t>(W) * D;
  if (full_stride_bh < static_cast<int64_t>(W) * D) return FA_ERR_SHAPE;
  AppendParams p{};
  p.k_new = k_new; p.v_new = v_new; p.k_full = k_full; p.v_full = v_full;
  p.full_stride = full_stride_bh; p.B = B; p.Hkv = Hkv; p.D = D; p.W = W; p.slot = slot;
  p.seq_slot = seq_slot; p.seq_nmid = seq_nmid; p.n_cap = n_cap; p.T = T;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  const hipError_t prior = hipPeekAtLastError();
  if (evict) {
    if (Dkc < 0 || Dkc > D || Dvc < 0 || Dvc > D) return FA_ERR_SHAPE;
    if (M < 1 || T < 1 || M > T || n_mid < 0 || n_mid >= T) return FA_ERR_SHAPE;
    if (M > FA_MAX_STATES) return FA_ERR_UNSUPPORTED;
    if (!kmask || !vmask) return FA_ERR_NULL;
    if ((Dkc > 0 && !ck) || (Dvc > 0 && !cv) || (Dkc < D && !k_keep) || (Dvc < D && !v_keep)) return FA_ERR_NULL;
    // the slabs hold every token that may be written: n_mid + 1 of them, or the stated capacity
    const int64_t tokens = seq_nmid ? n_cap : n_mid + 1;
    const int64_t kk_dense = tokens * ((D - Dkc + 7) & ~7);
    const int64_t vk_dense = (tokens + 7) / 8 * 8 * (D - Dvc);
    if (kk_stride_bh == 0) kk_stride_bh = kk_dense;
    if (vk_stride_bh == 0) vk_stride_bh = vk_dense;
    if (kk_stride_bh < kk_dense || vk_stride_bh < vk_dense) return FA_ERR_SHAPE;
    p.kmask = kmask; p.vmask = vmask; p.ck = ck; p.cv = cv; p.k_keep = k_keep; p.v_keep = v_keep;
    p.kk_stride = kk_stride_bh; p.vk_stride = vk_stride_bh;
    p.Dkc = Dkc; p.Dvc = Dvc; p.M = M; p.n_mid = n_mid;
  } else {
    p.n_mid = -1;
  }
  const int dims = append_dims(B * Hkv, D);
  const dim3 grid(B * Hkv, 2, (D + dims - 1) / dims);
#define FA_APPEND(T_) \
  if (dims == 16) hipLaunchKernelGGL((append_token<T_, 16>), grid, dim3(kABlock), 0, st, p); \
  else if (dims == 32) hipLaunchKernelGGL((append_token<T_, 32>), grid, dim3(kABlock), 0, st, p); \
  else hipLaunchKernelGGL((append_token<T_, 64>), grid, dim3(kABlock), 0, st, p)
  if (dtype == FA_F32) { FA_APPEND(float); } else { FA_APPEND(bf16_t); }
#undef FA_APPEND
  // only this call's launches are reported: an error an earlier, unrelated HIP call left behind is
  // neither returned nor cleared
  return (hipPeekAtLastError() == hipSuccess || prior != hipSuccess) ? FA_OK : FA_ERR_HIP;
}

extern "C" int fa_append(const void* k_new, const void* v_new, int dtype, int B, int Hkv, int D,
                         void* k_full, void* v_full, int W, int64_t full_stride_bh, int slot, int evict,
                         const uint8_t* kmask, int Dkc, const uint8_t* vmask, int Dvc, int M, int T,
                         int n_mid, float* ck, float* cv, void* k_keep, int64_t kk_stride_bh,
                         void* v_keep, int64_t vk_stride_bh, void* hip_stream) {
  return append_impl(k_new, v_new, dtype, B, Hkv, D, k_full, v_full, W, full_stride_bh, slot, evict, kmask, Dkc,
                     vmask, Dvc, M, T, n_mid, ck, cv, k_keep, kk_stride_bh, v_keep, vk_stride_bh, hip_stream,
                     nullptr, nullptr, 0);
}

extern "C" int fa_append_varlen(const void* k_new, const void* v_new, int dtype, int B, int Hkv, int D,
                                void* k_full, void* v_full, int W, int64_t full_stride_bh,
                                const int32_t* seq_slot, const uint8_t* kmask, int Dkc, const uint8_t* vmask,
                                int Dvc, int M, int T, const int32_t* seq_nmid, int n_cap, float* ck, float* cv,
                                void* k_keep, int64_t kk_stride_bh, void* v_keep, int64_t vk_stride_bh,
                                void* hip_stream) {
  if (!seq_slot || !seq_nmid) return FA_ERR_NULL;
  if (n_cap < 1 || n_cap > T) return FA_ERR_SHAPE;
  return append_impl(k_new, v_new, dtype, B, Hkv, D, k_full, v_full, W, full_stride_bh, 0, 1, kmask, Dkc, vmask,
                     Dvc, M, T, 0, ck, cv, k_keep, kk_stride_bh, v_keep, vk_stride_bh, hip_stream, seq_slot,
                     seq_nmid, n_cap);
}
