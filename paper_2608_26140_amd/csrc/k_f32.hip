// fp32 path of the recompute block.  On gfx950 the fp32 matrix and fp32
// vector peaks are equal (157 TFLOP/s); what the fp32 MFMA (16x16x4, products
// and sums in fp32) saves is operand traffic: a lane's 16-byte loads along the
// contraction feed it as they are, so the small products, the attention and
// the scores need no staging of their operands and split the contraction (or
// the keys) over the waves of a workgroup.  Rotary angles are reduced in
// fp64 so the fp32 outputs stay within a few ulp at any position.
#include <algorithm>
#include <type_traits>

#include "device.h"
#include "internal.h"

namespace acache {

namespace {

// ---------------------------------------------------------------- GEMM  C = X W^T (+ C)
constexpr int TM = 64, TN = 64, TK = 16;

__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ X, const float* __restrict__ W,
                                                       float* __restrict__ C, int64_t ldc, int M, int N,
                                                       int K, int accumulate) {
  __shared__ float sA[TK][TM + 4];
  __shared__ float sB[TK][TN + 4];
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TN;
  float c[4][4] = {};
  // the next K tile is loaded into registers while the current one computes
  float ra[4], rb[4];
  auto load = [&](int k0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int idx = threadIdx.x + i * 256;
      const int r = idx / TK, kk = idx % TK;
      const int m = m0 + r, n = n0 + r, k = k0 + kk;
      ra[i] = (m < M && k < K) ? X[(int64_t)m * K + k] : 0.f;
      rb[i] = (n < N && k < K) ? W[(int64_t)n * K + k] : 0.f;
    }
  };
  load(0);
  for (int k0 = 0; k0 < K; k0 += TK) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int idx = threadIdx.x + i * 256;
      const int r = idx / TK, kk = idx % TK;
      sA[kk][r] = ra[i];
      sB[kk][r] = rb[i];
    }
    __syncthreads();
    if (k0 + TK < K) load(k0 + TK);
#pragma unroll
    for (int kk = 0; kk < TK; ++kk) {
      float av[4], bv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) av[i] = sA[kk][ty + 16 * i];
#pragma unroll
      for (int j = 0; j < 4; ++j) bv[j] = sB[kk][tx + 16 * j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) c[i][j] = fmaf(av[i], bv[j], c[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int m = m0 + ty + 16 * i, n = n0 + tx + 16 * j;
      if (m < M && n < N) {
        float* p = C + (int64_t)m * ldc + n;
        *p = accumulate ? *p + c[i][j] : c[i][j];
      }
    }
}

// ---------------------------------------------------------------- small products
// 16x16x4 fp32 MFMA: lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16]
// and receives D[4 (l / 16) + r][l % 16], r = 0..3.
__device__ __forceinline__ f32x4 mfma16x16x4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
// p[k .. k + 3], zero from k = n on.  VEC: n % 4 == 0, p 16-byte aligned and
// k a multiple of 4, so the four are all in or all out.
template <bool VEC>
__device__ __forceinline__ f32x4 load4(const float* __restrict__ p, int k, int n) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if constexpr (VEC) {
    if (k < n) v = *reinterpret_cast<const f32x4*>(p + k);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (k + i < n) v[i] = p[k + i];
  }
  return v;
}

// A few rows against a few hundred columns: nothing but latency.  One
// workgroup per 16 x 16 outputs, its 8 waves taking every eighth 16-wide
// slice of K (4 MFMAs on two 16-byte loads per lane, all of them in flight),
// their sums added in wave order through LDS.  90 rows, 768 x 256 / 256 x
// 688: 23 / 60 us with the 64 x 64 tiles above (8 to 44 workgroups, K walked
// serially), 4.5 / 5.8 us with this.  It re-reads its operands from L2 once per
// 16 rows, so the larger tiles win where they give every CU one: 512 x 2048 x
// 512 (256 tiles) takes 33 us here and 47 there, 1024 x 2048 x 1024 (512) 116
// and 101.
constexpr int kSmallWaves = 8;
constexpr int kSmallTiles = 256;  // 64 x 64 tiles up to which this kernel is taken

template <bool VEC>
__global__ __launch_bounds__(64 * kSmallWaves) void gemm_f32_small_kernel(const float* __restrict__ X,
                                                                          const float* __restrict__ W,
                                                                          float* __restrict__ C, int64_t ldc, int M,
                                                                          int N, int K, int accumulate) {
  __shared__ f32x4 red[kSmallWaves][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i16 = lane & 15, g = lane >> 4;
  const int n0 = blockIdx.x * 16, m0 = blockIdx.y * 16;
  const float* wr = W + (int64_t)min(n0 + i16, N - 1) * K;
  const float* xr = X + (int64_t)min(m0 + i16, M - 1) * K;
  f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = acc0;
#pragma unroll 4
  for (int k0 = 16 * wave; k0 < K; k0 += 16 * kSmallWaves) {
    const f32x4 a = load4<VEC>(wr, k0 + 4 * g, K);
    const f32x4 b = load4<VEC>(xr, k0 + 4 * g, K);
    acc0 = mfma16x16x4(a[0], b[0], acc0);
    acc1 = mfma16x16x4(a[1], b[1], acc1);
    acc0 = mfma16x16x4(a[2], b[2], acc0);
    acc1 = mfma16x16x4(a[3], b[3], acc1);
  }
  red[wave][lane] = acc0 + acc1;
  __syncthreads();
  if (wave != 0) return;
  f32x4 t = red[0][lane];
#pragma unroll
  for (int w = 1; w < kSmallWaves; ++w) t += red[w][lane];
  const int m = m0 + i16;
  if (m >= M) return;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int n = n0 + 4 * g + r;
    if (n < N) {
      float* p = C + (int64_t)m * ldc + n;
      *p = accumulate ? *p + t[r] : t[r];
    }
  }
}

// ---------------------------------------------------------------- rotary + K/V store
__global__ __launch_bounds__(256) void rope_scatter_f32_kernel(const float* __restrict__ qkv, int H, int Hkv,
                                                               int dh, const int32_t* __restrict__ pos,
                                                               float rope_base, float* __restrict__ q_out,
                                                               const int32_t* __restrict__ wslots,
                                                               float* __restrict__ kp, float* __restrict__ vp,
                                                               int64_t pool_ld, int64_t n_slots) {
  const int64_t m = blockIdx.x;
  const int half = dh / 2;
  const int width = (H + 2 * Hkv) * dh;
  const float* row = qkv + m * width;
  const int64_t slot = wslots[m];
  const bool slot_ok = slot >= 0 && slot < n_slots;
  const double p = (double)pos[m];
  // rotated pairs of the Q and K heads
  for (int c = threadIdx.x; c < (H + Hkv) * half; c += blockDim.x) {
    const int head = c / half, i = c % half;
    const double ang = p * exp2(-(2.0 * i / dh) * log2((double)rope_base));
    double sn, cs;
    sincos(ang, &sn, &cs);
    const float x1 = row[head * dh + i], x2 = row[head * dh + i + half];
    const float o1 = (float)(x1 * cs - x2 * sn), o2 = (float)(x2 * cs + x1 * sn);
    if (head < H) {
      q_out[m * H * dh + head * dh + i] = o1;
      q_out[m * H * dh + head * dh + i + half] = o2;
    } else if (slot_ok) {
      const int kh = head - H;
      kp[slot * pool_ld + kh * dh + i] = o1;
      kp[slot * pool_ld + kh * dh + i + half] = o2;
    }
  }
  if (slot_ok)
    for (int c = threadIdx.x; c < Hkv * dh; c += blockDim.x) vp[slot * pool_ld + c] = row[(H + Hkv) * dh + c];
}

__global__ __launch_bounds__(256) void swiglu_f32_kernel(const float* __restrict__ gu, int M, int F,
                                                         float* __restrict__ h) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)M * F) return;
  const int64_t m = t / F, f = t % F;
  const float g = gu[m * 2 * F + f], u = gu[m * 2 * F + F + f];
  h[t] = g / (1.f + expf(-g)) * u;
}

// ---------------------------------------------------------------- attention
struct RowsArgs {
  int batch;
  int row_start[kMaxBatch + 1];
  int key_start[kMaxBatch + 1];
  int key_len[kMaxBatch + 1];
  int tile_start[kMaxBatch + 1];  // cumulative 16-row tiles
};

__device__ __forceinline__ int request_of(const RowsArgs& a, int tile) {
  int lo = 0, hi = a.batch - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (a.tile_start[mid] <= tile) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// 16 query rows of one head per workgroup; its 8 waves take every eighth tile
// of 16 keys with an online softmax each, merged in wave order through LDS.
// Keys are the MFMA A operand, so a lane holds four logits of one query and
// they are the B operand of the product with V as they stand.  A key whose
// slot is out of range has logit 0 and a zero V row.
// q_rows (nullable): query row i is row q_rows[i] (zeros where it is outside
// [0, q_n_rows)).  LSE_ONLY: no output rows, only their log-sum-exp.
// Latency-bound at the sizes that run in fp32: 90 rows, 4 heads of 64, 192
// keys took 62 us with a wave per row and head that walked its keys one lane
// each, 11 us with this.
constexpr int kAttWaves = 8;

template <int ND, bool VEC, bool LSE_ONLY>
__global__ __launch_bounds__(64 * kAttWaves) void attention_f32_kernel(
    RowsArgs a, int H, int Hkv, int dh, const float* __restrict__ q, int64_t q_ld, int64_t q_n_rows,
    const int32_t* __restrict__ q_rows, const int32_t* __restrict__ read_slots, const float* __restrict__ kp,
    const float* __restrict__ vp, int64_t pool_ld, int64_t n_slots, float* __restrict__ out,
    float* __restrict__ lse) {
  __shared__ float sm[kAttWaves][16], sl[kAttWaves][16];
  __shared__ f32x4 so[LSE_ONLY ? 1 : kAttWaves][LSE_ONLY ? 1 : ND][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i16 = lane & 15, g = lane >> 4;
  const int h = blockIdx.y;
  const int b = request_of(a, blockIdx.x);
  const int row0 = a.row_start[b] + (blockIdx.x - a.tile_start[b]) * 16;
  const int nrow = min(16, a.row_start[b + 1] - row0);
  const int S = a.key_len[b];
  const int32_t* slots = read_slots + a.key_start[b];
  const int64_t koff = (int64_t)(h / (H / Hkv)) * dh;
  const float scale = rsqrtf((float)dh);

  f32x4 qf[ND];
  {
    int64_t r = row0 + min(i16, nrow - 1);
    if (q_rows) r = q_rows[r];
    const bool ok = r >= 0 && r < q_n_rows;
    const float* qr = q + (ok ? r : 0) * q_ld + (int64_t)h * dh;
#pragma unroll
    for (int c = 0; c < ND; ++c) {
      qf[c] = load4<VEC>(qr, 16 * c + 4 * g, dh);
      if (!ok) qf[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  float m = -INFINITY, l = 0.f;  // of query i16 over this wave's keys (l: this lane's share)
  f32x4 o[ND];
#pragma unroll
  for (int c = 0; c < ND; ++c) o[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int t = wave * 16; t < S; t += 16 * kAttWaves) {
    int64_t sl16 = t + i16 < S ? slots[t + i16] : -1;
    if (sl16 < 0 || sl16 >= n_slots) sl16 = -1;
    const float* kr = kp + (sl16 < 0 ? 0 : sl16) * pool_ld + koff;
    f32x4 kf[ND];
#pragma unroll
    for (int c = 0; c < ND; ++c) {
      kf[c] = load4<VEC>(kr, 16 * c + 4 * g, dh);
      if (sl16 < 0) kf[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    float vf[LSE_ONLY ? 1 : ND][4];
    if constexpr (!LSE_ONLY) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int vs = __shfl((int)sl16, 4 * g + r);
        const float* vr = vp + (int64_t)(vs < 0 ? 0 : vs) * pool_ld + koff;
#pragma unroll
        for (int c = 0; c < ND; ++c) vf[c][r] = (vs >= 0 && 16 * c + i16 < dh) ? vr[16 * c + i16] : 0.f;
      }
    }
    f32x4 z0 = {0.f, 0.f, 0.f, 0.f}, z1 = z0;
#pragma unroll
    for (int c = 0; c < ND; ++c) {
      z0 = mfma16x16x4(kf[c][0], qf[c][0], z0);
      z1 = mfma16x16x4(kf[c][1], qf[c][1], z1);
      z0 = mfma16x16x4(kf[c][2], qf[c][2], z0);
      z1 = mfma16x16x4(kf[c][3], qf[c][3], z1);
    }
    float z[4], mt = m;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      z[r] = t + 4 * g + r < S ? (z0[r] + z1[r]) * scale : -INFINITY;
      mt = fmaxf(mt, z[r]);
    }
    mt = fmaxf(mt, __shfl_xor(mt, 16));
    mt = fmaxf(mt, __shfl_xor(mt, 32));
    if (mt > m) {
      const float f = expf(m - mt);
      l *= f;
      if constexpr (!LSE_ONLY) {
#pragma unroll
        for (int c = 0; c < ND; ++c) o[c] *= f;
      }
      m = mt;
    }
    // a query whose logits were all -inf so far: against 0, which gives zeros
    const float m_use = m == -INFINITY ? 0.f : m;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      z[r] = expf(z[r] - m_use);
      l += z[r];
    }
    if constexpr (!LSE_ONLY) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < ND; ++c) o[c] = mfma16x16x4(vf[c][r], z[r], o[c]);
    }
  }
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  if (g == 0) {
    sm[wave][i16] = m;
    sl[wave][i16] = l;
  }
  if constexpr (!LSE_ONLY) {
#pragma unroll
    for (int c = 0; c < ND; ++c) so[wave][c][lane] = o[c];
  }
  __syncthreads();
  // the tile's keys span at least wave 0, so the merged maximum is a logit
  float M = sm[0][i16], L = 0.f;
#pragma unroll
  for (int w = 1; w < kAttWaves; ++w) M = fmaxf(M, sm[w][i16]);
  float f[kAttWaves];
#pragma unroll
  for (int w = 0; w < kAttWaves; ++w) {
    f[w] = expf(sm[w][i16] - M);
    L += sl[w][i16] * f[w];
  }
  if (i16 >= nrow) return;
  const int64_t row = row0 + i16;
  if (lse && wave == 0 && g == 0) lse[row * H + h] = M + logf(L);
  if constexpr (!LSE_ONLY) {
    const float inv = 1.f / L;
    for (int c = wave; c < ND; c += kAttWaves) {
      f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < kAttWaves; ++w) t += so[w][c][lane] * f[w];
      float* op = out + row * H * dh + (int64_t)h * dh;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (16 * c + 4 * g + r < dh) op[16 * c + 4 * g + r] = t[r] * inv;
    }
  }
}

// ---------------------------------------------------------------- probe scores (Eq. 4-5)
// One workgroup per (16 affix keys, head, request); its 8 waves take every
// eighth tile of 16 masked queries.  Queries are the MFMA A operand, so a
// lane holds four queries of one key: it adds their weights, and the lanes of
// a key and then the waves are added in a fixed order.
template <int ND, bool VEC>
__global__ __launch_bounds__(64 * kAttWaves) void score_colsum_f32_kernel(
    RowsArgs a, int H, int Hkv, int dh, const float* __restrict__ q, int64_t q_ld, int64_t q_n_rows,
    const int32_t* __restrict__ q_rows, const float* __restrict__ kp, int64_t pool_ld, int64_t n_slots,
    const int32_t* __restrict__ affix_slots, int L, const float* __restrict__ lse, int lse_by_qrow,
    float* __restrict__ part) {
  __shared__ float red[kAttWaves][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i16 = lane & 15, g = lane >> 4;
  const int h = blockIdx.y, b = blockIdx.z;
  const int j = blockIdx.x * 16 + i16;
  int64_t sl = j < L ? affix_slots[j] : -1;
  if (sl < 0 || sl >= n_slots) sl = -1;
  const float* kr = kp + (sl < 0 ? 0 : sl) * pool_ld + (int64_t)(h / (H / Hkv)) * dh;
  f32x4 kf[ND];
#pragma unroll
  for (int c = 0; c < ND; ++c) kf[c] = load4<VEC>(kr, 16 * c + 4 * g, dh);
  const float scale = rsqrtf((float)dh);
  float acc = 0.f;
  for (int q0 = a.row_start[b] + 16 * wave; q0 < a.row_start[b + 1]; q0 += 16 * kAttWaves) {
    const int qi = q0 + i16;
    int64_t row = qi < a.row_start[b + 1] ? q_rows[qi] : -1;
    if (row < 0 || row >= q_n_rows) row = -1;
    const float* qr = q + (row < 0 ? 0 : row) * q_ld + (int64_t)h * dh;
    // a query that is not there weighs nothing
    const float lq = row < 0 ? INFINITY : lse[(lse_by_qrow ? (int64_t)qi : row) * H + h];
    f32x4 z0 = {0.f, 0.f, 0.f, 0.f}, z1 = z0;
#pragma unroll
    for (int c = 0; c < ND; ++c) {
      const f32x4 qf = load4<VEC>(qr, 16 * c + 4 * g, dh);
      z0 = mfma16x16x4(qf[0], kf[c][0], z0);
      z1 = mfma16x16x4(qf[1], kf[c][1], z1);
      z0 = mfma16x16x4(qf[2], kf[c][2], z0);
      z1 = mfma16x16x4(qf[3], kf[c][3], z1);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float lr = __shfl(lq, 4 * g + r);
      acc += lr == INFINITY ? 0.f : expf((z0[r] + z1[r]) * scale - lr);
    }
  }
  acc += __shfl_xor(acc, 16);
  acc += __shfl_xor(acc, 32);
  if (g == 0) red[wave][i16] = acc;
  __syncthreads();
  if (threadIdx.x < 16 && j < L) {
    float t = red[0][i16];
#pragma unroll
    for (int w = 1; w < kAttWaves; ++w) t += red[w][i16];
    part[((int64_t)b * H + h) * L + j] = sl < 0 ? 0.f : t;
  }
}

RowsArgs rows_args(const int* starts, int batch) {
  RowsArgs a = {};
  a.batch = batch;
  for (int b = 0; b <= batch; ++b) a.row_start[b] = starts[b];
  for (int b = 0; b < batch; ++b) a.tile_start[b + 1] = a.tile_start[b] + (starts[b + 1] - starts[b] + 15) / 16;
  return a;
}

// f(ND, VEC): ND 16-wide slices of a head; VEC: 16-byte loads along it.
template <typename F>
hipError_t by_head_dim(int dh, bool vec, F f) {
  auto go = [&](auto nd) {
    if (vec) f(nd, std::true_type());
    else f(nd, std::false_type());
  };
  switch ((dh + 15) / 16) {
    case 1: go(std::integral_constant<int, 1>()); break;
    case 2: go(std::integral_constant<int, 2>()); break;
    case 3: go(std::integral_constant<int, 3>()); break;
    case 4: go(std::integral_constant<int, 4>()); break;
    case 5: go(std::integral_constant<int, 5>()); break;
    case 6: go(std::integral_constant<int, 6>()); break;
    case 7: go(std::integral_constant<int, 7>()); break;
    case 8: go(std::integral_constant<int, 8>()); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// 16-byte loads along a head of q and of the pools
bool head_vec(int dh, const float* q, int64_t q_ld, const float* kp, int64_t pool_ld) {
  return dh % 4 == 0 && q_ld % 4 == 0 && pool_ld % 4 == 0 && (uintptr_t)q % 16 == 0 && (uintptr_t)kp % 16 == 0;
}

}  // namespace

hipError_t launch_gemm_f32(const float* X, const float* W, float* C, int64_t ldc, int M, int N,
                           int K, int accumulate, hipStream_t s) {
  const int tiles = ((N + TN - 1) / TN) * ((M + TM - 1) / TM);
  if (tiles <= kSmallTiles && (M + 15) / 16 <= 65535) {
    const dim3 grid((N + 15) / 16, (M + 15) / 16), block(64 * kSmallWaves);
    const bool vec = K % 4 == 0 && (uintptr_t)X % 16 == 0 && (uintptr_t)W % 16 == 0;
    if (vec)
      hipLaunchKernelGGL(gemm_f32_small_kernel<true>, grid, block, 0, s, X, W, C, ldc, M, N, K, accumulate);
    else
      hipLaunchKernelGGL(gemm_f32_small_kernel<false>, grid, block, 0, s, X, W, C, ldc, M, N, K, accumulate);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(gemm_f32_kernel, dim3((N + TN - 1) / TN, (M + TM - 1) / TM), dim3(256), 0, s, X,
                     W, C, ldc, M, N, K, accumulate);
  return hipGetLastError();
}

hipError_t launch_rope_scatter_f32(const float* qkv, int M, int H, int Hkv, int dh,
                                   const int32_t* pos, float rope_base, float* q_out,
                                   const int32_t* write_slots, float* k_pool, float* v_pool,
                                   int64_t pool_ld, int64_t n_slots, hipStream_t s) {
  hipLaunchKernelGGL(rope_scatter_f32_kernel, dim3(M), dim3(256), 0, s, qkv, H, Hkv, dh, pos, rope_base,
                     q_out, write_slots, k_pool, v_pool, pool_ld, n_slots);
  return hipGetLastError();
}

hipError_t launch_swiglu_f32(const float* gu, int M, int F, float* h, hipStream_t s) {
  const int64_t n = (int64_t)M * F;
  hipLaunchKernelGGL(swiglu_f32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, gu, M, F, h);
  return hipGetLastError();
}

hipError_t launch_attention_f32(const Ragged& rg, int H, int Hkv, int dh, const float* q,
                                const int32_t* read_slots, const float* k_pool,
                                const float* v_pool, int64_t pool_ld, int64_t n_slots, float* out,
                                float* lse, hipStream_t s) {
  RowsArgs a = rows_args(rg.cu_rows, rg.batch);
  for (int b = 0; b < rg.batch; ++b) {
    a.key_start[b] = rg.cu_keys[b];
    a.key_len[b] = rg.cu_keys[b + 1] - rg.cu_keys[b];
  }
  const int rows = rg.cu_rows[rg.batch];
  if (rows == 0) return hipSuccess;
  const int64_t q_ld = (int64_t)H * dh;
  return by_head_dim(dh, head_vec(dh, q, q_ld, k_pool, pool_ld), [&](auto nd, auto vec) {
    hipLaunchKernelGGL((attention_f32_kernel<decltype(nd)::value, decltype(vec)::value, false>),
                       dim3(a.tile_start[a.batch], H), dim3(64 * kAttWaves), 0, s, a, H, Hkv, dh, q, q_ld,
                       (int64_t)rows, nullptr, read_slots, k_pool, v_pool, pool_ld, n_slots, out, lse);
  });
}

hipError_t launch_score_lse_f32(int batch, const int* cu_q, int H, int Hkv, int dh, const float* q,
                                int64_t q_ld, int64_t q_n_rows, const int32_t* q_rows,
                                const float* k_pool, int64_t pool_ld, int64_t n_slots,
                                const int32_t* affix_slots, int L, float* lse_out, hipStream_t s) {
  const int n = cu_q[batch];
  if (n == 0) return hipSuccess;
  const int all[2] = {0, n};  // every request's queries against the same keys
  RowsArgs a = rows_args(all, 1);
  a.key_len[0] = L;
  return by_head_dim(dh, head_vec(dh, q, q_ld, k_pool, pool_ld), [&](auto nd, auto vec) {
    hipLaunchKernelGGL((attention_f32_kernel<decltype(nd)::value, decltype(vec)::value, true>),
                       dim3(a.tile_start[1], H), dim3(64 * kAttWaves), 0, s, a, H, Hkv, dh, q, q_ld, q_n_rows,
                       q_rows, affix_slots, k_pool, nullptr, pool_ld, n_slots, nullptr, lse_out);
  });
}

hipError_t launch_score_colsum_f32(int batch, const int* cu_q, int H, int Hkv, int dh,
                                   const float* q, int64_t q_ld, int64_t q_n_rows,
                                   const int32_t* q_rows, const float* k_pool, int64_t pool_ld,
                                   int64_t n_slots, const int32_t* affix_slots, int L,
                                   const float* lse, int lse_by_qrow, float* part, hipStream_t s) {
  RowsArgs a = rows_args(cu_q, batch);
  return by_head_dim(dh, head_vec(dh, q, q_ld, k_pool, pool_ld), [&](auto nd, auto vec) {
    hipLaunchKernelGGL((score_colsum_f32_kernel<decltype(nd)::value, decltype(vec)::value>),
                       dim3((L + 15) / 16, H, batch), dim3(64 * kAttWaves), 0, s, a, H, Hkv, dh, q, q_ld, q_n_rows,
                       q_rows, k_pool, pool_ld, n_slots, affix_slots, L, lse, lse_by_qrow, part);
  });
}

}  // namespace acache
