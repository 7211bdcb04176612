// bf16 MFMA GEMM for a few activation rows (a decode step's block rows, the
// head's): C[m, n] = sum_k X[m, k] W[n, k], M <= kRowsMax.
//
// Bound by reading the weights once.  With the 256-wide tiles of k_gemm.hip
// the layer's matrices make 32 to 148 workgroups: too few CUs pull on HBM
// (2.5 TB/s), and most of a tile is padding.  Here a workgroup takes all M
// activation rows and 32 WN weight rows, WN chosen so that the workgroups
// come out close below the CU count.  WN waves hold 32 weight rows each
// (2 x NB MFMA 16x16x32 tiles); where WN is small, WK such sets take every
// WK-th 64-wide K step and their sums are added in order at the end.
//
// Both operands are copied to LDS, 8 whole 128-byte rows an instruction
// (straight from memory into MFMA operands a lane's 16 bytes are a tag lookup
// of their own: 25-35 B/ns per CU, measured, however deep the prefetch), in a
// ring of ST K steps per set: enough in flight per CU (64-140 KB) to cover
// HBM, one wait and, with WN > 1, one barrier per step.  Chunk c (16 B) of row
// r sits at c ^ ((r >> 1) & 7), as in gemm_bf16_w4_kernel.
//
// Where a row of the operands is a multiple of 4 KB, all rows' lines of one K
// step fall on few memory channels; workgroup t then starts kStagger t steps
// into K and wraps around.
//
// Measured (weights not in cache; before = the tiles of k_gemm.hip, us):
//   24576 x 4096   M 32: 82 -> 39, 64: 88 -> 40, 128: 93 -> 49, 256: 90 -> 64
//   12288 x 4096   M 32: 45 -> 23, 64: 46 -> 27, 128: 47 -> 33, 256: 82 -> 58
//   37888 x 3584   M 32: 78 -> 48, 64: 83 -> 50, 128: 87 -> 59, 192: 84 -> 70
//   126464 x 4096  M 32: 233 -> 178 (5.8 TB/s), 128: 256 -> 211, 192: 276 -> 245
// Above 192 rows a wave's registers are full (2 to 5 spilled, 20 to 37 in the
// rotary epilogue): still faster than the tiles there (layers of 4096 columns,
// 224 rows 278 -> 231 us, 256 rows 285 -> 240).
#include <algorithm>
#include <type_traits>

#include "device.h"
#include "internal.h"

namespace acache {

namespace {

constexpr uint32_t kPast = 0xFFFFFFF0u;  // past the end of every operand: copies zeros

struct RowsMap {
  int n_tiles;  // workgroups along the weight rows
  int units;    // 32-row units of the weight in all
  int splits;   // K splits (EPI_PARTIAL)
  int nk;       // 64-wide K steps
  int stagger;  // workgroup t starts stagger * t steps into its K range
};

// First weight row of half `a` (16 rows) of unit u.  The pair epilogues hold
// the first members of 16 pairs in half 0 and their partners (rotary, up
// projection) in half 1.
template <int EPI>
__device__ __forceinline__ int half_row(int u, int a, int F) {
  if constexpr (EPI == EPI_QKV) return (u >> 2) * 128 + (u & 3) * 16 + a * 64;
  else if constexpr (EPI == EPI_SWIGLU) return u * 16 + a * F;
  else return u * 32 + a * 16;
}

__device__ __forceinline__ void store4(bf16* p, const f32x4& v) {
  const bf16x4 o = {(bf16)v[0], (bf16)v[1], (bf16)v[2], (bf16)v[3]};
  *reinterpret_cast<bf16x4*>(p) = o;
}

// Epilogue of 16 activation rows (16 b ..) and one 32-row unit: lane l holds
// activation row l % 16, columns 4 (l / 16) .. + 3 of each half.
template <int EPI>
__device__ __forceinline__ void finish(const GemmParams& p, const RowsMap& rm, int sp, int u, int b, int lane, f32x4 lo,
                                       f32x4 hi) {
  const int m = b * 16 + (lane & 15), q4 = 4 * (lane >> 4);
  if (u >= rm.units || m >= p.M) return;
  if constexpr (EPI == EPI_SWIGLU) {
    // SiLU with the hardware reciprocal, as the large tiles
#pragma unroll
    for (int r = 0; r < 4; ++r) lo[r] = lo[r] * __builtin_amdgcn_rcpf(1.f + __expf(-lo[r])) * hi[r];
    store4((bf16*)p.C + (int64_t)m * p.ldc + u * 16 + q4, lo);
  } else if constexpr (EPI == EPI_QKV) {
    const int col0 = (u >> 2) * 128, d0 = (u & 3) * 16 + q4;
    const bool is_v = col0 >= p.hq_cols + p.hkv_cols;
    bf16* dst;
    if (col0 < p.hq_cols) {
      dst = (bf16*)p.q_out + (int64_t)m * p.hq_cols + col0;
    } else {
      const int64_t slot = p.write_slots[m];
      if (slot < 0 || slot >= p.n_slots) return;
      dst = (bf16*)(is_v ? p.v_pool : p.k_pool) + slot * p.pool_ld +
            (is_v ? col0 - p.hq_cols - p.hkv_cols : col0 - p.hq_cols);
    }
    if (!is_v) {
      const float* rt = p.rope_cs + (int64_t)m * 128 + 2 * d0;
      const f32x4 t0 = *reinterpret_cast<const f32x4*>(rt), t1 = *reinterpret_cast<const f32x4*>(rt + 4);
      const float cs[4] = {t0[0], t0[2], t1[0], t1[2]}, sn[4] = {t0[1], t0[3], t1[1], t1[3]};
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float x1 = lo[r], x2 = hi[r];
        lo[r] = x1 * cs[r] - x2 * sn[r];
        hi[r] = x2 * cs[r] + x1 * sn[r];
      }
    }
    store4(dst + d0, lo);
    store4(dst + d0 + 64, hi);
  } else if constexpr (EPI == EPI_PARTIAL) {
    float* dst = p.P + ((int64_t)sp * p.M + m) * p.N + u * 32 + q4;
    *reinterpret_cast<f32x4*>(dst) = lo;
    *reinterpret_cast<f32x4*>(dst + 16) = hi;
  } else {
    bf16* dst = (bf16*)p.C + (int64_t)m * p.ldc + u * 32 + q4;
    if constexpr (EPI == EPI_ACCUM) {
      const bf16x4 o0 = *reinterpret_cast<const bf16x4*>(dst), o1 = *reinterpret_cast<const bf16x4*>(dst + 16);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        lo[r] += (float)o0[r];
        hi[r] += (float)o1[r];
      }
    }
    store4(dst, lo);
    store4(dst + 16, hi);
  }
}

// Rings of a set of waves, in 64-wide K steps: its activation rows (all waves
// read them, one extra wave copies them) and its weight rows (each wave copies
// and reads its own 32).  A wave's copies complete in issue order, so one wave
// could not run far ahead with the weights, which come from HBM, and stay
// close with the activations, which come from L2; two can.
// nb: 16-row tiles of the activation rows (M <= 16 nb).
struct RowsRing {
  int wk;   // sets of waves along K
  int xst;  // K steps of activation rows
  int wst;  // K steps of weight rows
};
constexpr int kLdsB = 160 * 1024;
constexpr RowsRing rows_ring(int nb, int wn, int s) {
  const int xb = nb * 2048, wb = wn * s * 4096, xst = 3;
  // more sets where that leaves each at least four weight steps
  int wk = 1;
  if (s > 1) wk = 1;
  else if (wn == 1 && 4 * (xst * xb + 4 * wb) <= kLdsB) wk = 4;
  else if (wn <= 2 && 2 * (xst * xb + 4 * wb) <= kLdsB) wk = 2;
  const int wst = (kLdsB / wk - xst * xb) / wb;
  return {wk, xst, wst > 16 ? 16 : wst};
}

template <int NB, int WN, int S>
struct RowsCfg {
  static constexpr RowsRing R = rows_ring(NB, WN, S);
  static constexpr int WK = R.wk, XST = R.xst, WST = R.wst;
  static constexpr int NBW = NB / S;    // 16-row activation tiles of a wave
  static constexpr int kUnits = WN * S;  // 32-row weight units of a workgroup
  static constexpr int kXB = NB * 2048, kWB = kUnits * 4096;
  static constexpr int kSetB = XST * kXB + WST * kWB;
  // copying waves of a set: one, or as many as make five waves in all (with
  // four or fewer the compiler sees 512 registers a wave, keeps the
  // accumulators in AGPRs and moves them around: 10-20% slower)
  static constexpr int NL = (kUnits + 1) * WK >= 5 ? 1 : (5 + WK - 1) / WK - kUnits;
  static constexpr int kXCopies = (2 * NB + NL - 1) / NL;  // of a copying wave, per step
  static constexpr int kThreads = 64 * (kUnits + NL) * WK;
  static_assert(NB % S == 0 && (S == 1 || WK == 1), "wave tiles");
  static_assert(WST >= 2 && (WST - 2) * 4 < 64 && (XST - 2) * kXCopies < 64, "ring depth");
  static_assert(WK == 1 || WK * WN * 2 * NB * 1024 <= WK * kSetB, "reduction space");
};

// S == 1: WN waves of 32 weight rows x all activation rows.  S == 2 (many
// activation rows): 2 WN waves of 64 weight rows x half the activation rows,
// which reads a third less from LDS per MFMA.
template <int EPI, int NB, int WN, int S>
__global__ __launch_bounds__((RowsCfg<NB, WN, S>::kThreads)) void gemm_rows_kernel(GemmParams p, RowsMap rm) {
  using C = RowsCfg<NB, WN, S>;
  constexpr int WK = C::WK, XST = C::XST, WST = C::WST, NBW = C::NBW, UN = C::kUnits;
  __shared__ __attribute__((aligned(1024))) char ring[WK * C::kSetB];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wc = __builtin_amdgcn_readfirstlane(wave % (UN + C::NL));
  const int wk = __builtin_amdgcn_readfirstlane(wave / (UN + C::NL));
  const rsrc_words wres = buffer_words(p.W, (uint32_t)p.N * (uint32_t)p.K * 2u);
  const rsrc_words xres = buffer_words(p.X, (uint32_t)p.M * (uint32_t)p.K * 2u);
  const int K = p.K, items = rm.n_tiles * rm.splits;
  char* const xring = ring + wk * C::kSetB;
  char* const wring = xring + XST * C::kXB;
  const int lrow = lane >> 3, lch = lane & 7;

  // a walk over the K steps of this workgroup's items, in order
  struct Cursor {
    int item, tile, sp, kb, ke, rot, i, n;
  };
  auto open = [&](Cursor& c, int item) __attribute__((always_inline)) {
    c.item = item;
    c.i = 0;
    if (item < items) {
      c.tile = item % rm.n_tiles;
      c.sp = item / rm.n_tiles;
      c.kb = c.sp * rm.nk / rm.splits;
      c.ke = (c.sp + 1) * rm.nk / rm.splits;
      c.rot = (int)((int64_t)c.tile * rm.stagger % (c.ke - c.kb));
      c.n = (c.ke - c.kb + WK - 1) / WK;
    }
  };
  // byte offset along K of the cursor's step for this set; past: none
  auto step_offset = [&](const Cursor& c, bool& in) __attribute__((always_inline)) {
    int j = c.kb + c.i * WK + wk;
    in = c.item < items && j < c.ke;
    j += c.rot;
    if (j >= c.ke) j -= c.ke - c.kb;
    return (uint32_t)j * 128u;
  };

  // Copies move 8 rows an instruction: lane l row l / 8, physical chunk l % 8.
  // Rows past the last unit or the last activation row repeat it.  Steps past
  // the K range of an item or past the last item copy zeros, so that every
  // step has the same number of copies in flight and computes no branch.
  if (wc >= UN) {
    constexpr int XC = C::kXCopies;
    const int x0 = (wc - UN) * XC;  // a wave past the last copy repeats it
    uint32_t xofs[XC];
#pragma unroll
    for (int c = 0; c < XC; ++c) {
      const int e = min(x0 + c, 2 * NB - 1);
      xofs[c] = (uint32_t)(min(8 * e + lrow, p.M - 1) * K + (lch ^ (4 * (e & 1) + (lane >> 4))) * 8) * 2u;
    }
    Cursor ahead, at;
    open(ahead, blockIdx.x);
    open(at, blockIdx.x);
    int xs = 0;  // stage of the next copies
    auto issue = [&]() __attribute__((always_inline)) {
      bool in;
      const uint32_t ko = step_offset(ahead, in);
#pragma unroll
      for (int c = 0; c < XC; ++c)
        dma16_asm(xres, in ? xofs[c] + ko : kPast, xring + xs * C::kXB + min(x0 + c, 2 * NB - 1) * 1024);
      xs = xs + 1 == XST ? 0 : xs + 1;
      if (ahead.item < items && ++ahead.i == ahead.n) open(ahead, ahead.item + gridDim.x);
    };
#pragma unroll
    for (int i = 0; i < XST - 1; ++i) issue();
    auto next = [&]() __attribute__((always_inline)) {  // the barrier before a step, and one after the last
      wait_vm_asm<(XST - 2) * XC>();
      bare_barrier();
      issue();  // into the stage every wave left before this barrier
    };
    next();
    while (at.item < items) {
      for (; at.i < at.n; ++at.i) next();
      open(at, at.item + gridDim.x);
    }
    wait_vm_asm<0>();
    if constexpr (WK > 1) {
      bare_barrier();
      __syncthreads();
    }
    return;
  }

  // weight units wn S .. + S - 1 of the tile, activation tiles wm NBW .. + NBW - 1
  const int wn = wc / S, wm = wc % S;
  const int i16 = lane & 15, g4 = lane >> 4;
  uint32_t wofs[4];
  Cursor ahead, at;
  auto open_ahead = [&](int item) __attribute__((always_inline)) {
    open(ahead, item);
    if (item < items) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int u = min(ahead.tile * UN + wc, rm.units - 1);
        const int row = half_row<EPI>(u, c >> 1, p.N >> 1) + 8 * (c & 1) + lrow;
        wofs[c] = (uint32_t)(row * K + (lch ^ (4 * (c & 1) + (lane >> 4))) * 8) * 2u;
      }
    }
  };
  open_ahead(blockIdx.x);
  open(at, blockIdx.x);
  int ws = 0;
  auto issue = [&]() __attribute__((always_inline)) {
    bool in;
    const uint32_t ko = step_offset(ahead, in);
#pragma unroll
    for (int c = 0; c < 4; ++c)
      dma16_asm(wres, in ? wofs[c] + ko : kPast, wring + ws * C::kWB + (wc * 32 + 8 * c) * 128);
    ws = ws + 1 == WST ? 0 : ws + 1;
    if (ahead.item < items && ++ahead.i == ahead.n) open_ahead(ahead.item + gridDim.x);
  };
#pragma unroll
  for (int i = 0; i < WST - 1; ++i) issue();
  // A step is two units of 32 along K.  Unit 0's MFMAs run while unit 1's
  // fragments are read, and unit 1's while the next step's unit 0 is, which
  // may be the next item's.
  int xr = 0, wr = 0;  // stages of the step read
  bf16x8 wf[2][2 * S], xf[2][NBW];
  auto read = [&](int h) __attribute__((always_inline)) {
    const char* xp = xring + xr * C::kXB + wm * NBW * 2048;
    const char* wp = wring + wr * C::kWB + wn * S * 4096;
    const int co = ((4 * h + g4) ^ (i16 >> 1)) * 16;
#pragma unroll
    for (int a = 0; a < 2 * S; ++a) wf[h][a] = *reinterpret_cast<const bf16x8*>(wp + (a * 16 + i16) * 128 + co);
#pragma unroll
    for (int b = 0; b < NBW; ++b) xf[h][b] = *reinterpret_cast<const bf16x8*>(xp + (b * 16 + i16) * 128 + co);
  };
  // this wave's weight rows of the next step have landed and its LDS reads of
  // the step before are done; with the barrier, in every wave, and so have
  // the activation rows
  auto meet = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((WST - 2) * 4) : "memory");
    bare_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  meet();
  read(0);
  issue();
  while (at.item < items) {
    f32x4 acc[2 * S][NBW];
#pragma unroll
    for (int a = 0; a < 2 * S; ++a)
#pragma unroll
      for (int b = 0; b < NBW; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto mfmas = [&](int h) __attribute__((always_inline)) {
#pragma unroll
      for (int b = 0; b < NBW; ++b)
#pragma unroll
        for (int a = 0; a < 2 * S; ++a)
          acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[h][a], xf[h][b], acc[a][b], 0, 0, 0);
    };
    for (; at.i < at.n; ++at.i) {
      read(1);
      mfmas(0);
      meet();
      xr = xr + 1 == XST ? 0 : xr + 1;
      wr = wr + 1 == WST ? 0 : wr + 1;
      read(0);
      issue();  // into the weight stage of the step before
      mfmas(1);
    }
    if constexpr (WK == 1) {
#pragma unroll
      for (int u = 0; u < S; ++u)
#pragma unroll
        for (int b = 0; b < NBW; ++b)
          finish<EPI>(p, rm, at.sp, at.tile * UN + wn * S + u, wm * NBW + b, lane, acc[2 * u][b], acc[2 * u + 1][b]);
    } else {
      // one item per workgroup here; no copy is in flight when LDS is reused
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
      bare_barrier();
      f32x4* red = reinterpret_cast<f32x4*>(ring);  // [WK][WN * NB][2][64]
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) red[(((wk * WN + wn) * NB + b) * 2 + a) * 64 + lane] = acc[a][b];
      __syncthreads();
      for (int f = wk * WN + wn; f < WN * NB; f += WN * WK) {
        f32x4 lo = red[f * 128 + lane], hi = red[f * 128 + 64 + lane];
#pragma unroll
        for (int w = 1; w < WK; ++w) {
          lo += red[(w * WN * NB + f) * 128 + lane];
          hi += red[(w * WN * NB + f) * 128 + 64 + lane];
        }
        finish<EPI>(p, rm, at.sp, at.tile * WN + f / NB, f % NB, lane, lo, hi);
      }
    }
    open(at, at.item + gridDim.x);
  }
  wait_vm_asm<0>();
}

// odd, and not one of the WN (kStagger == WN puts the workgroups' lines back
// on the same channels: 126,464 x 4096, M 32, WN 4: 0 215 us, 1 178, 4 284,
// 13 178)
constexpr int kStagger = 13;
constexpr int kMinSplitSteps = 4;  // K steps of a split at least
constexpr int kCus = 256;  // workgroups at a time the plan counts on (one per CU)

int rows_nb(int M) {
  const int nb = (M + 15) / 16;
  return nb <= 2 ? 2 : nb <= 4 ? 4 : nb <= 6 ? 6 : nb <= 8 ? 8 : nb <= 12 ? 12 : 16;
}

// S of the kernel, and the largest WN it is built for, at nb activation tiles.
constexpr int rows_s(int nb) { return nb > 8 ? 2 : 1; }
constexpr int rows_wn_max(int nb) { return nb > 12 ? 2 : nb > 8 ? 3 : 6; }

// Units per workgroup and K splits with the least estimated time (us): rounds
// of workgroups x K steps x the larger of a step's HBM share (about 5.3 TB/s
// over the CUs at work, at most what its ring has in flight per 2.3 us for
// one) and its own length (a step's barrier and LDS reads, then its MFMAs:
// fitted to 126,464 x 4096, 0.75 us at 64 rows to 1.16 at 256), and, with
// splits, the fp32 partials written and read back at 6 TB/s.
struct RowsPlan {
  int wn, splits;
  float us;
};
RowsPlan rows_plan(bool partial, int M, int N, int K) {
  const int nb = rows_nb(M), sq = rows_s(nb), units = N / 32, nk = K / 64;
  RowsPlan best = {1, 1, 1e30f};
  for (int wn = 1; wn <= rows_wn_max(nb); ++wn) {
    const RowsRing r = rows_ring(nb, wn, sq);
    const int un = wn * sq, tiles = (units + un - 1) / un;
    const float own = (0.15f + 0.05f * un + 0.05f * nb) * (r.wk > 1 ? 0.75f : 1.f);
    const float flight = r.wk * (r.wst - 1) * un * 4.096f / 2.3f;  // B/ns
    for (int s = 1; s <= (partial ? 16 : 1); ++s) {
      if (s > 1 && (nk / s < kMinSplitSteps || (size_t)s * M * N * 4 > gemm_bf16_sk_ws_bytes())) break;
      const int wgs = tiles * s;
      const float hbm = un * 4.096f / std::min(flight, 5300.f / std::min(wgs, kCus));
      const float us = (float)((wgs + kCus - 1) / kCus) * ((nk + s - 1) / s) * (std::max(hbm, own) + 0.03f) +
                       (partial ? 2.f * s * M * N * 4 / 6e6f : 0.f);
      if (us < best.us) best = {wn, s, us};
    }
  }
  return best;
}

template <int EPI, int NB, int WN>
hipError_t launch(const GemmParams& p, hipStream_t s) {
  using C = RowsCfg<NB, WN, rows_s(NB)>;
  RowsMap rm = {};
  rm.units = p.N / 32;
  rm.n_tiles = (rm.units + C::kUnits - 1) / C::kUnits;
  rm.splits = EPI == EPI_PARTIAL ? p.splits : 1;
  rm.nk = p.K / 64;
  rm.stagger = p.K % 2048 == 0 ? kStagger : 0;
  const int items = rm.n_tiles * rm.splits;
  hipLaunchKernelGGL((gemm_rows_kernel<EPI, NB, WN, rows_s(NB)>), dim3(C::WK == 1 ? std::min(items, kCus) : items),
                     dim3(C::kThreads), 0, s, p, rm);
  return hipGetLastError();
}

template <int EPI, int NB>
hipError_t by_units(int wn, const GemmParams& p, hipStream_t s) {
  switch (wn) {
    case 1: return launch<EPI, NB, 1>(p, s);
    case 2: return launch<EPI, NB, 2>(p, s);
    default: break;
  }
  if constexpr (rows_wn_max(NB) >= 3) {
    if (wn == 3) return launch<EPI, NB, 3>(p, s);
  }
  if constexpr (rows_wn_max(NB) >= 6) {
    switch (wn) {
      case 4: return launch<EPI, NB, 4>(p, s);
      case 5: return launch<EPI, NB, 5>(p, s);
      case 6: return launch<EPI, NB, 6>(p, s);
      default: break;
    }
  }
  return hipErrorInvalidValue;
}

template <int EPI>
hipError_t by_rows(const GemmParams& p, hipStream_t s) {
  const int wn = rows_plan(EPI == EPI_PARTIAL, p.M, p.N, p.K).wn;
  switch (rows_nb(p.M)) {
    case 2: return by_units<EPI, 2>(wn, p, s);
    case 4: return by_units<EPI, 4>(wn, p, s);
    case 6: return by_units<EPI, 6>(wn, p, s);
    case 8: return by_units<EPI, 8>(wn, p, s);
    case 12: return by_units<EPI, 12>(wn, p, s);
    default: return by_units<EPI, 16>(wn, p, s);
  }
}

}  // namespace

int gemm_rows_splits(int M, int N, int K) { return rows_plan(true, M, N, K).splits; }

double gemm_rows_us(int M, int N, int K) { return rows_plan(false, M, N, K).us; }

hipError_t launch_gemm_rows(GemmEpi epi, const GemmParams& p, hipStream_t s) {
  // A narrow product whose tiles leave CUs idle goes through K splits where
  // the caller lends space for the partials (4096 x 12,288 at 128 rows 66 us
  // whole, 37 split with the sum, which costs a launch and what waits for it:
  // 4096 x 4096 at 32 rows 13 whole, 15 split).
  if ((epi == EPI_STORE || epi == EPI_ACCUM) && p.sk_ws && p.N <= 8192 && p.ldc == p.N) {
    const RowsPlan split = rows_plan(true, p.M, p.N, p.K);
    // Above 192 rows the accumulating epilogue waits for the old values of one
    // 16-row tile after the other, 3 us more than a plain store, and the sum is
    // cheap up to 2048 columns (512 x 512 at 193 rows 13.3 whole, 10.3 split;
    // 2048 x 768 16.4 and 12.3; 4096 x 768 at 256 rows 16.5 and 17.0).
    const float sum = epi == EPI_ACCUM && p.M > 192 && p.N <= 2048 ? 3.f : 9.f;
    if (split.splits > 1 && split.us + sum < rows_plan(false, p.M, p.N, p.K).us) {
      GemmParams q = p;
      q.splits = split.splits;
      q.P = p.sk_ws;
      hipError_t e = by_rows<EPI_PARTIAL>(q, s);
      if (e != hipSuccess) return e;
      return epi == EPI_ACCUM
                 ? launch_reduce_residual(p.C, q.P, q.splits, p.M, p.N, nullptr, nullptr, 0.f, s)
                 : launch_reduce_store(p.C, q.P, q.splits, p.M, p.N, s);
    }
  }
  switch (epi) {
    case EPI_STORE: return by_rows<EPI_STORE>(p, s);
    case EPI_ACCUM: return by_rows<EPI_ACCUM>(p, s);
    case EPI_PARTIAL: return by_rows<EPI_PARTIAL>(p, s);
    case EPI_QKV: return by_rows<EPI_QKV>(p, s);
    default: return by_rows<EPI_SWIGLU>(p, s);
  }
}

}  // namespace acache
