// The split path's x_proj (with the conv in front) and out_proj for small
// batches, where the row panels' serial walk over K sets the time: a few
// hundred rows are a handful of 128-row workgroups, each taking K's chunks one
// after another on one CU, loads, conversions and MFMAs. Here a workgroup owns
// 32 rows and its wavefronts take one 64-wide chunk of K each, W's fragments
// straight from memory into registers. Only the MFMAs stay in K's order: the
// accumulators go from wavefront to wavefront through LDS, the second column
// block a step behind the first, so every sum is that of the panel kernels
// (gemm_split.hip, gemm_f16s.hip), bit for bit.
//
// Bound by latency: a launch, one chunk's loads and conversions, the chain of
// MFMAs. 8 programs of up to 25 tokens, d 256: conv + x_proj 28.6 -> 15.0 us, out_proj
// 20.2 -> 14.4; 64 programs, d 64: 11.3 -> 8.7, 9.7 -> 7.7.
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace tcl {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kRows = 32;                     // rows per workgroup
constexpr int kCW = 64;                       // k per wavefront
constexpr int kNS = kCW / 16;                 // MFMA k-steps per wavefront
constexpr int kCols = 64;                     // columns per workgroup
constexpr int kPA = kCW + 4;                  // fp32 pitch of a parked row (conflict-free 16-byte reads)
constexpr uint32_t kOutOfRange = 0x80000000u;  // beyond every resource used here

__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// x[0..7] -> the three bf16 parts of each (exact: split3_pair)
__device__ __forceinline__ void split8(const float* x, bf16x8& p1, bf16x8& p2, bf16x8& p3) {
  u32x4 a, b, c;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t h, m, l;
    split3_pair(x[2 * i], x[2 * i + 1], h, m, l);
    a[i] = h;
    b[i] = m;
    c[i] = l;
  }
  p1 = __builtin_bit_cast(bf16x8, a);
  p2 = __builtin_bit_cast(bf16x8, b);
  p3 = __builtin_bit_cast(bf16x8, c);
}

// A column block's accumulators as the wavefront before handed them on (the
// first one finds the zeros it handed itself: no condition on the reads).
__device__ __forceinline__ floatx16 take(const float* sP, int lane) {
  floatx16 a;
#pragma unroll
  for (int r = 0; r < 16; ++r) a[r] = sP[r * 64 + lane];
  return a;
}
__device__ __forceinline__ void hand(float* sP, int lane, const floatx16& a) {
#pragma unroll
  for (int r = 0; r < 16; ++r) sP[r * 64 + lane] = a[r];
}

// u = SiLU(conv) and xdbl = u W^T of 32 rows, wavefront w taking channels
// 64 w .. 64 w + 63 (gemm_split32conv_kernel's conv, row by row the same)
template <int KCH, bool XB>
__global__ __launch_bounds__(KCH * 64) void small_conv_kernel(GemmArgs p, ConvIn cv, const uint16_t* Ws, int ldws) {
  constexpr int XR = kRows + 3;
  __shared__ __attribute__((aligned(16))) float sA[KCH * kRows * kPA];
  __shared__ float sP[2][16 * 64];
  const int tid = threadIdx.x;
  const int c = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int li = lane & 31, lg = lane >> 5;
  const int M = p.Mdev ? *p.Mdev : p.Mmax;
  const int row0 = blockIdx.x * kRows;
  if (row0 >= M) return;
  const int E = p.K;

  int tp = 3;
  if (lane < 32 && row0 + lane < M) tp = min((int)cv.tpos[row0 + lane], 3);
  const int xr0 = max(row0 - 3, 0);
  const int xrows = min(M, row0 + kRows) - xr0;
  const int64_t ld = XB ? 64 : cv.ldx;
  const __amdgpu_buffer_rsrc_t xres =
      raw_rsrc(cv.x + (XB ? ((int64_t)c * cv.xblk_rows + xr0) * 64 : (int64_t)xr0 * ld + c * kCW),
               (uint32_t)(((xrows - 1) * ld + kCW) * 4));
  uint32_t xw[XR];
#pragma unroll
  for (int i = 0; i < XR; ++i) {
    const int row = row0 - 3 + i;  // rows before the first and past the last read zero
    const uint32_t off = row >= 0 && row < xr0 + xrows ? (uint32_t)((row - xr0) * ld + lane) * 4u : kOutOfRange;
    xw[i] = __builtin_amdgcn_raw_buffer_load_b32(xres, off, 0, 0);
  }
  const int e = c * kCW + lane;
  const floatx4 cw = *reinterpret_cast<const floatx4*>(cv.w + (int64_t)e * 4);
  const float bias = cv.b[e];
  // W's fragments of this chunk: row n = 32 nb + l % 32, k = 16 ks + 8 (l / 32)
  const __amdgpu_buffer_rsrc_t wres = raw_rsrc(Ws, (uint32_t)(3 * p.N * ldws * 2));
  u32x4 wf[2][3][kNS];
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int part = 0; part < 3; ++part)
#pragma unroll
      for (int ks = 0; ks < kNS; ++ks) {
        const int n = nb * 32 + li, k = c * kCW + 16 * ks + 8 * lg;
        wf[nb][part][ks] = __builtin_amdgcn_raw_buffer_load_b128(
            wres, n < p.N ? (uint32_t)(((part * p.N + n) * ldws + k) * 2) : kOutOfRange, 0, 0);
      }

  const uint32_t p0 = (uint32_t)__builtin_amdgcn_readfirstlane(tp);
  const uint32_t starts = (uint32_t)__builtin_amdgcn_ballot_w64(lane >= 1 && lane < 32 && tp == 0);
  // the rows before the first row that lie in an earlier program
  if (p0 < 3) xw[0] = 0u;
  if (p0 < 2) xw[1] = 0u;
  if (p0 < 1) xw[2] = 0u;
  float* mine = &sA[c * kRows * kPA];
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    // row r starts a program: the three rows before it are no longer anyone's taps
    if (r > 0 && ((starts >> r) & 1u)) xw[r] = xw[r + 1] = xw[r + 2] = 0u;
    float a = bias;
    a = fmaf(cw.x, __uint_as_float(xw[r]), a);
    a = fmaf(cw.y, __uint_as_float(xw[r + 1]), a);
    a = fmaf(cw.z, __uint_as_float(xw[r + 2]), a);
    a = fmaf(cw.w, __uint_as_float(xw[r + 3]), a);
    mine[r * kPA + lane] = silu(a);
  }
  wave_lds_order();
  {
    const __amdgpu_buffer_rsrc_t ures =
        raw_rsrc(cv.u + (int64_t)row0 * E, (uint32_t)(min(kRows, M - row0) * E * 4));
#pragma unroll
    for (int i = 0; i < kRows / 4; ++i) {
      const int r = 4 * i + (lane >> 4), k = 4 * (lane & 15);
      const u32x4 v = *reinterpret_cast<const u32x4*>(&mine[r * kPA + k]);
      __builtin_amdgcn_raw_buffer_store_b128(v, ures, (uint32_t)(r * E + c * kCW + k) * 4u, 0, 0);
    }
  }
  bf16x8 a1[kNS], a2[kNS], a3[kNS];
#pragma unroll
  for (int ks = 0; ks < kNS; ++ks) {
    const float* ap = &mine[li * kPA + 16 * ks + 8 * lg];
    float x[8];
    *reinterpret_cast<floatx4*>(x) = *reinterpret_cast<const floatx4*>(ap);
    *reinterpret_cast<floatx4*>(x + 4) = *reinterpret_cast<const floatx4*>(ap + 4);
    split8(x, a1[ks], a2[ks], a3[ks]);
  }
  // the chunk's MFMAs on column block nb, the panel's order of part products
  const __amdgpu_buffer_rsrc_t cres =
      raw_rsrc(p.C + (int64_t)row0 * p.ldc, (uint32_t)(min(kRows, M - row0) * p.ldc * 4));
  auto chain = [&](auto NB) {
    constexpr int nb = decltype(NB)::value;
    floatx16 acc = take(sP[nb], lane);
#pragma unroll
    for (int ks = 0; ks < kNS; ++ks) {
      const bf16x8 w0 = __builtin_bit_cast(bf16x8, wf[nb][0][ks]), w1 = __builtin_bit_cast(bf16x8, wf[nb][1][ks]),
                   w2 = __builtin_bit_cast(bf16x8, wf[nb][2][ks]);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a3[ks], w0, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a2[ks], w1, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[ks], w2, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a2[ks], w0, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[ks], w1, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[ks], w0, acc, 0, 0, 0);
    }
    if (c < KCH - 1) {
      hand(sP[nb], lane, acc);
    } else {
      const int col = nb * 32 + li;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int rl = 8 * (r >> 2) + 4 * lg + (r & 3);
        const float v = acc[r];
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), cres,
                                              col < p.N ? (uint32_t)((rl * p.ldc + col) * 4) : kOutOfRange, 0, 0);
      }
    }
  };
  if (c == 0) {
    floatx16 none;
#pragma unroll
    for (int r = 0; r < 16; ++r) none[r] = 0.f;
    hand(sP[0], lane, none);
    hand(sP[1], lane, none);
  }
  for (int step = 0; step <= KCH; ++step) {  // wavefront-uniform branches, every wavefront at every barrier
    if (step == c) chain(std::integral_constant<int, 0>{});
    if (step == c + 1) chain(std::integral_constant<int, 1>{});
    __syncthreads();
  }
}

// 2^e as a float, e in [-126, 127]; floor(log2(x)) of a positive normal float
__device__ __forceinline__ float pow2f(int e) { return __uint_as_float((uint32_t)(e + 127) << 23); }
__device__ __forceinline__ int exponent_of(float x) { return (int)((__float_as_uint(x) >> 23) & 0xFF) - 127; }

// C (=|+=) A W^T (+ bias) on two-part fp16 operands with unscaled low parts:
// gemm_f16acc_kernel's 128-wide chunks of K, two wavefronts each, under its
// running power-of-two row scale. 32 rows x 64 columns per workgroup.
template <int KCH, int FL>
__global__ __launch_bounds__(KCH * 64) void small_f16acc_kernel(GemmArgs p, const uint16_t* Wh, int ldwh) {
  __shared__ float sP[2][16 * 64];
  __shared__ float sM[KCH][32];
  const int tid = threadIdx.x;
  const int c = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int li = lane & 31, lg = lane >> 5;
  const int M = p.Mdev ? *p.Mdev : p.Mmax;
  const int row0 = blockIdx.x * kRows, cb = blockIdx.y * kCols;
  if (row0 >= M) return;

  const int grow = row0 + li;
  const bool rok = grow < M;
  const float* arow = p.A + (rok ? (int64_t)grow * p.lda : 0);
  float x[kNS][8];
  float mx = 0.f;
#pragma unroll
  for (int s = 0; s < kNS; ++s) {
    const int k = c * kCW + 16 * s + 8 * lg;
    const bool ok0 = rok && k < p.K, ok1 = rok && k + 4 < p.K;
    const floatx4 v0 = *reinterpret_cast<const floatx4*>(arow + (ok0 ? k : 0));
    const floatx4 v1 = *reinterpret_cast<const floatx4*>(arow + (ok1 ? k + 4 : 0));
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      x[s][j] = ok0 ? v0[j] : 0.f;
      x[s][4 + j] = ok1 ? v1[j] : 0.f;
    }
  }
  const __amdgpu_buffer_rsrc_t wres = raw_rsrc(Wh, (uint32_t)(2 * p.N * ldwh * 2));
  u32x4 wf[2][2][kNS];
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int part = 0; part < 2; ++part)
#pragma unroll
      for (int ks = 0; ks < kNS; ++ks) {
        const int n = cb + nb * 32 + li, k = c * kCW + 16 * ks + 8 * lg;
        wf[nb][part][ks] = __builtin_amdgcn_raw_buffer_load_b128(
            wres, n < p.N && k < ldwh ? (uint32_t)(((part * p.N + n) * ldwh + k) * 2) : kOutOfRange, 0, 0);
      }
  // the last wavefront finishes the rows: its residuals are in flight from here
  const uint32_t rows_bytes = (uint32_t)(min(kRows, M - row0) * p.ldc * 4);
  const __amdgpu_buffer_rsrc_t cres = raw_rsrc(p.C + (int64_t)row0 * p.ldc, rows_bytes);
  const __amdgpu_buffer_rsrc_t rres =
      raw_rsrc((p.R ? p.R : p.C) + (int64_t)row0 * p.ldc, (FL & kResid) != 0 ? rows_bytes : 0);
  float res[2][16];
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      res[nb][r] = 0.f;
      if constexpr ((FL & kResid) != 0) {
        const int col = cb + nb * 32 + li, rl = 8 * (r >> 2) + 4 * lg + (r & 3);
        const uint32_t off = c == KCH - 1 && col < p.N ? (uint32_t)((rl * p.ldc + col) * 4) : kOutOfRange;
        res[nb][r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rres, off, 0, 0));
      }
    }

#pragma unroll
  for (int s = 0; s < kNS; ++s)
#pragma unroll
    for (int j = 0; j < 8; ++j) mx = fmaxf(mx, fabsf(x[s][j]));
  mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
  if (lane < 32) sM[c][lane] = mx;
  __syncthreads();
  // the row's running scale up to this chunk of 128, and up to the one before
  int erun = 100, eold = 100;
#pragma unroll
  for (int q = 0; q < (KCH + 1) / 2; ++q) {
    const float m = fmaxf(sM[2 * q][li], 2 * q + 1 < KCH ? sM[2 * q + 1 < KCH ? 2 * q + 1 : 0][li] : 0.f);
    const int ec = m > 0.f ? min(14 - exponent_of(m), 100) : 100;
    if (q <= c / 2) erun = min(erun, ec);
    if (q < c / 2) eold = min(eold, ec);
  }
  const float sc = pow2f(erun);
  const int dlt = erun - eold;  // <= 0
  f16x8 ah[kNS], al[kNS];
#pragma unroll
  for (int ks = 0; ks < kNS; ++ks)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float v = x[ks][j] * sc;
      ah[ks][j] = (_Float16)v;
      al[ks][j] = (_Float16)(v - (float)ah[ks][j]);
    }
  // row 8 (r / 4) + 4 lg + r % 4 of an accumulator: its exponents are held by
  // the lane of that row
  float fs[16], fr[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int rl = 8 * (r >> 2) + 4 * lg + (r & 3);
    fs[r] = pow2f(max(__shfl(dlt, rl, 64), -126));
    fr[r] = pow2f(-(__shfl(erun, rl, 64) + kF16WeightExp));
  }
  const bool rescale = c > 0 && c % 2 == 0;  // the first wavefront of a later chunk of 128
  auto chain = [&](auto NB) {
    constexpr int nb = decltype(NB)::value;
    floatx16 acc = take(sP[nb], lane);
    if (rescale) {
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] *= fs[r];
    }
#pragma unroll
    for (int ks = 0; ks < kNS; ++ks) {  // the small part products first, the large last
      const f16x8 w0 = __builtin_bit_cast(f16x8, wf[nb][0][ks]), w1 = __builtin_bit_cast(f16x8, wf[nb][1][ks]);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(al[ks], w0, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah[ks], w1, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah[ks], w0, acc, 0, 0, 0);
    }
    if (c < KCH - 1) {
      hand(sP[nb], lane, acc);
    } else {
      const int col = cb + nb * 32 + li;
      const float bias = (FL & kBias) != 0 ? p.bias[col < p.N ? col : 0] : 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int rl = 8 * (r >> 2) + 4 * lg + (r & 3);
        float v = fmaf(acc[r], fr[r], bias + res[nb][r]);
        if (p.relu) v = fmaxf(v, 0.f);
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), cres,
                                              col < p.N ? (uint32_t)((rl * p.ldc + col) * 4) : kOutOfRange, 0, 0);
      }
    }
  };
  if (c == 0) {
    floatx16 none;
#pragma unroll
    for (int r = 0; r < 16; ++r) none[r] = 0.f;
    hand(sP[0], lane, none);
    hand(sP[1], lane, none);
  }
  for (int step = 0; step <= KCH; ++step) {  // wavefront-uniform branches, every wavefront at every barrier
    if (step == c) chain(std::integral_constant<int, 0>{});
    if (step == c + 1) chain(std::integral_constant<int, 1>{});
    __syncthreads();
  }
}

template <int FL>
hipError_t launch_small_acc(const GemmArgs& a, const uint16_t* Wh, int ldwh, hipStream_t s) {
  const dim3 grid((a.Mmax + kRows - 1) / kRows, (a.N + kCols - 1) / kCols);
#define TCL_SMALL(KCH)                                                                                     \
  case KCH: hipLaunchKernelGGL((small_f16acc_kernel<KCH, FL>), grid, dim3(KCH * 64), 0, s, a, Wh, ldwh); break
  switch ((a.K + kCW - 1) / kCW) {
    TCL_SMALL(1);
    TCL_SMALL(2);
    TCL_SMALL(4);
    TCL_SMALL(8);
    default: return hipErrorInvalidValue;
  }
#undef TCL_SMALL
  return hipGetLastError();
}

}  // namespace

// Up to 16,384 padded rows, 512 workgroups: at K = 512 two of them fit on a CU, and a
// third round costs more than the panels' chain, one panel a CU up to 32,768
// rows. Measured, us a launch against the panels, by padded rows with every length 25 (in
// brackets 5 to 25): K = 512 -14 (-15) at 6,400, +1.5 (-12) at 12,800, -2 (-2) at 16,384,
// +7 (-2) at 18,432, +16 (-3) at 25,600; K = 256 -3 (-6) at 10,000, -2 (-1) at 16,384,
// +6 (0) at 20,000, +6 (-2) at 24,500; K = 128 -1 (-2.5) at 10,000, 0 (0) at 15,000, +1 (0)
// at 20,000; K = 64 -0.4 at 10,000, 0.2 at 15,000 and 18,000.
bool small_conv_wanted(const GemmArgs& a) {
  const int ch = a.K / kCW;
  return a.Mmax <= 16384 && a.K % kCW == 0 && (ch == 1 || ch == 2 || ch == 4 || ch == 8);
}

hipError_t launch_small_conv(const GemmArgs& a, const ConvIn& cv, const uint16_t* Ws, int ldws, hipStream_t s) {
  const int grid = (a.Mmax + kRows - 1) / kRows;
  if (grid <= 0) return hipSuccess;
#define TCL_SMALL(KCH)                                                                                            \
  case KCH:                                                                                                       \
    if (cv.xblk_rows > 0)                                                                                         \
      hipLaunchKernelGGL((small_conv_kernel<KCH, true>), dim3(grid), dim3(KCH * 64), 0, s, a, cv, Ws, ldws);       \
    else                                                                                                          \
      hipLaunchKernelGGL((small_conv_kernel<KCH, false>), dim3(grid), dim3(KCH * 64), 0, s, a, cv, Ws, ldws);      \
    break
  switch (a.K / kCW) {
    TCL_SMALL(1);
    TCL_SMALL(2);
    TCL_SMALL(4);
    TCL_SMALL(8);
    default: return hipErrorInvalidValue;
  }
#undef TCL_SMALL
  return hipGetLastError();
}

// Up to 416 workgroups of 32 x 64, by padded rows: with full lengths the second
// workgroup on a CU (from 256) costs what shorter ones gain up to there. Measured,
// us a launch against the panels, every length 25 (in brackets 5 to 25): K = 512, N =
// 256 -8 (-6) at 200 workgroups, +4 (-7) at 312, +3 (-8) at 412, +5 (+4) at 500; K = 256, N = 128
// -2 (-3) at 188, 0 (-2) at 312, -1 (+1) at 412, +5 (-1) at 626; K = 128, N = 128 -1 (-1) at 188, +2 (-1)
// at 312, +2 (+1.5) at 412; K = 128, N = 64 -2 at 250, 0 (-1) at 416, +1.5 (0) at 625.
bool small_f16acc_wanted(const GemmArgs& a) {
  const int ch = (a.K + kCW - 1) / kCW;
  return (int64_t)a.Mmax * a.N <= 416 * kRows * kCols && (ch == 1 || ch == 2 || ch == 4 || ch == 8);
}

hipError_t launch_small_f16acc(const GemmArgs& a, const uint16_t* Wh, int ldwh, int flags, hipStream_t s) {
  if (a.Mmax <= 0) return hipSuccess;
  switch (flags) {
    case 0: return launch_small_acc<0>(a, Wh, ldwh, s);
    case kBias: return launch_small_acc<kBias>(a, Wh, ldwh, s);
    case kResid: return launch_small_acc<kResid>(a, Wh, ldwh, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace tcl
