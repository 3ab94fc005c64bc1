// HIP kernels specific to the SOAP owner step (fp32): the first-moment pass that also lays out the
// gradient for the products, Adam in the eigenbasis, and the blocked Householder QR that refreshes
// a basis. The products themselves run on the Shampoo GEMM.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "mfsdp_internal.h"
#include "soap_internal.h"

namespace mfsdp {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) float g_f32;
typedef __attribute__((address_space(1))) const float g_cf32;
typedef __attribute__((address_space(1))) f32x4 g_f32x4;
typedef __attribute__((address_space(1))) const f32x4 g_cf32x4;

constexpr int kTile = kShCopyTile;  // 64 x 64 tiles of the elementwise passes

template <typename D>
__device__ __forceinline__ int find_desc(const D* d, int count, int b) {
  int lo = 0, hi = count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (d[mid].tile_begin <= b) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Compile-time loop: f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>), so that
// register arrays indexed by the loop variable stay in registers.
template <typename F, int... I>
__device__ __forceinline__ void unrolled_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void unrolled(F&& f) {
  unrolled_impl(f, std::make_integer_sequence<int, N>{});
}

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, false));
}

// Sum over the 64 lanes of a wave (all lanes active), the same value in every lane, in a fixed
// order: DPP butterflies within each 16-lane row (quad_perm [1,0,3,2], quad_perm [2,3,0,1],
// row_half_mirror, row_mirror: every lane of a row then holds the row sum; the partners' adds are
// commutative, so all lanes agree bit for bit), then the four row sums read from lanes 0, 16, 32,
// 48 and added in that order.
__device__ __forceinline__ float wave_sum(float x) {
  x += dpp<0xB1>(x);
  x += dpp<0x4E>(x);
  x += dpp<0x141>(x);
  x += dpp<0x140>(x);
  const int xi = __float_as_int(x);
  const float r0 = __int_as_float(__builtin_amdgcn_readlane(xi, 0));
  const float r1 = __int_as_float(__builtin_amdgcn_readlane(xi, 16));
  const float r2 = __int_as_float(__builtin_amdgcn_readlane(xi, 32));
  const float r3 = __int_as_float(__builtin_amdgcn_readlane(xi, 48));
  return ((r0 + r1) + r2) + r3;
}

// Sum of x over the four 16-lane rows of a wave, in every lane of the same column (all lanes
// active): rows 0 + 1 and 2 + 3 by swapping odd and even rows, then the two halves by swapping them
// (v_permlane16_swap, v_permlane32_swap: vector ALU exchanges, no LDS round trip). Each add has the
// same two operands in every lane that forms it, so all lanes of a column agree bit for bit.
__device__ __forceinline__ float sum_rows4(float x) {
  const uint32_t xi = __float_as_uint(x);
  const auto p = __builtin_amdgcn_permlane16_swap(xi, xi, false, false);
  const float y = __uint_as_float(p[0]) + __uint_as_float(p[1]);  // (row 2k) + (row 2k + 1)
  const uint32_t yi = __float_as_uint(y);
  const auto q = __builtin_amdgcn_permlane32_swap(yi, yi, false, false);
  return __uint_as_float(q[0]) + __uint_as_float(q[1]);  // (rows 0, 1) + (rows 2, 3)
}

// Reduce-scatter of 16 values over the 16 lanes of a DPP row (all lanes active): afterwards lane l
// of each row holds that row's sum of value l (l = lane mod 16). Four exchange rounds with the lane
// at distance 1, 2, 4 and 8 (quad_perm [1,0,3,2], quad_perm [2,3,0,1], row_shl/row_shr 4,
// row_ror 8): each lane keeps the half of its values whose index bit matches its own lane bit and
// adds the partner's copy of them; every sum is formed by exactly one lane, in a fixed order.
__device__ __forceinline__ float row_reduce_scatter16(const float (&v)[16], int l16) {
  const bool b0 = l16 & 1, b1 = (l16 >> 1) & 1, b2 = (l16 >> 2) & 1, b3 = (l16 >> 3) & 1;
  float s1[8], s2[4], s3[2];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float keep = b0 ? v[2 * j + 1] : v[2 * j], send = b0 ? v[2 * j] : v[2 * j + 1];
    s1[j] = keep + dpp<0xB1>(send);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float keep = b1 ? s1[2 * j + 1] : s1[2 * j], send = b1 ? s1[2 * j] : s1[2 * j + 1];
    s2[j] = keep + dpp<0x4E>(send);
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const float keep = b2 ? s2[2 * j + 1] : s2[2 * j], send = b2 ? s2[2 * j] : s2[2 * j + 1];
    const float from_up = dpp<0x104>(send);    // row_shl 4: lane l reads lane l + 4
    const float from_down = dpp<0x114>(send);  // row_shr 4: lane l reads lane l - 4
    s3[j] = keep + (b2 ? from_down : from_up);
  }
  const float keep = b3 ? s3[1] : s3[0], send = b3 ? s3[0] : s3[1];
  return keep + dpp<0x128>(send);  // row_ror 8: lane l reads lane l ^ 8
}

__global__ __launch_bounds__(256) void soap_prep_kernel(const SoapPrepDesc* __restrict__ descs, int count,
                                                        float beta1) {
  __shared__ float tg[kTile][kTile + 1];
  __shared__ float tm[kTile][kTile + 1];
  const int e = find_desc(descs, count, blockIdx.x);
  const SoapPrepDesc& d = descs[e];
  const int lt = blockIdx.x - d.tile_begin;
  const int ti = lt / d.tiles_n, tj = lt - ti * d.tiles_n;
  const int t = threadIdx.x, c = t & 63, rr = t >> 6;
  const int64_t gc = int64_t(tj) * kTile + c;
  typedef __attribute__((address_space(1))) uint16_t g_u16;
  g_f32* Gp = (g_f32*)(d.Gp);
  g_f32* GMt = (g_f32*)(d.GMt);
  g_f32* GM = (g_f32*)(d.GM);
  g_f32* Mr = (g_f32*)(d.Mr);
  // G (and G^T) as bf16: the value's upper 16 bits, exact for a bf16 gradient
  auto put_g = [&](g_f32* base, int64_t i, float v) {
    if (d.g_bf16) ((g_u16*)base)[i] = uint16_t(__float_as_uint(v) >> 16);
    else base[i] = v;
  };
#pragma unroll 4
  for (int i = 0; i < 16; ++i) {
    const int r = rr + 4 * i;
    const int64_t gr = int64_t(ti) * kTile + r;
    float g = 0.0f, mo = 0.0f;
    if (gr < d.m && gc < d.n) {
      const int64_t o = gr * d.n + gc;
      g = d.grad_dtype == kDtBF16
              ? __uint_as_float(uint32_t(static_cast<const uint16_t*>(d.grad)[o]) << 16)
              : static_cast<const float*>(d.grad)[o];
      mo = beta1 * d.exp_avg[o] + (1.0f - beta1) * g;
      d.exp_avg[o] = mo;
    }
    if (Gp) put_g(Gp, gr * d.np + gc, g);
    if (Mr) Mr[gr * d.np + gc] = mo;
    if (GM) {
      GM[gr * 2 * d.np + gc] = g;
      GM[gr * 2 * d.np + d.np + gc] = mo;
    }
    tg[r][c] = g;
    tm[r][c] = mo;
  }
  if (!GMt) return;  // (uniform over the workgroup: no barrier is skipped by part of it)
  __syncthreads();
#pragma unroll 4
  for (int i = 0; i < 16; ++i) {
    const int r = rr + 4 * i;  // row of the transposed tile = column of the source tile
    const int64_t o = (int64_t(tj) * kTile + r) * d.mp + int64_t(ti) * kTile + c;
    put_g(GMt, o, tg[c][r]);
    if (!Mr) GMt[o + d.np * d.mp] = tm[c][r];
  }
}

__global__ __launch_bounds__(256) void soap_adam_kernel(const SoapAdamDesc* __restrict__ descs, int count,
                                                        float beta2, float eps, float inv_bc1,
                                                        float inv_sqrt_bc2) {
  __shared__ float tn[kTile][kTile + 1];
  const int e = find_desc(descs, count, blockIdx.x);
  const SoapAdamDesc& d = descs[e];
  const int lt = blockIdx.x - d.tile_begin;
  const int ti = lt / d.tiles_n, tj = lt - ti * d.tiles_n;
  const int t = threadIdx.x, c = t & 63, rr = t >> 6;
  const int64_t gc = int64_t(tj) * kTile + c;
  const g_cf32* GMr = (const g_cf32*)(d.GMr);
#pragma unroll 4
  for (int i = 0; i < 16; ++i) {
    const int r = rr + 4 * i;
    const int64_t gr = int64_t(ti) * kTile + r;
    float np_ = 0.0f;
    if (gr < d.m && gc < d.n) {
      const float gq = GMr[gr * 2 * d.np + gc];
      const float mq = GMr[gr * 2 * d.np + d.np + gc];
      const int64_t o = gr * d.n + gc;
      const float v = beta2 * d.exp_avg_sq[o] + (1.0f - beta2) * (gq * gq);
      d.exp_avg_sq[o] = v;
      np_ = (mq * inv_bc1) / (sqrtf(v) * inv_sqrt_bc2 + eps);
    }
    tn[r][c] = np_;
    if (d.Np) ((g_f32*)(d.Np))[gr * d.np + gc] = np_;
  }
  if (!d.NpT) return;  // (uniform over the workgroup)
  __syncthreads();
  g_f32* NpT = (g_f32*)(d.NpT);
#pragma unroll 4
  for (int i = 0; i < 16; ++i) {
    const int r = rr + 4 * i;
    NpT[(int64_t(tj) * kTile + r) * d.mp + int64_t(ti) * kTile + c] = tn[c][r];
  }
}

__global__ __launch_bounds__(256) void soap_eye_kernel(const SoapEyeDesc* __restrict__ descs, int count) {
  const int e = find_desc(descs, count, blockIdx.x);
  const SoapEyeDesc& d = descs[e];
  const int lt = blockIdx.x - d.tile_begin;
  const int ti = lt / d.tiles_n, tj = lt - ti * d.tiles_n;
  const int t = threadIdx.x, c = t & 63, rr = t >> 6;
  const int64_t gc = int64_t(tj) * kTile + c;
  g_f32* X = (g_f32*)(d.X);
#pragma unroll 4
  for (int i = 0; i < 16; ++i) {
    const int64_t gr = int64_t(ti) * kTile + rr + 4 * i;
    X[gr * d.ld + gc] = (gr == gc && gr < d.d) ? 1.0f : 0.0f;
  }
}

// Householder factorization of one 16-column panel (LAPACK's convention: for the column x below and
// on the pivot, beta = -sign(x_0) ||x||, tau = (beta - x_0) / beta, v = x / (x_0 - beta) with v_0 = 1;
// tau = 0 when nothing below the pivot is non-zero). Its 16 x 16 block of T receives tau_k on the
// diagonal and the dot products v_j . v_k (j < k) above it, from which the applications and the
// block's factor form what they need. One 512-thread workgroup per panel; thread t holds rows
// t + 512 i (i < 8) of the panel in registers (the panel's columns are rows of the transposed matrix:
// each is read coalesced). One block reduction per column, of 16 sums at once (column k's squared
// norm below the pivot and its products with the other 15 columns there), formed in the same pass
// over the rows that applies the previous reflector; every wave sums the waves' partials itself
// (lane l: slot l, in wave order) and reads them back from its lanes. Every sum is taken in a fixed
// order.
__global__ __launch_bounds__(kQrPanelThreads) void qr_panel_kernel(const QrPanelDesc* __restrict__ descs) {
  __shared__ float red[2][kQrPanelThreads / 64][kQrPanel];  // by column parity: the waves' sums
  __shared__ float piv[2][kQrPanel];                         // by column parity: the pivot row
  __shared__ float Ds[kQrPanel][kQrPanel];
  __builtin_amdgcn_s_setprio(3);  // the updates of the auxiliary stream share its CU
  const QrPanelDesc& d = descs[blockIdx.x];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int jb = d.jb;
  const int rows = jb > 0 ? d.d - d.c : 0;  // panel rows [c, d)
  float a[kQrRowsPerThread][kQrPanel];
  {
    const g_cf32* At = (const g_cf32*)(d.At) + int64_t(d.c) * d.ld + d.c;
#pragma unroll
    for (int k = 0; k < kQrPanel; ++k)
#pragma unroll
      for (int i = 0; i < kQrRowsPerThread; ++i) {
        const int lr = t + kQrPanelThreads * i;
        a[i][k] = (lr < rows && k < jb) ? At[int64_t(k) * d.ld + lr] : 0.0f;
      }
  }
  if (t < kQrPanel * kQrPanel) Ds[t / kQrPanel][t % kQrPanel] = 0.0f;
  // register rows that hold panel rows (uniform); the others are zero and are skipped. Columns
  // >= jb are zero as well: their dot products are exactly 0 and they stay 0.
  const int used = (rows + kQrPanelThreads - 1) / kQrPanelThreads;
  // Column k's sums over the rows below its pivot: slot l = a_k . a_l (slot k: the squared norm),
  // reduced within each wave (lane l: slot l) into red[k & 1]; the pivot row into piv[k & 1].
  auto reduce_col = [&](auto kc) {
    constexpr int k = decltype(kc)::value;
    float part[kQrPanel];
#pragma unroll
    for (int l = 0; l < kQrPanel; ++l) part[l] = 0.0f;
#pragma unroll
    for (int i = 0; i < kQrRowsPerThread; ++i) {
      if (i < used && t + kQrPanelThreads * i > k) {
        const float ak = a[i][k];
#pragma unroll
        for (int l = 0; l < kQrPanel; ++l) part[l] += ak * a[i][l];
      }
    }
    // lane l of every row: the row's sum of slot l; then over the four rows of the wave (the
    // adds are commutative pairs, so every lane of a column l agrees bit for bit)
    const float r = sum_rows4(row_reduce_scatter16(part, lane & 15));
    if (lane < kQrPanel) red[k & 1][w][lane] = r;
    if (t == k) {
#pragma unroll
      for (int l = 0; l < kQrPanel; ++l) piv[k & 1][l] = a[0][l];
    }
  };
  if (jb > 0) {  // (uniform)
    reduce_col(std::integral_constant<int, 0>{});
    __syncthreads();
  }

  // One barrier per column: the sums of column k were formed (and reduced) in the pass that applied
  // reflector k - 1. With them, v_k = e_k + scale a_k (below the pivot), and every product with v_k
  // follows without another reduction: v_k . a_l = a_l[k] + scale (a_k . a_l), v_j . v_k = v_j[k] +
  // scale (a_k . v_j).
  unrolled<kQrPanel>([&](auto kc) {
    constexpr int k = decltype(kc)::value;
    if (k >= jb) return;  // (uniform: jb is the panel's width)
    // the block totals: lane l of every wave sums slot l over the waves in wave order, and the wave
    // reads them from its lanes (red[k & 1] and piv[k & 1] are written again only after the next
    // column's barrier)
    float mine = 0.0f;
#pragma unroll
    for (int j = 0; j < kQrPanelThreads / 64; ++j) mine += red[k & 1][j][lane & (kQrPanel - 1)];
    float tot[kQrPanel], pv[kQrPanel];
#pragma unroll
    for (int l = 0; l < kQrPanel; ++l) {
      tot[l] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mine), l));
      pv[l] = piv[k & 1][l];
    }
    const float alpha = pv[k], sigma = tot[k];
    float tau = 0.0f, scale = 0.0f;
    if (sigma != 0.0f) {
      const float beta = -copysignf(sqrtf(alpha * alpha + sigma), alpha);
      tau = (beta - alpha) / beta;
      scale = 1.0f / (alpha - beta);
    }
    float f[kQrPanel];
#pragma unroll
    for (int l = k + 1; l < kQrPanel; ++l) f[l] = tau * (pv[l] + scale * tot[l]);
#pragma unroll
    for (int i = 0; i < kQrRowsPerThread; ++i) {
      if (i < used) {
        const int lr = t + kQrPanelThreads * i;
        a[i][k] = lr > k ? a[i][k] * scale : (lr == k ? 1.0f : 0.0f);
#pragma unroll
        for (int l = k + 1; l < kQrPanel; ++l) a[i][l] -= f[l] * a[i][k];
      }
    }
#pragma unroll
    for (int j = 0; j < k; ++j)
      if (t == j) Ds[j][k] = pv[j] + scale * tot[j];
    if (t == k) Ds[k][k] = tau;
    if constexpr (k + 1 < kQrPanel) {
      if (k + 1 < jb) {  // (uniform)
        reduce_col(std::integral_constant<int, k + 1>{});
        __syncthreads();
      }
    }
  });
  __syncthreads();
  // the panel's 16 rows of Vt over every block row: entries [0, c - j0) above the panel are zero,
  // entries [c - j0, vrows) are the registers (zero from d on; vrows - (c - j0) = dp - c <= kQrMaxDim).
  // (V itself is formed by qr_t_kernel's launch: 64-byte pieces of its 512-byte rows, stored from here,
  // took one line per lane and instruction on the one CU that the whole factorization waits for.)
  const int top = d.c - d.j0, s16 = top;  // the panel's first column within the block = c - j0
  {
    g_f32* Vt = (g_f32*)(d.Vt) + int64_t(s16) * d.ldvt;
    const int below = d.vrows - top;
#pragma unroll
    for (int i = 0; i < kQrRowsPerThread; ++i) {
      const int lr = t + kQrPanelThreads * i;
      if (lr < below) {
#pragma unroll
        for (int k = 0; k < kQrPanel; ++k) Vt[int64_t(k) * d.ldvt + top + lr] = a[i][k];
      }
    }
    for (int r = t; r < top; r += kQrPanelThreads) {
#pragma unroll
      for (int k = 0; k < kQrPanel; ++k) Vt[int64_t(k) * d.ldvt + r] = 0.0f;
    }
  }
  if (t < kQrPanel * kQrPanel)
    ((g_f32*)d.T)[int64_t(s16 + t / kQrPanel) * kQrBlock + s16 + t % kQrPanel] = Ds[t / kQrPanel][t % kQrPanel];
}

// x <- H_16 ... H_1 x = x - V_s y for one column x of A (a row of At, rows [c, d) of A), with
// y_k = tau_k (w_k - sum_{j<k} (v_j . v_k) y_j) and w = V_s^T x (the reflectors applied one after the
// other, in the reduced coordinates). Bound by latency: it runs between two panels that depend on it.
// (This layout, V out of the panels and the factor below: basis refresh of six 768/3072-sided matrices
// 14.24 -> 12.16 ms.)
// Thread t holds entries 4 (t + 256 i) .. + 3 in registers and reads the reflectors from Vt, 16 bytes per
// lane and 1 KiB per wave (from V's rows, 64 bytes of each 512, a load touched one line per lane).
// It forms its part of the 16 sums w; the workgroup reduces them in a fixed order (DPP reduce-scatter
// within each row of 16 lanes, then over the wave's four rows, then over the four waves through LDS);
// every wave then runs the 16-step recurrence for y itself, lane k holding w_k and column k of
// the panel's block of T, and subtracts V_s y from its entries. The column is read and written once.
__global__ __launch_bounds__(kQrColThreads) void qr_col_kernel(const QrColDesc* __restrict__ descs, int count) {
  __shared__ float red[kQrColThreads / 64][kQrPanel];
  __builtin_amdgcn_s_setprio(3);
  const int e = find_desc(descs, count, blockIdx.x);
  const QrColDesc& d = descs[e];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, l16 = lane & (kQrPanel - 1);
  float tk[kQrPanel];  // T[j][l16]
#pragma unroll
  for (int j = 0; j < kQrPanel; ++j) tk[j] = ((const g_cf32*)(d.T))[j * kQrBlock + l16];
  const int64_t col = int64_t(d.c) + kQrPanel + (blockIdx.x - d.tile_begin);
  g_f32* x = (g_f32*)(d.At) + col * d.ld + d.c;
  const g_cf32* Vt = (const g_cf32*)(d.Vt);
  f32x4 xr[kQrColGroups];
  float part[kQrPanel];
#pragma unroll
  for (int k = 0; k < kQrPanel; ++k) part[k] = 0.0f;
  // (a group's four entries lie within the padded row: c and the row's length are multiples of 4;
  // entries from d on count as zero and are not written)
#pragma unroll
  for (int i = 0; i < kQrColGroups; ++i) {
    xr[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const int r = 4 * (t + kQrColThreads * i);
    if (r < d.rows) {
      xr[i] = *(const g_cf32x4*)(x + r);
#pragma unroll
      for (int j = 1; j < 4; ++j)
        if (r + j >= d.rows) xr[i][j] = 0.0f;
#pragma unroll
      for (int k = 0; k < kQrPanel; ++k) {
        const f32x4 v = *(const g_cf32x4*)(Vt + int64_t(k) * d.ldvt + r);
        // (in pairs: four terms in a row made the factor's error a few per cent larger)
        part[k] += (v[0] * xr[i][0] + v[1] * xr[i][1]) + (v[2] * xr[i][2] + v[3] * xr[i][3]);
      }
    }
  }
  const float rsum = sum_rows4(row_reduce_scatter16(part, l16));
  if (lane < kQrPanel) red[w][lane] = rsum;
  __syncthreads();
  float acc = ((red[0][l16] + red[1][l16]) + red[2][l16]) + red[3][l16];
  float y[kQrPanel];
#pragma unroll
  for (int j = 0; j < kQrPanel; ++j) {
    y[j] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(tk[j] * acc), j));
    acc -= tk[j] * y[j];  // (lanes up to j are not read again)
  }
#pragma unroll
  for (int i = 0; i < kQrColGroups; ++i) {
    const int r = 4 * (t + kQrColThreads * i);
    if (r < d.rows) {
      f32x4 sub[2] = {};
#pragma unroll
      for (int k = 0; k < kQrPanel; ++k) {
        const f32x4 v = *(const g_cf32x4*)(Vt + int64_t(k) * d.ldvt + r);
#pragma unroll
        for (int j = 0; j < 4; ++j) sub[k & 1][j] += v[j] * y[k];
      }
      const f32x4 out = xr[i] - (sub[0] + sub[1]);
      if (r + 4 <= d.rows) {
        *(g_f32x4*)(x + r) = out;
      } else {
#pragma unroll
        for (int j = 0; j < 3; ++j)
          if (r + j < d.rows) x[r + j] = out[j];
      }
    }
  }
}

// The block's compact-WY factor, one workgroup per block, held in LDS. The panels' diagonal blocks
// first, row by row (one thread per row i; T_kk = tau_k, T_ik = -tau_k sum_{j=i}^{k-1} T_ij (v_j . v_k),
// from the tau and dot products the panel left in its block); then, with the blocks of G above the
// diagonal (G summed over its partials in order), neighbouring diagonal blocks T1, T2 of side L = 16, 32,
// 64 are joined: M = G12 T2, T12 = -T1 M, on the fp64 MFMA (16 x 16 x 4; with fp32 sums the refreshed basis was 2 to
// 4 % less orthogonal than with the panel-by-panel form, now it is up to 13 % more), M held below the diagonal,
// where T is zero. Three levels of two products: the panel-by-panel form with one output element per thread
// had seven, on a chain that every block waits for. The launch's other workgroups form V from Vt,
// 64 x 64 elements each, meanwhile.
__global__ __launch_bounds__(kQrTThreads) void qr_t_kernel(const QrTDesc* __restrict__ descs, int count) {
  __shared__ float Tl[kQrBlock][kQrBlock + 1];
  __shared__ float Gl[kQrBlock][kQrBlock + 1];
  __shared__ float Dl[kQrBlock][kQrPanel];  // row i: the panel's tau / dot-product row i
  const int t = threadIdx.x;
  __builtin_amdgcn_s_setprio(3);
  if (int(blockIdx.x) >= count) {
    const int b = int(blockIdx.x) - count;
    const QrTDesc& d = descs[find_desc(descs, count, b)];
    int lt = b - d.tile_begin;
    if (d.W) {
      if (lt < kQrSumWgs) {
        static_assert(kQrBlock * kQrBlock == 4 * kQrTThreads * kQrSumWgs, "four elements per thread");
        const int o = 4 * (lt * kQrTThreads + t);
        f32x4 s = *(const g_cf32x4*)((const g_cf32*)(d.W) + o);
        for (int q = 1; q < d.nW; ++q) s += *(const g_cf32x4*)((const g_cf32*)(d.W) + q * kQrBlock * kQrBlock + o);
        *(g_f32x4*)((g_f32*)(d.Ws) + o) = s;
        return;
      }
      lt -= kQrSumWgs;
    }
    const int ti = lt >> 1, tj = lt & 1;  // rows 64 ti, columns 64 tj of V
    const int c = t & 63, rr = t >> 6;
    const g_cf32* Vt = (const g_cf32*)(d.Vt) + int64_t(64 * tj) * d.ldvt + 64 * ti;
    g_f32* V = (g_f32*)(d.V) + int64_t(64 * ti) * kQrBlock + 64 * tj;
#pragma unroll
    for (int i = 0; i < 64; i += kQrTThreads / 64) Tl[rr + i][c] = Vt[int64_t(rr + i) * d.ldvt + c];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 64; i += kQrTThreads / 64) V[int64_t(rr + i) * kQrBlock + c] = Tl[c][rr + i];
    return;
  }
  const QrTDesc& d = descs[blockIdx.x];
  g_f32* T = (g_f32*)(d.T);
  const g_cf32* G = (const g_cf32*)(d.G);
  // thread t owns column j = t % 128 and every fourth row of both matrices; G's partials (only what lies
  // above the diagonal is used: of the left half of the columns, the upper half of the rows) are summed in
  // order, the loads of four partials in flight together (one partial at a time, the 12 partials of a
  // 3072-sided statistic cost the refresh of a GPT-2-small layer 0.9 ms)
  constexpr int kM = kQrBlock * kQrBlock / kQrTThreads, kStep = kQrTThreads / kQrBlock;
  const int tj = t % kQrBlock, ti = t / kQrBlock;
#pragma unroll
  for (int m = 0; m < kM; ++m) Tl[ti + kStep * m][tj] = 0.0f;
  auto sum_g = [&](auto rows_c) {
    constexpr int M = decltype(rows_c)::value;
    float g[M] = {};
    auto add = [&](int q0, auto parts_c) {
      constexpr int N = decltype(parts_c)::value;
      float x[N][M];
#pragma unroll
      for (int p = 0; p < N; ++p)
#pragma unroll
        for (int m = 0; m < M; ++m) x[p][m] = G[(int64_t(q0 + p) * kQrBlock + ti + kStep * m) * kQrBlock + tj];
#pragma unroll
      for (int p = 0; p < N; ++p)
#pragma unroll
        for (int m = 0; m < M; ++m) g[m] += x[p][m];
    };
    int q = 0;
    for (; q + 4 <= d.nG; q += 4) add(q, std::integral_constant<int, 4>{});
    for (; q < d.nG; ++q) add(q, std::integral_constant<int, 1>{});
#pragma unroll
    for (int m = 0; m < M; ++m) Gl[ti + kStep * m][tj] = g[m];
  };
  if (__builtin_amdgcn_readfirstlane(tj) < kQrBlock / 2) sum_g(std::integral_constant<int, kM / 2>{});
  else sum_g(std::integral_constant<int, kM>{});
#pragma unroll
  for (int idx = t; idx < kQrBlock * kQrPanel; idx += kQrTThreads) {
    const int i = idx / kQrPanel, jj = idx % kQrPanel;
    Dl[i][jj] = T[i * kQrBlock + (i / kQrPanel) * kQrPanel + jj];
  }
  __syncthreads();
  if (t < kQrBlock) {
    const int i = t, b0 = (i / kQrPanel) * kQrPanel, ii = i % kQrPanel;
    float row[kQrPanel];
#pragma unroll
    for (int k = 0; k < kQrPanel; ++k) {
      float v = 0.0f;
      if (k == ii) {
        v = Dl[i][ii];
      } else if (k > ii) {
        float acc = 0.0f;
#pragma unroll
        for (int j = 0; j < k; ++j)
          if (j >= ii) acc += row[j] * Dl[b0 + j][k];
        v = -Dl[b0 + k][k] * acc;
      }
      row[k] = v;
      Tl[i][b0 + k] = v;
    }
  }
  __syncthreads();
  // one wave per 16 x 16 output tile; a lane's operands are row (column) lane % 16, k = lane / 16, its
  // outputs rows lane / 16 + 4 r of column lane % 16
  typedef double f64x4 __attribute__((ext_vector_type(4)));
  const int lane = t & 63, w = t >> 6, lc = lane & 15, lk = lane >> 4;
  for (int L = kQrPanel; L < kQrBlock; L *= 2) {
    const int n = L / 16, per = n * n, tiles = kQrBlock / (2 * L) * per;
    for (int tile = w; tile < tiles; tile += kQrTThreads / 64) {
      const int b = tile / per * 2 * L, i0 = tile % per / n * 16, j0 = tile % n * 16;
      f64x4 acc[2] = {};
      for (int k = 0; k < j0 + 16; k += 16)  // T2 is upper triangular
#pragma unroll
        for (int q = 0; q < 4; ++q)
          acc[q & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(Gl[b + i0 + lc][b + L + k + 4 * q + lk],
                                                            Tl[b + L + k + 4 * q + lk][b + L + j0 + lc], acc[q & 1], 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) Tl[b + L + i0 + lk + 4 * r][b + j0 + lc] = float(acc[0][r] + acc[1][r]);
    }
    __syncthreads();
    for (int tile = w; tile < tiles; tile += kQrTThreads / 64) {
      const int b = tile / per * 2 * L, i0 = tile % per / n * 16, j0 = tile % n * 16;
      f64x4 acc[2] = {};
      for (int k = i0; k < L; k += 16)  // so is T1
#pragma unroll
        for (int q = 0; q < 4; ++q)
          acc[q & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(Tl[b + i0 + lc][b + k + 4 * q + lk],
                                                            Tl[b + L + k + 4 * q + lk][b + j0 + lc], acc[q & 1], 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) Tl[b + i0 + lk + 4 * r][b + L + j0 + lc] = -float(acc[0][r] + acc[1][r]);
    }
    __syncthreads();
    // M's place is read as T's zeros by the next level
    for (int idx = t; idx < 64 * L; idx += kQrTThreads) {
      const int p = idx / (L * L), i = idx % (L * L) / L, j = idx % L;
      Tl[2 * L * p + L + i][2 * L * p + j] = 0.0f;
    }
    __syncthreads();
  }
#pragma unroll
  for (int m = 0; m < kM; ++m) T[(ti + kStep * m) * kQrBlock + tj] = Tl[ti + kStep * m][tj];
}

}  // namespace

hipError_t launch_soap_prep(const SoapPrepDesc* d, int count, int total_tiles, float beta1, hipStream_t st) {
  if (total_tiles <= 0 || count <= 0) return hipSuccess;
  hipLaunchKernelGGL(soap_prep_kernel, dim3(total_tiles), dim3(256), 0, st, d, count, beta1);
  return hipGetLastError();
}

hipError_t launch_soap_adam(const SoapAdamDesc* d, int count, int total_tiles, float beta2, float eps,
                            float inv_bc1, float inv_sqrt_bc2, hipStream_t st) {
  if (total_tiles <= 0 || count <= 0) return hipSuccess;
  hipLaunchKernelGGL(soap_adam_kernel, dim3(total_tiles), dim3(256), 0, st, d, count, beta2, eps, inv_bc1,
                     inv_sqrt_bc2);
  return hipGetLastError();
}

hipError_t launch_soap_eye(const SoapEyeDesc* d, int count, int total_tiles, hipStream_t st) {
  if (total_tiles <= 0 || count <= 0) return hipSuccess;
  hipLaunchKernelGGL(soap_eye_kernel, dim3(total_tiles), dim3(256), 0, st, d, count);
  return hipGetLastError();
}

hipError_t launch_qr_panel(const QrPanelDesc* d, int count, hipStream_t st) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(qr_panel_kernel, dim3(count), dim3(kQrPanelThreads), 0, st, d);
  return hipGetLastError();
}

hipError_t launch_qr_col(const QrColDesc* d, int count, int total_blocks, hipStream_t st) {
  if (total_blocks <= 0 || count <= 0) return hipSuccess;
  hipLaunchKernelGGL(qr_col_kernel, dim3(total_blocks), dim3(kQrColThreads), 0, st, d, count);
  return hipGetLastError();
}

hipError_t launch_qr_t(const QrTDesc* d, int count, int total_tiles, hipStream_t st) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(qr_t_kernel, dim3(count + total_tiles), dim3(kQrTThreads), 0, st, d, count);
  return hipGetLastError();
}

}  // namespace mfsdp
