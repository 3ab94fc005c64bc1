// Kernels of the inverse fourth root (Shampoo's preconditioners): its products on split-fp16 operands
// (h2_core.h), the conversion of a statistic into the iteration's first M, and of its result into the
// caller's fp32 matrix.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "h2_core.h"
#include "mfsdp_internal.h"
#include "shampoo_internal.h"

namespace mfsdp {
namespace {

typedef __attribute__((address_space(1))) float g_f32;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) f32x4 g_f32x4;
typedef __attribute__((address_space(1))) const f32x4 g_cf32x4;

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

// One 128 x 128 upper tile of one product per workgroup (4 waves of 64 x 64, 80 KiB of LDS: two workgroups
// per CU, so that one multiplies while the other is in its epilogue). Bound by the matrix pipe at the
// power-limited clock, the operand loads and the LDS reads: a launch with one product of each of 24 sides
// (4 of 3072, 20 of 768; 1.31e11 flop on the upper tiles) takes 0.38 to 0.47 ms, 1000 TFLOP/s of fp16 MFMA (the
// six bf16 products per 16 k of the general kernel: 0.68 ms); the matrix pipe is busy 70 % of the cycles in
// which its CU has work. 256 x 128 tiles (a quarter fewer operand bytes) took the same time, and so did
// splitting the sides over two streams to fill the launches' tails.
// Epilogue: the tile's image (64 blocks of 1 KiB) is formed in LDS. E, if any, is first copied there as it
// lies by direct global->LDS loads; every lane then replaces its own elements by the result. The blocks
// leave whole, as they are and (mirror) through transposing LDS reads. Results are stored exactly symmetric:
// only blocks on and above the diagonal are stored, with their mirrors, and a block on the diagonal takes
// its lower triangle from its upper one.
using Core = H2Core<2, 2, 2, 2, 5>;
__global__ __launch_bounds__(256, 2) void h2_root_kernel(const RootDesc* __restrict__ descs,
                                                         const TileRef* __restrict__ tiles) {
  __shared__ __attribute__((aligned(1024))) uint8_t smem[Core::NST * Core::STAGE];
  const TileRef tr = tiles[blockIdx.x];
  const RootDesc& d = descs[tr.e];
  const int bi = tr.bi, bj = tr.bj;
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);

  // coefficients (scaled) from the row that the residual selects
  const float r = *d.conv_in;
  const bool done = r == kRootDone, fin = root_ends(*d.sum_in);
  if (bi == 0 && bj == 0 && t == 0) {
    if (d.clear) {
      *d.clear = fin ? kRootDone : 0.0f;
      *d.sum_clear = 0;
    }
    if (d.xsel && !done) *d.xsel = d.out_idx;
  }
  if (done || (fin && d.op >= kRootT2)) return;
  const bool agg = !(r < kRootSwitch);
  const float ca = agg ? kRootAggressive[0] : kRootFinal[0];
  const float cb = agg ? kRootAggressive[1] : kRootFinal[1];
  const float cc = agg ? kRootAggressive[2] : kRootFinal[2];
  const float sx = d.sc[3];  // X's scale
  float alpha = 1.0f, beta = 0.0f, diag = 0.0f;
  switch (d.op) {
    case kRootFirst: alpha = cc * sx / (kScM * kScM); beta = cb * sx / kScM; diag = ca * sx; break;
    case kRootU: alpha = cc * kScU / (kScM * kScM); beta = cb * kScU / kScM; break;
    case kRootX: alpha = 1.0f / kScU; beta = ca; break;
    case kRootT2:
      if (d.E) {
        alpha = kScT2 / (kScU * kScU);
        beta = 2.0f * ca * (kScT2 / kScU);
        diag = ca * ca * kScT2;
      } else {
        alpha = kScT2 / sx / sx;
      }
      break;
    case kRootT4: alpha = kScT4 / (kScT2 * kScT2); break;
    default: alpha = 1.0f / kScT4; break;
  }

  h2_f32x16 acc[Core::MI][Core::NI];
#pragma unroll
  for (int i = 0; i < Core::MI; ++i)
#pragma unroll
    for (int j = 0; j < Core::NI; ++j) acc[i][j] = h2_f32x16{};
  const int64_t panel = int64_t(d.K) << 5;  // 16-bit units per 16-row panel
  const int np = d.K >> 4;                  // panels
  const int r0 = bi * Core::PP, c0 = bj * Core::QP;  // first block row and column
  {
    const uint16_t* ps[Core::PL];
    const uint16_t* qs[Core::QL];
#pragma unroll
    for (int i = 0; i < Core::PL; ++i) ps[i] = d.P + (r0 + i * Core::NW + w) * panel + lane * 8;
#pragma unroll
    for (int i = 0; i < Core::QL; ++i) qs[i] = d.Q + (c0 + i * Core::NW + w) * panel + lane * 8;
    Core::loop(ps, qs, np, smem, w, lane, acc);
  }

  // image block (rp, cb) of the tile at (8 rp + cb) KiB
  static_assert(Core::NST * Core::STAGE >= 65536, "image of a tile");
  const uint16_t* E = d.E;
  h2_lds* img = (h2_lds*)smem;
  h2_gu16* C = (h2_gu16*)d.C;
  const int wm = w / Core::WN, wn = w % Core::WN;
  const int fr = lane & 31, fh = lane >> 5;
  const int sw = h2_swz(fr & 15);
  const H2BlockLane bl(lane);
  float res = 0.0f, sum = 0.0f;
  if (E) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int b = i * 4 + w;
      __builtin_amdgcn_global_load_lds(
          (const void*)(E + (r0 + (b >> 3)) * panel + int64_t(c0 + (b & 7)) * 512 + lane * 8), img + b * 1024, 16, 0, 0);
    }
    H2_WAIT_VMCNT(0);
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < Core::MI; ++i)
#pragma unroll
    for (int j = 0; j < Core::NI; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        // element (gr, gc + k) of the matrix
        const int gr = r0 * 16 + wm * (Core::MI * 32) + i * 32 + fr;
        const int gc = c0 * 16 + wn * (Core::NI * 32) + j * 32 + g * 8 + fh * 4;
        h2_lds* at = img + ((wm * 4 + i * 2 + (fr >> 4)) * 8 + wn * (Core::NI * 2) + j * 2 + (g >> 1)) * 1024 +
                     (fr & 15) * 32 + (((g & 1) ^ sw) << 4) + fh * 8;
        float v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = alpha * acc[i][j][4 * g + k];
        if (E) {
          const h2_u32x2 eh = *(h2_lu2*)at, el = *(h2_lu2*)(at + 512);
          float e0, e1, e2, e3;
          h2_join2(eh.x, el.x, e0, e1);
          h2_join2(eh.y, el.y, e2, e3);
          v[0] += beta * e0;
          v[1] += beta * e1;
          v[2] += beta * e2;
          v[3] += beta * e3;
        }
        if (diag != 0.0f) {
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (gr == gc + k) v[k] += diag;
        }
        if (d.resid_out) {
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (gr <= gc + k && gr < d.valid && gc + k < d.valid) {
              const float dv = fabsf(v[k] * (1.0f / kScM) - (gr == gc + k ? 1.0f : 0.0f));
              res = (dv > res || dv != dv) ? dv : res;  // keeps a NaN
              sum += (gr == gc + k ? 1.0f : 2.0f) * (dv * dv);
            }
        }
        uint32_t h0, l0, h1, l1;
        h2_split2(v[0], v[1], h0, l0);
        h2_split2(v[2], v[3], h1, l1);
        *(h2_lu2*)at = h2_u32x2{h0, h1};
        *(h2_lu2*)(at + 512) = h2_u32x2{l0, l1};
      }
  __syncthreads();
#pragma unroll 4
  for (int i = 0; i < 16; ++i) {
    const int b = i * 4 + w;
    const int rp = r0 + (b >> 3), cb = c0 + (b & 7);  // (uniform over the wave)
    if (rp > cb) continue;
    h2_u32x4 v = bl.read(img + b * 1024);
    const h2_u32x4 tv = bl.read_t(img + b * 1024);
    if (rp == cb) v = bl.mirror(v, tv);
    *(h2_gu4*)(C + rp * panel + int64_t(cb) * 512 + bl.off / 2) = v;
    if (rp != cb) *(h2_gu4*)(C + cb * panel + int64_t(rp) * 512 + bl.off / 2) = tv;
  }
  if (d.resid_out) {
    // NaN propagates as the largest bit pattern, so a diverged side never counts as converged
    uint32_t rb = __float_as_uint(res);
    if (res != res) rb = 0x7fc00000u;
    for (int o = 32; o > 0; o >>= 1) {
      rb = max(rb, uint32_t(__shfl_xor(int(rb), o)));
      sum += __shfl_xor(sum, o);
    }
    if (lane == 0) {
      atomicMax(reinterpret_cast<unsigned int*>(d.resid_out), rb);
      atomicAdd(d.sum_out, (unsigned long long)(root_sum_term(sum)));
    }
  }
}

// M_0 = z (S + rho I) in h2 from the padded fp32 statistic: one 64 x 64 tile per workgroup; a half wave
// converts one 16 x 16 block (lane: 8 consecutive columns of a row, 32 bytes in, 16 + 16 out).
__global__ __launch_bounds__(256) void h2_root_init_kernel(const RootConvDesc* __restrict__ descs, int count) {
  const int e = find_desc(descs, count, blockIdx.x);
  const RootConvDesc& d = descs[e];
  const int lt = blockIdx.x - d.tile_begin, tn = d.dp / 64;
  const int ti = lt / tn, tj = lt - ti * tn;
  const int t = threadIdx.x;
  if (lt == 0 && t < 2) {
    d.resid[t] = t == 0 ? 0.0f : 3.0e38f;
    d.sum[t] = t == 0 ? 0 : kRootSumOpen;
  }
  const float rho = d.sc[0], zs = d.sc[1] * kScM;
  const int l = t & 31, row = l & 15, ch = l >> 4;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int b = (t >> 5) + 8 * i, rb = b >> 2, cb = b & 3;
    const int gr = ti * 64 + rb * 16 + row, gc = tj * 64 + cb * 16 + ch * 8;
    const float* s = d.S + int64_t(gr) * d.dp + gc;
    const f32x4 x0 = *(g_cf32x4*)s, x1 = *(g_cf32x4*)(s + 4);
    float v[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
    h2_u32x4 hi, lo;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      uint32_t h, q;
      h2_split2(zs * (v[2 * k] + (gr == gc + 2 * k ? rho : 0.0f)),
                zs * (v[2 * k + 1] + (gr == gc + 2 * k + 1 ? rho : 0.0f)), h, q);
      hi[k] = h;
      lo[k] = q;
    }
    h2_gu16* m = (h2_gu16*)d.M + h2_index(gr, gc, d.dp);
    *(h2_gu4*)m = hi;
    *(h2_gu4*)(m + kH2Lo) = lo;
  }
}

// The root in fp32 (dp x dp row-major): z^(1/4) X from the X buffer the side ended in.
__global__ __launch_bounds__(256) void h2_root_out_kernel(const RootConvDesc* __restrict__ descs, int count) {
  const int e = find_desc(descs, count, blockIdx.x);
  const RootConvDesc& d = descs[e];
  const int lt = blockIdx.x - d.tile_begin, tn = d.dp / 64;
  const int ti = lt / tn, tj = lt - ti * tn;
  const int t = threadIdx.x;
  const float zp = d.sc[2] / d.sc[3];
  const uint16_t* X = *d.xsel ? d.X1 : d.X0;
  const int l = t & 31, row = l & 15, ch = l >> 4;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int b = (t >> 5) + 8 * i, rb = b >> 2, cb = b & 3;
    const int gr = ti * 64 + rb * 16 + row, gc = tj * 64 + cb * 16 + ch * 8;
    const h2_gcu16* x = (h2_gcu16*)X + h2_index(gr, gc, d.dp);
    const h2_u32x4 hi = *(__attribute__((address_space(1))) const h2_u32x4*)x;
    const h2_u32x4 lo = *(__attribute__((address_space(1))) const h2_u32x4*)(x + kH2Lo);
    float v[8];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      h2_join2(hi[k], lo[k], v[2 * k], v[2 * k + 1]);
      v[2 * k] *= zp;
      v[2 * k + 1] *= zp;
    }
    float* o = d.out + int64_t(gr) * d.dp + gc;
    *(g_f32x4*)o = f32x4{v[0], v[1], v[2], v[3]};
    *(g_f32x4*)(o + 4) = f32x4{v[4], v[5], v[6], v[7]};
  }
}

}  // namespace

hipError_t launch_root(const RootDesc* d, const TileRef* tiles, int total_tiles, hipStream_t st) {
  if (total_tiles <= 0) return hipSuccess;
  hipLaunchKernelGGL(h2_root_kernel, dim3(total_tiles), dim3(256), 0, st, d, tiles);
  return hipGetLastError();
}
hipError_t launch_root_conv(const RootConvDesc* d, int count, int total_tiles, int dir, hipStream_t st) {
  if (total_tiles <= 0 || count <= 0) return hipSuccess;
  if (dir == 0)
    hipLaunchKernelGGL(h2_root_init_kernel, dim3(total_tiles), dim3(256), 0, st, d, count);
  else
    hipLaunchKernelGGL(h2_root_out_kernel, dim3(total_tiles), dim3(256), 0, st, d, count);
  return hipGetLastError();
}

}  // namespace mfsdp
