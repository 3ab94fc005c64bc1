// The fp32 Newton-Schulz path: its products on split-fp16 operands (h2_core.h), the split of the momentum
// pass's fp32 u into the first iterate, and the parameter update in the last product's epilogue.
//
// Buffers are padded to 64 and tiles are 128 x 128 or 64 x 64, so a tile may reach past the last panel: such
// panels read the last one again and are not stored.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "h2_core.h"
#include "mfsdp_internal.h"

namespace mfsdp {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) float g_f32;
typedef __attribute__((address_space(1))) const float g_cf32;
typedef __attribute__((address_space(1))) f32x4 g_f32x4;
typedef __attribute__((address_space(1))) const f32x4 g_cf32x4;
typedef __attribute__((address_space(3))) float l_f32;
typedef __attribute__((address_space(3))) f32x4 l_f32x4;

template <typename D>
__device__ __forceinline__ int find_entry(const D* descs, int count, int key) {
  int lo = 0, hi = count - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (descs[mid].tile_begin <= key) lo = mid; else hi = mid - 1;
  }
  return lo;
}

constexpr int kGram = 0, kSquare = 1, kUpdate = 2, kApply = 3;

// Scales. A product's result is split as it is stored, so its buffer's power-of-two scale 2^e must follow from
// what is known before the product. Two ways, chosen by the host from the coefficients (h2_exponents):
//   static  bounds on the singular values carried from step to step by the coefficients; no cost here.
//   DYN     where those bounds leave the singular values behind (a step's polynomial may take the bound outside
//           the next one's stable interval, from where it grows without end): bounds that start anew in
//           every step from the data. For X with K columns and A = X X^T:
//             |A_ij| <= min(K max |X|^2, lambda_max(A))               (|A_ij| <= the row norms' squares)
//             |B'_ij| <= |a| + |b| max |A| + |c| ||A||_F max |A|       (|(A A)_ij| <= lambda_max(A) max |A|)
//             |X'_ij| <= max |sqrt(y) (a + b y + c y^2)|, 0 <= y <= sqrt(||A A||_F)    (>= lambda_max(A))
//                                                         or 0 <= y <= lambda_max(A)'s bound from the last step
//           The maxima and the norms (sums of squares, in integers, so that their order does not matter) are
//           taken by the epilogues, which costs 1 us per launch and 7 % at 768 x 3072; the last bound squared
//           is the next step's lambda_max(A). They exceed the largest element by up to about r^(1/4) in the
//           singular values (2^8 for X' at r = 4096): parts lose bits from 2^-28 of the bound down.
struct TileStats {
  float big = 0.0f, sq = 0.0f;  // largest |v| (NaN: kept) and sum of v^2 of the thread's elements
  __device__ __forceinline__ void add(float v, float weight) {
    const float m = fabsf(v);
    big = m > big || m != m ? m : big;
    sq += weight * (v * v);
  }
};
// The workgroup's (NW waves') statistics of values held under the scale 2^e into the matrix's slots: the largest
// |value| and, if sum is set, the sum of squares under the scale, rounded up, at most 2^45 per tile. lds: NW
// x 8 bytes that nobody else uses.
template <int NW>
__device__ __forceinline__ void put_stats(TileStats s, int e, uint32_t* max_slot, unsigned long long* sum, float* lds) {
  uint32_t big = __float_as_uint(s.big);
  if (s.big != s.big) big = 0x7fc00000u;
  float sq = s.sq;
  for (int o = 32; o > 0; o >>= 1) {
    big = max(big, uint32_t(__shfl_xor(int(big), o)));
    sq += __shfl_xor(sq, o);
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    lds[2 * w] = __uint_as_float(big);
    lds[2 * w + 1] = sq;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < NW; ++k) {
      big = max(big, __float_as_uint(lds[2 * k]));
      sq += lds[2 * k + 1];
    }
    if (max_slot) atomicMax(max_slot, __float_as_uint(ldexpf(__uint_as_float(big), -e)));
    if (sum) atomicAdd(sum, sq < 0x1p45f ? (unsigned long long)(sq) + 1ull : 1ull << 45);
  }
}

__device__ __forceinline__ NsH2State* ns_state(const float* scale) {
  return reinterpret_cast<NsH2State*>(reinterpret_cast<uintptr_t>(scale) + kNsH2StateOffset);
}
__device__ __forceinline__ const int32_t* ns_small(const float* scale) {
  return reinterpret_cast<const int32_t*>(scale) + 1;
}
__device__ __forceinline__ int gram_exponent(float lam, float xmax, int K) {
  return ns_h2_exponent(fminf(lam, float(K) * xmax * xmax));
}

// One tile of one product per workgroup, 128 x 128 (4 waves of 64 x 64, 80 KiB of LDS) or 64 x 64 (32 x 32,
// 64 KiB), two workgroups per CU. Bound by the matrix pipe and operand loads at large sizes (2048 x 8192, five
// steps: 1.95 ms, 318 TFLOP/s of the 3 r^2 s + r^3 fp32 flop; the fp32 MFMA kernel before it 6.18 ms) and by
// launches and the serial K loop at small ones (256 x 512: 239 -> 112 us; seven 768/3072/1024x4096 matrices
// 2.20 -> 0.84 ms). Errors against 64 bits after five steps: 768 x 768 2.7e-6 -> 1.1e-6, 2048 x 8192 4.8e-6 -> 1.5e-6.
// PK: the product; its epilogue is
//   Gram, square  C (upper tiles, mirrored; stored exactly symmetric), the square with the addend E = A and a I
//   Gram, split   the fp32 partial tile of K range ks into CT (the iterate's other buffer, free here)
//   update        X' in C and X'^T in CT
//   apply         the parameter update (or the standalone output) in the parameter's orientation
// ca, cb, cc: this step's a, b, c.
template <typename Core, int PK, bool DYN>
__global__ __launch_bounds__(256, 2) void ns_h2_kernel(const GemmDesc* __restrict__ descs, int count, int parity,
                                                       float ca, float cb, float cc, NsH2Exponents he) {
  constexpr int T = Core::TM, PB = T / 16;  // tile side, panels per side
  static_assert(Core::TM == Core::TN && Core::NST * Core::STAGE >= T * T * 4 + 8 * Core::NW, "square tile, image in LDS");
  __shared__ __attribute__((aligned(1024))) uint8_t smem[Core::NST * Core::STAGE];
  const GemmDesc& d = descs[find_entry(descs, count, blockIdx.x)];
  int lt = blockIdx.x - d.tile_begin, ks = 0;
  const int nks = PK == kGram && d.nks > 1 ? d.nks : 1;
  if (nks > 1) {
    ks = lt % nks;
    lt /= nks;
  }
  int bi, bj;
  if constexpr (PK <= kSquare) {
    bi = 0;
    int rem = lt;
    while (rem >= d.tiles_n - bi) rem -= d.tiles_n - bi++;
    bj = bi + rem;
  } else {
    bi = lt / d.tiles_n;
    bj = lt - bi * d.tiles_n;
  }
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int mp = d.M >> 4, np = d.N >> 4;      // panels of C's rows and columns
  const int r0 = bi * PB, c0 = bj * PB;

  // the matrix's state (loaded here, beside the operands' first loads, and used after the loop)
  NsH2State* st = ns_state(d.scale);
  // (small by a vector load, the oldest outstanding one during the loop: a scalar one was waited for before the
  // operands' loads, 1.3 % of a step on seven 768/3072/1024x4096 matrices against 0.2 %)
  int zero = 0;
  asm volatile("" : "+v"(zero));
  const int vsmall = DYN ? 0 : ns_small(d.scale)[zero];
  int ex = 0, ea = he.ea, eb = he.eb, eq_in = 0;
  float lam = 0.0f, xmax = 0.0f, amax = 0.0f, a2 = 0.0f, q2 = 0.0f;
  if constexpr (DYN) {
    ex = st->ex[parity];
    ea = st->ea;
    eb = st->eb;
    eq_in = st->eq;
    lam = st->lam[parity];
    xmax = __uint_as_float(st->xmax[parity]);
    amax = __uint_as_float(st->amax);
    a2 = float(st->a2);
    q2 = float(st->q2);
  }

  h2_f32x16 acc[Core::MI][Core::NI];
#pragma unroll
  for (int i = 0; i < Core::MI; ++i)
#pragma unroll
    for (int j = 0; j < Core::NI; ++j) acc[i][j] = h2_f32x16{};
  {
    const int nk = (d.K >> 4) / nks;
    const uint16_t* ps[Core::PL];
    const uint16_t* qs[Core::QL];
    const uint16_t* P = static_cast<const uint16_t*>(d.P[parity]) + int64_t(ks) * nk * 512 + lane * 8;
    const uint16_t* Q = static_cast<const uint16_t*>(d.Q[parity]) + int64_t(ks) * nk * 512 + lane * 8;
    const int64_t panel = int64_t(d.K) << 5;
#pragma unroll
    for (int i = 0; i < Core::PL; ++i) ps[i] = P + min(r0 + i * Core::NW + w, mp - 1) * panel;
#pragma unroll
    for (int i = 0; i < Core::QL; ++i) qs[i] = Q + min(c0 + i * Core::NW + w, np - 1) * panel;
    Core::loop(ps, qs, nk, smem, w, lane, acc);
  }

  const int small = __builtin_amdgcn_readfirstlane(vsmall);
  if constexpr (!DYN) ex = he.ex + max(0, small + he.gx);

  // the result's scale 2^eo, and 2^ep that of acc
  const bool first = bi == 0 && bj == 0 && ks == 0 && t == 0;
  const int ep = PK == kGram ? 2 * ex : PK == kSquare ? 2 * ea : eb + ex;
  int eo = PK == kGram ? ea : PK == kSquare ? eb : he.exn + max(0, small + he.gxn), eq = 0;
  if constexpr (DYN && PK == kGram) {
    eo = gram_exponent(lam, xmax, d.K);
    if (first) {
      st->q2 = 0;
      st->ea = eo;
    }
  } else if constexpr (DYN && PK == kSquare) {
    const float q = ldexpf(sqrtf(a2), -ea) * amax;  // bounds A A's elements
    eq = ns_h2_exponent(q);
    eo = ns_h2_exponent(fabsf(ca) + fabsf(cb) * amax + fabsf(cc) * q);
    if (first) {
      st->xmax[parity ^ 1] = 0;
      st->eb = eo;
      st->eq = eq;
    }
  } else if constexpr (DYN && PK == kUpdate) {
    const float bound = fminf(ns_h2_next_bound(sqrtf(ldexpf(sqrtf(q2), -eq_in)), ca, cb, cc),
                              ns_h2_next_bound(lam, ca, cb, cc));
    eo = ns_h2_exponent(bound);
    if (first) {
      st->amax = 0;
      st->a2 = 0;
      st->ex[parity ^ 1] = eo;
      st->lam[parity ^ 1] = fmaxf(bound * bound, 0x1p-120f);
    }
  }

  const int wm = w / Core::WN, wn = w % Core::WN;
  const int fr = lane & 31, fh = lane >> 5;
  // this lane's values: rows il(i), columns jl(j, g) .. + 3 of the tile
  auto il = [&](int i) { return wm * (Core::MI * 32) + i * 32 + fr; };
  auto jl = [&](int j, int g) { return wn * (Core::NI * 32) + j * 32 + g * 8 + fh * 4; };
  h2_lds* img = (h2_lds*)smem;

  if (PK == kGram && nks > 1) {
    // (the scale is applied by the sum)
    g_f32* part = (g_f32*)d.CT[parity] + (int64_t(upper_index(bi, bj, d.tiles_n)) * nks + ks) * (T * T);
#pragma unroll
    for (int i = 0; i < Core::MI; ++i)
#pragma unroll
      for (int j = 0; j < Core::NI; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *(g_f32x4*)(part + il(i) * T + jl(j, g)) = f32x4{acc[i][j][4 * g], acc[i][j][4 * g + 1],
                                                           acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
    return;
  }

  if constexpr (PK == kApply) {
    // O through LDS (rows of T fp32 in the parameter's orientation, 16-byte slots XOR-permuted by the row),
    // then whole row segments: 16-byte slots when n % 4 == 0, else element by element, 64 in a row at a
    // time. The old parameter is loaded before the exchange (loaded after it, four at a time, the launch
    // took 136 us instead of 110 on seven 768/3072/1024x4096 fp32 matrices).
    const ApplyDesc& a = *d.fused;
    const bool tall = a.m > a.n;
    constexpr int SL = T / 4;  // slots per row
    auto at = [&](int r, int c) { return r * (T * 4) + (((c >> 2) ^ (r & (SL - 1))) << 4) + (c & 3) * 4; };
    const int64_t pr0 = int64_t(tall ? bj : bi) * T, pc0 = int64_t(tall ? bi : bj) * T;
    // (mode 1, the standalone output: p <- O, the words are not used)
    auto put = [&](const ParamWords<4>& p, int64_t i, const float (&o)[4]) {
      if (a.mode == 0) p.store(a.param, a.param_dtype, a.update_out, i, a.decay, a.step, o);
      else ParamWords<4>::write(a.param, a.param_dtype, i, o);
    };
    auto put1 = [&](const ParamWords<1>& p, int64_t i, const float (&o)[1]) {
      if (a.mode == 0) p.store(a.param, a.param_dtype, a.update_out, i, a.decay, a.step, o);
      else ParamWords<1>::write(a.param, a.param_dtype, i, o);
    };
    auto exchange = [&] {
#pragma unroll
      for (int i = 0; i < Core::MI; ++i)
#pragma unroll
        for (int j = 0; j < Core::NI; ++j)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const f32x4 o = f32x4{ldexpf(acc[i][j][4 * g], -ep), ldexpf(acc[i][j][4 * g + 1], -ep),
                                  ldexpf(acc[i][j][4 * g + 2], -ep), ldexpf(acc[i][j][4 * g + 3], -ep)};
            if (!tall) {
              *(l_f32x4*)(img + at(il(i), jl(j, g))) = o;
            } else {
#pragma unroll
              for (int k = 0; k < 4; ++k) *(l_f32*)(img + at(jl(j, g) + k, il(i))) = o[k];
            }
          }
      __syncthreads();
    };
    if ((a.n & 3) == 0) {
      constexpr int RPW = 64 / SL, NIT = T / (4 * RPW);  // rows per wave and pass, passes
      ParamWords<4> pw[NIT];
      auto row = [&](int it) { return (it * 4 + w) * RPW + lane / SL; };
      const int c = (lane % SL) * 4;
      const bool in = pc0 + c < a.n;
#pragma unroll
      for (int it = 0; it < NIT; ++it)
        if (a.mode == 0 && in && pr0 + row(it) < a.m) pw[it].load(a.param, a.param_dtype, (pr0 + row(it)) * a.n + pc0 + c);
      exchange();
#pragma unroll
      for (int it = 0; it < NIT; ++it)
        if (in && pr0 + row(it) < a.m) {
          const f32x4 o = *(l_f32x4*)(img + at(row(it), c));
          put(pw[it], (pr0 + row(it)) * a.n + pc0 + c, {o[0], o[1], o[2], o[3]});
        }
    } else {
      constexpr int CP = T / 64, NIT = T / 4 * CP;  // column passes, passes
      ParamWords<1> pw[NIT];
      auto row = [&](int it) { return (it / CP) * 4 + w; };
      auto col = [&](int it) { return (it % CP) * 64 + lane; };
#pragma unroll
      for (int it = 0; it < NIT; ++it)
        if (a.mode == 0 && pr0 + row(it) < a.m && pc0 + col(it) < a.n)
          pw[it].load(a.param, a.param_dtype, (pr0 + row(it)) * a.n + pc0 + col(it));
      exchange();
#pragma unroll
      for (int it = 0; it < NIT; ++it)
        if (pr0 + row(it) < a.m && pc0 + col(it) < a.n)
          put1(pw[it], (pr0 + row(it)) * a.n + pc0 + col(it), {*(l_f32*)(img + at(row(it), col(it)))});
    }
    return;
  } else {
    const int sw = h2_swz(fr & 15);
    const uint16_t* E = PK == kSquare ? static_cast<const uint16_t*>(d.E[parity]) : nullptr;
    const int64_t epanel = int64_t(d.lde) << 5;
    if constexpr (PK == kSquare) {
      // the addend's image as it lies; every lane then replaces its own elements
#pragma unroll
      for (int i = 0; i < PB * PB / 4; ++i) {
        const int b = i * 4 + w;
        __builtin_amdgcn_global_load_lds((const void*)(E + min(r0 + b / PB, mp - 1) * epanel +
                                                       int64_t(min(c0 + b % PB, np - 1)) * 512 + lane * 8),
                                         img + b * 1024, 16, 0, 0);
      }
      H2_WAIT_VMCNT(0);
      __syncthreads();
    }
    const float weight = PK != kUpdate && bi != bj ? 2.0f : 1.0f;  // a tile off the diagonal is stored twice
    const float kc = ldexpf(cc, eo - ep), kb = ldexpf(cb, eo - ea), diag = ldexpf(ca, eo);  // (square)
    TileStats stats;
#pragma unroll
    for (int i = 0; i < Core::MI; ++i)
#pragma unroll
      for (int j = 0; j < Core::NI; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          h2_lds* p = img + ((il(i) >> 4) * PB + (jl(j, g) >> 4)) * 1024 + (fr & 15) * 32 + (((g & 1) ^ sw) << 4) + fh * 8;
          float v[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const float x = acc[i][j][4 * g + k];
            v[k] = PK == kSquare ? kc * x : ldexpf(x, eo - ep);
            if constexpr (DYN) stats.add(PK == kSquare ? ldexpf(x, eq - ep) : v[k], weight);
          }
          if constexpr (PK == kSquare) {
            const h2_u32x2 eh = *(h2_lu2*)p, el = *(h2_lu2*)(p + 512);
            float e[4];
            h2_join2(eh.x, el.x, e[0], e[1]);
            h2_join2(eh.y, el.y, e[2], e[3]);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              v[k] += kb * e[k];
              if (bi == bj && il(i) == jl(j, g) + k) v[k] += diag;
            }
          }
          uint32_t h0, l0, h1, l1;
          h2_split2(v[0], v[1], h0, l0);
          h2_split2(v[2], v[3], h1, l1);
          *(h2_lu2*)p = h2_u32x2{h0, h1};
          *(h2_lu2*)(p + 512) = h2_u32x2{l0, l1};
        }
    if constexpr (DYN)  // (with a barrier of its own)
      put_stats<Core::NW>(stats, eo, PK == kGram ? &st->amax : PK == kUpdate ? &st->xmax[parity ^ 1] : nullptr,
                          PK == kGram ? &st->a2 : PK == kSquare ? &st->q2 : nullptr,
                          reinterpret_cast<float*>(smem + T * T * 4));
    else
      __syncthreads();
    const H2BlockLane bl(lane);
    h2_gu16* C = (h2_gu16*)d.C[parity];
    h2_gu16* CT = (h2_gu16*)(PK == kUpdate ? d.CT[parity] : d.C[parity]);
    const int64_t cpanel = int64_t(d.ldc) << 5, tpanel = int64_t(PK == kUpdate ? d.ldct : d.ldc) << 5;
#pragma unroll 4
    for (int i = 0; i < PB * PB / 4; ++i) {
      const int b = i * 4 + w, rp = r0 + b / PB, cb = c0 + b % PB;  // (uniform over the wave)
      if (rp >= mp || cb >= np || (PK != kUpdate && rp > cb)) continue;
      h2_u32x4 v = bl.read(img + b * 1024);
      const h2_u32x4 tv = bl.read_t(img + b * 1024);
      if (PK != kUpdate && rp == cb) v = bl.mirror(v, tv);
      *(h2_gu4*)(C + rp * cpanel + int64_t(cb) * 512 + bl.off / 2) = v;
      if (PK == kUpdate || rp != cb) *(h2_gu4*)(CT + cb * tpanel + int64_t(rp) * 512 + bl.off / 2) = tv;
    }
  }
}

// Sum of a split Gram product's partial tiles: one workgroup per 16-row slab of an upper tile. Thread t adds
// the ranges' 8 consecutive columns 8 (t % (T / 8)) of row t / (T / 8) in order, and stores them and, through
// LDS, the mirrored block rows. The block on the diagonal takes its lower triangle from its upper one, as in the
// unsplit product: (i, j) and (j, i) add their mixed products in different orders.
template <int T, bool DYN>
__global__ __launch_bounds__(2 * T) void ns_h2_sum_kernel(const GemmDesc* __restrict__ descs, int count, int parity,
                                                          NsH2Exponents he) {
  __shared__ float tt[16][T + 1];
  __shared__ float red[T / 16];
  int lo = 0, hi = count - 1;  // (ldct holds the problem's first block of this launch)
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (descs[mid].ldct <= int(blockIdx.x)) lo = mid; else hi = mid - 1;
  }
  const GemmDesc& d = descs[lo];
  if (d.nks <= 1) return;
  const int lb = int(blockIdx.x) - int(d.ldct);
  const int slab = lb % (T / 16), nks = d.nks;
  int rem = lb / (T / 16), bi = 0;
  const int64_t idx = rem;
  while (rem >= d.tiles_n - bi) rem -= d.tiles_n - bi++;
  const int bj = bi + rem;
  const int rp = bi * (T / 16) + slab, np = d.M >> 4;
  if (rp >= np) return;
  const int t = threadIdx.x, row = t / (T / 8), c8 = t % (T / 8);
  const g_cf32* part = (const g_cf32*)d.CT[parity] + idx * nks * (T * T) + (slab * 16 + row) * T + c8 * 8;
  f32x4 a = *(g_cf32x4*)part, b = *(g_cf32x4*)(part + 4);
  for (int k = 1; k < nks; ++k) {
    a += *(g_cf32x4*)(part + int64_t(k) * (T * T));
    b += *(g_cf32x4*)(part + int64_t(k) * (T * T) + 4);
  }
  NsH2State* st = ns_state(d.scale);
  const int ep = 2 * (DYN ? st->ex[parity] : he.ex + max(0, *ns_small(d.scale) + he.gx));
  const int eo = DYN ? gram_exponent(st->lam[parity], __uint_as_float(st->xmax[parity]), d.K) : he.ea;
  float v[8];
  TileStats stats;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    v[k] = ldexpf(a[k], eo - ep);
    v[4 + k] = ldexpf(b[k], eo - ep);
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    tt[row][c8 * 8 + k] = v[k];
    if constexpr (DYN) stats.add(v[k], bi != bj ? 2.0f : 1.0f);
  }
  h2_gu16* C = (h2_gu16*)d.C[parity];
  const int64_t ldc = d.ldc;
  auto put = [&](int64_t r, int64_t k0) {
    h2_u32x4 h, l;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      uint32_t x, y;
      h2_split2(v[2 * k], v[2 * k + 1], x, y);
      h[k] = x;
      l[k] = y;
    }
    h2_gu16* o = C + h2_index(r, k0, ldc);
    *(h2_gu4*)o = h;
    *(h2_gu4*)(o + kH2Lo) = l;
  };
  if constexpr (DYN) put_stats<T / 32>(stats, eo, &st->amax, &st->a2, red);  // (with a barrier of its own)
  else __syncthreads();
  const int gc = bj * T + c8 * 8;
  if ((gc >> 4) < np && (gc >> 4) >= rp) {
    if ((gc >> 4) == rp) {  // (then bi == bj)
      const int c0 = c8 * 8 - slab * 16;  // the thread's first column within the block
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (c0 + k < row) v[k] = tt[c0 + k][slab * 16 + row];
    }
    put(rp * 16 + row, gc);
  }
  // mirror: row `c` of the tile's columns, its 8 values of slab rows 8 h .. 8 h + 7
  const int c = t >> 1, h = t & 1, gm = bj * T + c;
  if ((gm >> 4) >= np || (gm >> 4) <= rp) return;
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = tt[8 * h + k][c];
  put(gm, rp * 16 + 8 * h);
}

// First iterate: X_0 = scale u in both layouts, from the momentum pass's fp32 u (panel blocked, stored
// orientation). One 64 x 64 tile per workgroup: a half wave converts a 16 x 16 block (8 consecutive columns
// per lane), the transposed blocks through LDS. HBM bound: 4 B read and 8 B written per element.
__global__ __launch_bounds__(256) void ns_h2_split_kernel(const PrepDesc* __restrict__ descs, int count) {
  __shared__ float tile[64][65];
  const PrepDesc& d = descs[find_entry(descs, count, blockIdx.x)];
  const int lt = blockIdx.x - d.tile_begin;
  const int64_t row0 = int64_t(lt / d.tiles_n) * 64, col0 = int64_t(lt % d.tiles_n) * 64;
  // (X_0's buffer in the stored orientation precedes the one that u is in; the matrix's scale follows its
  // partial sums)
  const int64_t tiles = int64_t(d.tiles_m) * d.tiles_n;
  uint8_t* x_out = static_cast<uint8_t*>(d.d_out) - tiles * (64 * 64 * 4);
  const float* scale = reinterpret_cast<const float*>(reinterpret_cast<const uint8_t*>(d.partials) +
                                                      ((tiles * 4 + 255) & ~int64_t(255)));
  const int small = *ns_small(scale);
  const float s = ldexpf(*scale, kNsH2First + small);
  if (lt == 0 && threadIdx.x == 0) {
    NsH2State* st = ns_state(scale);
    st->ex[0] = kNsH2First + small;
    st->lam[0] = ldexpf(1.0f, -2 * small);   // ||X_0||_F <= 2^-small
    st->xmax[0] = __float_as_uint(ldexpf(1.0f, -small));
    st->amax = 0;
    st->a2 = 0;
  }
  const int t = threadIdx.x, l = t & 31, row = l & 15, ch = l >> 4;
  auto put = [&](void* base, int64_t r, int64_t k0, int64_t ld, const float (&v)[8]) {
    h2_u32x4 h, q;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      uint32_t x, y;
      h2_split2(v[2 * k], v[2 * k + 1], x, y);
      h[k] = x;
      q[k] = y;
    }
    h2_gu16* o = (h2_gu16*)base + h2_index(r, k0, ld);
    *(h2_gu4*)o = h;
    *(h2_gu4*)(o + kH2Lo) = q;
  };
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int b = (t >> 5) + 8 * i;
    const int r = (b >> 2) * 16 + row, c = (b & 3) * 16 + ch * 8;
    const g_cf32* u = (const g_cf32*)d.d_out + blk_index(row0 + r, col0 + c, d.ld_d);
    const f32x4 x0 = *(g_cf32x4*)u, x1 = *(g_cf32x4*)(u + 4);
    float v[8];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = s * x0[k];
      v[4 + k] = s * x1[k];
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) tile[r][c + k] = v[k];
    put(x_out, row0 + r, col0 + c, d.ld_d, v);
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int b = (t >> 5) + 8 * i;
    const int r = (b >> 2) * 16 + row, c = (b & 3) * 16 + ch * 8;  // of the transposed tile
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = tile[c + k][r];
    put(d.t_out, col0 + r, row0 + c, d.ld_t, v);
  }
}

template <typename Core, bool DYN>
void launch_products(const GemmDesc* d, int count, int tiles, int product, int parity, float ca, float cb, float cc,
                     const NsH2Exponents& he, hipStream_t st) {
  switch (product) {
    case kGram: hipLaunchKernelGGL((ns_h2_kernel<Core, kGram, DYN>), dim3(tiles), dim3(256), 0, st, d, count, parity, ca, cb, cc, he); break;
    case kSquare: hipLaunchKernelGGL((ns_h2_kernel<Core, kSquare, DYN>), dim3(tiles), dim3(256), 0, st, d, count, parity, ca, cb, cc, he); break;
    case kUpdate: hipLaunchKernelGGL((ns_h2_kernel<Core, kUpdate, DYN>), dim3(tiles), dim3(256), 0, st, d, count, parity, ca, cb, cc, he); break;
    default: hipLaunchKernelGGL((ns_h2_kernel<Core, kApply, DYN>), dim3(tiles), dim3(256), 0, st, d, count, parity, ca, cb, cc, he); break;
  }
}
template <int T, bool DYN>
void launch_sum(const GemmDesc* d, int count, int blocks, int parity, const NsH2Exponents& he, hipStream_t st) {
  hipLaunchKernelGGL((ns_h2_sum_kernel<T, DYN>), dim3(blocks), dim3(2 * T), 0, st, d, count, parity, he);
}

}  // namespace

hipError_t launch_ns_h2(const GemmDesc* d, int count, int total_tiles, int product, int parity, float ca, float cb,
                        float cc, const NsH2Exponents* he, int tile, hipStream_t st) {
  using Small = H2Core<2, 2, 1, 1, 8>;
  using Large = H2Core<2, 2, 2, 2, 5>;
  const NsH2Exponents none{};
  if (total_tiles <= 0) return hipSuccess;
  if (tile == 64) {
    if (he) launch_products<Small, false>(d, count, total_tiles, product, parity, ca, cb, cc, *he, st);
    else launch_products<Small, true>(d, count, total_tiles, product, parity, ca, cb, cc, none, st);
  } else {
    if (he) launch_products<Large, false>(d, count, total_tiles, product, parity, ca, cb, cc, *he, st);
    else launch_products<Large, true>(d, count, total_tiles, product, parity, ca, cb, cc, none, st);
  }
  return hipGetLastError();
}
hipError_t launch_ns_h2_sum(const GemmDesc* d, int count, int blocks, int parity, const NsH2Exponents* he, int tile,
                            hipStream_t st) {
  const NsH2Exponents none{};
  if (blocks <= 0) return hipSuccess;
  if (tile == 64) {
    if (he) launch_sum<64, false>(d, count, blocks, parity, *he, st);
    else launch_sum<64, true>(d, count, blocks, parity, none, st);
  } else {
    if (he) launch_sum<128, false>(d, count, blocks, parity, *he, st);
    else launch_sum<128, true>(d, count, blocks, parity, none, st);
  }
  return hipGetLastError();
}
hipError_t launch_ns_h2_split(const PrepDesc* d, int count, int total_tiles, hipStream_t st) {
  if (total_tiles <= 0) return hipSuccess;
  hipLaunchKernelGGL(ns_h2_split_kernel, dim3(total_tiles), dim3(256), 0, st, d, count);
  return hipGetLastError();
}

}  // namespace mfsdp
