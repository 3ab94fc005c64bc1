// Split-fp16 operands ("h2") and the MFMA main loop over them: fp32-accurate products at a third of the
// fp16 matrix rate.
//
// An fp32 value x, scaled by a power of two s so that |x s| stays below 2^15, is held as two fp16 numbers,
// hi = fp16(x s) and lo = fp16(2^11 (x s - hi)): 22 to 23 significant bits down to 2^-28 of the buffer's
// bound, and an absolute error of at most 2^-51 of it below. A product of two such operands takes three fp16
// MFMAs per 16 k: hi.hi into one accumulator, lo.hi and hi.lo into another that is added at the end times
// 2^-11 (lo.lo is below 2^-22 of |x||y|, random in sign). The main accumulator is rounded a sixth as often as
// with the six products of a three-way bf16 split, so the error against 64 bits is smaller from K = 64 on.
//
// Layout of an R x K operand (K a multiple of 16, rows padded to 16): 16 x 16 blocks of 1 KiB, the blocks
// of a 16-row panel one after another along K; a block is its 512-byte plane of hi parts and then the
// plane of lo parts, each 16 rows of two 16-byte chunks (8 consecutive k), chunk c of row r in slot
// c ^ h2_swz(r). The footprint is fp32's. One global_load_lds wave instruction moves one block into
// LDS as it lies; 8 consecutive rows' fragments then fall in distinct banks (32 or 64 of 4 B).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mfsdp {

__host__ __device__ constexpr int h2_swz(int r) { return ((r >> 2) ^ (r >> 3)) & 1; }
// Index (in 16-bit units) of the hi part of element (r, k) of a buffer with K columns; its lo part is
// kH2Lo further. Eight consecutive k from a multiple of 8 are contiguous.
constexpr int kH2Lo = 256;
__host__ __device__ constexpr int64_t h2_index(int64_t r, int64_t k, int64_t K) {
  return (r >> 4) * (K << 5) + ((k >> 4) << 9) + ((r & 15) << 4) + ((((k >> 3) & 1) ^ h2_swz(int(r & 15))) << 3) +
         (k & 7);
}

typedef _Float16 h2_f16x8 __attribute__((ext_vector_type(8)));
typedef short h2_s16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 h2_f16x2 __attribute__((ext_vector_type(2)));
typedef float h2_f32x2 __attribute__((ext_vector_type(2)));
typedef float h2_f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t h2_u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t h2_u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) h2_u32x2 h2_gu2;
typedef __attribute__((address_space(1))) h2_u32x4 h2_gu4;
typedef __attribute__((address_space(1))) uint16_t h2_gu16;
typedef __attribute__((address_space(1))) const uint16_t h2_gcu16;
typedef __attribute__((address_space(3))) uint8_t h2_lds;
typedef __attribute__((address_space(3))) h2_u32x2 h2_lu2;
typedef __attribute__((address_space(3))) h2_u32x4 h2_lu4;
typedef __attribute__((address_space(3))) h2_s16x4 h2_ls4;

constexpr float kH2LoScale = 2048.0f;
// The two parts of two scaled values, packed (first value in the low half); round to nearest even.
__device__ __forceinline__ void h2_split2(float a, float b, uint32_t& hi, uint32_t& lo) {
  const h2_f16x2 h = __builtin_convertvector(h2_f32x2{a, b}, h2_f16x2);
  hi = __builtin_bit_cast(uint32_t, h);
  lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(h2_f32x2{kH2LoScale * (a - float(h.x)), kH2LoScale * (b - float(h.y))},
                                                         h2_f16x2));
}
// The two (scaled) values of packed parts.
__device__ __forceinline__ void h2_join2(uint32_t hi, uint32_t lo, float& a, float& b) {
  const h2_f16x2 h = __builtin_bit_cast(h2_f16x2, hi), l = __builtin_bit_cast(h2_f16x2, lo);
  a = float(h.x) + (1.0f / kH2LoScale) * float(l.x);
  b = float(h.y) + (1.0f / kH2LoScale) * float(l.y);
}

// s_waitcnt with only vmcnt constrained; with only lgkmcnt(0)
#define H2_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 0xF) | (((n) >> 4) << 14) | (7 << 4) | (0xF << 8))
#define H2_WAIT_LGKM0() __builtin_amdgcn_s_waitcnt(0xF | (7 << 4) | (0 << 8) | (3 << 14))

// WM x WN waves on a TM x TN output tile, each MI x NI blocks of 32 x 32; a stage holds one K step of 16
// (TM / 16 blocks of P, then TN / 16 of Q), and a ring of NST stages is filled by direct global->LDS loads,
// NST - 1 steps ahead of their use.
template <int WM_, int WN_, int MI_, int NI_, int NST_>
struct H2Core {
  static constexpr int WM = WM_, WN = WN_, MI = MI_, NI = NI_, NST = NST_;
  static constexpr int NW = WM * WN, TM = WM * MI * 32, TN = WN * NI * 32;
  static constexpr int PP = TM / 16, QP = TN / 16;   // panels of P and Q
  static constexpr int PL = PP / NW, QL = QP / NW;   // blocks per wave and step
  static constexpr int DLOADS = PL + QL;
  static constexpr int STAGE = (PP + QP) * 1024;
  static constexpr int NMF = MI * NI, NRD = MI + NI;
  static_assert(PP % NW == 0 && QP % NW == 0 && PL >= 1 && QL >= 1, "whole blocks per wave");

  // psrc[i] / qsrc[i]: this wave's i-th panel of P / Q (panel i NW + w) at k = 0, in 16-bit units, already
  // holding the lane's offset lane * 8.
  static __device__ __forceinline__ void issue(const uint16_t* const (&psrc)[PL], const uint16_t* const (&qsrc)[QL],
                                               int kt, h2_lds* stage, int w) {
#pragma unroll
    for (int i = 0; i < PL; ++i)
      __builtin_amdgcn_global_load_lds((const void*)(psrc[i] + int64_t(kt) * 512), stage + (i * NW + w) * 1024, 16, 0, 0);
#pragma unroll
    for (int i = 0; i < QL; ++i)
      __builtin_amdgcn_global_load_lds((const void*)(qsrc[i] + int64_t(kt) * 512), stage + (PP + i * NW + w) * 1024,
                                       16, 0, 0);
  }

  // The products of nk steps (even, >= 2) into acc (zero on entry). One barrier per step, between its hi.hi and its
  // two mixed products: before it a wave waits for its own loads of step kt + 1, after it the loads of step
  // kt + NST - 1 go into the stage of step kt - 1, whose fragments every wave has consumed, and the next
  // step's hi parts are read while the mixed products run.
  static __device__ __forceinline__ void loop(const uint16_t* const (&psrc)[PL], const uint16_t* const (&qsrc)[QL], int nk,
                                              uint8_t* smem, int w, int lane, h2_f32x16 (&acc)[MI][NI]) {
    const int wm = w / WN, wn = w % WN;
    const int fr = lane & 31, fh = lane >> 5;
    const int in = (fr & 15) * 32 + ((fh ^ h2_swz(fr & 15)) << 4);
    const int pbase = (wm * MI * 2 + (fr >> 4)) * 1024 + in;
    const int qbase = (PP + wn * NI * 2 + (fr >> 4)) * 1024 + in;
#pragma unroll
    for (int s = 0; s < NST - 1; ++s) issue(psrc, qsrc, s < nk ? s : nk - 1, (h2_lds*)(smem + s * STAGE), w);
    H2_WAIT_VMCNT((NST - 2) * DLOADS);
    __builtin_amdgcn_s_barrier();
    h2_f16x8 ph0[MI], qh0[NI], ph1[MI], qh1[NI], pl[MI], ql[NI];
    auto rd = [&](const uint8_t* sb, int part, h2_f16x8 (&pf)[MI], h2_f16x8 (&qf)[NI]) {
#pragma unroll
      for (int i = 0; i < MI; ++i) pf[i] = *reinterpret_cast<const h2_f16x8*>(sb + pbase + i * 2048 + part * 512);
#pragma unroll
      for (int i = 0; i < NI; ++i) qf[i] = *reinterpret_cast<const h2_f16x8*>(sb + qbase + i * 2048 + part * 512);
    };
    auto mm = [&](h2_f32x16 (&c)[MI][NI], const h2_f16x8 (&pf)[MI], const h2_f16x8 (&qf)[NI]) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) c[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(qf[j], pf[i], c[i][j], 0, 0, 0);
    };
    h2_f32x16 mix[MI][NI];  // 2^11 times the mixed products
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) mix[i][j] = h2_f32x16{};
    int cs = 0, ns = 1, fs = NST - 1;
    auto step = [&](int kt, h2_f16x8 (&ph)[MI], h2_f16x8 (&qh)[NI], h2_f16x8 (&phn)[MI], h2_f16x8 (&qhn)[NI]) {
      // the lo parts of this step are read while hi.hi multiplies
      rd(smem + cs * STAGE, 1, pl, ql);
      mm(acc, ph, qh);
#pragma unroll
      for (int i = 0; i < (NMF > NRD ? NMF : NRD); ++i) {
        if (i < NMF) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (i < NRD) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      // step kt + 1 has landed (later ones may be in flight); every wave is done with step kt - 1
      H2_WAIT_VMCNT((NST - 3) * DLOADS);
      __builtin_amdgcn_s_barrier();
      const int kl = kt + NST - 1;
      issue(psrc, qsrc, kl < nk ? kl : nk - 1, (h2_lds*)(smem + fs * STAGE), w);
      rd(smem + ns * STAGE, 0, phn, qhn);
      mm(mix, pl, qh);
      mm(mix, ph, ql);
#pragma unroll
      for (int i = 0; i < (2 * NMF > DLOADS ? 2 * NMF : DLOADS); ++i) {
        if (i < 2 * NMF) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (i < DLOADS) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        if (i < NRD) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      cs = ns;
      ns = ns + 1 == NST ? 0 : ns + 1;
      fs = fs + 1 == NST ? 0 : fs + 1;
    };
    rd(smem, 0, ph0, qh0);
    for (int kt = 0; kt < nk; kt += 2) {
      step(kt, ph0, qh0, ph1, qh1);
      step(kt + 1, ph1, qh1, ph0, qh0);
    }
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[i][j] += (1.0f / kH2LoScale) * mix[i][j];
    // the clamped tail loads have landed and every wave is done reading: the LDS is free
    H2_WAIT_VMCNT(0);
    __builtin_amdgcn_s_barrier();
  }
};

// Lane addressing of one 16 x 16 block's image (1 KiB) when a wave stores it with 16 bytes per lane: lane =
// 32 plane + 16 chunk + row. off: the lane's 16 bytes of the image. t0, t1: the LDS addresses of the two 4 x 16
// transposing reads whose results are the lane's 16 bytes of the transposed block (8 consecutive rows of
// column `row`); lane 4 r + c of each 16 addresses row r (+ 4), columns 4 c .. 4 c + 3.
struct H2BlockLane {
  int row, ch, off, t0, t1;
  __device__ __forceinline__ explicit H2BlockLane(int lane) {
    const int plane = lane >> 5;
    row = lane & 15;
    ch = (lane >> 4) & 1;
    off = plane * 512 + row * 32 + ((ch ^ h2_swz(row)) << 4);
    const int c = lane & 3, r0 = 8 * ch + ((lane >> 2) & 3), r1 = r0 + 4;
    t0 = plane * 512 + r0 * 32 + (((c >> 1) ^ h2_swz(r0)) << 4) + (c & 1) * 8;
    t1 = plane * 512 + r1 * 32 + (((c >> 1) ^ h2_swz(r1)) << 4) + (c & 1) * 8;
  }
  __device__ __forceinline__ h2_u32x4 read(const h2_lds* blk) const { return *(const h2_lu4*)(blk + off); }
  __device__ __forceinline__ h2_u32x4 read_t(h2_lds* blk) const {
    const h2_s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((h2_ls4*)(blk + t0));
    const h2_s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((h2_ls4*)(blk + t1));
    return __builtin_bit_cast(h2_u32x4, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
  }
  // v with the elements below the block's diagonal taken from the transposed block's bytes tv
  __device__ __forceinline__ h2_u32x4 mirror(h2_u32x4 v, h2_u32x4 tv) const {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int c = ch * 8 + 2 * k;
      const uint32_t m = (c < row ? 0xffffu : 0u) | (c + 1 < row ? 0xffff0000u : 0u);
      v[k] = (v[k] & ~m) | (tv[k] & m);
    }
    return v;
  }
};

}  // namespace mfsdp
