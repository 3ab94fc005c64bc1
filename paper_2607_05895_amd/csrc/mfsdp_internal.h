// Internal descriptors and kernel launchers shared by the host library and the HIP kernels.
//
// Data layout in HBM for one Muon entry with stored shape m x n (r = min, s = max):
//   the NS iterate is kept in both layouts, zero padded to the NS tile size:
//     X[0], X[1]   r_pad x s_pad   (K = s_pad columns)   -- ping-pong over NS steps
//     XT[0], XT[1] s_pad x r_pad   (K = r_pad)           -- X^T of the same iterate
//     G            r_pad x r_pad   A = X X^T (symmetric)
//     H            r_pad x r_pad   B' = b A + c A A + a I (symmetric)
//   Zero padding is exact for the iteration: padded rows/columns of X give zero rows/columns of
//   A and B', and stay zero in B' X.
//   Every NS product is then an "NT" product C = P Q^T with both operands K-contiguous:
//     Gram      A = X X^T             P = Q = X,  K = s_pad
//     square    A A = A A^T           P = Q = A,  K = r_pad   (A symmetric)
//     update    B' X = B' (X^T)^T     P = B', Q = X^T, K = r_pad
//   The square product stores B' = c A A + b A + a I, so the update X' = a X + B X = B' X is a plain
//   product with no addend. It writes X' in both layouts so the next step again reads
//   K-contiguous operands.
//
//   All of these buffers are panel blocked (blk_index below): rows in blocks of 16, columns in
//   blocks of 32, each 16 x 32 block contiguous (1 KiB in bf16), the blocks of one 16-row panel
//   following each other along K. One K step of a 16-row slice of an operand is then one
//   contiguous KiB, which the GEMM's direct-to-LDS loads fetch as eight whole 128-B lines.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm_schedule.h"

namespace mfsdp {

// Element (r, k) of a panel-blocked buffer with K columns (K a multiple of 32, rows a multiple of
// 16). Eight consecutive k starting at a multiple of 8 are contiguous.
constexpr int kBlkRows = 16;
constexpr int kBlkCols = 32;
__host__ __device__ constexpr int64_t blk_index(int64_t r, int64_t k, int64_t K) {
  return (r >> 4) * (K << 4) + ((k >> 5) << 9) + ((r & 15) << 5) + (k & 31);
}

// Two floats to packed bf16 (lo in bits 0..15), round to nearest even, one v_cvt_pk_bf16_f32.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

constexpr int kDtF32 = 0;
constexpr int kDtBF16 = 1;

// A parameter update p <- p decay - step O of V = 1 or 4 consecutive elements, in two halves: the old words are
// loaded long before O is there. Four elements are one access at any address of their own type's alignment (rows
// of odd n): global memory takes unaligned vectors, split by the hardware only where they cross a line.
template <int V>
struct ParamWords {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2), aligned(2)));
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));
  template <typename T>
  using gptr = __attribute__((address_space(1))) T*;
  uint32_t w[V];  // fp32 bits
  __device__ __forceinline__ void load(const void* param, int dt, int64_t i) {
    if (dt == kDtBF16) {
      const gptr<const uint16_t> p = (gptr<const uint16_t>)param + i;
      if constexpr (V == 4) {
        const u32x2 x = *(gptr<const u32x2>)p;
        w[0] = x.x << 16;
        w[1] = x.x & 0xffff0000u;
        w[2] = x.y << 16;
        w[3] = x.y & 0xffff0000u;
      } else {
        w[0] = uint32_t(*p) << 16;
      }
    } else {
      const gptr<const uint32_t> p = (gptr<const uint32_t>)param + i;
      if constexpr (V == 4) {
        const u32x4 x = *(gptr<const u32x4>)p;
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = x[k];
      } else {
        w[0] = *p;
      }
    }
  }
  static __device__ __forceinline__ void write(void* param, int dt, int64_t i, const float (&r)[V]) {
    if (dt == kDtBF16) {
      const gptr<uint16_t> p = (gptr<uint16_t>)param + i;
      if constexpr (V == 4) *(gptr<u32x2>)p = u32x2{pack_bf16x2(r[0], r[1]), pack_bf16x2(r[2], r[3])};
      else *p = uint16_t(pack_bf16x2(r[0], 0.0f));
    } else {
      const gptr<uint32_t> p = (gptr<uint32_t>)param + i;
      if constexpr (V == 4)
        *(gptr<u32x4>)p = u32x4{__float_as_uint(r[0]), __float_as_uint(r[1]), __float_as_uint(r[2]), __float_as_uint(r[3])};
      else *p = __float_as_uint(r[0]);
    }
  }
  __device__ __forceinline__ void store(void* param, int dt, float* update_out, int64_t i, float decay, float step,
                                        const float (&o)[V]) const {
    float r[V];
#pragma unroll
    for (int k = 0; k < V; ++k) r[k] = __uint_as_float(w[k]) * decay - step * o[k];
    if (update_out) write(update_out, kDtF32, i, o);
    write(param, dt, i, r);
  }
};

// ---------------------------------------------------------------------------------------------
// prep: momentum EMA + Nesterov (or a plain copy for standalone NS), Sum u^2 partials, and the
// NS input written in both layouts. One 64 x 64 tile of the stored m x n matrix per workgroup.
constexpr int kMaxGradParts = 64;

struct PrepDesc {
  const void* grad;      // m x n, grad_dtype (the NS input for standalone NS); unused if nparts > 0
  float* momentum;       // m x n fp32, or null for standalone NS
  void* d_out;           // u in stored orientation, padded, panel blocked with ld_d columns
  void* t_out;           // u^T, panel blocked with ld_t columns (fp32 path: X_0's other layout, which
                         // the split pass writes)
  float* partials;       // one Sum u^2 per tile
  int64_t m, n;          // stored shape
  int64_t ld_d, ld_t;
  int32_t tiles_m, tiles_n;  // over the padded domain, 64 x 64
  int32_t grad_dtype;
  int32_t tile_begin;    // first global tile index of this entry
  // owner-side reduction: g = gscale * (parts[0] + ... + parts[nparts - 1]) in fp32, in that order,
  // optionally stored to gout (grad_dtype); nparts == 0 reads grad instead
  int32_t nparts;
  float gscale;
  void* gout;
  const void* parts[kMaxGradParts];
};

// norm finalize: scale = 1 / max(sqrt(Sum partials), eps), deterministic order.
struct NormDesc {
  const float* partials;
  int32_t count;
  float* scale;
};

// apply: p <- p (1 - lr wd) - lr f (oscale O), or out <- oscale O for standalone NS.
struct ApplyDesc {
  const void* o;         // O in stored orientation (ns dtype), panel blocked with ld_o columns
  void* param;           // m x n, param dtype (or NS output)
  float* update_out;     // optional fp32 m x n
  const float* scale;    // norm scale, applied when no NS step ran (K = 0)
  int64_t m, n, ld_o;
  int32_t param_dtype;
  int32_t use_scale;
  int32_t mode;          // 0 = Muon parameter update, 1 = write O to param (standalone NS)
  float decay;           // 1 - lr wd
  float step;            // lr f
  int32_t tiles_m, tiles_n;
  int32_t tile_begin;
};

// Grouped NT GEMM problem: C = alpha * P Q^T + beta * E, stored in C and/or transposed in CT.
// Every operand is panel blocked; the ld* fields are the column counts. Both ping-pong alternatives are kept, indexed by step parity.
struct GemmDesc {
  const void* P[2];
  const void* Q[2];
  const void* E[2];
  void* C[2];
  void* CT[2];
  const float* scale;    // per-matrix norm scale (used on the first NS step), may be null
  int64_t ldp, ldq, lde, ldc, ldct;
  int32_t M, N, K;       // padded sizes, multiples of the tile
  float alpha, beta;     // (the square product takes its coefficients per launch instead)
  int32_t alpha_scale_pow;  // on the first step alpha *= scale^pow
  int32_t beta_scale_pow;
  int32_t sym;           // 1: only tiles bi <= bj, stored to (bi,bj) and mirrored to (bj,bi)
  int32_t tiles_m, tiles_n;
  int32_t tile_begin;    // prefix over the problems of one launch
  int32_t tile_count;
  int32_t last_c, last_ct;  // on the last step: write C / CT (1) or skip (0)
  // update product: on the last step, apply the parameter update (or write the standalone NS
  // output) from the fp32 accumulators instead of storing the final iterate
  const ApplyDesc* fused;
  // bf16 Gram product with a split contraction (nks > 1): tile (bi, bj, range ks) stores its fp32
  // partial product in part (one 256 x 256 row-major tile per upper tile and range, at
  // ((upper index of (bi, bj)) * nks + ks) * 65536 floats) and a second pass adds the ranges in
  // order and stores A; 0 or 1: not split. (On the fp32 path the partials go to CT, the iterate's
  // other buffer, which is free then, and ldct is the problem's first block in the second pass.)
  float* part;
  int32_t nks;
  int32_t kper;  // bf16 path: K steps of 32 per range (the last range may be shorter)
};
// The fp32 path's scales (kernels_ns_h2.hip): a buffer's elements are held times 2^e, e from a bound on them. One
// step's exponents of X, A, B' and X' where the host's bounds hold for every matrix; else one matrix's state,
// formed on the device step by step, which lies kNsH2StateOffset bytes after the matrix's norm scale (the pairs
// alternate with the iterate's buffers).
struct NsH2Exponents {
  int32_t ex, ea, eb, exn;
  // A matrix whose norm is below eps starts at ||X_0||_F <= 2^-small (an int beside its norm scale, else 0) and stays
  // that far below the bounds but for the steps' growth: X and X' take 2^max(0, small + gx) and
  // 2^max(0, small + gxn) more.
  int32_t gx, gxn;
};
constexpr size_t kNsH2StateOffset = 64;
constexpr int kNsH2First = 15;  // X_0's exponent: its elements are at most 1
constexpr int kNsH2MaxSmall = 60;
struct NsH2State {
  int32_t ex[2], ea, eb, eq;  // exponents of X, A, B' and of A A in q2
  float lam[2];               // bound on lambda_max(A) of the step that reads this X
  uint32_t xmax[2], amax;     // largest |X|, |A| (bit patterns)
  unsigned long long a2, q2;  // sums of squares of A's and A A's elements, each times 2^e
};
static_assert(kNsH2StateOffset + sizeof(NsH2State) <= 256, "the norm scale's block");
// The exponent under which a buffer with this bound (>= 0, inf or NaN: unknown) stays below 2^14, a factor of four
// inside fp16's range.
__host__ __device__ __forceinline__ int ns_h2_exponent(float bound) {
  return 140 - int(__builtin_bit_cast(uint32_t, bound) >> 23 & 0xff);
}
// Bound on the singular values (and so the elements) of X' = (a + b A + c A^2) X where lam bounds A's eigenvalues:
// the largest |sqrt(y) (a + b y + c y^2)| over [0, lam], at its end or where a + 3 b y + 5 c y^2 = 0; 1 % for
// rounding.
__host__ __device__ __forceinline__ float ns_h2_next_bound(float lam, float a, float b, float c) {
  const float end = 1.001f * lam;
  float best = 0.0f;
  auto at = [&](float y) {
    if (!(y > 0.0f && y <= end)) return;
    const float p = __builtin_sqrtf(y) * __builtin_fabsf(a + y * (b + c * y));
    if (!(p <= best)) best = p;  // (keeps a NaN)
  };
  at(end);
  if (!(end < 3.0e38f)) return end;
  const float disc = 9.0f * b * b - 20.0f * a * c;
  if (disc >= 0.0f) {  // the roots q / (10 c) and 2 a / q, neither by a difference of like numbers
    const float q = -3.0f * b - __builtin_copysignf(__builtin_sqrtf(disc), b);
    if (c != 0.0f) at(q / (10.0f * c));
    if (q != 0.0f) at(2.0f * a / q);
  }
  return 1.01f * best;
}
// Upper index of tile (bi, bj), bi <= bj, of a symmetric problem with tm tiles per side (row-major
// over the upper triangle).
__host__ __device__ constexpr int upper_index(int bi, int bj, int tm) { return bi * tm - bi * (bi - 1) / 2 + (bj - bi); }

constexpr int kAdamWMaxPerLaunch = 32;
struct AdamWDesc {
  void* param;
  const void* grad;
  float* exp_avg;
  float* exp_avg_sq;
  int64_t numel;
  int32_t param_dtype, grad_dtype;
  int32_t block_begin;
};
struct AdamWBatch {
  AdamWDesc d[kAdamWMaxPerLaunch];
  int32_t count;
  float decay;           // 1 - lr wd
  float beta1, beta2;
  float omb1, omb2;      // 1 - beta1, 1 - beta2 (formed in double)
  float step_size;       // lr / (1 - beta1^t)
  float inv_sqrt_bc2;    // 1 / sqrt(1 - beta2^t)
  float eps;
};
constexpr int kAdamWBlockElems = 2048;

// Launchers (return hipError_t of the launch).
// reduce: the descriptors' gradients are reductions of gradient parts (nparts >= 1 for all)
hipError_t launch_prep(const PrepDesc* d_descs, int count, int total_tiles, int ns_dtype,
                       int reduce, float beta, float one_minus_beta, int nesterov, hipStream_t st);
hipError_t launch_norm(const NormDesc* d_descs, int count, float eps, hipStream_t st);
// product: 0 Gram, 1 square, 2 update (the order of the products in one NS step); 3 the last update with
// the fused parameter update (its descriptors carry `fused`)
// (ca, cb, cc): the NS step's coefficients (a_k, b_k, c_k), used by the square product.
// tile: the output tile, kTileBF16 or kTileBF16Small; the descriptors' tile grids and the schedule are in
// that tile.
hipError_t launch_gemm(const GemmDesc* d_descs, int total_tiles, const TileRef* d_sched, int ngroups, int product,
                       int parity, int first_step, int last_step, float ca, float cb, float cc, int tile,
                       hipStream_t st);
// The fp32 path's products (on split fp16): one workgroup per tile (and K range) in the order of the
// descriptors; ca, cb, cc: the step's a, b, c; he: its scales, or null for scales formed on the device. tile: 128 or
// 64.
hipError_t launch_ns_h2(const GemmDesc* d, int count, int total_tiles, int product, int parity, float ca, float cb,
                        float cc, const NsH2Exponents* he, int tile, hipStream_t st);
// Second pass of a split Gram product there (blocks: tile / 16 per upper tile of every problem).
hipError_t launch_ns_h2_sum(const GemmDesc* d, int count, int blocks, int parity, const NsH2Exponents* he, int tile,
                            hipStream_t st);
// X_0 = scale u in both layouts from the momentum pass's u; starts the matrix's NsH2State.
hipError_t launch_ns_h2_split(const PrepDesc* d, int count, int total_tiles, hipStream_t st);
hipError_t launch_apply(const ApplyDesc* d_descs, int count, int total_tiles, int ns_dtype,
                        hipStream_t st);
// The second pass of a split Gram product: for each job (problem e in the Gram launch's order,
// upper tile bi <= bj) the problem's nks partial tiles added in range order, scaled as the Gram
// epilogue scales, stored as A (bf16) at (bi, bj) and mirrored at (bj, bi).
hipError_t launch_gram_sum(const GemmDesc* d_descs, const TileRef* d_jobs, int njobs, int parity,
                           int first, int tile, hipStream_t st);
hipError_t launch_adamw(const AdamWBatch& batch, int total_blocks, hipStream_t st);

// NS tile sizes (padding granularity of the workspace buffers).
constexpr int kTileBF16 = 256;
// The bf16 products of a launch with few 256 x 256 tiles run on 128 x 128 tiles, two workgroups per CU
// (buffers stay padded to 256; where every product of a call runs on them, they cover the matrices padded to 128).
constexpr int kTileBF16Small = 128;
// The fp32 path pads to 64; its products run on 128 x 128 or 64 x 64 tiles, which may reach past the padding.
constexpr int kTileF32 = 64;
constexpr int kPrepRows = 64;                    // prep tile rows
constexpr int kPrepColsBF16 = 256;              // prep tile columns on the bf16 path (divides 256)
constexpr int kPrepColsF32 = 64;                 // prep tile columns on the fp32 path
constexpr int kApplyCols = 128;                 // apply tile columns (8 per thread per row)
constexpr int kApplyRows = 16384 / kApplyCols;  // 16 K elements per tile: 64 per thread

}  // namespace mfsdp
