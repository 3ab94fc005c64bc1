// Descriptors and launchers of the Shampoo owner step (fp32 throughout).
//
// Every matrix the step works on lives in the workspace as a zero-padded row-major fp32 buffer
// whose row and column counts are multiples of kShTile (128), so the GEMM needs no edge
// handling. Caller buffers (gradient, parameter, statistics, preconditioners) keep their natural
// m x n / m x m / n x n row-major layout; small copy kernels move data across that boundary.
//
// Zero padding is exact for every product: a padded statistic S is block diagonal (the real block
// and a zero block), the root iteration keeps that structure (products of block-diagonal matrices),
// and the padded rows and columns of the gradient are zero, so they add nothing to P_L G P_R.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm_schedule.h"
#include "root_rule.h"

namespace mfsdp {

constexpr int kShTile = 128;     // GEMM output tile and padding granularity
constexpr int kShCopyTile = 64;  // copy / init / apply tile
// Convergence of the Newton inverse-root iteration (p = 1, 2): once max |M_k - I| over the real block
// is below this, the remaining change of X is below 5e-6 relative (T_k = I - (M_k - I)/p, then
// quadratic), and the side's remaining products are skipped.
constexpr float kShConvTol = 1e-5f;

// The fourth-root iteration (p = 4; root_rule.h):
constexpr float kRootDone = -1.0f;  // residual slot of a side whose last X update is done
// Every iterate is held as split fp16 (h2_core.h) under a power-of-two scale from a bound on its
// eigenvalues, which bound its elements: M <= 1, |U| <= 0.9, T^2 <= 3.46, T^4 <= 11.93 (each times its scale at
// most 2^14, a factor of four inside fp16's range) and X <= (z rho)^(-1/4), whose scale the scalar
// kernel forms. X lacks the factor z^(1/4) until it is converted back.
constexpr double kRootBound = 16384.0;
constexpr float kScM = 16384.0f, kScU = 16384.0f, kScT2 = 4096.0f, kScT4 = 1024.0f;
// Products of one iteration (RootDesc::op); a is the current row's a.
constexpr int kRootFirst = 1;  // T_0 = c M M + b M + a I (is X_1)
constexpr int kRootU = 2;      // U = T - a I = c M M + b M
constexpr int kRootX = 3;      // X' = X U + a X (small while M is: keeps X's rounding errors down)
constexpr int kRootT2 = 4;     // T^2 = U U + 2 a U + a^2 I (T_0 T_0 in the first iteration)
constexpr int kRootT4 = 5;     // T^4 = T^2 T^2
constexpr int kRootM = 6;      // M' = T^4 M

// C = alpha * P Q^T + beta * E + diag * I over one padded problem (P: M x K, Q: N x K, all
// row-major with the given row strides; M, N and K multiples of kShTile). sym: only tiles bi <= bj are computed; each is stored at
// (bi, bj) and transposed at (bj, bi). E may alias C (each element is read before it is written,
// by the same thread).
struct ShGemmDesc {
  const float* P;
  const float* Q;
  const float* E;
  float* C;
  int64_t ldp, ldq, lde, ldc;
  int32_t K;
  int32_t tiles_n;     // N / kShTile (= M / kShTile when sym)
  int32_t sym;
  int32_t tile_begin;  // prefix over the problems of one launch
  float alpha, beta, diag;
  // Newton inverse-root iteration only (null otherwise). Each side has two residual slots; iteration k
  // (parity q) reads slot q^1 (written by iteration k-1) and writes slot q:
  const float* conv_in;  // skip the product when this residual is below kShConvTol (and, with
                         // copy_on_skip, copy the tile of E into C instead)
  float* clear;          // set to 0 by the problem's first block before anything else
  float* resid_out;      // max |C - I| over the real block (rows, cols < valid), atomic max
  int32_t copy_on_skip;
  int32_t valid;
  // operand stored as bf16 (a bf16 gradient; row stride in elements): both P and Q, or Q alone
  int32_t p_bf16, q_bf16;
  // kShX3U: apply the parameter update p <- p decay - step C (and C to update_out) to the real block instead of
  // storing C
  const struct ShApplyDesc* fused;
};

// Boundary copies over 64 x 64 tiles of a padded rows_pad x cols_pad domain.
// in  (dir 0): dst[r][c] = src[r][c] inside rows x cols, 0 elsewhere; optional dstT[c][r] too
//              (dst may be null when dstT is set); both fp32, or both bf16 when dst_bf16 (for a
//              bf16 source: the copy is exact).
// out (dir 1): dst (caller, rows x cols fp32, row stride ld_dst) = src (padded fp32) inside.
struct ShCopyDesc {
  const void* src;
  void* dst;
  void* dstT;
  int64_t rows, cols;
  int64_t ld_src, ld_dst, ld_dstT;
  int32_t src_dtype;   // kDtF32 / kDtBF16 (dir 0)
  int32_t tiles_n;     // column tiles of the domain
  int32_t tile_begin;
  int32_t dst_bf16;    // dir 0: dst and dstT hold bf16
};

// Sum of squares and trace of a padded d_pad x d_pad statistic, in row chunks (fp64 partials).
struct ShNormDesc {
  const float* S;
  int64_t ld;
  int32_t rows_pad;
  int32_t chunk_rows;
  double* partials;    // 2 doubles per chunk: (sum S^2, trace part)
  int32_t nchunks;
  int32_t tile_begin;  // first block of this problem in the launch
};

// Root scalars of one problem from its partials: rho = eps + eps_rel ||S||_F,
// z over the real dimension d (p = 4: 1 / ||S + rho I||_F; else (1 + p) / (2 ||S + rho I||_F));
// out = {rho, z, z^(1/p)} and for p = 4 X's scale.
struct ShScalarDesc {
  const double* partials;
  int32_t nchunks;
  int32_t d;
  float* out;
};

// M = z (S + rho I), X = z^(1/p) I over the padded domain (the padded diagonal is rho as well).
struct ShInitDesc {
  const float* S;
  float* M;
  float* X;
  float* resid;        // the two residual slots: {0, not converged}
  int64_t ld;
  const float* sc;     // {rho, z, z^(1/p)}
  int32_t tiles_n;
  int32_t tile_begin;
};

// One product of the fourth-root iteration: C = alpha P Q + beta E + diag I on dp x dp symmetric h2
// operands (K = dp, a multiple of 128), alpha, beta and diag from op and the side's residual.
struct RootDesc {
  const uint16_t* P;
  const uint16_t* Q;
  const uint16_t* E;     // may be null
  uint16_t* C;
  const float* sc;       // {rho, z, z^(1/4), X's scale}
  // two residual slots per side; iteration k (parity q) reads slot q^1 and writes slot q
  const float* conv_in;
  float* clear;          // (tile (0, 0)) set to 0, or to kRootDone in the side's last iteration
  float* resid_out;      // max |C - I| over the real block, atomic max
  // and two slots of ||C - I||_F^2 over the real block (root_rule.h), read, cleared and added to alike
  const unsigned long long* sum_in;
  unsigned long long* sum_clear;
  unsigned long long* sum_out;
  int32_t* xsel;         // (tile (0, 0)) receives out_idx, the index of the X buffer written
  int32_t out_idx;
  int32_t K;
  int32_t valid;
  int32_t op;
};

// Conversions over the padded domain: in, M = z (S + rho I) in h2 from fp32; out, z^(1/4) X in fp32 from
// the X buffer that xsel names.
struct RootConvDesc {
  const float* S;
  uint16_t* M;
  const uint16_t* X0;
  const uint16_t* X1;
  float* out;
  const float* sc;
  float* resid;          // the two residual slots: {0, not converged}
  unsigned long long* sum;  // the two sum slots, likewise
  const int32_t* xsel;
  int32_t dp;
  int32_t tile_begin;    // 64 x 64 tiles
};

// p <- p (1 - lr wd) - lr U (U padded fp32), and optionally update_out = U.
struct ShApplyDesc {
  const float* U;
  int64_t ldu;
  void* param;
  float* update_out;
  int64_t m, n;
  int32_t param_dtype;
  int32_t tiles_n;
  int32_t tile_begin;
};

// kind: three-way bf16 splits (operands of any range), without or with the parameter update in every problem, the
// same of P with a bf16 Q, or all operands bf16; decay and step are those of the parameter update (kShX3U)
enum { kShX3, kShX3U, kShX1, kShB };
hipError_t launch_sh_gemm(const ShGemmDesc* d, int count, int total_tiles, int kind, float decay, float step,
                          hipStream_t st);
hipError_t launch_sh_copy(const ShCopyDesc* d, int count, int total_tiles, int dir, hipStream_t st);
hipError_t launch_sh_norm(const ShNormDesc* d, int count, int total_blocks, hipStream_t st);
hipError_t launch_sh_scalars(const ShScalarDesc* d, int count, double eps, double eps_rel, int p,
                             hipStream_t st);
hipError_t launch_sh_init(const ShInitDesc* d, int count, int total_tiles, hipStream_t st);
// tiles: one upper 128 x 128 tile per workgroup, in launch order
hipError_t launch_root(const RootDesc* d, const TileRef* tiles, int total_tiles, hipStream_t st);
hipError_t launch_root_conv(const RootConvDesc* d, int count, int total_tiles, int dir, hipStream_t st);
hipError_t launch_sh_apply(const ShApplyDesc* d, int count, int total_tiles, float decay, float step,
                           hipStream_t st);

}  // namespace mfsdp
