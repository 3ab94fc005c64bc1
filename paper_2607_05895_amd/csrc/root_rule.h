// The fourth-root iteration's coefficients and its rules for switching and ending (plain C++ with no HIP
// dependency, so that the CPU tests can follow the rules on their own).
//
// X <- X T, M <- T^4 M with T = a I + b M + c M^2, M_0 = z (S + rho I), z = 1 / ||S + rho I||_F, so that the
// spectrum of every M stays in (0, 1] (rounding aside).
#pragma once

#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace mfsdp {

// While max |M - I| >= kRootSwitch the coefficients are the aggressive row: the quadratic q for which
// f(x) = x q(x)^4 has its inner maximum and f(1) equal to 1 and its inner minimum equal to 0.7. Small
// eigenvalues grow by a^4 = 11.9 per iteration (Newton: (5/4)^4 = 2.44), and [0.0863, 1] maps into
// [0.7, 1], so no eigenvalue already near 1 is pushed far down again (which would cost it its relative
// accuracy: the unconstrained minimax quadratic grows 37-fold but loses a digit or two). Below
// kRootSwitch the row is the expansion of x^(-1/4) about 1 (third-order convergence; small eigenvalues grow by
// a^4 = 3.9). The switch looks at elements, which a few small eigenvalues hardly move: they then grow at the
// second row's rate, and the end waits for them.
constexpr float kRootAggressive[3] = {1.85835485f, -2.08442379f, 1.22606893f};
constexpr float kRootFinal[3] = {45.0f / 32.0f, -18.0f / 32.0f, 5.0f / 32.0f};
constexpr float kRootSwitch = 0.31f;

// The end: once ||M - I||_F, which no eigenvalue of M - I exceeds, is below kRootFinalTol, one last X update
// follows, nothing else (an eigenvalue 1 - e of M leaves 0.117 e^3 of X: 1.5e-8 at most). The largest element
// would not do: one eigenvalue 1 - x whose eigenvector is spread over d entries moves it by (1 - x) / d only.
// The squares are summed in units of 2^-40 (integers: their order does not matter), each addend rounded up
// and held to 2^4, so that the at most 2^19 addends (65536 x 65536, four waves per 128 x 128 upper tile) fit.
constexpr float kRootFinalTol = 5e-3f;
constexpr float kRootSumUnit = 1099511627776.0f;  // 2^40
constexpr uint64_t kRootSumOpen = uint64_t(1) << 62;  // before the first sum
constexpr uint64_t root_sum_term(float s) {  // (NaN: the largest)
  return s < 16.0f ? uint64_t(s * kRootSumUnit) + 1 : uint64_t(1) << 44;
}
constexpr bool root_ends(uint64_t sum) {
  return float(sum) * (1.0f / kRootSumUnit) < kRootFinalTol * kRootFinalTol;
}

// Iterations after which a side with this relative ridge has converged: the smallest eigenvalue of M_0 is at
// least eps_rel / (1 + eps_rel sqrt(d)) (half of it is taken, for rounding) and grows at least by the second row's
// a^4 per iteration up to 0.5; then 0.5 -> 0.918 -> 1 - 3e-4 -> 1 - 1e-11, the last X update, and one to
// spare. (Sides that end earlier skip their later products on the device.)
inline int root4_iters(double eps_rel, int64_t d, int iters) {
  const double l0 = 0.5 * eps_rel / (1.0 + eps_rel * std::sqrt(double(d)));
  if (!(l0 > 1e-30)) return iters;
  const double grow = std::pow(double(kRootFinal[0]), 4.0);
  const int k = int(std::ceil(std::max(0.0, std::log(0.5 / l0) / std::log(grow))));
  return std::min(iters, k + 5);
}

}  // namespace mfsdp
