// CPU check of the fourth-root iteration's rules (root_rule.h) in 64-bit arithmetic, on spectra whose eigenvectors
// are spread over all entries, so that the largest element of M - I says little about its spectrum: every
// eigenvalue's root is accurate when the rules end the iteration, within the host's cap, and the end
// is not put off on easy spectra. Exit code 0 on success; every failure prints what it found.
#include <cstdio>
#include <utility>
#include <vector>

#include "root_rule.h"

using namespace mfsdp;

static int g_fail = 0;

struct Group {
  double lam;    // eigenvalue
  double count;  // how many
};

// Runs the iteration; returns the iterations taken and the largest relative error of a root's eigenvalue.
// max |M - I| is that of the diagonal, the mean of the eigenvalues of M - I: what eigenvectors that are spread
// evenly leave, and the smallest that any eigenvectors can.
static std::pair<int, double> run(const std::vector<Group>& g, double eps_rel, int cap) {
  double n2 = 0, d = 0;
  for (const Group& x : g) n2 += x.count * x.lam * x.lam, d += x.count;
  const double rho = eps_rel * std::sqrt(n2);
  double f2 = 0;
  for (const Group& x : g) f2 += x.count * (x.lam + rho) * (x.lam + rho);
  const double z = 1.0 / std::sqrt(f2);
  std::vector<double> M, X(g.size(), 1.0);
  for (const Group& x : g) M.push_back(z * (x.lam + rho));
  const std::vector<double> M0 = M;
  float resid = 3.0e38f;
  uint64_t sum = kRootSumOpen;
  int k = 0;
  for (bool end = false; k < cap && !end; ++k) {
    end = root_ends(sum);
    const float* t = resid < kRootSwitch ? kRootFinal : kRootAggressive;
    double mean = 0;
    f2 = 0;
    for (size_t i = 0; i < g.size(); ++i) {
      const double T = t[0] + M[i] * (t[1] + M[i] * t[2]);
      X[i] *= T;
      M[i] *= T * T * T * T;
      mean += g[i].count * (M[i] - 1.0) / d;
      f2 += g[i].count * (M[i] - 1.0) * (M[i] - 1.0);
    }
    resid = float(std::fabs(mean));
    sum = 0;  // many addends
    for (int w = 0; w < 4096; ++w) sum += root_sum_term(float(f2 / 4096));
  }
  double err = 0;
  for (size_t i = 0; i < g.size(); ++i) err = std::max(err, std::fabs(X[i] / std::pow(M0[i], -0.25) - 1.0));
  return {k, err};
}

int main() {
  for (double d : {2.0, 64.0, 384.0, 768.0, 2048.0, 8192.0, 12288.0, 65536.0})
    for (double eps_rel : {1e-4, 1e-6, 1e-7, 1e-8, 1e-9})
      for (double part : {0.0, 1.0 / d, 0.05, 0.12, 0.2, 0.3, 0.75, 0.999})
        for (double low : {0.0, 1e-3, 1e-4}) {
          const double n = std::max(part > 0.0 ? 1.0 : 0.0, std::floor(part * d));
          if (n >= d) continue;
          std::vector<Group> g;
          const int large = int(std::min(16.0, d - n));
          for (int i = 0; i < large; ++i) g.push_back(Group{0.5 + i / 15.0, (d - n) / large});
          if (n > 0) g.push_back(Group{low, n});
          const auto [k, err] = run(g, eps_rel, root4_iters(eps_rel, int64_t(d), 100));
          if (!(err <= 1e-6)) {
            ++g_fail;
            std::printf("FAIL d %g eps_rel %g, %g of eigenvalue %g: error %.2e after %d iterations\n", d, eps_rel, n, low,
                        err, k);
          }
          if (n == 0 && k > 7) {
            ++g_fail;
            std::printf("FAIL d %g eps_rel %g, flat: %d iterations\n", d, eps_rel, k);
          }
        }
  // the caller's own cap stays
  if (root4_iters(1e-6, 768, 5) != 5 || root4_iters(0.0, 768, 33) != 33) ++g_fail;
  // a NaN and huge sums never end it, and do not wrap
  if (root_ends(root_sum_term(std::nanf("")) * (uint64_t(1) << 19)) || root_ends(root_sum_term(3e38f))) ++g_fail;
  if (!root_ends(root_sum_term(0.0f) * (uint64_t(1) << 19))) ++g_fail;
  if (g_fail == 0) std::printf("root rule check ok\n");
  return g_fail ? 1 : 0;
}
