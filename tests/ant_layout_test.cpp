// Antennas behind lists of baselines (ant_layout.h), on the CPU: reads cases
// "n keep autos order jitter" from the command line, draws an array and its
// list, and prints what was found, for tests/test_antennas.py to judge.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <set>
#include <vector>

#include "../paper_2005_09316_amd/csrc/ant_layout.h"

using namespace vp;

int main(int argc, char **argv) {
  if (argc != 6) return 2;
  const int n = atoi(argv[1]), autos = atoi(argv[3]), order = atoi(argv[4]), T = 3;
  const double keep = atof(argv[2]), jitter = atof(argv[5]);
  std::mt19937_64 rng(n * 1000 + order);
  std::uniform_real_distribution<double> U(-1500.0, 1500.0), U1(0.0, 1.0);
  std::vector<std::vector<double>> X(T, std::vector<double>(3 * n));
  for (auto &x : X)
    for (double &v : x) v = U(rng);
  std::vector<std::pair<int, int>> pairs;
  for (int i = 0; i < n; ++i)
    for (int j = i + (autos ? 0 : 1); j < n; ++j)
      if (U1(rng) < keep) pairs.push_back(order == 1 ? std::make_pair(j, i) : std::make_pair(i, j));
  if (pairs.empty()) pairs.push_back({0, n - 1});
  if (order == 2) std::shuffle(pairs.begin(), pairs.end(), rng);
  const int B = (int)pairs.size();
  std::vector<double> uvw((size_t)3 * B * T);
  for (int t = 0; t < T; ++t)
    for (int b = 0; b < B; ++b)
      for (int c = 0; c < 3; ++c)
        uvw[3 * ((size_t)t * B + b) + c] = X[t][3 * pairs[b].second + c] - X[t][3 * pairs[b].first + c];
  if (jitter > 0) uvw[3 * ((size_t)(T - 1) * B + B / 2) + 1] += jitter;  // one row at the last time
  const double tol = 1e-9;
  const AntLayout L = find_antennas(T, B, uvw.data(), tol, (int)(2.2 * std::sqrt((double)B)) + 8);
  // every row a pair of its own whose difference is the row, at every time
  int bad = 0;
  std::set<std::pair<int, int>> seen;
  for (int b = 0; b < B && L.n > 0; ++b) {
    const int p = L.p[b], q = L.q[b];
    if (p < 0 || q < 0 || p >= L.n || q >= L.n || !seen.insert({std::min(p, q), std::max(p, q)}).second) {
      ++bad;
      continue;
    }
    for (int t = 0; t < T; ++t)
      for (int c = 0; c < 3; ++c) {
        const double d = L.xyz[((size_t)t * L.n + q) * 3 + c] - L.xyz[((size_t)t * L.n + p) * 3 + c];
        if (!(std::fabs(d - uvw[3 * ((size_t)t * B + b) + c]) <= tol)) ++bad;
      }
  }
  // the macros cover every block pair of the upper triangle once per channel
  int channels = 0, uncovered = 0;
  if (L.n > 0) {
    const std::vector<AntMacro> M = ant_macros(L.n, &channels);
    const int nb = (L.n + kAntBlk - 1) / kAntBlk;
    std::multiset<std::vector<int>> got;
    for (const AntMacro &m : M) {
      if (m.nsup < 1 || m.nsup > kAntSup) ++uncovered;
      for (int w = 0; w < kAntWaves; ++w) {
        if (m.a[w] < 0) continue;
        if (m.a[w] >= m.nsup || m.b[w] >= m.nsup) ++uncovered;
        auto at = [&](int i, int j) {
          if (m.dk[i] != m.dk[j]) ++uncovered;
          got.insert({m.blk[i], m.blk[j], m.dk[i]});
        };
        if (m.tri[w]) {
          at(m.a[w], m.a[w]);
          if (m.b[w] >= 0) at(m.b[w], m.b[w]);
        } else {
          at(m.a[w], m.b[w]);
        }
      }
    }
    for (int i = 0; i < nb; ++i)
      for (int j = i; j < nb; ++j)
        for (int k = 0; k < channels; ++k)
          if (got.count({i, j, k}) != 1) ++uncovered;
    if ((int)got.size() != nb * (nb + 1) / 2 * channels) ++uncovered;
  }
  printf("%d %d %d %.3g %d %d\n", B, L.n, bad, L.dev, channels, uncovered);
  return 0;
}
