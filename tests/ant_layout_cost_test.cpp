// What the search for antennas costs on lists that share coordinates, repeat
// baselines or have nothing to find: reads "n keep kind" from the command line and
// prints rows, antennas found, rows that disagree, and seconds, for
// tests/test_antenna_finder_cost.py to judge.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include "../paper_2005_09316_amd/csrc/ant_layout.h"

using namespace vp;

int main(int argc, char **argv) {
  if (argc != 4) return 2;
  const int n = atoi(argv[1]);
  const double keep = atof(argv[2]);
  const char *kind = argv[3];
  auto is = [&](const char *s) { return strcmp(kind, s) == 0; };
  std::mt19937_64 rng(n);
  std::uniform_real_distribution<double> U(-1500.0, 1500.0), U1(0.0, 1.0);
  std::vector<double> X(3 * (size_t)n), uvw;
  const int side = (int)std::ceil(std::sqrt((double)n));
  for (int i = 0; i < n; ++i) {
    for (int c = 0; c < 3; ++c) X[3 * i + c] = U(rng);
    if (is("plane") || is("line")) X[3 * i] = 0.0;
    if (is("line")) X[3 * i + 1] = 0.0;
    if (is("lattice")) X[3 * i] = 14.0 * (i % side), X[3 * i + 1] = 14.0 * (i / side), X[3 * i + 2] = 0.0;
    if (is("rail")) X[3 * i] = 5.0 * i, X[3 * i + 1] = X[3 * i + 2] = 0.0;
    if (is("one-place")) X[3 * i] = X[3 * i + 1] = X[3 * i + 2] = 0.0;
  }
  for (int i = 0; i < n; ++i)
    for (int j = i + 1; j < n; ++j)
      if (U1(rng) < keep)
        for (int c = 0; c < 3; ++c) uvw.push_back(is("random") ? U(rng) : X[3 * j + c] - X[3 * i + c]);
  const int B = (int)(uvw.size() / 3);
  const auto t0 = std::chrono::steady_clock::now();
  const double tol = 1.6e-10;
  const AntLayout L = find_antennas(1, B, uvw.data(), tol, std::min(1024, (int)(2.2 * std::sqrt((double)B)) + 8), false);
  const double s = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
  int bad = 0;
  for (int b = 0; b < B && L.n > 0; ++b)
    for (int c = 0; c < 3; ++c)
      if (!(std::fabs(L.xyz[3 * (size_t)L.q[b] + c] - L.xyz[3 * (size_t)L.p[b] + c] - uvw[3 * (size_t)b + c]) <= tol)) ++bad;
  printf("%d %d %d %.4f\n", B, L.n, bad, s);
  return 0;
}
