// ant_layout.cpp -- see ant_layout.h.
#include "ant_layout.h"

#include <algorithm>
#include <cmath>

namespace vp {

namespace {

// Points in space, looked up by coordinate to a tolerance: open addressing on
// the cell of a projection whose weights no array's symmetry knows (rows of one
// list may well share one or two coordinates).  Points that coincide share a cell
// all the same: probes() counts what the look-ups touched, for the caller to bound.
class Places {
 public:
  Places(double tol, int most) : tol_(tol), cell_(std::max(1e-3, 8.0 * tol)) {
    int bits = 4;
    while ((1 << bits) < 2 * most) ++bits;
    shift_ = 64 - bits;
    slot_.assign((size_t)1 << bits, -1);
    pos_.reserve(3 * (size_t)most);
  }
  void add(const double *x) { put(x, false); }
  void add_once(const double *x) { put(x, true); }  // not beside one within tol (of the same cell)
  int size() const { return (int)(pos_.size() / 3); }
  int64_t probes() const { return probes_; }
  const double *at(int i) const { return &pos_[3 * (size_t)i]; }
  bool near(int i, const double *x) const {
    const double *y = at(i);
    return std::fabs(y[0] - x[0]) <= tol_ && std::fabs(y[1] - x[1]) <= tol_ && std::fabs(y[2] - x[2]) <= tol_;
  }
  // Calls f(index) for every point within tol of x until it returns true.
  template <typename F>
  bool each(const double *x, F f) const {
    const double k = key(x);
    const int64_t lo = cell(k - kReach * tol_), hi = cell(k + kReach * tol_);
    for (int64_t c = lo; c <= hi; ++c)
      for (size_t h = hash(c); slot_[h] >= 0; h = next(h)) {
        ++probes_;
        if (near(slot_[h], x) && cell(key(at(slot_[h]))) == c && f(slot_[h])) return true;
      }
    return false;
  }

 private:
  static constexpr double kReach = 2.5;  // above the sum of the weights
  static double key(const double *x) { return x[0] + 0.7548776662466927 * x[1] + 0.5698402909980532 * x[2]; }
  int64_t cell(double v) const { return (int64_t)std::floor(v / cell_); }
  size_t hash(int64_t c) const { return (size_t)(((uint64_t)c * 0x9e3779b97f4a7c15ull) >> shift_); }
  size_t next(size_t h) const { return (h + 1) & (slot_.size() - 1); }
  void put(const double *x, bool once) {
    size_t h = hash(cell(key(x)));
    for (; slot_[h] >= 0; h = next(h)) {
      ++probes_;
      if (once && near(slot_[h], x)) return;
    }
    slot_[h] = size();
    pos_.insert(pos_.end(), x, x + 3);
  }
  double tol_, cell_;
  int shift_;
  std::vector<int> slot_;
  std::vector<double> pos_;
  mutable int64_t probes_ = 0;
};

// Probes of the tables that a search over b rows may have made: a list in general
// position takes some 2 a row, and up to 50 a new antenna and candidate for its
// place (5e6 at 900 antennas with gaps).  Where many antennas coincide, or
// baselines repeat, the tables degenerate into lists, and the search, quadratic
// then, is given up.
int64_t most_probes(int64_t b) { return 40 * b + 4000000; }

void plus(const double *x, const double *d, double *y) {
  for (int c = 0; c < 3; ++c) y[c] = x[c] + d[c];
}

// One pass over the first time step's rows.  rows (or null): the rows' own
// vectors, asked where a new antenna stands: at the place that the most other
// antennas have a row to.
struct Pass {
  std::vector<int32_t> P, Q;
  std::vector<int32_t> from, via;  // antenna a > 0: X_a = X_from[a] + uvw of row via[a] (- uvw of row ~via[a])
  bool run(int B, const double *uvw, double tol, int max_n, const Places *rows) {
    P.assign(B, -1);
    Q.assign(B, -1);
    from.assign(1, 0);
    via.assign(1, -1);
    Places places(tol, max_n);
    const double origin[3] = {0.0, 0.0, 0.0};
    places.add(origin);
    std::vector<char> used((size_t)max_n * max_n, 0);  // unordered pairs taken by earlier rows
    auto free_pair = [&](int p, int q) { return !used[(size_t)std::min(p, q) * max_n + std::max(p, q)]; };
    int cur = 0, last = 0;
    int64_t looks = 0;
    for (int b = 0; b < B; ++b) {
      const double *d = uvw + 3 * (size_t)b;
      const int n = places.size();
      int p = -1, q = -1;
      double y[3];
      // a complete list's next row ...
      plus(places.at(cur), d, y);
      if (last + 1 < n && places.near(last + 1, y) && free_pair(cur, last + 1)) {
        p = cur;
        q = last + 1;
      } else if (cur + 2 < n) {
        plus(places.at(cur + 1), d, y);
        if (places.near(cur + 2, y) && free_pair(cur + 1, cur + 2)) {
          p = cur + 1;
          q = cur + 2;
        }
      }
      // ... or any antennas found so far (on a complete list, the next one at most)
      for (int s = 0; s < (rows ? n : std::min(n, 2)) && q < 0; ++s) {
        p = cur + s < n ? cur + s : cur + s - n;
        ++looks;
        plus(places.at(p), d, y);
        places.each(y, [&](int c) {
          if (!free_pair(p, c)) return false;
          q = c;
          return true;
        });
      }
      if (q < 0) {  // a further antenna: the row's second, seen from the first, or its first
        if (n >= max_n) return false;
        int a = cur;
        double sign = 1.0;
        if (rows && n > 2) {
          const int m = std::min(n, 24);
          int best = -1;
          for (int s = 0; s < 2 * n && best < (m + 2) / 3; ++s) {
            const int i = cur + s / 2 < n ? cur + s / 2 : cur + s / 2 - n;
            const double g = s % 2 ? -1.0 : 1.0, w[3] = {g * d[0], g * d[1], g * d[2]};
            plus(places.at(i), w, y);
            int votes = 0;
            for (int k = 0; k < m; ++k) {
              const double *x = places.at((int)((int64_t)k * n / m));
              const double v[3] = {y[0] - x[0], y[1] - x[1], y[2] - x[2]}, r[3] = {-v[0], -v[1], -v[2]};
              auto any = [](int) { return true; };
              votes += rows->each(v, any) || rows->each(r, any);
            }
            looks += 8;
            if (votes > best) {
              best = votes;
              a = i;
              sign = g;
            }
          }
        }
        const double w[3] = {sign * d[0], sign * d[1], sign * d[2]};
        plus(places.at(a), w, y);
        places.add(y);
        from.push_back(a);
        via.push_back(sign > 0 ? b : ~b);
        p = sign > 0 ? a : n;
        q = sign > 0 ? n : a;
      }
      // lists in no order cost a search of every antenna per row: left alone
      if (looks > 3 * (int64_t)b + 2 * (int64_t)n * n + 1024) return false;
      if (places.probes() + (rows ? rows->probes() : 0) > most_probes(b)) return false;
      used[(size_t)std::min(p, q) * max_n + std::max(p, q)] = 1;
      P[b] = p;
      Q[b] = q;
      cur = p;
      last = q;
    }
    return true;
  }
};

}  // namespace

AntLayout find_antennas(int T, int B, const double *uvw, double tol, int max_n, bool check) {
  AntLayout r;
  if (T <= 0 || B <= 0 || max_n < 2 || !(tol > 0.0)) return r;
  // coordinates beyond this overflow the lookup's cells (and are no array's)
  for (int64_t i = 0; i < 3 * (int64_t)B; ++i)
    if (!(std::fabs(uvw[i]) < 1e9)) return r;
  Pass s;
  bool ok = s.run(B, uvw, tol, max_n, nullptr);
  const int64_t n0 = (int64_t)s.from.size();
  if (!ok || (B != n0 * (n0 - 1) / 2 && B != n0 * (n0 + 1) / 2)) {
    // not a complete list: place its antennas by vote
    Places rows(tol, B);
    bool fits = true;
    for (int b = 0; b < B && fits; ++b) {
      rows.add_once(uvw + 3 * (size_t)b);  // (asked for their presence only)
      fits = rows.probes() <= most_probes(b);
    }
    Pass v;
    if (fits && v.run(B, uvw, tol, max_n, &rows) && (!ok || v.from.size() < s.from.size())) {
      s = v;
      ok = true;
    }
  }
  if (!ok) return r;
  const std::vector<int32_t> &P = s.P, &Q = s.Q;
  const int n = (int)s.from.size();
  std::vector<double> xyz((size_t)T * n * 3);
  double dev = 0.0;
  for (int t = 0; t < T; ++t) {
    double *X = &xyz[(size_t)t * n * 3];
    const double *U = uvw + (size_t)t * B * 3;
    for (int c = 0; c < 3; ++c) X[c] = 0.0;
    for (int a = 1; a < n; ++a) {
      const double g = s.via[a] >= 0 ? 1.0 : -1.0, *u = U + 3 * (size_t)(s.via[a] >= 0 ? s.via[a] : ~s.via[a]);
      for (int c = 0; c < 3; ++c) X[3 * a + c] = X[3 * s.from[a] + c] + g * u[c];
    }
    if (t > 0 && !check) continue;
    double d0 = 0.0, d1 = 0.0, d2 = 0.0;
    for (int b = 0; b < B; ++b) {
      const double *x = X + 3 * (size_t)P[b], *y = X + 3 * (size_t)Q[b], *u = U + 3 * (size_t)b;
      const double e0 = std::fabs(y[0] - x[0] - u[0]), e1 = std::fabs(y[1] - x[1] - u[1]), e2 = std::fabs(y[2] - x[2] - u[2]);
      d0 = e0 > d0 ? e0 : d0;
      d1 = e1 > d1 ? e1 : d1;
      d2 = e2 > d2 ? e2 : d2;
    }
    dev = std::max(dev, std::max(d0, std::max(d1, d2)));
    if (!(dev <= tol)) return r;
  }
  r.n = n;
  r.xyz.swap(xyz);
  r.p.swap(s.P);
  r.q.swap(s.Q);
  r.dev = dev;
  return r;
}

std::vector<AntMacro> ant_macros(int n, int *channels) {
  std::vector<AntMacro> out;
  const int nb = (n + kAntBlk - 1) / kAntBlk;
  *channels = nb == 1 ? 4 : nb == 2 ? 2 : 1;
  auto fresh = []() {
    AntMacro m;
    m.nsup = 0;
    for (int i = 0; i < kAntSup; ++i) m.blk[i] = m.dk[i] = 0;
    for (int w = 0; w < kAntWaves; ++w) {
      m.a[w] = m.b[w] = -1;
      m.tri[w] = 0;
    }
    return m;
  };
  // Groups of up to 4 blocks: a group's own upper triangle (4 triangles and 6
  // pairs: 36 of the 16 x 16 tiles over 8 waves, two triangles to a wave) ...
  for (int g = 0; g < nb; g += 4) {
    const int ng = std::min(4, nb - g);
    AntMacro m = fresh();
    int w = 0;
    for (int dk = 0; dk < *channels; ++dk)
      for (int i = 0; i < ng; ++i) {
        m.blk[m.nsup] = g + i;
        m.dk[m.nsup] = dk;
        ++m.nsup;
      }
    // waves w and w + 4 share a SIMD: triangle waves (6 tiles) come first, so
    // that each meets a pair (4 tiles)
    const int nt = m.nsup;
    const bool two = *channels * ng * (ng - 1) / 2 + nt > kAntWaves;  // two triangles to a wave
    for (int i = 0; i < nt; i += two ? 2 : 1, ++w) {
      m.tri[w] = 1;
      m.a[w] = i;
      m.b[w] = two && i + 1 < nt ? i + 1 : -1;
    }
    for (int dk = 0; dk < *channels; ++dk)
      for (int i = 0; i < ng; ++i)
        for (int j = i + 1; j < ng; ++j, ++w) {
          m.a[w] = dk * ng + i;
          m.b[w] = dk * ng + j;
        }
    out.push_back(m);
  }
  // ... and between groups, 2 blocks by up to 4: a pair to a wave
  for (int g = 0; g < nb; g += 4)
    for (int h = g + 4; h < nb; h += 4) {
      const int ng = std::min(4, nb - g), nh = std::min(4, nb - h);
      for (int i0 = 0; i0 < ng; i0 += 2) {
        AntMacro m = fresh();
        const int ni = std::min(2, ng - i0);
        for (int i = 0; i < ni; ++i) m.blk[m.nsup++] = g + i0 + i;
        for (int j = 0; j < nh; ++j) m.blk[m.nsup++] = h + j;
        int w = 0;
        for (int i = 0; i < ni; ++i)
          for (int j = 0; j < nh; ++j, ++w) {
            m.a[w] = i;
            m.b[w] = ni + j;
          }
        out.push_back(m);
      }
    }
  return out;
}

}  // namespace vp
