// dispatch.h -- which kernel a call's points, Gaussians and shapelets take: sizes
// in, decision out, free of any device code (tests/ evaluates the rules for its own
// cases).  Every line lies where measurement put it; both sides stand beside it.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "shp_nodes.h"

namespace vp {

constexpr double kLightSpeed = 299792458.0;  // m/s

// Tile geometry.  A tile is kTileRows consecutive (time, baseline) rows times
// a block of channels; one workgroup of kTileRows threads processes a tile.
constexpr int kTileRows = 256;
constexpr int kPgChan = 8;     // channels per point/Gaussian tile (per thread)
constexpr int kShpChan = 4;    // channels per shapelet tile
constexpr int kChunk = 64;     // components staged in LDS at a time
constexpr int kFlush = 8;      // components summed plainly before a Kahan step
constexpr int kFlushMixed = 16; // mixed path: components per FP64 add (two kFlush partials, summed in FP32)
constexpr int kNmaxLimit = 96; // largest n1 + n2
constexpr int kMBMax = 4;      // 32-row blocks of the n1 axis: ceil(97 / 32)

// The MFMA shapelet kernels keep only the 32 x 32 blocks of the signed
// coefficient matrix (32 rows of n1 by 32 orders of n2) that meet the
// triangle n1 + n2 <= N: block (chunk ch, row block mb) with
// 32 (ch + mb) <= N, chunk-major.  With q = N / 32 there are
// (q + 1)(q + 2) / 2 of them.
constexpr int shp_pairs(int nmax) { return (nmax / 32 + 1) * (nmax / 32 + 2) / 2; }
constexpr int kAbfPerPair = 2 * 64 * 8;  // BF16 values of one split part: [parity][lane][8]

// Precision paths, numbered as VP_PREC_*; 5 (the FP32-MFMA contraction of the
// mixed path) is retired and refused at the boundary.
enum Prec : int { kFP64 = 0, kMixed = 1, kMixedBf16 = 2, kFP32 = 3, kMixedBf16x2 = 4, kLut = 6 };

// ---------------------------------------------------------------------------
// points and Gaussians by channels
// ---------------------------------------------------------------------------

constexpr int kPgSplitTiles = 640;  // up to this many tiles, the components may be split too

// Whether an observation is so small that rows, channels and components are all
// split (k_pg_nodes over channels).  1,000 Gaussians, us each, against the tiles
// with split components: mixed, 2 tiles 0.040 for 0.068, 32 tiles 0.064 for
// 0.069, 128 tiles 0.21 for 0.12; FP64, where the tiles rotate phasors between
// channels, 0.13 for 0.15, then 0.26 for 0.15, and on irregular channels 0.26 for
// 0.34 at 32 tiles.
inline bool pg_small(bool f64, int64_t nt, int n, bool uniform) {
  // (a few components leave most lanes without one: a point on 2 tiles, 8.5 us for
  // 5.9 on the tiles in FP64)
  if (n < (f64 && !uniform ? 8 : 16)) return false;
  return nt <= (f64 ? (uniform ? 4 : 64) : 40);
}

// Whether the components are split over a workgroup's waves.  Per Gaussian, us: tiles
// by workgroups a CU (1 / 2 / 3), mixed 0.295, 0.44, 0.59, FP64 0.57, 1.03, 1.5;
// split, which fills the device evenly, 0.02 + 0.00079 a tile and 0.045 + 0.0021 (128
// to 635 tiles).  A wave takes whole groups of a chunk: of a few components, most
// waves have none, which costs about the root of the idle share (10 points, 508
// tiles, FP64: split 30 us, tiles 15.6; mixed 15.2 and 12.0).
inline bool pg_split(bool f64, int64_t nt, int P, int G) {
  const int n = P + G;
  if (nt > kPgSplitTiles || n == 0) return false;
  const int group = f64 ? kFlush : kFlushMixed;
  auto slots = [&](int m) {  // of the waves' time, in components
    const int rest = m % kChunk;
    return m - rest + 4 * group * (((rest + group - 1) / group + 3) / 4);
  };
  const double idle = (double)(slots(P) + slots(G)) / n * (1.0 + 3.0 / n);
  const int per_cu = (int)std::min<int64_t>(3, (nt + 255) / 256);
  const double tile = f64 ? (per_cu == 1 ? 0.57 : per_cu == 2 ? 1.03 : 1.5) : (per_cu == 1 ? 0.295 : per_cu == 2 ? 0.44 : 0.59);
  return (f64 ? 0.045 + 0.0021 * nt : 0.02 + 0.00079 * nt) * std::sqrt(idle) < tile;
}

// ---------------------------------------------------------------------------
// points and Gaussians by nodes
// ---------------------------------------------------------------------------

constexpr int kPgNB = 6;  // nodes (or channels) a lane of k_pg_nodes holds

// Rows of a workgroup of k_pg_nodes: those whose rounds of workgroups (as many as
// the CUs hold at the kernel's registers) end soonest, a component's staging and
// reads weighing the more the fewer rows share them.
inline int pg_node_rows(bool f64, int Mp, int64_t nrows, int64_t *slots) {
  const int nw = (Mp + kPgNB - 1) / kPgNB;
  *slots = 256 * std::max(1, 4 * (f64 ? 3 : 5) / nw);
  int LR = 64;
  double best = 0.0;
  for (int r = 64; r >= 16; r /= 2) {
    const int64_t wgs = (nrows + r - 1) / r;
    const double t = (double)((wgs + *slots - 1) / *slots) * (r + 4);
    if (best == 0.0 || t < best) {
      best = t;
      LR = r;
    }
  }
  return LR;
}

// Whether P points and G Gaussians cost less by nodes than by channels.  By nodes a
// launch, the staging of every 64 components and the outputs cost something before
// the first component is summed, and in FP64 a node costs what two channels of a
// regular grid do, where phasors are rotated.  Times in us, fitted to 1 to 300
// components on 190 to 69,000 rows x 16 to 384 channels by 6 to 48 nodes (rms 10% by
// channels, 13% and 19% by nodes; hence the margins, with which 4 of 1,625 measured
// calls are over 5% slower than by channels, and 2% of the gain is lost).  One
// point, 2,016 rows x 384 channels, mixed: 16.6 us by nodes, 9.7 by channels; 30
// points and 10 Gaussians, 32,512 rows x 64 channels by 20 nodes in FP64: 113 and 68.
inline bool pg_nodes_pay(bool f64, int P, int G, int Mp, int64_t nrows, int K, bool uniform) {
  int64_t slots = 0;
  const int LR = pg_node_rows(f64, Mp, nrows, &slots), nw = (Mp + kPgNB - 1) / kPgNB;
  const int64_t wgs = (nrows + LR - 1) / LR, nt = (nrows + kTileRows - 1) / kTileRows * ((K + kPgChan - 1) / kPgChan);
  const double full = (double)wgs / slots, values = 1e-6 * nrows * K;
  const double rounds = full > 1.0 ? 0.5 * (std::ceil(full) + full) : 0.6 + 0.4 * full;
  const int chunks = (P + kChunk - 1) / kChunk + (G + kChunk - 1) / kChunk;
  const double outs = LR / 16.0 * ((K + 15) / 16) / nw;  // of a wave
  if (f64) {
    const double node = 7.3 + rounds * ((1.43 * P + 2.68 * G) * LR / 64.0 + 2.45 * chunks + outs * (0.77 + 0.053 * Mp)) + 3.2 * values;
    const double chan = 7.4 + 4.35 * values + (1.07 * P + 1.72 * G) * (0.064 + 0.001 * nt) * (uniform ? 1.0 : 2.5);
    return node < 0.75 * chan;
  }
  const double node = 6.0 + rounds * ((0.43 * P + 0.69 * G) * LR / 64.0 + 2.54 * chunks + outs * (0.09 + 0.071 * Mp)) + 1.7 * values;
  const double chan = 6.9 + 2.03 * values + (0.35 * P + 0.64 * G) * (0.088 + 0.001 * nt) * (uniform ? 1.0 : 1.1);
  return node < 0.85 * chan;
}

// Nodes of points and Gaussians, or 0: where three channels or more go to a node, and
// there are components enough (pg_nodes_pay).  A row's phase per component is at
// most its length (b_max, metres, the longest) times the distance of the
// component's direction from the phase centre (apart, of unit vectors, the largest).
inline int pg_plan_nodes(bool f64, int P, int G, double apart, double b_max, double amax, double f_lo, double f_hi,
                         double beam_fwhm, double beam_nu_ref, int64_t nrows, int K, bool uniform) {
  if (P + G == 0 || K < 12) return 0;
  const double half = 0.5 * (f_hi - f_lo) / kLightSpeed, mid = 0.5 * (f_lo + f_hi) / kLightSpeed;
  const double reach = b_max * apart * (1.0 + 1e-9);
  if (!(reach * f_hi / kLightSpeed <= 262144.0)) return 0;  // the mixed kernel's phases are fixed-point, up to 2^19 turns
  const double w = 6.283185307179586477 * reach * half, delta = half / mid;
  double beam = 0.0;  // exponent of the beam, furthest component, middle of the band (see flux_at)
  if (beam_fwhm > 0.0) {
    const double rho = std::min(1.57079632679489662, 2.0 * std::asin(0.5 * apart) * (1.0 + 1e-9));
    const double x = rho * mid * kLightSpeed / (beam_fwhm * beam_nu_ref);
    beam = 4.0 * 0.69314718055994530942 * x * x;
  }
  if (!(pg_spread(delta, amax, beam) <= (f64 ? kPgSpreadFp64 : kPgSpreadMixed))) return 0;
  const int M = pg_nodes(w, delta, amax, f64 ? kNodesTolFp64 : kNodesTolMixed, beam);
  return M > 0 && 3 * M <= K && pg_nodes_pay(f64, P, G, (M + 3) / 4 * 4, nrows, K, uniform) ? M : 0;
}

// ---------------------------------------------------------------------------
// shapelets
// ---------------------------------------------------------------------------

constexpr int kF64Chunk = 16;     // orders of the second axis that the FP64 kernels hold at a time
constexpr int kNodeThreads = 256;

// Doubles of LDS the node values of S shapelets take.
constexpr size_t node_lds(int S, int Mp, int R) { return (size_t)S * 2 * Mp * R; }

// What an envelope of a shapelet costs goes by this: (N + 1)(N + 2) / 1000 on the
// FP64 path (coefficients), pairs of 32 orders on the mixed one (contractions).
inline double shp_size(int prec, int nmax) {
  return prec == kFP64 ? 1e-3 * (nmax + 1) * (nmax + 2) : shp_pairs(nmax);
}
// Channels of a workgroup of the mixed path's shapelet tiles: fewer where the tiles
// would leave CUs without one (2,524 rows x 13 channels: 40 workgroups of four
// channels, 48 us, 130 of one, 17 us).
inline int shp_channels(int64_t n_rb, int K) {
  int kc = kShpChan;
  while (kc > 1 && n_rb * ((K + kc - 1) / kc) < 256) kc /= 2;
  return kc;
}

// LDS beside the node values: the mixed path's coefficient tiles, the FP64
// path's chunk.
inline size_t node_base_bytes(int prec, int max_nmax) {
  if (prec == kFP64) return (size_t)(kNmaxLimit + 1) * kF64Chunk * sizeof(double);
  return (size_t)(prec == kMixedBf16x2 ? 2 : 3) * shp_pairs(max_nmax) * kAbfPerPair * sizeof(uint16_t);
}

// Rows of a workgroup, a multiple of 16 (the outputs' tile): those with which
// the last workgroups end soonest.  A workgroup takes as many passes of its
// threads over the envelopes as its (row, node) pairs need (quads of nodes on
// the FP64 path), staging and outputs beside them; two workgroups share a CU
// (registers) where the LDS holds both, and one alone there runs some 1.5 times as
// fast.  The costs, in cycles, are rough: they have to tell a last pass or round
// nearly empty from a full one (113,792 rows, 9 nodes of two shapelets of order
// 70: 112 rows, 98% of the lanes and 99% of two rounds at work, where 128 left
// 10% and 13%).  0: LDS for not even 16.
inline int node_rows(int prec, int max_nmax, int S, int M, int Mp, int64_t nrows) {
  const size_t base = node_base_bytes(prec, max_nmax), half = 81920, all = 163840;
  const bool f64 = prec == kFP64;
  const double eval = f64 ? 12.5 * (max_nmax + 1) * (max_nmax + 2) : 2200.0 * shp_pairs(max_nmax);
  int best_r = 0;
  double best = 0.0;
  for (int R = 16; R <= 128; R += 16) {
    const size_t lds = base + node_lds(S, Mp, R) * sizeof(double);
    if (lds > all) break;
    const int64_t items = f64 ? (int64_t)R * (Mp / 4) : (int64_t)R * M, wgs = (nrows + R - 1) / R;
    const double work = S * ((double)((items + kNodeThreads - 1) / kNodeThreads) * eval + 3000.0 + 75.0 * R);
    const int64_t slots = lds <= half ? 512 : 256, rest = wgs % slots;
    const double one = 1.0 / 1.5;
    const double t = work * ((wgs / slots) * (slots == 512 ? 1.0 : one) + (rest == 0 ? 0.0 : rest > 256 ? 1.0 : one));
    if (best_r == 0 || t < best) {
      best = t;
      best_r = R;
    }
  }
  return best_r;
}

// Whether the shapelets of a sky (their sizes together, see shp_size) cost less by
// nodes than by channels.  Both kernels evaluate envelopes in passes of 256 threads,
// two workgroups a CU (one alone takes 0.67 to 0.78 of the time); by nodes a pass
// holds as many (row, node) pairs as the LDS keeps rows of every shapelet's node
// values, 16 at the least: with many shapelets most of its lanes repeat others.
// Times in us a shapelet and round, fitted to 1 to 75 shapelets of order 8 to 70 on
// 9,400 to 69,000 rows x 12 to 150 channels (rms 4 to 8%; no choice of them costs
// over 3%).  20 of order 40, 32,512 rows x 20 channels in FP64: 1.80 ms by nodes, 1.00 by
// channels; 45 of order 20, 12 channels, mixed: by nodes 2.2 times the channels'.
inline bool shp_nodes_pay(int prec, int max_nmax, int S, double size, int M, int64_t nrows, int K) {
  const int Mp = (M + 3) / 4 * 4;
  const bool f64 = prec == kFP64;
  const int R = node_rows(prec, max_nmax, S, M, Mp, nrows);
  if (R == 0) return false;
  auto rounds = [](int64_t wgs, int64_t slots, double alone) {
    const int64_t rest = wgs % slots;
    return (wgs / slots) * (slots == 512 ? 1.0 : alone) + (rest == 0 ? 0.0 : rest > 256 ? 1.0 : alone);
  };
  const size_t lds = node_base_bytes(prec, max_nmax) + node_lds(S, Mp, R) * sizeof(double);
  const int64_t items = f64 ? (int64_t)R * (Mp / 4) : (int64_t)R * M;
  const double passes = (double)((items + kNodeThreads - 1) / kNodeThreads), outs = R / 16 * ((K + 15) / 16) / 4.0;
  const int64_t n_rb = (nrows + kTileRows - 1) / kTileRows;
  if (f64) {
    const double node = 13.6 + (passes * (4.05 * S + 15.7 * size) + 1.64 * S * outs) * rounds((nrows + R - 1) / R, lds <= 81920 ? 512 : 256, 0.67);
    const double chan = 11.4 + (5.16 * S + 15.5 * size) * rounds(n_rb * ((K + kShpChan - 1) / kShpChan), 512, 0.66);
    return node < chan;
  }
  const int kc = shp_channels(n_rb, K);
  const double node = 8.5 + (passes * (0.9 * S + 1.85 * size) + 1.26 * S + 1.35 * S * outs) * rounds((nrows + R - 1) / R, lds <= 81920 ? 512 : 256, 0.78);
  const double chan = 10.5 + (kc * (1.0 * S + 1.75 * size) + 1.4 * S) * rounds(n_rb * ((K + kc - 1) / kc), 512, 0.71);
  return node < chan;
}

// Nodes of S shapelets (sizes together, see shp_size), or 0: where that saves a sixth
// of the envelopes or more (a channel's interpolation, phase and flux cost about 0.035
// of one), and the kernel is the faster (shp_nodes_pay).  The highest order's nodes
// serve all of the sky's shapelets.
inline int shp_plan_nodes(bool f64, int S, int max_nmax, double size, double f_lo, double f_hi, int64_t nrows, int K) {
  if (S == 0) return 0;
  const int M = shp_nodes(max_nmax, f_lo, f_hi, f64 ? kNodesTolFp64 : kNodesTolMixed);
  if (M == 0 || M + 0.035 * K > 0.85 * K) return 0;
  // Nor where the channels' own tiles run side by side, all in a first round of
  // two workgroups per CU (513 rows x 201 channels, order 92, FP64: 93 us, by nodes
  // 101).
  const int64_t n_rb = (nrows + kTileRows - 1) / kTileRows;
  if (n_rb * (f64 ? (K + kShpChan - 1) / kShpChan : K) <= 512) return 0;
  return shp_nodes_pay(f64 ? kFP64 : kMixed, max_nmax, S, size, M, nrows, K) ? M : 0;
}

}  // namespace vp
