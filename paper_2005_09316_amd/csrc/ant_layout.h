// ant_layout.h -- the antennas behind a list of baselines, free of any device
// code.
//
// The uvw of an interferometer's baselines are differences of its antennas'
// coordinates, uvw_b = X_q - X_p, at every time step.  A point component's
// phase is linear in uvw, so its term is a product of one factor per antenna,
// e^{2 pi i t_q} conj(e^{2 pi i t_p}), and the sum over points for all
// baselines of one (time, channel) is a Hermitian matrix product: n factors
// per component in place of up to n^2 / 2 sines and cosines.  An observation
// is described by uvw per row alone, so the antennas are found from them.
#pragma once

#include <stdint.h>

#include <vector>

namespace vp {

struct AntLayout {
  int n = 0;                  // antennas found; 0: the rows are no such list
  std::vector<double> xyz;    // [T][n][3] metres, antenna 0 at the origin
  std::vector<int32_t> p, q;  // [B] antennas of each row: uvw = X_q - X_p (p > q possible)
  double dev = 0.0;           // largest |uvw - (X_q - X_p)| component over all rows, metres
};

// Finds antennas for the B rows of every one of T time steps (uvw [T][B][3],
// metres): every row gets a pair (p, q), no two rows the same unordered pair,
// and X_q - X_p agrees with the row to tol metres at each time step.  Rows may
// come in any order, orientation and subset; lists grouped by one antenna (as
// correlators write them) give the true antennas, and rows that cannot be
// tied to antennas found before (a gap in the list) get further ones, which
// are as exact.  At most max_n antennas; n = 0 when that does not suffice or
// the rows do not agree over time.  check = false: only the first time step is
// looked at (dev is its own); whether the others agree is the caller's to find.
AntLayout find_antennas(int T, int B, const double *uvw, double tol, int max_n, bool check = true);

// Tiling of the (p, q) plane for the kernels that form it: antennas in blocks
// of 32, workgroups ("macros") of up to kAntWaves waves.  A macro stages up
// to kAntSup blocks (an antenna block of one of the workgroup's channels
// each); each wave takes one pair of different blocks, or one or two blocks
// with themselves (their upper triangles).
constexpr int kAntBlk = 32;
constexpr int kAntSup = 6;
constexpr int kAntWaves = 8;
struct AntMacro {
  int32_t nsup;              // blocks staged
  int32_t blk[kAntSup];      // antenna block
  int32_t dk[kAntSup];       // channel offset within the workgroup
  int32_t a[kAntWaves];      // first block (index into blk) of each wave's work, -1: none
  int32_t b[kAntWaves];      // second block; for a triangle wave: its second triangle, or -1
  int32_t tri[kAntWaves];    // 1: triangles (a, a) and (b, b); 0: the pair (a, b)
};

// The macros that cover the upper triangle of n antennas once, and the
// channels that one workgroup takes (more than one for few antennas).
std::vector<AntMacro> ant_macros(int n, int *channels);

}  // namespace vp
