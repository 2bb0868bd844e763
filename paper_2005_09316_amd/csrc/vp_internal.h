// vp_internal.h -- structures shared between the libvp host code and its
// gfx950 kernels.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dispatch.h"

namespace vp {

constexpr int kPairsMax = (kNmaxLimit / 32 + 1) * (kNmaxLimit / 32 + 2) / 2;
constexpr int kA32PerPair = 2 * 8 * 64;  // floats: [parity][K step of 2 orders][lane]

// Lookup table of the basis (the lookup-table variant): kLutSamples + 2 rows
// of kLutStride FP32 values.
constexpr int kLutSamples = 8192;
constexpr double kLutXMax = 32.0;
constexpr int kLutStride = 100;
constexpr size_t kLutBytes = (size_t)(kLutSamples + 2) * kLutStride * sizeof(float);

// By nodes: shapelet envelopes, or the sums of points and Gaussians, are
// evaluated at M Chebyshev nodes of the band and interpolated to the channels (M =
// 0: evaluated at every channel).
// Table: the nodes nu / c [kNodesStride], then the interpolation matrix as
// operands of 16 channels x 4 nodes: [K / 16][M / 4][64], both rounded up, lane
// l of a block holding channel 4 (l mod 4) + (l mod 16) / 4 and node l / 16 of it.
struct NodePlan {
  int M, Mp;                 // nodes, padded to a multiple of 4 (zero columns)
  double mid, half;          // the band in nu / c
};
constexpr int kPlans = 4;
constexpr int kNodesStride = 64;
inline size_t node_doubles(int K, int Mp) { return kNodesStride + (size_t)((K + 15) / 16) * 16 * Mp; }
constexpr int kNodesMaxChan = 4096;

// Per-(sky, observation) tables, built on the device.
struct Derived {
  double4 *pos;   // [J] (l, m, n-1, 0), components in order points, Gaussians, shapelets
  double4 *gq;    // [G] quadratic form of the Gaussian envelope exponent (base 2), metres^2
  double *sframe; // [S][12] a-vector(3), b-vector(3), (l, m, n-1)(3), pad(3)
  float *flux32;  // [J][Kpad]
  double *flux64; // [J][Kpad]
  // Nodes and interpolation (NodePlan; M = 0: none): [0] shapelets on the mixed
  // and [1] on the FP64 path, [2] points and Gaussians on the mixed and [3] on
  // the FP64 path, these with their fluxes at the nodes, [P + G][Mp].
  NodePlan plan[kPlans];
  double *interp[kPlans];
  double *nflux[2];
  // Points by antenna (null: not taken by antenna): sign(S) sqrt|S| x the
  // channel's scale [Kpad][Jp], then the largest |S| and 1 / scale^2 [Kpad] each.
  float *amp;
  double *amp_peak, *amp_unscale;
};

// Shapelet coefficient tiles (depend on the sky only).
struct ShpTiles {
  const float *a32;        // MFMA A-operand tiles, FP32
  const int64_t *a32_off;  // [S]
  const double *c64;       // dense signed coefficients [n1][ld], FP64
  const int64_t *c64_off;  // [S]
  const int32_t *c64_ld;   // [S] leading dimension (multiple of 8)
  const uint16_t *abf;     // BF16 split A tiles: [part][pair][parity][64][8]
  const int64_t *abf_off;  // [S]
  const int32_t *nmax;     // [S]
};

struct DeriveArgs {
  int P, G, S;
  const double *ra, *dec;          // [J]
  const double *g_maj, *g_min, *g_pa;  // [G]
  const double *s_beta1, *s_beta2, *s_pa;  // [S]
  double ra0, dec0;
  int K;                           // the interpolation tables (below), for plans with M > 0
  const double *fk;                // [Kpad] nu / c
  Derived d;
};

struct FluxArgs {
  int J, K, Kpad;
  const double *sref, *alpha;  // [J]
  const double *ra, *dec;      // [J], for the beam
  const double *freq;          // [K]
  double nu_ref;
  double ra0, dec0;
  double beam_fwhm, beam_nu_ref;
  int j0;                      // first shapelet component
  const int32_t *lpow;         // [J - j0] power q of ln(nu / nu_ref) multiplying a shapelet's flux, or null
  Derived d;                   // (its plans 2 and 3: fluxes at the nodes for the components before j0)
};

struct TileBuildArgs {
  int S;
  const int32_t *nmax;
  const int64_t *coeff_off;
  const double *coeffs;
  float *a32;
  const int64_t *a32_off;
  double *c64;
  const int64_t *c64_off;
  const int32_t *c64_ld;
  uint16_t *abf;
  const int64_t *abf_off;
};

constexpr int kOutPoints = 4;  // points that may go along with the outputs of shapelets by nodes

// Arguments common to the visibility tile kernels.
struct TileArgs {
  int64_t nrows;       // n_time * n_bl
  int K, Kpad;         // channels, padded to a multiple of kPgChan
  int n_rb, n_cb;      // row blocks, channel blocks (of the kernel's own channel width)
  const double *uvw;   // [nrows][3] metres
  const double *fk;    // [Kpad] nu_k / c (padded with the last channel)
  int P, G, S;
  Derived d;
  ShpTiles t;
  void *vis;           // output (predict) or data (subtract), [nrows][K] complex
  int subtract;        // 0: vis = V; 1: vis = vis - V
  int skip_points;     // 1: the points were taken by antenna; the Gaussians add to vis (or subtract from it)
  // The point/Gaussian kernels may take a part of the rows and channels (the
  // pointers above begin there, K and nrows are the part's): channels of a row of
  // vis, the part's first channel (a multiple of 16 by nodes), and the call's rows,
  // by which kernel and workgroups are chosen whatever the part.
  int ld, chan0;
  int64_t call_rows;
  const double2 *sums; // [nrows][K] the points' sums, to be added to the Gaussians' (null: they are in vis)
  int c64;             // 1: complex64, 0: complex128
  int conj;            // 1 when the exponent sign is -1
  const float *lut;    // basis table of the lookup-table variant, or null
  double dfk;          // (nu_{k+1} - nu_k) / c when the channels are uniformly spaced
  int uniform;         // 1: channels uniformly spaced (the mixed path rotates phasors by dfk)
  int shp_chan;        // channels of a workgroup of the mixed shapelet tile
  int out_points;      // points that the outputs of shapelets by nodes take along
  int fresh;           // 1: the shapelet pass starts from zero instead of reading vis (a
                       //    predict with no point/Gaussian pass before it)
};

// Lets a kernel without LDS of its own be launched with up to a CU's whole.  The
// setting is the kernel's, for every thread and context that launches it: always the
// same value, so that a launch never meets another's smaller one.
inline hipError_t whole_lds(const void *kernel) {
  return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 163840);
}

// Whether a grid of so many workgroups runs whole (its threads are counted in 32 bits:
// HIP launches a larger one cut short, without an error).
inline bool grid_fits(int64_t blocks, int threads) { return blocks <= 0xffffffffll / threads; }
constexpr int64_t kNodesMaxRows = 1ll << 28;  // so many, by nodes, whatever rows a workgroup takes (16 x 256 threads at the least)

// Points by antenna (vp_ant.hip).
constexpr int kAntMinPoints = 64;  // two blocks of 32 points: below, padding is most of the work
constexpr int kAntMaxN = 1024;     // antennas (the pair map takes 4 n^2 bytes)
struct AntMacro;
struct AntArgs {
  int T, B, K;            // time steps, baselines, channels
  int npad;               // antennas padded to whole blocks
  int J, Jp;              // points, padded to whole groups of blocks
  int nmac, max_sup;      // macros and the most blocks one of them stages
  int kpack, nkb;         // channels per workgroup, workgroups over the channels
  const AntMacro *mac;
  const double *xyz;      // [T][npad][3] antenna coordinates, metres (zero in the padding)
  const double *xyz_lo;   // [T][npad][3] what they are short of (FP64 path)
  const int32_t *rowmap;  // [npad][npad] row of pair (p, q) + 1, negative: conjugated, 0: none
  const double *fk;       // [Kpad] nu / c
  const double4 *pos;     // [J] l, m, n - 1
  const float *amp;       // [Kpad][Jp] (mixed path)
  const double *flux64;   // [J][Kpad] (FP64 path)
  int Kpad;
  const double *unscale;  // [Kpad] 1 / (the amplitudes' scale)^2 (mixed path)
  int neg;                // 1: some fluxes are negative
  int fine;               // 1: the more exact factors (irregular channels)
  void *vis;              // [T][B][K]
  int c64, conj, subtract;
};
struct AntAmpArgs {
  int J, Jp, Kpad;
  Derived d;
};

// Where the data are complex64, points by antenna hand their sums to the
// Gaussians' pass in FP64 (written to vis, they would be rounded to complex64
// between the two): through a workspace of [rows][channels] complex128, whole time
// steps at a time or, where one does not fit, some of the channels of one.  Such
// workspaces hold kSumsMin to kSumsMax bytes; a call's least part fits the former.
constexpr uint64_t kSumsMin = 64ull << 20, kSumsMax = 256ull << 20;
struct SumsSpace {
  double2 *p;
  uint64_t bytes;
};

// A serving job's mark: its sequence number, and the device wall clock when it
// was written (host-mapped memory).
struct ServeMark {
  uint64_t seq, clk;
};

// Kernel classes timed by vp_profile: tables, point/Gaussian, shapelet, calibration.
constexpr int kProfClasses = 4;

// Peel calibration (vp_calib.hip).
constexpr int kGainPairs = 128;           // up to this many, the solve keeps both tables of a cell on chip
constexpr int kPeelMaxAnt = 256;          // tiles per observation (one thread each)
constexpr size_t kPeelSmemMax = 163840;  // LDS per workgroup on gfx950
constexpr size_t kPeelWsMax = size_t(1) << 30;  // per-cell tables of one launch, bytes (at least one cell)

struct GainArgs {
  int T, B, K;            // cells are (time, channel); B baselines per time step
  int n_ant, n_iter, max_cg;
  double cg_tol2;         // squared relative residual that ends a CG solve
  const void *model;      // [T][B][K] complex ideal model I (same type as data)
  void *data;             // [T][B][K] complex data V; the residual on return when subtract
  int c64;                // 1: complex64, 0: complex128
  const int32_t *ant1, *ant2;  // [B] tiles of each baseline
  const int32_t *pair_bl;      // [n_ant (n_ant - 1) / 2] baseline of tile pair (i < j), -1 if none
  const int32_t *comp;         // [n_ant] connected component of each tile in the baseline graph, -1 if idle
  double2 *gains;         // [T][K][n_ant] output, or null
  double2 *gw;            // [T][n_ant][K] gains of every cell (workspace, read by the subtract pass)
  int cell0, ncell;       // the launch covers cells cell0 .. cell0 + ncell - 1 (cell = t K + k)
  // workspace: complex X and |I|^2 (float when w32, else double), [ncell][pairs]
  // up to kGainPairs tiles, else [ncell][n_ant][n_ant]
  void *xt;
  void *wf;
  int w32;                // 1 (mixed path): FP32 tables and FP32 W in the step's operator, FP64 sums
  int single_comp;        // 1: every tile with a baseline is in one connected component
};

// Device set-up (vp_kernels.hip): the recurrence constants, once per device
// and process (the device must be current).
constexpr int kMaxDevices = 64;
hipError_t device_init(int dev);
// Device address of this device's no-allocation scratch array (valid after
// device_init(dev) succeeded), or null.
void *noalloc_scratch(int dev);
// Size of that array: per-(sky, observation) tables of vp_predict_noalloc.
constexpr uint64_t kNoAllocScratchBytes = 64ull << 20;
// A second part of the array, behind the first, holds the points' amplitudes
// by antenna: 4 of the 12 bytes per (component, channel) above for the points
// padded to 32 (of 64 at the least) and 16 a channel, 6.2 bytes in place of 12,
// so that no pair the first part takes exceeds it.
constexpr uint64_t kNoAllocAmpBytes = 34ull << 20;
// A third part holds the interpolation tables of one path, shapelets' and points'
// (at most kNodesMaxChan channels x kNodesStride nodes each).
constexpr uint64_t kNoAllocNodeBytes = (uint64_t)kPlans / 2 * (kNodesMaxChan + 16) * kNodesStride * 8;
// A fourth, points' and Gaussians' fluxes at its nodes: room for every pair that the
// tables hold (12 bytes per component and padded channel in 64 MiB, 8 per
// component and node, at most half as many nodes as padded channels), so that the
// calls take the same kernels as vp_predict.
constexpr uint64_t kNoAllocNfluxBytes = 24ull << 20;

// A fifth, the points' sums on their way to the Gaussians (kSumsMin bytes).

// Host-side launchers (vp_kernels.hip).
hipError_t launch_derive(const DeriveArgs &a, hipStream_t s);
hipError_t launch_flux(const FluxArgs &a, hipStream_t s);
hipError_t launch_tiles_build(const TileBuildArgs &a, int max_nmax, hipStream_t s);
hipError_t launch_pg(const TileArgs &a, int prec, hipStream_t s);
hipError_t launch_shp(const TileArgs &a, int prec, int max_nmax, hipStream_t s);
hipError_t launch_pg_nodes(const TileArgs &a, int prec, hipStream_t s);
hipError_t launch_shp_nodes(const TileArgs &a, const NodePlan &p, int prec, int max_nmax, hipStream_t s);
hipError_t launch_lut_build(float *T, hipStream_t s);
hipError_t launch_ant_amp(const AntAmpArgs &a, hipStream_t s);
hipError_t launch_ant(const AntArgs &a, hipStream_t s);
hipError_t launch_ant_refine(int T, int B, int n, int npad, const double *uvw, const int32_t *rowmap, const double *xyz,
                             double *xyz_lo, unsigned long long *dev, hipStream_t s);
hipError_t launch_ant64(const AntArgs &a, hipStream_t s);
hipError_t launch_mark(ServeMark *m, uint64_t seq, hipStream_t s);
hipError_t launch_gain(const GainArgs &a, hipStream_t s);
hipError_t launch_gain_subtract(const GainArgs &a, hipStream_t s);
bool gain_supported(int n_ant);
size_t gain_smem_bytes(int n_ant, bool w64, int threads);
size_t gain_x_bytes(int n_ant, bool w32);     // of table X per cell
size_t gain_cell_bytes(int n_ant, bool w32);  // of tables X and W per cell

// sizes of per-shapelet tile storage
inline int64_t a32_floats(int nmax) { return (int64_t)shp_pairs(nmax) * kA32PerPair; }
inline int c64_ld(int nmax) { return ((nmax + 1) + 7) / 8 * 8; }
inline int64_t c64_doubles(int nmax) { return (int64_t)(nmax + 1) * c64_ld(nmax); }
inline int64_t abf_elems(int nmax) { return (int64_t)3 * shp_pairs(nmax) * kAbfPerPair; }

}  // namespace vp
