// vp_kernels.hip -- gfx950 kernels of libvp.
//
// Direct-Fourier visibility prediction (Line et al., Sec. 3): for every
// (time, baseline, channel) visibility, sum over point, Gaussian and shapelet
// components of flux x uv-envelope x phase term (Eqs. measure_eq_discrete,
// env_visi_def, gauss-env, shape-env).  A call takes its points on the matrix
// cores where that pays (vp_ant.hip), then points and Gaussians, then shapelets,
// each over tiles of (time, baseline) rows x a block of channels, or at a few
// frequencies of the band with interpolation to the channels (k_pg_nodes,
// k_shp_nodes, below):
//
//   k_pg_tile   points then Gaussians (k_pg_split: few tiles, the components
//               shared by four waves).  One thread owns one row and
//               kPgChan channels; component lists are staged through LDS in
//               chunks and read as wave-uniform broadcasts.  Phase per
//               (row, component) is t0 = u l + v m + w (n-1) in metres (FP64);
//               per channel t = t0 nu/c, reduced to a fraction of a turn in
//               FP64, then sin/cos of 2 pi t in FP32 on the transcendental
//               unit (input in turns); with uniformly spaced channels the
//               mixed path evaluates 3 of every 8 channels and the channel
//               step and rotates the other phasors.  Sums are plain FP32
//               over kFlush components; the mixed path adds two such
//               partials in FP32 and then into FP64 sums (the FP32-only
//               path: Kahan-compensated FP32 sums).
//   k_shp_mfma  shapelets.  Per (visibility, shapelet): rotate uvw into the
//               shapelet's frame, walk the rescaled Hermite recurrence for
//               both axes (FP64 on the mixed path: it costs the same issue
//               slots as FP32 on this chip and removes the argument-rounding
//               and underflow error of an FP32 recurrence), contract against
//               the signed coefficient matrix on MFMA (n1 on M, n2 on K split
//               by parity into real/imaginary accumulators, 32 visibilities on
//               N; 32 x 32 blocks that meet the n1 + n2 <= N triangle only;
//               v_mfma_f32_32x32x16_bf16 on 3-way BF16 splits of the FP64
//               values on the mixed path, v_mfma_f32_32x32x2_f32 on the
//               FP32-only path), fold each block's n1 sum against the first
//               axis (FP64 on the mixed path), and add flux x envelope x
//               phase into an FP64 accumulator held in LDS.
//   k_shp_fp64  the FP64 path of the shapelet term on the vector ALU (and
//               the lookup-table variant of the basis).
//
// All arithmetic is done with the exponent sign +1; a sign of -1 is applied
// by conjugating at the output, which is exact.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "shp_nodes.h"
#include "vp_internal.h"

namespace vp {

typedef float floatx16 __attribute__((ext_vector_type(16)));

__constant__ double c_sqn[128];   // sqrt(n)
__constant__ double c_isqn1[128]; // 1 / sqrt(n + 1)
__constant__ double c_half[128];   // n / 2
// scales of the rescaled Hermite values (see shp_tile): [0] = s_16 / s_0,
// [k] = s_{32k+16} / s_{32k-16} for k = 1, 2, 3, with s_n = sqrt(2^n / n!)
__constant__ double c_sc[4];

static constexpr double kPiM14 = 0.75112554446494248285870300477622; // pi^(-1/4)
static constexpr double kHalfLog2e = 0.72134752044448170367996234050095; // log2(e) / 2

// ---------------------------------------------------------------------------
// helpers
// ---------------------------------------------------------------------------

// The hardware dispatches consecutive workgroups round-robin over the 8 XCDs;
// give each XCD a contiguous range of logical tiles so that tiles sharing a
// channel block (and its flux-table rows) share that XCD's L2.
__device__ __forceinline__ int xcd_tile(int b, int nt) {
  const int q = nt >> 3, r = nt & 7, x = b & 7, i = b >> 3;
  return x * q + (x < r ? x : r) + i;
}

// cos/sin of 2 pi t for an FP64 phase in turns: exact FP64 reduction to
// [0, 1), then the FP32 transcendental unit (which takes turns).
__device__ __forceinline__ void turns_sincos_mixed(double t, float &c, float &s) {
  const float r = (float)__builtin_amdgcn_fract(t);
  s = __builtin_amdgcn_sinf(r);
  c = __builtin_amdgcn_cosf(r);
}

// The same of t0 f, |t0 f| < 2^19, by one fused multiply-add onto 1.5 2^20: the
// low word of the sum is the fraction in units of 2^-32, signed.
__device__ __forceinline__ void turns_sincos_fixed(double t0, double f, float &c, float &s) {
  const float r = (float)__double2loint(fma(t0, f, 1572864.0)) * 2.3283064365386963e-10f;
  s = __builtin_amdgcn_sinf(r);
  c = __builtin_amdgcn_cosf(r);
}

__device__ __forceinline__ void turns_sincos_f32(float t, float &c, float &s) {
  const float r = __builtin_amdgcn_fractf(t);
  s = __builtin_amdgcn_sinf(r);
  c = __builtin_amdgcn_cosf(r);
}

__device__ __forceinline__ void turns_sincos_f64(double t, double &c, double &s) {
  const double r = t - rint(t);  // exact, |r| <= 1/2
  sincospi(2.0 * r, &s, &c);
}

template <typename T>
__device__ __forceinline__ void kahan_add(T &sum, T &cmp, T x) {
  const T y = x - cmp;
  const T t = sum + y;
  cmp = (t - sum) - y;
  sum = t;
}

// Four channels of one row, from k on (n of them within the row): vis = (add ?
// vis : 0) + (re, im).  complex64 goes as two 16-byte accesses where every such
// group is aligned (wide: even rows on a 16-byte base); as single values, lanes
// apart by rows, each access leaves most of its sectors unused (119 -> 96 us of
// outputs at 32,640 rows x 384 channels).
__device__ __forceinline__ bool vis_wide(const TileArgs &a) { return a.c64 && a.ld % 2 == 0 && ((uintptr_t)a.vis & 15) == 0; }
__device__ __forceinline__ void vis_put4(const TileArgs &a, bool wide, bool add, int64_t idx, int n, const double (&re)[4],
                                         const double (&im)[4]) {
  if (wide && n >= 4) {
    float4 *o = (float4 *)((float2 *)a.vis + idx);
    float4 x = make_float4(0.f, 0.f, 0.f, 0.f), y = x;
    if (add) {
      x = o[0];
      y = o[1];
    }
    o[0] = make_float4((float)(re[0] + x.x), (float)(im[0] + x.y), (float)(re[1] + x.z), (float)(im[1] + x.w));
    o[1] = make_float4((float)(re[2] + y.x), (float)(im[2] + y.y), (float)(re[3] + y.z), (float)(im[3] + y.w));
    return;
  }
  if (!a.c64 && n >= 4) {  // (no test between the accesses: all four in flight)
    double2 *o = (double2 *)a.vis + idx;
    double2 d[4] = {make_double2(0.0, 0.0), make_double2(0.0, 0.0), make_double2(0.0, 0.0), make_double2(0.0, 0.0)};
    if (add)
#pragma unroll
      for (int r = 0; r < 4; ++r) d[r] = o[r];
#pragma unroll
    for (int r = 0; r < 4; ++r) o[r] = make_double2(re[r] + d[r].x, im[r] + d[r].y);
    return;
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (r >= n) break;
    if (a.c64) {
      float2 *o = (float2 *)a.vis + idx + r;
      const float2 d = add ? *o : make_float2(0.f, 0.f);
      *o = make_float2((float)(re[r] + d.x), (float)(im[r] + d.y));
    } else {
      double2 *o = (double2 *)a.vis + idx + r;
      const double2 d = add ? *o : make_double2(0.0, 0.0);
      *o = make_double2(re[r] + d.x, im[r] + d.y);
    }
  }
}

// (re, im) -= or += the points' sums of four channels of one row, from k on
// (signs as the Gaussians' in re, im).
__device__ __forceinline__ void add_sums(const TileArgs &a, int64_t row, int k, double (&re)[4], double (&im)[4]) {
  if (!a.sums) return;
  const double2 *s = a.sums + row * a.K;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double2 x = s[min(k + r, a.K - 1)];
    re[r] += a.subtract ? -x.x : x.x;
    im[r] += a.subtract ? -x.y : x.y;
  }
}

// ---------------------------------------------------------------------------
// per-(sky, observation) tables
// ---------------------------------------------------------------------------

// Direction cosines of every component relative to the phase centre, the
// Gaussian envelope's quadratic form, and each shapelet's frame vectors.
__device__ __forceinline__ void derive_one(const DeriveArgs &a, int j) {
  const double ra = a.ra[j], dec = a.dec[j];
  const double da = ra - a.ra0;
  const double sd = sin(dec), cd = cos(dec), sd0 = sin(a.dec0), cd0 = cos(a.dec0);
  // m = sin(dec) cos(dec0) - cos(dec) sin(dec0) cos(da) and n - 1 from
  // differences and half angles, where nothing large cancels
  const double dd = dec - a.dec0;
  const double hda = sin(0.5 * da), hdd = sin(0.5 * dd);
  const double l = cd * sin(da);
  const double m = fma(2.0 * cd * sd0, hda * hda, sin(dd));
  const double nm1 = -2.0 * fma(cd * cd0, hda * hda, hdd * hdd);
  a.d.pos[j] = make_double4(l, m, nm1, 0.0);
  if (j >= a.P && j < a.P + a.G) {
    // exponent of Eq. gauss-env in base 2:
    //   q = pi^2 / (4 ln2 ln2) * (kx^2 maj^2 + ky^2 min^2),
    //   kx = cos(pa) v + sin(pa) u, ky = -sin(pa) v + cos(pa) u
    // expanded in u^2, v^2, u v (metres; the channel scales it by (nu/c)^2).
    const int g = j - a.P;
    const double pa = a.g_pa[g], sp = sin(pa), cp = cos(pa);
    const double M2 = a.g_maj[g] * a.g_maj[g], N2 = a.g_min[g] * a.g_min[g];
    const double k = 3.14159265358979323846 * 3.14159265358979323846 /
                     (4.0 * 0.69314718055994530942 * 0.69314718055994530942);
    a.d.gq[g] = make_double4(k * (sp * sp * M2 + cp * cp * N2),   // u^2
                             k * (cp * cp * M2 + sp * sp * N2),   // v^2
                             k * 2.0 * sp * cp * (M2 - N2),       // u v
                             0.0);
  } else if (j >= a.P + a.G) {
    // Shapelet frame: (u', v', w') = T(ra_j, dec_j) T(ra0, dec0)^T (u, v, w),
    // T's rows being the east, north and pointing unit vectors.  Then
    // a = kappa beta1 (cos(pa) v' + sin(pa) u'), b = kappa beta2 (cos(pa) u' - sin(pa) v').
    const int s = j - a.P - a.G;
    const double sa0 = sin(a.ra0), ca0 = cos(a.ra0), sa = sin(ra), ca = cos(ra);
    const double T0[3][3] = {{-sa0, ca0, 0.0}, {-sd0 * ca0, -sd0 * sa0, cd0}, {cd0 * ca0, cd0 * sa0, sd0}};
    const double Tj[2][3] = {{-sa, ca, 0.0}, {-sd * ca, -sd * sa, cd}};
    double R[2][3];
    for (int r = 0; r < 2; ++r)
      for (int c = 0; c < 3; ++c) R[r][c] = Tj[r][0] * T0[c][0] + Tj[r][1] * T0[c][1] + Tj[r][2] * T0[c][2];
    const double kappa = 3.14159265358979323846 / sqrt(2.0 * 0.69314718055994530942);
    const double pa = a.s_pa[s], sp = sin(pa), cp = cos(pa);
    const double ka = kappa * a.s_beta1[s], kb = kappa * a.s_beta2[s];
    double *f = a.d.sframe + 12 * s;
    for (int c = 0; c < 3; ++c) {
      f[c] = ka * (sp * R[0][c] + cp * R[1][c]);
      f[3 + c] = kb * (cp * R[0][c] - sp * R[1][c]);
    }
    f[6] = l; f[7] = m; f[8] = nm1; f[9] = 0.0; f[10] = 0.0; f[11] = 0.0;
  }
}

// Node m of a plan (nu / c), and the sine of its angle.
__device__ __forceinline__ double node_at(const NodePlan &p, int m, double &sn) {
  double cs;
  sincospi((2 * m + 1) / (2.0 * p.M), &sn, &cs);
  return fma(p.half, cs, p.mid);
}

// Row k (a channel) of the interpolation matrix of plan i, one wave a row and
// one lane a node: barycentric weights of the Chebyshev nodes, normalised; a
// channel on a node takes that node alone.  Channels past the last and padding
// nodes are zero.
__device__ __forceinline__ void interp_row(const DeriveArgs &a, int i, int k) {
  const NodePlan &p = a.d.plan[i];
  const int m = threadIdx.x & 63;
  double *tab = a.d.interp[i];
  double sn;
  const double fm = node_at(p, m, sn);
  if (k == 0) tab[m] = m < p.M ? fm : p.mid;
  double w = 0.0;
  if (k < a.K) {
    const double dx = a.fk[k] - fm;
    const unsigned long long hit = __ballot(m < p.M && dx == 0.0);
    if (hit)
      w = m == __ffsll(hit) - 1 ? 1.0 : 0.0;
    else if (m < p.M)
      w = ((m & 1) ? -sn : sn) / dx;
  }
  double sum = w;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) sum += __shfl_xor(sum, o);
  if (k < a.K) w /= sum;
  const int c = k & 15;  // channel 4 g + r of its block is operand row 4 r + g
  if (m < p.Mp)
    tab[kNodesStride + ((size_t)(k >> 4) * (p.Mp >> 2) + (m >> 2)) * 64 + (m & 3) * 16 + 4 * (c & 3) + (c >> 2)] = w;
}

// Blocks of 128 threads: the components first, then two rows of the
// interpolation tables each.
__global__ __launch_bounds__(128) void k_derive(DeriveArgs a) {
  const int J = a.P + a.G + a.S, nj = (J + 127) / 128;
  if ((int)blockIdx.x < nj) {
    const int j = blockIdx.x * 128 + threadIdx.x;
    if (j < J) derive_one(a, j);
    return;
  }
  int row = 2 * ((int)blockIdx.x - nj) + (int)(threadIdx.x >> 6);
  const int K16 = (a.K + 15) / 16 * 16;
#pragma unroll
  for (int i = 0; i < kPlans; ++i) {
    if (a.d.plan[i].M == 0) continue;
    if (row < K16) {
      interp_row(a, i, row);
      return;
    }
    row -= K16;
  }
}

// S_j(nu) = S_ref (nu / nu_ref)^alpha * B_j(nu).
__device__ __forceinline__ double flux_at(const FluxArgs &a, int j, double nu) {
  double S = a.sref[j] * pow(nu / a.nu_ref, a.alpha[j]);
  if (a.lpow && j >= a.j0) {
    // spectral term q of a shapelet's coefficients: ln(nu / nu_ref)^q
    const double x = log(nu / a.nu_ref);
    for (int q = a.lpow[j - a.j0]; q > 0; --q) S *= x;
  }
  if (a.beam_fwhm > 0.0) {
    // distance from the phase centre: sin(rho) = sqrt(l^2 + m^2)
    const double dec = a.dec[j], da = a.ra[j] - a.ra0;
    const double l = cos(dec) * sin(da);
    const double m = sin(dec) * cos(a.dec0) - cos(dec) * sin(a.dec0) * cos(da);
    const double rho = asin(sqrt(l * l + m * m));
    const double th = a.beam_fwhm * a.beam_nu_ref / nu;
    S *= exp(-4.0 * 0.69314718055994530942 * rho * rho / (th * th));
  }
  return S;
}

// The channels' table, flat index j * Kpad + k (zero in the channel padding),
// then the nodes', j * Mp + m (zero in the node padding).
__global__ void k_flux(FluxArgs a) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t n = (int64_t)a.J * a.Kpad;
  if (a.d.amp && idx < a.Kpad) a.d.amp_peak[idx] = 0.0;  // k_ant_peak, next on the stream, takes the maximum
  if (idx < n) {
    const int j = (int)(idx / a.Kpad), k = (int)(idx % a.Kpad);
    const double S = k < a.K ? flux_at(a, j, a.freq[k]) : 0.0;
    a.d.flux32[idx] = (float)S;
    a.d.flux64[idx] = S;
    return;
  }
  idx -= n;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const NodePlan &p = a.d.plan[2 + i];
    if (p.M == 0) continue;
    const int64_t nn = (int64_t)a.j0 * p.Mp;
    if (idx < nn) {
      const int j = (int)(idx / p.Mp), m = (int)(idx % p.Mp);
      double sn;
      a.d.nflux[i][idx] = m < p.M ? flux_at(a, j, node_at(p, m, sn) * kLightSpeed) : 0.0;
      return;
    }
    idx -= nn;
  }
}

// Coefficient tiles.  Signed coefficients C''[n1][n2] = C[n1][n2] (-1)^floor((n1+n2)/2),
// so that xi = sum_{n1+n2 even} C'' phi phi + i sum_{n1+n2 odd} C'' phi phi
// equals sum C i^(n1+n2) phi phi.  The MFMA tiles hold the 32 x 32 blocks that
// meet the triangle, in pair order (chunk ch of 32 n2-orders outer, row block
// mb inner, 32 (ch + mb) <= N):
//   a32: [pair][parity][s][lane]: lane l supplies A[row = l % 32][k = l / 32] of
//        the 32x32x2 FP32 MFMA for n1 = 32 mb + l % 32,
//        n2 = 32 ch + 4 s + 2 (l / 32) + parity;
//   abf: [part][pair][parity][lane][8]: BF16 hi/mid/lo splits for the
//        32x32x16 MFMA, element e of lane l: n1 = 32 mb + l % 32,
//        n2 = 32 ch + 16 (l / 32) + 2 e + parity;
//   c64: [n1][ld], zero outside the triangle.
// The MFMA tiles hold C'' (s_n1 / s_{32 mb + 16}) (s_n2 / s_{32 ch + 16}): the
// kernels walk the rescaled Hermite values of psi_next (FP64 bases at the
// middle of each block), and these factors undo the rescaling.

// s_n / s_b with s_n = sqrt(2^n / n!), as a product of sqrt(2 / (k + 1)).
__host__ __device__ inline double herm_scale(int b, int n) {
  double r = 1.0;
  for (int k = b; k < n; ++k) r *= sqrt(2.0 / (k + 1));
  for (int k = n; k < b; ++k) r /= sqrt(2.0 / (k + 1));
  return r;
}

__device__ __forceinline__ double signed_coeff(const double *c, int N, int n1, int n2) {
  if (n1 < 0 || n2 < 0 || n1 > N || n2 > N - n1) return 0.0;
  const int64_t off = (int64_t)n1 * (N + 1) - (int64_t)n1 * (n1 - 1) / 2;
  const double v = c[off + n2];
  return (((n1 + n2) >> 1) & 1) ? -v : v;
}

__device__ __forceinline__ uint16_t bf16_rne(float x) {
  uint32_t u = __float_as_uint(x);
  const uint32_t lsb = (u >> 16) & 1u;
  u += 0x7fffu + lsb;
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf16_to_f(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

// (chunk, row block) of pair p; q = N / 32
__device__ __forceinline__ void pair_coords(int q, int p, int &ch, int &mb) {
  ch = 0;
  while (p > q - ch) {
    p -= q - ch + 1;
    ++ch;
  }
  mb = p;
}

__global__ void k_tiles(TileBuildArgs a) {
  const int s = blockIdx.y;
  if (s >= a.S) return;
  const int N = a.nmax[s];
  const double *C = a.coeffs + a.coeff_off[s];
  const int q = N / 32, npairs = shp_pairs(N);
  // FP32 MFMA tiles
  const int n32 = npairs * kA32PerPair;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n32; i += gridDim.x * blockDim.x) {
    const int lane = i & 63, st = (i >> 6) & 7, par = (i >> 9) & 1, p = i >> 10;
    int ch, mb;
    pair_coords(q, p, ch, mb);
    const int n1 = 32 * mb + (lane & 31), n2 = 32 * ch + 4 * st + 2 * (lane >> 5) + par;
    const double v = signed_coeff(C, N, n1, n2);
    a.a32[a.a32_off[s] + i] =
        v == 0.0 ? 0.f : (float)(v * herm_scale(32 * mb + 16, n1) * herm_scale(32 * ch + 16, n2));
  }
  // FP64 dense
  const int ld = a.c64_ld[s];
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < (N + 1) * ld; i += gridDim.x * blockDim.x) {
    const int n1 = i / ld, n2 = i % ld;
    a.c64[a.c64_off[s] + i] = signed_coeff(C, N, n1, n2);
  }
  // BF16 three-way split tiles
  const int nbf = npairs * kAbfPerPair;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nbf; i += gridDim.x * blockDim.x) {
    const int e = i & 7, lane = (i >> 3) & 63, par = (i >> 9) & 1, p = i >> 10;
    int ch, mb;
    pair_coords(q, p, ch, mb);
    const int n1 = 32 * mb + (lane & 31), n2 = 32 * ch + 16 * (lane >> 5) + 2 * e + par;
    const double v = signed_coeff(C, N, n1, n2);
    // split the FP64 value itself: each residual is formed in FP64 (exactly),
    // so the three parts carry ~27 bits instead of an FP32 rounding's 24
    const double x = v == 0.0 ? 0.0 : v * herm_scale(32 * mb + 16, n1) * herm_scale(32 * ch + 16, n2);
    const uint16_t hi = bf16_rne((float)x);
    const double r1 = x - (double)bf16_to_f(hi);
    const uint16_t mid = bf16_rne((float)r1);
    const double r2 = r1 - (double)bf16_to_f(mid);
    const uint16_t lo = bf16_rne((float)r2);
    uint16_t *dst = a.abf + a.abf_off[s];
    dst[i] = hi;
    dst[nbf + i] = mid;
    dst[2 * nbf + i] = lo;
  }
}

// ---------------------------------------------------------------------------
// point + Gaussian tile kernel
// ---------------------------------------------------------------------------

template <int PREC>
struct PgTypes {
  typedef float acc_t;
};
template <>
struct PgTypes<kFP64> {
  typedef double acc_t;
};

template <typename T>
struct PgSmem {
  double4 pos[kChunk];
  double4 gq[kChunk];
  T flux[kChunk][kPgChan];
};

// One tile: kTileRows rows x kPgChan channels starting at channel block cb.
// UNI (uniformly spaced channels): on the mixed path the phasors of channels
// 0, 3 and 6 of the tile are evaluated (FP64 phase, FP32 sincos) and the
// others are those rotated by one channel step, e^{+-2 pi i t0 dnu/c}: 4
// sincos and 5 complex rotations per (row, component) instead of 8 sincos,
// with at most one rotation between a channel and an evaluated phasor.  On
// the FP64 path channel 0 and the step are evaluated and channels 1-7 are
// reached by successive rotations.
// SPLIT (observations of a few tiles): the workgroup's four waves take the same
// 64 rows and a quarter of the components each, their sums meeting in LDS (part),
// so that four times as many workgroups have a quarter of the work.
template <int PREC, bool UNI = false, bool SPLIT = false>
__device__ __forceinline__ void pg_tile(const TileArgs &a, int rb, int cb,
                                        PgSmem<typename PgTypes<PREC>::acc_t> &sm,
                                        double (*part)[kPgChan][64][2] = nullptr) {
  static_assert(!UNI || ((PREC == kMixed || PREC == kFP64) && kPgChan == 8),
                "channel rotation: mixed and FP64 paths, 8-channel tiles");
  typedef typename PgTypes<PREC>::acc_t acc_t;
  constexpr int KB = kPgChan;
  double4 *s_pos = sm.pos;
  double4 *s_gq = sm.gq;
  auto &s_flux = sm.flux;
  const int k0 = cb * KB;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t row = SPLIT ? (int64_t)rb * 64 + (tid & 63) : (int64_t)rb * kTileRows + tid;
  const bool valid = row < a.nrows;
  const int64_t rowc = valid ? row : a.nrows - 1;
  const double u = a.uvw[3 * rowc], v = a.uvw[3 * rowc + 1], w = a.uvw[3 * rowc + 2];

  double f[KB];
#pragma unroll
  for (int k = 0; k < KB; ++k) f[k] = a.fk[k0 + k];

  // Partial sums over kFlush components in acc_t; across them, the mixed
  // path adds each pair of partials in FP32 (hld + prt; the pair's rounding
  // error stays within kFlush units of roundoff of its terms' magnitude) and
  // that into FP64 sums (FP64 adds issue at the FP32 rate here, and three
  // operations per value and pair replace Kahan's eight), the FP32-only path
  // keeps Kahan-compensated FP32 sums and the FP64 path Kahan-compensated
  // FP64 sums of its FP64 partials.
  acc_t sum_re[KB], sum_im[KB], cmp_re[KB], cmp_im[KB], prt_re[KB], prt_im[KB], hld_re[KB], hld_im[KB];
  double dsum_re[KB], dsum_im[KB];
#pragma unroll
  for (int k = 0; k < KB; ++k) {
    sum_re[k] = sum_im[k] = cmp_re[k] = cmp_im[k] = prt_re[k] = prt_im[k] = hld_re[k] = hld_im[k] = 0;
    dsum_re[k] = dsum_im[k] = 0.0;
  }

  // FP32-path copies of the row's coordinates
  const float uf = (float)u, vf = (float)v, wf = (float)w;
  float ff[KB], f2[KB];
#pragma unroll
  for (int k = 0; k < KB; ++k) {
    ff[k] = (float)f[k];
    f2[k] = (float)(f[k] * f[k]);
  }
  const acc_t uu = (acc_t)(u * u), vv = (acc_t)(v * v), uv = (acc_t)(u * v);
  // anchors of the rotation scheme: nu/c of tile channels 3 and 6 on the
  // uniform grid (also when they lie past the last channel)
  const double fa3 = fma(3.0, a.dfk, f[0]), fa6 = fma(6.0, a.dfk, f[0]);

  const int J0[2] = {a.skip_points ? a.P : 0, a.P};
  const int JN[2] = {a.P, a.P + a.G};
#pragma unroll
  for (int kind = 0; kind < 2; ++kind) {  // 0: points, 1: Gaussians
    for (int j0 = J0[kind]; j0 < JN[kind]; j0 += kChunk) {
      const int n = min(kChunk, JN[kind] - j0);
      __syncthreads();
      if (tid < n) {
        s_pos[tid] = a.d.pos[j0 + tid];
        if (kind == 1) s_gq[tid] = a.d.gq[j0 - a.P + tid];
      }
      for (int i = tid; i < n * KB; i += kTileRows) {
        const int jj = i / KB, k = i % KB;
        const int64_t fi = (int64_t)(j0 + jj) * a.Kpad + k0 + k;
        if (PREC == kFP64)
          s_flux[jj][k] = (acc_t)a.d.flux64[fi];
        else
          s_flux[jj][k] = (acc_t)a.d.flux32[fi];
      }
      __syncthreads();
      // one component's terms into the plain partial sums
      auto term = [&](int jj) {
        const double4 p = s_pos[jj];
        acc_t Q = 0;
        if (kind == 1) {
          const double4 g = s_gq[jj];
          if (PREC == kFP64)
            Q = fma(g.x, u * u, fma(g.y, v * v, g.z * (u * v)));
          else
            Q = fmaf((float)g.x, (float)uu, fmaf((float)g.y, (float)vv, (float)g.z * (float)uv));
        }
        if (PREC == kFP64 && UNI) {
          // FP64: channel 0's phasor and the channel step are evaluated,
          // channels 1-7 follow by successive rotations (each adds ~2e-16 of
          // the term: FP64 keeps a chain of seven far below its error bar)
          const double t0 = fma(u, p.x, fma(v, p.y, w * p.z));
          double c[KB], s[KB], cd, sd;
          turns_sincos_f64(t0 * f[0], c[0], s[0]);
          turns_sincos_f64(t0 * a.dfk, cd, sd);
#pragma unroll
          for (int k = 1; k < KB; ++k) {
            c[k] = fma(c[k - 1], cd, -s[k - 1] * sd);
            s[k] = fma(s[k - 1], cd, c[k - 1] * sd);
          }
          // Gaussian envelope 2^(-Q f_k^2) on the same grid f_k = f_0 + k df:
          // e_{k+1} = e_k r_k and r_{k+1} = r_k q, with r_0 = 2^(-Q df (2 f_0 + df))
          // and q = 2^(-2 Q df^2) (three exponentials instead of eight)
          double e = 1.0, r = 1.0, q = 1.0;
          if (kind == 1) {
            e = exp2(-(double)Q * (f[0] * f[0]));
            r = exp2(-(double)Q * a.dfk * (2.0 * f[0] + a.dfk));
            q = exp2(-2.0 * (double)Q * a.dfk * a.dfk);
          }
#pragma unroll
          for (int k = 0; k < KB; ++k) {
            double S = (double)s_flux[jj][k];
            if (kind == 1) {
              S *= e;
              e *= r;
              r *= q;
            }
            prt_re[k] = fma(S, c[k], (double)prt_re[k]);
            prt_im[k] = fma(S, s[k], (double)prt_im[k]);
          }
        } else if (PREC == kFP64) {
          const double t0 = fma(u, p.x, fma(v, p.y, w * p.z));
#pragma unroll
          for (int k = 0; k < KB; ++k) {
            double c, s;
            turns_sincos_f64(t0 * f[k], c, s);
            double S = (double)s_flux[jj][k];
            if (kind == 1) S *= exp2(-(double)Q * (f[k] * f[k]));
            prt_re[k] = fma(S, c, (double)prt_re[k]);
            prt_im[k] = fma(S, s, (double)prt_im[k]);
          }
        } else if (PREC == kFP32) {
          const float t0 = fmaf(uf, (float)p.x, fmaf(vf, (float)p.y, wf * (float)p.z));
#pragma unroll
          for (int k = 0; k < KB; ++k) {
            float c, s;
            turns_sincos_f32(t0 * ff[k], c, s);
            float S = (float)s_flux[jj][k];
            if (kind == 1) S *= __builtin_amdgcn_exp2f(-(float)Q * f2[k]);
            prt_re[k] = fmaf(S, c, (float)prt_re[k]);
            prt_im[k] = fmaf(S, s, (float)prt_im[k]);
          }
        } else if (UNI) {
          const double t0 = fma(u, p.x, fma(v, p.y, w * p.z));
          float c[KB], s[KB], cd, sd;
          turns_sincos_mixed(t0 * f[0], c[0], s[0]);
          turns_sincos_mixed(t0 * fa3, c[3], s[3]);
          turns_sincos_mixed(t0 * fa6, c[6], s[6]);
          turns_sincos_mixed(t0 * a.dfk, cd, sd);
          // one step up from channels 0, 3, 6; one step down from 3, 6
          c[1] = fmaf(c[0], cd, -s[0] * sd);
          s[1] = fmaf(s[0], cd, c[0] * sd);
          c[4] = fmaf(c[3], cd, -s[3] * sd);
          s[4] = fmaf(s[3], cd, c[3] * sd);
          c[7] = fmaf(c[6], cd, -s[6] * sd);
          s[7] = fmaf(s[6], cd, c[6] * sd);
          c[2] = fmaf(c[3], cd, s[3] * sd);
          s[2] = fmaf(s[3], cd, -c[3] * sd);
          c[5] = fmaf(c[6], cd, s[6] * sd);
          s[5] = fmaf(s[6], cd, -c[6] * sd);
#pragma unroll
          for (int k = 0; k < KB; ++k) {
            float S = (float)s_flux[jj][k];
            if (kind == 1) S *= __builtin_amdgcn_exp2f(-(float)Q * f2[k]);
            prt_re[k] = fmaf(S, c[k], (float)prt_re[k]);
            prt_im[k] = fmaf(S, s[k], (float)prt_im[k]);
          }
        } else {
          const double t0 = fma(u, p.x, fma(v, p.y, w * p.z));
#pragma unroll
          for (int k = 0; k < KB; ++k) {
            float c, s;
            turns_sincos_mixed(t0 * f[k], c, s);
            float S = (float)s_flux[jj][k];
            if (kind == 1) S *= __builtin_amdgcn_exp2f(-(float)Q * f2[k]);
            prt_re[k] = fmaf(S, c, (float)prt_re[k]);
            prt_im[k] = fmaf(S, s, (float)prt_im[k]);
          }
        }
      };
      // mixed path: a group's first kFlush terms are held aside and added to
      // the second kFlush terms' partial in FP32 before the FP64 add
      auto hold_partials = [&]() {
#pragma unroll
        for (int k = 0; k < KB; ++k) {
          hld_re[k] = prt_re[k];
          hld_im[k] = prt_im[k];
          prt_re[k] = prt_im[k] = 0;
        }
      };
      auto flush_partials = [&]() {
#pragma unroll
        for (int k = 0; k < KB; ++k) {
          if constexpr (PREC == kMixed) {
            dsum_re[k] += (double)(prt_re[k] + hld_re[k]);
            dsum_im[k] += (double)(prt_im[k] + hld_im[k]);
            hld_re[k] = hld_im[k] = 0;
          } else {
            kahan_add(sum_re[k], cmp_re[k], prt_re[k]);
            kahan_add(sum_im[k], cmp_im[k], prt_im[k]);
          }
          prt_re[k] = prt_im[k] = 0;
        }
      };
      // groups of kGroup components, unrolled, then the remainder
      constexpr int kGroup = PREC == kMixed ? kFlushMixed : kFlush;
      int jg = SPLIT ? wave * kGroup : 0;
      // FP64 terms hold twice the registers: two at a time keep two waves per SIMD
      constexpr int kUnroll = PREC == kFP64 ? 2 : kGroup;
      for (; jg + kGroup <= n; jg += SPLIT ? 4 * kGroup : kGroup) {
#pragma unroll kUnroll
        for (int jo = 0; jo < kGroup; ++jo) {
          if (kGroup > kFlush && jo == kFlush) hold_partials();
          term(jg + jo);
        }
        flush_partials();
      }
      if (jg < n) {  // (split: the wave whose group is the incomplete one)
        for (int jj = jg; jj < n; ++jj) {
          if (kGroup > kFlush && jj - jg == kFlush) hold_partials();
          term(jj);
        }
        flush_partials();
      }
    }
  }

  double tre[KB], tim[KB];
#pragma unroll
  for (int c = 0; c < KB; ++c) {
    tre[c] = PREC == kMixed ? dsum_re[c] : (double)sum_re[c] - (double)cmp_re[c];
    tim[c] = PREC == kMixed ? dsum_im[c] : (double)sum_im[c] - (double)cmp_im[c];
  }
  if constexpr (SPLIT) {
    if (wave > 0) {
#pragma unroll
      for (int c = 0; c < KB; ++c) {
        part[wave - 1][c][tid & 63][0] = tre[c];
        part[wave - 1][c][tid & 63][1] = tim[c];
      }
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int c = 0; c < KB; ++c)
      for (int q = 0; q < 3; ++q) {
        tre[c] += part[q][c][tid][0];
        tim[c] += part[q][c][tid][1];
      }
  }
  if (!valid) return;
  const bool wide = vis_wide(a), add = a.subtract || (a.skip_points && !a.sums);
#pragma unroll
  for (int k = 0; k < KB; k += 4) {
    if (k0 + k >= a.K) break;
    double re[4], im[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int c = k + r;
      re[r] = tre[c];
      im[r] = tim[c];
      if (a.subtract) re[r] = -re[r];
      if (a.subtract != a.conj) im[r] = -im[r];
    }
    add_sums(a, row, k0 + k, re, im);
    vis_put4(a, wide, add, row * a.ld + k0 + k, a.K - k0 - k, re, im);
  }
}

template <int PREC, bool UNI = false>
__global__ __launch_bounds__(kTileRows) void k_pg_tile(TileArgs a) {
  __shared__ PgSmem<typename PgTypes<PREC>::acc_t> sm;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  pg_tile<PREC, UNI>(a, tile % a.n_rb, tile / a.n_rb, sm);
}
template <int PREC, bool UNI>
__global__ __launch_bounds__(kTileRows) void k_pg_split(TileArgs a, int n_rb) {
  __shared__ PgSmem<typename PgTypes<PREC>::acc_t> sm;
  __shared__ double part[3][kPgChan][64][2];
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  pg_tile<PREC, UNI, true>(a, tile % n_rb, tile / n_rb, sm, part);
}

// ---------------------------------------------------------------------------
// shapelet tile on MFMA (mixed and FP32-only paths)
// ---------------------------------------------------------------------------

// Hermite recurrence step, phi_{n+1} = (sqrt2 x phi_n - sqrt(n) phi_{n-1}) / sqrt(n+1).
template <typename R>
__device__ __forceinline__ R herm_step(R sx, R pn, R pm1, int n) {
  return (R)c_isqn1[n] * fma(sx, pn, -(R)c_sqn[n] * pm1);
}

// Rescaled Hermite functions.  With s_n = sqrt(2^n / n!) and a base order b,
// u_n = phi_n s_b / s_n obeys u_{n+1} = x u_n - (n / 2) u_{n-1}: two
// operations per order and a constant that is a short immediate (n / 2 is a
// half-integer).  The MFMA path walks u with b at the middle of each 32-order
// block (|log10 (s_b / s_n)| <= 14 there) and multiplies the coefficient tiles
// by (s_n1 / s_b1)(s_n2 / s_b2), so that the products are unchanged.
template <typename R>
__device__ __forceinline__ R psi_next(R x, R un, R um1, R half_n) {
  return fma(x, un, -half_n * um1);
}

// Contraction modes: FP32 MFMA, or the coefficients and the second axis's
// Hermite values split into BF16 parts (x = hi + mid + lo) with the partial
// products summed on v_mfma_f32_32x32x16_bf16: 3 parts / 6 products, or
// 2 parts / 3 products.
enum Contraction : int { kCmF32 = 0, kCmBf16x2 = 2, kCmBf16x3 = 3 };

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// LDS of the shapelet tile: the coefficient blocks of one shapelet and the
// tile's visibility sums (one slot per thread and channel, FP64 on the mixed
// paths; kept here rather than in registers, which the MFMA loop needs).
template <int CM>
struct ShpA {
  float A[kPairsMax * kA32PerPair];
};
template <>
struct ShpA<kCmBf16x2> {
  uint4 A[2 * kPairsMax * kAbfPerPair / 8];
};
template <>
struct ShpA<kCmBf16x3> {
  uint4 A[3 * kPairsMax * kAbfPerPair / 8];
};
template <int CM>
struct ShpSmem : ShpA<CM> {
  double acc_re[kShpChan][kTileRows], acc_im[kShpChan][kTileRows];
};

// Per (visibility, shapelet) start value and phasor.  The synthetic envelopes
// reach ~15x their value at the uv origin, so on the mixed path these O(1)
// steps run in FP64 (exp, sincospi, product and sum) to keep their relative
// error from being magnified against the component's total flux.
template <typename R>
__device__ __forceinline__ R shp_phi0(R x);
template <>
__device__ __forceinline__ double shp_phi0<double>(double x) {
  return kPiM14 * exp(-0.5 * x * x);
}
template <>
__device__ __forceinline__ float shp_phi0<float>(float x) {
  return (float)kPiM14 * __builtin_amdgcn_exp2f(-x * x * (float)kHalfLog2e);
}

// Exchange between the two halves of a wave (v_permlane32_swap).  Every lane
// passes (p, q); afterwards lanes 0-31 hold (their own p, the p of lane + 32)
// and lanes 32-63 hold (the q of lane - 32, their own q).  When p is the value
// the lower half needs from a lane's visibility and q the one the upper half
// needs, p ends up as the value for the lower half's visibility and q as the
// value for the upper half's visibility, in every lane.
__device__ __forceinline__ void half_swap(float &p, float &q) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(p), __float_as_uint(q), false, false);
  p = __uint_as_float(r[0]);
  q = __uint_as_float(r[1]);
}
__device__ __forceinline__ void half_swap(uint32_t &p, uint32_t &q) {
  const auto r = __builtin_amdgcn_permlane32_swap(p, q, false, false);
  p = r[0];
  q = r[1];
}
// Fold one 32 x 32 block's FP32 accumulators into the DOT-precision sums:
// walk the first-axis recurrence (rescaled, psi_next) over the block's rows
// n0 + 8 g + r (this lane's visibility), 8 rows at a time, bring each row value to the lanes
// whose accumulator holds that row (half_swap) and add value x accumulator.
// Accumulator register i of a lane in half h holds block row
// 8 (i / 4) + 4 h + i % 4, of parity i % 2; even-n2 accumulators (E) pair
// with even rows for the real part.  Only the first ng 8-row groups are
// walked and folded (the rest of the block lies outside the triangle); with
// ng = 4, (prev, cur) leave as the next block's start values.
template <typename REC, typename DOT>
__device__ __forceinline__ void shp_fold(REC x, REC &prev, REC &cur, int n0, int ng, const floatx16 &E0,
                                         const floatx16 &O0, const floatx16 &E1, const floatx16 &O1, DOT &xr0,
                                         DOT &xi0, DOT &xr1, DOT &xi1) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    if (g < ng) {
    REC ra[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      ra[r] = cur;
      const REC nx = psi_next<REC>(x, cur, prev, (REC)(0.5 * (n0 + 8 * g + r)));
      prev = cur;
      cur = nx;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 4 * g + r;
      DOT p0 = (DOT)ra[r], p1 = (DOT)ra[4 + r];
      half_swap(p0, p1);
      const DOT e0 = (DOT)E0[i], o0 = (DOT)O0[i], e1 = (DOT)E1[i], o1 = (DOT)O1[i];
      if ((i & 1) == 0) {
        xr0 = fma(p0, e0, xr0);
        xi0 = fma(p0, o0, xi0);
        xr1 = fma(p1, e1, xr1);
        xi1 = fma(p1, o1, xi1);
      } else {
        xr0 = fma(p0, o0, xr0);
        xi0 = fma(p0, e0, xi0);
        xr1 = fma(p1, o1, xr1);
        xi1 = fma(p1, e1, xi1);
      }
    }
    }
    // keep the 8-row groups in order: hoisting the recurrence ahead of the
    // folds would hold all 32 of the block's values
    __builtin_amdgcn_sched_barrier(0);
  }
}

// One tile of the FP32-only path's shapelet pass: kTileRows rows x kShpChan
// channels starting at channel block cb.  Lane l of wave w owns row 64 w + l
// and runs both Hermite recurrences of its visibility in FP32.  The MFMA's N
// dimension is 32 visibilities: group 0 is the lower half-wave's, group 1 the
// upper's, and each operand value reaches the lane that supplies it through
// one half_swap per pair of values.  M is a 32-row block of the first axis, K
// runs over the second axis's orders (v_mfma_f32_32x32x2f32, K steps of 4
// orders inside the triangle) with even orders in one accumulator and odd
// orders in the other, folded into FP32 sums every 4 steps.
__device__ __forceinline__ void shp_tile_f32(const TileArgs &a, int rb, int cb, ShpSmem<kCmF32> &sm) {
  using REC = float;
  using DOT = float;
  constexpr int KB = kShpChan;
  const int k0 = cb * KB;
  const int tid = threadIdx.x, lane = tid & 63;
  const int64_t row = (int64_t)rb * kTileRows + tid;
  const bool valid = row < a.nrows;
  const int64_t rowc = valid ? row : a.nrows - 1;
  const int K = a.K;

  // sums start from what the point/Gaussian pass left (from zero without one)
#pragma unroll
  for (int c = 0; c < KB; ++c) {
    double sr = 0, si = 0;
    if (valid && k0 + c < K && !a.fresh) {
      const int64_t idx = row * K + k0 + c;
      if (a.c64) {
        const float2 x = ((const float2 *)a.vis)[idx];
        sr = x.x;
        si = a.conj ? -x.y : x.y;
      } else {
        const double2 x = ((const double2 *)a.vis)[idx];
        sr = x.x;
        si = a.conj ? -x.y : x.y;
      }
    }
    sm.acc_re[c][tid] = sr;
    sm.acc_im[c][tid] = si;
  }

  const DOT sgn = a.subtract ? -1 : 1;
  const floatx16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int j = 0; j < a.S; ++j) {
    const int N = a.t.nmax[j];
    const int q = N / 32;
    const int npairs = (q + 1) * (q + 2) / 2;
    __syncthreads();  // the previous shapelet's blocks are no longer read
    {
      const uint4 *src = (const uint4 *)(a.t.a32 + a.t.a32_off[j]);
      uint4 *dst = (uint4 *)&sm.A[0];
      for (int i = tid; i < npairs * kA32PerPair / 4; i += kTileRows) dst[i] = src[i];
    }
    const double *fr = a.d.sframe + 12 * j;
    const double u = a.uvw[3 * rowc], v = a.uvw[3 * rowc + 1], w = a.uvw[3 * rowc + 2];
    const double am = fma(fr[0], u, fma(fr[1], v, fr[2] * w));
    const double bm = fma(fr[3], u, fma(fr[4], v, fr[5] * w));
    const double t0 = fma(fr[6], u, fma(fr[7], v, fr[8] * w));
    __syncthreads();
    const int jg = a.P + a.G + j;
    for (int c = 0; c < KB; ++c) {
      if (k0 + c >= K) break;
      const double f = a.fk[k0 + c];
      const DOT S = (DOT)a.d.flux32[(int64_t)jg * a.Kpad + k0 + c];
      const REC xa = (REC)am * (REC)f;
      const REC xb = (REC)bm * (REC)f;
      // rescaled walks (psi_next): block or chunk k of 32 orders uses base
      // order 32 k + 16; carried values are rescaled when the base moves
      REC pb_m1 = 0, pb_n = shp_phi0<REC>(xb) * (REC)c_sc[0];
      // start values (u_{32 mb - 1}, u_{32 mb}) of the first axis's blocks,
      // filled in while chunk 0 walks every block
      REC sam[kMBMax], san[kMBMax];
      sam[0] = 0;
      san[0] = shp_phi0<REC>(xa) * (REC)c_sc[0];
#pragma unroll
      for (int k = 1; k < kMBMax; ++k) {
        sam[k] = 0;
        san[k] = 0;
      }
      DOT xr0 = 0, xi0 = 0, xr1 = 0, xi1 = 0;  // partial sums for groups 0 and 1
      int pbase = 0;
      for (int ch = 0; ch <= q; ++ch) {
        // second axis, this lane's visibility: orders 32 ch + t, in groups of
        // 8; groups past N (last chunk only) are zero
        float ob[32];
        {
          const int nb8 = min(4, (N - 32 * ch) / 8 + 1);
          REC prev = pb_m1, cur = pb_n;
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            if (g < nb8) {
#pragma unroll
              for (int t = 8 * g; t < 8 * g + 8; ++t) {
                ob[t] = (float)cur;
                const REC nx = psi_next<REC>(xb, cur, prev, (REC)c_half[32 * ch + t]);
                prev = cur;
                cur = nx;
              }
            } else {
#pragma unroll
              for (int t = 8 * g; t < 8 * g + 8; ++t) ob[t] = 0.f;
            }
          }
          // next chunk's base
          const REC rs = ch < 3 ? (REC)c_sc[ch + 1] : (REC)1;
          pb_m1 = prev * rs;
          pb_n = cur * rs;
        }
        // B operands of both groups (K = 2): lanes of half h supply orders
        // 4 s + 2 h + parity of K step s, stored at [2 s + parity]
        float bg0[16], bg1[16];
#pragma unroll
        for (int t = 0; t < 16; ++t) {
          const int lo = 4 * (t >> 1) + (t & 1);
          float p = ob[lo], qv = ob[lo + 2];
          half_swap(p, qv);
          bg0[t] = p;
          bg1[t] = qv;
        }
        const int nmb = q - ch + 1;
#pragma unroll
        for (int mb = 0; mb < kMBMax; ++mb) {
          if (mb >= nmb) break;
          const int p = pbase + mb;
          REC prev = sam[mb], cur = san[mb];
          // 8-row groups of this block that meet the triangle; all four while
          // chunk 0 walks towards a further block's start values
          const int ng = (ch == 0 && mb < q) ? 4 : min(4, (N - 32 * (ch + mb)) / 8 + 1);
          // K steps of this block inside the triangle: 32 (ch + mb) + 4 s <= N,
          // in two halves of 4 steps, each folded as soon as it is summed; the
          // second fold walks the rows again
          const int smax = min(8, (N - 32 * (ch + mb)) / 4 + 1);
          const float *Ap = &sm.A[p * kA32PerPair];
          const REC prev0 = prev, cur0 = cur;
          const int nh = smax > 4 ? 2 : 1;
#pragma nounroll
          for (int hf = 0; hf < nh; ++hf) {
            floatx16 E0 = zero16, O0 = zero16, E1 = zero16, O1 = zero16;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const int st = 4 * hf + k;
              if (st < smax) {
                const float ae = Ap[st * 64 + lane], ao = Ap[(8 + st) * 64 + lane];
                const float b0e = hf ? bg0[8 + 2 * k] : bg0[2 * k], b0o = hf ? bg0[9 + 2 * k] : bg0[2 * k + 1];
                const float b1e = hf ? bg1[8 + 2 * k] : bg1[2 * k], b1o = hf ? bg1[9 + 2 * k] : bg1[2 * k + 1];
                E0 = __builtin_amdgcn_mfma_f32_32x32x2f32(ae, b0e, E0, 0, 0, 0);
                O0 = __builtin_amdgcn_mfma_f32_32x32x2f32(ao, b0o, O0, 0, 0, 0);
                E1 = __builtin_amdgcn_mfma_f32_32x32x2f32(ae, b1e, E1, 0, 0, 0);
                O1 = __builtin_amdgcn_mfma_f32_32x32x2f32(ao, b1o, O1, 0, 0, 0);
              }
            }
            prev = prev0;
            cur = cur0;
            shp_fold<REC, DOT>(xa, prev, cur, 32 * mb, ng, E0, O0, E1, O1, xr0, xi0, xr1, xi1);
          }
          if (mb + 1 < kMBMax && ch == 0 && mb < q) {
            sam[mb + 1] = prev * (REC)c_sc[mb + 1];
            san[mb + 1] = cur * (REC)c_sc[mb + 1];
          }
        }
        pbase += nmb;
      }
      // each group's two half-wave partial sums, brought to the owning lane
      half_swap(xr0, xr1);
      half_swap(xi0, xi1);
      const DOT xr = xr0 + xr1, xi = xi0 + xi1;
      float cs, sn;
      turns_sincos_f32((float)t0 * (float)f, cs, sn);
      const DOT tr = sgn * S * (xr * cs - xi * sn);
      const DOT ti = sgn * S * (xr * sn + xi * cs);
      sm.acc_re[c][tid] = (double)((DOT)sm.acc_re[c][tid] + tr);
      sm.acc_im[c][tid] = (double)((DOT)sm.acc_im[c][tid] + ti);
    }
  }
  if (!valid) return;
#pragma unroll
  for (int c = 0; c < KB; ++c) {
    if (k0 + c >= K) break;
    const int64_t idx = row * K + k0 + c;
    const double re = sm.acc_re[c][tid], im = sm.acc_im[c][tid];
    if (a.c64)
      ((float2 *)a.vis)[idx] = make_float2((float)re, (float)(a.conj ? -im : im));
    else
      ((double2 *)a.vis)[idx] = make_double2(re, a.conj ? -im : im);
  }
}

// ---------------------------------------------------------------------------
// shapelet tile, BF16-split contraction (mixed path)
// ---------------------------------------------------------------------------

// The products of one MFMA group: even-n2 (E) and odd-n2 (O) accumulators of
// one 32 x 32 block, the two chains interleaved; smallest products first:
// (mid, mid), (lo, hi), (hi, lo), (mid, hi), (hi, mid), (hi, hi), or for the
// 2-way split (mid, hi), (hi, mid), (hi, hi).
template <int CM>
__device__ __forceinline__ void shp_group_mfma(const bf16x8 (&A)[3][2], const bf16x8 (&Bg)[3][2], floatx16 &E,
                                               floatx16 &O) {
  const floatx16 z = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (CM == kCmBf16x3) {
    E = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[1][0], Bg[1][0], z, 0, 0, 0);
    O = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[1][1], Bg[1][1], z, 0, 0, 0);
    E = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[2][0], Bg[0][0], E, 0, 0, 0);
    O = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[2][1], Bg[0][1], O, 0, 0, 0);
    E = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[0][0], Bg[2][0], E, 0, 0, 0);
    O = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[0][1], Bg[2][1], O, 0, 0, 0);
    E = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[1][0], Bg[0][0], E, 0, 0, 0);
    O = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[1][1], Bg[0][1], O, 0, 0, 0);
  } else {
    E = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[1][0], Bg[0][0], z, 0, 0, 0);
    O = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[1][1], Bg[0][1], z, 0, 0, 0);
  }
  E = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[0][0], Bg[1][0], E, 0, 0, 0);
  O = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[0][1], Bg[1][1], O, 0, 0, 0);
  E = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[0][0], Bg[0][0], E, 0, 0, 0);
  O = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[0][1], Bg[0][1], O, 0, 0, 0);
}

// The envelope of one shapelet of order N at this lane's (xa, xb), with the
// coefficient tiles Ab in LDS (parts part_stride apart); every lane of the wave
// takes part.  See shp_tile_bf.
template <int CM>
__device__ __forceinline__ void shp_eval_bf(double xa, double xb, int N, const __bf16 *Ab, int part_stride, double &xr,
                                            double &xi) {
  constexpr int parts = CM == kCmBf16x3 ? 3 : 2;
  const int q = N / 32;
  double pb_m1 = 0, pb_n = shp_phi0<double>(xb) * c_sc[0];
  const double ua0 = shp_phi0<double>(xa) * c_sc[0];
  double sr[4] = {0, 0, 0, 0}, si[4] = {0, 0, 0, 0};
  int pbase = 0;
  for (int ch = 0; ch <= q; ++ch) {
    const int nb8 = min(4, (N - 32 * ch) / 8 + 1);
    // second-axis operands of both groups: Bv[group][part][parity]
    bf16x8 Bv[2][3][2];
    {
      // pkb[part][parity][hc] element jj holds orders 16 hc + 4 jj +
      // parity (low half) and 16 hc + 4 jj + 2 + parity (high half)
      u32x4 pkb[3][2][2];
      double prev = pb_m1, cur = pb_n;
#pragma unroll
      for (int s4 = 0; s4 < 8; ++s4) {
        const int hc = s4 >> 2, jj = s4 & 3;
        if (s4 < 2 * nb8) {
          double v4[4];
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            v4[t] = cur;
            const double nx = psi_next<double>(xb, cur, prev, c_half[32 * ch + 4 * s4 + t]);
            prev = cur;
            cur = nx;
          }
#pragma unroll
          for (int par = 0; par < 2; ++par) {
            const double x0 = v4[par], x1 = v4[par + 2];
            const float2v xf = {(float)x0, (float)x1};
            const bf16x2v h = __builtin_convertvector(xf, bf16x2v);
            const float2v hf = __builtin_convertvector(h, float2v);
            const float2v rf = {(float)(x0 - (double)hf[0]), (float)(x1 - (double)hf[1])};
            const bf16x2v m = __builtin_convertvector(rf, bf16x2v);
            pkb[0][par][hc][jj] = __builtin_bit_cast(uint32_t, h);
            pkb[1][par][hc][jj] = __builtin_bit_cast(uint32_t, m);
            if (CM == kCmBf16x3) {
              const bf16x2v l = __builtin_convertvector(rf - __builtin_convertvector(m, float2v), bf16x2v);
              pkb[2][par][hc][jj] = __builtin_bit_cast(uint32_t, l);
            }
          }
        } else {
#pragma unroll
          for (int part = 0; part < 3; ++part)
#pragma unroll
            for (int par = 0; par < 2; ++par) pkb[part][par][hc][jj] = 0u;
        }
      }
      const double rs = ch < 3 ? c_sc[ch + 1] : 1.0;
      pb_m1 = prev * rs;
      pb_n = cur * rs;
      // group 0's operand: orders 0-15 of the lower half's visibility in
      // lanes 0-31, its orders 16-31 in lanes 32-63; group 1's likewise
      // for the upper half's visibility
#pragma unroll
      for (int part = 0; part < 3; ++part)
#pragma unroll
        for (int par = 0; par < 2; ++par) {
          u32x4 g0 = pkb[part][par][0], g1 = pkb[part][par][1];
          if (part < parts) {
#pragma unroll
            for (int jj = 0; jj < 4; ++jj)
              if (jj < 2 * nb8) {  // else both registers are zero in every lane
                uint32_t a0 = g0[jj], a1 = g1[jj];
                half_swap(a0, a1);
                g0[jj] = a0;
                g1[jj] = a1;
              }
          }
          Bv[0][part][par] = __builtin_bit_cast(bf16x8, g0);
          Bv[1][part][par] = __builtin_bit_cast(bf16x8, g1);
        }
    }
    const int nmb = q - ch + 1;
    double prev = 0, cur = ua0;
#pragma unroll
    for (int mb = 0; mb < kMBMax; ++mb) {
      if (mb >= nmb) break;
      if (mb > 0) {  // the next block's base order
        prev *= c_sc[mb];
        cur *= c_sc[mb];
      }
      const int p = pbase + mb;
      bf16x8 Av[3][2];  // [part][parity]
      {
        const int oe = p * kAbfPerPair + (threadIdx.x & 63) * 8, oo = oe + 64 * 8;
#pragma unroll
        for (int part = 0; part < 3; ++part) {
          const int pp = part < parts ? part : parts - 1;
          Av[part][0] = *(const bf16x8 *)(Ab + pp * part_stride + oe);
          Av[part][1] = *(const bf16x8 *)(Ab + pp * part_stride + oo);
        }
      }
      floatx16 E0, O0, E1, O1;
      shp_group_mfma<CM>(Av, Bv[0], E0, O0);
      shp_group_mfma<CM>(Av, Bv[1], E1, O1);
      // 8-row groups of this block inside the triangle
      const int ng = min(4, (N - 32 * (ch + mb)) / 8 + 1);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        if (g < ng) {
          double ra[8];
#pragma unroll
          for (int r = 0; r < 8; ++r) {
            ra[r] = cur;
            const double nx = psi_next<double>(xa, cur, prev, 0.5 * (32 * mb + 8 * g + r));
            prev = cur;
            cur = nx;
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int i = 4 * g + r;
            float e0 = E0[i], e1 = E1[i], o0 = O0[i], o1 = O1[i];
            half_swap(e0, e1);
            half_swap(o0, o1);
            // rows 8 g + r (set 0) and 8 g + 4 + r (set 1), both of parity r % 2;
            // four independent FP64 sums per part (set x row parity)
            const int k = 2 * (r & 1);
            if ((r & 1) == 0) {
              sr[k] = fma(ra[r], (double)e0, sr[k]);
              si[k] = fma(ra[r], (double)o0, si[k]);
              sr[k + 1] = fma(ra[4 + r], (double)e1, sr[k + 1]);
              si[k + 1] = fma(ra[4 + r], (double)o1, si[k + 1]);
            } else {
              sr[k] = fma(ra[r], (double)o0, sr[k]);
              si[k] = fma(ra[r], (double)e0, si[k]);
              sr[k + 1] = fma(ra[4 + r], (double)o1, sr[k + 1]);
              si[k + 1] = fma(ra[4 + r], (double)e1, si[k + 1]);
            }
          }
        }
      }
    }
    pbase += nmb;
  }
  xr = (sr[0] + sr[1]) + (sr[2] + sr[3]);
  xi = (si[0] + si[1]) + (si[2] + si[3]);
}

// One tile of the mixed path's shapelet pass: kTileRows rows x a.shp_chan (up
// to kShpChan) channels of channel block cb.  Lane l of wave w owns row 64 w + l
// and runs both Hermite recurrences of its visibility in FP64 (rescaled,
// psi_next).  The MFMA's N dimension is 32 visibilities: group 0 is the lower
// half-wave's, group 1 the upper's.  M is a 32-row block of the first axis, K
// the second axis's orders, even orders in one accumulator (E) and odd orders
// in the other (O).
//   * Second axis, per chunk of 32 orders: each lane walks its own
//     visibility, splits every value into BF16 parts from its FP64 value
//     (the residual after the high part is formed in FP64, exactly, so the
//     parts carry ~27 bits instead of an FP32 rounding's 24; that rounding
//     measured as the largest single error term of the contraction), packs
//     them two per register and exchanges half of them with the other half
//     of the wave, one v_permlane32_swap per register.
//   * First axis, per block: both groups' MFMAs; then each accumulator
//     register of group 0 is exchanged with the same register of group 1, so
//     that every lane holds all 8 rows of each 8-row group for its own
//     visibility (accumulator register i then holds row 8 (i / 4) + i % 4 in
//     group 0's set and row 8 (i / 4) + 4 + i % 4 in group 1's); the lane
//     walks its own first-axis recurrence over the block and folds the rows
//     into FP64 sums.  No row value crosses lanes.
// The first axis is walked from order 0 in each chunk, carried from one
// block into the next (only a chunk's last block is partial).  The sums are
// added to what the point/Gaussian pass left (with one).
template <int CM>
__device__ __forceinline__ void shp_tile_bf(const TileArgs &a, int rb, int cb, ShpSmem<CM> &sm) {
  static_assert(CM == kCmBf16x3 || CM == kCmBf16x2, "BF16-split contraction modes only");
  constexpr int KB = kShpChan;
  constexpr int parts = CM == kCmBf16x3 ? 3 : 2;
  const int kc = a.shp_chan, k0 = cb * kc;
  const int tid = threadIdx.x;
  const int64_t row = (int64_t)rb * kTileRows + tid;
  const bool valid = row < a.nrows;
  const int64_t rowc = valid ? row : a.nrows - 1;
  const int K = a.K;

#pragma unroll
  for (int c = 0; c < KB; ++c) sm.acc_re[c][tid] = sm.acc_im[c][tid] = 0.0;

  const double sgn = a.subtract ? -1 : 1;
  for (int j = 0; j < a.S; ++j) {
    const int N = a.t.nmax[j];
    const int q = N / 32;
    const int npairs = (q + 1) * (q + 2) / 2;
    __syncthreads();  // the previous shapelet's blocks are no longer read
    {
      const uint4 *src = (const uint4 *)(a.t.abf + a.t.abf_off[j]);
      uint4 *dst = &sm.A[0];
      for (int i = tid; i < parts * npairs * kAbfPerPair / 8; i += kTileRows) dst[i] = src[i];
    }
    const double *fr = a.d.sframe + 12 * j;
    const double u = a.uvw[3 * rowc], v = a.uvw[3 * rowc + 1], w = a.uvw[3 * rowc + 2];
    const double am = fma(fr[0], u, fma(fr[1], v, fr[2] * w));
    const double bm = fma(fr[3], u, fma(fr[4], v, fr[5] * w));
    const double t0 = fma(fr[6], u, fma(fr[7], v, fr[8] * w));
    __syncthreads();
    const int jg = a.P + a.G + j;
    const __bf16 *Ab = (const __bf16 *)&sm.A[0];
    const int part_stride = npairs * kAbfPerPair;
    for (int c = 0; c < kc; ++c) {
      if (k0 + c >= K) break;
      const double f = a.fk[k0 + c];
      const double S = a.d.flux64[(int64_t)jg * a.Kpad + k0 + c];
      const double xa = am * f, xb = bm * f;
      double xr, xi;
      shp_eval_bf<CM>(xa, xb, N, Ab, part_stride, xr, xi);
      double cs, sn;
      turns_sincos_f64(t0 * f, cs, sn);
      sm.acc_re[c][tid] += sgn * S * (xr * cs - xi * sn);
      sm.acc_im[c][tid] += sgn * S * (xr * sn + xi * cs);
    }
  }
  if (!valid) return;
  static_assert(KB == 4, "one vis_put4");
  double re[4], im[4];
#pragma unroll
  for (int c = 0; c < KB; ++c) {
    re[c] = sm.acc_re[c][tid];
    im[c] = a.conj ? -sm.acc_im[c][tid] : sm.acc_im[c][tid];
  }
  vis_put4(a, vis_wide(a), !a.fresh, row * K + k0, min(kc, K - k0), re, im);
}

template <int CM>
__global__ __launch_bounds__(kTileRows) __attribute__((amdgpu_waves_per_eu(2))) void k_shp_mfma(TileArgs a) {
  __shared__ ShpSmem<CM> sm;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  if constexpr (CM == kCmF32)
    shp_tile_f32(a, tile % a.n_rb, tile / a.n_rb, sm);
  else
    shp_tile_bf<CM>(a, tile % a.n_rb, tile / a.n_rb, sm);
}

// ---------------------------------------------------------------------------
// shapelet kernel, FP64 path (vector ALU)
// ---------------------------------------------------------------------------

// One thread per row of the tile, for the tile's kShpChan channels.  The
// second axis is taken in chunks of orders whose Hermite values sit in
// registers; per chunk the matching columns of the signed coefficient matrix
// are staged in LDS and each row n1 of them is dotted with those values while
// the first axis's recurrence advances with n1.  The recurrence path takes
// the four channels together (16-order chunks), the lookup-table variant one
// channel at a time (32-order chunks).
// Lookup-table variant of the basis (the paper's simulator interpolates a
// 1-D table of the basis, Sec. 3.2): phi_n at x_i = i dx, 0 <= i <= kLutSamples,
// dx = kLutXMax / kLutSamples, FP32, rows of kLutStride orders; phi_n(-x) =
// (-1)^n phi_n(x) covers x < 0 and the table reads zero beyond kLutXMax
// (phi_96(32) ~ 1e-78).  Built once per context from the FP64 recurrence.
__global__ __launch_bounds__(256) void k_lut_build(float *T) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i > kLutSamples + 1) return;
  const double x = i * (kLutXMax / kLutSamples);
  const double sx = 1.41421356237309504880 * x;
  double p = kPiM14 * exp(-0.5 * x * x), pm1 = 0.0;
  float *row = T + (int64_t)i * kLutStride;
  for (int n = 0; n < kLutStride; ++n) {
    row[n] = n <= kNmaxLimit ? (float)p : 0.0f;
    if (n < kNmaxLimit) {
      const double nx = herm_step<double>(sx, p, pm1, n);
      pm1 = p;
      p = nx;
    }
  }
}

// Interpolation position in the table: row pointer, fraction and the sign
// of odd orders.
struct LutPos {
  const float *r0;
  float fr, odd;
  bool in;
};

__device__ __forceinline__ LutPos lut_pos(const float *T, double x) {
  LutPos q;
  const double t = fabs(x) * (kLutSamples / kLutXMax);
  q.in = t < (double)kLutSamples;
  const int i = q.in ? (int)t : 0;
  q.fr = q.in ? (float)(t - i) : 0.0f;
  q.r0 = T + (int64_t)i * kLutStride;
  q.odd = x < 0.0 ? -1.0f : 1.0f;
  return q;
}

// Orders n0 .. n0 + 31 of the basis at q: linear interpolation between the
// two bracketing rows, the sign (-1)^n for x < 0, zero past kNmaxLimit and
// beyond the table.  The rows are read with 16-byte loads: a lane's orders
// are contiguous in its rows, and one 4-byte load per order made every load
// instruction touch a cache line per lane.  n0 is a multiple of 32 and rows
// are 16-byte aligned (kLutStride x 4 B); orders past kLutStride read the
// following row (inside the table, which has a spare row) before they are
// masked.
__device__ __forceinline__ void lut_chunk(const LutPos &q, int n0, float (&v)[32]) {
  const float4 *p0 = (const float4 *)(q.r0 + n0), *p1 = (const float4 *)(q.r0 + kLutStride + n0);
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const float4 a = p0[k], b = p1[k];
    v[4 * k] = fmaf(q.fr, b.x - a.x, a.x);
    v[4 * k + 1] = fmaf(q.fr, b.y - a.y, a.y);
    v[4 * k + 2] = fmaf(q.fr, b.z - a.z, a.z);
    v[4 * k + 3] = fmaf(q.fr, b.w - a.w, a.w);
  }
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    const int n = n0 + i;
    const float x = (n & 1) ? q.odd * v[i] : v[i];
    v[i] = q.in && n <= kNmaxLimit ? x : 0.0f;
  }
}

// Second-axis orders per chunk of the FP64 recurrence path: the values of a
// chunk for the tile's four channels (4 x 16 FP64) stay in registers.

// The envelopes of shapelet j (order N) at the four frequencies f4 (nu / c) of
// this thread's row; sC: the workgroup's chunk of coefficients.  Every thread of
// the workgroup takes part (barriers).
__device__ __forceinline__ void shp_eval4_fp64(const ShpTiles &t, int j, int N, double am, double bm,
                                               const double (&f4)[kShpChan], double *sC, double (&xr)[kShpChan],
                                               double (&xi)[kShpChan]) {
  constexpr int KB = kShpChan;
  const int tid = threadIdx.x;
  // The second axis in chunks of kF64Chunk orders (its recurrence carried
  // across chunks, per channel); per chunk the first axis is walked from
  // order 0 for all of the tile's channels at once, and each row n1 is
  // dotted with the chunk's part of row n1 of the signed coefficient
  // matrix.  Every coefficient read from LDS (a broadcast to all lanes)
  // feeds the tile's four channels: with one channel per read the LDS
  // return path, not the FP64 units, set the pace.  Channels past the
  // last (a ragged tile) are computed on the padded frequency table and
  // not used.
  const double *C = t.c64 + t.c64_off[j];
  const int ld = t.c64_ld[j];
  double bn[KB], bm1[KB], pa0[KB];  // per channel
#pragma unroll
  for (int c = 0; c < KB; ++c) {
    const double xb = f4[c] * bm, xa = f4[c] * am;
    bn[c] = kPiM14 * exp(-0.5 * xb * xb);
    pa0[c] = kPiM14 * exp(-0.5 * xa * xa);
    bm1[c] = xr[c] = xi[c] = 0.0;
  }
  for (int ch = 0; kF64Chunk * ch <= N; ++ch) {
    const int m0 = kF64Chunk * ch;
    __syncthreads();  // the previous chunk is no longer read
    for (int i = tid; i < (N - m0 + 1) * kF64Chunk; i += kTileRows) {
      const int col = m0 + (i % kF64Chunk);
      sC[i] = col < ld ? C[(int64_t)(i / kF64Chunk) * ld + col] : 0.0;
    }
    __syncthreads();
    double pb[KB][kF64Chunk];
#pragma unroll
    for (int c = 0; c < KB; ++c) {
      const double sxb = 1.41421356237309504880 * (f4[c] * bm);
#pragma unroll
      for (int i = 0; i < kF64Chunk; ++i) {
        pb[c][i] = bn[c];
        const double nx = herm_step<double>(sxb, bn[c], bm1[c], m0 + i);  // orders <= 127: table size
        bm1[c] = bn[c];
        bn[c] = nx;
      }
    }
    double pa[KB], pam1[KB], sxa[KB];
#pragma unroll
    for (int c = 0; c < KB; ++c) {
      pa[c] = pa0[c];
      pam1[c] = 0.0;
      sxa[c] = 1.41421356237309504880 * (f4[c] * am);
    }
    // one row n1: its dots with the chunk's second-axis values, folded
    // with the first axis into the real or imaginary sums by the parity
    // of n1 (rows are taken in pairs, so the parity is a constant)
    auto row = [&](int n1, auto ODD) {
      const double *Cr = sC + n1 * kF64Chunk;
      double te[KB], to[KB];
#pragma unroll
      for (int b8 = 0; b8 < kF64Chunk / 8; ++b8) {
        if (b8 == 0 || 8 * b8 <= N - m0 - n1) {
#pragma unroll
          for (int e = 0; e < 8; e += 2) {
            const double ce = Cr[8 * b8 + e], co = Cr[8 * b8 + e + 1];
#pragma unroll
            for (int c = 0; c < KB; ++c) {
              if (b8 == 0 && e == 0) {
                te[c] = ce * pb[c][0];
                to[c] = co * pb[c][1];
              } else {
                te[c] = fma(ce, pb[c][8 * b8 + e], te[c]);
                to[c] = fma(co, pb[c][8 * b8 + e + 1], to[c]);
              }
            }
          }
        }
      }
#pragma unroll
      for (int c = 0; c < KB; ++c) {
        if constexpr (decltype(ODD)::value) {
          xr[c] = fma(pa[c], to[c], xr[c]);
          xi[c] = fma(pa[c], te[c], xi[c]);
        } else {
          xr[c] = fma(pa[c], te[c], xr[c]);
          xi[c] = fma(pa[c], to[c], xi[c]);
        }
        const double nx = herm_step<double>(sxa[c], pa[c], pam1[c], n1);
        pam1[c] = pa[c];
        pa[c] = nx;
      }
    };
    for (int n1 = 0; n1 <= N - m0; n1 += 2) {
      row(n1, std::integral_constant<bool, false>());
      if (n1 + 1 <= N - m0) row(n1 + 1, std::integral_constant<bool, true>());
    }
  }
}

template <bool LUT>
__global__ __launch_bounds__(kTileRows) __attribute__((amdgpu_waves_per_eu(2))) void k_shp_fp64(TileArgs a) {
  constexpr int KB = kShpChan;
  // one 32-column chunk of the signed coefficient matrix (rows 0 .. N - m0),
  // staged in LDS for the whole workgroup and read as broadcasts: from
  // global memory every row dot waited on its wave-uniform loads
  __shared__ double sC[(kNmaxLimit + 1) * 32];
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int cb = tile / a.n_rb, rb = tile % a.n_rb;
  const int k0 = cb * KB;
  const int nc = min(KB, a.K - k0);  // channels of this tile
  const int tid = threadIdx.x;
  const int64_t row = (int64_t)rb * kTileRows + tid;
  const bool valid = row < a.nrows;
  const int64_t rowc = valid ? row : a.nrows - 1;
  const double u = a.uvw[3 * rowc], v = a.uvw[3 * rowc + 1], w = a.uvw[3 * rowc + 2];

  double acc_re[KB], acc_im[KB];
#pragma unroll
  for (int c = 0; c < KB; ++c) acc_re[c] = acc_im[c] = 0.0;
  for (int j = 0; j < a.S; ++j) {
    const int N = a.t.nmax[j];
    const double *fr = a.d.sframe + 12 * j;
    const double am = fma(fr[0], u, fma(fr[1], v, fr[2] * w));
    const double bm = fma(fr[3], u, fma(fr[4], v, fr[5] * w));
    const double t0 = fma(fr[6], u, fma(fr[7], v, fr[8] * w));
    if constexpr (!LUT) {
      double f4[KB], xr[KB], xi[KB];
#pragma unroll
      for (int c = 0; c < KB; ++c) f4[c] = a.fk[k0 + c];
      shp_eval4_fp64(a.t, j, N, am, bm, f4, sC, xr, xi);
#pragma unroll
      for (int c = 0; c < KB; ++c) {
        if (c >= nc) break;
        const double f = a.fk[k0 + c];
        double cs, sn;
        turns_sincos_f64(t0 * f, cs, sn);
        const double S = a.d.flux64[(int64_t)(a.P + a.G + j) * a.Kpad + k0 + c];
        acc_re[c] += S * (xr[c] * cs - xi[c] * sn);
        acc_im[c] += S * (xr[c] * sn + xi[c] * cs);
      }
    } else {
      // Lookup-table basis: the second axis in chunks of 32 orders, one
      // channel at a time; per chunk and channel each row n1 is dotted with
      // the chunk's part of row n1 of the signed coefficient matrix (staged in
      // LDS), and the first axis's table values are read 32 rows at a time,
      // all in flight before the rows that use them: a table read per row,
      // waited on by that row, left the kernel waiting on memory.
      const double *C = a.t.c64 + a.t.c64_off[j];
      const int ld = a.t.c64_ld[j];
      double xr[KB], xi[KB];
#pragma unroll
      for (int c = 0; c < KB; ++c) xr[c] = xi[c] = 0.0;
      for (int ch = 0; 32 * ch <= N; ++ch) {
        const int m0 = 32 * ch;
        __syncthreads();  // the previous chunk is no longer read
        for (int i = tid; i < (N - m0 + 1) * 32; i += kTileRows) {
          const int col = m0 + (i & 31);
          sC[i] = col < ld ? C[(int64_t)(i >> 5) * ld + col] : 0.0;
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < KB; ++c) {
          if (c >= nc) break;
          const double f = a.fk[k0 + c];
          const LutPos qa = lut_pos(a.lut, f * am), qb = lut_pos(a.lut, f * bm);
          double pb[32];
          {
            float pbf[32];
            lut_chunk(qb, m0, pbf);
#pragma unroll
            for (int i = 0; i < 32; ++i) pb[i] = (double)pbf[i];
          }
          for (int r0 = 0; r0 <= N - m0; r0 += 32) {
            float pa[32];  // rows past N - m0 are read but not used
            lut_chunk(qa, r0, pa);
#pragma unroll
            for (int r = 0; r < 32; ++r) {
              const int n1 = r0 + r;  // r0 is a multiple of 32: n1 has the parity of r
              if (n1 > N - m0) break;
              const double *Cr = sC + n1 * 32;
              double te = 0.0, to = 0.0;
#pragma unroll
              for (int b8 = 0; b8 < 4; ++b8) {
                if (8 * b8 <= N - m0 - n1) {
#pragma unroll
                  for (int e = 0; e < 8; e += 2) {
                    te = fma(Cr[8 * b8 + e], pb[8 * b8 + e], te);
                    to = fma(Cr[8 * b8 + e + 1], pb[8 * b8 + e + 1], to);
                  }
                }
              }
              const double pv = (double)pa[r];
              if (r & 1) {
                xr[c] = fma(pv, to, xr[c]);
                xi[c] = fma(pv, te, xi[c]);
              } else {
                xr[c] = fma(pv, te, xr[c]);
                xi[c] = fma(pv, to, xi[c]);
              }
            }
          }
        }
      }
#pragma unroll
      for (int c = 0; c < KB; ++c) {
        if (c >= nc) break;
        const double f = a.fk[k0 + c];
        double cs, sn;
        turns_sincos_f64(t0 * f, cs, sn);
        const double S = a.d.flux64[(int64_t)(a.P + a.G + j) * a.Kpad + k0 + c];
        acc_re[c] += S * (xr[c] * cs - xi[c] * sn);
        acc_im[c] += S * (xr[c] * sn + xi[c] * cs);
      }
    }
  }
  if (!valid) return;
#pragma unroll
  for (int c = 0; c < KB; ++c) {
    if (c >= nc) break;
    const int64_t idx = row * a.K + k0 + c;
    double2 *o = (double2 *)a.vis;
    float2 *o32 = (float2 *)a.vis;
    double xr = 0.0, xi = 0.0;
    if (a.fresh) {
      // no point/Gaussian pass wrote this visibility
    } else if (a.c64) {
      const float2 x = o32[idx];
      xr = x.x;
      xi = a.conj ? -x.y : x.y;
    } else {
      const double2 x = o[idx];
      xr = x.x;
      xi = a.conj ? -x.y : x.y;
    }
    if (a.subtract) {
      xr -= acc_re[c];
      xi -= acc_im[c];
    } else {
      xr += acc_re[c];
      xi += acc_im[c];
    }
    if (a.conj) xi = -xi;
    if (a.c64)
      o32[idx] = make_float2((float)xr, (float)xi);
    else
      o[idx] = make_double2(xr, xi);
  }
}

// ---------------------------------------------------------------------------
// shapelets by nodes
// ---------------------------------------------------------------------------
//
// The envelope of a shapelet along a baseline is a smooth function of
// frequency (see shp_nodes.h): it is evaluated at M Chebyshev nodes of the band
// and interpolated to the channels, where flux and phase are applied as ever.
// A workgroup takes R rows: the envelopes of every shapelet at the nodes go to
// LDS (FP64), lanes holding (row, node) pairs, and then each wave forms 16 rows
// x 16 channels at a time, the interpolation on v_mfma_f64_16x16x4f64 (the
// matrix from global memory, 4 nodes a step) and the sums over the shapelets in
// FP64 registers, one write per visibility.  What bounds it: the envelopes, M
// in place of K of them; a channel then costs M / 4 FP64 MFMAs per 128 outputs
// and ~35 vector instructions for its phase and flux, a fiftieth to a twentieth
// of an envelope.
typedef double double4w __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void node_outputs(const TileArgs &a, int Mp, const double *tab, const double *xs, int R,
                                             int64_t row0, int wave, int nwaves) {
  const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
  const int ncb = (a.K + 15) / 16, ntask = (R / 16) * ncb, steps = Mp / 4;
  const bool wide = vis_wide(a);
  for (int task = wave; task < ntask; task += nwaves) {
    const int rg = task / ncb, cb = task - rg * ncb;
    const int rr = rg * 16 + n, k = cb * 16 + 4 * g;  // this lane's row and first of four channels
    const int64_t row = row0 + rr;
    if (row0 + rg * 16 >= a.nrows) break;  // whole groups past the last row (wave-uniform)
    const bool valid = row < a.nrows;
    const int64_t rowc = valid ? row : a.nrows - 1;
    const double u = a.uvw[3 * rowc], v = a.uvw[3 * rowc + 1], w = a.uvw[3 * rowc + 2];
    double f[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) f[r] = a.fk[min(k + r, a.Kpad - 1)];
    double sre[4] = {0, 0, 0, 0}, sim[4] = {0, 0, 0, 0};
    for (int j = 0; j < a.S + a.out_points; ++j) {
      const bool pt = j >= a.S;  // a point: an envelope of 1
      const double *xr = xs + node_lds(pt ? 0 : j, Mp, R), *xi = xr + (size_t)Mp * R;
      const double *L = tab + kNodesStride + (size_t)cb * steps * 64 + lane;
      const double one = pt ? 1.0 : 0.0;
      double4w er = {one, one, one, one}, ei = {0, 0, 0, 0};
      for (int s = 0; s < (pt ? 0 : steps); ++s) {
        const double l = L[64 * s];
        const int at = (4 * s + g) * R + rr;
        er = __builtin_amdgcn_mfma_f64_16x16x4f64(l, xr[at], er, 0, 0, 0);
        ei = __builtin_amdgcn_mfma_f64_16x16x4f64(l, xi[at], ei, 0, 0, 0);
      }
      const double *fr = pt ? (const double *)(a.d.pos + (j - a.S)) : a.d.sframe + 12 * j + 6;
      const double t0 = fma(fr[0], u, fma(fr[1], v, fr[2] * w));
      double c, s, cd = 0, sd = 0;
      turns_sincos_f64(t0 * f[0], c, s);
      if (a.uniform) turns_sincos_f64(t0 * a.dfk, cd, sd);
      const double *fl = a.d.flux64 + (int64_t)(pt ? j - a.S : a.P + a.G + j) * a.Kpad;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (r > 0) {
          if (a.uniform) {
            const double cn = fma(c, cd, -s * sd);
            s = fma(s, cd, c * sd);
            c = cn;
          } else {
            turns_sincos_f64(t0 * f[r], c, s);
          }
        }
        const double S = fl[min(k + r, a.Kpad - 1)];
        sre[r] += S * (er[r] * c - ei[r] * s);
        sim[r] += S * (er[r] * s + ei[r] * c);
      }
    }
    if (!valid) continue;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (a.subtract) sre[r] = -sre[r];
      if (a.subtract != a.conj) sim[r] = -sim[r];
    }
    vis_put4(a, wide, !a.fresh, row * a.K + k, a.K - k, sre, sim);
  }
}

template <int CM>
__global__ __launch_bounds__(kNodeThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_shp_nodes(
    TileArgs a, NodePlan p, const double *tab, int R, int a_bytes) {
  extern __shared__ __align__(16) unsigned char node_sm[];
  constexpr int parts = CM == kCmBf16x3 ? 3 : 2;
  uint4 *sA = (uint4 *)node_sm;
  double *xs = (double *)(node_sm + a_bytes);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t row0 = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * R;
  // padding nodes (zero columns of the matrix) hold zeros
  for (int i = tid; i < a.S * 2 * (p.Mp - p.M) * R; i += kNodeThreads) {
    const int c = i / ((p.Mp - p.M) * R), e = i % ((p.Mp - p.M) * R);
    xs[(size_t)c * p.Mp * R + (size_t)p.M * R + e] = 0.0;
  }
  const int pairs = R * p.M;  // (row, node), 64 of them a wave's share
  for (int j = 0; j < a.S; ++j) {
    const int N = a.t.nmax[j];
    const int npairs = shp_pairs(N);
    __syncthreads();  // the previous shapelet's blocks are no longer read
    {
      const uint4 *src = (const uint4 *)(a.t.abf + a.t.abf_off[j]);
      for (int i = tid; i < parts * npairs * kAbfPerPair / 8; i += kNodeThreads) sA[i] = src[i];
    }
    __syncthreads();
    const double *fr = a.d.sframe + 12 * j;
    double *xr_s = xs + node_lds(j, p.Mp, R), *xi_s = xr_s + (size_t)p.Mp * R;
    for (int i0 = 64 * wave; i0 < pairs; i0 += kNodeThreads) {
      const int i = min(i0 + lane, pairs - 1), m = i / R, rr = i - m * R;
      const int64_t row = min(row0 + rr, a.nrows - 1);
      const double f = tab[m];
      const double u = a.uvw[3 * row], v = a.uvw[3 * row + 1], w = a.uvw[3 * row + 2];
      const double am = fma(fr[0], u, fma(fr[1], v, fr[2] * w));
      const double bm = fma(fr[3], u, fma(fr[4], v, fr[5] * w));
      double xr, xi;
      shp_eval_bf<CM>(am * f, bm * f, N, (const __bf16 *)sA, npairs * kAbfPerPair, xr, xi);
      if (i0 + lane < pairs) {
        xr_s[i] = xr;
        xi_s[i] = xi;
      }
    }
  }
  __syncthreads();
  node_outputs(a, p.Mp, tab, xs, R, row0, wave, kNodeThreads / 64);
}

// The FP64 path: four nodes of one row a thread (padding nodes repeat the
// middle of the band), as many passes as the workgroup's R rows x M / 4 need.
__global__ __launch_bounds__(kNodeThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_shp_nodes64(
    TileArgs a, NodePlan p, const double *tab, int R) {
  extern __shared__ __align__(16) unsigned char node_sm[];
  double *sC = (double *)node_sm;
  double *xs = sC + (kNmaxLimit + 1) * kF64Chunk;
  const int tid = threadIdx.x;
  const int64_t row0 = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * R;
  const int quads = p.Mp / 4;
  for (int j = 0; j < a.S; ++j) {
    const int N = a.t.nmax[j];
    const double *fr = a.d.sframe + 12 * j;
    double *xr_s = xs + node_lds(j, p.Mp, R), *xi_s = xr_s + (size_t)p.Mp * R;
    for (int i0 = 0; i0 < R * quads; i0 += kNodeThreads) {
      const int i = min(i0 + tid, R * quads - 1);
      const int rr = i % R, q = i / R;
      const int64_t row = min(row0 + rr, a.nrows - 1);
      const double u = a.uvw[3 * row], v = a.uvw[3 * row + 1], w = a.uvw[3 * row + 2];
      const double am = fma(fr[0], u, fma(fr[1], v, fr[2] * w));
      const double bm = fma(fr[3], u, fma(fr[4], v, fr[5] * w));
      double f4[kShpChan], xr[kShpChan], xi[kShpChan];
#pragma unroll
      for (int c = 0; c < kShpChan; ++c) f4[c] = tab[4 * q + c];
      shp_eval4_fp64(a.t, j, N, am, bm, f4, sC, xr, xi);
      if (i0 + tid < R * quads) {
#pragma unroll
        for (int c = 0; c < kShpChan; ++c) {
          xr_s[(4 * q + c) * R + rr] = xr[c];
          xi_s[(4 * q + c) * R + rr] = xi[c];
        }
      }
    }
  }
  __syncthreads();
  node_outputs(a, p.Mp, tab, xs, R, row0, __builtin_amdgcn_readfirstlane(tid >> 6), kNodeThreads / 64);
}

// ---------------------------------------------------------------------------
// points and Gaussians by nodes
// ---------------------------------------------------------------------------
//
// In a narrow field a row's sum over points and Gaussians is a smooth function
// of frequency (see pg_nodes in shp_nodes.h): it is summed at M Chebyshev nodes
// of the band and interpolated to the channels.  A workgroup takes LR rows; wave
// i holds nodes kPgNB i .. kPgNB (i + 1) - 1, lane l row l % LR and every
// (64 / LR)-th component (fewer rows where more workgroups are wanted), sums as
// on the tile of channels (FP32 partials of kFlush components into FP64 on the
// mixed path, Kahan sums on the FP64 path).  The sums go to LDS and each wave
// interpolates 16 rows x 16 channels at a time on v_mfma_f64_16x16x4f64.
//
// What bounds it: vector instructions, 8 a value of a point (phase, sine and
// cosine, two multiply-adds), 12 of a Gaussian.  128 antennas x 4 times, 384
// channels by 28 nodes (0.5 degrees): 1,791 Gaussians 1.08 ms for 7.07 on
// channels, 4,540 points 1.85 ms for 10.7 (1.75 by antenna); FP64 6.4 and 11.1 ms
// for 19.6 and 30.6.  Six nodes a lane hold five waves a SIMD (96 registers);
// at four, 1,016 workgroups took two rounds: 1.43 ms and 2.57.
// Waves of a workgroup, at most.
constexpr int pg_node_waves(bool f64, bool nodes) { return nodes || f64 ? kPgNodesMax / kPgNB : 16; }

struct PgNodeLds {
  double4 pos[kChunk], gq[kChunk];
};

// NODES false: the same split over channels instead of nodes, without
// interpolation, for observations whose tiles (256 rows x 8 channels a workgroup)
// would leave most CUs idle: workgroup (x, y) takes LR rows and the y-th kPgNB nw
// channels, CS groups of nw waves sharing the components.  2,524 rows x 13
// channels, 90 Gaussians: 14.5 us for 33.5 on tiles; 496 rows x 4 channels in
// FP64, 100 points and 10 Gaussians: 16 us for 26 (points by antenna) and 9.4.
template <bool F64, bool NODES>
__global__ __launch_bounds__(64 * pg_node_waves(F64, NODES)) __attribute__((amdgpu_waves_per_eu(F64 ? 3 : NODES ? 5 : 4))) void k_pg_nodes(
    TileArgs a, int LR, int CS) {
  typedef typename std::conditional<F64, double, float>::type T;
  extern __shared__ __align__(16) unsigned char node_sm[];
  const NodePlan &p = a.d.plan[2 + F64];
  const double *tab = a.d.interp[2 + F64], *nf = a.d.nflux[F64];
  const int tid = threadIdx.x, lane = tid & 63, nt = blockDim.x;
  const int nw = NODES ? nt / 64 : nt / 64 / CS, FS = kPgNB * nw;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6), wave = NODES ? wid : wid % nw, cp = NODES ? 0 : wid / nw;
  PgNodeLds &sm = *(PgNodeLds *)node_sm;
  T *s_flux = (T *)(node_sm + sizeof(PgNodeLds));       // [kChunk][FS]
  double *xr = (double *)(s_flux + kChunk * FS), *xi = xr + p.Mp * LR;  // [Mp][LR] each
  const int k0 = NODES ? 0 : blockIdx.y * FS;
  const int64_t row0 = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * LR;
  const int rr = lane % LR, sub = lane / LR + 64 / LR * cp, nsub = 64 / LR * (NODES ? 1 : CS);
  const int64_t row = min(row0 + rr, a.nrows - 1);
  const double u = a.uvw[3 * row], v = a.uvw[3 * row + 1], w = a.uvw[3 * row + 2];
  double f[kPgNB], sre[kPgNB], sim[kPgNB], cre[kPgNB], cim[kPgNB];
  T f2[kPgNB], pre[kPgNB], pim[kPgNB];
#pragma unroll
  for (int k = 0; k < kPgNB; ++k) {
    f[k] = NODES ? tab[min(wave * kPgNB + k, kNodesStride - 1)] : a.fk[min(k0 + wave * kPgNB + k, a.Kpad - 1)];
    f2[k] = (T)(f[k] * f[k]);
    sre[k] = sim[k] = cre[k] = cim[k] = 0.0;
    pre[k] = pim[k] = 0;
  }
  const T uu = (T)(u * u), vv = (T)(v * v), uv = (T)(u * v);
  const int J0[2] = {a.skip_points ? a.P : 0, a.P}, JN[2] = {a.P, a.P + a.G};
#pragma unroll
  for (int kind = 0; kind < 2; ++kind) {  // 0: points, 1: Gaussians
    for (int j0 = J0[kind]; j0 < JN[kind]; j0 += kChunk) {
      const int n = min(kChunk, JN[kind] - j0);
      __syncthreads();
      for (int i = tid; i < n; i += nt) {
        sm.pos[i] = a.d.pos[j0 + i];
        if (kind == 1) sm.gq[i] = a.d.gq[j0 - a.P + i];
      }
      for (int i = tid; i < n * FS; i += nt) {
        const int jj = i / FS, m = i - jj * FS;
        if (NODES)
          s_flux[i] = m < p.Mp ? (T)nf[(int64_t)(j0 + jj) * p.Mp + m] : (T)0;
        else if (F64)
          s_flux[i] = k0 + m < a.K ? (T)a.d.flux64[(int64_t)(j0 + jj) * a.Kpad + k0 + m] : (T)0;
        else
          s_flux[i] = k0 + m < a.K ? (T)a.d.flux32[(int64_t)(j0 + jj) * a.Kpad + k0 + m] : (T)0;
      }
      __syncthreads();
      auto term = [&](int jj) {
        const double4 q = sm.pos[jj];
        T Q = 0;
        if (kind == 1) {
          const double4 g = sm.gq[jj];
          Q = fma((T)g.x, uu, fma((T)g.y, vv, (T)g.z * uv));
        }
        const double t0 = fma(u, q.x, fma(v, q.y, w * q.z));
        const T *fl = s_flux + jj * FS + wave * kPgNB;
#pragma unroll
        for (int k = 0; k < kPgNB; ++k) {
          T c, s, S = fl[k];
          if constexpr (F64) {
            turns_sincos_f64(t0 * f[k], c, s);
            if (kind == 1) S *= exp2(-Q * f2[k]);
          } else {
            if (NODES)
              turns_sincos_fixed(t0, f[k], c, s);
            else
              turns_sincos_mixed(t0 * f[k], c, s);
            if (kind == 1) S *= __builtin_amdgcn_exp2f(-Q * f2[k]);
          }
          pre[k] = fma(S, c, pre[k]);
          pim[k] = fma(S, s, pim[k]);
        }
      };
      auto flush = [&]() {
#pragma unroll
        for (int k = 0; k < kPgNB; ++k) {
          if constexpr (F64) {
            kahan_add(sre[k], cre[k], pre[k]);
            kahan_add(sim[k], cim[k], pim[k]);
          } else {
            sre[k] += (double)pre[k];
            sim[k] += (double)pim[k];
          }
          pre[k] = pim[k] = 0;
        }
      };
      int jj = sub;
      constexpr int kUnroll = F64 ? 1 : 4;
      for (; jj + (kFlush - 1) * nsub < n; jj += kFlush * nsub) {
#pragma unroll kUnroll
        for (int i = 0; i < kFlush; ++i) term(jj + i * nsub);
        flush();
      }
      for (; jj < n; jj += nsub) term(jj);
      flush();
    }
  }
#pragma unroll
  for (int k = 0; k < kPgNB; ++k) {
    const int m = wave * kPgNB + k;
    double re = sre[k] - cre[k], im = sim[k] - cim[k];
    for (int o = LR; o < 64; o *= 2) {
      re += __shfl_xor(re, o);
      im += __shfl_xor(im, o);
    }
    if (NODES && sub == 0 && m < p.Mp) {
      xr[m * LR + rr] = re;
      xi[m * LR + rr] = im;
    }
    if (!NODES) {
      sre[k] = re;
      sim[k] = im;
    }
  }
  if constexpr (!NODES) {
    // the waves' shares of the components, [CS - 1][nw][kPgNB][LR] each
    double *ex = (double *)(s_flux + kChunk * FS), *ey = ex + (CS - 1) * nw * kPgNB * LR;
    if (cp > 0 && lane < LR) {
#pragma unroll
      for (int k = 0; k < kPgNB; ++k) {
        const int at = (((cp - 1) * nw + wave) * kPgNB + k) * LR + rr;
        ex[at] = sre[k];
        ey[at] = sim[k];
      }
    }
    __syncthreads();
    const int k = k0 + wave * kPgNB;
    if (cp > 0 || lane >= LR || row0 + rr >= a.nrows || k >= a.K) return;
#pragma unroll
    for (int i = 0; i < kPgNB; ++i) {
      for (int c = 1; c < CS; ++c) {
        const int at = (((c - 1) * nw + wave) * kPgNB + i) * LR + rr;
        sre[i] += ex[at];
        sim[i] += ey[at];
      }
      if (a.subtract) sre[i] = -sre[i];
      if (a.subtract != a.conj) sim[i] = -sim[i];
    }
    static_assert(kPgNB == 6, "four channels and two");
    double r0[4] = {sre[0], sre[1], sre[2], sre[3]}, i0[4] = {sim[0], sim[1], sim[2], sim[3]};
    double r1[4] = {sre[4], sre[5], 0, 0}, i1[4] = {sim[4], sim[5], 0, 0};
    const bool wide = vis_wide(a), add = a.subtract || (a.skip_points && !a.sums);
    add_sums(a, row, k, r0, i0);
    add_sums(a, row, k + 4, r1, i1);
    vis_put4(a, wide, add, row * a.ld + k, min(4, a.K - k), r0, i0);
    vis_put4(a, wide, add, row * a.ld + k + 4, min(2, a.K - k - 4), r1, i1);
    return;
  }
  __syncthreads();
  const int n16 = lane & 15, g = lane >> 4, ncb = (a.K + 15) / 16, cb0 = a.chan0 / 16, steps = p.Mp / 4;
  const bool wide = vis_wide(a);
  for (int task = wave; task < (LR / 16) * ncb; task += nw) {
    const int rg = task / ncb, cb = task - rg * ncb, ro = rg * 16 + n16, k = cb * 16 + 4 * g;
    const double *L = tab + kNodesStride + (size_t)(cb0 + cb) * steps * 64 + lane;
    double4w er = {0, 0, 0, 0}, ei = {0, 0, 0, 0};
    for (int s = 0; s < steps; ++s) {
      const double l = L[64 * s];
      const int at = (4 * s + g) * LR + ro;
      er = __builtin_amdgcn_mfma_f64_16x16x4f64(l, xr[at], er, 0, 0, 0);
      ei = __builtin_amdgcn_mfma_f64_16x16x4f64(l, xi[at], ei, 0, 0, 0);
    }
    if (row0 + ro >= a.nrows) continue;
    double re[4], im[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      re[r] = a.subtract ? -er[r] : er[r];
      im[r] = a.subtract != a.conj ? -ei[r] : ei[r];
    }
    add_sums(a, row0 + ro, k, re, im);
    vis_put4(a, wide, a.subtract || (a.skip_points && !a.sums), (row0 + ro) * a.ld + k, a.K - k, re, im);
  }
}

// A serving job's mark on its stream (see ServeMark): the clock, then the
// sequence number that tells the host that the clock is there.
__global__ void k_mark(ServeMark *m, uint64_t seq) {
  __hip_atomic_store(&m->clk, wall_clock64(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __hip_atomic_store(&m->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

// Per-device set-up, once per device and process: the recurrence constants
// into __constant__ memory.
static std::once_flag g_init_once[kMaxDevices];
static hipError_t g_init_err[kMaxDevices];

static hipError_t init_constants() {
  double sq[128], isq[128], half[128], sc[4];
  for (int n = 0; n < 128; ++n) {
    sq[n] = sqrt((double)n);
    isq[n] = 1.0 / sqrt((double)n + 1.0);
    half[n] = 0.5 * n;
  }
  sc[0] = herm_scale(0, 16);
  for (int k = 1; k < 4; ++k) sc[k] = herm_scale(32 * k - 16, 32 * k + 16);
  hipError_t e = hipMemcpyToSymbol(HIP_SYMBOL(c_sqn), sq, sizeof(sq));
  if (e == hipSuccess) e = hipMemcpyToSymbol(HIP_SYMBOL(c_isqn1), isq, sizeof(isq));
  if (e == hipSuccess) e = hipMemcpyToSymbol(HIP_SYMBOL(c_half), half, sizeof(half));
  if (e == hipSuccess) e = hipMemcpyToSymbol(HIP_SYMBOL(c_sc), sc, sizeof(sc));
  return e;
}

// Scratch of vp_predict_noalloc (the per-(sky, observation) tables of one
// call), one array per device for the life of the process.  In host code the
// name is only a stand-in: its device address, which differs per device, is
// looked up once per device below and used everywhere instead.
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes + kNoAllocAmpBytes + kNoAllocNodeBytes +
                                                              kNoAllocNfluxBytes + kSumsMin];
static void *g_scratch[kMaxDevices];

hipError_t device_init(int dev) {
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::call_once(g_init_once[dev], [dev]() {
    // the caller has made `dev` current
    hipError_t e = init_constants();
    if (e == hipSuccess) {
      void *p = nullptr;
      e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      if (e == hipSuccess) g_scratch[dev] = p;
    }
    g_init_err[dev] = e;
  });
  return g_init_err[dev];
}

void *noalloc_scratch(int dev) {
  if (dev < 0 || dev >= kMaxDevices || device_init(dev) != hipSuccess) return nullptr;
  return g_scratch[dev];
}

static hipError_t upload_tables() {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  return device_init(dev);
}

hipError_t launch_derive(const DeriveArgs &a, hipStream_t s) {
  const int J = a.P + a.G + a.S;
  int rows = 0;
  for (const NodePlan &p : a.d.plan) rows += p.M > 0 ? (a.K + 15) / 16 * 16 : 0;
  if (J == 0 && rows == 0) return hipSuccess;
  hipLaunchKernelGGL(k_derive, dim3((J + 127) / 128 + (rows + 1) / 2), dim3(128), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_flux(const FluxArgs &a, hipStream_t s) {
  int64_t n = (int64_t)a.J * a.Kpad;
  for (int i = 0; i < 2; ++i)
    if (a.d.plan[2 + i].M > 0) n += (int64_t)a.j0 * a.d.plan[2 + i].Mp;
  if (a.d.amp) n = std::max<int64_t>(n, a.Kpad);
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_flux, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_tiles_build(const TileBuildArgs &a, int max_nmax, hipStream_t s) {
  (void)max_nmax;
  if (a.S == 0) return hipSuccess;
  hipLaunchKernelGGL(k_tiles, dim3(16, a.S), dim3(256), 0, s, a);
  return hipGetLastError();
}

static int64_t pg_tiles(const TileArgs &a) { return (a.call_rows + kTileRows - 1) / kTileRows * (a.Kpad / kPgChan); }
static hipError_t launch_pg_small(const TileArgs &a, bool f64, hipStream_t s);

hipError_t launch_pg(const TileArgs &a, int prec, hipStream_t s) {
  hipError_t e = upload_tables();
  if (e != hipSuccess) return e;
  const int64_t nt = (int64_t)a.n_rb * a.n_cb;
  if (nt <= 0) return hipSuccess;
  if (nt > 0x7fffffff) return hipErrorInvalidValue;
  const bool f64 = prec == kFP64 || prec == kLut;
  const int points = a.skip_points ? 0 : a.P;
  if (prec != kFP32 && pg_small(f64, pg_tiles(a), points + a.G, a.uniform)) return launch_pg_small(a, f64, s);
  if (prec != kFP32 && pg_split(f64, pg_tiles(a), points, a.G)) {
    const int n_rb = (int)((a.nrows + 63) / 64);
    const dim3 g((unsigned)((int64_t)n_rb * a.n_cb)), b(kTileRows);
    if (prec == kFP64 || prec == kLut) {
      if (a.uniform)
        hipLaunchKernelGGL((k_pg_split<kFP64, true>), g, b, 0, s, a, n_rb);
      else
        hipLaunchKernelGGL((k_pg_split<kFP64, false>), g, b, 0, s, a, n_rb);
    } else if (a.uniform)
      hipLaunchKernelGGL((k_pg_split<kMixed, true>), g, b, 0, s, a, n_rb);
    else
      hipLaunchKernelGGL((k_pg_split<kMixed, false>), g, b, 0, s, a, n_rb);
    return hipGetLastError();
  }
  switch (prec) {
    case kFP64:
    case kLut:  // the lookup-table variant differs from the FP64 path in the shapelet basis only
      if (a.uniform)
        hipLaunchKernelGGL((k_pg_tile<kFP64, true>), dim3((unsigned)nt), dim3(kTileRows), 0, s, a);
      else
        hipLaunchKernelGGL((k_pg_tile<kFP64, false>), dim3((unsigned)nt), dim3(kTileRows), 0, s, a);
      break;
    case kFP32:
      hipLaunchKernelGGL(k_pg_tile<kFP32>, dim3((unsigned)nt), dim3(kTileRows), 0, s, a);
      break;
    default:
      if (a.uniform)
        hipLaunchKernelGGL((k_pg_tile<kMixed, true>), dim3((unsigned)nt), dim3(kTileRows), 0, s, a);
      else
        hipLaunchKernelGGL((k_pg_tile<kMixed, false>), dim3((unsigned)nt), dim3(kTileRows), 0, s, a);
      break;
  }
  return hipGetLastError();
}

hipError_t launch_shp(const TileArgs &a, int prec, int max_nmax, hipStream_t s) {
  hipError_t e = upload_tables();
  if (e != hipSuccess) return e;
  const int64_t nt = (int64_t)a.n_rb * a.n_cb;
  if (nt <= 0 || a.S == 0) return hipSuccess;
  if (nt > 0x7fffffff) return hipErrorInvalidValue;
  if (max_nmax < 0 || max_nmax > kNmaxLimit) return hipErrorInvalidValue;
  const dim3 g((unsigned)nt), b(kTileRows);
  switch (prec) {
    case kFP64:
      hipLaunchKernelGGL(k_shp_fp64<false>, g, b, 0, s, a);
      break;
    case kLut:
      if (!a.lut) return hipErrorInvalidValue;
      hipLaunchKernelGGL(k_shp_fp64<true>, g, b, 0, s, a);
      break;
    case kFP32:
      hipLaunchKernelGGL(k_shp_mfma<kCmF32>, g, b, 0, s, a);
      break;
    case kMixed:
    case kMixedBf16:
    case kMixedBf16x2: {
      TileArgs t = a;
      t.shp_chan = shp_channels(t.n_rb, a.K);
      t.n_cb = (a.K + t.shp_chan - 1) / t.shp_chan;
      const dim3 gt((unsigned)((int64_t)t.n_rb * t.n_cb));
      if (prec == kMixedBf16x2)
        hipLaunchKernelGGL(k_shp_mfma<kCmBf16x2>, gt, b, 0, s, t);
      else
        hipLaunchKernelGGL(k_shp_mfma<kCmBf16x3>, gt, b, 0, s, t);
      break;
    }
    default:
      return hipErrorNotSupported;
  }
  return hipGetLastError();
}

hipError_t launch_pg_nodes(const TileArgs &a, int prec, hipStream_t s) {
  const bool f64 = prec == kFP64 || prec == kLut;
  const NodePlan &p = a.d.plan[2 + f64];
  if (p.M < 1 || p.M > kPgNodesMax || p.M > p.Mp || p.Mp > kNodesStride || p.Mp % 4 || a.K > kNodesMaxChan)
    return hipErrorInvalidValue;
  int64_t slots = 0;
  const int nw = (p.Mp + kPgNB - 1) / kPgNB, LR = pg_node_rows(f64, p.Mp, a.call_rows, &slots);
  const int64_t nt = (a.nrows + LR - 1) / LR;
  if (nt > 0x7fffffff) return hipErrorInvalidValue;
  const size_t sm = sizeof(PgNodeLds) + (size_t)kChunk * kPgNB * nw * (f64 ? 8 : 4) + (size_t)2 * p.Mp * LR * 8;
  const void *k = f64 ? (const void *)k_pg_nodes<true, true> : (const void *)k_pg_nodes<false, true>;
  hipError_t e = whole_lds(k);
  if (e != hipSuccess) return e;
  if (f64)
    hipLaunchKernelGGL((k_pg_nodes<true, true>), dim3((unsigned)nt), dim3(64 * nw), sm, s, a, LR, 1);
  else
    hipLaunchKernelGGL((k_pg_nodes<false, true>), dim3((unsigned)nt), dim3(64 * nw), sm, s, a, LR, 1);
  return hipGetLastError();
}

// Points and Gaussians of a small observation, channel by channel.
static hipError_t launch_pg_small(const TileArgs &a, bool f64, hipStream_t s) {
  const int nw = std::min(4, (a.K + kPgNB - 1) / kPgNB), ny = (a.K + kPgNB * nw - 1) / (kPgNB * nw);
  // fewer rows a wave, then more waves to the components, until two waves a SIMD
  const int comps = a.G + (a.skip_points ? 0 : a.P);
  int LR = 64, CS = 1;
  while (LR > 16 && (a.nrows + LR - 1) / LR * ny < 512) LR /= 2;
  const int64_t wgs = (a.nrows + LR - 1) / LR * ny;
  while (2 * CS * nw <= pg_node_waves(f64, false) && wgs * nw * CS < 2048 && comps >= 64 / LR * CS * 4) CS *= 2;
  const dim3 g((unsigned)((a.nrows + LR - 1) / LR), (unsigned)ny), b(64 * nw * CS);
  const size_t sm = sizeof(PgNodeLds) + (size_t)kChunk * kPgNB * nw * (f64 ? 8 : 4) + (size_t)2 * (CS - 1) * nw * kPgNB * LR * 8;
  const void *k = f64 ? (const void *)k_pg_nodes<true, false> : (const void *)k_pg_nodes<false, false>;
  hipError_t e = whole_lds(k);
  if (e != hipSuccess) return e;
  if (f64)
    hipLaunchKernelGGL((k_pg_nodes<true, false>), g, b, sm, s, a, LR, CS);
  else
    hipLaunchKernelGGL((k_pg_nodes<false, false>), g, b, sm, s, a, LR, CS);
  return hipGetLastError();
}

template <typename K, typename... A>
static hipError_t launch_node_kernel(K k, unsigned grid, size_t sm, hipStream_t s, A... args) {
  hipError_t e = whole_lds((const void *)k);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(grid), dim3(kNodeThreads), sm, s, args...);
  return hipGetLastError();
}

hipError_t launch_shp_nodes(const TileArgs &a, const NodePlan &p, int prec, int max_nmax, hipStream_t s) {
  hipError_t e = upload_tables();
  if (e != hipSuccess) return e;
  const int R = node_rows(prec, max_nmax, a.S, p.M, p.Mp, a.nrows);
  if (R == 0 || p.M < 1 || p.M > p.Mp || p.Mp > kNodesStride || p.Mp % 4 || max_nmax < 0 || max_nmax > kNmaxLimit)
    return hipErrorInvalidValue;
  const int64_t nt = (a.nrows + R - 1) / R;
  if (nt > 0x7fffffff) return hipErrorInvalidValue;
  const size_t base = node_base_bytes(prec, max_nmax), sm = base + node_lds(a.S, p.Mp, R) * sizeof(double);
  const double *tab = a.d.interp[prec == kFP64];
  if (prec == kFP64) return launch_node_kernel(k_shp_nodes64, (unsigned)nt, sm, s, a, p, tab, R);
  if (prec == kMixedBf16x2)
    return launch_node_kernel(k_shp_nodes<kCmBf16x2>, (unsigned)nt, sm, s, a, p, tab, R, (int)base);
  return launch_node_kernel(k_shp_nodes<kCmBf16x3>, (unsigned)nt, sm, s, a, p, tab, R, (int)base);
}

hipError_t launch_lut_build(float *T, hipStream_t s) {
  hipError_t e = upload_tables();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_lut_build, dim3((kLutSamples + 2 + 255) / 256), dim3(256), 0, s, T);
  return hipGetLastError();
}

hipError_t launch_mark(ServeMark *m, uint64_t seq, hipStream_t s) {
  hipLaunchKernelGGL(k_mark, dim3(1), dim3(1), 0, s, m, seq);
  return hipGetLastError();
}

}  // namespace vp
