// vp_ant.hip -- point components by antenna (gfx950 matrix cores).
//
// A baseline's uvw is the difference of two antennas' coordinates, so a point
// component's phasor is a product of one factor per antenna, and the sum over
// points for all baselines of one (time, channel) is the Hermitian product
//   V_pq = sum_j F_qj conj(F_pj),  F_pj = sqrt(S_j) e^{2 pi i X_p . l_j nu / c}:
// n sines and cosines per component in place of n^2 / 2, and a complex
// multiply-add per visibility on the matrix cores in place of the vector ALU.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "ant_layout.h"
#include "vp_internal.h"

namespace vp {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float2w __attribute__((ext_vector_type(2)));
typedef float float4w __attribute__((ext_vector_type(4)));
typedef uint32_t uint4w __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// mixed path: FP16 pairs
// ---------------------------------------------------------------------------
//
// One workgroup (8 waves) forms the tiles of one macro (up to 128 x 128
// antennas' upper triangle) for one (time, channel) and all points, 32 points
// at a time: the factors of the next 32 points are evaluated into one LDS
// buffer while the matrix cores take the 32 in the other.
//   * Factors: the phase in fixed point (FP64 multiply-adds onto a constant
//     that leaves its fraction of a turn in the low 32 bits), FP32 polynomials
//     for sine and cosine, times sqrt|S| (FP32, from the FP64 flux), split into
//     two FP16 parts (x = hi + lo to 2^-23 of x).  The workgroup's antennas x
//     32 points are divided over the waves as (64 antennas) x (8 points).
//   * Products: v_mfma_f32_16x16x32_f16 on hi/lo, lo/hi and hi/hi, the small
//     products first; lo/lo (2^-24) is dropped.  Each 32-point block's FP32
//     result is added to FP64 sums: the MFMA rounds its 32 products and its
//     addend to ~1.3 units of the largest of them (measured), so that a running
//     FP32 sum would cost its own magnitude's rounding twelve times per block.
// What bounds it: the vector instructions (27 per factor, 16 wave-wide factors
// per SIMD and block at 128 antennas, 144 more for the FP64 adds) and the
// matrix instructions (108 of 16 cycles) in turn: beside other work an MFMA
// still holds the issue of about two vector instructions.  Evaluation and
// products therefore share each wave's instruction stream.  MWA-like points
// (128 antennas, 14 x 32 (time, channel), 20,000 points): 2.5 ms, against 14.7
// ms on the vector path (vector instructions hold 0.47 of the SIMDs' cycles, matrix
// instructions 0.33, in sum 0.95 of those with a workgroup on the CU); 256 antennas
// x 384 channels x 100,000: 42 ms against 233 ms.  Error against FP64 over the
// result's norm: 1.27e-7 (vector path 1.43e-7), irregular channels 1.12e-7
// (1.18e-7).
constexpr int kAntK = 32;  // points per block

__device__ __forceinline__ int ant_xcd(int b, int nt) {
  const int q = nt >> 3, r = nt & 7, x = b & 7, i = b >> 3;
  return x * q + (x < r ? x : r) + i;
}

// LDS offset (in 16-byte units) of part (0 re hi, 1 re lo, 2 im hi, 3 im lo),
// point group g (8 points) and staged antenna r of R.
__device__ __forceinline__ int ant_at(int R, int part, int g, int r) { return (part * 4 + g) * R + r; }

struct AntParts {
  half8 rh, rl, ih, il;
};

__device__ __forceinline__ half8 h8_xor(half8 x, uint4w m) {
  return __builtin_bit_cast(half8, __builtin_bit_cast(uint4w, x) ^ m);
}

__device__ __forceinline__ AntParts ant_load(const half8 *F, int R, int r, int g) {
  AntParts p;
  p.rh = F[ant_at(R, 0, g, r)];
  p.rl = F[ant_at(R, 1, g, r)];
  p.ih = F[ant_at(R, 2, g, r)];
  p.il = F[ant_at(R, 3, g, r)];
  return p;
}

__device__ __forceinline__ float4w ant_mfma(half8 a, half8 b, float4w c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// One 16 x 16 tile (rows: antennas p from A, columns: antennas q from B) of
// F_q conj(F_p) over a block of points.
struct AntTile {
  float4w re, im;
};

// Step e of the products, the small ones first: e = 0..3 hi/lo and lo/hi,
// e = 4, 5 hi/hi (nih, nil: the A side's imaginary parts negated).  The caller
// takes all of its tiles through one step before the next, so that no MFMA
// waits for the one before it.
template <int E>
__device__ __forceinline__ void ant_step(AntTile &t, const AntParts &A, half8 nih, half8 nil, const AntParts &B) {
  const float4w z = {0.f, 0.f, 0.f, 0.f};
  if (E == 0) {
    t.re = ant_mfma(A.rh, B.rl, z);
    t.im = ant_mfma(A.rh, B.il, z);
  } else if (E == 1) {
    t.re = ant_mfma(A.rl, B.rh, t.re);
    t.im = ant_mfma(A.rl, B.ih, t.im);
  } else if (E == 2) {
    t.re = ant_mfma(A.ih, B.il, t.re);
    t.im = ant_mfma(nih, B.rl, t.im);
  } else if (E == 3) {
    t.re = ant_mfma(A.il, B.ih, t.re);
    t.im = ant_mfma(nil, B.rh, t.im);
  } else if (E == 4) {
    t.re = ant_mfma(A.rh, B.rh, t.re);
    t.im = ant_mfma(A.rh, B.ih, t.im);
  } else {
    t.re = ant_mfma(A.ih, B.ih, t.re);
    t.im = ant_mfma(nih, B.rh, t.im);
  }
}

struct AntSum {
  double re[4], im[4];
};

__device__ __forceinline__ void ant_clear(AntSum &s) {
#pragma unroll
  for (int i = 0; i < 4; ++i) s.re[i] = s.im[i] = 0.0;
}
__device__ __forceinline__ void ant_add(AntSum &s, const AntTile &t) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    s.re[i] += (double)t.re[i];
    s.im[i] += (double)t.im[i];
  }
}

// Writes one tile's visibilities: element i of lane l is (p0 + 4 (l / 16) + i,
// q0 + l % 16), with F64 (the FP64 MFMA's layout) row p0 + 4 i + l / 16; the map
// gives the row of each pair (+: as it is, -: conjugated).
template <bool F64 = false>
__device__ __forceinline__ void ant_store(const AntArgs &a, const AntSum &s, int p0, int q0, int64_t t, int k) {
  const int lane = threadIdx.x & 63;
  const int q = q0 + (lane & 15);
  const double un = F64 ? 1.0 : a.unscale[k];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int p = p0 + (F64 ? 4 * i + (lane >> 4) : 4 * (lane >> 4) + i);
    const int m = a.rowmap[(int64_t)p * a.npad + q];
    if (m == 0) continue;
    const double re = s.re[i] * un, im0 = s.im[i] * un;
    const double im = (m < 0) != (a.conj != 0) ? -im0 : im0;
    const int64_t idx = (t * a.B + (m < 0 ? -m : m) - 1) * a.K + k;
    if (a.c64) {
      float2 *o = (float2 *)a.vis + idx;
      if (a.subtract) {
        const float2 d = *o;
        *o = make_float2((float)((double)d.x - re), (float)((double)d.y - im));
      } else {
        *o = make_float2((float)re, (float)im);
      }
    } else {
      double2 *o = (double2 *)a.vis + idx;
      if (a.subtract) {
        const double2 d = *o;
        *o = make_double2(d.x - re, d.y - im);
      } else {
        *o = make_double2(re, im);
      }
    }
  }
}

// Fixed-point phase: a phase of |t| < 2^19 turns added to this is rounded to
// 2^-32 turns, its fraction in the low 32 bits of the sum.
constexpr double kAntTurn = 1572864.0;  // 1.5 x 2^20

// |am| x (cosine, sine) of the phase whose fraction of a turn is lo / 2^32.
// Twice lo, as a signed number, is the distance from the nearest half turn
// (|f| <= 1/4), and the top bit of lo + 2^30 says whether that half turn is
// odd: the sign of both.  Polynomials in f^2 (minimax fits: 7e-9 and 9e-10);
// rms error 5e-8 of the pair against 7e-8 from v_sin and v_cos of an FP32
// fraction.  FINE: the distance from the nearest quarter turn (|f| <= 1/8),
// shorter polynomials (2e-9, 2e-10) and an exchange where the quarter is odd:
// 3e-8 for four instructions more.  The vector path multiplies two phasors for
// most channels of a uniform grid, as the products here do, but takes an
// irregular grid's one by one: only FINE is as exact as that.
template <bool FINE>
__device__ __forceinline__ void ant_factor(uint32_t lo, float am, float &c, float &s) {
  if constexpr (FINE) {
    const float f = (float)(int32_t)(lo << 2) * 5.8207660913467407e-11f;  // 2^-34
    const float x = f * f;
    float ps = fmaf(-75.4016127f, x, 81.5925429f);
    ps = fmaf(ps, x, -41.3416626f);
    ps = fmaf(ps, x, 6.28318529f);
    ps *= f;
    float pc = fmaf(59.2201690f, x, -85.4428447f);
    pc = fmaf(pc, x, 64.9393161f);
    pc = fmaf(pc, x, -19.7392087f);
    pc = fmaf(pc, x, 1.0f);
    const uint32_t w = lo + 0x20000000u, w1 = w << 1;  // the quarter in the top two bits
    const bool odd = (int32_t)w1 < 0;
    s = __builtin_copysignf(am, __uint_as_float(w)) * (odd ? pc : ps);
    c = __builtin_copysignf(am, __uint_as_float(w ^ w1)) * (odd ? ps : pc);
    return;
  }
  const float f = (float)(int32_t)(lo << 1) * 1.16415321826934814453125e-10f;  // 2^-33
  const float x = f * f;
  float ps = fmaf(39.759826660f, x, -76.58116912f);
  ps = fmaf(ps, x, 81.602478027f);
  ps = fmaf(ps, x, -41.34168243f);
  ps = fmaf(ps, x, 6.2831854820f);
  float pc = fmaf(-25.21816253f, x, 60.179039001f);
  pc = fmaf(pc, x, -85.45536041f);
  pc = fmaf(pc, x, 64.939384460f);
  pc = fmaf(pc, x, -19.73920822f);
  pc = fmaf(pc, x, 1.0f);
  const float a = __builtin_copysignf(am, __uint_as_float(lo + 0x40000000u));
  s = a * (ps * f);
  c = a * pc;
}

// What the workgroup stages beside the factors: the points' positions (block b
// in slot b mod 2) and amplitudes per staged antenna block (in slot b mod 4:
// the products of block b still ask for their signs).
struct AntPoints {
  double x[2][kAntK], y[2][kAntK], z[2][kAntK];
  float am[4][kAntSup][kAntK];
};

struct AntPack {
  uint4w rh, rl, ih, il;
};

// One wave's share of the factors of a block: 64 staged antennas (one a lane)
// x 8 points, two points at a time.
template <bool FINE>
struct AntGen {
  double x, y, z;  // this lane's antenna, coordinates x nu / c
  int r, g, sup;   // staged antenna, point group, the antenna's staged block
  bool on;
  __device__ __forceinline__ void pair(AntPack &o, const AntPoints &pt, int blk, int e) const {
    const int slot = blk & 1, j = g * 8 + 2 * e;
    float2w cs, sn;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const double u = fma(x, pt.x[slot][j + h], fma(y, pt.y[slot][j + h], fma(z, pt.z[slot][j + h], kAntTurn)));
      float c, s;
      ant_factor<FINE>((uint32_t)__double_as_longlong(u), pt.am[blk & 3][sup][j + h], c, s);
      cs[h] = c;
      sn[h] = s;
    }
    const half2v ch = __builtin_convertvector(cs, half2v), sh = __builtin_convertvector(sn, half2v);
    const float2w cr = {__builtin_fmaf((float)ch[0], -1.f, cs[0]), __builtin_fmaf((float)ch[1], -1.f, cs[1])};
    const float2w sr = {__builtin_fmaf((float)sh[0], -1.f, sn[0]), __builtin_fmaf((float)sh[1], -1.f, sn[1])};
    o.rh[e] = __builtin_bit_cast(uint32_t, ch);
    o.ih[e] = __builtin_bit_cast(uint32_t, sh);
    o.rl[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(cr, half2v));
    o.il[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(sr, half2v));
  }
  __device__ __forceinline__ void store(const AntPack &o, half8 *F, int R) const {
    if (!on) return;
    F[ant_at(R, 0, g, r)] = __builtin_bit_cast(half8, o.rh);
    F[ant_at(R, 1, g, r)] = __builtin_bit_cast(half8, o.rl);
    F[ant_at(R, 2, g, r)] = __builtin_bit_cast(half8, o.ih);
    F[ant_at(R, 3, g, r)] = __builtin_bit_cast(half8, o.il);
  }
};

__device__ __forceinline__ void ant_negate(AntParts &p, uint4w m) {
  p.rh = h8_xor(p.rh, m);
  p.rl = h8_xor(p.rl, m);
  p.ih = h8_xor(p.ih, m);
  p.il = h8_xor(p.il, m);
}

// Sign bits of the 8 points of this lane's group, as FP16 sign masks (points
// of negative flux enter the product with a minus sign).
__device__ __forceinline__ uint4w ant_signs(const float *am) {
  const int g = (threadIdx.x & 63) >> 4;
  const uint32_t *s = (const uint32_t *)(am + g * 8);
  uint4w m;
#pragma unroll
  for (int e = 0; e < 4; ++e) m[e] = ((s[2 * e] >> 16) & 0x8000u) | (s[2 * e + 1] & 0x80000000u);
  return m;
}

template <typename F>
__device__ __forceinline__ void ant_steps(F f) {
  f(std::integral_constant<int, 0>());
  f(std::integral_constant<int, 1>());
  f(std::integral_constant<int, 2>());
  f(std::integral_constant<int, 3>());
  f(std::integral_constant<int, 4>());
  f(std::integral_constant<int, 5>());
}

// A block of points for a wave on the pair of blocks (ia, ib): four tiles.
// side(e) runs beside step e.
template <bool NEG, typename F>
__device__ __forceinline__ void ant_pair_block(AntSum (&s)[4], const half8 *B_, int R, int ia, int ib, const float *neg_am,
                                               F side) {
  const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
  const uint4w neg = {0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u};
  AntParts A[2], B[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    A[i] = ant_load(B_, R, ia * kAntBlk + 16 * i + r, g);
    B[i] = ant_load(B_, R, ib * kAntBlk + 16 * i + r, g);
  }
  if constexpr (NEG) {
    const uint4w m = ant_signs(neg_am);
    ant_negate(B[0], m);
    ant_negate(B[1], m);
  }
  half8 nih[2], nil[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    nih[i] = h8_xor(A[i].ih, neg);
    nil[i] = h8_xor(A[i].il, neg);
  }
  AntTile t[4];
  ant_steps([&](auto E) {
    constexpr int e = decltype(E)::value;
#pragma unroll
    for (int i = 0; i < 4; ++i) ant_step<e>(t[i], A[i >> 1], nih[i >> 1], nil[i >> 1], B[i & 1]);
    side(E);
  });
#pragma unroll
  for (int i = 0; i < 4; ++i) ant_add(s[i], t[i]);
}

// A block of points for a wave on the upper triangle of block ia: three tiles.
template <bool NEG, typename F>
__device__ __forceinline__ void ant_tri_block(AntSum (&s)[3], const half8 *B_, int R, int ia, const float *neg_am, F side) {
  const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
  const uint4w neg = {0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u};
  const AntParts A0 = ant_load(B_, R, ia * kAntBlk + r, g), A1 = ant_load(B_, R, ia * kAntBlk + 16 + r, g);
  AntParts B0 = A0, B1 = A1;
  if constexpr (NEG) {
    const uint4w m = ant_signs(neg_am);
    ant_negate(B0, m);
    ant_negate(B1, m);
  }
  const half8 n0h = h8_xor(A0.ih, neg), n0l = h8_xor(A0.il, neg);
  const half8 n1h = h8_xor(A1.ih, neg), n1l = h8_xor(A1.il, neg);
  AntTile t[3];
  ant_steps([&](auto E) {
    constexpr int e = decltype(E)::value;
    ant_step<e>(t[0], A0, n0h, n0l, B0);
    ant_step<e>(t[1], A0, n0h, n0l, B1);
    ant_step<e>(t[2], A1, n1h, n1l, B1);
    side(E);
  });
#pragma unroll
  for (int i = 0; i < 3; ++i) ant_add(s[i], t[i]);
}

// ITEMS: 64-antenna x 8-point shares of the factors per wave and block (1 for
// up to 128 staged antennas, 2 beyond).
template <int ITEMS, bool NEG, bool FINE>
__global__ __launch_bounds__(64 * kAntWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_ant_mixed(AntArgs a) {
  extern __shared__ __align__(16) unsigned char ant_sm[];
  const int tile = ant_xcd(blockIdx.x, gridDim.x);
  // macros fastest, then channels: workgroups of neighbouring channels, whose
  // outputs share cache lines, run close together on one XCD
  const int mi = tile % a.nmac, kb = (tile / a.nmac) % a.nkb;
  const int64_t t = tile / (a.nmac * a.nkb);
  const AntMacro &mac = a.mac[mi];
  const int R = mac.nsup * kAntBlk, k0 = kb * a.kpack;
  AntPoints &pt = *(AntPoints *)ant_sm;
  half8 *F = (half8 *)(ant_sm + sizeof(AntPoints));  // [2][4 parts][4 groups][R]
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nc = a.Jp / kAntK;

  AntGen<FINE> gen[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int it = wave + i * kAntWaves;
    const int r = (it >> 2) * 64 + (tid & 63);
    gen[i].on = r < R;
    gen[i].r = gen[i].on ? r : R - 1;
    gen[i].g = it & 3;
    gen[i].sup = gen[i].r >> 5;
    const int k = min(k0 + mac.dk[gen[i].sup], a.K - 1);
    const double *X = a.xyz + (t * a.npad + mac.blk[gen[i].sup] * kAntBlk + (gen[i].r & 31)) * 3;
    const double f = a.fk[k];
    gen[i].x = X[0] * f;
    gen[i].y = X[1] * f;
    gen[i].z = X[2] * f;
  }
  // this thread's part of a block's positions and amplitudes: doubles of the
  // positions for the first 96 threads, amplitudes for the next 32 nsup
  const int pj = tid & 31, pc = tid >> 5;
  const bool is_pos = pc < 3, is_am = pc >= 3 && pc < 3 + mac.nsup;
  const float *am_src = a.amp + (int64_t)min(k0 + mac.dk[is_am ? pc - 3 : 0], a.K - 1) * a.Jp + pj;
  auto fetch = [&](int c, double &dv, float &fv) {
    const int j = min(c, nc - 1) * kAntK + pj;
    if (is_pos) dv = ((const double *)(a.pos + min(j, a.J - 1)))[pc];
    if (is_am) fv = am_src[min(c, nc - 1) * kAntK];
  };
  auto place = [&](int c, double dv, float fv) {
    if (is_pos) (pc == 0 ? pt.x[c & 1] : pc == 1 ? pt.y[c & 1] : pt.z[c & 1])[pj] = dv;
    if (is_am) pt.am[c & 3][pc - 3][pj] = fv;
  };
  double dv = 0.0;
  float fv = 0.f;
  fetch(0, dv, fv);
  place(0, dv, fv);
  fetch(1, dv, fv);
  place(1, dv, fv);
  fetch(2, dv, fv);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    AntPack o;
#pragma unroll
    for (int e = 0; e < 4; ++e) gen[i].pair(o, pt, 0, e);
    gen[i].store(o, F, R);
  }
  const int ia = mac.a[wave], ib = mac.b[wave];
  const int stride = 16 * R;
  // Iteration c multiplies block c and evaluates block c + 1 (at the end, the
  // last block once more, into the buffer that is not read again); the points
  // of block c + 2 go to LDS, those of c + 3 are fetched.  The slot they go to
  // held block c, whose evaluation ended before the barrier.  Every wave passes
  // the same barriers, one per block.
  auto head = [&](int c) {
    __syncthreads();
    place(c + 2, dv, fv);
    fetch(c + 3, dv, fv);
  };
  AntPack o;
  auto side = [&](int c, auto E) {  // steps 0 to 3: a fourth of the wave's share each
    constexpr int e = decltype(E)::value;
    if constexpr (e < 4) {
#pragma unroll
      for (int h = 0; h < ITEMS; ++h) {
        const int n = ITEMS * e + h;
        gen[n >> 2].pair(o, pt, c + 1, n & 3);
        if ((n & 3) == 3) gen[n >> 2].store(o, F + ((c + 1) & 1) * stride, R);
      }
    }
  };
  auto idle = [](auto) {};
  if (mac.tri[wave]) {
    AntSum s[2][3];
#pragma unroll
    for (int i = 0; i < 6; ++i) ant_clear(s[i / 3][i % 3]);
    for (int c = 0; c < nc; ++c) {
      head(c);
      const half8 *cur = F + (c & 1) * stride;
      ant_tri_block<NEG>(s[0], cur, R, ia, pt.am[c & 3][ia], [&](auto E) { side(c, E); });
      if (ib >= 0) ant_tri_block<NEG>(s[1], cur, R, ib, pt.am[c & 3][ib], idle);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int b = i ? ib : ia;
      if (b < 0) continue;
      const int k = k0 + mac.dk[b], p = mac.blk[b] * kAntBlk;
      if (k >= a.K) continue;
      ant_store(a, s[i][0], p, p, t, k);
      ant_store(a, s[i][1], p, p + 16, t, k);
      ant_store(a, s[i][2], p + 16, p + 16, t, k);
    }
  } else if (ia >= 0) {
    AntSum s[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) ant_clear(s[i]);
    for (int c = 0; c < nc; ++c) {
      head(c);
      ant_pair_block<NEG>(s, F + (c & 1) * stride, R, ia, ib, pt.am[c & 3][ia], [&](auto E) { side(c, E); });
    }
    const int k = k0 + mac.dk[ia], p = mac.blk[ia] * kAntBlk, q = mac.blk[ib] * kAntBlk;
    if (k < a.K) {
#pragma unroll
      for (int i = 0; i < 4; ++i) ant_store(a, s[i], p + 16 * (i >> 1), q + 16 * (i & 1), t, k);
    }
  } else {
    for (int c = 0; c < nc; ++c) {
      head(c);
      ant_steps([&](auto E) { side(c, E); });
    }
  }
}

// ---------------------------------------------------------------------------
// FP64 path
// ---------------------------------------------------------------------------
//
// The same product in FP64 on v_mfma_f64_16x16x4f64, 16 points at a time (they
// come from faint to bright, so that the running sums stay small for longest).
// The factors' phases are dots of
// coordinates (wavelengths) with (l, m, n - 1): each product is taken with its
// rounding error and reduced to a fraction of a turn before the sum, so that
// the phase is good to an ulp of a turn and not of the whole phase (the error of
// two factors would otherwise exceed that of the vector path's one phase).
// What bounds it: the matrix cores (12 MFMAs of 64 cycles per four tiles and 4
// points: 0.58 of the cycles in which a CU holds a workgroup), with ~55 vector
// instructions per factor (0.23) and what the two wait for each other.
typedef double double4a __attribute__((ext_vector_type(4)));
constexpr int kAntK64 = 16;  // points per block

// Cosine and sine of the phase (xh + xl) l + (yh + yl) m + (zh + zl) n turns.
struct AntXyz {
  double xh, yh, zh, xl, yl, zl;
};
__device__ __forceinline__ void ant_sincos64(const AntXyz &X, double l, double m, double n, double &c, double &s) {
  const double px = X.xh * l, py = X.yh * m, pz = X.zh * n;
  double e = fma(X.xh, l, -px);
  e = fma(X.xl, l, e);
  e += fma(X.yl, m, fma(X.yh, m, -py));
  e += fma(X.zl, n, fma(X.zh, n, -pz));
  const double t = ((px - rint(px)) + (py - rint(py))) + ((pz - rint(pz)) + e);
  // nearest quarter turn (its number modulo 4 in the low bits of u), |f| <= 1/8
  const double u = t + 1688849860263936.0;  // 1.5 x 2^50
  const uint32_t q = (uint32_t)__double_as_longlong(u);
  const double f = t - (u - 1688849860263936.0), x = f * f;
  // minimax fits of sin(2 pi f) / f (2e-17) and (cos(2 pi f) - 1) / f^2 (1e-19)
  double ps = fma(3.7808689593022955184, x, -15.093804209987113512);
  ps = fma(ps, x, 42.058685020160894047);
  ps = fma(ps, x, -76.705859704274550647);
  ps = fma(ps, x, 81.605249275948035209);
  ps = fma(ps, x, -41.341702240399636207);
  ps = fma(ps, x, 6.2831853071795864572) * f;
  double pc = fma(-1.6990343940660636356, x, 7.9032069115696784291);
  pc = fma(pc, x, -26.426253275854721364);
  pc = fma(pc, x, 60.244641352702008933);
  pc = fma(pc, x, -85.456817206643804246);
  pc = fma(pc, x, 64.939394022668242743);
  pc = fma(pc, x, -19.73920880217871723);
  pc = fma(pc, x, 1.0);
  const bool odd = q & 1;
  const double a = odd ? ps : pc, b = odd ? pc : ps;
  const uint32_t w = q << 30;
  s = __longlong_as_double(__double_as_longlong(b) ^ ((int64_t)(w & 0x80000000u) << 32));
  c = __longlong_as_double(__double_as_longlong(a) ^ ((int64_t)((w + 0x40000000u) & 0x80000000u) << 32));
}

struct AntPoints64 {
  double x[2][kAntK64], y[2][kAntK64], z[2][kAntK64];
  double am[4][kAntSup][kAntK64];  // sign(S) sqrt|S| per staged antenna block
};

// Antennas against rows, a workgroup per time step and 32 antennas: dev receives
// the largest disagreement (as the bits of a non-negative double), and xyz_lo
// what a row's average disagreement says an antenna lies beside xyz: the
// least-squares correction for a complete list (sums over each antenna's rows,
// of residuals formed without rounding; order fixed).  Rows are rounded to 1e-16
// of their length; an antenna seen through one row alone would carry that
// rounding into all of its baselines.  Once per observation; 25 us at 128
// antennas x 14 times, bound by its dependent loads.
__global__ __launch_bounds__(256) void k_ant_refine(int B, int n, int npad, const double *uvw, const int32_t *rowmap,
                                                    const double *xyz, double *xyz_lo, unsigned long long *dev) {
  const int64_t t = blockIdx.x;
  const double *X = xyz + 3 * t * npad;
  double worst = 0.0;
  // 32 antennas x 8 shares of their rows
  __shared__ double part[8][32][4];
  const int a32 = threadIdx.x & 31, sh = threadIdx.x >> 5, p = blockIdx.y * 32 + a32;
  double s[3] = {0, 0, 0};
  {
    int deg = 0;
    for (int q = sh; q < n && p < n; q += 8) {
      const int lo = min(p, q), hi = max(p, q);
      const int m = rowmap[(int64_t)lo * npad + hi];
      if (m == 0) continue;
      ++deg;
      const double *u = uvw + 3 * (t * B + (m < 0 ? -m : m) - 1);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const double a = X[3 * hi + c], b = X[3 * lo + c], v = m < 0 ? -u[c] : u[c];
        // a - b = d + r exactly
        const double d = a - b, bb = d - a, r = (a - (d - bb)) - (b + bb);
        const double e = (v - d) - r;
        worst = fmax(worst, fabs(e));
        s[c] += p == hi ? e : -e;
      }
    }
    for (int c = 0; c < 3; ++c) part[sh][a32][c] = s[c];
    part[sh][a32][3] = deg;
  }
  __syncthreads();
  if (sh == 0) {
    double d[4] = {0, 0, 0, 0};
    for (int i = 0; i < 8; ++i)
      for (int c = 0; c < 4; ++c) d[c] += part[i][a32][c];
    for (int c = 0; c < 3; ++c) xyz_lo[3 * (t * npad + p) + c] = d[c] / (d[3] + 1.0);
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) worst = fmax(worst, __shfl_xor(worst, o));
  if ((threadIdx.x & 63) == 0) atomicMax(dev, (unsigned long long)__double_as_longlong(worst));
}

hipError_t launch_ant_refine(int T, int B, int n, int npad, const double *uvw, const int32_t *rowmap, const double *xyz,
                             double *xyz_lo, unsigned long long *dev, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_ant_refine, dim3((unsigned)T, (unsigned)(npad / kAntBlk)), dim3(256), 0, s, B, n, npad, uvw,
                     rowmap, xyz, xyz_lo, dev);
  return hipGetLastError();
}

// Sums over points of Ar Br, Ai Bi and (Ar + Ai)(Bi - Br), for conj(A) B with three
// real products instead of four.
struct AntTile64 {
  double4a rr, ii, mx;
};

__device__ __forceinline__ double4a ant_mfma64(double a, double b, double4a c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ double ant_flip(double x, double sign_of) {
  return __longlong_as_double(__double_as_longlong(x) ^ (__double_as_longlong(sign_of) & (int64_t)0x8000000000000000ull));
}

// The operands of one wave's tiles for four points (step st of a block), and
// their products: NT = 4, the pair of blocks (ia, ib), or 3, the upper triangle
// of block ia.  F: [re, im][16 points][R].
template <int NT>
struct AntOps64 {
  double Ar[2], Ai[2], Br[NT == 4 ? 2 : 1], Bi[NT == 4 ? 2 : 1], sg;
  __device__ __forceinline__ void load(const double *F, int R, int ia, int ib, int st, const double *am) {
    const int lane = threadIdx.x & 63, j = 4 * st + (lane >> 4), r = lane & 15;
    const double *re = F + j * R, *im = re + kAntK64 * R;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      Ar[i] = re[ia * kAntBlk + 16 * i + r];
      Ai[i] = im[ia * kAntBlk + 16 * i + r];
      if constexpr (NT == 4) {
        Br[i] = re[ib * kAntBlk + 16 * i + r];
        Bi[i] = im[ib * kAntBlk + 16 * i + r];
      }
    }
    sg = am[j];
  }
  template <bool NEG>
  __device__ __forceinline__ void products(AntTile64 (&t)[NT]) const {
    double br[2], bi[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if constexpr (NT == 4) {
        br[i] = Br[i];
        bi[i] = Bi[i];
      } else {
        br[i] = Ar[i];
        bi[i] = Ai[i];
      }
      if constexpr (NEG) {
        br[i] = ant_flip(br[i], sg);
        bi[i] = ant_flip(bi[i], sg);
      }
    }
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int p = i >> 1, q = NT == 4 ? i & 1 : (i + 1) >> 1;
      t[i].rr = ant_mfma64(Ar[p], br[q], t[i].rr);
      t[i].ii = ant_mfma64(Ai[p], bi[q], t[i].ii);
    }
    const double sa[2] = {Ar[0] + Ai[0], Ar[1] + Ai[1]}, db[2] = {bi[0] - br[0], bi[1] - br[1]};
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int p = i >> 1, q = NT == 4 ? i & 1 : (i + 1) >> 1;
      t[i].mx = ant_mfma64(sa[p], db[q], t[i].mx);
    }
  }
};

__device__ __forceinline__ void ant_zero64(AntTile64 &t) { t.rr = t.ii = t.mx = double4a{0.0, 0.0, 0.0, 0.0}; }
__device__ __forceinline__ AntSum ant_sum64(const AntTile64 &t) {
  AntSum s;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    s.re[e] = t.rr[e] + t.ii[e];
    s.im[e] = t.mx[e] + (t.rr[e] - t.ii[e]);
  }
  return s;
}

// 128 antennas, 14 times x 32 channels, 20,000 points: 12.9 ms (the vector
// kernel: 39.6; 15.3 with four real products), 5.2 us per block and round of
// workgroups.  The MFMAs of 64 cycles take 3.2 us of it where a SIMD has a triangle
// (18 a step) and a pair (12); the rest is the factors, which the two waves of a
// SIMD mostly evaluate at the same time, between barriers.
// Error against 80-bit sums, 4,000 points: 6.6e-14 of the visibilities' norm
// (1.7e-13 before, most of it from direction cosines with cancelling terms),
// 6.4e-16 over a 0.1 degree field (5.6e-14), with four real products and with three.
// ITEMS: (64 antennas) x (4 points) shares of the factors per wave and block.
template <int ITEMS, bool NEG>
__global__ __launch_bounds__(64 * kAntWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_ant_fp64(AntArgs a) {
  extern __shared__ __align__(16) unsigned char ant_sm[];
  const int tile = ant_xcd(blockIdx.x, gridDim.x);
  const int mi = tile % a.nmac, kb = (tile / a.nmac) % a.nkb;
  const int64_t t = tile / (a.nmac * a.nkb);
  const AntMacro &mac = a.mac[mi];
  const int R = mac.nsup * kAntBlk, k0 = kb * a.kpack;
  AntPoints64 &pt = *(AntPoints64 *)ant_sm;
  double *F = (double *)(ant_sm + sizeof(AntPoints64));  // [2 buffers][re, im][16 points][R]
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nc = (a.J + kAntK64 - 1) / kAntK64;

  AntXyz X[ITEMS];
  int gr[ITEMS], gg[ITEMS], gs[ITEMS];
  bool on[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int it = wave + i * kAntWaves, r = (it >> 2) * 64 + (tid & 63);
    on[i] = r < R;
    gr[i] = on[i] ? r : R - 1;
    gg[i] = it & 3;
    gs[i] = gr[i] >> 5;
    const double *x = a.xyz + (t * a.npad + mac.blk[gs[i]] * kAntBlk + (gr[i] & 31)) * 3;
    const double *xl = a.xyz_lo + (x - a.xyz);
    const double f = a.fk[min(k0 + mac.dk[gs[i]], a.K - 1)];
    X[i].xh = x[0] * f;
    X[i].yh = x[1] * f;
    X[i].zh = x[2] * f;
    X[i].xl = fma(xl[0], f, fma(x[0], f, -X[i].xh));
    X[i].yl = fma(xl[1], f, fma(x[1], f, -X[i].yh));
    X[i].zl = fma(xl[2], f, fma(x[2], f, -X[i].zh));
  }
  // one point of a block a thread: position components for the first 48
  // threads, amplitudes (per staged block) for the next 16 nsup
  const int pj = tid & 15, pc = tid >> 4;
  const bool is_pos = pc < 3, is_am = pc >= 3 && pc < 3 + mac.nsup;
  const int ka = min(k0 + mac.dk[is_am ? pc - 3 : 0], a.K - 1);
  auto fetch = [&](int c) {
    const int j = min(c, nc - 1) * kAntK64 + pj;
    double v = 0.0;
    if (is_pos) v = ((const double *)(a.pos + min(j, a.J - 1)))[pc];
    if (is_am && j < a.J) v = a.flux64[(int64_t)j * a.Kpad + ka];
    return v;
  };
  auto place = [&](int c, double v) {
    if (is_pos) (pc == 0 ? pt.x[c & 1] : pc == 1 ? pt.y[c & 1] : pt.z[c & 1])[pj] = v;
    if (is_am) pt.am[c & 3][pc - 3][pj] = copysign(sqrt(fabs(v)), v);
  };
  const int stride = 2 * kAntK64 * R;
  // point e of this wave's four of block b
  auto factor = [&](int i, int b, int e) {
    const int j = 4 * gg[i] + e;
    double c, s;
    ant_sincos64(X[i], pt.x[b & 1][j], pt.y[b & 1][j], pt.z[b & 1][j], c, s);
    const double m = fabs(pt.am[b & 3][gs[i]][j]);
    if (on[i]) {
      double *o = F + (b & 1) * stride + j * R + gr[i];
      o[0] = m * c;
      o[kAntK64 * R] = m * s;
    }
  };
  place(0, fetch(0));
  place(1, fetch(1));
  double next = fetch(2);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < ITEMS; ++i)
    for (int e = 0; e < 4; ++e) factor(i, 0, e);
  const int ia = mac.a[wave], ib = mac.b[wave];
  // Iteration c multiplies block c and evaluates block c + 1 (at the end, the
  // last block's points once more, into the buffer that is not read again).
  auto head = [&](int c) {
    __syncthreads();
    place(c + 2, next);
    next = fetch(c + 3);
  };
  auto side = [&](int c, int st) {
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) factor(i, c + 1, st);
  };
  // Each step's operands are read while the step before multiplies.
  if (mac.tri[wave]) {
    AntTile64 w[2][3];
#pragma unroll
    for (int i = 0; i < 6; ++i) ant_zero64(w[i / 3][i % 3]);
    for (int c = 0; c < nc; ++c) {
      head(c);
      const double *cur = F + (c & 1) * stride;
      const int i1 = ib >= 0 ? ib : ia;
      const double *am0 = pt.am[c & 3][ia], *am1 = pt.am[c & 3][i1];
      AntOps64<3> o0, o1;
      o0.load(cur, R, ia, ia, 0, am0);
#pragma unroll
      for (int st = 0; st < 4; ++st) {
        o1.load(cur, R, i1, i1, st, am1);
        o0.template products<NEG>(w[0]);
        if (st < 3) o0.load(cur, R, ia, ia, st + 1, am0);
        if (ib >= 0) o1.template products<NEG>(w[1]);
        side(c, st);
      }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int b = i ? ib : ia;
      if (b < 0) continue;
      const int k = k0 + mac.dk[b], p = mac.blk[b] * kAntBlk;
      if (k >= a.K) continue;
      ant_store<true>(a, ant_sum64(w[i][0]), p, p, t, k);
      ant_store<true>(a, ant_sum64(w[i][1]), p, p + 16, t, k);
      ant_store<true>(a, ant_sum64(w[i][2]), p + 16, p + 16, t, k);
    }
  } else if (ia >= 0) {
    AntTile64 w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) ant_zero64(w[i]);
    for (int c = 0; c < nc; ++c) {
      head(c);
      const double *cur = F + (c & 1) * stride, *am = pt.am[c & 3][ia];
      AntOps64<4> o[2];
      o[0].load(cur, R, ia, ib, 0, am);
#pragma unroll
      for (int st = 0; st < 4; ++st) {
        if (st < 3) o[(st + 1) & 1].load(cur, R, ia, ib, st + 1, am);
        o[st & 1].template products<NEG>(w);
        side(c, st);
      }
    }
    const int k = k0 + mac.dk[ia], p = mac.blk[ia] * kAntBlk, q = mac.blk[ib] * kAntBlk;
    if (k < a.K) {
#pragma unroll
      for (int i = 0; i < 4; ++i) ant_store<true>(a, ant_sum64(w[i]), p + 16 * (i >> 1), q + 16 * (i & 1), t, k);
    }
  } else {
    for (int c = 0; c < nc; ++c) {
      head(c);
#pragma unroll
      for (int st = 0; st < 4; ++st) side(c, st);
    }
  }
}

// The points' largest |S| in each channel, beam and spectrum in it (as the bits
// of a non-negative double; k_flux cleared it).  Workgroup (x, y): 8 channels,
// runs of kPeakRows points; memory bound.
constexpr int kPeakRows = 1024;
__global__ __launch_bounds__(256) void k_ant_peak(AntAmpArgs a) {
  const int k = blockIdx.x * 8 + (threadIdx.x & 7);
  double m = 0.0;
  for (int64_t j0 = (int64_t)blockIdx.y * kPeakRows; j0 < a.J; j0 += (int64_t)gridDim.y * kPeakRows) {
    const int64_t j1 = min(j0 + kPeakRows, (int64_t)a.J);
#pragma unroll 4
    for (int64_t j = j0 + (threadIdx.x >> 3); j < j1; j += 32) m = fmax(m, fabs(a.d.flux64[j * a.Kpad + k]));
  }
#pragma unroll
  for (int o = 8; o < 64; o *= 2) m = fmax(m, __shfl_xor(m, o));
  if ((threadIdx.x & 63) < 8)
    atomicMax((unsigned long long *)(a.d.amp_peak + k), (unsigned long long)__double_as_longlong(m));
}

// Amplitudes of the factors: sign(S) sqrt|S| x scale per (channel, point),
// zero past the last point (blocks of 32 points are taken whole).  The factors
// are FP16 pairs (2^-24 .. 2^16): a channel's scale is the power of two that
// brings the largest of its amplitudes to 2^11 .. 2^12, whatever beam and
// spectrum have left of it.
__global__ __launch_bounds__(256) void k_ant_amp(AntAmpArgs a) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (int64_t)a.Jp * a.Kpad) return;
  const int j = (int)(i / a.Kpad), k = (int)(i % a.Kpad);
  const double peak = a.d.amp_peak[k];
  int e = 12;
  if (peak > 0.0) (void)frexp(sqrt(peak), &e);
  double s = 0.0;
  if (j < a.J) s = a.d.flux64[(int64_t)j * a.Kpad + k];
  a.d.amp[(int64_t)k * a.Jp + j] = (float)copysign(ldexp(sqrt(fabs(s)), 12 - e), s);
  if (j == 0) a.d.amp_unscale[k] = ldexp(1.0, 2 * (e - 12));
}

hipError_t launch_ant_amp(const AntAmpArgs &a, hipStream_t s) {
  const int64_t n = (int64_t)a.Jp * a.Kpad;
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_ant_peak, dim3((unsigned)(a.Kpad / 8), (unsigned)min(1024, (a.J - 1) / kPeakRows + 1)), dim3(256), 0, s,
                     a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_ant_amp, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

template <int ITEMS, bool NEG, bool FINE>
static hipError_t launch_ant_mixed(const AntArgs &a, int nt, size_t sm, hipStream_t s) {
  hipError_t e = whole_lds((const void *)k_ant_mixed<ITEMS, NEG, FINE>);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_ant_mixed<ITEMS, NEG, FINE>), dim3((unsigned)nt), dim3(64 * kAntWaves), sm, s, a);
  return hipGetLastError();
}
template <int ITEMS>
static hipError_t launch_ant_items(const AntArgs &a, int nt, size_t sm, hipStream_t s) {
  if (a.neg)
    return a.fine ? launch_ant_mixed<ITEMS, true, true>(a, nt, sm, s) : launch_ant_mixed<ITEMS, true, false>(a, nt, sm, s);
  return a.fine ? launch_ant_mixed<ITEMS, false, true>(a, nt, sm, s) : launch_ant_mixed<ITEMS, false, false>(a, nt, sm, s);
}

hipError_t launch_ant(const AntArgs &a, hipStream_t s) {
  const int64_t nt = (int64_t)a.T * a.nkb * a.nmac;
  if (nt <= 0) return hipSuccess;
  if (nt > 0x7fffffff || a.J <= 0 || a.max_sup < 1 || a.max_sup > kAntSup || a.Jp % kAntK) return hipErrorInvalidValue;
  const int R = a.max_sup * kAntBlk;
  const size_t sm = sizeof(AntPoints) + (size_t)2 * 16 * R * sizeof(half8);
  return R <= 16 * kAntWaves ? launch_ant_items<1>(a, (int)nt, sm, s) : launch_ant_items<2>(a, (int)nt, sm, s);
}

template <int ITEMS, bool NEG>
static hipError_t launch_ant_fp64(const AntArgs &a, int nt, size_t sm, hipStream_t s) {
  hipError_t e = whole_lds((const void *)k_ant_fp64<ITEMS, NEG>);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_ant_fp64<ITEMS, NEG>), dim3((unsigned)nt), dim3(64 * kAntWaves), sm, s, a);
  return hipGetLastError();
}

hipError_t launch_ant64(const AntArgs &a, hipStream_t s) {
  const int64_t nt = (int64_t)a.T * a.nkb * a.nmac;
  if (nt <= 0) return hipSuccess;
  if (nt > 0x7fffffff || a.J <= 0 || a.max_sup < 1 || a.max_sup > kAntSup) return hipErrorInvalidValue;
  const int R = a.max_sup * kAntBlk;
  const size_t sm = sizeof(AntPoints64) + (size_t)2 * 2 * kAntK64 * R * sizeof(double);
  if (R <= 16 * kAntWaves)
    return a.neg ? launch_ant_fp64<1, true>(a, (int)nt, sm, s) : launch_ant_fp64<1, false>(a, (int)nt, sm, s);
  return a.neg ? launch_ant_fp64<2, true>(a, (int)nt, sm, s) : launch_ant_fp64<2, false>(a, (int)nt, sm, s);
}

}  // namespace vp
