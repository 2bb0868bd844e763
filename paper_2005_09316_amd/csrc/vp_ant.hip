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
// (128 antennas, 14 x 32 (time, channel), 20,000 points): 2.7 ms, against 14.7
// ms on the vector path; 256 antennas x 384 channels x 100,000: 39 ms against
// 233 ms.  Error against FP64 over the result's norm: 1.27e-7 (vector path
// 1.43e-7), irregular channels 1.12e-7 (1.18e-7).
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
// q0 + l % 16); the map gives the row of each pair (+: as it is, -: conjugated).
__device__ __forceinline__ void ant_store(const AntArgs &a, const AntSum &s, int p0, int q0, int64_t t, int k) {
  const int lane = threadIdx.x & 63;
  const int q = q0 + (lane & 15);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int p = p0 + 4 * (lane >> 4) + i;
    const int m = a.rowmap[(int64_t)p * a.npad + q];
    if (m == 0) continue;
    const double re = s.re[i] * a.unscale, im0 = s.im[i] * a.unscale;
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

// Amplitudes of the factors: sign(S) sqrt|S| x scale per (channel, point),
// zero past the last point (blocks of 32 points are taken whole).
__global__ __launch_bounds__(256) void k_ant_amp(AntAmpArgs a) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (int64_t)a.Jp * a.Kpad) return;
  const int j = (int)(i / a.Kpad), k = (int)(i % a.Kpad);
  double s = 0.0;
  if (j < a.J) s = a.flux64[(int64_t)j * a.Kpad + k];
  a.amp[(int64_t)k * a.Jp + j] = (float)copysign(sqrt(fabs(s)) * a.scale, s);
}

hipError_t launch_ant_amp(const AntAmpArgs &a, hipStream_t s) {
  const int64_t n = (int64_t)a.Jp * a.Kpad;
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_ant_amp, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

template <int ITEMS, bool NEG, bool FINE>
static hipError_t launch_ant_mixed(const AntArgs &a, int nt, size_t sm, hipStream_t s) {
  hipError_t e = hipFuncSetAttribute((const void *)k_ant_mixed<ITEMS, NEG, FINE>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm);
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

}  // namespace vp
