// vp_api.cpp -- C ABI of libvp: contexts, observations, sky models, predict
// and subtract.  Serving (vp_submit / vp_poll) lives in vp_serve.cpp.
#include <hip/hip_runtime.h>
#include <rocprofiler-sdk-roctx/roctx.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <utility>
#include <vector>

#include "../../include/vp.h"
#include "ant_layout.h"
#include "shp_nodes.h"
#include "vp_internal.h"
#include "vp_objects.h"

namespace vp {

static thread_local std::string g_err;

int set_error(int code, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

int hip_error(hipError_t e, const char *what) {
  return set_error(e == hipErrorOutOfMemory ? VP_ENOMEM : VP_EDEVICE, "%s: %s", what, hipGetErrorString(e));
}

DeviceGuard::DeviceGuard(int dev) {
  ok = hipGetDevice(&prev) == hipSuccess && hipSetDevice(dev) == hipSuccess;
}
DeviceGuard::~DeviceGuard() {
  if (ok) (void)hipSetDevice(prev);
}

static bool finite_all(const double *p, int64_t n) {
  uint64_t all = 0;  // (no early exit, so that it vectorises)
  for (int64_t i = 0; i < n; ++i) {
    uint64_t u;
    std::memcpy(&u, p + i, sizeof(u));
    all |= (u & 0x7fffffffffffffffull) + 0x0010000000000000ull;  // an exponent of ones carries into the sign
  }
  return all >> 63 == 0;
}

template <typename T>
static hipError_t upload(T **dst, const T *src, int64_t n, DeviceMem &mem) {
  *dst = nullptr;
  if (n <= 0) return hipSuccess;
  hipError_t e = mem.alloc((void **)dst, sizeof(T) * (size_t)n);
  if (e != hipSuccess) return e;
  return hipMemcpy(*dst, src, sizeof(T) * (size_t)n, hipMemcpyHostToDevice);
}

hipError_t DeviceMem::alloc(void **p, size_t bytes) {
  hipError_t e = hipMalloc(p, bytes);
  if (e == hipSuccess) {
    ptrs.push_back(*p);
    total += bytes;
  }
  return e;
}

void DeviceMem::release() {
  for (void *p : ptrs) (void)hipFree(p);
  ptrs.clear();
  total = 0;
}

// ---------------------------------------------------------------------------
// derived (sky, obs) tables
// ---------------------------------------------------------------------------

static int shapelet_nodes(const vp_sky *sky, const vp_obs *obs, int i) {
  double size = 0.0;
  for (int j = 0; j < sky->S; ++j) size += shp_size(i == 0 ? kMixed : kFP64, sky->h_nmax[j]);
  return shp_plan_nodes(i == 1, sky->S, sky->max_nmax, size, obs->f_lo, obs->f_hi, (int64_t)obs->T * obs->B, obs->K);
}

static int pg_sum_nodes(const vp_sky *sky, const vp_obs *obs, int i) {
  // the furthest direction, bounded through the sky's middle:
  // |s - s'|^2 = 4 sin^2(d dec / 2) + 4 cos(dec) cos(dec') sin^2(d ra / 2)
  const double sd = std::sin(0.5 * (sky->pg_dec - obs->dec0)), sa = std::sin(0.5 * (sky->pg_ra - obs->ra0));
  const double to_mid = 2.0 * std::sqrt(sd * sd + std::fabs(std::cos(sky->pg_dec) * std::cos(obs->dec0)) * sa * sa);
  return pg_plan_nodes(i == 3, sky->P, sky->G, std::min(2.0, to_mid + sky->pg_reach), obs->b_max, sky->pg_amax, obs->f_lo,
                       obs->f_hi, obs->beam_fwhm, obs->beam_nu_ref, (int64_t)obs->T * obs->B, obs->K,
                       i == 3 ? obs->uniform64 : obs->uniform);
}

NodePlan node_plan(const vp_sky *sky, const vp_obs *obs, int i) {
  NodePlan p{0, 0, 0.0, 0.0};
  if (obs->K > kNodesMaxChan || (int64_t)obs->T * obs->B > kNodesMaxRows) return p;
  // the fluxes at the nodes lengthen the flux tables' grid
  if (i >= 2 && !grid_fits(((int64_t)(sky->P + sky->G + sky->S) * obs->Kpad + 2ll * (sky->P + sky->G) * kNodesStride) / 256 + 1, 256))
    return p;
  const int M = i < 2 ? shapelet_nodes(sky, obs, i) : pg_sum_nodes(sky, obs, i);
  if (M == 0) return p;
  const int Mp = (M + 3) / 4 * 4;
  p.M = M;
  p.Mp = Mp;
  p.mid = 0.5 * (obs->f_lo + obs->f_hi) / kLightSpeed;
  p.half = 0.5 * (obs->f_hi - obs->f_lo) / kLightSpeed;
  return p;
}

uint64_t plan_bytes(const vp_obs *obs, const NodePlan &p) {
  return p.M > 0 ? sizeof(double) * (uint64_t)node_doubles(obs->K, p.Mp) : 0;
}
uint64_t nflux_bytes(const vp_sky *sky, const NodePlan &p, int i) {
  return i >= 2 && p.M > 0 ? sizeof(double) * (uint64_t)(sky->P + sky->G) * p.Mp : 0;
}

// Points by antenna: whole blocks of 32 points.
int ant_jp(const vp_sky *sky) { return (sky->P + 31) / 32 * 32; }
uint64_t ant_amp_bytes(const vp_sky *sky, const vp_obs *obs) {
  return (sizeof(float) * (uint64_t)ant_jp(sky) + 2 * sizeof(double)) * obs->Kpad;
}
static void place_amp(Derived &d, char *at, const vp_sky *sky, const vp_obs *obs) {
  d.amp = (float *)at;
  d.amp_peak = (double *)(d.amp + (size_t)ant_jp(sky) * obs->Kpad);
  d.amp_unscale = d.amp_peak + obs->Kpad;
}

bool ant_pair(const vp_sky *sky, const vp_obs *obs) {
  if (sky->P < kAntMinPoints || obs->ant_n == 0) return false;
  // Every channel's amplitudes are scaled by their own largest (k_ant_amp), so
  // that beam and spectrum may take any share of the fluxes; these have to be
  // finite (as a product of the largest S_ref and the largest growth), and not so
  // steep that the points' order by S_ref, faint to bright, says nothing about
  // the order in the band.
  if (!grid_fits((int64_t)ant_jp(sky) * obs->Kpad / 256 + 1, 256)) return false;
  const double x = std::max(std::fabs(std::log(obs->f_lo / sky->nu_ref)), std::fabs(std::log(obs->f_hi / sky->nu_ref)));
  const double grow = std::exp(sky->p_amax * x);
  return sky->p_smax >= 1e-30 && sky->p_smax * grow <= 1e30 && grow <= 1048576.0;
}

// Whether a call takes the points by antenna: the mixed paths, where the
// antennas agree with the rows to 1e-10 turns (the path's own phases are good
// to 3e-8) and lie within 2^17 wavelengths (fixed-point phases hold 2^19 turns;
// |n - 1| <= 2), and the matrix kernel is the faster.  Its time goes by blocks
// of 32 points and rounds of one workgroup per CU, a workgroup being a (time,
// channels, macro): 2.1 us each (128 antennas, one round and six; 256, six; 1.8
// at 64 and 96, 1.3 at up to 32).  The vector kernels' goes by points and tiles:
// 0.32 us per point and 768 (128 antennas, 1,780 tiles), or 0.0005 a tile, 0.045
// at least, where few tiles split their components.
//
// The FP64 path: where the antennas agree with the rows to 1e-12 turns (its bar
// is 1e-11 of the flux), and not when complex64 data would take the Gaussians
// in a pass of their own (a rounding more).  Per block of 16 points and round of
// workgroups 5.4 us (measured at 128 to 256 antennas; 4.1 at 64 and 96, 2.7 at
// up to 32: smaller macros), and the vector kernels 0.29 us a point and tile
// per CU (32 to 256 antennas, 1 to 14 times 8 to 32 channels), or 0.0012 a tile,
// 0.09 at least, where few tiles split their components.
// 128 antennas, 14 times, 32 channels: 0.65 against 1.98 us a point.
//
// Where the points may go by nodes instead (plan), that kernel's time decides:
// 2.3e6 values (row, node, point) a us on the mixed path, 0.47e6 in FP64 (32,512
// rows x 30 and 36 nodes), and not below 0.1 and 0.3 us a point.  128 antennas,
// 4 times x 384 channels: 0.41 us a point by nodes, 0.39 by antenna.
static bool use_ant(const vp_sky *sky, const vp_obs *obs, int precision, int dtype, const NodePlan &plan) {
  const bool f64 = precision == kFP64 || precision == kLut;
  if (sky->P < kAntMinPoints) return false;  // (first: such skies' observations may have their antennas found meanwhile)
  if (!grid_fits((int64_t)obs->T * ((obs->K + obs->ant_kpack - 1) / obs->ant_kpack) * obs->ant_nmac, 64 * kAntWaves)) return false;
  const double rows = (double)obs->T * obs->B;
  const double node_us = plan.M == 0 ? 1e30 : sky->P * (f64 ? std::max(0.3, rows * plan.Mp / 0.47e6) : std::max(0.1, rows * plan.Mp / 2.3e6));
  if (precision == kFP64 || precision == kLut) {
    if (obs->ant_n == 0 || !(obs->ant_dev <= 1e-12) || !(obs->ant_reach <= 1e12)) return false;
    if (dtype == VP_C64 && sky->G > 0) return false;
    const double wgs = (double)obs->T * ((obs->K + obs->ant_kpack - 1) / obs->ant_kpack) * obs->ant_nmac;
    const double blk_us = obs->ant_n <= 32 ? 2.7 : obs->ant_n <= 96 ? 4.1 : 5.4;
    const double ant_us = std::ceil(wgs / 256.0) * ((sky->P + 15) / 16) * blk_us + 10.0;
    const double tiles = (double)(((int64_t)obs->T * obs->B + kTileRows - 1) / kTileRows) * (obs->Kpad / kPgChan);
    return ant_us < std::min(node_us, sky->P * (tiles <= kPgSplitTiles ? std::max(0.09, 0.02 + 0.0012 * tiles) : 0.29 * std::ceil(tiles / 256.0)));
  }
  if (precision != kMixed && precision != kMixedBf16 && precision != kMixedBf16x2) return false;
  if (!ant_pair(sky, obs) || !(obs->ant_dev <= 1e-10) || !(obs->ant_reach <= 131072.0)) return false;
  const double wgs = (double)obs->T * ((obs->K + obs->ant_kpack - 1) / obs->ant_kpack) * obs->ant_nmac;
  const double blk_us = obs->ant_n <= 32 ? 1.3 : obs->ant_n <= 96 ? 1.8 : 2.1;
  const double ant_us = std::ceil(wgs / 256.0) * ant_jp(sky) / 32.0 * blk_us + 8.0;
  const double tiles = (double)(((int64_t)obs->T * obs->B + kTileRows - 1) / kTileRows) * (obs->Kpad / kPgChan);
  const double vec_us = sky->P * (tiles <= kPgSplitTiles ? std::max(0.045, 0.015 + 0.0005 * tiles) : 0.32 * tiles / 768.0);
  if (!(ant_us < std::min(node_us, vec_us))) return false;
  // What either costs whatever the points: a round's first block, the visibilities
  // (scattered by antenna, in rows by the vector kernels) and, beside Gaussians, a pass
  // of their own over the data.  100 points and 20 Gaussians, 128 antennas, 4 times x 32
  // channels: 49 us by antenna, 40 together; 64 points, 150 antennas, 2 x 100: 60, 43.
  const double vis = 1e-6 * rows * obs->K;
  return ant_us - 8.0 + 4.9 + 3.9 * std::ceil(wgs / 256.0) + 5.7 * vis + (sky->G > 0 ? 10.0 + 4.8 * vis : 0.0) <
         vec_us * (obs->uniform ? 1.0 : 1.1) + 7.5 + 2.0 * vis;
}

// Whether any mixed call on the pair may take its points by antenna: by nodes
// allowed or not (use_ant asks for the type on the FP64 path only).
bool ant_mixed(const vp_sky *sky, const vp_obs *obs) {
  const NodePlan none{0, 0, 0.0, 0.0};
  return use_ant(sky, obs, kMixed, VP_C128, node_plan(sky, obs, 2)) || use_ant(sky, obs, kMixed, VP_C128, none);
}

// The path whose tables by nodes and by antenna a precision works with: 0 mixed,
// 1 FP64, -1 none.
static int table_path(int precision) {
  return precision == kFP32 ? -1 : precision == kFP64 || precision == kLut ? 1 : 0;
}

// One path's tables by nodes and by antenna, into d.
static hipError_t alloc_path(const vp_sky *sky, const vp_obs *obs, int path, Derived &d, DeviceMem &mem) {
  hipError_t e = hipSuccess;
  for (int i = path; i < kPlans && e == hipSuccess; i += 2) {
    const NodePlan p = d.plan[i] = node_plan(sky, obs, i);
    if (p.M == 0) continue;
    e = mem.alloc((void **)&d.interp[i], plan_bytes(obs, p));
    if (e == hipSuccess && i >= 2) e = mem.alloc((void **)&d.nflux[i - 2], nflux_bytes(sky, p, i));
  }
  if (path == 0 && e == hipSuccess && ant_mixed(sky, obs)) {
    char *amp = nullptr;
    e = mem.alloc((void **)&amp, ant_amp_bytes(sky, obs));
    if (e == hipSuccess) place_amp(d, amp, sky, obs);
  }
  return e;
}

// d with the tables of one path only (-1: of none).
static Derived of_path(Derived d, int path) {
  for (int i = 0; i < kPlans; ++i)
    if (path < 0 || i % 2 != path) d.plan[i].M = 0;
  if (path != 0) d.amp = nullptr;
  return d;
}

static int alloc_derived(const vp_sky *sky, const vp_obs *obs, DerivedEntry **out) {
  DerivedEntry *d = new DerivedEntry();
  const int J = sky->P + sky->G + sky->S;
  const int Jc = std::max(J, 1), Gc = std::max(sky->G, 1), Sc = std::max(sky->S, 1);
  hipError_t e = d->mem.alloc((void **)&d->d.pos, sizeof(double4) * Jc);
  if (e == hipSuccess) e = d->mem.alloc((void **)&d->d.gq, sizeof(double4) * Gc);
  if (e == hipSuccess) e = d->mem.alloc((void **)&d->d.sframe, sizeof(double) * 12 * Sc);
  if (e == hipSuccess) e = d->mem.alloc((void **)&d->d.flux32, sizeof(float) * (size_t)Jc * obs->Kpad);
  if (e == hipSuccess) e = d->mem.alloc((void **)&d->d.flux64, sizeof(double) * (size_t)Jc * obs->Kpad);
  if (e != hipSuccess) {
    d->mem.release();
    delete d;
    return hip_error(e, "allocating per-(sky, observation) tables");
  }
  *out = d;
  return VP_OK;
}

DeriveArgs make_derive_args(const vp_sky *sky, const vp_obs *obs, const Derived &d) {
  DeriveArgs da;
  da.P = sky->P; da.G = sky->G; da.S = sky->S;
  da.ra = sky->ra; da.dec = sky->dec;
  da.g_maj = sky->g_maj; da.g_min = sky->g_min; da.g_pa = sky->g_pa;
  da.s_beta1 = sky->s_beta1; da.s_beta2 = sky->s_beta2; da.s_pa = sky->s_pa;
  da.ra0 = obs->ra0; da.dec0 = obs->dec0;
  da.K = obs->K;
  da.fk = obs->fk;
  da.d = d;
  return da;
}

FluxArgs make_flux_args(const vp_sky *sky, const vp_obs *obs, const Derived &d) {
  FluxArgs fa;
  fa.J = sky->P + sky->G + sky->S; fa.K = obs->K; fa.Kpad = obs->Kpad;
  fa.sref = sky->sref; fa.alpha = sky->alpha; fa.ra = sky->ra; fa.dec = sky->dec; fa.freq = obs->freq;
  fa.nu_ref = sky->nu_ref; fa.ra0 = obs->ra0; fa.dec0 = obs->dec0;
  fa.beam_fwhm = obs->beam_fwhm; fa.beam_nu_ref = obs->beam_nu_ref;
  fa.j0 = sky->P + sky->G;
  fa.lpow = sky->lpow;
  fa.d = d;
  return fa;
}

static hipError_t build_amp(const vp_sky *sky, const vp_obs *obs, const Derived &d, hipStream_t stream) {
  if (!d.amp) return hipSuccess;
  AntAmpArgs a;
  a.J = sky->P; a.Jp = ant_jp(sky); a.Kpad = obs->Kpad;
  a.d = d;
  return launch_ant_amp(a, stream);
}

static uint64_t entry_bytes(const DerivedEntry *d) { return d->mem.total + d->path[0].mem.total + d->path[1].mem.total; }

static void free_entry(vp_ctx *ctx, DerivedEntry *d) {
  // caller holds ctx->mu and has removed d from ctx->derived
  ctx->lib_bytes -= entry_bytes(d);
  for (hipEvent_t e : {d->ready, d->path[0].ready, d->path[1].ready})
    if (e) {
      (void)hipEventSynchronize(e);
      (void)hipEventDestroy(e);
    }
  d->path[0].mem.release();
  d->path[1].mem.release();
  d->mem.release();
  delete d;
}

int get_derived(vp_ctx *ctx, const vp_sky *sky, const vp_obs *obs, hipStream_t stream, int precision, bool serving,
                Derived *out, DerivedEntry **entry, int *built, int *kernels) {
  const auto key = std::make_pair(sky->id, obs->id);
  const int path = table_path(precision);
  std::lock_guard<std::mutex> lk(ctx->mu);
  auto it = ctx->derived.find(key);
  const bool base = it == ctx->derived.end();
  DerivedEntry *d = nullptr;
  if (base) {
    int rc = alloc_derived(sky, obs, &d);
    if (rc != VP_OK) return rc;
  } else {
    d = it->second;
  }
  DerivedEntry::Path *x = path >= 0 ? &d->path[path] : nullptr;
  hipError_t e = hipSuccess;
  bool own = false;  // this call builds the path's tables
  if (x && !x->built) {
    // Not under capture, where they would be built by the graph: the call then does
    // without them, as it does without the memory for them.
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    own = base || (hipStreamIsCapturing(stream, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone);
    x->mem.release();
    if (own && alloc_path(sky, obs, path, d->d, x->mem) != hipSuccess) {
      x->mem.release();
      own = false;
    }
    if (!own) (void)hipGetLastError();
  }
  // before the path's tables, too: the amplitudes come from the components' fluxes
  if (!base && d->ready_stream != stream) e = hipStreamWaitEvent(stream, d->ready, 0);
  if (e == hipSuccess && !own && x && x->built && x->ready && x->ready_stream != stream)
    e = hipStreamWaitEvent(stream, x->ready, 0);
  if (e != hipSuccess) {
    if (own) x->mem.release();
    return hip_error(e, "hipStreamWaitEvent");
  }
  int n = 0;
  if (base || own) {
    const Derived part = of_path(d->d, own ? path : -1);
    DeriveArgs da = make_derive_args(sky, obs, part);
    FluxArgs fa = make_flux_args(sky, obs, part);
    bool any = base && fa.J > 0;
    for (int i = 0; i < kPlans; ++i) any = any || part.plan[i].M > 0;
    if (!base) {  // the components' own are there, and may be being read
      da.P = da.G = da.S = 0;
      fa.J = 0;
    }
    ProfScope ps(serving || !(any || part.amp) ? nullptr : ctx, stream, 0);
    if (any) {
      e = launch_derive(da, stream);
      if (e == hipSuccess) e = launch_flux(fa, stream);
      n += 2;
    } else if (part.amp) {
      e = launch_flux(fa, stream);  // (clears the peaks)
      n += 1;
    }
    if (e == hipSuccess && part.amp) {
      e = build_amp(sky, obs, part, stream);
      n += 2;
    }
    ps.end();
    if (e == hipSuccess && base) {
      e = hipEventCreateWithFlags(&d->ready, hipEventDisableTiming);
      if (e == hipSuccess) e = hipEventRecord(d->ready, stream);
      d->ready_stream = stream;
    } else if (e == hipSuccess && n > 0) {
      if (!x->ready) e = hipEventCreateWithFlags(&x->ready, hipEventDisableTiming);
      if (e == hipSuccess) e = hipEventRecord(x->ready, stream);
      x->ready_stream = stream;
    }
    if (e != hipSuccess) {
      (void)hipStreamSynchronize(stream);
      if (base) {
        ctx->lib_bytes += entry_bytes(d);  // (free_entry takes it off)
        free_entry(ctx, d);
      } else {
        x->mem.release();
      }
      return hip_error(e, "building per-(sky, observation) tables");
    }
    if (own) x->built = true;
    ctx->lib_bytes += base ? entry_bytes(d) : x->mem.total;
  }
  if (base) {
    d->serve_built = serving;
    ctx->derived[key] = d;
  }
  if (serving)
    d->serve_users += 1;
  else
    d->serve_built = false;  // a direct call's kernels may read it from now on: never evicted by serving
  if (built) *built = (base ? kBuiltBase : 0) | (own ? kBuiltPath : 0);
  if (kernels) *kernels = n;
  *out = of_path(d->d, x && x->built ? path : -1);
  if (entry) *entry = d;
  return VP_OK;
}

void serve_release_derived(vp_ctx *ctx, DerivedEntry *d) {
  std::lock_guard<std::mutex> lk(ctx->mu);
  d->serve_users -= 1;
}

void serve_abandon_derived(vp_ctx *ctx, DerivedEntry *d, int built) {
  std::lock_guard<std::mutex> lk(ctx->mu);
  d->serve_users -= 1;
  if (!(built & kBuiltBase)) {
    ctx->lib_bytes -= d->path[0].mem.total;
    d->path[0].built = false;  // serving is mixed; the next call builds them anew
    d->path[0].mem.release();
    return;
  }
  for (auto it = ctx->derived.begin(); it != ctx->derived.end(); ++it)
    if (it->second == d) {
      ctx->derived.erase(it);
      free_entry(ctx, d);
      return;
    }
}

uint64_t serve_evictable_bytes(vp_ctx *ctx) {
  std::lock_guard<std::mutex> lk(ctx->mu);
  uint64_t b = 0;
  for (auto &kv : ctx->derived)
    if (kv.second->serve_built && kv.second->serve_users == 0) b += entry_bytes(kv.second);
  return b;
}

void serve_evict(vp_ctx *ctx) {
  std::lock_guard<std::mutex> lk(ctx->mu);
  for (auto it = ctx->derived.begin(); it != ctx->derived.end();) {
    DerivedEntry *d = it->second;
    if (d->serve_built && d->serve_users == 0) {
      it = ctx->derived.erase(it);
      free_entry(ctx, d);
    } else {
      ++it;
    }
  }
}

void drop_derived(vp_ctx *ctx, uint64_t sky_id, uint64_t obs_id) {
  // caller holds ctx->mu; an id of 0 matches nothing
  for (auto it = ctx->derived.begin(); it != ctx->derived.end();) {
    if ((sky_id && it->first.first == sky_id) || (obs_id && it->first.second == obs_id)) {
      DerivedEntry *d = it->second;
      it = ctx->derived.erase(it);
      free_entry(ctx, d);
    } else {
      ++it;
    }
  }
}

void drop_all_derived(vp_ctx *ctx) {
  // caller holds ctx->mu
  for (auto &kv : ctx->derived) free_entry(ctx, kv.second);
  ctx->derived.clear();
}

// ---------------------------------------------------------------------------
// profiling
// ---------------------------------------------------------------------------

TraceRange::TraceRange(const char *name) { roctxRangePushA(name); }
TraceRange::~TraceRange() { roctxRangePop(); }

ProfScope::ProfScope(vp_ctx *c, hipStream_t s, int k) : ctx(c), stream(s), kind(k) {
  if (ctx && ctx->profile) {
    if (hipEventCreate(&e0) == hipSuccess && hipEventCreate(&e1) == hipSuccess &&
        hipEventRecord(e0, stream) == hipSuccess)
      active = true;
  }
}

void ProfScope::end() {
  if (!active) return;
  active = false;
  if (hipEventRecord(e1, stream) == hipSuccess) {
    std::lock_guard<std::mutex> lk(ctx->prof_mu);
    ctx->prof_pending.push_back({kind, e0, e1});
  } else {
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
  }
}

ProfScope::~ProfScope() { end(); }

// ---------------------------------------------------------------------------
// predict / subtract
// ---------------------------------------------------------------------------

// The basis table of the lookup-table variant, built once per context (the
// build is synchronous: later calls on any stream find it complete).
static int get_lut(vp_ctx *ctx, hipStream_t stream, const float **out) {
  std::lock_guard<std::mutex> lk(ctx->mu);
  if (!ctx->lut) {
    void *p = nullptr;
    hipError_t e = ctx->lut_mem.alloc(&p, kLutBytes);
    if (e == hipSuccess) e = launch_lut_build((float *)p, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) {
      ctx->lut_mem.release();
      return hip_error(e, "building the basis lookup table");
    }
    ctx->lut = (float *)p;
  }
  *out = ctx->lut;
  return VP_OK;
}

void SumsPool::release() {
  for (Slot &s : slot) {
    if (s.done) {
      (void)hipEventSynchronize(s.done);
      (void)hipEventDestroy(s.done);
    }
    if (s.p) (void)hipFree(s.p);
    s = Slot();
  }
}

SumsSpace SumsLease::take(SumsPool &pool, uint64_t want, hipStream_t stream) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) {
    (void)hipGetLastError();
    return {nullptr, 0};
  }
  uint64_t bytes = kSumsMin;
  while (bytes < want && bytes < kSumsMax) bytes *= 2;
  std::unique_lock<std::mutex> lk(pool.mu);
  SumsPool::Slot *s = nullptr;
  for (SumsPool::Slot &x : pool.slot)  // this stream's own: nothing to wait for
    if (!s && x.used && x.last == stream) s = &x;
  for (SumsPool::Slot &x : pool.slot)
    if (!s && !x.p) s = &x;
  if (!s) {
    s = &pool.slot[pool.next];
    pool.next = (pool.next + 1) % SumsPool::kSlots;
  }
  hipError_t e = s->done ? hipSuccess : hipEventCreateWithFlags(&s->done, hipEventDisableTiming);
  if (e == hipSuccess && s->bytes < bytes) {
    void *p = nullptr;
    if (hipMalloc(&p, bytes) == hipSuccess) {
      if (s->p) {
        (void)hipEventSynchronize(s->done);
        (void)hipFree(s->p);
      }
      s->p = p;
      s->bytes = bytes;
    } else {
      (void)hipGetLastError();  // the smaller one, if there is one, will do in parts
    }
  }
  if (e == hipSuccess && s->used) e = hipStreamWaitEvent(stream, s->done, 0);
  if (e != hipSuccess || !s->p) {
    (void)hipGetLastError();
    return {nullptr, 0};
  }
  lk_ = std::move(lk);
  slot_ = s;
  stream_ = stream;
  return {(double2 *)s->p, s->bytes};
}

SumsLease::~SumsLease() {
  if (!slot_) return;
  if (hipEventRecord(slot_->done, stream_) != hipSuccess) (void)hipStreamSynchronize(stream_);
  slot_->last = stream_;
  slot_->used = true;
}

// How a call's points and Gaussians go.
struct PgRoute {
  bool by_nodes;  // Gaussians, and points unless by antenna
  bool ant;       // points by antenna
  bool sums;      // their sums go to the Gaussians through a workspace
  int step;       // channels by which parts of a time step are counted
};
static PgRoute pg_route(const vp_sky *sky, const vp_obs *obs, int precision, int dtype, const Derived &d, bool nodes) {
  PgRoute r;
  const bool ant64 = precision == kFP64 || precision == kLut;
  r.by_nodes = d.plan[2 + ant64].M > 0 && precision != kFP32 && (nodes || ant64);
  r.ant = (ant64 || d.amp) && use_ant(sky, obs, precision, dtype, r.by_nodes ? d.plan[2 + ant64] : NodePlan{0, 0, 0.0, 0.0});
  r.sums = r.ant && !ant64 && dtype == VP_C64 && sky->G > 0;
  r.step = r.by_nodes ? 16 : 8;
  if (r.sums && sizeof(double2) * (uint64_t)obs->B * std::min(r.step, obs->K) > kSumsMin) r.ant = r.sums = false;
  return r;
}

uint64_t sums_bytes(const vp_sky *sky, const vp_obs *obs, int precision, int dtype, const Derived &d, bool nodes) {
  if (!pg_route(sky, obs, precision, dtype, d, nodes).sums) return 0;
  return sizeof(double2) * (uint64_t)obs->T * obs->B * obs->K;
}

int launch_passes(vp_ctx *prof, const vp_sky *sky, const vp_obs *obs, int precision, int dtype, void *vis,
                  int subtract, hipStream_t stream, const Derived &d, const float *lut, SumsSpace sums, int *kernels,
                  bool nodes) {
  TileArgs a;
  a.nrows = (int64_t)obs->T * obs->B;
  a.K = obs->K;
  a.Kpad = obs->Kpad;
  a.uvw = obs->uvw;
  a.fk = obs->fk;
  a.P = sky->P; a.G = sky->G; a.S = sky->S;
  a.d = d;
  a.t = sky->tiles;
  a.vis = vis;
  a.subtract = subtract;
  a.c64 = dtype == VP_C64;
  a.conj = obs->sign < 0;
  a.n_rb = (int)((a.nrows + kTileRows - 1) / kTileRows);
  a.n_cb = obs->Kpad / kPgChan;
  a.lut = lut;
  a.shp_chan = kShpChan;
  a.ld = a.K;
  a.chan0 = 0;
  a.call_rows = a.nrows;
  a.sums = nullptr;
  a.dfk = obs->dfk;
  a.uniform = precision == kFP64 || precision == kLut ? obs->uniform64 : obs->uniform;
  // A sky of shapelets only skips the point/Gaussian pass, which would only
  // write zeros (predict) or rewrite the data unchanged (subtract).
  const bool ant64 = precision == kFP64 || precision == kLut;
  PgRoute route = pg_route(sky, obs, precision, dtype, d, nodes);
  if (route.sums && !sums.p) route.ant = route.sums = false;
  const bool by_nodes = route.by_nodes, ant = route.ant;
  const int path = precision == kFP64 ? 1 : precision == kFP32 || precision == kLut ? -1 : 0;
  const bool shp_by_nodes = sky->S > 0 && nodes && path >= 0 && d.plan[path].M > 0;
  // A handful of points goes along with the shapelets' outputs by nodes, as
  // envelopes of 1: some 4 us each where a pass of their own over the data takes 26
  // (113,792 rows x 32 channels).
  a.out_points = shp_by_nodes && !ant && sky->G == 0 && sky->P <= kOutPoints ? sky->P : 0;
  const bool pg_pass = a.out_points > 0 ? false : ant ? sky->G > 0 : sky->P + sky->G > 0 || sky->S == 0;
  a.skip_points = ant;
  a.fresh = !pg_pass && !ant && !subtract;
  hipError_t e = hipSuccess;
  AntArgs p;
  if (ant) {
    p.T = obs->T; p.B = obs->B; p.K = obs->K;
    p.npad = obs->ant_npad;
    p.J = sky->P; p.Jp = ant_jp(sky);
    p.nmac = obs->ant_nmac; p.max_sup = obs->ant_max_sup;
    p.kpack = obs->ant_kpack; p.nkb = (obs->K + p.kpack - 1) / p.kpack;
    p.mac = obs->ant_mac; p.xyz = obs->ant_xyz; p.xyz_lo = obs->ant_lo; p.rowmap = obs->ant_rowmap;
    p.fk = obs->fk; p.pos = d.pos; p.amp = d.amp;
    p.flux64 = d.flux64; p.Kpad = obs->Kpad;
    p.unscale = d.amp_unscale;
    p.neg = sky->p_neg;
    p.fine = !obs->uniform;
    p.vis = vis; p.c64 = a.c64; p.conj = a.conj; p.subtract = subtract;
  }
  auto points = [&](const AntArgs &x) {
    ProfScope ps(prof, stream, 1);
    if (kernels) ++*kernels;
    return ant64 ? launch_ant64(x, stream) : launch_ant(x, stream);
  };
  auto gaussians = [&](const TileArgs &x) {  // (and the points, if not by antenna)
    ProfScope ps(prof, stream, 1);
    if (kernels) ++*kernels;
    return by_nodes ? launch_pg_nodes(x, precision, stream) : launch_pg(x, precision, stream);
  };
  if (route.sums) {
    // parts of the call, of like sizes: whole time steps, or channels of one
    const uint64_t chan = sizeof(double2) * (uint64_t)obs->B, whole = chan * obs->K;
    int tc = 1, kc = obs->K;
    if (whole <= sums.bytes) {
      tc = (int)std::min<uint64_t>(obs->T, sums.bytes / whole);
      const int parts = (obs->T + tc - 1) / tc;
      tc = (obs->T + parts - 1) / parts;
    } else {
      const int most = (int)(sums.bytes / chan) / route.step * route.step, parts = (obs->K + most - 1) / most;
      kc = ((obs->K + parts - 1) / parts + route.step - 1) / route.step * route.step;
    }
    const size_t vis_size = a.c64 ? sizeof(float2) : sizeof(double2);
    for (int t0 = 0; t0 < obs->T && e == hipSuccess; t0 += tc)
      for (int k0 = 0; k0 < obs->K && e == hipSuccess; k0 += kc) {
        const int nt = std::min(tc, obs->T - t0), nk = std::min(kc, obs->K - k0);
        AntArgs x = p;
        x.T = nt; x.K = nk;
        x.nkb = (nk + x.kpack - 1) / x.kpack;
        x.xyz += (size_t)t0 * x.npad * 3; x.xyz_lo += (size_t)t0 * x.npad * 3;
        x.fk += k0; x.amp += (size_t)k0 * x.Jp; x.unscale += k0; x.flux64 += k0;
        x.vis = sums.p; x.c64 = 0; x.subtract = 0;
        e = points(x);
        TileArgs y = a;
        const int64_t row0 = (int64_t)t0 * obs->B;
        y.nrows = (int64_t)nt * obs->B; y.K = nk; y.chan0 = k0;
        y.n_rb = (int)((y.nrows + kTileRows - 1) / kTileRows);
        y.n_cb = (nk + kPgChan - 1) / kPgChan;
        y.uvw += 3 * row0; y.fk += k0; y.d.flux32 += k0; y.d.flux64 += k0;
        y.vis = (char *)vis + vis_size * (row0 * obs->K + k0);
        y.sums = sums.p;
        if (e == hipSuccess) e = gaussians(y);
      }
    if (e != hipSuccess) return hip_error(e, "launching the points by antenna and the Gaussians");
  } else {
    if (ant) e = points(p);
    if (e != hipSuccess) return hip_error(e, "launching the kernel of the points by antenna");
    if (pg_pass) e = gaussians(a);
    if (e != hipSuccess) return hip_error(e, "launching the point/Gaussian kernel");
  }
  if (sky->S > 0) {
    a.n_cb = (obs->K + kShpChan - 1) / kShpChan;
    ProfScope ps(prof, stream, 2);
    a.uniform = obs->uniform64;  // (the outputs by nodes turn FP64 phasors by dfk)
    if (shp_by_nodes)
      e = launch_shp_nodes(a, d.plan[path], precision, sky->max_nmax, stream);
    else
      e = launch_shp(a, precision, sky->max_nmax, stream);
    if (kernels) ++*kernels;
    if (e == hipErrorNotSupported) return set_error(VP_EINVAL, "precision %d has no shapelet kernel", precision);
    if (e != hipSuccess) return hip_error(e, "launching the shapelet kernel");
  }
  return VP_OK;
}

int run_tiles(vp_ctx *ctx, const vp_sky *sky, const vp_obs *obs, int precision, int dtype, void *vis,
              int subtract, hipStream_t stream, bool nodes) {
  Derived d;
  int rc = get_derived(ctx, sky, obs, stream, precision, false, &d);
  if (rc != VP_OK) return rc;
  const float *lut = nullptr;
  if (precision == kLut && sky->S > 0) {
    rc = get_lut(ctx, stream, &lut);
    if (rc != VP_OK) return rc;
  }
  SumsLease lease;
  const uint64_t want = sums_bytes(sky, obs, precision, dtype, d, nodes);
  const SumsSpace sums = want ? lease.take(ctx->sums, want, stream) : SumsSpace{nullptr, 0};
  return launch_passes(ctx, sky, obs, precision, dtype, vis, subtract, stream, d, lut, sums, nullptr, nodes);
}

int check_call(vp_ctx *ctx, const vp_sky *sky, const vp_obs *obs, int precision, int dtype, void *vis) {
  if (!ctx || !sky || !obs) return set_error(VP_EINVAL, "NULL context, sky or observation");
  if (sky->ctx != ctx || obs->ctx != ctx) return set_error(VP_EINVAL, "sky or observation belongs to another context");
  if (precision < VP_PREC_FP64 || precision > VP_PREC_LUT)
    return set_error(VP_EINVAL, "unknown precision %d", precision);
  if (precision == VP_PREC_MIXED_F32MMA)
    return set_error(VP_EINVAL, "precision %d (FP32 MFMA contraction) is retired", precision);
  if (dtype != VP_C128 && dtype != VP_C64) return set_error(VP_EINVAL, "unknown dtype %d", dtype);
  if (!vis) return set_error(VP_EINVAL, "NULL visibility buffer");
  return VP_OK;
}

}  // namespace vp

using namespace vp;

extern "C" {

const char *vp_last_error(void) { return g_err.c_str(); }

const char *vp_version(void) { return "libvp 0.1 (gfx950)"; }

int vp_create_ctx(int hip_device, uint64_t hbm_budget_bytes, vp_ctx **out) {
  if (!out) return set_error(VP_EINVAL, "NULL out");
  int n = 0;
  hipError_t e = hipGetDeviceCount(&n);
  if (e != hipSuccess) return hip_error(e, "hipGetDeviceCount");
  if (hip_device < 0 || hip_device >= n) return set_error(VP_EINVAL, "device %d out of range (%d devices)", hip_device, n);
  DeviceGuard g(hip_device);
  if (!g.ok) return set_error(VP_EDEVICE, "cannot select device %d", hip_device);
  e = device_init(hip_device);
  if (e != hipSuccess) return hip_error(e, "initialising the device");
  size_t free_b = 0, total_b = 0;
  e = hipMemGetInfo(&free_b, &total_b);
  if (e != hipSuccess) return hip_error(e, "hipMemGetInfo");
  vp_ctx *c = new vp_ctx();
  c->device = hip_device;
  c->budget = hbm_budget_bytes ? hbm_budget_bytes : (uint64_t)(0.9 * (double)free_b);
  *out = c;
  return VP_OK;
}

int vp_destroy_ctx(vp_ctx *ctx) {
  if (!ctx) return set_error(VP_EINVAL, "NULL context");
  if (serve_pending(ctx)) return set_error(VP_EBUSY, "serving jobs still pending");
  serve_shutdown(ctx);
  DeviceGuard g(ctx->device);
  {
    std::lock_guard<std::mutex> lk(ctx->mu);
    drop_all_derived(ctx);
    for (vp_obs *o : ctx->obs) {
      o->mem.release();
      delete o;
    }
    for (vp_sky *s : ctx->skies) {
      s->mem.release();
      delete s;
    }
    ctx->obs.clear();
    ctx->skies.clear();
  }
  {
    std::lock_guard<std::mutex> lk(ctx->prof_mu);
    for (auto &r : ctx->prof_pending) {
      (void)hipEventDestroy(r.e0);
      (void)hipEventDestroy(r.e1);
    }
  }
  if (ctx->peel) {
    if (ctx->peel->done) {
      (void)hipEventSynchronize(ctx->peel->done);
      (void)hipEventDestroy(ctx->peel->done);
    }
    ctx->peel->mem.release();
    delete ctx->peel;
  }
  ctx->sums.release();
  ctx->lut_mem.release();
  delete ctx;
  return VP_OK;
}

// The antennas behind the rows, if there are any (see ant_layout.h), and the
// tables by which the kernels work on them.  The search and its upload take 20 us
// (6 antennas) to 1 ms (256, a seventh of the baselines flagged), more than a
// small sky's predictions, so they wait for a sky that may use them: done where
// the second of the two is created, none is left to a call on them.
static hipError_t upload_antennas(vp_obs *o, const double *uvw) {
  // a complete list of n antennas has B = n (n - 1) / 2 rows; half of them
  // flagged, n = 2 sqrt(B)
  const int max_n = std::min(kAntMaxN, (int)(2.2 * std::sqrt((double)o->B)) + 8);
  const double f = o->f_hi / kLightSpeed;
  const AntLayout L = find_antennas(o->T, o->B, uvw, 1e-10 / f, max_n, false);
  const int np = (L.n + kAntBlk - 1) / kAntBlk * kAntBlk;
  // (few baselines over very many times: the padding would outgrow the uvw)
  if (L.n == 0 || (np > o->B && (int64_t)o->T * np > 1 << 20)) return hipSuccess;
  const std::vector<AntMacro> mac = ant_macros(L.n, &o->ant_kpack);
  // one buffer: largest disagreement, coordinates, their corrections, pair map, macros
  const size_t n_xyz = sizeof(double) * 3 * (size_t)o->T * np, n_map = sizeof(int32_t) * (size_t)np * np;
  const size_t o_xyz = 16, o_lo = o_xyz + n_xyz, o_map = o_lo + n_xyz, o_mac = o_map + n_map;
  std::vector<char> buf(o_mac + sizeof(AntMacro) * mac.size(), 0);
  double *xyz = (double *)(buf.data() + o_xyz);
  int32_t *map = (int32_t *)(buf.data() + o_map);
  std::memcpy(buf.data() + o_mac, mac.data(), sizeof(AntMacro) * mac.size());
  for (int b = 0; b < o->B; ++b) {
    const int p = L.p[b], q = L.q[b];
    if (p <= q)
      map[(size_t)p * np + q] = b + 1;
    else
      map[(size_t)q * np + p] = -(b + 1);
  }
  for (int t = 0; t < o->T; ++t)
    std::copy(&L.xyz[(size_t)t * L.n * 3], &L.xyz[(size_t)t * L.n * 3] + 3 * (size_t)L.n, &xyz[(size_t)t * np * 3]);
  char *dev = nullptr;
  hipError_t e = upload(&dev, buf.data(), (int64_t)buf.size(), o->mem);
  if (e != hipSuccess) return e;
  o->ant_xyz = (double *)(dev + o_xyz);
  o->ant_lo = (double *)(dev + o_lo);
  o->ant_rowmap = (int32_t *)(dev + o_map);
  o->ant_mac = (AntMacro *)(dev + o_mac);
  double worst = 0.0;
  e = launch_ant_refine(o->T, o->B, L.n, np, o->uvw, o->ant_rowmap, o->ant_xyz, o->ant_lo, (unsigned long long *)dev, nullptr);
  if (e == hipSuccess) e = hipMemcpy(&worst, dev, sizeof(worst), hipMemcpyDeviceToHost);
  if (e != hipSuccess) return e;
  if (!(worst * f <= 1e-10)) return hipSuccess;  // other time steps have other antennas
  o->ant_n = L.n;
  o->ant_npad = np;
  o->ant_nmac = (int)mac.size();
  for (const AntMacro &m : mac) o->ant_max_sup = std::max(o->ant_max_sup, (int)m.nsup);
  o->ant_dev = worst * f;
  for (size_t i = 0; i < L.xyz.size(); i += 3)
    o->ant_reach = std::max(o->ant_reach, f * (std::fabs(L.xyz[i]) + std::fabs(L.xyz[i + 1]) + std::fabs(L.xyz[i + 2])));
  return hipSuccess;
}

// uvw: the rows on the host, or NULL to read them back.
static hipError_t look_for_antennas(vp_obs *o, const double *uvw) {
  o->ant_looked = true;
  if (o->B > (int64_t)kAntMaxN * (kAntMaxN + 1) / 2 || !grid_fits(o->T, 256)) return hipSuccess;
  hipError_t e = hipSuccess;
  try {
    std::vector<double> rows;
    if (!uvw) {
      rows.resize(3 * (size_t)o->T * o->B);
      e = hipMemcpy(rows.data(), o->uvw, sizeof(double) * rows.size(), hipMemcpyDeviceToHost);
      uvw = rows.data();
    }
    if (e == hipSuccess) e = upload_antennas(o, uvw);
  } catch (const std::bad_alloc &) {  // without the antennas, points go the vector path
    o->ant_n = 0;
  }
  return e;
}

int vp_create_obs(vp_ctx *ctx, const vp_obs_desc *desc, vp_obs **out) {
  if (!ctx || !desc || !out) return set_error(VP_EINVAL, "NULL argument");
  if (desc->n_time <= 0 || desc->n_bl <= 0 || desc->n_chan <= 0)
    return set_error(VP_EINVAL, "n_time, n_bl, n_chan must be positive");
  const int64_t nrows = (int64_t)desc->n_time * desc->n_bl;
  if (nrows > (int64_t)1 << 30 || desc->n_chan > (1 << 20))
    return set_error(VP_EINVAL, "observation too large");
  if (!desc->uvw_m || !desc->freq_hz) return set_error(VP_EINVAL, "NULL uvw or frequency array");
  if (desc->sign != 1 && desc->sign != -1) return set_error(VP_EINVAL, "sign must be +1 or -1");
  if (!finite_all(desc->uvw_m, 3 * nrows)) return set_error(VP_EINVAL, "non-finite uvw");
  if (!finite_all(desc->freq_hz, desc->n_chan)) return set_error(VP_EINVAL, "non-finite frequency");
  for (int k = 0; k < desc->n_chan; ++k)
    if (desc->freq_hz[k] <= 0) return set_error(VP_EINVAL, "frequency %d not positive", k);
  if (!std::isfinite(desc->ra0) || !std::isfinite(desc->dec0)) return set_error(VP_EINVAL, "non-finite phase centre");
  if (!std::isfinite(desc->beam_fwhm_rad) || desc->beam_fwhm_rad < 0)
    return set_error(VP_EINVAL, "beam FWHM must be finite and >= 0");
  if (desc->beam_fwhm_rad > 0 && !(desc->beam_nu_ref_hz > 0 && std::isfinite(desc->beam_nu_ref_hz)))
    return set_error(VP_EINVAL, "beam reference frequency must be positive");
  DeviceGuard g(ctx->device);
  if (!g.ok) return set_error(VP_EDEVICE, "cannot select device");
  vp_obs *o = new vp_obs();
  o->ctx = ctx;
  o->T = desc->n_time;
  o->B = desc->n_bl;
  o->K = desc->n_chan;
  o->Kpad = (desc->n_chan + kPgChan - 1) / kPgChan * kPgChan;
  o->ra0 = desc->ra0;
  o->dec0 = desc->dec0;
  o->sign = desc->sign;
  o->beam_fwhm = desc->beam_fwhm_rad;
  o->beam_nu_ref = desc->beam_nu_ref_hz;
  o->h_freq.assign(desc->freq_hz, desc->freq_hz + desc->n_chan);
  o->f_lo = *std::min_element(o->h_freq.begin(), o->h_freq.end());
  o->f_hi = *std::max_element(o->h_freq.begin(), o->h_freq.end());
  double longest[4] = {0, 0, 0, 0};  // (four chains: one would wait on itself)
  for (int64_t r = 0; r < nrows; r += 4)
    for (int64_t i = 0; i < 4; ++i) {
      const double *b = desc->uvw_m + 3 * std::min(r + i, nrows - 1), l = b[0] * b[0] + b[1] * b[1] + b[2] * b[2];
      longest[i] = l > longest[i] ? l : longest[i];
    }
  o->b_max = std::sqrt(*std::max_element(longest, longest + 4));
  std::vector<double> fk(o->Kpad);
  for (int k = 0; k < o->Kpad; ++k) fk[k] = desc->freq_hz[std::min(k, o->K - 1)] / kLightSpeed;
  if (o->K >= 2) {
    // uniformly spaced channels let the kernels rotate phasors between
    // channels: the mixed path while the grid holds to 1e-12 of nu/c (phase
    // error below 1e-8 turns for |t0| up to 1e4 m), the FP64 path while it
    // holds to 1e-15 (1e-11 turns)
    const double d = (fk[o->K - 1] - fk[0]) / (o->K - 1);
    double dev = 0.0;
    for (int k = 0; k < o->K; ++k) dev = std::max(dev, std::fabs(fk[k] - std::fma((double)k, d, fk[0])));
    const bool uni = d != 0.0 && dev <= 1e-12 * std::fabs(fk[0]);
    o->uniform = uni ? 1 : 0;
    o->uniform64 = uni && dev <= 1e-15 * std::fabs(fk[0]) ? 1 : 0;
    o->dfk = uni ? d : 0.0;
  }
  hipError_t e = upload(&o->uvw, desc->uvw_m, 3 * nrows, o->mem);
  if (e == hipSuccess) e = upload(&o->freq, desc->freq_hz, (int64_t)o->K, o->mem);
  if (e == hipSuccess) e = upload(&o->fk, fk.data(), (int64_t)o->Kpad, o->mem);
  bool look;
  {
    std::lock_guard<std::mutex> lk(ctx->mu);
    look = ctx->ant_skies > 0;
  }
  if (e == hipSuccess && look) e = look_for_antennas(o, desc->uvw_m);
  std::lock_guard<std::mutex> lk(ctx->mu);
  // (a first such sky may have come since)
  if (e == hipSuccess && ctx->ant_skies > 0 && !o->ant_looked) e = look_for_antennas(o, desc->uvw_m);
  if (e != hipSuccess) {
    o->mem.release();
    delete o;
    return hip_error(e, "uploading the observation");
  }
  o->id = ++ctx->next_id;
  ctx->obs.insert(o);
  ctx->lib_bytes += o->mem.total;
  *out = o;
  return VP_OK;
}

int vp_destroy_obs(vp_obs *obs) {
  if (!obs) return set_error(VP_EINVAL, "NULL observation");
  vp_ctx *ctx = obs->ctx;
  DeviceGuard g(ctx->device);
  std::lock_guard<std::mutex> lk(ctx->mu);
  if (obs->jobs > 0) return set_error(VP_EBUSY, "observation used by pending jobs");
  drop_derived(ctx, 0, obs->id);
  ctx->obs.erase(obs);
  ctx->lib_bytes -= obs->mem.total;
  obs->mem.release();
  delete obs;
  return VP_OK;
}

// The points from faint to bright, to a quarter of an octave (a counting sort
// on the leading bits; points of one bin keep their order).  The kernels sum
// points in short FP32 groups, on the matrix cores with roundings of ~1.3 units
// of the group's largest term: groups of one brightness keep a bright point's
// rounding off the faint ones' sum (MWA-like points by antenna: 2.1e-7 of the
// result's norm as given), and a point much brighter than all others comes last
// in its group, after which nothing is rounded at its size (first, it costs a
// rounding for each that follows).  FP64 sums stay small for longest, too.
static std::vector<int32_t> by_flux(const double *s, int n) {
  constexpr int kBins = 2048 << 2;  // exponent and two bits of the mantissa
  std::vector<int32_t> at(kBins + 1, 0), ord(n);
  auto bin = [&](int i) {
    uint64_t u;
    std::memcpy(&u, &s[i], 8);
    return (int)((u << 1) >> 51);
  };
  for (int i = 0; i < n; ++i) ++at[bin(i) + 1];
  for (int b = 0; b < kBins; ++b) at[b + 1] += at[b];
  for (int i = 0; i < n; ++i) ord[at[bin(i)]++] = i;
  return ord;
}

int vp_create_sky(vp_ctx *ctx, const vp_sky_desc *d, vp_sky **out) {
  if (!ctx || !d || !out) return set_error(VP_EINVAL, "NULL argument");
  if (d->n_point < 0 || d->n_gauss < 0 || d->n_shp < 0) return set_error(VP_EINVAL, "negative component count");
  if (!(d->nu_ref_hz > 0) || !std::isfinite(d->nu_ref_hz)) return set_error(VP_EINVAL, "nu_ref must be positive");
  const int P = d->n_point, G = d->n_gauss, Sd = d->n_shp;
  if ((int64_t)P + G + Sd > (1 << 28)) return set_error(VP_EINVAL, "too many components");
  if (P > 0 && (!d->p_ra || !d->p_dec || !d->p_sref || !d->p_alpha)) return set_error(VP_EINVAL, "NULL point array");
  if (G > 0 && (!d->g_ra || !d->g_dec || !d->g_sref || !d->g_alpha || !d->g_maj || !d->g_min || !d->g_pa))
    return set_error(VP_EINVAL, "NULL Gaussian array");
  if (Sd > 0 && (!d->s_ra || !d->s_dec || !d->s_sref || !d->s_alpha || !d->s_beta1 || !d->s_beta2 || !d->s_pa ||
                 !d->s_nmax || !d->s_coeff_off || !d->coeffs))
    return set_error(VP_EINVAL, "NULL shapelet array");
  const double *pa[] = {d->p_ra, d->p_dec, d->p_sref, d->p_alpha};
  for (auto p : pa)
    if (P > 0 && !finite_all(p, P)) return set_error(VP_EINVAL, "non-finite point parameter");
  const double *ga[] = {d->g_ra, d->g_dec, d->g_sref, d->g_alpha, d->g_maj, d->g_min, d->g_pa};
  for (auto p : ga)
    if (G > 0 && !finite_all(p, G)) return set_error(VP_EINVAL, "non-finite Gaussian parameter");
  for (int g = 0; g < G; ++g)
    if (d->g_maj[g] < 0 || d->g_min[g] < 0) return set_error(VP_EINVAL, "Gaussian %d has a negative FWHM", g);
  const double *sa[] = {d->s_ra, d->s_dec, d->s_sref, d->s_alpha, d->s_beta1, d->s_beta2, d->s_pa};
  for (auto p : sa)
    if (Sd > 0 && !finite_all(p, Sd)) return set_error(VP_EINVAL, "non-finite shapelet parameter");
  // Shapelet components: one per spectral term of each shapelet (same
  // position and frame; term q's flux carries ln(nu / nu_ref)^q).
  std::vector<int> src;            // shapelet of the description
  std::vector<int32_t> lp;         // its spectral term
  std::vector<const double *> cp;  // its coefficients, packed for order d->s_nmax
  for (int s = 0; s < Sd; ++s) {
    const int N = d->s_nmax[s];
    if (N < 0 || N > VP_NMAX_LIMIT) return set_error(VP_EINVAL, "shapelet %d: nmax %d outside 0..%d", s, N, VP_NMAX_LIMIT);
    if (!(d->s_beta1[s] > 0) || !(d->s_beta2[s] > 0)) return set_error(VP_EINVAL, "shapelet %d: beta must be positive", s);
    if (d->s_coeff_off[s] < 0) return set_error(VP_EINVAL, "shapelet %d: negative coefficient offset", s);
    const int Q = d->s_nterm ? d->s_nterm[s] : 1;
    if (Q < 1 || Q > VP_NTERM_LIMIT)
      return set_error(VP_EINVAL, "shapelet %d: %d spectral terms outside 1..%d", s, Q, VP_NTERM_LIMIT);
    const int64_t cnt = (int64_t)(N + 1) * (N + 2) / 2;
    for (int q = 0; q < Q; ++q) {
      const double *c = d->coeffs + d->s_coeff_off[s] + q * cnt;
      if (!finite_all(c, cnt)) return set_error(VP_EINVAL, "shapelet %d: non-finite coefficient", s);
      src.push_back(s);
      lp.push_back(q);
      cp.push_back(c);
    }
  }
  const int S = (int)src.size();
  if ((int64_t)P + G + S > (1 << 28)) return set_error(VP_EINVAL, "too many components");
  int max_nmax = 0;
  std::vector<int32_t> nmax(S);
  std::vector<int64_t> coff(S);
  int64_t ncoef = 0;
  for (int i = 0; i < S; ++i) {
    const int N = d->s_nmax[src[i]];
    const double *c = cp[i];
    // effective order: the highest n1 + n2 with a non-zero coefficient (orders
    // above it contribute nothing, and the kernels' work follows the order)
    int neff = 0;
    for (int n1 = 0, j = 0; n1 <= N; ++n1)
      for (int n2 = 0; n2 <= N - n1; ++n2, ++j)
        if (c[j] != 0.0) neff = std::max(neff, n1 + n2);
    nmax[i] = neff;
    coff[i] = ncoef;
    ncoef += (int64_t)(neff + 1) * (neff + 2) / 2;
    max_nmax = std::max(max_nmax, neff);
  }
  DeviceGuard g(ctx->device);
  if (!g.ok) return set_error(VP_EDEVICE, "cannot select device");
  vp_sky *k = new vp_sky();
  k->ctx = ctx;
  k->P = P; k->G = G; k->S = S;
  k->nu_ref = d->nu_ref_hz;
  k->max_nmax = max_nmax;
  k->h_nmax = nmax;
  const int J = P + G + S;
  std::vector<double> ra(J), dec(J), sref(J), alpha(J), coeffs(ncoef), b1(S), b2(S), spa(S);
  for (int i = 0; i < P; ++i) {
    k->p_smax = std::max(k->p_smax, std::fabs(d->p_sref[i]));
    k->p_amax = std::max(k->p_amax, std::fabs(d->p_alpha[i]));
    if (d->p_sref[i] < 0) k->p_neg = 1;
  }
  const std::vector<int32_t> ord = by_flux(d->p_sref, P);
  for (int i = 0; i < P; ++i) {
    const int j = ord[i];
    ra[i] = d->p_ra[j]; dec[i] = d->p_dec[j]; sref[i] = d->p_sref[j]; alpha[i] = d->p_alpha[j];
  }
  for (int i = 0; i < G; ++i) { ra[P + i] = d->g_ra[i]; dec[P + i] = d->g_dec[i]; sref[P + i] = d->g_sref[i]; alpha[P + i] = d->g_alpha[i]; }
  if (P + G > 0) {
    auto turn = [](double x) {  // (one turn at most: right ascensions further out only loosen the bound)
      return x - (x > 3.141592653589793 ? 6.283185307179586477 : x < -3.141592653589793 ? -6.283185307179586477 : 0.0);
    };
    double ra_lo = 0, ra_hi = 0, dec_lo = dec[0], dec_hi = dec[0], r2 = 0;
    for (int i = 0; i < P + G; ++i) {
      const double x = turn(ra[i] - ra[0]);
      ra_lo = std::min(ra_lo, x);
      ra_hi = std::max(ra_hi, x);
      dec_lo = std::min(dec_lo, dec[i]);
      dec_hi = std::max(dec_hi, dec[i]);
      k->pg_amax = std::max(k->pg_amax, std::fabs(alpha[i]));
    }
    k->pg_ra = ra[0] + 0.5 * (ra_lo + ra_hi);
    k->pg_dec = 0.5 * (dec_lo + dec_hi);
    // |s - s'|^2 <= (d dec)^2 + cos(dec) cos(dec') (d ra)^2, cos(dec) <= cos(dec') + |d dec|
    const double c = std::fabs(std::cos(k->pg_dec));
    for (int i = 0; i < P + G; ++i) {
      const double da = turn(ra[i] - k->pg_ra), dd = std::fabs(dec[i] - k->pg_dec);
      r2 = std::max(r2, dd * dd + c * (c + dd) * da * da);
    }
    k->pg_reach = std::sqrt(r2);
  }
  bool terms = false;
  for (int i = 0; i < S; ++i) {
    const int s = src[i];
    ra[P + G + i] = d->s_ra[s]; dec[P + G + i] = d->s_dec[s]; sref[P + G + i] = d->s_sref[s]; alpha[P + G + i] = d->s_alpha[s];
    b1[i] = d->s_beta1[s]; b2[i] = d->s_beta2[s]; spa[i] = d->s_pa[s];
    terms = terms || lp[i] > 0;
    // packed n1-major over n1 + n2 <= nmax, re-packed for the effective order
    const int N = d->s_nmax[s], M = nmax[i];
    const double *c = cp[i];
    double *o = coeffs.data() + coff[i];
    for (int n1 = 0; n1 <= M; ++n1)
      for (int n2 = 0; n2 <= M - n1; ++n2)
        *o++ = c[(int64_t)n1 * (N + 1) - (int64_t)n1 * (n1 - 1) / 2 + n2];
  }
  std::vector<int64_t> a32_off(S), c64_off(S), abf_off(S);
  std::vector<int32_t> ld(S);
  int64_t n32 = 0, n64 = 0, nbf = 0;
  for (int s = 0; s < S; ++s) {
    a32_off[s] = n32; n32 += a32_floats(nmax[s]);
    ld[s] = c64_ld(nmax[s]);
    c64_off[s] = n64; n64 += c64_doubles(nmax[s]);
    abf_off[s] = nbf; nbf += abf_elems(nmax[s]);
  }
  int32_t *d_nmax = nullptr;
  int64_t *d_coff = nullptr, *d_a32off = nullptr, *d_c64off = nullptr, *d_abfoff = nullptr;
  int32_t *d_ld = nullptr;
  double *d_coeffs = nullptr;
  float *d_a32 = nullptr;
  double *d_c64 = nullptr;
  uint16_t *d_abf = nullptr;
  hipError_t e = hipSuccess;
  if (e == hipSuccess) e = upload(&k->ra, ra.data(), J, k->mem);
  if (e == hipSuccess) e = upload(&k->dec, dec.data(), J, k->mem);
  if (e == hipSuccess) e = upload(&k->sref, sref.data(), J, k->mem);
  if (e == hipSuccess) e = upload(&k->alpha, alpha.data(), J, k->mem);
  if (e == hipSuccess) e = upload(&k->g_maj, d->g_maj, G, k->mem);
  if (e == hipSuccess) e = upload(&k->g_min, d->g_min, G, k->mem);
  if (e == hipSuccess) e = upload(&k->g_pa, d->g_pa, G, k->mem);
  if (e == hipSuccess) e = upload(&k->s_beta1, b1.data(), S, k->mem);
  if (e == hipSuccess) e = upload(&k->s_beta2, b2.data(), S, k->mem);
  if (e == hipSuccess) e = upload(&k->s_pa, spa.data(), S, k->mem);
  if (e == hipSuccess && terms) e = upload(&k->lpow, lp.data(), S, k->mem);
  if (e == hipSuccess) e = upload(&d_nmax, nmax.data(), S, k->mem);
  if (e == hipSuccess) e = upload(&d_coff, coff.data(), S, k->mem);
  if (e == hipSuccess) e = upload(&d_coeffs, coeffs.data(), ncoef, k->mem);
  if (e == hipSuccess) e = upload(&d_a32off, a32_off.data(), S, k->mem);
  if (e == hipSuccess) e = upload(&d_c64off, c64_off.data(), S, k->mem);
  if (e == hipSuccess) e = upload(&d_abfoff, abf_off.data(), S, k->mem);
  if (e == hipSuccess) e = upload(&d_ld, ld.data(), S, k->mem);
  if (e == hipSuccess && n32 > 0) e = k->mem.alloc((void **)&d_a32, sizeof(float) * n32);
  if (e == hipSuccess && n64 > 0) e = k->mem.alloc((void **)&d_c64, sizeof(double) * n64);
  if (e == hipSuccess && nbf > 0) e = k->mem.alloc((void **)&d_abf, sizeof(uint16_t) * nbf);
  if (e == hipSuccess && S > 0) {
    TileBuildArgs ta;
    ta.S = S; ta.nmax = d_nmax; ta.coeff_off = d_coff; ta.coeffs = d_coeffs;
    ta.a32 = d_a32; ta.a32_off = d_a32off; ta.c64 = d_c64; ta.c64_off = d_c64off; ta.c64_ld = d_ld;
    ta.abf = d_abf; ta.abf_off = d_abfoff;
    e = launch_tiles_build(ta, max_nmax, nullptr);
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
  }
  if (e != hipSuccess) {
    k->mem.release();
    delete k;
    return hip_error(e, "uploading the sky model");
  }
  k->tiles.a32 = d_a32; k->tiles.a32_off = d_a32off;
  k->tiles.c64 = d_c64; k->tiles.c64_off = d_c64off; k->tiles.c64_ld = d_ld;
  k->tiles.abf = d_abf; k->tiles.abf_off = d_abfoff;
  k->tiles.nmax = d_nmax;
  std::lock_guard<std::mutex> lk(ctx->mu);
  if (P >= kAntMinPoints) {
    for (vp_obs *o : ctx->obs) {
      if (o->ant_looked) continue;
      const size_t before = o->mem.total;
      e = look_for_antennas(o, nullptr);
      ctx->lib_bytes += o->mem.total - before;
      if (e == hipErrorOutOfMemory) {  // (the observation does without them)
        (void)hipGetLastError();
        e = hipSuccess;
      }
      if (e != hipSuccess) {
        k->mem.release();
        delete k;
        return hip_error(e, "looking for the antennas of an observation");
      }
    }
    ++ctx->ant_skies;
  }
  k->id = ++ctx->next_id;
  ctx->skies.insert(k);
  ctx->lib_bytes += k->mem.total;
  *out = k;
  return VP_OK;
}

int vp_destroy_sky(vp_sky *sky) {
  if (!sky) return set_error(VP_EINVAL, "NULL sky");
  vp_ctx *ctx = sky->ctx;
  DeviceGuard g(ctx->device);
  std::lock_guard<std::mutex> lk(ctx->mu);
  if (sky->jobs > 0) return set_error(VP_EBUSY, "sky used by pending jobs");
  drop_derived(ctx, sky->id, 0);
  ctx->skies.erase(sky);
  if (sky->P >= kAntMinPoints) --ctx->ant_skies;
  ctx->lib_bytes -= sky->mem.total;
  sky->mem.release();
  delete sky;
  return VP_OK;
}

int vp_predict(vp_ctx *ctx, const vp_sky *sky, const vp_obs *obs, int precision, int dtype, void *vis_dev,
               void *hip_stream) {
  TraceRange tr("vp_predict");
  int rc = check_call(ctx, sky, obs, precision, dtype, vis_dev);
  if (rc != VP_OK) return rc;
  DeviceGuard g(ctx->device);
  if (!g.ok) return set_error(VP_EDEVICE, "cannot select device");
  return run_tiles(ctx, sky, obs, precision, dtype, vis_dev, 0, (hipStream_t)hip_stream);
}

int vp_predict_noalloc(vp_ctx *ctx, const vp_sky *sky, const vp_obs *obs, int precision, int dtype, void *vis_dev,
                       void *hip_stream) {
  TraceRange tr("vp_predict_noalloc");
  int rc = check_call(ctx, sky, obs, precision, dtype, vis_dev);
  if (rc != VP_OK) return rc;
  if (precision == VP_PREC_LUT)
    return set_error(VP_EINVAL, "vp_predict_noalloc: the lookup-table variant needs a per-context table");
  // the pair's tables, laid out in the device's scratch array (256-byte aligned parts)
  const int J = sky->P + sky->G + sky->S;
  const uint64_t Jc = (uint64_t)std::max(J, 1), Gc = (uint64_t)std::max(sky->G, 1);
  const uint64_t Sc = (uint64_t)std::max(sky->S, 1), Kp = (uint64_t)obs->Kpad;
  auto up = [](uint64_t b) { return (b + 255) & ~(uint64_t)255; };
  const uint64_t o_gq = up(sizeof(double4) * Jc);
  const uint64_t o_sf = o_gq + up(sizeof(double4) * Gc);
  const uint64_t o_f32 = o_sf + up(sizeof(double) * 12 * Sc);
  const uint64_t o_f64 = o_f32 + up(sizeof(float) * Jc * Kp);
  const uint64_t need = o_f64 + up(sizeof(double) * Jc * Kp);
  if (need > kNoAllocScratchBytes)
    return set_error(VP_EINVAL,
                     "vp_predict_noalloc: %d components x %d padded channels need %llu bytes of tables; "
                     "the scratch holds %llu",
                     J, obs->Kpad, (unsigned long long)need, (unsigned long long)kNoAllocScratchBytes);
  DeviceGuard g(ctx->device);
  if (!g.ok) return set_error(VP_EDEVICE, "cannot select device %d", ctx->device);
  char *base = (char *)noalloc_scratch(ctx->device);
  if (!base) return set_error(VP_EDEVICE, "no scratch address for device %d", ctx->device);
  Derived d{};
  d.pos = (double4 *)base;
  d.gq = (double4 *)(base + o_gq);
  d.sframe = (double *)(base + o_sf);
  d.flux32 = (float *)(base + o_f32);
  d.flux64 = (double *)(base + o_f64);
  char *part = base + kNoAllocScratchBytes + kNoAllocAmpBytes;
  const int path = table_path(precision);
  for (int i = path; path >= 0 && i < kPlans; i += 2) {
    d.plan[i] = node_plan(sky, obs, i);
    if (nflux_bytes(sky, d.plan[i], i) > kNoAllocNfluxBytes) d.plan[i].M = 0;
    d.interp[i] = (double *)(part + i / 2 * (kNoAllocNodeBytes / 2));
    if (i >= 2) d.nflux[i - 2] = (double *)(part + kNoAllocNodeBytes);
  }
  if (path == 0 && use_ant(sky, obs, precision, dtype, d.plan[2]) && ant_amp_bytes(sky, obs) <= kNoAllocAmpBytes)
    place_amp(d, base + kNoAllocScratchBytes, sky, obs);
  const hipStream_t stream = (hipStream_t)hip_stream;
  // every entry the tile kernels read is written here first (the flux table
  // includes its zero padding), so nothing is cleared
  hipError_t e = launch_derive(make_derive_args(sky, obs, d), stream);
  if (e == hipSuccess) e = launch_flux(make_flux_args(sky, obs, d), stream);
  if (e == hipSuccess) e = build_amp(sky, obs, d, stream);
  if (e != hipSuccess) return hip_error(e, "building the tables in the scratch array");
  const SumsSpace sums = {(double2 *)(part + kNoAllocNodeBytes + kNoAllocNfluxBytes), kSumsMin};
  return launch_passes(nullptr, sky, obs, precision, dtype, vis_dev, 0, stream, d, nullptr, sums);
}

int vp_subtract(vp_ctx *ctx, const vp_sky *sky, const vp_obs *obs, int precision, int dtype, void *data_dev,
                void *hip_stream) {
  TraceRange tr("vp_subtract");
  int rc = check_call(ctx, sky, obs, precision, dtype, data_dev);
  if (rc != VP_OK) return rc;
  DeviceGuard g(ctx->device);
  if (!g.ok) return set_error(VP_EDEVICE, "cannot select device");
  return run_tiles(ctx, sky, obs, precision, dtype, data_dev, 1, (hipStream_t)hip_stream);
}

int vp_profile(vp_ctx *ctx, int enable) {
  if (!ctx) return set_error(VP_EINVAL, "NULL context");
  ctx->profile = enable != 0;
  return VP_OK;
}

int vp_profile_read(vp_ctx *ctx, int64_t *counts, double *total_ms) {
  if (!ctx || !counts || !total_ms) return set_error(VP_EINVAL, "NULL argument");
  DeviceGuard g(ctx->device);
  std::vector<ProfRecord> recs;
  {
    std::lock_guard<std::mutex> lk(ctx->prof_mu);
    recs.swap(ctx->prof_pending);
  }
  int64_t c[kProfClasses] = {0, 0, 0, 0};
  double t[kProfClasses] = {0, 0, 0, 0};
  int rc = VP_OK;
  for (auto &r : recs) {
    float ms = 0.f;
    hipError_t e = hipEventSynchronize(r.e1);
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, r.e0, r.e1);
    if (e != hipSuccess && rc == VP_OK) rc = hip_error(e, "reading kernel timings");
    if (e == hipSuccess && r.kind >= 0 && r.kind < kProfClasses) {
      c[r.kind] += 1;
      t[r.kind] += ms;
    }
    (void)hipEventDestroy(r.e0);
    (void)hipEventDestroy(r.e1);
  }
  if (rc != VP_OK) return rc;
  for (int i = 0; i < kProfClasses; ++i) {
    counts[i] = c[i];
    total_ms[i] = t[i];
  }
  return VP_OK;
}

}  // extern "C"
