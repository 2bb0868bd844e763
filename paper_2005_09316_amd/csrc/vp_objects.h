// vp_objects.h -- host-side objects behind the opaque handles of vp.h.
#pragma once

#include <hip/hip_runtime.h>

#include <map>
#include <atomic>
#include <mutex>
#include <set>
#include <utility>
#include <vector>

#include "vp_internal.h"

struct vp_ctx;

namespace vp {

struct Scheduler;

// Device allocations owned by one object; released together.
struct DeviceMem {
  std::vector<void *> ptrs;
  size_t total = 0;
  hipError_t alloc(void **p, size_t bytes);
  void release();
};

// Device workspace of vp_peel: the model visibilities, the baseline tables,
// the per-cell tables of the gain solve and the gains of every cell.  Calls on one context take turns on it (mu, and the event of the
// previous call's last kernel).
struct PeelWork {
  std::mutex mu;
  DeviceMem mem;
  void *model = nullptr;
  size_t model_bytes = 0;
  int32_t *tab = nullptr;  // ant1 [B], ant2 [B], pair_bl [n_pairs], comp [n_ant]
  size_t tab_n = 0;
  void *ws = nullptr;      // per-cell tables of the gain solve
  size_t ws_bytes = 0;
  void *gw = nullptr;      // gains of every cell, [T][n_ant][K] complex128
  size_t gw_bytes = 0;
  hipEvent_t done = nullptr;
};

// Workspaces for points' sums (SumsSpace) of the calls on one context: up to
// kSlots, each in use by one call's kernels at a time (the event of the last one's
// end orders the next, on whatever stream), freed with the context.
struct SumsPool {
  static constexpr int kSlots = 4;
  struct Slot {
    void *p = nullptr;
    uint64_t bytes = 0;
    hipEvent_t done = nullptr;
    hipStream_t last = nullptr;
    bool used = false;  // done was recorded, on last
  };
  std::mutex mu;
  Slot slot[kSlots];
  int next = 0;
  void release();
};

// One call's hold on a workspace while it enqueues its kernels.
class SumsLease {
 public:
  // Up to `want` bytes, at least kSumsMin of it, for work enqueued on `stream`
  // from here until the lease ends; p null when there is none to have: memory is
  // short, or the stream is being captured (the graph would use the workspace
  // beside later calls).
  SumsSpace take(SumsPool &pool, uint64_t want, hipStream_t stream);
  ~SumsLease();

 private:
  std::unique_lock<std::mutex> lk_;
  SumsPool::Slot *slot_ = nullptr;
  hipStream_t stream_ = nullptr;
};

struct DerivedEntry {
  Derived d{};
  DeviceMem mem;
  hipEvent_t ready = nullptr;  // recorded after the kernels that build the tables
  hipStream_t ready_stream = nullptr;
  // What one path's kernels by nodes and by antenna need beside the components'
  // own: [0] mixed, [1] FP64, each built by the first call that works on it.
  struct Path {
    DeviceMem mem;
    bool built = false;
    hipEvent_t ready = nullptr;  // null: built with the components' own
    hipStream_t ready_stream = nullptr;
  } path[2];
  bool serve_built = false;    // built for serving and not handed to a direct call since (guarded by ctx->mu)
  int serve_users = 0;         // admitted serving jobs that use the tables (guarded by ctx->mu)
};

struct ProfRecord {
  int kind;
  hipEvent_t e0, e1;
};

// Records a pair of events around the kernels launched in its lifetime when
// profiling is enabled on the context.
struct ProfScope {
  vp_ctx *ctx;
  hipStream_t stream;
  int kind;
  bool active = false;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  ProfScope(vp_ctx *c, hipStream_t s, int k);
  void end();
  ~ProfScope();
};

// A named range on the host timeline (roctx) for the lifetime of the guard;
// rocprofv3 --marker-trace records it, and without a profiler it costs a call.
struct TraceRange {
  explicit TraceRange(const char *name);
  ~TraceRange();
  TraceRange(const TraceRange &) = delete;
  TraceRange &operator=(const TraceRange &) = delete;
};

// Selects a HIP device for the lifetime of the guard, restoring the previous one.
struct DeviceGuard {
  int prev = 0;
  bool ok = false;
  explicit DeviceGuard(int dev);
  ~DeviceGuard();
};

int set_error(int code, const char *fmt, ...);
int hip_error(hipError_t e, const char *what);
int run_tiles(vp_ctx *ctx, const struct ::vp_sky *sky, const struct ::vp_obs *obs, int precision, int dtype,
              void *vis, int subtract, hipStream_t stream, bool nodes = true);
int check_call(vp_ctx *ctx, const struct ::vp_sky *sky, const struct ::vp_obs *obs, int precision, int dtype,
               void *vis);
// Launch the passes over the visibility tiles with the pair's tables `d`.
// prof: the context whose profiling records the launches, or null; sums: the
// workspace that sums_bytes asks for, or {null, 0} (the points then go with the
// Gaussians); *kernels (when given) grows by the number of kernels launched;
// nodes = false (vp_peel except in FP64): summed channel by channel (of the
// lookup-table path, whose points and Gaussians are FP64, only the shapelets).
int launch_passes(vp_ctx *prof, const struct ::vp_sky *sky, const struct ::vp_obs *obs, int precision, int dtype,
                  void *vis, int subtract, hipStream_t stream, const Derived &d, const float *lut, SumsSpace sums,
                  int *kernels = nullptr, bool nodes = true);
// Bytes of workspace with which a call takes one pass over its sums (fewer:
// several), 0 when it needs none.
uint64_t sums_bytes(const struct ::vp_sky *sky, const struct ::vp_obs *obs, int precision, int dtype, const Derived &d,
                    bool nodes = true);
// Per-(sky, observation) tables, built on `stream` at first use and cached, those
// by nodes and by antenna for the path that `precision` works on; later callers on
// other streams wait for the build.  *out: the tables as this call may use them
// (without a path's, which a capture or short memory kept from being built, the
// call goes by channels and rows).  serving: the caller is an admitted job, counted
// in the entry's users until serve_release_derived.  *built (when given): what this
// call enqueued the build of, *kernels: in how many kernels.
constexpr int kBuiltBase = 1, kBuiltPath = 2;
int get_derived(vp_ctx *ctx, const struct ::vp_sky *sky, const struct ::vp_obs *obs, hipStream_t stream, int precision,
                bool serving, Derived *out, DerivedEntry **entry = nullptr, int *built = nullptr, int *kernels = nullptr);
// A serving job is done with the pair's tables.
void serve_release_derived(vp_ctx *ctx, DerivedEntry *d);
// The tables a serving job was to build may never have been built (its work
// was abandoned): drop them, so that no later call finds them ready.
void serve_abandon_derived(vp_ctx *ctx, DerivedEntry *d, int built);
// Bytes of tables that serving jobs built and no admitted job or direct call
// uses, and their release (hipFree: waits for the device).
uint64_t serve_evictable_bytes(vp_ctx *ctx);
void serve_evict(vp_ctx *ctx);
// The pair's plans by nodes (Derived::plan; M = 0: none).
NodePlan node_plan(const struct ::vp_sky *sky, const struct ::vp_obs *obs, int i);
// Bytes of a plan's tables: nodes and interpolation, and the fluxes at the nodes.
uint64_t plan_bytes(const struct ::vp_obs *obs, const NodePlan &p);
uint64_t nflux_bytes(const struct ::vp_sky *sky, const NodePlan &p, int i);
// Whether the pair's points may be taken by antenna on the mixed paths, were it the
// faster.  Its tables then hold the amplitudes, Jp x Kpad of them, and two doubles a
// channel beside them.
bool ant_pair(const struct ::vp_sky *sky, const struct ::vp_obs *obs);
// Whether a mixed call on the pair may do so.
bool ant_mixed(const struct ::vp_sky *sky, const struct ::vp_obs *obs);
int ant_jp(const struct ::vp_sky *sky);
uint64_t ant_amp_bytes(const struct ::vp_sky *sky, const struct ::vp_obs *obs);
DeriveArgs make_derive_args(const struct ::vp_sky *sky, const struct ::vp_obs *obs, const Derived &d);
FluxArgs make_flux_args(const struct ::vp_sky *sky, const struct ::vp_obs *obs, const Derived &d);
void drop_derived(vp_ctx *ctx, uint64_t sky_id, uint64_t obs_id);
void drop_all_derived(vp_ctx *ctx);

// serving hooks (vp_serve.cpp)
uint64_t job_footprint(const struct ::vp_sky *sky, const struct ::vp_obs *obs, int dtype);
bool serve_pending(vp_ctx *ctx);
void serve_shutdown(vp_ctx *ctx);

}  // namespace vp

struct vp_obs {
  vp_ctx *ctx = nullptr;
  uint64_t id = 0;
  int T = 0, B = 0, K = 0, Kpad = 0;
  double ra0 = 0, dec0 = 0;
  int sign = -1;
  double beam_fwhm = 0, beam_nu_ref = 0;
  double *uvw = nullptr;  // device [T*B][3]
  double *freq = nullptr; // device [K]
  double *fk = nullptr;   // device [Kpad], nu/c
  double dfk = 0;         // channel step of nu/c when uniform
  int uniform = 0;        // channels uniformly spaced (to 1e-12 of nu/c)
  int uniform64 = 0;      // ... to 1e-15 of nu/c (enough for the FP64 path)
  std::vector<double> h_freq;
  double f_lo = 0, f_hi = 0;  // lowest and highest channel frequency, Hz
  double b_max = 0;           // longest row, metres
  // antennas behind the baselines (ant_layout.h); ant_n 0: none found.  They are
  // looked for once the context holds a sky that may use them (ant_looked, under
  // the context's lock), and read only for such skies.
  bool ant_looked = false;
  int ant_n = 0, ant_npad = 0, ant_nmac = 0, ant_max_sup = 0, ant_kpack = 1;
  double ant_dev = 0;           // their largest disagreement with a row, in turns at the highest frequency
  double ant_reach = 0;         // largest antenna coordinate (a sum of magnitudes), in wavelengths at the highest frequency
  double *ant_xyz = nullptr, *ant_lo = nullptr;  // device [T][npad][3], [T][npad][3]
  int32_t *ant_rowmap = nullptr;  // device [npad][npad]
  vp::AntMacro *ant_mac = nullptr;
  int jobs = 0;           // pending serving jobs using it (guarded by ctx->mu)
  vp::DeviceMem mem;
};

struct vp_sky {
  vp_ctx *ctx = nullptr;
  uint64_t id = 0;
  int P = 0, G = 0, S = 0;
  double nu_ref = 0;
  int max_nmax = 0;
  std::vector<int32_t> h_nmax;
  double p_smax = 0, p_amax = 0;  // points: largest |S_ref| and largest |spectral index|
  int p_neg = 0;                  // points: 1 if an S_ref is negative
  // points and Gaussians: a direction in their middle, a bound on their distance
  // from it (of unit vectors), and the largest |spectral index|
  double pg_ra = 0, pg_dec = 0, pg_reach = 0, pg_amax = 0;
  double *ra = nullptr, *dec = nullptr, *sref = nullptr, *alpha = nullptr;  // device [J]
  double *g_maj = nullptr, *g_min = nullptr, *g_pa = nullptr;               // device [G]
  double *s_beta1 = nullptr, *s_beta2 = nullptr, *s_pa = nullptr;          // device [S]
  int32_t *lpow = nullptr;  // device [S]: spectral term of each shapelet component, or null (all 0)
  vp::ShpTiles tiles;
  int jobs = 0;
  vp::DeviceMem mem;
};

struct vp_ctx {
  int device = 0;
  uint64_t budget = 0;
  std::mutex mu;  // guards the object sets, the derived cache and job counts
  uint64_t next_id = 0;
  std::set<vp_obs *> obs;
  std::set<vp_sky *> skies;
  int ant_skies = 0;  // of these, skies with kAntMinPoints points or more
  std::map<std::pair<uint64_t, uint64_t>, vp::DerivedEntry *> derived;
  uint64_t lib_bytes = 0;
  bool profile = false;
  std::mutex prof_mu;
  std::vector<vp::ProfRecord> prof_pending;
  // created by the first vp_submit (under mu), read by vp_poll without it
  std::atomic<vp::Scheduler *> sched{nullptr};
  vp::PeelWork *peel = nullptr;
  vp::SumsPool sums;
  float *lut = nullptr;    // basis table of VP_PREC_LUT, built at its first use (guarded by mu)
  vp::DeviceMem lut_mem;
};
