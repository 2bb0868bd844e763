// vp_serve.cpp -- continuous batching: vp_submit / vp_poll.
//
// The scheduling policy (FIFO admission by HBM footprint, tickets, the
// scheduler thread) is ServeCore (serve_core.cpp); this file is its device
// side.  An admitted job's kernels -- its tables, when its (sky, observation)
// pair has none yet, then the passes of vp_predict / vp_subtract, by the same
// launch function, so that a job's result is the same alone and in a mix --
// are enqueued at once on one of kServeStreams streams, the one with the
// fewest jobs in flight.  Jobs on different streams share the device: a job's
// last, thinly filled wave of workgroups runs beside the next job's first.
// Two one-thread kernels around the job's own write the device clock and the
// job's sequence number to host-mapped memory, which the scheduler thread
// reads; an event behind them confirms the job's end.
//
// This replaced a persistent kernel per pass that pulled tiles from
// host-published rings.  Its tile functions shared one kernel's registers
// (165 against 122 for the point/Gaussian tile), its phases met at the host
// (tables, point/Gaussian, shapelets: a host round trip and an idle tail of up
// to 100 us each), and it could run nothing but those tiles.
#include <hip/hip_runtime.h>
#include <time.h>

#include <algorithm>
#include <atomic>
#include <cstring>
#include <mutex>
#include <vector>

#include "../../include/vp.h"
#include "serve_core.h"
#include "serve_spans.h"
#include "vp_internal.h"
#include "vp_objects.h"

namespace vp {

static uint64_t node_table_bytes(const vp_sky *sky, const vp_obs *obs) {
  uint64_t b = 0;
  for (int i = 0; i < kPlans; i += 2) {  // (serving is mixed)
    const NodePlan p = node_plan(sky, obs, i);
    b += plan_bytes(obs, p) + nflux_bytes(sky, p, i);
  }
  return b;
}

uint64_t job_footprint(const vp_sky *sky, const vp_obs *obs, int dtype) {
  const uint64_t nvis = (uint64_t)obs->T * obs->B * obs->K;
  const uint64_t J = (uint64_t)sky->P + sky->G + sky->S;
  const uint64_t tables = 32 * (J ? J : 1) + 32 * (sky->G ? sky->G : 1) + 96 * (sky->S ? sky->S : 1) +
                          12 * (J ? J : 1) * (uint64_t)obs->Kpad +
                          node_table_bytes(sky, obs) + (ant_mixed(sky, obs) ? ant_amp_bytes(sky, obs) : 0);
  return nvis * (dtype == VP_C64 ? 8 : 16) + tables;
}

static int check_job(vp_ctx *ctx, const vp_job *job) {
  if (!ctx || !job) return set_error(VP_EINVAL, "NULL context or job");
  if (job->kind != VP_JOB_PREDICT && job->kind != VP_JOB_SUBTRACT)
    return set_error(VP_EINVAL, "unknown job kind %d", job->kind);
  int rc = check_call(ctx, job->sky, job->obs, job->precision, job->dtype, job->vis_dev);
  if (rc != VP_OK) return rc;
  if (job->precision != VP_PREC_MIXED)
    return set_error(VP_EINVAL, "serving runs the mixed-precision path (VP_PREC_MIXED)");
  if (job->sky->max_nmax > kNmaxLimit) return set_error(VP_EINVAL, "shapelet order too large");
  return VP_OK;
}

constexpr int kServeSlots = 1024;  // jobs in flight
constexpr int kServeStreams = 4;   // as many as a process has hardware queues

// What the device tells the host about each slot's job (host-mapped, coherent).
struct ServeHost {
  ServeMark started[kServeSlots], finished[kServeSlots];
};

// What the device side keeps per job.
struct JobExt {
  vp_job job{};
  int slot = -1, stream = 0;
  uint64_t seq = 0;        // the job's sequence number in its slot's marks
  int kernels = 0;         // kernels launched for it
  DerivedEntry *d = nullptr;
  int built = 0;           // what this job enqueued the build of (kBuiltBase, kBuiltPath)
  uint64_t floor = 0;      // SpanUnion's, from its admission
};

static JobExt &ext(CoreJob &j) { return *(JobExt *)j.payload; }

class HipExecutor : public ServeExecutor {
 public:
  vp_ctx *ctx = nullptr;
  ServeHost *H = nullptr;      // host pointer
  ServeHost *H_dev = nullptr;  // the same memory as seen by the device
  std::vector<int> free_slots;
  std::vector<hipEvent_t> done;  // per slot, created at its first use
  uint64_t next_seq = 1;
  hipStream_t streams[kServeStreams] = {};
  int in_flight[kServeStreams] = {};
  double ticks_per_ms = 1e5;

  int init(vp_ctx *c);
  void teardown();
  void stats(uint64_t *n, double *ms);

  void thread_start() override { (void)hipSetDevice(ctx->device); }
  bool has_room(const CoreJob &) override { return !free_slots.empty(); }
  uint64_t evictable_bytes() override { return serve_evictable_bytes(ctx); }
  void evict() override { serve_evict(ctx); }
  int admit(CoreJob &j) override;
  bool poll(CoreJob &j) override;
  int kick() override;
  void idle() override {}
  void abandon(const std::vector<CoreJob *> &running, int rc) override;
  void finished(CoreJob &j) override;
  void retired(CoreJob &j) override;

 private:
  std::mutex stats_mu;     // the two below, read by vp_serve_stats
  uint64_t launches = 0;   // kernels of finished jobs
  SpanUnion spans;         // their device intervals
};

struct Scheduler {
  HipExecutor ex;
  ServeCore *core = nullptr;
};

int HipExecutor::admit(CoreJob &j) {
  JobExt &x = ext(j);
  int si = 0;
  for (int i = 1; i < kServeStreams; ++i)
    if (in_flight[i] < in_flight[si]) si = i;
  hipStream_t st = streams[si];
  TraceRange tr("vp_serve: job");
  DerivedEntry *d = nullptr;
  Derived tables;
  int rc = get_derived(ctx, x.job.sky, x.job.obs, st, x.job.precision, true, &tables, &d, &x.built, &x.kernels);
  if (rc != VP_OK) return rc;
  const int slot = free_slots.back();
  hipError_t e = hipSuccess;
  if (!done[slot]) e = hipEventCreateWithFlags(&done[slot], hipEventDisableTiming);
  x.seq = next_seq++;
  if (e == hipSuccess) e = launch_mark(&H_dev->started[slot], x.seq, st);
  if (e != hipSuccess) {
    rc = hip_error(e, "starting a serving job");
  } else {
    SumsLease lease;
    const uint64_t want = sums_bytes(x.job.sky, x.job.obs, x.job.precision, x.job.dtype, tables);
    const SumsSpace sums = want ? lease.take(ctx->sums, want, st) : SumsSpace{nullptr, 0};
    rc = launch_passes(nullptr, x.job.sky, x.job.obs, x.job.precision, x.job.dtype, x.job.vis_dev,
                       x.job.kind == VP_JOB_SUBTRACT, st, tables, nullptr, sums, &x.kernels);
  }
  if (rc == VP_OK) {
    e = launch_mark(&H_dev->finished[slot], x.seq, st);
    if (e == hipSuccess) e = hipEventRecord(done[slot], st);
    if (e != hipSuccess) rc = hip_error(e, "ending a serving job");
  }
  if (rc != VP_OK) {
    // what was enqueued ends before the caller hears of the failure
    (void)hipStreamSynchronize(st);
    serve_release_derived(ctx, d);
    return rc;
  }
  free_slots.pop_back();
  x.slot = slot;
  x.stream = si;
  x.d = d;
  ++in_flight[si];
  std::lock_guard<std::mutex> lk(stats_mu);
  x.floor = spans.admit();
  return VP_OK;
}

bool HipExecutor::poll(CoreJob &j) {
  JobExt &x = ext(j);
  if (j.t_start == 0 && __atomic_load_n(&H->started[x.slot].seq, __ATOMIC_ACQUIRE) == x.seq) {
    timespec ts;
    clock_gettime(CLOCK_MONOTONIC, &ts);
    j.t_start = (uint64_t)ts.tv_sec * 1000000000ull + (uint64_t)ts.tv_nsec;
  }
  if (__atomic_load_n(&H->finished[x.slot].seq, __ATOMIC_ACQUIRE) != x.seq) return false;
  const hipError_t e = hipEventQuery(done[x.slot]);
  if (e == hipErrorNotReady) return false;
  j.dev_start = __atomic_load_n(&H->started[x.slot].clk, __ATOMIC_RELAXED);
  j.dev_done = __atomic_load_n(&H->finished[x.slot].clk, __ATOMIC_RELAXED);
  j.status = e == hipSuccess ? VP_OK : hip_error(e, "serving job");
  return true;
}

// A device failure: every stream's work is lost with it.
int HipExecutor::kick() {
  for (int i = 0; i < kServeStreams; ++i) {
    if (!in_flight[i]) continue;
    const hipError_t e = hipStreamQuery(streams[i]);
    if (e != hipSuccess && e != hipErrorNotReady) return hip_error(e, "serving streams");
  }
  return VP_OK;
}

void HipExecutor::finished(CoreJob &j) {
  JobExt &x = ext(j);
  {
    std::lock_guard<std::mutex> lk(stats_mu);
    launches += (uint64_t)x.kernels;
    spans.finish(x.floor, j.dev_start, j.dev_done);
  }
  --in_flight[x.stream];
  free_slots.push_back(x.slot);
  serve_release_derived(ctx, x.d);
}

void HipExecutor::retired(CoreJob &j) {
  JobExt *x = (JobExt *)j.payload;
  {
    std::lock_guard<std::mutex> lk(ctx->mu);
    const_cast<vp_sky *>(x->job.sky)->jobs -= 1;
    const_cast<vp_obs *>(x->job.obs)->jobs -= 1;
  }
  delete x;
  j.payload = nullptr;
}

void HipExecutor::stats(uint64_t *n, double *ms) {
  std::lock_guard<std::mutex> lk(stats_mu);
  *n = launches;
  *ms = (double)spans.ticks() / ticks_per_ms;
}

// The device failed under the running jobs: they end with that error.  Their
// streams are drained first, so that nothing still runs into buffers their
// callers may free, and tables they were to build are dropped, since nothing
// says that they were.
void HipExecutor::abandon(const std::vector<CoreJob *> &running, int rc) {
  (void)rc;
  for (hipStream_t s : streams) (void)hipStreamSynchronize(s);
  for (CoreJob *j : running)
    if (!ext(*j).built) serve_release_derived(ctx, ext(*j).d);
  for (CoreJob *j : running)
    if (ext(*j).built) serve_abandon_derived(ctx, ext(*j).d, ext(*j).built);
  for (CoreJob *j : running) {
    free_slots.push_back(ext(*j).slot);
    --in_flight[ext(*j).stream];
    std::lock_guard<std::mutex> lk(stats_mu);
    spans.drop(ext(*j).floor);
  }
}

int HipExecutor::init(vp_ctx *c) {
  ctx = c;
  DeviceGuard g(ctx->device);
  hipError_t e = hipHostMalloc((void **)&H, sizeof(ServeHost), hipHostMallocMapped | hipHostMallocCoherent);
  if (e == hipSuccess) {
    std::memset(H, 0, sizeof(ServeHost));
    e = hipHostGetDevicePointer((void **)&H_dev, H, 0);
  }
  for (int i = 0; i < kServeStreams && e == hipSuccess; ++i)
    e = hipStreamCreateWithFlags(&streams[i], hipStreamNonBlocking);
  int rate_khz = 0;
  if (e == hipSuccess) e = hipDeviceGetAttribute(&rate_khz, hipDeviceAttributeWallClockRate, ctx->device);
  if (e != hipSuccess) {
    int rc = hip_error(e, "starting the serving scheduler");
    teardown();
    return rc;
  }
  if (rate_khz > 0) ticks_per_ms = rate_khz;
  done.assign(kServeSlots, nullptr);
  for (int i = kServeSlots - 1; i >= 0; --i) free_slots.push_back(i);
  return VP_OK;
}

void HipExecutor::teardown() {
  DeviceGuard g(ctx->device);
  for (hipStream_t &s : streams) {
    if (!s) continue;
    (void)hipStreamSynchronize(s);
    (void)hipStreamDestroy(s);
    s = nullptr;
  }
  for (hipEvent_t &e : done)
    if (e) (void)hipEventDestroy(e);
  done.clear();
  if (H) (void)hipHostFree(H);
  H = H_dev = nullptr;
}

bool serve_pending(vp_ctx *ctx) {
  Scheduler *s = ctx->sched.load(std::memory_order_acquire);
  return s && s->core->pending();
}

void serve_shutdown(vp_ctx *ctx) {
  Scheduler *s = ctx->sched.exchange(nullptr, std::memory_order_acq_rel);
  if (!s) return;
  // not under ctx->mu: the scheduler thread takes it while retiring jobs
  delete s->core;  // drains (nothing is pending here) and stops the thread
  s->ex.teardown();
  delete s;
}

}  // namespace vp

using namespace vp;

extern "C" {

int vp_job_footprint(vp_ctx *ctx, const vp_job *job, uint64_t *bytes) {
  if (!bytes) return set_error(VP_EINVAL, "NULL out");
  if (!ctx || !job || !job->sky || !job->obs) return set_error(VP_EINVAL, "NULL context, job, sky or observation");
  if (job->dtype != VP_C128 && job->dtype != VP_C64) return set_error(VP_EINVAL, "unknown dtype %d", job->dtype);
  *bytes = job_footprint(job->sky, job->obs, job->dtype);
  return VP_OK;
}

int vp_submit(vp_ctx *ctx, const vp_job *job, uint64_t *ticket) {
  TraceRange tr("vp_submit");
  if (!ticket) return set_error(VP_EINVAL, "NULL ticket");
  int rc = check_job(ctx, job);
  if (rc != VP_OK) return rc;
  const uint64_t fp = job_footprint(job->sky, job->obs, job->dtype);
  if (fp > ctx->budget)
    return set_error(VP_ECAPACITY, "job footprint %llu bytes exceeds the HBM budget %llu", (unsigned long long)fp,
                     (unsigned long long)ctx->budget);
  Scheduler *s = nullptr;
  {
    std::lock_guard<std::mutex> lk(ctx->mu);
    s = ctx->sched.load(std::memory_order_relaxed);
    if (!s) {
      Scheduler *n = new Scheduler();
      rc = n->ex.init(ctx);
      if (rc != VP_OK) {
        delete n;
        return rc;
      }
      n->core = new ServeCore(&n->ex, ctx->budget);
      ctx->sched.store(n, std::memory_order_release);
      s = n;
    }
  }
  JobExt *x = new JobExt();
  x->job = *job;
  {
    // the job holds its sky and observation from here until it retires
    std::lock_guard<std::mutex> lk(ctx->mu);
    const_cast<vp_sky *>(job->sky)->jobs += 1;
    const_cast<vp_obs *>(job->obs)->jobs += 1;
  }
  if (x->job.t_arrival_ns == 0) {
    timespec ts;
    clock_gettime(CLOCK_MONOTONIC, &ts);
    x->job.t_arrival_ns = (uint64_t)ts.tv_sec * 1000000000ull + (uint64_t)ts.tv_nsec;
  }
  CoreJob *j = new CoreJob();
  j->footprint = fp;
  j->payload = x;
  rc = s->core->submit(j, ticket);
  if (rc != VP_OK) {  // not reached: the footprint was checked above
    {
      std::lock_guard<std::mutex> lk(ctx->mu);
      const_cast<vp_sky *>(job->sky)->jobs -= 1;
      const_cast<vp_obs *>(job->obs)->jobs -= 1;
    }
    delete x;
    delete j;
    return set_error(rc, "job refused by the scheduler");
  }
  return VP_OK;
}

int vp_poll(vp_ctx *ctx, uint64_t ticket, vp_job_result *res) {
  if (!ctx || !res) return set_error(VP_EINVAL, "NULL context or result");
  Scheduler *s = ctx->sched.load(std::memory_order_acquire);
  if (!s) return set_error(VP_ENOTFOUND, "unknown ticket %llu", (unsigned long long)ticket);
  CoreJob j;
  const int rc = s->core->poll(ticket, &j);
  if (rc == VP_ENOTFOUND) return set_error(VP_ENOTFOUND, "unknown ticket %llu", (unsigned long long)ticket);
  if (rc != VP_OK) return rc;
  res->status = j.status;
  res->t_submit = j.t_submit;
  res->t_admit = j.t_admit;
  res->t_start = j.t_start;
  res->t_done = j.t_done;
  res->dev_first_tile = j.dev_start;
  res->dev_last_tile = j.dev_done;
  return VP_OK;
}

int vp_serve_stats(vp_ctx *ctx, uint64_t *launches, double *resident_ms) {
  if (!ctx || !launches || !resident_ms) return set_error(VP_EINVAL, "NULL argument");
  Scheduler *s = ctx->sched.load(std::memory_order_acquire);
  if (!s) {
    *launches = 0;
    *resident_ms = 0.0;
    return VP_OK;
  }
  s->ex.stats(launches, resident_ms);
  return VP_OK;
}

}  // extern "C"
