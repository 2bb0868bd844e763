// serve_submit_test.cpp -- callers of the scheduler while it launches a job: an
// executor whose admit() takes until the test lets it go on.  Built with g++ (also
// with -fsanitize=thread) by test_serve_submit.py; exits non-zero on failure.
#include <stdio.h>

#include <atomic>
#include <chrono>
#include <string>
#include <thread>
#include <vector>

#include "serve_core.h"
#include "vp.h"

using namespace vp;
using Clock = std::chrono::steady_clock;

struct SlowExec : public ServeExecutor {
  std::atomic<int> admitting{0}, let{0};
  std::atomic<bool> gave_up{false};
  int fail = 0;                     // the job (by its number) whose admission fails
  std::vector<std::string> events;  // of the core's thread; read once it has ended
  static int number(const CoreJob &j) { return (int)(intptr_t)j.payload; }
  bool has_room(const CoreJob &) override { return true; }
  uint64_t evictable_bytes() override { return 0; }
  void evict() override {}
  int admit(CoreJob &j) override {
    const int n = number(j);
    admitting = n;
    const auto t0 = Clock::now();
    while (let < n && !gave_up) {
      if (Clock::now() - t0 > std::chrono::seconds(5)) gave_up = true;
      std::this_thread::sleep_for(std::chrono::microseconds(100));
    }
    events.push_back("admit" + std::to_string(n));
    return n == fail ? VP_ENOMEM : VP_OK;
  }
  bool poll(CoreJob &) override { return true; }
  int kick() override { return VP_OK; }
  void idle() override {}
  void abandon(const std::vector<CoreJob *> &, int) override {}
  void finished(CoreJob &j) override { events.push_back("finish" + std::to_string(number(j))); }
  void retired(CoreJob &j) override { events.push_back("retire" + std::to_string(number(j))); }
};

static uint64_t submit(ServeCore &core, int n) {
  CoreJob *j = new CoreJob();
  j->footprint = 10;
  j->payload = (void *)(intptr_t)n;
  uint64_t t = 0;
  if (core.submit(j, &t) != VP_OK) return 0;
  return t;
}

int main() {
  SlowExec ex;
  ex.fail = 2;
  int bad = 0;
  {
    ServeCore core(&ex, 100);
    uint64_t t[4] = {0, submit(core, 1), 0, 0};
    while (ex.admitting < 1) std::this_thread::yield();
    // job 1 is being launched: others are taken, and asked for, all the same
    t[2] = submit(core, 2);
    t[3] = submit(core, 3);
    CoreJob out;
    if (core.poll(t[1], &out) != VP_EAGAIN || core.poll(t[3], &out) != VP_EAGAIN) ++bad;
    if (!core.pending() || core.in_use() != 10) ++bad;
    if (ex.gave_up) ++bad;
    ex.let = 3;
    const int want[4] = {0, VP_OK, VP_ENOMEM, VP_OK};
    for (int n = 1; n <= 3; ++n) {
      while (core.poll(t[n], &out) == VP_EAGAIN) std::this_thread::sleep_for(std::chrono::microseconds(100));
      if (out.status != want[n]) ++bad;
    }
    if (core.in_use() != 0) ++bad;
  }
  // a job that has ended leaves before the next is launched, not after all of them
  const std::vector<std::string> want = {"admit1", "finish1", "retire1", "admit2", "retire2", "admit3", "finish3", "retire3"};
  if (ex.events != want) ++bad;
  for (const std::string &e : ex.events) printf("%s ", e.c_str());
  printf("\n%s\n", bad ? "FAIL" : "PASS");
  return bad != 0;
}
