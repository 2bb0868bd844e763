// SpanUnion (serve_spans.h) against a count tick by tick: jobs in flight together,
// ending in any order, with the total asked for at any time.  Prints the number of
// wrong answers and the most intervals held.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "../paper_2005_09316_amd/csrc/serve_spans.h"

int main(int argc, char **argv) {
  if (argc != 3) return 2;
  std::mt19937_64 rng(atoi(argv[1]));
  const int jobs = atoi(argv[2]);
  struct Job {
    uint64_t floor, from, to;
  };
  vp::SpanUnion u;
  std::vector<Job> run;
  std::vector<char> covered;
  uint64_t now = 1, count = 0;
  int wrong = 0, done = 0;
  size_t held = 0;
  while (done < jobs) {
    const int what = rng() % 8;
    if (what < 3 && run.size() < 6) {  // admitted: begins a little later
      Job j;
      j.floor = u.admit();
      j.from = now + 1 + rng() % 5;
      j.to = j.from + rng() % 40;
      run.push_back(j);
    } else if (what < 6 && !run.empty()) {  // one of the running jobs has ended: the host sees its clock
      const size_t i = rng() % run.size();
      const Job j = run[i];
      run.erase(run.begin() + i);
      if (rng() % 16 == 0) {
        u.drop(j.floor);
      } else {
        u.finish(j.floor, j.from, j.to);
        if (covered.size() < j.to) covered.resize(j.to, 0);
        for (uint64_t t = j.from; t < j.to; ++t) {
          count += !covered[t];
          covered[t] = 1;
        }
      }
      now = now > j.to ? now : j.to;
      ++done;
    } else if (what == 6) {
      now += rng() % 4;
    } else if (u.ticks() != count) {
      ++wrong;
    }
    held = held > u.held() ? held : u.held();
  }
  if (u.ticks() != count) ++wrong;
  printf("%d %zu\n", wrong, held);
  return 0;
}
