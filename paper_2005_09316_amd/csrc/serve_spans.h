// serve_spans.h -- how long at least one serving job was on the device, free of
// any device code: the union of the finished jobs' intervals on the device's clock,
// in bounded memory.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <set>
#include <utility>
#include <vector>

namespace vp {

// Jobs are admitted and end in any order.  A job admitted once the host has seen
// the clock at c begins after c: intervals that end before every running job's c
// can meet no later one and are kept as a sum only.
class SpanUnion {
 public:
  // A job is admitted: the clock it begins after, to be handed back at its end.
  uint64_t admit() {
    floors_.insert(seen_);
    return seen_;
  }
  // It ended, having been on the device from `from` to `to`.
  void finish(uint64_t floor, uint64_t from, uint64_t to) {
    drop(floor);
    seen_ = std::max(seen_, to);
    spans_.emplace_back(from, to);
    if (spans_.size() >= 2 * kept_ + 4096) merge();
  }
  // It ended without an interval.
  void drop(uint64_t floor) {
    auto it = floors_.find(floor);
    if (it != floors_.end()) floors_.erase(it);
  }
  // The union's length.
  uint64_t ticks() {
    merge();
    uint64_t t = past_;
    for (const auto &s : spans_) t += s.second - s.first;
    return t;
  }
  size_t held() const { return spans_.size(); }

 private:
  void merge() {
    std::sort(spans_.begin(), spans_.end());
    const uint64_t horizon = floors_.empty() ? seen_ : *floors_.begin();
    std::vector<std::pair<uint64_t, uint64_t>> u;
    for (const auto &s : spans_) {
      if (s.second <= s.first) continue;
      if (!u.empty() && s.first <= u.back().second)
        u.back().second = std::max(u.back().second, s.second);
      else
        u.push_back(s);
    }
    spans_.clear();
    for (const auto &s : u) {
      if (s.second <= horizon)
        past_ += s.second - s.first;
      else
        spans_.push_back(s);
    }
    kept_ = spans_.size();
  }
  std::multiset<uint64_t> floors_;  // of the running jobs
  uint64_t seen_ = 0;               // latest clock the host has seen
  uint64_t past_ = 0;               // length of the intervals that nothing can meet any more
  std::vector<std::pair<uint64_t, uint64_t>> spans_;
  size_t kept_ = 0;                 // disjoint intervals that the last merge kept
};

}  // namespace vp
