// rdx_graphs.hpp -- the captured graphs an engine keeps, by launch shape.
//
// A sequence of windows needs one graph, or two that alternate (an odd number
// of windows per graph: a graph starts at one parity of the step index).  All
// that a sequence needs are at hand before its first replay, so nothing is
// captured, and no capture can fail, between two replays; and a graph is only
// destroyed once every replay has ended.
#pragma once

#include <cstddef>
#include <map>
#include <utility>

namespace rdx {

template <typename Exec>
class GraphCache {
 public:
  typedef std::pair<int, long long> Key;  // windows, everything of the arguments that can change
  static constexpr size_t kMost = 16;     // graphs kept; a sequence needs two at most

  // out[j] = the graph of keys[j].  Where the missing ones do not fit, all
  // graphs are dropped first: idle() returns once no replay is under way,
  // destroy(exec) drops one.  capture(j, &exec) makes that of keys[j]; what it
  // returns other than zero ends the call.
  template <typename Capture, typename Idle, typename Destroy>
  int take(const Key* keys, int n, Exec* out, Capture capture, Idle idle, Destroy destroy) {
    size_t missing = 0;
    for (int j = 0; j < n; ++j) missing += execs_.count(keys[j]) ? 0 : 1;
    if (missing > 0 && execs_.size() + missing > kMost) {
      idle();
      clear(destroy);
    }
    for (int j = 0; j < n; ++j) {
      auto it = execs_.find(keys[j]);
      if (it == execs_.end()) {
        Exec e{};
        const int st = capture(j, &e);
        if (st != 0) return st;
        it = execs_.emplace(keys[j], e).first;
      }
      out[j] = it->second;
    }
    return 0;
  }

  template <typename Destroy>
  void clear(Destroy destroy) {
    for (auto& g : execs_) destroy(g.second);
    execs_.clear();
  }

 private:
  std::map<Key, Exec> execs_;
};

}  // namespace rdx
