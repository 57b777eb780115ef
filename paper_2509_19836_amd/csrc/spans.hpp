// Which buffers of a call's steps may share memory.  Host only.
#pragma once
#include <algorithm>
#include <cstdint>
#include <vector>

namespace burst {

// Addresses from the first to the last element (empty: begin == end).  Overlapping spans may still name different elements.
struct Span {
  uintptr_t begin, end;
};
inline bool overlap(const Span& a, const Span& b) { return a.begin < b.end && b.begin < a.end; }

// A span that a step reads or writes.  What all steps write together (dQ) is a step of its own.
struct Use {
  Span span;
  int step;
  bool written;
};

// Whether no step writes what another one reads or writes.  In order of their first address, a span meets an earlier one of
// another step exactly if the furthest end of those lies behind its beginning.  (A backward call of 1024 steps up to its first launch,
// all pairs compared: 16.7 ms; so: 0.6-0.9.)
inline bool steps_apart(std::vector<Use>& uses) {
  struct Furthest {
    int step = INT32_MIN;
    uintptr_t end = 0, other = 0;   // of `step`, which reaches furthest, and of the other steps
    void add(const Use& u) {
      if (u.step == step) {
        end = std::max(end, u.span.end);
      } else if (u.span.end > end) {
        other = end;
        end = u.span.end;
        step = u.step;
      } else {
        other = std::max(other, u.span.end);
      }
    }
    uintptr_t without(int s) const { return s == step ? other : end; }
  } all, writes;
  std::sort(uses.begin(), uses.end(), [](const Use& a, const Use& b) { return a.span.begin < b.span.begin; });
  for (const Use& u : uses) {
    if (u.span.begin == u.span.end) continue;
    if ((u.written ? all : writes).without(u.step) > u.span.begin) return false;
    all.add(u);
    if (u.written) writes.add(u);
  }
  return true;
}

}  // namespace burst
