// Placement of a model's activations in one arena by lifetime (host only, internal to
// the library).
#pragma once
#include <algorithm>
#include <cstddef>
#include <vector>

namespace rafiki {

// First fit over the free ranges, lowest offset first; sizes rounded to 256 bytes.
struct FreeList {
  struct B { size_t off, size; };
  std::vector<B> free;
  size_t top = 0;
  static size_t rounded(size_t n) { return (std::max<size_t>(n, 1) + 255) / 256 * 256; }
  size_t alloc(size_t n) {
    n = rounded(n);
    for (size_t i = 0; i < free.size(); ++i) {
      if (free[i].size >= n) {
        size_t off = free[i].off;
        free[i].off += n;
        free[i].size -= n;
        if (free[i].size == 0) free.erase(free.begin() + i);
        return off;
      }
    }
    size_t off = top;
    top += n;
    return off;
  }
  void release(size_t off, size_t n) {
    free.push_back({off, rounded(n)});
    std::sort(free.begin(), free.end(), [](const B& a, const B& b) { return a.off < b.off; });
    std::vector<B> merged;
    for (auto& b : free) {
      if (!merged.empty() && merged.back().off + merged.back().size == b.off) merged.back().size += b.size;
      else merged.push_back(b);
    }
    free.swap(merged);
  }
};

// One step of a forward pass: reads tensors in[0] and in[1] (negative: not in the arena),
// writes tensor out, and uses scratch while it runs.
struct ArenaStep {
  int in[2] = {-1, -1};
  int out = -1;
  size_t out_bytes = 0;       // 0: the output lies elsewhere
  size_t scratch_bytes = 0;
  int last = -1;              // last step of the launch that may run this step with later ones
};

struct ArenaPlan {
  std::vector<size_t> off;        // per tensor
  std::vector<size_t> scratch;    // per step
  size_t bytes = 0;
};

// A tensor lives from the step that writes it to the last step of any launch that reads or
// writes it: a launch of several steps reads its inputs while it writes each of its outputs,
// and may do so at any of its steps.  After that its range is free.
inline ArenaPlan plan_arena(const std::vector<ArenaStep>& steps, int tensors) {
  ArenaPlan plan;
  plan.off.assign(tensors, 0);
  plan.scratch.assign(steps.size(), 0);
  std::vector<int> until(tensors, -1);
  std::vector<size_t> size(tensors, 0);
  for (size_t i = 0; i < steps.size(); ++i)
    for (int t : {steps[i].in[0], steps[i].in[1], steps[i].out})
      if (t >= 0) until[t] = std::max({until[t], (int)i, steps[i].last});
  std::vector<std::vector<int>> ends(steps.size());
  for (int t = 0; t < tensors; ++t)
    if (until[t] >= 0) ends[until[t]].push_back(t);
  FreeList fl;
  for (size_t i = 0; i < steps.size(); ++i) {
    const ArenaStep& s = steps[i];
    if (s.scratch_bytes) plan.scratch[i] = fl.alloc(s.scratch_bytes);
    if (s.out_bytes) {
      plan.off[s.out] = fl.alloc(s.out_bytes);
      size[s.out] = s.out_bytes;
    }
    if (s.scratch_bytes) fl.release(plan.scratch[i], s.scratch_bytes);
    for (int t : ends[i])
      if (size[t]) fl.release(plan.off[t], size[t]);
  }
  plan.bytes = fl.top;
  return plan;
}

}  // namespace rafiki
