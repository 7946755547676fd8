#include "mlmq_shape.h"

#include <algorithm>
#include <cmath>
#include <vector>

namespace mlmq {

namespace {

constexpr uint32_t kSample = 2048;       // vertices of a search
constexpr uint32_t kSampleEdges = 65536;  // and the edges it looks at, at most
constexpr uint32_t kTable = 8192;         // places of its hash table

// One search: vertices seen and hops taken; 0 hops when it ended early.
double radius_from(int32_t n, const int32_t* off, const int32_t* col, int32_t start, uint32_t want,
                   std::vector<int32_t>* queue, std::vector<int32_t>* table) {
  std::fill(table->begin(), table->end(), -1);
  auto add = [&](int32_t v) {
    uint32_t h = ((uint32_t)v * 2654435761u) >> 19;  // the upper 13 bits
    while ((*table)[h] >= 0 && (*table)[h] != v) h = (h + 1u) & (kTable - 1u);
    if ((*table)[h] == v) return;
    (*table)[h] = v;
    queue->push_back(v);
  };
  queue->clear();
  add(start);
  std::vector<uint32_t> within = {1};  // vertices within so many hops
  uint32_t edges = 0;
  size_t at = 0;
  while (at < queue->size() && queue->size() < want && edges < kSampleEdges) {
    const size_t level = queue->size();
    for (; at < level && queue->size() < want + kSample; ++at)
      for (int32_t e = off[(*queue)[at]]; e < off[(*queue)[at] + 1] && queue->size() < want + kSample; ++e, ++edges)
        add(col[e]);
    within.push_back((uint32_t)queue->size());
  }
  if (queue->size() < want && edges < kSampleEdges) return 0;
  const uint32_t r = (uint32_t)within.size() - 1;
  const double half = 0.5 * r;
  const uint32_t lo = (uint32_t)half;
  const double then = within[lo] + (within[std::min(lo + 1, r)] - (double)within[lo]) * (half - lo);
  const double power = std::max(0.5, std::log2(within[r] / then));
  return r * std::pow((double)n / within[r], 1.0 / power);
}

}  // namespace

uint32_t estimate_radius(int32_t n, const int32_t* off, const int32_t* col) {
  const uint32_t want = std::min(kSample, std::max(64u, (uint32_t)n / 4u));
  std::vector<int32_t> queue, table(kTable);
  queue.reserve(2 * kSample + 1);
  double most = 0;
  // places spread evenly, in an order that any few of them are spread as well
  for (int64_t k = 0, found = 0; k < 16 && found < 4; ++k) {
    const int64_t slot = ((k & 1) << 3) | ((k & 2) << 1) | ((k & 4) >> 1) | ((k & 8) >> 3);
    int32_t start = (int32_t)((2 * slot + 1) * n / 32);
    for (int i = 0; i < 64 && start + 1 < n && off[start + 1] == off[start]; ++i) ++start;
    const double r = radius_from(n, off, col, start, want, &queue, &table);
    if (r > 0) ++found;
    most = std::max(most, r);
  }
  return (uint32_t)std::min(1e9, most);
}

}  // namespace mlmq
