// How a launch's element tiles are dealt to its workgroups (host code; no device calls).
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <vector>

namespace esdg {

// Contiguous tile ranges for G workgroups, range c holding tiles r[c] .. r[c+1]-1 (cum: costs
// summed up to each tile).  A launch of few tiles per workgroup ends with its most loaded one,
// so first comes the smallest possible largest range (by bisection; a greedy fill tests a
// bound), then the ranges lie as near to equal shares as that bound lets them.  (Equal shares
// alone, each rounded up to a whole tile, overload a workgroup by up to a tile: an ensemble of
// 45944 elements, N = 2..4, FP32, 66.2 us a stage, 60.6 so; with fewer tiles than workgroups, one
// each: 6038 elements 15.3 -> 8.5.  Of the ensembles timed one lost: 18198 elements 29.2 -> 30.9.)
inline std::vector<int32_t> split_tiles(const std::vector<long long> &cum, int G) {
  const int n = int(cum.size()) - 1;
  auto past = [&](int from, long long cap) {       // end of the longest range from `from` on
    return int(std::upper_bound(cum.begin() + from, cum.end(), cum[from] + cap) - cum.begin()) - 1;
  };
  long long lo = 0, hi = cum[n];                   // ranges of at most hi exist, of at most lo not
  while (hi - lo > 1) {
    const long long cap = lo + (hi - lo) / 2;
    int t = 0;
    for (int c = 0; c < G && t < n; ++c) {
      const int e = past(t, cap);
      if (e == t) break;
      t = e;
    }
    (t == n ? hi : lo) = cap;
  }
  // first[c]: the first tile that ranges c .. G-1 can start at and still hold all the rest
  std::vector<int32_t> first(G + 1, n), r(G + 1, n);
  for (int c = G - 1; c >= 0; --c) {
    const auto at = std::lower_bound(cum.begin(), cum.begin() + first[c + 1] + 1, cum[first[c + 1]] - hi);
    first[c] = int32_t(at - cum.begin());
  }
  r[0] = 0;
  for (int c = 0; c + 1 < G; ++c) {
    const long long share = (long long)((__int128)cum[n] * (c + 1) / G);
    int near = int(std::lower_bound(cum.begin(), cum.end(), share) - cum.begin());
    if (near > 0 && share - cum[near - 1] < cum[near] - share) --near;
    r[c + 1] = std::min(std::max(near, std::max(first[c + 1], r[c])), past(r[c], hi));
  }
  return r;
}

// The ranges of a launch of `kinds` element kinds on G workgroups, or none (equal numbers of tiles):
// one kind's tiles cost the same, and with a workgroup for every tile there is nothing to split.
inline std::vector<int32_t> tile_ranges(const std::vector<long long> &cum, size_t kinds, int G) {
  if (kinds <= 1 || cum.size() <= size_t(G) + 1) return {};
  return split_tiles(cum, G);
}

}  // namespace esdg
