// Pairing of the target layers of the mid-tile-barrier k-split kernel (host
// only, plain C++).
#pragma once

#include <stdint.h>

namespace kvx {

// Order in which the g_n <= 64 target layers of a group are paired: positions 2 j
// and 2 j + 1 of `order` form pair j.  idx[l * k + i]: the sources of layer l of
// the group.  sh[i][j] below is the number of layer j's sources that layer i also
// lists (the slots of a pair's second layer that read the first layer's).
//
// Each CU keeps its pair for the whole launch, so the pairs that share nothing
// set the time: match as many layers as possible to a partner that shares a
// source.  Min-degree greedy: the unmatched layer with the fewest unmatched
// sharing partners takes the partner that shares the most (then the one with the
// fewest partners left); the rest are paired in order.
//
// A call on an idle GPU waits for this between its first launch and the map
// kernel's, so it works on bit sets of layers: what it visits is the pairs of
// layers that share a source, not all pairs of list entries (64 layers, k = 4, 40
// sources: 54 us that way, 9.5 us this way).
inline void ks2_pair_order(const uint8_t* idx, int k, int g_n, uint8_t* order) {
  uint64_t lists[256];                // layers that list a source
  uint8_t sh[64][64] = {};
  uint64_t near[64] = {};             // layers that share a source with layer i
  for (int e = 0; e < g_n * k; ++e) lists[idx[e]] = 0;
  for (int i = 0; i < g_n; ++i)
    for (int r = 0; r < k; ++r) lists[idx[i * k + r]] |= 1ull << i;
  for (int j = 0; j < g_n; ++j)
    for (int r = 0; r < k; ++r) {
      const uint64_t m = lists[idx[j * k + r]];
      near[j] |= m;
      for (uint64_t b = m; b != 0; b &= b - 1) ++sh[__builtin_ctzll(b)][j];
    }
  uint8_t deg[64];                    // unmatched partners
  for (int i = 0; i < g_n; ++i) {
    near[i] &= ~(1ull << i);
    deg[i] = (uint8_t)__builtin_popcountll(near[i]);
  }
  auto s = [&](int i, int j) { return sh[i][j] > sh[j][i] ? sh[i][j] : sh[j][i]; };
  uint64_t open = g_n == 64 ? ~0ull : (1ull << g_n) - 1;   // unmatched layers
  int n = 0;
  for (;;) {
    int i = -1;
    for (uint64_t b = open; b != 0; b &= b - 1) {
      const int c = __builtin_ctzll(b);
      if (deg[c] > 0 && (i < 0 || deg[c] < deg[i])) i = c;
    }
    if (i < 0) break;
    int j = -1;
    for (uint64_t b = open & near[i]; b != 0; b &= b - 1) {
      const int c = __builtin_ctzll(b);
      if (j < 0 || s(i, c) > s(i, j) || (s(i, c) == s(i, j) && deg[c] < deg[j])) j = c;
    }
    const int a = sh[i][j] >= sh[j][i] ? i : j, b = a == i ? j : i;
    order[n++] = (uint8_t)a;
    order[n++] = (uint8_t)b;
    open &= ~(1ull << i) & ~(1ull << j);
    for (uint64_t m = open & near[i]; m != 0; m &= m - 1) --deg[__builtin_ctzll(m)];
    for (uint64_t m = open & near[j]; m != 0; m &= m - 1) --deg[__builtin_ctzll(m)];
  }
  for (; open != 0; open &= open - 1) order[n++] = (uint8_t)__builtin_ctzll(open);
}

}  // namespace kvx
