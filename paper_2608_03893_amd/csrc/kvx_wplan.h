// How the W-stationary kernel cuts a call's tokens (host only, plain C++).
#pragma once

#include <stdint.h>

namespace kvx {

// Time of the W-stationary kernel in tiles of 256 tokens when every workgroup
// takes n of them, one fits a CU (256 of them) and staging its map costs about
// one tile's time: the full ranges of all tasks first, then their shorter last
// ranges on the CUs that are free earliest.
inline int64_t w_span(int64_t tasks, int64_t tiles, int64_t n) {
  const int64_t full = tiles / n * tasks, a = n + 1, b = tiles % n + 1;
  const int64_t q = full / 256, r = full % 256;
  if (b == 1) return (q + (r > 0)) * a;
  int64_t t = (full * a + tasks * b + 255) / 256;
  if (t < q * a + b) t = q * a + b;
  if (r > 0 && t < (q + 1) * a) t = (q + 1) * a;
  while ((256 - r) * ((t - q * a) / b) + (t > (q + 1) * a ? r * ((t - (q + 1) * a) / b) : 0) < tasks) ++t;
  return t;
}

// Tokens per workgroup of the W-stationary kernel, at most 16 tiles.  A fixed
// 4096 tokens left 240 CUs idle for one layer of 4096 tokens and 8 heads (a call
// of 190 us; 256 tokens a workgroup: 26.5 us).  Calls that w_span shortens by less
// than a tenth keep 16 tiles (63 layers, one head, k = 1, 15015 tokens: 266 us, with
// 15 tiles, a count of 32 for 34, 281 us).
inline int w_tokens_per_wg(int64_t tasks, int64_t T) {
  const int64_t tiles = (T + 255) / 256;
  const int64_t most = w_span(tasks, tiles, 16);
  int64_t best = 16, span = most;
  for (int64_t n = 15; n >= 1; --n)
    if (const int64_t s = w_span(tasks, tiles, n); s < span) {
      best = n;
      span = s;
    }
  return (int)(10 * span <= 9 * most ? best : 16) * 256;
}

}  // namespace kvx
