// Which memory the idle compute units of an attention launch read ahead.  Plain C++ without HIP: a test on the CPU checks
// the rule.
#pragma once
#include <stdint.h>

namespace et {

// Memory that the launches behind this one read and that is in no cache yet (weights), in the order of its use: where an
// attention launch leaves compute units idle, further workgroups of it read these ranges once, so that they come from the
// last-level cache then.
struct WarmRanges {
  static constexpr int kMax = 4;
  const void *ptr[kMax] = {};
  uint32_t bytes[kMax] = {};               // multiples of 16
};

// What `idle` units read of `all` beside an attention whose workgroups walk `tiles` key tiles one after the other.
// A unit fetches some 40 KB per microsecond and the launch ends when the last one is done: all of the weights where a unit's share
// takes about as long as the attention, 512 KB beside one tile and 768 KB beside three; else 192 KB each, the first weights to be
// used.  Measured, us per block, none / all / 192 KB (width 1152 unless said; share of a unit when all is read): 1 x 729
// 72.0 / 67.0 / 70.4 (465 KB), 4 x 169 67.2 / 65.4 / 65.7 (465), 12 heads of 96 6 x 361 123.9 / 121.3 / 122.7 (743 KB, three
// tiles); one tile: 6 x 100, 18 heads 67.5 / 70.4 / 66.6 (743 KB), 2 x 196 at a width of 1536 79.9 / 83.3 / 78.6 (864), 5 x 169 68.8
// / 90.1 / 68.4 (1858); three: 5 x 361 104.5 / 122.7 / 104.5 (1858).  Where the encoder's weights fit in the last-level
// cache, nothing is gained or lost (12 blocks at a width of 768, 1 to 4 x 196: 43.1 / 42.6, 45.3 / 45.4, 47.2 / 47.1, 50.0 / 49.7).
inline WarmRanges read_ahead_of(const WarmRanges &all, int idle, int tiles) {
  WarmRanges w;
  if (idle < 16) return w;
  uint64_t total = 0;
  for (int i = 0; i < WarmRanges::kMax; ++i) total += all.bytes[i];
  const uint64_t share = (uint64_t)idle * 1024;
  uint64_t left = total <= share * (tiles >= 3 ? 768 : 512) ? total : share * 192;
  for (int i = 0; i < WarmRanges::kMax; ++i) {
    w.ptr[i] = all.ptr[i];
    w.bytes[i] = all.bytes[i] < left ? all.bytes[i] : (uint32_t)left;
    left -= w.bytes[i];
  }
  return w;
}

}  // namespace et
