/* The tile words of the compaction, on the host: launches without bucket counts between two bucket launches whose epochs
 * are the same, and the second one's words becoming visible in every order. Prints "lookback ok". */
#include <cstdio>

#include "lookback.h"

typedef unsigned long long u64;

int main() {
  using namespace rp;
  const u64 tiles = 7;
  u64 words[kVals] = {};  // one tile's, zero when first used
  const auto store = [&](int k, u64 w) { words[k] = w; };
  u64 launch = 3;
  const u64 again = launch + kEpochs;
  if (launch_epoch(launch * tiles + tiles - 1, tiles) != launch_epoch(again * tiles, tiles)) return 1;
  {
    const long long first[kVals] = {10, 11, 12, 13, 14};
    publish_words(launch_epoch(launch * tiles, tiles), first, store);
  }
  for (++launch; launch < again; ++launch) {
    const long long v[kVals - 1] = {20, 21, 22, 23};
    publish_words(launch_epoch(launch * tiles, tiles), v, store);
  }
  const u64 epoch = launch_epoch(again * tiles, tiles);
  const long long now[kVals] = {30, 31, 32, 33, 34};
  u64 fresh[kVals] = {};
  publish_words(epoch, now, [&](int k, u64 w) { fresh[k] = w; });
  for (unsigned seen = 0; seen < 1u << kVals; ++seen) {  // the words that a waiting tile sees already
    long long got[kVals];
    const bool ok = fetch_words(epoch, got, [&](int k) { return seen >> k & 1u ? fresh[k] : words[k]; });
    if (ok != (seen + 1 == 1u << kVals)) {
      std::printf("words seen %#x: %s\n", seen, ok ? "stale sums accepted" : "sums refused");
      return 1;
    }
    for (int k = 0; ok && k < kVals; ++k)
      if (got[k] != now[k]) return 1;
  }
  std::puts("lookback ok");
  return 0;
}
