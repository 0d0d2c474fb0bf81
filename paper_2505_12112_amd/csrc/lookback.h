// The words that a compaction's tiles publish for each other (see k_compact), without
// any device code, so that a host program can check the protocol.
#pragma once

#ifdef __HIP__
#define RP_HOST_DEVICE __host__ __device__
#else
#define RP_HOST_DEVICE
#endif

namespace rp {

// Per-tile sums carried by the compaction: marked vertices, their out-degrees,
// their in-degrees, marked vertices of the first bitmap, and in the bucket form (NV
// = kVals, else one fewer) their bucket counts.
constexpr int kVals = 5;

// Published tile sums: each 64-bit word holds the launch epoch (1..65535) above a
// 48-bit value, so a word is valid on its own, in whatever order a tile's words become
// visible. Epochs come round again every 65535 launches, so words of earlier launches
// are never mistaken for current ones only because every launch rewrites all kVals
// words of its tiles, those it has no sum for (the bucket counts outside the bucket
// form) as zeros.
constexpr int kEpochShift = 48;
constexpr unsigned long long kEpochs = 65535;
constexpr unsigned long long kValueMask = (1ull << kEpochShift) - 1;

// The epoch of the launch that holds ticket `ticket`, each launch taking `tiles`.
RP_HOST_DEVICE inline unsigned long long launch_epoch(unsigned long long ticket, unsigned long long tiles) {
  return ticket / tiles % kEpochs + 1;
}

// store(k, word): word k of the tile.
template <int NV, typename Store>
RP_HOST_DEVICE inline void publish_words(unsigned long long epoch, const long long (&v)[NV], Store store) {
  static_assert(NV <= kVals, "a tile has kVals words");
#pragma unroll
  for (int k = 0; k < kVals; ++k)
    store(k, epoch << kEpochShift | (k < NV ? static_cast<unsigned long long>(v[k < NV ? k : 0]) & kValueMask : 0ull));
}

// load(k): word k of the tile. False if one of its first NV words is not this epoch's.
template <int NV, typename Load>
RP_HOST_DEVICE inline bool fetch_words(unsigned long long epoch, long long (&v)[NV], Load load) {
  static_assert(NV <= kVals, "a tile has kVals words");
  bool ok = true;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const unsigned long long w = load(k);
    ok = ok && (w >> kEpochShift) == epoch;
    v[k] = static_cast<long long>(w & kValueMask);
  }
  return ok;
}

}  // namespace rp
