// Frontier and message kernels.
//
// Per layer l the dirty set D^l (vertices whose layer-(l-1) contribution changed)
// pushes its delta rows along every post-batch out-arc into the cached aggregate
// S^l (Sec. IV-C.1: a message carries the new minus the old embedding and the
// receiver adds it to its mailbox), and the affected set
//   A^l = out(D^l) u sinks(net arcs) u D^l
// is collected in two bitmaps (one for the out-arc sinks, so that their distinct
// count is known exactly) and compacted into a sorted list by a popcount prefix
// sum, which also yields each listed vertex's first out-arc index for the next
// layer's scatter. A pushing layer with a small frontier instead lists A^l in its
// own scatter, in no particular order: the first setter of a member's bit appends
// it (see ScatterList). The layer-1 dirty set of a batch without GCN terms is
// listed by the correction kernel itself, with its deltas.
#include <type_traits>

#include "internal.h"
#include "lookback.h"

namespace rp {

namespace {

constexpr int kCompactThreads = 256;
constexpr int kCompactWaves = kCompactThreads / kWave;
// Vertices per compaction tile: eight per thread, or sixteen on graphs of more than
// 2^19 vertices (half as many tiles for the look-back to cross; at 2.45M vertices
// 598 tiles).
constexpr int kTileSmall = 8 * kCompactThreads, kTileLarge = 16 * kCompactThreads;
constexpr long long kTileLargeFrom = 1LL << 19;
inline int tile_vertices(long long n) { return n > kTileLargeFrom ? kTileLarge : kTileSmall; }
// Tiles that are placed by block index: no more than the compute units, so that all
// are resident at once (graphs up to 2^20 vertices; larger ones go in ticket order).
constexpr long long kIndexTiles = 256;

__device__ inline int lane_id() { return threadIdx.x & (kWave - 1); }

__device__ inline long long global_wave() {
  return (static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x) / kWave;
}

__device__ inline long long num_waves() {
  return static_cast<long long>(gridDim.x) * blockDim.x / kWave;
}

__device__ inline int lanes_below(u64 mask) {
  return static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<unsigned>(mask >> 32),
                                                    __builtin_amdgcn_mbcnt_lo(static_cast<unsigned>(mask), 0u)));
}

// Sets v's bit; the old word is not read back, so nothing waits on it.
__device__ inline void mark_only(unsigned *bm, int v) { atomicOr(&bm[v >> 5], 1u << (v & 31)); }

inline int blocks_for(long long items, int threads, int cap = 4096) {
  long long b = (items + threads - 1) / threads;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return static_cast<int>(b);
}

// The inserted arcs' slots, the pre-batch corrections and the layer-1 dirty marks
// (see launch_corr_mark).
__global__ void k_corr_mark(int agg, LayerPtrs lp, Adj out, Adj in, const int *ins_rank, const float *arc_w,
                            const int *ddeg, const int *flist, const int *ins_src, const int *ins_dst,
                            const int *del_src, const int *del_dst, const float *ins_w, const float *del_w,
                            unsigned *bm, Counters *c, DirectList dl) {
  const long long nf = static_cast<long long>(c->n_feat);
  const long long ni = static_cast<long long>(c->n_ins);
  const long long na = ni + static_cast<long long>(c->n_del);
  if (aborted_with(c->abort, nf, na)) return;
  const int lane = lane_id();
  const int *out_len = out.len;
  if (dl.list != nullptr && blockIdx.x == 0) {
    // block 0 lists the dirty set (flist[0, nf), distinct vertices) with the
    // exclusive prefix of their post-batch out-degrees: four entries per thread
    constexpr int kPer = kDirectListMax / 256;
    static_assert(kPer * 256 == kDirectListMax, "four entries per thread");
    __shared__ long long wsum[4];
    int v[kPer], dg[kPer];
    long long sum = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const long long i = static_cast<long long>(threadIdx.x) * kPer + q;
      v[q] = i < nf ? flist[i] : -1;
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      dg[q] = v[q] >= 0 ? out_len[v[q]] : 0;
      sum += dg[q];
    }
    long long incl = sum;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const long long y = __shfl_up(incl, o);
      if (lane >= o) incl += y;
    }
    const int wave = threadIdx.x / kWave;
    if (lane == kWave - 1) wsum[wave] = incl;
    __syncthreads();
    long long pos = incl - sum, total = 0;
    for (int w = 0; w < 4; ++w) {
      if (w < wave) pos += wsum[w];
      total += wsum[w];
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const long long i = static_cast<long long>(threadIdx.x) * kPer + q;
      if (i < nf) {
        dl.list[i] = v[q];
        dl.doff[i] = pos;
      }
      pos += dg[q];
    }
    if (threadIdx.x == 0) {
      const long long listed = nf < kDirectListMax ? nf : kDirectListMax;
      dl.doff[listed] = total;
      *dl.count = static_cast<u64>(listed);
      *dl.out_total = static_cast<u64>(total);
      if (nf > kDirectListMax) atomicOr(&c->err, 2ull);
    }
  }
  if (dl.delta != nullptr) {
    // layer-0 deltas of the listed vertices, one wave per row from the grid's last
    // wave down (the corrections start at wave 0); x' is staged, X keeps x
    const float *feat = dl.in->feat;
    const long long nl = nf < kDirectListMax ? nf : kDirectListMax;
    for (long long j = num_waves() - 1 - global_wave(); j < nl; j += num_waves()) {
      const int u = flist[j];
      const float *xu = dl.X + static_cast<long long>(u) * dl.d0;
      const float *xn = feat + static_cast<long long>(dl.frow[j]) * dl.d0;
      float *dj = dl.delta + j * dl.ld;
      float *sj = dl.stage + j * dl.ld;
      for (int k = lane; k < dl.d0; k += kWave) {
        const float x1 = xn[k];
        dj[k] = x1 - xu[k];
        sj[k] = x1;
      }
    }
  }
  {
    // item w = 2 * arc + direction: its row's inserts follow the kept entries, in
    // rank order
    const long long stride = static_cast<long long>(gridDim.x) * blockDim.x;
    for (long long w = blockIdx.x * blockDim.x + threadIdx.x; w < 2 * ni; w += stride) {
      const long long arc = w >> 1;
      const int dir = static_cast<int>(w & 1);
      const int row = dir == 0 ? ins_src[arc] : ins_dst[arc];
      const int entry = dir == 0 ? ins_dst[arc] : ins_src[arc];
      const Adj &a = dir ? in : out;
      const long long slot = a.off[row] + (a.len[row] - a.inscnt[row]) + ins_rank[w];
      a.col[slot] = entry;
      if (a.wt != nullptr) a.wt[slot] = arc_w[arc];
    }
  }
  const long long items = na * lp.L;
  for (long long it = global_wave(); it < items; it += num_waves()) {
    const long long arc = it / lp.L;
    const int l = static_cast<int>(it % lp.L) + 1;
    const bool ins = arc < ni;
    const int u = ins ? ins_src[arc] : del_src[arc - ni];
    const int v = ins ? ins_dst[arc] : del_dst[arc - ni];
    float coef = ins ? 1.0f : -1.0f;
    if (agg == kGcn) coef *= 1.0f / sqrtf(static_cast<float>(out_len[u] - ddeg[u]) + 1.0f);
    if (ins_w != nullptr) coef *= ins ? ins_w[arc] : del_w[arc - ni];  // the arc's weight
    const int d = lp.sw[l];
    const float *hu = lp.src[l] + static_cast<long long>(u) * d;
    float *sv = lp.S[l] + static_cast<long long>(v) * d;
    for (int k = lane; k < d; k += kWave) unsafeAtomicAdd(&sv[k], coef * hu[k]);
  }
  const long long total = nf + (agg == kGcn ? na : 0);
  const long long stride = static_cast<long long>(gridDim.x) * blockDim.x;
  for (long long i = blockIdx.x * blockDim.x + threadIdx.x + (dl.list != nullptr ? nf : 0); i < total; i += stride) {
    if (i < nf) {
      mark_only(bm, flist[i]);
    } else {
      const long long a = i - nf;
      const int u = a < ni ? ins_src[a] : del_src[a - ni];
      if (ddeg[u] != 0) mark_only(bm, u);
    }
  }
}

// Exclusive block scan of NV values at once (one LDS round; the caller's next
// barrier frees lds).
template <int NV>
__device__ inline void block_scan(const long long (&v)[NV], long long (&excl)[NV], long long (&total)[NV],
                                  long long (*lds)[NV]) {
  const int lane = lane_id(), wave = threadIdx.x / kWave;
  long long x[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) x[k] = v[k];
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const long long y = __shfl_up(x[k], o);
      if (lane >= o) x[k] += y;
    }
  }
  if (lane == kWave - 1) {
#pragma unroll
    for (int k = 0; k < NV; ++k) lds[wave][k] = x[k];
  }
  __syncthreads();
  long long before[NV] = {}, all[NV] = {};
#pragma unroll 1  // (unrolled, the waves' sums take 40 registers at once)
  for (int w = 0; w < kCompactWaves; ++w) {
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const long long t = lds[w][k];
      if (w < wave) before[k] += t;
      all[k] += t;
    }
  }
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    excl[k] = before[k] + x[k] - v[k];
    total[k] = all[k];
  }
}

constexpr int kSpinLimit = 1 << 20;

// A tile's sums to and from its words (see lookback.h).
template <int NV>
__device__ inline void publish(u64 *p, u64 epoch, const long long (&v)[NV]) {
  publish_words(epoch, v,
                [p](int k, u64 w) { __hip_atomic_store(p + k, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); });
}

template <int NV>
__device__ inline bool fetch(const u64 *p, u64 epoch, long long (&v)[NV]) {
  return fetch_words(epoch, v,
                     [p](int k) { return __hip_atomic_load(p + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); });
}

// V consecutive values from p (16-byte aligned), zeros past `left` of them.
template <int V>
__device__ inline void load_run(const int *p, long long left, int (&x)[V]) {
  if (left >= V) {
    const int4 *q = reinterpret_cast<const int4 *>(p);
#pragma unroll
    for (int i = 0; i < V / 4; ++i) {
      const int4 t = q[i];
      x[4 * i] = t.x;
      x[4 * i + 1] = t.y;
      x[4 * i + 2] = t.z;
      x[4 * i + 3] = t.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < V; ++i) x[i] = i < left ? p[i] : 0;
  }
}

// The tile's offsets of one kind into out[first ..): member j of the tile gets base
// plus the sum of x over the tile's members before it (run: that sum before this
// thread's first member, which is member `at` of the tile). Through LDS, so that the
// members' offsets go out as whole runs.
template <int V>
__device__ inline void write_offsets(unsigned bits, int at, long long run, const int (&x)[V], long long base,
                                     int members, long long *stage, long long *out) {
#pragma unroll
  for (int i = 0; i < V; ++i) {
    if (bits >> i & 1u) {
      stage[at++] = base + run;
      run += x[i];
    }
  }
  __syncthreads();
  for (int j = threadIdx.x; j < members; j += kCompactThreads) out[j] = stage[j];
  __syncthreads();
}

// Single-pass compaction (a decoupled look-back prefix scan) of tiles of
// V * kCompactThreads vertices, V consecutive vertices per thread. A thread's bits,
// degrees and bucket counts come in one round of 16-byte loads (on large graphs the
// degrees in a second round, and only where a bit is set). Tiles go to blocks by
// index when all of them fit on the GPU at once, else in ticket order; either way a
// tile's predecessors are running or done when it waits for them. Each tile
// publishes its sums at once, then walks back over its predecessors, one per thread
// and round, adding their sums; in ticket order the walk ends at the nearest
// predecessor that has published its inclusive prefix. A tile publishes its own sums
// before it waits, so every wait is for work that needs no waiting: all waits end. A
// wait that outlasts kSpinLimit polls (a predecessor that never ran) sets bit 2 of
// the error word and counts the tile as empty (the batch then fails loudly instead
// of hanging). Output: the marked vertices of both bitmaps as a sorted list with
// prefix sums of their out-degrees and bucket counts, membership words and per-word
// prefix counts, each staged in LDS and written as whole runs; both bitmaps and the
// bucket counters are cleared.
// Bound by latency (a load round, the look-back, the stores) up to some 10^5
// vertices and by the degree reads and list writes beyond. Tiles are this small to
// spread a dense frontier: with tiles of 32K vertices (6 blocks on 169K vertices, 75
// on 2.45M) and one thread walking the set bits of 128 vertices, a compaction took
// 50 us on average on the 3-layer mean workload at batch 1000 (169K vertices; now
// 8.3), 73 us on the RMAT graph of 2^20 vertices at batch 2500 (now 13, and 20 with
// bucket counts) and 103 us on dense_large at batch 1000 (2.45M; now 32 and 48).
template <int V, bool BKT>
__global__ __launch_bounds__(kCompactThreads, 3) void k_compact(unsigned *bm_a, unsigned *bm_b, long long n,
                                                             CompactOut o, u64 *agg, u64 *inc, u64 *ticket,
                                                             u64 *err) {
  constexpr int kTile = V * kCompactThreads;
  constexpr int NV = BKT ? kVals : kVals - 1;
  typedef typename std::conditional<V == 8, unsigned char, unsigned short>::type Bits;  // a thread's bits of a bitmap
  static_assert(sizeof(Bits) * 8 == V, "a thread's bits are one load");
  __shared__ long long red[kCompactWaves][NV];
  __shared__ int red_incl[kCompactWaves];
  __shared__ u64 epoch_s, ticket_s, long_base;
  __shared__ int long_count;
  __shared__ long long stage[kTile];
  const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  if (tid == 0) long_count = 0;  // published by the scan's barrier
  const long long tiles = gridDim.x;
  // Up to kIndexTiles tiles all fit on the GPU at once, so block b takes tile b and
  // its ticket (for the epoch) is in flight beside the loads. Beyond that, tiles go
  // in ticket order, so a tile's predecessors are running or done however the blocks
  // are dispatched.
  const bool by_ticket = tiles > kIndexTiles;
  u64 ticket_no = 0;
  if (by_ticket) {
    if (tid == 0) ticket_s = atomicAdd(ticket, 1ull);
    __syncthreads();
    ticket_no = ticket_s;
  }
  const long long tile = by_ticket ? static_cast<long long>(ticket_no % static_cast<u64>(tiles)) : blockIdx.x;
  const long long v0 = tile * kTile + static_cast<long long>(tid) * V;
  const long long left = n - v0;  // vertices from v0 on (may be <= 0)
  const bool in_bm = v0 < (n + 31) / 32 * 32;  // the bitmaps cover whole words
  const int *odeg = o.doff != nullptr || o.out_total != nullptr ? o.out_deg : nullptr;
  const int *ideg = o.in_deg;
  Bits *pa = reinterpret_cast<Bits *>(bm_a) + v0 / V, *pb = reinterpret_cast<Bits *>(bm_b) + v0 / V;
  unsigned bits = 0, bits_a = 0;
  int od[V] = {}, id[V] = {}, bc[V] = {};
  if (in_bm) {
    bits_a = *pa;
    bits = *pb;
  }
  // (the counters cover whole tiles, and those past n stay zero)
  if (BKT) load_run<V>(o.bkt_cnt + v0, V, bc);
  if (V == 8) {
    if (odeg != nullptr && left > 0) load_run<V>(odeg + v0, left, od);
    if (ideg != nullptr && left > 0) load_run<V>(ideg + v0, left, id);
  }
  if (!by_ticket && tid == 0) ticket_no = atomicAdd(ticket, 1ull);  // in flight beside the loads
  int bkt_any = 0;
#pragma unroll
  for (int i = 0; i < V; ++i) {  // the bucket form's sinks, from their counts, count as first-bitmap bits
    bits_a |= (bc[i] > 0 ? 1u : 0u) << i;
    bkt_any |= bc[i];
  }
  bits |= bits_a;
  if (V != 8 && bits != 0) {
    if (odeg != nullptr) load_run<V>(odeg + v0, left, od);
    if (ideg != nullptr) load_run<V>(ideg + v0, left, id);
  }
  long long st[NV] = {__popc(bits), 0, 0, __popc(bits_a)};
#pragma unroll
  for (int i = 0; i < V; ++i) {
    const bool on = bits >> i & 1u;
    st[1] += on ? od[i] : 0;
    st[2] += on ? id[i] : 0;
    if constexpr (BKT) st[4] += bc[i];
  }
  // The ticket counter only grows and every launch on this scratch has the same
  // number of blocks, each taking one ticket, so launch k holds tickets k * tiles
  // .. k * tiles + tiles - 1: the ticket's quotient names the launch.
  if (tid == 0) epoch_s = launch_epoch(ticket_no, static_cast<u64>(tiles));
  long long ex[NV], tot[NV];
  block_scan(st, ex, tot, red);  // its barrier also publishes epoch_s
  const u64 epoch = epoch_s;
  if (tid == 0) publish((by_ticket && tile == 0 ? inc : agg) + tile * kVals, epoch, tot);
  long long base[NV] = {};
  bool timed_out = false, done = false;
  for (long long j = tile - 1; j >= 0 && !done; j -= kCompactThreads) {
    const long long p = j - tid;
    long long v[NV] = {};
    bool incl = p < 0;  // threads before tile 0 end the walk with zeros
    if (p >= 0) {
      for (int it = 0;; ++it) {
        long long va[NV];  // in ticket order both words are read in the same round
        const bool got_agg = fetch(agg + p * kVals, epoch, va);
        if (by_ticket && fetch(inc + p * kVals, epoch, v)) {
          incl = true;
          break;
        }
        if (got_agg) {
#pragma unroll
          for (int k = 0; k < NV; ++k) v[k] = va[k];
          break;
        }
        if (it >= kSpinLimit) {
          timed_out = true;
#pragma unroll
          for (int k = 0; k < NV; ++k) v[k] = 0;
          break;
        }
        __builtin_amdgcn_s_sleep(2);
      }
    }
    // the wave's predecessors up to the nearest inclusive one, then the block's
    const u64 im = __ballot(incl);
    const int first = im ? __ffsll(static_cast<long long>(im)) - 1 : kWave;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      long long x = lane <= first ? v[k] : 0;
#pragma unroll
      for (int s = kWave / 2; s > 0; s >>= 1) x += __shfl_xor(x, s);
      v[k] = x;
    }
    __syncthreads();  // red: the scan's or the previous round's reads are over
    if (lane == 0) {
#pragma unroll
      for (int k = 0; k < NV; ++k) red[wave][k] = v[k];
      red_incl[wave] = first < kWave ? 1 : 0;
    }
    __syncthreads();
#pragma unroll 1
    for (int w = 0; w < kCompactWaves && !done; ++w) {
#pragma unroll
      for (int k = 0; k < NV; ++k) base[k] += red[w][k];
      done = red_incl[w] != 0;
    }
  }
  if (timed_out) atomicOr(err, 4ull);
  if (by_ticket && tile > 0 && tid == 0) {
    long long incv[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) incv[k] = base[k] + tot[k];
    publish(inc + tile * kVals, epoch, incv);
  }
  const int members = static_cast<int>(tot[0]);
  const int at = static_cast<int>(ex[0]);  // this thread's first member among the tile's
  if (o.memb != nullptr) {
    // a word's bits from its 32 / V threads, stored by the first of them
    constexpr int kPer = 32 / V;
    unsigned w = bits << (V * (tid % kPer));
#pragma unroll
    for (int s = 1; s < kPer; s <<= 1) w |= __shfl_xor(w, s);
    if (in_bm && tid % kPer == 0) o.memb[v0 / 32] = make_uint2(w, static_cast<unsigned>(base[0] + at));
  }
  if (in_bm) {
    *pa = 0;
    *pb = 0;
  }
  if (BKT && bkt_any != 0) {  // the counters are spent
    int4 *z = reinterpret_cast<int4 *>(o.bkt_cnt + v0);
#pragma unroll
    for (int i = 0; i < V / 4; ++i) z[i] = make_int4(0, 0, 0, 0);
  }
  if (o.list != nullptr) {
    int *ids = reinterpret_cast<int *>(stage);
    int k = at;
#pragma unroll
    for (int i = 0; i < V; ++i)
      if (bits >> i & 1u) ids[k++] = static_cast<int>(v0) + i;
    __syncthreads();
    for (int j = tid; j < members; j += kCompactThreads) o.list[base[0] + j] = ids[j];
    __syncthreads();
  }
  if (o.doff != nullptr) write_offsets<V>(bits, at, ex[1], od, base[1], members, stage, o.doff + base[0]);
  if constexpr (BKT) write_offsets<V>(bits, at, ex[4], bc, base[4], members, stage, o.boff + base[0]);
  if (o.longs != nullptr) {  // the tile's long in-rows take their places with one atomic
    unsigned lm = 0;
#pragma unroll
    for (int i = 0; i < V; ++i) lm |= ((bits >> i & 1u) && id[i] > kPullLong ? 1u : 0u) << i;
    const int place = lm != 0 ? atomicAdd(&long_count, __popc(lm)) : 0;
    __syncthreads();
    if (tid == 0 && long_count > 0) long_base = atomicAdd(o.nlong, static_cast<u64>(long_count));
    __syncthreads();
    int *out = o.longs + long_base + place;
    for (; lm != 0; lm &= lm - 1) *out++ = static_cast<int>(v0) + __ffs(lm) - 1;
  }
  if (tile == tiles - 1 && tid == 0) {
    const long long total = base[0] + tot[0];
    *o.count = static_cast<u64>(total);
    if (o.doff != nullptr) o.doff[total] = base[1] + tot[1];
    if constexpr (BKT) o.boff[total] = base[4] + tot[4];
    if (o.out_total != nullptr) *o.out_total = static_cast<u64>(base[1] + tot[1]);
    if (o.in_total != nullptr) *o.in_total = static_cast<u64>(base[2] + tot[2]);
    if (o.sinks_a != nullptr) *o.sinks_a = static_cast<u64>(base[3] + tot[3]);
  }
}

// First index i in [lo, hi) with a[i] > x (hi if none).
__device__ inline long long upper_bound(const long long *a, long long lo, long long hi, long long x) {
  while (lo < hi) {
    const long long mid = (lo + hi) >> 1;
    if (a[mid] <= x) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// Last index j in [lo, hi) with a[j] <= x, for non-decreasing a with a[lo] <= x.
// The whole wave searches together: each round probes 64 evenly spaced entries
// with one load and keeps the gap after the last probe that is <= x, so a search
// over m entries takes ceil(log64 m) dependent loads instead of log2 m.
__device__ inline long long wave_last_le(const long long *a, long long lo, long long hi, long long x) {
  const int lane = lane_id();
  while (hi - lo > kWave) {
    const long long step = (hi - lo + kWave - 1) / kWave;
    const long long idx = lo + lane * step;
    const bool le = idx < hi && a[idx] <= x;
    const int last = __popcll(__ballot(le)) - 1;  // probes <= x form a prefix
    lo = lo + last * step;
    hi = lo + step < hi ? lo + step : hi;
  }
  const long long idx = lo + lane;
  const bool le = idx < hi && a[idx] <= x;
  return lo + __popcll(__ballot(le)) - 1;
}

// wave_last_le over [0, n) that also hands back its last round's loads: lane t
// holds a[w0 + t] (1 << 62 past n), w0 <= the answer.
__device__ inline long long wave_last_le_win(const long long *a, long long n, long long x, long long &win,
                                             long long &w0) {
  const int lane = lane_id();
  long long lo = 0, hi = n;
  while (hi - lo > kWave) {
    const long long step = (hi - lo + kWave - 1) / kWave;
    const long long idx = lo + lane * step;
    const bool le = idx < hi && a[idx] <= x;
    const int last = __popcll(__ballot(le)) - 1;
    lo = lo + last * step;
    hi = lo + step < hi ? lo + step : hi;
  }
  const long long idx = lo + lane;
  win = idx < n ? a[idx] : (1LL << 62);
  w0 = lo;
  return lo + __popcll(__ballot(idx < hi && win <= x)) - 1;
}

// Same answer as wave_last_le(a, from, n1, x), for a lower bound `from` whose
// answer is usually close: one round of 64 probes from `from`, and the full
// search only when every probe is <= x. Used when a wave walks consecutive arcs.
__device__ inline long long owner_from(const long long *a, long long from, long long n1, long long x) {
  const int lane = lane_id();
  const long long hi = from + kWave < n1 ? from + kWave : n1;
  const long long idx = from + lane;
  const bool le = idx < hi && a[idx] <= x;
  const int cnt = __popcll(__ballot(le));
  if (cnt == hi - from && hi < n1) return wave_last_le(a, hi - 1, n1, x);
  return from + cnt - 1;
}

// One wave per listed vertex (see Delta0Args). list holds cap entries: the wave's
// first vertex is fetched with the count (an entry past the count is dropped).
__global__ void k_delta0(Delta0Args z, const int *list, const u64 *count, long long cap) {
  const long long j0 = global_wave();
  const int u0 = j0 < cap ? list[j0] : 0;
  const long long m = static_cast<long long>(*count);
  const float *feat = z.in->feat;
  // (an entry past the count may hold anything: it joins the test as an unsigned
  // half, which is never negative)
  if (aborted_with(z.c->abort, m, static_cast<unsigned>(u0) >> 1)) return;
  const int lane = lane_id();
  for (long long j = j0; j < m; j += num_waves()) {
    const int u = j == j0 ? u0 : list[j];
    const int fo = z.fop[u];
    float cn = 1.0f, co = 1.0f;
    if (z.agg == kGcn) {
      const int dout = z.out_len[u];
      cn = 1.0f / sqrtf(static_cast<float>(dout) + 1.0f);
      co = 1.0f / sqrtf(static_cast<float>(dout - z.ddeg[u]) + 1.0f);
    }
    float *xu = z.X + static_cast<long long>(u) * z.d0;
    const float *xn = fo >= 0 ? feat + static_cast<long long>(z.ops[fo].feat_row) * z.d0 : xu;
    float *dj = z.delta + j * z.ld;
    for (int k = lane; k < z.d0; k += kWave) {
      const float xo = xu[k];
      const float x1 = xn[k];
      dj[k] = cn * x1 - co * xo;
      xu[k] = x1;
    }
  }
}

// Arc e = e0 + lane (e <= elast) of the scatter's numbering, for a run whose first
// and last arcs belong to list positions ja and jb: its sink (-1 past elast).
__device__ inline int run_sink(const long long *doff, const int *list, const Adj &out, long long e0,
                               long long elast, long long ja, long long jb) {
  const int lane = lane_id();
  const long long e = e0 + lane;
  const bool active = e <= elast;
  int j = static_cast<int>(ja);
  if (jb > ja) {
    if (jb - ja < kWave) {
      const long long mine = ja + lane <= jb ? doff[ja + lane] : (1LL << 62);
      int cnt_le = 0;
      for (int t = 0; t <= static_cast<int>(jb - ja); ++t) cnt_le += __shfl(mine, t) <= e ? 1 : 0;
      j = static_cast<int>(ja) + cnt_le - 1;
    } else if (active) {
      j = static_cast<int>(upper_bound(doff, ja, jb + 1, e) - 1);
    }
  }
  if (!active) return -1;
  const int u = list[j];
  return out.col[out.off[u] + (e - doff[j])];
}

// One mark per lane (v < 0: none) by a scatter that lists A^l itself (see
// ScatterList): the membership and sink bits are set with returning atomics, the
// degrees are read beside them, and the lanes that set a membership bit first take
// consecutive list positions and out-arc offsets with one atomic for the wave.
__device__ inline void list_mark(int v, bool sink, const ScatterList &lo, unsigned *bm_out, unsigned *bm_x) {
  const int lane = lane_id();
  bool fresh = false, fresh_sink = false;
  long long dv = 0, iv = 0;
  if (v >= 0) {
    const unsigned bit = 1u << (v & 31);
    const unsigned om = atomicOr(&bm_x[v >> 5], bit);
    const unsigned os = sink ? atomicOr(&bm_out[v >> 5], bit) : bit;
    dv = lo.doff != nullptr ? lo.out_len[v] : 0;
    iv = lo.in_len[v];
    fresh = (om & bit) == 0;
    fresh_sink = (os & bit) == 0;
  }
  const u64 ms = __ballot(fresh_sink);
  const u64 m = __ballot(fresh);
  if ((m | ms) == 0) return;
  if (!fresh) dv = iv = 0;
  long long dinc = dv, itot = iv;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const long long y = __shfl_up(dinc, o);
    if (lane >= o) dinc += y;
    itot += __shfl_xor(itot, o);
  }
  const long long dtot = __shfl(dinc, kWave - 1);
  const int leader = __ffsll(static_cast<long long>(m | ms)) - 1;
  u64 base = 0;
  if (lane == leader) {
    if (m != 0) base = atomicAdd(lo.app, static_cast<u64>(__popcll(m)) << kAppShift | static_cast<u64>(dtot));
    atomicAdd(lo.sinks, static_cast<u64>(__popcll(ms)) << kAppShift | static_cast<u64>(itot));
  }
  base = __shfl(base, leader);
  if (fresh) {
    const int below = lanes_below(m);
    const long long pos = static_cast<long long>(base >> kAppShift) + below;
    lo.list[pos] = v;
    if (lo.doff != nullptr) lo.doff[pos] = static_cast<long long>(base & kAppMask) + dinc - dv;
  }
}

// Edge-parallel scatter. Pushed arcs are numbered: arc e of listed vertex j has
// index doff[j] + its position in j's out-row. A wave takes a chunk of C
// consecutive arcs (C = 1 when there are few arcs, so that many waves run at
// once; up to 64 when there are many), each lane resolves one arc's source slot
// and sink and marks the sink, then G lanes per arc add the source's delta row
// into the sink's row of S with fp32 atomics (coalesced across the G lanes). The
// delta row stays in registers while consecutive arcs share a source, so a hub's
// arcs cost one row load per chunk; hubs spread over many waves.
template <int G, int NC, bool PUSH, bool LIST>
__global__ __launch_bounds__(256) void k_scatter(int d, int ld, const int *list, const u64 *count, const long long *doff,
                                                 const float *delta, Adj out, float *S, unsigned *bm_out,
                                                 unsigned *bm_x, const int *ins_dst, const int *del_dst,
                                                 const u64 *pushed, const Counters *c, int mark_list,
                                                 ScatterCopy copy, ScatterList lo, int packed_in) {
  const u64 cw = *count;
  const long long nD = static_cast<long long>(packed_in ? cw >> kAppShift : cw);
  const long long E = static_cast<long long>(packed_in ? cw & kAppMask : *pushed);
  const long long ni = static_cast<long long>(c->n_ins);
  const long long na = ni + static_cast<long long>(c->n_del);
  if (aborted_with(c->abort, nD, E, na)) return;
  const int lane = lane_id();
  {
    const long long stride = static_cast<long long>(gridDim.x) * blockDim.x;
    const long long t0 = blockIdx.x * blockDim.x + threadIdx.x;
    if (!LIST) {
      for (long long i = t0; i < na; i += stride) mark_only(bm_x, i < ni ? ins_dst[i] : del_dst[i - ni]);
      if (mark_list)
        for (long long j = t0; j < nD; j += stride) mark_only(bm_x, list[j]);
    } else {
      // the net arcs' heads, then D when it joins A^l: whole waves step together
      const long long marks = na + (mark_list ? nD : 0);
      for (long long b = t0 - lane; b < marks; b += stride) {
        const long long i = b + lane;
        const int v = i >= marks ? -1 : i < ni ? ins_dst[i] : i < na ? del_dst[i - ni] : list[i - na];
        list_mark(v, false, lo, bm_out, bm_x);
      }
    }
  }
  if (copy.dst != nullptr) {
    // the staged rows of the listed vertices, one wave each from the grid's last
    // wave down (nothing in this kernel reads them)
    for (long long j = num_waves() - 1 - global_wave(); j < nD; j += num_waves()) {
      float *xu = copy.dst + static_cast<long long>(list[j]) * copy.d;
      const float *sj = copy.stage + j * copy.ld;
      for (int k = lane; k < copy.d; k += kWave) xu[k] = sj[k];
    }
  }
  const long long waves = num_waves();
  if (LIST) {
    // A^l listed here: the sinks are marked 64 arcs per wave (one list append per
    // wave), by waves from the grid's last one down (the adds below start at wave 0)
    const long long groups = (E + kWave - 1) / kWave;
    for (long long g = waves - 1 - global_wave(); g < groups; g += waves) {
      const long long e0 = g * kWave;
      const long long elast = e0 + kWave - 1 < E - 1 ? e0 + kWave - 1 : E - 1;
      // the search's last round leaves doff[w0 .. w0 + 63] in the lanes (w0 <= ja):
      // when the group's last arc falls in that window (no more than 64 - (ja - w0)
      // owners), each arc's owner and offset come from it by shuffles, with no
      // further load of the offsets
      long long mine, w0;
      const long long ja = wave_last_le_win(doff, nD, e0, mine, w0);
      const int owners = __popcll(__ballot(mine <= elast));  // window entries starting at or before elast
      int v = -1;
      if (owners < kWave || w0 + kWave >= nD) {
        const long long e = e0 + lane;
        int cnt_le = 0;
        for (int t = static_cast<int>(ja - w0); t < owners; ++t) cnt_le += __shfl(mine, t) <= e ? 1 : 0;
        const int at = static_cast<int>(ja - w0) + (cnt_le > 0 ? cnt_le - 1 : 0);
        const long long start = __shfl(mine, at);
        if (e <= elast) {
          const int u = list[w0 + at];
          v = out.col[out.off[u] + (e - start)];
        }
      } else {
        v = run_sink(doff, list, out, e0, elast, ja, owner_from(doff, ja, nD, elast));
      }
      list_mark(v, true, lo, bm_out, bm_x);
    }
  }
  // the owner searches run over doff[0, n1): a compacted list's doff[nD] holds the
  // arc total; a scatter-built list has no such entry, and needs none, as every
  // arc index is below the total
  const long long n1 = packed_in ? nD : nD + 1;
  int C = 1;
  while (C < kWave && static_cast<long long>(C) * waves < E) C <<= 1;
  constexpr int kEdgesPerStep = kWave / G;
  const int grp = lane / G, k0 = lane % G;
  int cached = -1;
  float dreg[NC];
  const long long chunks = (E + C - 1) / C;
  // a wave takes a contiguous run of chunks, so each chunk's first source is
  // found from the previous chunk's
  const long long per = (chunks + waves - 1) / waves;
  const long long c0 = global_wave() * per;
  const long long c1 = c0 + per < chunks ? c0 + per : chunks;
  long long ja = -1;
  for (long long ch = c0; ch < c1; ++ch) {
    const long long e0 = ch * C;
    const long long elast = e0 + C - 1 < E - 1 ? e0 + C - 1 : E - 1;
    ja = ja < 0 ? wave_last_le(doff, 0, n1, e0) : owner_from(doff, ja, n1, e0);
    if (PUSH && ja != cached) {
      // the chunk's first source is known before its arcs are resolved: fetch its
      // delta row now so that the load overlaps the list / offset / column reads
      const float *dj = delta + ja * ld;
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        const int k = k0 + q * G;
        dreg[q] = k < d ? dj[k] : 0.0f;
      }
      cached = static_cast<int>(ja);
    }
    const long long jb = C == 1 ? ja : owner_from(doff, ja, n1, elast);
    const long long e = e0 + lane;
    const bool active = e <= elast;
    int j = static_cast<int>(ja);
    if (jb > ja) {
      if (jb - ja < kWave) {
        // the window's offsets, one per lane; every lane takes part in the shuffles
        const long long mine = ja + lane <= jb ? doff[ja + lane] : (1LL << 62);
        int cnt_le = 0;
        for (int t = 0; t <= static_cast<int>(jb - ja); ++t) cnt_le += __shfl(mine, t) <= e ? 1 : 0;
        j = static_cast<int>(ja) + cnt_le - 1;
      } else if (active) {
        j = static_cast<int>(upper_bound(doff, ja, jb + 1, e) - 1);
      }
    }
    int v = -1;
    float wv = 1.0f;  // the arc's weight (weighted graphs)
    if (active) {
      const int u = list[j];
      const long long slot = out.off[u] + (e - doff[j]);
      v = out.col[slot];
      if (PUSH && out.wt != nullptr) wv = out.wt[slot];
    }
    if (!LIST && v >= 0) mark_only(bm_out, v);
    const int cnt = PUSH ? static_cast<int>(elast - e0 + 1) : 0;
    for (int i = 0; i < cnt; i += kEdgesPerStep) {
      const int vv = __shfl(v, i + grp);
      const int jj = __shfl(j, i + grp);
      const float ww = __shfl(wv, i + grp);
      if (vv >= 0) {
        if (jj != cached) {
          const float *dj = delta + static_cast<long long>(jj) * ld;
#pragma unroll
          for (int q = 0; q < NC; ++q) {
            const int k = k0 + q * G;
            dreg[q] = k < d ? dj[k] : 0.0f;
          }
          cached = jj;
        }
        float *sv = S + static_cast<long long>(vv) * d;
#pragma unroll
        for (int q = 0; q < NC; ++q) {
          const int k = k0 + q * G;
          if (k < d) unsafeAtomicAdd(&sv[k], ww * dreg[q]);
        }
      }
    }
  }
}

constexpr int kBinArcs = 4;  // arcs per lane per chunk (the bucket passes)
constexpr int kBinChunk = kWave * kBinArcs;

// Exclusive prefix sums of a[0, n) in LDS, in place, by a block of kBinThreads
// threads (each a run of consecutive entries); ends with a barrier.
__device__ inline void block_exclusive_scan(int *a, int n, int *wave_sums) {
  const int t = threadIdx.x, lane = lane_id(), wave = t / kWave;
  const int per = (n + kBinThreads - 1) / kBinThreads;
  int s = 0;
  for (int i = 0; i < per; ++i) {
    const int k = t * per + i;
    if (k < n) s += a[k];
  }
  int incl = s;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int y = __shfl_up(incl, o);
    if (lane >= o) incl += y;
  }
  if (lane == kWave - 1) wave_sums[wave] = incl;
  __syncthreads();
  int base = incl - s;
  for (int w = 0; w < wave; ++w) base += wave_sums[w];
  for (int i = 0; i < per; ++i) {
    const int k = t * per + i;
    if (k < n) {
      const int x = a[k];
      a[k] = base;
      base += x;
    }
  }
  __syncthreads();
}

// The bucket form's passes over the pushed arcs (numbered as in the scatter), in
// chunks of up to kBinChunk consecutive arcs per wave (a contiguous run of chunks
// per wave, so that a block owns the same arcs in both passes), each lane up to
// kBinArcs consecutive arcs with all their loads in flight together. The arcs are
// sorted by sink in two levels: into bins of 2^shift consecutive sinks here, then
// by sink within each bin (k_bin_sort). Counting pass (SCATTER false): marks the
// net arcs' heads and, under a self term, D in bm_x, counts the block's arcs per
// bin in LDS, and adds each count to its bin's total with one atomic, which hands
// back the block's place in the bin. Scatter pass: the bins' first slots are the
// exclusive prefix of their totals (block 0 also stores them); each arc takes the
// next place of its block in its bin (an LDS cursor) and leaves its sink, its
// source's list position (its message row) and, when the model weights arcs, its
// weight there.
template <bool SCATTER>
__global__ __launch_bounds__(kBinThreads) void k_bin_arcs(const int *list, const u64 *count, const long long *doff,
                                                           Adj out, const u64 *pushed, Buckets b, unsigned *bm_x,
                                                           const int *ins_dst, const int *del_dst, int mark_list,
                                                           const Counters *c) {
  extern __shared__ int bins[];  // per bin: the block's count, or its cursor
  __shared__ int wave_sums[kBinThreads / kWave];
  const long long nD = static_cast<long long>(*count);
  const long long E = static_cast<long long>(*pushed);
  const long long ni = static_cast<long long>(c->n_ins);
  const long long na = ni + static_cast<long long>(c->n_del);
  if (aborted_with(c->abort, nD, E, na)) return;  // the same for the whole block
  const int lane = lane_id();
  const int nb = b.nbins;
  if (!SCATTER) {
    for (int i = threadIdx.x; i < nb; i += kBinThreads) bins[i] = 0;
    const long long stride = static_cast<long long>(gridDim.x) * kBinThreads;
    const long long t0 = blockIdx.x * static_cast<long long>(kBinThreads) + threadIdx.x;
    for (long long i = t0; i < na; i += stride) mark_only(bm_x, i < ni ? ins_dst[i] : del_dst[i - ni]);
    if (mark_list)
      for (long long j = t0; j < nD; j += stride) mark_only(bm_x, list[j]);
    __syncthreads();
  } else {
    for (int i = threadIdx.x; i < nb; i += kBinThreads) bins[i] = b.bin_total[i];
    __syncthreads();
    block_exclusive_scan(bins, nb, wave_sums);
    const int *own = b.block_off + static_cast<long long>(blockIdx.x) * nb;
    for (int i = threadIdx.x; i < nb; i += kBinThreads) {
      if (blockIdx.x == 0) b.bin_base[i] = bins[i];
      bins[i] += own[i];
    }
    __syncthreads();
  }
  const long long waves = num_waves();
  const long long n1 = nD + 1;  // a compacted list: doff[nD] holds the arc total
  int C = 1;
  while (C < kBinChunk && static_cast<long long>(C) * waves < E) C <<= 1;
  const int per_lane = C > kWave ? C / kWave : 1;
  const long long chunks = (E + C - 1) / C;
  const long long per = (chunks + waves - 1) / waves;
  const long long c0 = global_wave() * per;
  const long long c1 = c0 + per < chunks ? c0 + per : chunks;
  long long ja = -1;
  for (long long ch = c0; ch < c1; ++ch) {
    const long long e0 = ch * C;
    const long long elast = e0 + C - 1 < E - 1 ? e0 + C - 1 : E - 1;
    ja = ja < 0 ? wave_last_le(doff, 0, n1, e0) : owner_from(doff, ja, n1, e0);
    const long long jb = C == 1 ? ja : owner_from(doff, ja, n1, elast);
    long long e[kBinArcs];
    int r[kBinArcs];
    bool on[kBinArcs];
#pragma unroll
    for (int a = 0; a < kBinArcs; ++a) {
      e[a] = e0 + static_cast<long long>(lane) * per_lane + a;
      on[a] = a < per_lane && e[a] <= elast;
      r[a] = static_cast<int>(ja);
    }
    if (jb > ja) {
      if (jb - ja < kWave) {
        // the window's offsets, one per lane; every lane takes part in the shuffles
        const long long mine = ja + lane <= jb ? doff[ja + lane] : (1LL << 62);
        int cnt[kBinArcs] = {};
        for (int t = 0; t <= static_cast<int>(jb - ja); ++t) {
          const long long o = __shfl(mine, t);
#pragma unroll
          for (int a = 0; a < kBinArcs; ++a) cnt[a] += o <= e[a] ? 1 : 0;
        }
#pragma unroll
        for (int a = 0; a < kBinArcs; ++a) r[a] = static_cast<int>(ja) + cnt[a] - 1;
      } else {
#pragma unroll
        for (int a = 0; a < kBinArcs; ++a)
          if (on[a]) r[a] = static_cast<int>(upper_bound(doff, ja, jb + 1, e[a]) - 1);
      }
    }
    long long slot[kBinArcs];
    int v[kBinArcs];
#pragma unroll
    for (int a = 0; a < kBinArcs; ++a) {
      const int u = on[a] ? list[r[a]] : 0;
      slot[a] = on[a] ? out.off[u] + (e[a] - doff[r[a]]) : 0;
    }
#pragma unroll
    for (int a = 0; a < kBinArcs; ++a) v[a] = on[a] ? out.col[slot[a]] : 0;
    if (!SCATTER) {
#pragma unroll
      for (int a = 0; a < kBinArcs; ++a)
        if (on[a]) atomicAdd(&bins[v[a] >> b.shift], 1);
    } else {
      float w[kBinArcs];
#pragma unroll
      for (int a = 0; a < kBinArcs; ++a) w[a] = on[a] && b.tw != nullptr ? out.wt[slot[a]] : 1.0f;
#pragma unroll
      for (int a = 0; a < kBinArcs; ++a) {
        if (!on[a]) continue;
        const int p = atomicAdd(&bins[v[a] >> b.shift], 1);
        b.tv[p] = v[a];
        b.tj[p] = r[a];
        if (b.tw != nullptr) b.tw[p] = w[a];
      }
    }
  }
  if (!SCATTER) {
    // the block's counts into the bins' totals; a bin it has no arc in gets place 0
    __syncthreads();
    int *own = b.block_off + static_cast<long long>(blockIdx.x) * nb;
    for (int i = threadIdx.x; i < nb; i += kBinThreads) own[i] = bins[i] > 0 ? atomicAdd(&b.bin_total[i], bins[i]) : 0;
  }
}

// Second level of the bucket sort: block i takes bin i (sinks i 2^shift ..
// (i + 1) 2^shift - 1, its arcs in slots bin_base[i] .. + bin_total[i]). It counts
// the arcs per sink in LDS, stores the counts in cnt (from which the compaction
// lists the sinks and forms their buckets' offsets, the same prefix sums in vertex
// order), then places each arc at its sink's next slot: idx (and wt) hold each
// sink's bucket contiguously, buckets in vertex order. Resets the bin's total.
__global__ __launch_bounds__(kBinThreads) void k_bin_sort(long long n, const u64 *pushed, Buckets b,
                                                           const Counters *c) {
  extern __shared__ int cur[];  // per sink of the bin: its count, then its next slot
  __shared__ int wave_sums[kBinThreads / kWave];
  const long long E = static_cast<long long>(*pushed);
  if (aborted_with(c->abort, E)) return;
  const int bin = blockIdx.x;
  const int total = b.bin_total[bin];
  if (total == 0) return;  // the same for the whole block; its sinks' counters stay zero
  const int base = b.bin_base[bin];
  const int span = 1 << b.shift;
  const long long v0 = static_cast<long long>(bin) << b.shift;
  const int nv = static_cast<int>(n - v0 < span ? n - v0 : span);
  const int t = threadIdx.x;
  for (int i = t; i < span; i += kBinThreads) cur[i] = 0;
  __syncthreads();
  if (t == 0) b.bin_total[bin] = 0;  // every thread has read it
  constexpr int kU = 8;  // arcs per thread in flight
  for (int p0 = t; p0 < total; p0 += kU * kBinThreads) {
    int vv[kU];
#pragma unroll
    for (int q = 0; q < kU; ++q) {
      const int p = p0 + q * kBinThreads;
      vv[q] = p < total ? b.tv[base + p] : -1;
    }
#pragma unroll
    for (int q = 0; q < kU; ++q)
      if (vv[q] >= 0) atomicAdd(&cur[vv[q] - v0], 1);
  }
  __syncthreads();
  for (int i = t; i < nv; i += kBinThreads) b.cnt[v0 + i] = cur[i];
  block_exclusive_scan(cur, span, wave_sums);
  for (int p0 = t; p0 < total; p0 += kU * kBinThreads) {
    int vv[kU], jj[kU];
    float ww[kU];
#pragma unroll
    for (int q = 0; q < kU; ++q) {
      const int p = p0 + q * kBinThreads;
      const bool on = p < total;
      vv[q] = on ? b.tv[base + p] : -1;
      jj[q] = on ? b.tj[base + p] : 0;
      ww[q] = on && b.tw != nullptr ? b.tw[base + p] : 1.0f;
    }
#pragma unroll
    for (int q = 0; q < kU; ++q) {
      if (vv[q] < 0) continue;
      const int at = base + atomicAdd(&cur[vv[q] - v0], 1);
      b.idx[at] = jj[q];
      if (b.wt != nullptr) b.wt[at] = ww[q];
    }
  }
}

// The bucket form's sums (see launch_bucket_sum), on the recompute's split with
// bucket slots for in-arcs: ranges of C <= kBucketSeg consecutive slots, a
// contiguous run of them per wave; a range owns the first segment (up to
// kBucketSeg slots) of each sink whose bucket starts in it and at most one
// later segment of the sink before. Besides the message and aggregate rows, a
// range reads only three windows, which its wave fetches in one round of loads:
// the bucket starts and the vertices of the 64 sinks from the one before the
// range's first (lane t: boff and list at jf - 1 + t), and the 128 slots (message
// row and weight) from the range start, since a segment that starts in a range of
// at most 64 slots ends within 128 slots of its start. The windows of the wave's
// next range are fetched while the groups sum this range's segments, so a segment
// costs one round trip: its message rows, loaded together with its aggregate row.
// Sums are fp32; a one-segment bucket is added with a plain load and store, longer
// ones with atomics. Sinks with empty buckets are left alone.
template <int G, int NC, int U>
__global__ __launch_bounds__(256) void k_bucket_sum(int d, int ld, const int *list, const u64 *count,
                                                    const long long *boff, Buckets bk, const float *msg, float *S,
                                                    const Counters *c) {
  static_assert(kWave % G == 0 && G % U == 0 && kBucketSeg % U == 0, "steps of U slots");
  static_assert(kBucketSeg <= kWave, "a segment starting in a range ends within two windows of slots");
  constexpr int kSlots = 2 * kWave;
  constexpr int kSteps = kBucketSeg / U;
  constexpr int kGroups = kWave / G;
  __shared__ long long win_b[256 / kWave][kWave];
  __shared__ int win_v[256 / kWave][kWave];
  __shared__ int win_u[256 / kWave][kSlots];
  __shared__ float win_w[256 / kWave][kSlots];
  const int w = threadIdx.x / kWave;
  long long *wb = win_b[w];
  int *wv = win_v[w], *wu = win_u[w];
  float *ww = win_w[w];
  const long long nA = static_cast<long long>(*count);
  if (aborted_with(c->abort, nA) || nA == 0) return;
  const long long E = boff[nA];
  if (E == 0) return;  // no message reached any sink
  const int lane = lane_id();
  const int grp = lane / G, k0 = lane % G;
  const bool weighted = bk.wt != nullptr;
  // the weight window is loaded unconditionally (from the slot array when there are no weights)
  const float *wsrc = weighted ? bk.wt : reinterpret_cast<const float *>(bk.idx);
  const long long waves = num_waves();
  long long C = 16;
  while (C < kBucketSeg && C * waves < E) C <<= 1;
  const long long ranges = (E + C - 1) / C;
  const long long per = (ranges + waves - 1) / waves;
  const long long r0 = global_wave() * per;
  const long long r1 = r0 + per < ranges ? r0 + per : ranges;
  if (r0 >= r1) return;
  // the window registers of the next range (clamped loads: entries outside the
  // list or the slots repeat its ends and are never used, except boff past nA,
  // which reads E and so ends the search for the range's last sink)
  long long nb;
  int nv, nu0, nu1;
  float nw0, nw1;
  const auto fetch = [&](long long jf, long long R0) {
    const long long i = jf - 1 + lane;
    const long long ib = i < 0 ? 0 : i > nA ? nA : i;
    const long long iv = i < 0 ? 0 : i > nA - 1 ? nA - 1 : i;
    const long long s0 = R0 + lane < E ? R0 + lane : E - 1;
    const long long s1 = R0 + kWave + lane < E ? R0 + kWave + lane : E - 1;
    nb = boff[ib];
    nv = list[iv];
    nu0 = bk.idx[s0];
    nu1 = bk.idx[s1];
    nw0 = wsrc[s0];
    nw1 = wsrc[s1];
  };
  // first sink starting at or after the first range's start
  long long jf = r0 == 0 ? 0 : wave_last_le(boff, 0, nA + 1, r0 * C - 1) + 1;
  fetch(jf, r0 * C);
  for (long long r = r0; r < r1; ++r) {
    const long long R0 = r * C;
    const bool last_range = r == ranges - 1;
    const long long R1 = last_range ? (1LL << 62) : R0 + C;
    // the previous range's groups have read the windows: publish this range's
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    wb[lane] = nb;
    wv[lane] = nv;
    wu[lane] = nu0;
    wu[kWave + lane] = nu1;
    ww[lane] = nw0;
    ww[kWave + lane] = nw1;
    // the last sink starting before R1: the window's entries <= R1 - 1 form a prefix
    // (lane 0 stands for the sink before jf, or for nothing when jf = 0)
    long long jl = nA - 1;
    if (!last_range) {
      const bool le = jf - 1 + lane < 0 || nb <= R1 - 1;
      const int cnt = __popcll(__ballot(le));
      jl = jf + cnt - 2;
      if (cnt == kWave && jf - 1 + kWave <= nA) jl = wave_last_le(boff, jf - 2 + kWave, nA + 1, R1 - 1);
      if (jl > nA - 1) jl = nA - 1;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (r + 1 < r1) fetch(jl + 1, R0 + C);
    // the sink before jf covers slot R0 when its bucket ends past it: it may have a
    // segment starting in this range
    long long pstart = -1, pend = 0;
    if (jf >= 1) {
      const long long a = wb[0], b = wb[1];
      if (b > R0) {
        const long long s = (R0 - a + kBucketSeg - 1) / kBucketSeg;
        const long long st = a + s * kBucketSeg;
        if (st < R1 && st < b) {
          pstart = st;
          pend = st + kBucketSeg < b ? st + kBucketSeg : b;
        }
      }
    }
    const long long has_pred = pstart >= 0 ? 1 : 0;
    const long long sinks = jl >= jf ? jl - jf + 1 : 0;
    const long long items = has_pred + sinks;
    for (long long it = grp; it < items; it += kGroups) {  // the same bounds for a group's lanes
      long long a0, a1;
      bool whole;
      int v;
      if (it < has_pred) {
        a0 = pstart;
        a1 = pend;
        whole = false;
        v = wv[0];
      } else {
        const long long q = it - has_pred;  // sink jf + q: window entries q + 1 and q + 2
        long long a, b;
        if (q + 2 < kWave) {
          a = wb[q + 1];
          b = wb[q + 2];
          v = wv[q + 1];
        } else {
          a = boff[jf + q];
          b = boff[jf + q + 1];
          v = list[jf + q];
        }
        a0 = a;
        whole = b - a <= kBucketSeg;
        a1 = whole ? b : a + kBucketSeg;
      }
      const int na = static_cast<int>(a1 - a0);  // slots in the segment (<= kBucketSeg)
      if (na == 0) continue;                      // no message reached the sink (the same for the group)
      float *sv = S + static_cast<long long>(v) * d;
      // the row's current values, loaded with the message rows (used when the
      // bucket is one segment)
      float prev[NC];
#pragma unroll
      for (int p = 0; p < NC; ++p) prev[p] = sv[k0 + p * G];  // past d: the next row or the tail (never used)
      const int o0 = static_cast<int>(a0 - R0);  // the segment's first slot in the window
      float acc[NC];
#pragma unroll
      for (int p = 0; p < NC; ++p) acc[p] = 0.0f;
#pragma unroll
      for (int st = 0; st < kSteps; ++st) {
        if (st * U >= na) break;  // the same for the group's lanes
        // every lane loads (a slot past the segment repeats its last one, a column
        // past the end reads the next row or the tail) and the value is masked to
        // zero afterwards: the loads carry no branch and go out together
        float row[U][NC];
        float cc[U];
#pragma unroll
        for (int t = 0; t < U; ++t) {
          const int i = st * U + t;
          const int o = o0 + (i < na ? i : na - 1);
          const float *su = msg + static_cast<long long>(wu[o]) * ld + k0;
          cc[t] = weighted ? ww[o] : 1.0f;
          const unsigned keep = i < na ? ~0u : 0u;
#pragma unroll
          for (int p = 0; p < NC; ++p) row[t][p] = __uint_as_float(__float_as_uint(su[p * G]) & keep);
        }
#pragma unroll
        for (int t = 0; t < U; ++t)
#pragma unroll
          for (int p = 0; p < NC; ++p) acc[p] += cc[t] * row[t][p];
      }
#pragma unroll
      for (int p = 0; p < NC; ++p) {
        const int k = k0 + p * G;
        if (k < d) {
          if (whole) sv[k] = prev[p] + acc[p];
          else unsafeAtomicAdd(&sv[k], acc[p]);
        }
      }
    }
    jf = jl + 1;
  }
}

// Four floats at a 4-byte aligned address (one 16-byte access).
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));

// The pulls: for every sink v of a list (or all vertices), the sum over its in-arcs
// (u -> v) of rows of a table. MSG: the message rows of those sources that are dirty
// (member bit of u; a message row's place is u's rank among the members), added to
// S[v]; else every source's row (the bootstrap and the recompute form), summed in
// fp64 and stored as S[v]. A wave per sink. A row takes the fewest lanes
// that cover it at four floats each (G lanes, NC spans of 4 G floats), the wave's
// groups take arcs round robin, U rows of each in flight; of 64 in-arcs the dirty
// ones are first moved to the front, so that only message rows are loaded. The sinks
// ahead are prefetched: while this sink's rows arrive, the next one's member words
// (or out-degrees), the arcs of the one after, the row bounds of the third and the id
// of the fourth are in flight. Sinks of more than long_from in-arcs go to k_pull_long.
// Bound by the row reads that leave the L2s, 128 bytes at a time (a 47-wide row, 192
// bytes, costs 256; 6.2 TB/s of them on dense_large's third layer). The message pull
// there took 3.83 ms at batch 100 and 4.85 at batch 1000 when its lane groups loaded 4
// bytes per lane, walked windows of 64 arcs with the non-member arcs in place, and
// flushed with atomics; now 3.1 and 4.5; on the 3-layer mean workload at batch 1000
// (256 wide) 73 us, now 59; RMAT 2^20 at batch 2500 (64 wide) 1.05 ms, now 0.92; but RMAT
// 2^23 at batch 10000, where most sinks have few in-arcs, 8.7 ms and now 9.1; the
// bootstrap of dense_large 60, 30 and 15.6 ms for rows 256, 100 and 47 wide with one
// load of 4 bytes per lane in flight per wave, now 18.2, 8.8 and 5.2. Non-temporal row
// loads took the batch 100 pull from 2.4 to 3.9 ms (its short rows).
struct Sink {
  int v, deg;  // v < 0: none
  long long off;
};
// 64 in-arcs of a sink, one per lane (u < 0: none)
struct Arcs {
  int u;
  float w;
  uint2 aux;  // MSG: u's member word and the members before it; GCN: u's out-degree
};

template <bool MSG>
struct Puller {
  const PullArgs &p;
  int lane;
  __device__ Sink bounds(int v) const {
    if (v < 0) return Sink{-1, 0, 0};
    return Sink{v, p.in.len[v], p.in.off[v]};
  }
  __device__ Arcs arcs(long long e, int cnt) const {
    Arcs a{-1, 1.0f, make_uint2(0u, 0u)};
    if (lane < cnt) {
      a.u = __builtin_nontemporal_load(p.in.col + e + lane);
      if (p.in.wt != nullptr) a.w = __builtin_nontemporal_load(p.in.wt + e + lane);
    }
    return a;
  }
  __device__ void look_up(Arcs &a) const {
    if (a.u < 0) return;
    if (MSG) a.aux = p.memb[a.u >> 5];
    else if (p.gcn) a.aux.x = static_cast<unsigned>(p.out_len[a.u]);
  }
  // The arcs that carry a row, moved to lanes 0 .. cnt-1: the row's index (u on entry)
  // and coefficient.
  __device__ int resolve(Arcs &a, int cnt, double &coef) const {
    coef = static_cast<double>(a.w);
    if (!MSG) {
      if (p.gcn) coef *= 1.0 / sqrt(static_cast<double>(static_cast<int>(a.aux.x)) + 1.0);
      return cnt;
    }
    const unsigned bit = 1u << (a.u & 31);
    const bool on = a.u >= 0 && (a.aux.x & bit) != 0;
    const u64 m = __ballot(on);
    const int n = __popcll(m);
    const int below = lanes_below(m);
    const int to = (on ? below : n + lane - below) << 2;  // a permutation of the lanes
    a.u = __builtin_amdgcn_ds_permute(to, static_cast<int>(a.aux.y) + __popc(a.aux.x & (bit - 1u)));
    if (p.in.wt != nullptr)
      coef = static_cast<double>(__int_as_float(__builtin_amdgcn_ds_permute(to, __float_as_int(a.w))));
    return n;
  }
};

// Messages are summed in fp32, at most 256 in a row: by groups of up to 16 lanes, a
// sink's (1024 among 4 groups or more); by 32 or 64 lanes, those of 64 in-arcs, whose
// sums are then added up (at most 16); and of a row that a block sums those of 64
// in-arcs, whose sums are added up in fp64. (With one fp32 sum per group throughout, a
// hub of 60,000 equal messages was off by 2965 units of 2^-24 of the sum at 256 wide and
// 556 at 64, and 1024 messages at 256 wide by 144; now 8, 2 and 10.) Whole aggregates are
// summed in fp64.
template <bool MSG>
using PullAcc = typename std::conditional<MSG, float, double>::type;

// acc += arcs [i0, i0 + U * (groups)) of the wave, as far as cnt unless FULL says they
// are all there (lane i holds arc i). An arc past cnt repeats the last one, masked to
// zero; lanes past the row's width read its first columns.
template <int G, int NC, int U, bool COEF, bool FULL, typename T>
__device__ inline void pull_step(const PullArgs &p, int idx, double coef, int i0, int cnt, int k0, T (&acc)[NC][4]) {
  constexpr int kGroups = kWave / G;
  const int grp = (threadIdx.x & (kWave - 1)) / G;
  float4u row[U][NC];
  T cf[U];
#pragma unroll
  for (int t = 0; t < U; ++t) {
    const int i = i0 + t * kGroups + grp;
    const int ii = FULL || i < cnt ? i : cnt - 1;
    const int u = G == kWave ? __builtin_amdgcn_readlane(idx, ii) : __shfl(idx, ii);
    if (COEF) cf[t] = static_cast<T>(__shfl(coef, ii));
    const float *h = p.src + static_cast<long long>(u) * p.ld;
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      const int k = k0 + 4 * G * q;
      row[t][q] = *reinterpret_cast<const float4u *>(h + (k < p.d ? k : 0));
    }
  }
#pragma unroll
  for (int t = 0; t < U; ++t) {
    const unsigned keep = FULL || i0 + t * kGroups + grp < cnt ? ~0u : 0u;
#pragma unroll
    for (int q = 0; q < NC; ++q)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float x = FULL ? row[t][q][j] : __uint_as_float(__float_as_uint(row[t][q][j]) & keep);
        acc[q][j] += COEF ? cf[t] * static_cast<T>(x) : static_cast<T>(x);
      }
  }
}

// The wave's arcs [0, cnt) in full steps of U rows per group and the shortest step
// that covers the rest.
template <int G, int NC, int U, bool COEF, typename T>
__device__ inline void pull_rows(const PullArgs &p, int idx, double coef, int cnt, int k0, T (&acc)[NC][4]) {
  constexpr int kGroups = kWave / G;
  for (int i0 = 0; i0 < cnt; i0 += kGroups * U) {
    const int rest = cnt - i0;
    if (rest >= kGroups * U) pull_step<G, NC, U, COEF, true>(p, idx, coef, i0, cnt, k0, acc);
    else if (rest <= kGroups * (U / 4)) pull_step<G, NC, U / 4, COEF, false>(p, idx, coef, i0, cnt, k0, acc);
    else if (rest <= kGroups * (U / 2)) pull_step<G, NC, U / 2, COEF, false>(p, idx, coef, i0, cnt, k0, acc);
    else pull_step<G, NC, U, COEF, false>(p, idx, coef, i0, cnt, k0, acc);
  }
}

// Sums over the wave's groups, left in every group's lanes.
template <int G, int NC, typename T>
__device__ inline void pull_reduce(T (&acc)[NC][4]) {
#pragma unroll
  for (int s = G; s < kWave; s <<= 1)
#pragma unroll
    for (int q = 0; q < NC; ++q)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[q][j] += __shfl_xor(acc[q][j], s);
}

// S[v] (row sv) = acc, or with MSG the row it held (prev) plus acc.
template <int G, int NC, bool MSG>
__device__ inline void pull_store(float *sv, int d, int k0, const PullAcc<MSG> (&acc)[NC][4],
                                  const float4u (&prev)[NC]) {
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int k = k0 + 4 * G * q;
    float4u r;
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] = MSG ? prev[q][j] + static_cast<float>(acc[q][j]) : static_cast<float>(acc[q][j]);
    if (k + 4 <= d) {
      *reinterpret_cast<float4u *>(sv + k) = r;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (k + j < d) sv[k + j] = r[j];
    }
  }
}

constexpr int kPullWaves = 256 / kWave;

// A long in-row (more than kPullLong arcs) summed by the whole block: its waves take
// chunks of 64 arcs round robin, and their sums are added up in fp64 through LDS in
// wave order. (With one wave per row the bootstrap of RMAT, 2^20 vertices and 64 wide,
// waited on its hubs for 17.3 ms; now 1.2. In a launch of their own the long rows took
// 26 us of a 98,765-vertex graph's pull; here the other sinks hide them.)
template <int G, int NC, int U, bool MSG, bool COEF>
__device__ inline void pull_long(const PullArgs &p, const Puller<MSG> &pl, const Sink &s, int k0,
                                 double (*part)[4 * G * NC], int *messages) {
  const int lane = pl.lane, wave = threadIdx.x / kWave;
  const int deg = __builtin_amdgcn_readfirstlane(s.deg);
  double sum[NC][4] = {};
  int found = 0;
  constexpr int kStep = kPullWaves * kWave;
  int e0 = __builtin_amdgcn_readfirstlane(wave * kWave);
  Arcs a = pl.arcs(s.off + e0, deg - e0 < kWave ? deg - e0 : kWave);
  pl.look_up(a);
  for (; e0 < deg; e0 += kStep) {
    const int more = deg - e0 - kStep;
    Arcs b = a;
    if (more > 0) b = pl.arcs(s.off + e0 + kStep, more < kWave ? more : kWave);
    double coef;
    const int cnt = pl.resolve(a, deg - e0 < kWave ? deg - e0 : kWave, coef);
    found += cnt;
    if constexpr (MSG) {
      float acc[NC][4] = {};
      pull_rows<G, NC, U, COEF>(p, a.u, coef, cnt, k0, acc);
#pragma unroll
      for (int q = 0; q < NC; ++q)
#pragma unroll
        for (int j = 0; j < 4; ++j) sum[q][j] += static_cast<double>(acc[q][j]);
    } else {
      pull_rows<G, NC, U, COEF>(p, a.u, coef, cnt, k0, sum);
    }
    if (more > 0) pl.look_up(b);
    a = b;
  }
  pull_reduce<G, NC>(sum);
  if (lane < G) {
#pragma unroll
    for (int q = 0; q < NC; ++q)
#pragma unroll
      for (int j = 0; j < 4; ++j) part[wave][k0 + 4 * G * q + j] = sum[q][j];
  }
  if (lane == 0) messages[wave] = found;
  __syncthreads();
  int total = 0;
#pragma unroll
  for (int w = 0; w < kPullWaves; ++w) total += messages[w];
  if (total > 0) {  // (a long row has arcs: without MSG always)
    float *sv = p.S + static_cast<long long>(s.v) * p.d;
    for (int k = threadIdx.x; k < p.d; k += kPullWaves * kWave) {
      double row = MSG ? static_cast<double>(sv[k]) : 0.0;
#pragma unroll
      for (int w = 0; w < kPullWaves; ++w) row += part[w][k];
      sv[k] = static_cast<float>(row);
    }
    if (MSG && p.mark != nullptr && threadIdx.x == 0) mark_only(p.mark, s.v);
  }
  __syncthreads();
}

template <int G, int NC, int U, bool MSG, bool COEF>
__device__ inline void pull_body(const PullArgs &p) {
  __shared__ double part[kPullWaves][4 * G * NC];
  __shared__ int messages[kPullWaves];
  const long long nlong = p.nlong != nullptr ? static_cast<long long>(*p.nlong) : 0;
  long long M = p.n;
  if (p.count != nullptr) M = static_cast<long long>(*p.count);
  if (p.c != nullptr && aborted_with(p.c->abort, M, nlong)) return;
  const int lane = lane_id();
  const int k0 = 4 * (lane % G);
  const Puller<MSG> pl{p, lane};
  for (long long r = blockIdx.x; r < nlong; r += gridDim.x)
    pull_long<G, NC, U, MSG, COEF>(p, pl, pl.bounds(p.longs[r]), k0, part, messages);
  const int long_from = p.nlong != nullptr ? kPullLong : INT32_MAX;
  // the blocks with the fewest long rows take the first sinks
  const long long step = num_waves();
  long long j = step - 1 - global_wave();
  if (j >= M) return;
  const auto vertex = [&](long long i) { return i < M ? (p.list != nullptr ? p.list[i] : static_cast<int>(i)) : -1; };
  const auto first_arcs = [&](const Sink &s) { return pl.arcs(s.off, s.deg < kWave ? s.deg : kWave); };
  const int va = vertex(j), vb = vertex(j + step), vc = vertex(j + 2 * step);
  int v3 = vertex(j + 3 * step);
  Sink s0 = pl.bounds(va), s1 = pl.bounds(vb), s2 = pl.bounds(vc);
  Arcs a0 = first_arcs(s0), a1 = first_arcs(s1);
  pl.look_up(a0);
  for (; j < M; j += step) {
    Arcs a1n = a1;
    pl.look_up(a1n);
    const Arcs a2 = first_arcs(s2);
    const Sink s3 = pl.bounds(v3);
    v3 = vertex(j + 4 * step);
    const int v = __builtin_amdgcn_readfirstlane(s0.v), deg = __builtin_amdgcn_readfirstlane(s0.deg);
    if (deg <= long_from) {
      PullAcc<MSG> acc[NC][4] = {};
      // The sink's row, which comes with its first messages; where the sums of 64s are
      // folded, those first (both at once cost a wave per SIMD) and the row last.
      float4u prev[NC] = {};
      const bool fold = MSG && G >= 32 && deg > kWave;
      float *sv = p.S + static_cast<long long>(v) * p.d;
      const auto load_prev = [&] {
#pragma unroll
        for (int q = 0; q < NC; ++q) {
          const int k = k0 + 4 * G * q;
          prev[q] = *reinterpret_cast<const float4u *>(sv + (k < p.d ? k : 0));
        }
      };
      bool any = false;
      Arcs a = a0;
      for (int e0 = 0; e0 < deg; e0 += kWave) {
        const int more = deg - e0 - kWave;  // arcs after these
        Arcs b = a;
        if (more > 0) b = pl.arcs(s0.off + e0 + kWave, more < kWave ? more : kWave);
        double coef;
        const int cnt = pl.resolve(a, deg - e0 < kWave ? deg - e0 : kWave, coef);
        if (MSG && cnt > 0 && !any) {
          any = true;
          if (!fold) load_prev();
        }
        pull_rows<G, NC, U, COEF>(p, a.u, coef, cnt, k0, acc);
        if (fold) {
#pragma unroll
          for (int q = 0; q < NC; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              prev[q][j] += static_cast<float>(acc[q][j]);
              acc[q][j] = 0;
            }
        }
        if (more > 0) pl.look_up(b);
        a = b;
      }
      if (!MSG || any) {
        if (fold) {
#pragma unroll
          for (int q = 0; q < NC; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[q][j] = prev[q][j];
          load_prev();
        }
        pull_reduce<G, NC>(acc);
        if (lane < G) pull_store<G, NC, MSG>(sv, p.d, k0, acc, prev);
        if (MSG && p.mark != nullptr && lane == 0) mark_only(p.mark, v);
      }
    }
    s0 = s1;
    s1 = s2;
    s2 = s3;
    a0 = a1n;
    a1 = a2;
  }
}

// The bootstrap's pull, the recompute form's and the message pulls (names of their own
// in a kernel trace).
template <int G, int NC, int U, bool COEF>
__global__ __launch_bounds__(256) void k_pull(PullArgs p) {
  pull_body<G, NC, U, false, COEF>(p);
}
template <int G, int NC, int U, bool COEF>
__global__ __launch_bounds__(256) void k_recompute(PullArgs p) {
  pull_body<G, NC, U, false, COEF>(p);
}
// (At 65 to 96 and 129 to 192 columns four waves per SIMD fit, by a register or three. A
// batch of 1000 on 300,000 vertices and 12M arcs with dense layers 80 wide: 658 us, now
// 584; 160 wide, with its fp64 sums of long rows, 680 and 702; 100 wide 555 and 567.)
template <int G, int NC, int U, bool COEF>
__global__ __launch_bounds__(256, NC == 3 && !COEF ? 4 : 1) void k_pull_msgs(PullArgs p) {
  pull_body<G, NC, U, true, COEF>(p);
}

// The vertices of more than kPullLong in-arcs. A block counts those of its share, then
// takes their places with one atomic (one per wave took 131 us on dense_large, whose
// some 20K long rows are spread over as many waves).
__global__ __launch_bounds__(1024) void k_list_long(long long n, const int *in_len, int *longs, u64 *nlong,
                                                    const Counters *c) {
  if (c != nullptr && c->abort) return;
  __shared__ int count, place;
  __shared__ u64 base;
  if (threadIdx.x == 0) count = place = 0;
  __syncthreads();
  const long long per = (n + gridDim.x - 1) / gridDim.x;
  const long long v0 = blockIdx.x * per, v1 = v0 + per < n ? v0 + per : n;
  int mine = 0;
  for (long long v = v0 + threadIdx.x; v < v1; v += blockDim.x) mine += in_len[v] > kPullLong ? 1 : 0;
  if (mine > 0) atomicAdd(&count, mine);
  __syncthreads();
  if (count == 0) return;  // the same for the whole block
  if (threadIdx.x == 0) base = atomicAdd(nlong, static_cast<u64>(count));
  __syncthreads();
  if (mine == 0) return;
  for (long long v = v0 + threadIdx.x; v < v1; v += blockDim.x)
    if (in_len[v] > kPullLong) longs[base + atomicAdd(&place, 1)] = static_cast<int>(v);
}

__global__ void k_fill_i32(int *p, long long count, int value) {
  const long long stride = static_cast<long long>(gridDim.x) * blockDim.x;
  for (long long i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) p[i] = value;
}

__global__ void k_fill_u64(u64 *p, long long count, u64 value) {
  const long long stride = static_cast<long long>(gridDim.x) * blockDim.x;
  for (long long i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) p[i] = value;
}

__global__ void k_copy_i32(const int *src, long long count, int *out) {
  const long long stride = static_cast<long long>(gridDim.x) * blockDim.x;
  for (long long i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) out[i] = src[i];
}

__global__ void k_gather_rows(const float *src, int d, const int *ids, long long count, float *out) {
  const long long total = count * d;
  const long long stride = static_cast<long long>(gridDim.x) * blockDim.x;
  for (long long i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
    const long long r = i / d;
    const int k = static_cast<int>(i % d);
    out[i] = src[static_cast<long long>(ids[r]) * d + k];
  }
}

}  // namespace

void launch_corr_mark(hipStream_t s, int cap_feat, int cap_arcs, int agg, LayerPtrs lp, Adj out, Adj in,
                      const int *ins_rank, const float *arc_w, const int *ddeg, const int *flist, const int *ins_src,
                      const int *ins_dst, const int *del_src, const int *del_dst, const float *ins_w,
                      const float *del_w, unsigned *bm, Counters *c, const DirectList &direct) {
  const long long waves = 2LL * cap_arcs * lp.L;
  const long long threads = static_cast<long long>(cap_feat) + 2LL * cap_arcs;
  const long long items = waves * kWave > threads ? waves * kWave : threads;
  RP_LAUNCH(k_corr_mark, dim3(blocks_for(items, 256)), dim3(256), 0, s, agg, lp, out, in, ins_rank, arc_w,
                     ddeg, flist, ins_src, ins_dst, del_src, del_dst, ins_w, del_w, bm, c, direct);
}

int compact_blocks(long long n) {
  const long long t = tile_vertices(n);
  return static_cast<int>((n + t - 1) / t);
}

long long bucket_counter_slots(long long n) { return static_cast<long long>(compact_blocks(n)) * tile_vertices(n); }

void launch_compact(hipStream_t s, long long n, unsigned *bm_a, unsigned *bm_b, const CompactScratch &cs,
                    const CompactOut &o) {
  const int tiles = compact_blocks(n);
  u64 *inc = cs.words + static_cast<long long>(tiles) * kVals, *ticket = cs.words + 2LL * tiles * kVals;
#define RP_COMPACT(VV, BK) \
  RP_LAUNCH((k_compact<VV, BK>), dim3(tiles), dim3(kCompactThreads), 0, s, bm_a, bm_b, n, o, cs.words, inc, ticket, cs.err)
  const bool small = tile_vertices(n) == kTileSmall;
  if (o.bkt_cnt != nullptr) {
    if (small) RP_COMPACT(8, true);
    else RP_COMPACT(16, true);
  } else {
    if (small) RP_COMPACT(8, false);
    else RP_COMPACT(16, false);
  }
#undef RP_COMPACT
}

void launch_delta0(hipStream_t s, long long n, const Delta0Args &z, const int *list, const u64 *count) {
  RP_LAUNCH(k_delta0, dim3(blocks_for(n * kWave, 256, 2048)), dim3(256), 0, s, z, list, count, n);
}

long long compact_scratch_words(long long n) { return 2LL * compact_blocks(n) * kVals + 1; }

void launch_scatter(hipStream_t s, long long n, int d, int ld, const int *list, const u64 *count, const long long *doff,
                    const float *delta, Adj out, float *S, unsigned *bm_out, unsigned *bm_x, const int *ins_dst,
                    const int *del_dst, const u64 *pushed, const Counters *c, bool push, bool mark_list,
                    const ScatterCopy &copy, const ScatterList &lo, bool packed_in) {
  const int blocks = 2048;
#define RP_SCATTER_L(GV, NCV, P, LV)                                                                               \
  RP_LAUNCH((k_scatter<GV, NCV, P, LV>), dim3(blocks), dim3(256), 0, s, d, ld, list, count, doff, delta, out, \
                     S, bm_out, bm_x, ins_dst, del_dst, pushed, c, mark_list ? 1 : 0, copy, lo, packed_in ? 1 : 0)
#define RP_SCATTER(GV, NCV, P)                \
  do {                                        \
    if (P && lo.list != nullptr)              \
      RP_SCATTER_L(GV, NCV, P, P);            \
    else                                      \
      RP_SCATTER_L(GV, NCV, P, false);        \
  } while (0)
  if (!push) RP_SCATTER(64, 1, false);
  else if (d <= 16) RP_SCATTER(16, 1, true);
  else if (d <= 32) RP_SCATTER(32, 1, true);
  else if (d <= 64) RP_SCATTER(64, 1, true);
  else if (d <= 128) RP_SCATTER(64, 2, true);
  else if (d <= 256) RP_SCATTER(64, 4, true);
  else if (d <= 512) RP_SCATTER(64, 8, true);
  else RP_SCATTER(64, 16, true);
#undef RP_SCATTER
#undef RP_SCATTER_L
}

int bin_shift(long long n) {
  // bins of 8192 sinks (few enough bins that the scatter's runs into them combine
  // in L2), at most kMaxBins of them
  const int s = 13;
  return (n + (1LL << s) - 1) >> s <= kMaxBins ? s : -1;
}

void launch_bin_count(hipStream_t s, const int *list, const u64 *count, const long long *doff, Adj out,
                      const u64 *pushed, const Buckets &b, unsigned *bm_x, const int *ins_dst, const int *del_dst,
                      bool mark_list, const Counters *c) {
  RP_LAUNCH(k_bin_arcs<false>, dim3(kBinBlocks), dim3(kBinThreads), b.nbins * sizeof(int), s, list, count, doff, out,
            pushed, b, bm_x, ins_dst, del_dst, mark_list ? 1 : 0, c);
}

void launch_bin_scatter(hipStream_t s, const int *list, const u64 *count, const long long *doff, Adj out,
                        const u64 *pushed, const Buckets &b, const Counters *c) {
  RP_LAUNCH(k_bin_arcs<true>, dim3(kBinBlocks), dim3(kBinThreads), b.nbins * sizeof(int), s, list, count, doff, out,
            pushed, b, nullptr, nullptr, nullptr, 0, c);
}

void launch_bin_sort(hipStream_t s, long long n, const u64 *pushed, const Buckets &b, const Counters *c) {
  RP_LAUNCH(k_bin_sort, dim3(static_cast<unsigned>(b.nbins)), dim3(kBinThreads), (sizeof(int) << b.shift), s, n,
            pushed, b, c);
}

// (G, NC, U) by row width: lane groups of 16 up to 64 columns, whole waves above
#define RP_BY_WIDTH(M)                                                                                         \
  do {                                                                                                         \
    if (d <= 16) M(16, 1, 8);                                                                                  \
    else if (d <= 32) M(16, 2, 8);                                                                             \
    else if (d <= 48) M(16, 3, 8);                                                                             \
    else if (d <= 64) M(16, 4, 8);                                                                             \
    else if (d <= 128) M(64, 2, 8);                                                                            \
    else if (d <= 256) M(64, 4, 8);                                                                            \
    else if (d <= 512) M(64, 8, 4);                                                                            \
    else M(64, 16, 2);                                                                                         \
  } while (0)

// Rows per step of the bucket sums: whole-wave groups (rows over 64 wide) take at
// most four, since a bucket holds a handful of slots and the masked rows of a step
// of eight reload a 1 KB row (1% on dense_large's 256-wide second layer); 16-lane
// groups keep eight (with four, buckets of 5-8 slots cost a second round trip).
constexpr int bucket_rows_per_step(int g, int u) { return g == kWave && u > 4 ? 4 : u; }

void launch_bucket_sum(hipStream_t s, int d, int ld, const int *list, const u64 *count, const long long *boff,
                       const Buckets &bk, const float *msg, float *S, const Counters *c) {
  const int blocks = 2048;
#define RP_BSUM(GV, NCV, UV)                                                                                     \
  RP_LAUNCH((k_bucket_sum<GV, NCV, bucket_rows_per_step(GV, UV)>), dim3(blocks), dim3(256), 0, s, d, ld, list,    \
            count, boff, bk, msg, S, c)
  RP_BY_WIDTH(RP_BSUM);
#undef RP_BSUM
}
#undef RP_BY_WIDTH

namespace {

template <bool COEF>
void pull_by_width(hipStream_t s, const PullArgs &a) {
  const int blocks = blocks_for(a.n * kWave, 256, 2048);
#define RP_PULL(GV, NCV, UV)                                                                                     \
  do {                                                                                                           \
    if (a.memb != nullptr) RP_LAUNCH((k_pull_msgs<GV, NCV, UV, COEF>), dim3(blocks), dim3(256), 0, s, a);        \
    else if (a.list != nullptr) RP_LAUNCH((k_recompute<GV, NCV, UV, COEF>), dim3(blocks), dim3(256), 0, s, a);   \
    else RP_LAUNCH((k_pull<GV, NCV, UV, COEF>), dim3(blocks), dim3(256), 0, s, a);                               \
  } while (0)
  // the lane groups that cover a row with the fewest idle lanes
  const int d = a.d;
  if (d <= 16) RP_PULL(4, 1, 4);
  else if (d <= 32) RP_PULL(8, 1, 8);
  else if (d <= 64) RP_PULL(16, 1, 8);
  else if (d <= 96) RP_PULL(8, 3, 4);
  else if (d <= 128) RP_PULL(32, 1, 8);
  else if (d <= 192) RP_PULL(16, 3, 4);
  else if (d <= 256) RP_PULL(64, 1, 8);
  else if (d <= 512) RP_PULL(64, 2, 4);
  else RP_PULL(64, 4, 4);
#undef RP_PULL
}

}  // namespace

void launch_list_long(hipStream_t s, long long n, const int *in_len, int *longs, u64 *nlong, const Counters *c) {
  RP_LAUNCH(k_list_long, dim3(blocks_for(n, 4096, 512)), dim3(1024), 0, s, n, in_len, longs, nlong, c);
}

void launch_pull(hipStream_t s, const PullArgs &args) {
  PullArgs a = args;
  if (a.memb != nullptr) a.gcn = 0;  // the message rows carry the coefficients
  if (a.gcn || a.in.wt != nullptr) pull_by_width<true>(s, a);
  else pull_by_width<false>(s, a);
}

void launch_fill_i32(hipStream_t s, int *p, long long count, int value) {
  if (count <= 0) return;
  RP_LAUNCH(k_fill_i32, dim3(blocks_for(count, 256)), dim3(256), 0, s, p, count, value);
}

void launch_fill_u64(hipStream_t s, u64 *p, long long count, u64 value) {
  if (count <= 0) return;
  RP_LAUNCH(k_fill_u64, dim3(blocks_for(count, 256)), dim3(256), 0, s, p, count, value);
}

void launch_copy_i32(hipStream_t s, const int *src, long long count, int *out) {
  if (count <= 0) return;
  RP_LAUNCH(k_copy_i32, dim3(blocks_for(count, 256, 1024)), dim3(256), 0, s, src, count, out);
}

void launch_gather_rows(hipStream_t s, const float *src, int d, const int *ids, long long count, float *out) {
  if (count <= 0) return;
  RP_LAUNCH(k_gather_rows, dim3(blocks_for(count * d, 256)), dim3(256), 0, s, src, d, ids, count, out);
}

}  // namespace rp
