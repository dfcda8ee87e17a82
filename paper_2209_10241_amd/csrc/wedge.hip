// Triangles, 4-cycles and 4-cliques of the pairwise graph without adjacency
// bit rows: the counts behind the graph identities of the exact count
// (sparse.hip) and the per-pair statistics of the pair sampler.
//
// The nodes are ranked by degree (x before y: fewer pairwise neighbours, or
// as many in the same class of degrees) and the graph is kept once more in
// rank space, without the neighbours of degree 1, which close nothing (the
// core rows).  Every pair {x, u}, x before u, is walked from its later node
// u: one workgroup takes u, marks N(u) in LDS, and for each neighbour x
// before u walks the row of x.  A node w met there closes a triangle when it
// is marked, and, when w is before u, one more path u - x - w, counted per w
// in LDS: c such paths close C(c, 2) 4-cycles whose last node is u.  So the
// membership tests and the path counters are LDS operations, where a hash
// probe per position and a sort of one key per path went to memory before.
// Triangles and 4-cycles together: co-authorship (N = 10^6, 2 x 10^7
// positions) 3.8 -> 1.1 ms, communication (N = 5 x 10^4, 1.3 x 10^8
// positions) 14.0 -> 1.0 ms; 4-cliques 1.0 -> 0.16 and 6.4 -> 0.74 ms.
//
// The longest walks are split by the neighbours x into shares on several CUs,
// whose counters are summed by another launch.
//
// u is taken by the size of its walk: a wavefront with a hash table of 1,024
// slots (degree below 24), a workgroup of 256 threads with 4,096 slots (at
// most 3,072 nodes marked and met), or one of 1,024 threads with counters
// addressed by rank, a range of ranks at a time.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "hm_sparse.h"
#include "hm_wedge.h"

namespace hm {
namespace {

// ------------------------------------------------------------------ rank space
constexpr uint32_t kSmallDeg = 24;        // degrees below: one wavefront a node
constexpr uint32_t kSmallSlots = 1024;    // 23 x 23 paths and 23 neighbours: load at most 0.54
constexpr uint32_t kMidSlots = 4096;
constexpr uint32_t kMidMost = 3072;
constexpr uint32_t kRankBits = 8;
constexpr uint32_t kNarrowDeg = 16;       // degrees below: path counts of 4 bits

// Class of a degree: itself below 64, then eight classes per octave.
__device__ inline uint32_t degree_class(uint32_t d) {
  if (d < 64) return d;
  const uint32_t e = 31 - __clz(int(d));
  return min(255u, 64 + 8 * (e - 6) + ((d >> (e - 3)) & 7u));
}

// Graph in rank space: node ranks, core rows and, in them, the later
// neighbours alone (out rows).
struct Ranked {
  uint32_t n;                // nodes
  const uint32_t* rank_of;   // node -> rank
  const uint32_t* node_of;   // rank -> node
  const uint2* core;         // rank -> (first entry, entries) of the core row
  const uint2* out;          // rank -> the same of the out row
  const uint32_t* core_adj;  // ranks
  const uint32_t* core_eid;  // position in e2 of the entry's pair
  const uint32_t* out_adj;
  const uint32_t* out_eid;
  const uint32_t* degree;    // rank -> degree
  const uint32_t* weight;    // rank -> bound on the nodes marked and positions walked (degree >= kSmallDeg)
  const uint32_t* bounds;    // first rank of degree >= 2, of degree >= kSmallDeg, of degree >= 16
  const uint32_t* facts;     // kLongestOut ..
};

// Words of Ranked::facts: the longest out row, the nodes with more than
// 65,535 core neighbours, the split walks' nodes and shares, and the core
// rows' entries.
enum : int { kLongestOut = 0, kManyCore = 1, kSplitNodes = 2, kSplitShares = 3, kCoreEntries = 4, kFacts = 5 };

__global__ void k_rank_keys(const uint32_t* __restrict__ g2_off, uint32_t n, uint32_t* __restrict__ keys,
                            uint32_t* __restrict__ vals, uint32_t* __restrict__ bounds) {
  if (blockIdx.x == 0 && threadIdx.x < 3) bounds[threadIdx.x] = n;
  for (uint64_t x = blockIdx.x * blockDim.x + threadIdx.x; x < n; x += gridDim.x * blockDim.x) {
    keys[x] = degree_class(g2_off[x + 1] - g2_off[x]);
    vals[x] = uint32_t(x);
  }
}

__global__ void k_rank_assign(const uint32_t* __restrict__ keys, const uint32_t* __restrict__ node_of,
                              uint32_t n, uint32_t* __restrict__ rank_of, uint32_t* __restrict__ bounds) {
  for (uint64_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const uint32_t r = uint32_t(i);
    rank_of[node_of[r]] = r;
    const uint32_t k = keys[r], before = r ? keys[r - 1] : 0u;
    if (k >= 2 && (r == 0 || before < 2)) bounds[0] = r;
    if (k >= kSmallDeg && (r == 0 || before < kSmallDeg)) bounds[1] = r;
    if (k >= kNarrowDeg && (r == 0 || before < kNarrowDeg)) bounds[2] = r;
  }
}

// Per adjacency entry: whether it is in the core rows (low half) and in the
// out rows (high half), for one scan of both.  And per rank u (weight, zero
// before) a bound on what its walk marks and walks: its degree and the
// degrees of its neighbours before it.  A wavefront takes 64 consecutive
// entries, sums them by row with a segmented scan and adds once per row (a
// wavefront per row left the longest row, 1.1e5 entries, as a tail of 0.2 ms).
__global__ void k_core_flags(const uint32_t* __restrict__ g2_off, const uint32_t* __restrict__ g2_adj,
                             const uint32_t* __restrict__ g2_eid, const uint32_t* __restrict__ e2, uint64_t m,
                             const uint32_t* __restrict__ rank_of, const uint32_t* __restrict__ bounds,
                             unsigned long long* __restrict__ flag, uint32_t* __restrict__ weight) {
  const uint32_t r0 = bounds[0], r1 = bounds[1];
  const uint32_t lane = threadIdx.x & (kWave - 1);
  for (uint64_t base = (uint64_t(blockIdx.x) * blockDim.x + threadIdx.x) & ~uint64_t(kWave - 1); base < m;
       base += uint64_t(gridDim.x) * blockDim.x) {
    const uint64_t i = base + lane;
    uint32_t ro = kEmpty32, d = 0;
    if (i < m) {
      const uint32_t z = g2_adj[i];
      const uint64_t e = g2_eid[i];
      ro = rank_of[e2[2 * e] ^ e2[2 * e + 1] ^ z];
      const uint32_t rz = rank_of[z];
      flag[i] = rz >= r0 ? (1ull | ((unsigned long long)(rz > ro) << 32)) : 0ull;
      d = 1 + (rz < ro && ro >= r1 ? g2_off[z + 1] - g2_off[z] : 0u);
    }
    for (int s = 1; s < kWave; s <<= 1) {
      const uint32_t o = uint32_t(__shfl_up(int(ro), s, kWave)), dd = uint32_t(__shfl_up(int(d), s, kWave));
      if (int(lane) >= s && o == ro) d += dd;   // (a row's entries are consecutive)
    }
    const uint32_t after = uint32_t(__shfl_down(int(ro), 1, kWave));
    // (degrees add up to at most 2 |E2|, below 2^32)
    if (i < m && ro >= r1 && (lane == kWave - 1 || after != ro)) atomicAdd(&weight[ro], d);
  }
}

__global__ void k_core_fill(const uint32_t* __restrict__ g2_adj, const uint32_t* __restrict__ g2_eid, uint64_t m,
                            const uint32_t* __restrict__ rank_of, const unsigned long long* __restrict__ flag,
                            const unsigned long long* __restrict__ pos, uint32_t* __restrict__ core_adj,
                            uint32_t* __restrict__ core_eid, uint32_t* __restrict__ out_adj,
                            uint32_t* __restrict__ out_eid) {
  for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < m; i += uint64_t(gridDim.x) * blockDim.x) {
    const unsigned long long f = flag[i], p = pos[i];
    if (!f) continue;
    const uint32_t r = rank_of[g2_adj[i]], e = g2_eid[i];
    core_adj[uint32_t(p)] = r;
    core_eid[uint32_t(p)] = e;
    if (f >> 32) {
      out_adj[p >> 32] = r;
      out_eid[p >> 32] = e;
    }
  }
}

__global__ void k_core_rows(const uint32_t* __restrict__ g2_off, uint32_t n, uint64_t m,
                            const uint32_t* __restrict__ node_of, const unsigned long long* __restrict__ flag,
                            const unsigned long long* __restrict__ pos, uint2* __restrict__ core,
                            uint2* __restrict__ out, uint32_t* __restrict__ degree, uint32_t* __restrict__ facts) {
  uint32_t most = 0;
  auto at = [&](uint32_t i) { return i < m ? pos[i] : (m ? pos[m - 1] + flag[m - 1] : 0ull); };
  if (blockIdx.x == 0 && threadIdx.x == 0) facts[kCoreEntries] = uint32_t(at(uint32_t(m)));
  for (uint64_t r = blockIdx.x * blockDim.x + threadIdx.x; r < n; r += gridDim.x * blockDim.x) {
    const uint64_t x = node_of[r];
    const uint32_t g0 = g2_off[x], g1 = g2_off[x + 1];
    degree[r] = g1 - g0;
    const unsigned long long b = at(g0), e = at(g1);
    core[r] = make_uint2(uint32_t(b), uint32_t(e) - uint32_t(b));
    out[r] = make_uint2(uint32_t(b >> 32), uint32_t(e >> 32) - uint32_t(b >> 32));
    most = max(most, uint32_t(e >> 32) - uint32_t(b >> 32));
    if (uint32_t(e) - uint32_t(b) > 65535u) atomicAdd(&facts[kManyCore], 1u);
  }
  for (int d = kWave / 2; d > 0; d >>= 1) most = max(most, uint32_t(__shfl_xor(int(most), d, kWave)));
  if ((threadIdx.x & (kWave - 1)) == 0 && most > 2) atomicMax(&facts[kLongestOut], most);
}

// ------------------------------------------------------------------ the walk
// What a walk computes: the triangles of each pair (always); the number of
// 4-cycles; the 4-cycles through each pair too; or, from the triangles of
// each pair, the sums over the common neighbours.
enum : int { kTri = 0, kCycles = 1, kPairCycles = 2, kSums = 3 };

struct WalkArgs {
  Ranked g;
  uint32_t* tri_e;                  // triangles of each pair: written (zero before), or read by kSums
  unsigned long long* cycles;       // 4-cycles: kAccCopies counters
  unsigned long long* c4e;          // kPairCycles: 4-cycles of each pair (zero before)
  // kSums: over the common neighbours w of the pair {a < b}: triangles of
  // {a, w}, of {b, w}, pairwise degrees of w
  unsigned long long *sum_a, *sum_b, *sum_d;
  const uint32_t* core_tri;         // kSums: per core entry, its pair's triangles
  uint32_t* vals;                   // kSums: kBitWide values of each of 256 workgroups
};

// A set of ranks with a value each, open addressing in LDS.
template <uint32_t SLOTS>
struct HashTab {
  uint32_t *key, *val;
  uint32_t mask;
  __device__ void begin(uint32_t most) {
    uint32_t cap = 64;
    while (cap < 2 * most && cap < SLOTS) cap <<= 1;
    mask = cap - 1;
    for (uint32_t i = threadIdx.x; i < cap; i += blockDim.x) {
      key[i] = kEmpty32;
      val[i] = 0u;
    }
  }
  __device__ uint32_t home(uint32_t w) const { return (w * 0x9E3779B1u >> 16) & mask; }
  __device__ uint32_t insert(uint32_t w) const {
    uint32_t h = home(w);
    while (true) {
      const uint32_t cur = atomicCAS(&key[h], kEmpty32, w);
      if (cur == kEmpty32 || cur == w) return h;
      h = (h + 1) & mask;
    }
  }
  // slot of w, or kEmpty32
  __device__ uint32_t find(uint32_t w) const {
    uint32_t h = home(w);
    while (true) {
      const uint32_t cur = key[h];
      if (cur == w) return h;
      if (cur == kEmpty32) return kEmpty32;
      h = (h + 1) & mask;
    }
  }
  __device__ bool covers(uint32_t) const { return true; }
  __device__ void mark(uint32_t w) const { val[insert(w)] = 0x80000000u; }
  __device__ void put(uint32_t w, uint32_t v) const { val[insert(w)] = v; }
  __device__ bool marked(uint32_t w) const {
    const uint32_t h = find(w);
    return h != kEmpty32 && (val[h] >> 31);
  }
  // one more path to w; whether w is marked
  __device__ bool add(uint32_t w) const { return atomicAdd(&val[insert(w)], 1u) >> 31; }
  __device__ uint32_t paths(uint32_t w) const { return val[find(w)] & 0x7FFFFFFFu; }
  __device__ uint32_t get(uint32_t w) const {
    const uint32_t h = find(w);
    return h == kEmpty32 ? 0u : val[h];
  }
  // this thread's share of the sum of C(paths, 2)
  __device__ unsigned long long pairs() const {
    unsigned long long s = 0;
    for (uint32_t i = threadIdx.x; i <= mask; i += blockDim.x) {
      const unsigned long long c = val[i] & 0x7FFFFFFFu;
      s += c * (c - (c > 0)) / 2;
    }
    return s;
  }
  __device__ void end() const {}
};

// Values by rank for the ranks [lo, lo + n): path counts of 1 << lg bits
// beside a mark bit each, or mark bits alone for kTri.  All zero between
// walks.  A count holds every path u - x - w when w, or u, has no more core
// neighbours than it can: 4 bits for the ranks of degree below 16 (most), 16
// bits for the others, and 32 when u has more than 65,535 as well as another
// node.  Each range walks the same positions: 16 bits for all took 9 ranges for
// a coauthorship graph's 458,000 ranks, this four.  k_walk_large<2> there: 896
// -> 380 us; k_walk_large<1> on one a tenth as dense: 391 -> 180 us.
constexpr uint32_t kDirectRanks = 51200;   // 16-bit counts: 100 KB, marks 6.25 KB
constexpr uint32_t kDirectWords = kDirectRanks / 2;
constexpr uint32_t kDirectMarks = kDirectRanks / 32;
constexpr uint32_t kNarrowRanks = 163840;   // 4-bit counts: 80 KB, and their marks in the next 20
constexpr uint32_t kNarrowWords = kNarrowRanks / 8;
static_assert(kNarrowWords + kNarrowRanks / 32 == kDirectWords, "both in the same words");
struct DirectTab {
  uint32_t *cnt, *bits;
  uint32_t lo, n, lg;
  __device__ bool covers(uint32_t w) const { return w - lo < n; }
  __device__ void mark(uint32_t w) const { atomicOr(&bits[(w - lo) >> 5], 1u << ((w - lo) & 31)); }
  __device__ bool marked(uint32_t w) const { return (bits[(w - lo) >> 5] >> ((w - lo) & 31)) & 1u; }
  __device__ bool add(uint32_t w) const {
    const uint32_t i = (w - lo) << lg;   // (the count's first bit)
    atomicAdd(&cnt[(w - lo) >> (5 - lg)], 1u << (i & 31));
    return marked(w);
  }
  __device__ uint32_t paths(uint32_t w) const {
    const uint32_t v = cnt[(w - lo) >> (5 - lg)] >> (((w - lo) << lg) & 31);
    return lg == 5 ? v : v & ((1u << (1u << lg)) - 1u);
  }
  __device__ uint32_t words() const { return (n + (32u >> lg) - 1) >> (5 - lg); }
  // the pairs of paths a word of counts of 1 << lg bits holds
  static __device__ unsigned long long pairs_of(uint32_t v, uint32_t lg) {
    if (lg == 5) {
      const unsigned long long c = v;
      return c * (c - (c > 0)) / 2;
    }
    if (lg == 4) {
      const uint32_t a = v & 0xFFFFu, b = v >> 16;
      return (unsigned long long)(a * (a - (a > 0)) / 2) + b * (b - (b > 0)) / 2;
    }
    uint32_t s = 0;
    for (; v; v >>= 4) {
      const uint32_t c = v & 15u;
      s += c * (c - (c > 0)) / 2;
    }
    return s;
  }
  __device__ unsigned long long pairs() const {
    unsigned long long s = 0;
    for (uint32_t i = threadIdx.x; i < words(); i += blockDim.x) s += pairs_of(cnt[i], lg);
    return s;
  }
};

// Values of the neighbours of u among the ranks [lo, lo + n), for kSums: a bit
// per rank, the bits before every 64 ranks, and the values in the order of
// their ranks (of v0 .. v0 + cap of them), in LDS when they fit, so that one
// walk serves kBitRanks ranks.  (A value per rank held 25,600 of them: 18
// walks of the same positions for 460,000 ranks, 0.78 and 0.38 ms for a
// coauthorship graph where this takes 0.28 and 0.25.)
constexpr uint32_t kBitRanks = 458752;
constexpr uint32_t kBitWords = kBitRanks / 32, kBitPres = kBitRanks / 64;
constexpr uint32_t kBitVals = kDirectWords - kBitWords - kBitPres;   // 4,096
constexpr uint32_t kBitWide = 65536;                                 // values at once in device memory
struct BitTab {
  uint32_t *bits, *pre, *val;
  uint32_t lo, n, v0, cap;
  __device__ bool covers(uint32_t w) const { return w - lo < n; }
  __device__ uint32_t index(uint32_t w) const {
    const uint32_t i = w - lo;
    return pre[i >> 6] + (i & 32u ? uint32_t(__popc(bits[(i >> 5) - 1])) : 0u) +
           uint32_t(__popc(bits[i >> 5] & ((1u << (i & 31)) - 1u)));
  }
  __device__ uint32_t get(uint32_t w) const {
    const uint32_t i = w - lo;
    if (!((bits[i >> 5] >> (i & 31)) & 1u)) return 0u;
    const uint32_t k = index(w) - v0;
    return k < cap ? val[k] : 0u;
  }
  // Marks the row entries row[0, len); returns how many are covered.  Every
  // thread of the 1,024 calls this.
  __device__ uint32_t mark_all(const uint32_t* __restrict__ row, uint32_t len, uint32_t* wave_tot) {
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const uint32_t pairs = (n + 63) / 64;
    __syncthreads();   // the previous table is no longer read
    for (uint32_t i = tid; i < 2 * pairs; i += 1024) bits[i] = 0;
    __syncthreads();
    for (uint32_t i = tid; i < len; i += 1024) {
      const uint32_t w = row[i];
      if (covers(w)) atomicOr(&bits[(w - lo) >> 5], 1u << ((w - lo) & 31));
    }
    __syncthreads();
    constexpr uint32_t P = kBitPres / 1024;
    uint32_t c[P], sum = 0, tot;
#pragma unroll
    for (uint32_t k = 0; k < P; ++k) {
      const uint32_t i = tid * P + k;
      c[k] = i < pairs ? uint32_t(__popc(bits[2 * i]) + __popc(bits[2 * i + 1])) : 0u;
      sum += c[k];
    }
    uint32_t at = wave_exclusive_scan(sum, &tot);
    if (lane == 0) wave_tot[wv] = tot;
    __syncthreads();
    uint32_t all = 0;
    for (uint32_t q = 0; q < 1024 / kWave; ++q) {
      if (q == wv) at += all;
      all += wave_tot[q];
    }
#pragma unroll
    for (uint32_t k = 0; k < P; ++k) {
      const uint32_t i = tid * P + k;
      if (i < pairs) pre[i] = at;
      at += c[k];
    }
    __syncthreads();
    return all;
  }
  // Puts the values of the entries into the window [v0, v0 + cap).
  __device__ void put_all(const uint32_t* __restrict__ row, const uint32_t* __restrict__ tri, uint32_t len) const {
    for (uint32_t i = threadIdx.x; i < len; i += 1024) {
      const uint32_t w = row[i];
      if (!covers(w)) continue;
      const uint32_t k = index(w) - v0;
      if (k < cap) val[k] = tri[i] + 1u;
    }
    __syncthreads();
  }
};

// Neighbours of u before u, in chunks of XS: where each one's positions start
// in the chunk, its row, its entry in u's row, and what it collects.
template <uint32_t XS, int MODE>
struct WalkLds {
  uint32_t pos[XS], row[XS], ent[XS], tri[XS];
  unsigned long long sum[MODE == kPairCycles ? XS : 1];
  unsigned long long sums[MODE == kSums ? 3 * XS : 1];
  uint32_t wave_tot[1024 / kWave][2];
  uint32_t n, total;
};

// Every thread of the workgroup (T threads) calls this.  L consecutive
// positions per thread and round: one search for the first's row, then L
// loads in flight.
// The neighbours at entries [e0, e1) of u's core row are walked; passes
// [pass0, pass1): 0 counts, 1 (kPairCycles, after every path is counted) adds
// the cycles to the pairs.
template <uint32_t T, uint32_t XPT, uint32_t L, int MODE, typename Tab>
__device__ void walk_top(const WalkArgs& a, WalkLds<T * XPT, MODE>& S, const Tab& tab, uint32_t u, uint32_t e0,
                         uint32_t e1, int pass0, int pass1, bool shared_pairs) {
  constexpr uint32_t XS = T * XPT;
  const Ranked& g = a.g;
  const uint2 ru = g.core[u];
  const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
  // (a BitTab comes filled)
  if (pass0 == 0 && !std::is_same<Tab, BitTab>::value) {
#pragma unroll 4
    for (uint32_t i = tid; i < ru.y; i += T) {
      const uint32_t w = g.core_adj[ru.x + i];
      if (!tab.covers(w)) continue;
      if constexpr (MODE != kSums) tab.mark(w);
      else if constexpr (!std::is_same<Tab, BitTab>::value) tab.put(w, a.core_tri[ru.x + i] + 1u);
    }
  }
  for (int pass = pass0; pass < pass1; ++pass) {
    for (uint32_t base = e0; base < e1; base += XS) {
      if (pass == pass0 || e1 - e0 > XS) {
        // the chunk's neighbours before u, compacted with the positions
        // where their rows start
        uint32_t x[XPT], len[XPT], row[XPT], mine = 0, kept = 0;
#pragma unroll
        for (uint32_t k = 0; k < XPT; ++k) {
          const uint32_t i = base + tid * XPT + k;
          x[k] = i < e1 ? g.core_adj[ru.x + i] : kEmpty32;
        }
#pragma unroll
        for (uint32_t k = 0; k < XPT; ++k) {
          len[k] = 0;
          if (x[k] < u) {
            const uint2 r = g.core[x[k]];
            row[k] = r.x;
            len[k] = r.y;
            mine += r.y;
            ++kept;
          }
        }
        uint32_t tot_len, tot_n;
        uint32_t at = wave_exclusive_scan(mine, &tot_len), slot = wave_exclusive_scan(kept, &tot_n);
        __syncthreads();   // the previous chunk's arrays are no longer read
        if (T > kWave) {
          if (lane == 0) {
            S.wave_tot[wv][0] = tot_len;
            S.wave_tot[wv][1] = tot_n;
          }
          __syncthreads();
          tot_len = tot_n = 0;
          for (uint32_t q = 0; q < T / kWave; ++q) {
            if (q == wv) {
              at += tot_len;
              slot += tot_n;
            }
            tot_len += S.wave_tot[q][0];
            tot_n += S.wave_tot[q][1];
          }
        }
#pragma unroll
        for (uint32_t k = 0; k < XPT; ++k)
          if (x[k] < u) {
            S.pos[slot] = at;
            S.row[slot] = row[k];
            S.ent[slot] = ru.x + base + tid * XPT + k;
            S.tri[slot] = 0;
            if constexpr (MODE == kPairCycles) S.sum[slot] = 0;
            if constexpr (MODE == kSums) S.sums[slot] = S.sums[XS + slot] = S.sums[2 * XS + slot] = 0;
            at += len[k];
            ++slot;
          }
        if (tid == 0) {
          S.n = tot_n;
          S.total = tot_len;
        }
      }
      __syncthreads();
      const uint32_t n = S.n, total = S.total;
      for (uint32_t p0 = tid * L; p0 < total; p0 += T * L) {
        uint32_t lo = 0, hi = n;   // pos[lo] <= p0 < pos[hi]
        while (hi - lo > 1) {
          const uint32_t m = (lo + hi) >> 1;
          if (S.pos[m] <= p0) lo = m; else hi = m;
        }
        uint32_t next = lo + 1 < n ? S.pos[lo + 1] : total, shift = S.row[lo] - S.pos[lo];
        uint32_t k[L], q[L], w[L];
#pragma unroll
        for (uint32_t r = 0; r < L; ++r) {
          const uint32_t p = min(p0 + r, total - 1);
          if (p >= next) {   // (every row holds u at least)
            ++lo;
            next = lo + 1 < n ? S.pos[lo + 1] : total;
            shift = S.row[lo] - S.pos[lo];
          }
          k[r] = lo;
          q[r] = shift + p;
        }
#pragma unroll
        for (uint32_t r = 0; r < L; ++r) w[r] = g.core_adj[q[r]];
        if constexpr (MODE == kSums) {
          // the common neighbours among them: both loads of each out before
          // any is used; summed in registers as long as the row is the same
          uint32_t t[L], tx[L], d[L];
#pragma unroll
          for (uint32_t r = 0; r < L; ++r) {
            t[r] = p0 + r < total && w[r] != u && tab.covers(w[r]) ? tab.get(w[r]) : 0u;
            tx[r] = t[r] ? a.core_tri[q[r]] : 0u;
            d[r] = t[r] ? g.degree[w[r]] : 0u;
          }
          unsigned long long sx = 0, su = 0;
          uint32_t sd = 0, at = k[0];   // (degrees add up to at most 2 |E2|, below 2^32)
          auto add = [&]() {
            if (!sd) return;
            if (sx) atomicAdd(&S.sums[at], sx);
            if (su) atomicAdd(&S.sums[XS + at], su);
            atomicAdd(&S.sums[2 * XS + at], (unsigned long long)sd);
          };
#pragma unroll
          for (uint32_t r = 0; r < L; ++r) {
            if (k[r] != at) {
              add();
              sx = su = 0;
              sd = 0;
              at = k[r];
            }
            sx += tx[r];
            su += t[r] ? t[r] - 1 : 0u;
            sd += d[r];
          }
          add();
        } else {
#pragma unroll
          for (uint32_t r = 0; r < L; ++r) {
            if (p0 + r >= total || w[r] == u || !tab.covers(w[r])) continue;
            if (pass == 0) {
              bool hit;
              if (MODE != kTri && w[r] < u) hit = tab.add(w[r]);
              else hit = tab.marked(w[r]);
              if (hit) atomicAdd(&S.tri[k[r]], 1u);
            } else if (w[r] < u) {
              // a path of c to w closes c - 1 cycles, each holding its two pairs
              const uint32_t c = tab.paths(w[r]);
              if (c >= 2) {
                atomicAdd(&S.sum[k[r]], (unsigned long long)(c - 1));
                atomicAdd(&a.c4e[g.core_eid[q[r]]], (unsigned long long)(c - 1));
              }
            }
          }
        }
      }
      __syncthreads();
      for (uint32_t i = tid; i < n; i += T) {
        const uint32_t e = g.core_eid[S.ent[i]];
        if constexpr (MODE == kSums) {
          if (!S.sums[XS + i] && !S.sums[i] && !S.sums[2 * XS + i]) continue;
          const bool x_first = g.node_of[g.core_adj[S.ent[i]]] < g.node_of[u];
          atomicAdd(x_first ? &a.sum_a[e] : &a.sum_b[e], S.sums[i]);
          atomicAdd(x_first ? &a.sum_b[e] : &a.sum_a[e], S.sums[XS + i]);
          atomicAdd(&a.sum_d[e], S.sums[2 * XS + i]);
        } else if (pass == 0) {
          if (S.tri[i]) {
            if (shared_pairs) atomicAdd(&a.tri_e[e], S.tri[i]);
            else a.tri_e[e] = S.tri[i];
          }
        } else if (MODE == kPairCycles && S.sum[i]) {
          atomicAdd(&a.c4e[e], S.sum[i]);
        }
      }
    }
    __syncthreads();
  }
}

constexpr bool counts_paths(int mode) { return mode == kCycles || mode == kPairCycles; }
constexpr int passes_of(int mode) { return mode == kPairCycles ? 2 : 1; }

// Sum of x over the workgroup (T threads) to one of the copies of *out.
template <uint32_t T>
__device__ void add_copies(unsigned long long x, unsigned long long* out) {
  __shared__ unsigned long long part[T / kWave];
  x = wave_sum(x);
  if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x / kWave] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long s = 0;
    for (uint32_t q = 0; q < T / kWave; ++q) s += part[q];
    if (s) atomicAdd(&out[blockIdx.x % kAccCopies], s);
  }
}

// Degree below kSmallDeg: a wavefront per node.
template <int MODE>
__global__ void __launch_bounds__(kWave) k_walk_small(WalkArgs a) {
  __shared__ WalkLds<kWave, MODE> S;
  __shared__ uint32_t key[kSmallSlots], val[kSmallSlots];
  HashTab<kSmallSlots> tab{key, val, 0};
  unsigned long long cycles = 0;
  const uint32_t r0 = a.g.bounds[0], r1 = a.g.bounds[1];
  for (uint64_t at = uint64_t(r0) + blockIdx.x; at < r1; at += gridDim.x) {
    const uint32_t u = uint32_t(at);
    const uint2 row = a.g.core[u];
    if (row.y < 2) continue;   // one neighbour of degree 2 or more closes nothing
    // what the walk may meet: every path, when the table holds paths
    uint32_t most = row.y;
    if (counts_paths(MODE)) {
      const uint32_t x = threadIdx.x < row.y ? a.g.core_adj[row.x + threadIdx.x] : kEmpty32;
      most += wave_sum_u32(x < u ? a.g.core[x].y : 0u);
    }
    __syncthreads();   // the previous node's table is no longer read
    tab.begin(most);
    __syncthreads();
    walk_top<kWave, 1, 2, MODE>(a, S, tab, u, 0, row.y, 0, passes_of(MODE), false);
    if (counts_paths(MODE)) cycles += tab.pairs();
  }
  if (counts_paths(MODE)) add_copies<kWave>(cycles, a.cycles);
}

// The ranks of the workgroups' shares are strided; each takes up to T
// candidates at a time, drops those of the other classes, and walks the rest,
// the latest (longest) first.
template <uint32_t T, typename F, typename G>
__device__ void for_candidates(uint64_t count, uint32_t* list, uint32_t* n_list, F keep, G body) {
  for (uint64_t base = 0; base + blockIdx.x < count; base += uint64_t(T) * gridDim.x) {
    const uint64_t c = base + uint64_t(threadIdx.x) * gridDim.x + blockIdx.x;
    const bool on = c < count && keep(c);
    __syncthreads();
    if (threadIdx.x == 0) *n_list = 0;
    __syncthreads();
    // in order: a wavefront's kept candidates after those of the wavefronts
    // before it
    const unsigned long long m = __ballot(on);
    for (uint32_t q = 0; q < T / kWave; ++q) {
      if (threadIdx.x / kWave == q) {
        const uint32_t lane = threadIdx.x & (kWave - 1);
        const uint32_t at = *n_list;
        if (on) list[at + uint32_t(__popcll(m & ((1ull << lane) - 1ull)))] = threadIdx.x;
        wave_sync();
        if (lane == 0) *n_list = at + uint32_t(__popcll(m));
      }
      __syncthreads();
    }
    const uint32_t n = *n_list;
    for (uint32_t i = 0; i < n; ++i) body(base + uint64_t(list[i]) * gridDim.x + blockIdx.x);
  }
}

template <int MODE>
__global__ void __launch_bounds__(256) k_walk_mid(WalkArgs a) {
  __shared__ WalkLds<1024, MODE> S;
  __shared__ uint32_t key[kMidSlots], val[kMidSlots];
  __shared__ uint32_t list[256], n_list;
  HashTab<kMidSlots> tab{key, val, 0};
  unsigned long long cycles = 0;
  const uint32_t n = a.g.n, r1 = a.g.bounds[1];
  for_candidates<256>(
      n - r1, list, &n_list, [&](uint64_t c) { return a.g.weight[n - 1 - uint32_t(c)] <= kMidMost; },
      [&](uint64_t c) {
        const uint32_t u = n - 1 - uint32_t(c);
        __syncthreads();
        tab.begin(a.g.weight[u]);
        __syncthreads();
        walk_top<256, 4, 4, MODE>(a, S, tab, u, 0, a.g.core[u].y, 0, passes_of(MODE), false);
        if (counts_paths(MODE)) cycles += tab.pairs();
      });
  if (counts_paths(MODE)) add_copies<256>(cycles, a.cycles);
}

// A 16-bit count holds every path u - x - w when u or w has at most 65,535
// core neighbours: always, unless u and another node have more.
__device__ inline bool wide_counts(const Ranked& g, uint32_t u) {
  return g.core[u].y > 65535u && g.facts[kManyCore] >= 2u;
}

// The walks of more than kSplitWork positions are split into shares of about
// as many (communication: the longest, on one CU, took 1.6 ms beside 0.3 ms
// of evenly spread work).  Split nodes are marked in weight.
constexpr uint32_t kSplitWork = 1u << 17;
constexpr uint32_t kSplitWalk = 0xFFFFFFFFu;
constexpr uint32_t kSplitRanks = 4096;     // only the latest ranks are looked at
constexpr uint32_t kSplitMostShares = 64;  // per node
struct SplitNode {
  uint32_t u, first, shares;   // rank; its shares are [first, first + shares)
};

__global__ void __launch_bounds__(1024) k_split_plan(Ranked g, uint32_t* __restrict__ weight, uint32_t capacity,
                                                     SplitNode* __restrict__ nodes, uint32_t* __restrict__ facts) {
  __shared__ uint32_t wave_tot[2][1024 / kWave];
  constexpr uint32_t P = kSplitRanks / 1024;
  const uint32_t lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
  uint32_t shares[P], mine = 0, n_mine = 0;
#pragma unroll
  for (uint32_t k = 0; k < P; ++k) {
    const uint32_t i = threadIdx.x * P + k;
    shares[k] = 0;
    if (i < g.n && g.n - 1 - i >= g.bounds[1]) {
      const uint32_t u = g.n - 1 - i, w = weight[u];
      if (w > kSplitWork && !wide_counts(g, u)) shares[k] = min(kSplitMostShares, (w + kSplitWork - 1) / kSplitWork);
    }
    mine += shares[k];
    n_mine += shares[k] != 0;
  }
  uint32_t tot, n_tot;
  uint32_t at = wave_exclusive_scan(mine, &tot), slot = wave_exclusive_scan(n_mine, &n_tot);
  if (lane == 0) {
    wave_tot[0][wv] = tot;
    wave_tot[1][wv] = n_tot;
  }
  __syncthreads();
  for (uint32_t q = 0; q < wv; ++q) {
    at += wave_tot[0][q];
    slot += wave_tot[1][q];
  }
  // in rank order, as many as the shares' counters hold: those taken are a
  // prefix, so the last one taken ends the totals
#pragma unroll
  for (uint32_t k = 0; k < P; ++k) {
    if (!shares[k]) continue;
    if (at + shares[k] <= capacity) {
      const uint32_t u = g.n - 1 - (threadIdx.x * P + k);
      nodes[slot] = SplitNode{u, at, shares[k]};
      weight[u] = kSplitWalk;
      atomicMax(&facts[kSplitNodes], slot + 1);
      atomicMax(&facts[kSplitShares], at + shares[k]);
    }
    at += shares[k];
    ++slot;
  }
}

// Threads' neighbours per chunk (the LDS beside the table).
template <int MODE>
constexpr uint32_t direct_xpt() { return MODE == kSums ? 1 : 2; }

// Range `part` of the ranks a mode's table holds at once, from the first of
// degree 2; empty past the last.  kTri and kSums take ranges of one size.  The
// modes that count paths take the ranks of degree below 16 by kNarrowRanks (lg
// 2) and the others by kDirectRanks (lg 4) where that makes fewer ranges, for
// each one walks every position again, and otherwise all by kDirectRanks: the
// communication graph's 50,000 ranks fit one, and as two ranges k_walk_large
// took 422 us in place of 141.
struct RankRange {
  uint32_t first, size, lg;
};
template <int MODE>
__device__ inline RankRange range_of(const Ranked& g, uint32_t part) {
  uint32_t first = g.bounds[0], end = g.n, step = MODE == kTri ? kDirectWords * 32 : kBitRanks, lg = 0;
  if (counts_paths(MODE)) {
    auto ranges = [](uint32_t ranks, uint32_t r) { return ranks / r + (ranks % r != 0); };
    const uint32_t mid = g.bounds[2], narrow = ranges(mid - first, kNarrowRanks);
    const bool both = narrow + ranges(end - mid, kDirectRanks) < ranges(end - first, kDirectRanks);
    step = kDirectRanks;
    lg = 4;
    if (both && part < narrow) {
      end = mid;
      step = kNarrowRanks;
      lg = 2;
    } else if (both) {
      first = mid;
      part -= narrow;
    }
  }
  const uint64_t at = first + uint64_t(part) * step;
  return at < end ? RankRange{uint32_t(at), min(step, end - uint32_t(at)), lg} : RankRange{0, 0, lg};
}

// kSums over the ranks [first, first + size) for u's entries [e0, e1).
template <uint32_t XPT>
__device__ void walk_sums(const WalkArgs& a, WalkLds<1024 * XPT, kSums>& S, uint32_t* words, uint32_t u, uint32_t first,
                          uint32_t size, uint32_t e0, uint32_t e1) {
  const uint2 ru = a.g.core[u];
  BitTab tab{words, words + kBitWords, words + kBitWords + kBitPres, first, size, 0, kBitVals};
  const uint32_t marked = tab.mark_all(a.g.core_adj + ru.x, ru.y, &S.wave_tot[0][0]);
  if (marked > kBitVals) {
    tab.val = a.vals + uint64_t(blockIdx.x) * kBitWide;
    tab.cap = kBitWide;
  }
  for (tab.v0 = 0; tab.v0 < marked; tab.v0 += tab.cap) {
    tab.put_all(a.g.core_adj + ru.x, a.core_tri + ru.x, ru.y);
    walk_top<1024, XPT, 8, kSums>(a, S, tab, u, e0, e1, 0, 1, true);
    __syncthreads();
  }
}

template <int MODE>
__global__ void __launch_bounds__(1024) k_walk_large(WalkArgs a, uint32_t parts) {
  constexpr uint32_t XPT = direct_xpt<MODE>();
  __shared__ WalkLds<1024 * XPT, MODE> S;
  __shared__ uint32_t words[kDirectWords];
  __shared__ uint32_t marks[MODE == kTri || MODE == kSums ? 1 : kDirectMarks];
  __shared__ uint32_t list[1024], n_list;
  for (uint32_t i = threadIdx.x; i < kDirectWords; i += 1024) words[i] = 0;
  if (MODE != kTri && MODE != kSums)
    for (uint32_t i = threadIdx.x; i < kDirectMarks; i += 1024) marks[i] = 0;
  unsigned long long cycles = 0;
  const uint32_t n = a.g.n, r1 = a.g.bounds[1];
  for_candidates<1024>(
      uint64_t(n - r1) * parts, list, &n_list,
      [&](uint64_t c) {
        const uint32_t w = a.g.weight[n - 1 - uint32_t(c / parts)];
        return w > kMidMost && w != kSplitWalk && range_of<MODE>(a.g, uint32_t(c % parts)).size;
      },
      [&](uint64_t c) {
        const uint32_t u = n - 1 - uint32_t(c / parts);
        const RankRange q = range_of<MODE>(a.g, uint32_t(c % parts));
        if constexpr (MODE == kSums) {
          walk_sums<XPT>(a, S, words, u, q.first, q.size, 0, a.g.core[u].y);
        } else {
          const bool narrow = counts_paths(MODE) && q.lg == 2u;
          const bool wide = counts_paths(MODE) && !narrow && wide_counts(a.g, u);
          const uint32_t step = wide ? kDirectRanks / 2 : q.size;
          for (uint32_t at = 0; at < q.size; at += step) {
            DirectTab tab{words, MODE == kTri ? words : narrow ? words + kNarrowWords : marks, q.first + at,
                          q.size - at < step ? q.size - at : step, wide ? 5u : q.lg};
            __syncthreads();
            walk_top<1024, XPT, 8, MODE>(a, S, tab, u, 0, a.g.core[u].y, 0, passes_of(MODE), parts > 1 || wide);
            if (counts_paths(MODE)) cycles += tab.pairs();
            __syncthreads();
            if (counts_paths(MODE))
              for (uint32_t i = threadIdx.x; i < tab.words(); i += 1024) words[i] = 0;
            for (uint32_t i = threadIdx.x; i < (tab.n + 31) / 32; i += 1024) tab.bits[i] = 0;
          }
        }
      });
  if (counts_paths(MODE)) add_copies<1024>(cycles, a.cycles);
}

// The shares of the split walks, a (share, range of ranks) per workgroup.
// Counting modes leave a share's counts in `dump` (kDirectWords per task) for
// k_split_sum; with SECOND, the pass of kPairCycles over the summed counts.
template <int MODE, bool SECOND>
__global__ void __launch_bounds__(1024) k_walk_split(WalkArgs a, const SplitNode* __restrict__ nodes, uint32_t parts,
                                                     uint32_t* __restrict__ dump) {
  constexpr uint32_t XPT = direct_xpt<MODE>();
  __shared__ WalkLds<1024 * XPT, MODE> S;
  __shared__ uint32_t words[kDirectWords];
  __shared__ uint32_t marks[MODE == kSums ? 1 : kDirectMarks];
  const uint32_t n_nodes = a.g.facts[kSplitNodes], n_shares = a.g.facts[kSplitShares];
  for (uint64_t t = blockIdx.x; t < uint64_t(n_shares) * parts; t += gridDim.x) {
    const uint32_t share = uint32_t(t / parts), part = uint32_t(t % parts);
    const RankRange q = range_of<MODE>(a.g, part);
    if (!q.size) continue;
    uint32_t lo = 0, hi = n_nodes;   // nodes[lo].first <= share < nodes[hi].first
    while (hi - lo > 1) {
      const uint32_t m = (lo + hi) >> 1;
      if (nodes[m].first <= share) lo = m; else hi = m;
    }
    const SplitNode node = nodes[lo];
    const uint32_t s = share - node.first, len = a.g.core[node.u].y;
    const uint32_t e0 = uint32_t(uint64_t(len) * s / node.shares), e1 = uint32_t(uint64_t(len) * (s + 1) / node.shares);
    if constexpr (MODE == kSums) {
      walk_sums<XPT>(a, S, words, node.u, q.first, q.size, e0, e1);
    } else {
      DirectTab tab{words, q.lg == 2 ? words + kNarrowWords : marks, q.first, q.size, q.lg};
      __syncthreads();   // the previous task's tables are no longer read
      const uint32_t used = tab.words();
      if (SECOND) {
        const uint32_t* summed = dump + (uint64_t(node.first) * parts + part) * kDirectWords;
        for (uint32_t i = threadIdx.x; i < used; i += 1024) words[i] = summed[i];
      } else {
        for (uint32_t i = threadIdx.x; i < used; i += 1024) words[i] = 0;
        for (uint32_t i = threadIdx.x; i < (tab.n + 31) / 32; i += 1024) tab.bits[i] = 0;
      }
      __syncthreads();
      walk_top<1024, XPT, 8, MODE>(a, S, tab, node.u, e0, e1, SECOND ? 1 : 0, SECOND ? 2 : 1, true);
      if (!SECOND) {
        uint32_t* out = dump + t * kDirectWords;
        for (uint32_t i = threadIdx.x; i < used; i += 1024) out[i] = words[i];
      }
    }
  }
}

// The counts of each split node's shares summed into its first share's, and
// the 4-cycles they close.  (Several counts per word: no count's sum over the
// shares passes its bits, see DirectTab.)
__global__ void __launch_bounds__(1024) k_split_sum(Ranked g, const SplitNode* __restrict__ nodes, uint32_t parts,
                                                    uint32_t* __restrict__ dump, unsigned long long* __restrict__ out) {
  const uint32_t n_nodes = g.facts[kSplitNodes];
  unsigned long long cycles = 0;
  for (uint64_t t = blockIdx.x; t < uint64_t(n_nodes) * parts; t += gridDim.x) {
    const SplitNode node = nodes[t / parts];
    const uint32_t part = uint32_t(t % parts);
    const RankRange q = range_of<kCycles>(g, part);
    const uint32_t words = q.size ? (q.size + (32u >> q.lg) - 1) >> (5 - q.lg) : 0u;
    uint32_t* base = dump + (uint64_t(node.first) * parts + part) * kDirectWords;
    for (uint32_t i = threadIdx.x; i < words; i += 1024) {
      uint32_t v = 0;
      for (uint32_t s = 0; s < node.shares; ++s) v += base[uint64_t(s) * parts * kDirectWords + i];
      base[i] = v;
      cycles += DirectTab::pairs_of(v, q.lg);
    }
  }
  add_copies<1024>(cycles, out);
}

// ------------------------------------------------------------------ 4-cliques
// A 4-clique is counted at its first node lo, as a triangle among the later
// neighbours D of lo: the pairs of G2 inside D are found by walking the out
// rows of D against a hash table of D, as bit rows over D; a second walk adds,
// for each pair of D, the common neighbours (the members of D after both, or
// with EDGE every member adjacent to both: the 4-cliques through lo and the
// pair).  D of at most CAP nodes, one workgroup of T threads per lo.
template <uint32_t T, uint32_t CAP, bool EDGE>
struct CliqueLds {
  static constexpr uint32_t kWords = CAP / 32;
  uint32_t pos[CAP], row[CAP];
  uint32_t bits[CAP * (kWords + 1)];   // rows an odd number of words apart (fewer bank conflicts)
  uint32_t key[2 * CAP], val[2 * CAP];
  uint32_t own[EDGE ? CAP : 1];
  uint32_t wave_tot[T / kWave];
};

template <uint32_t T, uint32_t CAP, bool EDGE>
__global__ void __launch_bounds__(T) k_clique(Ranked g, uint32_t least, unsigned long long* __restrict__ acc,
                                              unsigned long long* __restrict__ k4e) {
  using Lds = CliqueLds<T, CAP, EDGE>;
  constexpr uint32_t DPT = CAP / T, STRIDE = Lds::kWords + 1, SLOTS = 2 * CAP, L = 4;
  __shared__ Lds S;
  __shared__ uint32_t list[T], n_list;
  if (g.facts[kLongestOut] < least) return;   // (launched on a bound of it)
  const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
  unsigned long long cliques = 0;
  const uint32_t r0 = g.bounds[0];
  auto keep = [&](uint64_t c) {
    const uint32_t n = g.out[r0 + uint32_t(c)].y;
    return n >= least && n <= CAP;
  };
  for_candidates<T>(g.n - r0, list, &n_list, keep, [&](uint64_t c) {
    const uint32_t lo = r0 + uint32_t(c);
    const uint2 d = g.out[lo];
    const uint32_t words = (d.y + 31) / 32;
    __syncthreads();   // the previous node's arrays are no longer read
    for (uint32_t i = tid; i < SLOTS; i += T) S.key[i] = kEmpty32;
    for (uint32_t i = tid; i < d.y * STRIDE; i += T) S.bits[i] = 0;
    uint32_t x[DPT], len[DPT], row[DPT], mine = 0;
#pragma unroll
    for (uint32_t k = 0; k < DPT; ++k) {
      const uint32_t i = tid * DPT + k;
      x[k] = i < d.y ? g.out_adj[d.x + i] : 0u;
    }
#pragma unroll
    for (uint32_t k = 0; k < DPT; ++k) {
      const uint32_t i = tid * DPT + k;
      const uint2 r = i < d.y ? g.out[x[k]] : make_uint2(0u, 0u);
      row[k] = r.x;
      len[k] = r.y;
      mine += r.y;
      if (EDGE && i < d.y) S.own[i] = 0;
    }
    uint32_t total;
    uint32_t at = wave_exclusive_scan(mine, &total);
    if (lane == 0) S.wave_tot[wv] = total;
    __syncthreads();
    total = 0;
    for (uint32_t q = 0; q < T / kWave; ++q) {
      if (q == wv) at += total;
      total += S.wave_tot[q];
    }
#pragma unroll
    for (uint32_t k = 0; k < DPT; ++k) {
      const uint32_t i = tid * DPT + k;
      if (i < d.y) {
        S.pos[i] = at;
        S.row[i] = row[k];
        at += len[k];
        uint32_t h = (x[k] * 0x9E3779B1u >> 16) & (SLOTS - 1);
        while (atomicCAS(&S.key[h], kEmpty32, x[k]) != kEmpty32) h = (h + 1) & (SLOTS - 1);
        S.val[h] = i;
      }
    }
    __syncthreads();
    for (int pass = 0; pass < 2; ++pass) {
      for (uint32_t p0 = tid * L; p0 < total; p0 += T * L) {
        uint32_t a = 0, b = d.y;   // the last row that starts at or before p0
        while (b - a > 1) {
          const uint32_t m = (a + b) >> 1;
          if (S.pos[m] <= p0) a = m; else b = m;
        }
        uint32_t i[L], q[L], w[L];
#pragma unroll
        for (uint32_t r = 0; r < L; ++r) {
          const uint32_t p = min(p0 + r, total - 1);
          while (a + 1 < d.y && S.pos[a + 1] <= p) ++a;   // (rows may be empty)
          i[r] = a;
          q[r] = S.row[a] + (p - S.pos[a]);
        }
#pragma unroll
        for (uint32_t r = 0; r < L; ++r) w[r] = g.out_adj[q[r]];
#pragma unroll
        for (uint32_t r = 0; r < L; ++r) {
          if (p0 + r >= total) continue;
          uint32_t h = (w[r] * 0x9E3779B1u >> 16) & (SLOTS - 1);
          uint32_t cur = S.key[h];
          while (cur != w[r] && cur != kEmpty32) {
            h = (h + 1) & (SLOTS - 1);
            cur = S.key[h];
          }
          if (cur == kEmpty32) continue;
          const uint32_t j = S.val[h];
          if (pass == 0) {
            atomicOr(&S.bits[i[r] * STRIDE + (j >> 5)], 1u << (j & 31));
            if (EDGE) atomicOr(&S.bits[j * STRIDE + (i[r] >> 5)], 1u << (i[r] & 31));
          } else {
            uint32_t c = 0;
            for (uint32_t k = 0; k < words; ++k) c += __popc(S.bits[i[r] * STRIDE + k] & S.bits[j * STRIDE + k]);
            if (!c) continue;
            cliques += c;
            if (EDGE) {
              atomicAdd(&S.own[i[r]], c);
              atomicAdd(&S.own[j], c);
              atomicAdd(&k4e[g.out_eid[q[r]]], (unsigned long long)c);
            }
          }
        }
      }
      __syncthreads();
    }
    if (EDGE)
      for (uint32_t i = tid; i < d.y; i += T)
        if (S.own[i]) atomicAdd(&k4e[g.out_eid[d.x + i]], (unsigned long long)(S.own[i] / 2));
  });
  // (with EDGE each 4-clique was met at the three pairs of D it holds)
  add_copies<T>(cliques, acc);
}

// D of more nodes than an LDS bit matrix holds: its rows in device memory
// (`cap` rows of cap / 32 words per workgroup), filled by probing every pair.
template <bool EDGE>
__global__ void __launch_bounds__(1024) k_clique_wide(Ranked g, View v, uint32_t least, uint32_t cap,
                                                      uint32_t* __restrict__ matrix,
                                                      unsigned long long* __restrict__ acc,
                                                      unsigned long long* __restrict__ k4e,
                                                      const uint32_t* __restrict__ g2_eid) {
  if (g.facts[kLongestOut] < least) return;
  const uint32_t cap_words = (cap + 31) / 32;
  uint32_t* M = matrix + uint64_t(blockIdx.x) * cap * cap_words;
  unsigned long long cliques = 0;
  for (uint32_t lo = g.bounds[0] + blockIdx.x; lo < g.n; lo += gridDim.x) {
    const uint2 d = g.out[lo];
    if (d.y < least) continue;
    const uint32_t words = (d.y + 31) / 32;
    // a thread owns a word: 32 members of D against one
    for (uint64_t t = threadIdx.x; t < uint64_t(d.y) * words; t += 1024) {
      const uint32_t i = uint32_t(t / words), w = uint32_t(t % words);
      const uint32_t x = g.node_of[g.out_adj[d.x + i]];
      uint32_t word = 0;
      for (uint32_t b = 0; b < 32; ++b) {
        const uint32_t j = 32 * w + b;
        if (j < d.y && j != i && has2(v.hs2, x, g.node_of[g.out_adj[d.x + j]])) word |= 1u << b;
      }
      __hip_atomic_store(&M[uint64_t(i) * cap_words + w], word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();   // (the words are read back past the L1 cache)
    auto word_of = [&](uint32_t i, uint32_t w) {
      return __hip_atomic_load(&M[uint64_t(i) * cap_words + w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    // a thread owns a member: its pairs in D, their common members
    for (uint32_t i = threadIdx.x; i < d.y; i += 1024) {
      unsigned long long own = 0;
      for (uint32_t w = 0; w < words; ++w)
        for (uint32_t rest = word_of(i, w); rest; rest &= rest - 1) {
          const uint32_t j = 32 * w + uint32_t(__ffs(rest) - 1);
          if (!EDGE && j < i) continue;
          // (without EDGE the members after both, so that each 4-clique is
          // met once)
          uint32_t c = 0;
          for (uint32_t k = EDGE ? 0 : w; k < words; ++k)
            c += __popc(word_of(i, k) & word_of(j, k) & (EDGE ? ~0u : mask_gt(j, k)));
          own += c;
          if (j < i || !c) continue;
          cliques += c;
          if (EDGE) {
            const uint32_t x = g.node_of[g.out_adj[d.x + i]], y = g.node_of[g.out_adj[d.x + j]];
            uint32_t p = v.g2_off[x], e = v.g2_off[x + 1];
            while (p < e) {
              const uint32_t m = p + ((e - p) >> 1);
              if (v.g2_adj[m] < y) p = m + 1; else e = m;
            }
            atomicAdd(&k4e[g2_eid[p]], (unsigned long long)c);
          }
        }
      if (EDGE && own) atomicAdd(&k4e[g.out_eid[d.x + i]], own / 2);
    }
    __syncthreads();
  }
  add_copies<1024>(cliques, acc);
}

__global__ void k_sum_copies(const unsigned long long* __restrict__ copies, unsigned long long* __restrict__ out) {
  unsigned long long s = threadIdx.x < kAccCopies ? copies[threadIdx.x] : 0ull;
  s = wave_sum(s);
  if (threadIdx.x == 0) *out = s;
}

unsigned grid_of(uint64_t items, uint64_t per_block, unsigned cap) {
  return unsigned(std::max<uint64_t>(1, std::min<uint64_t>((items + per_block - 1) / per_block, cap)));
}

// H's pairwise graph in rank space, in buffers of tmp; *most receives, when
// asked for, the largest out row (one host read-back) or, for a graph with bit
// rows, a bound on it, as calls on those do not wait for the stream.  (The
// bound: an out row of m entries belongs to a node of m neighbours or more, and
// its entries are of the same class of degrees or a later one, whose degrees
// are more than 8/9 of the node's.  So 8/9 m^2 is at most the sum of all
// degrees, 2 n2.)
int ranked_graph(hm_graph* H, hipStream_t st, Scratch& tmp, Ranked* out, uint32_t* most) {
  HM_TRY(ensure_ranks(H, st));
  const uint32_t n = H->n_nodes;
  const uint64_t n2 = H->n_by_size[2], m = 2 * n2;
  unsigned long long *flag = nullptr, *pos = nullptr;
  uint32_t *core_adj = nullptr, *core_eid = nullptr, *out_adj = nullptr, *out_eid = nullptr, *weight = nullptr,
           *degree = nullptr, *facts = nullptr;
  uint2 *core = nullptr, *rows = nullptr;
  HM_TRY(tmp.get(&weight, n));
  HM_TRY(tmp.get(&degree, n));
  HM_TRY(tmp.get(&core, n));
  HM_TRY(tmp.get(&rows, n));
  HM_TRY(tmp.get(&facts, kFacts));
  HM_TRY(tmp.get(&flag, m));
  HM_TRY(tmp.get(&pos, m));
  HM_TRY(tmp.get(&core_adj, m));
  HM_TRY(tmp.get(&core_eid, m));
  HM_TRY(tmp.get(&out_adj, n2));
  HM_TRY(tmp.get(&out_eid, n2));
  HM_TRY(fill_u32(facts, 0, kFacts, st));
  HM_TRY(fill_u32(weight, 0, n, st));
  k_core_flags<<<grid_of(m, 256, 4096), 256, 0, st>>>(H->g2_off, H->g2_adj, H->g2_eid, H->e2, m, H->rank_of,
                                                      H->rank_bounds, flag, weight);
  HM_HIP(hipGetLastError());
  HM_TRY(scan_exclusive_u64(flag, pos, m, st));
  k_core_fill<<<grid_of(m, 256, 4096), 256, 0, st>>>(H->g2_adj, H->g2_eid, m, H->rank_of, flag, pos, core_adj,
                                                     core_eid, out_adj, out_eid);
  k_core_rows<<<grid_of(n, 256, 1024), 256, 0, st>>>(H->g2_off, n, m, H->node_of, flag, pos, core, rows, degree, facts);
  HM_HIP(hipGetLastError());
  *out = Ranked{n, H->rank_of, H->node_of, core, rows, core_adj, core_eid, out_adj, out_eid, degree, weight,
                H->rank_bounds, facts};
  if (most && H->bits) {
    *most = uint32_t(std::min<double>(n, 1.5 * std::sqrt(double(n2)) + 1.0));
  } else if (most) {
    HM_HIP(hipMemcpyAsync(most, facts + kLongestOut, sizeof(uint32_t), hipMemcpyDeviceToHost, st));
    HM_HIP(hipStreamSynchronize(st));
  }
  return HM_OK;
}

// Split walks of one graph: their nodes, and room for the shares' counts.
struct Split {
  SplitNode* nodes = nullptr;
  uint32_t* dump = nullptr;
  uint32_t parts = 0;   // ranges of ranks of the counting modes
};

// Ranges of ranks of a mode (an upper bound; see range_of): at most n2 / 8
// nodes have 16 neighbours.
template <int MODE>
uint32_t parts_of(uint32_t n, uint64_t n2) {
  auto ranges = [](uint64_t ranks, uint64_t r) { return uint32_t(std::max<uint64_t>(1, (ranks + r - 1) / r)); };
  if (!counts_paths(MODE)) return ranges(n, MODE == kTri ? kDirectWords * 32 : kBitRanks);
  return std::min(ranges(n, kDirectRanks),
                  ranges(n, kNarrowRanks) + ranges(std::min<uint64_t>(n, n2 / 8), kDirectRanks));
}

// Plans the split walks (marking their nodes in g.weight), with counters for
// 1,024 (share, range) tasks (100 MB).
int plan_split(const Ranked& g, uint64_t n2, Scratch& tmp, Split* sp, hipStream_t st) {
  sp->parts = parts_of<kCycles>(g.n, n2);
  const uint32_t capacity = 1024 / sp->parts;
  HM_TRY(tmp.get(&sp->nodes, kSplitRanks));
  HM_TRY(tmp.get(&sp->dump, uint64_t(std::max<uint32_t>(capacity, 1)) * sp->parts * kDirectWords));
  k_split_plan<<<1, 1024, 0, st>>>(g, const_cast<uint32_t*>(g.weight), capacity, sp->nodes,
                                   const_cast<uint32_t*>(g.facts));
  HM_HIP(hipGetLastError());
  return HM_OK;
}

// The walk launches of one mode, the longest walks first.
template <int MODE>
int launch_walks(const WalkArgs& a, uint64_t n2, const Split& sp, const char* name, hipStream_t st) {
  ProfileScope ps(name, st);
  const uint32_t parts = parts_of<MODE>(a.g.n, n2);
  if constexpr (MODE != kTri) {
    k_walk_split<MODE, false><<<256, 1024, 0, st>>>(a, sp.nodes, parts, sp.dump);
    if constexpr (counts_paths(MODE)) k_split_sum<<<256, 1024, 0, st>>>(a.g, sp.nodes, parts, sp.dump, a.cycles);
    if constexpr (MODE == kPairCycles) k_walk_split<MODE, true><<<256, 1024, 0, st>>>(a, sp.nodes, parts, sp.dump);
  }
  k_walk_large<MODE><<<256, 1024, 0, st>>>(a, parts);
  k_walk_mid<MODE><<<768, 256, 0, st>>>(a);
  k_walk_small<MODE><<<grid_of(a.g.n, 1, 3072), kWave, 0, st>>>(a);
  HM_HIP(hipGetLastError());
  return HM_OK;
}

template <bool EDGE>
int launch_cliques(const hm_graph* H, const Ranked& g, uint32_t most, unsigned long long* copies,
                   unsigned long long* k4e, hipStream_t st, Scratch& tmp) {
  ProfileScope ps("k_clique", st);
  if (most > 512) {
    // at most 2 GiB of matrices
    const uint64_t each = uint64_t(most) * ((most + 31) / 32);
    const unsigned blocks = unsigned(std::max<uint64_t>(1, std::min<uint64_t>(256, (1ull << 29) / each)));
    uint32_t* matrix = nullptr;
    HM_TRY(tmp.get(&matrix, each * blocks));
    k_clique_wide<EDGE><<<blocks, 1024, 0, st>>>(g, view_of(H), 513, most, matrix, copies, k4e, H->g2_eid);
  }
  if (most > 64) k_clique<256, 512, EDGE><<<768, 256, 0, st>>>(g, 65, copies, k4e);
  if (most > 2) k_clique<64, 64, EDGE><<<grid_of(g.n, 1, 4096), 64, 0, st>>>(g, 3, copies, k4e);
  HM_HIP(hipGetLastError());
  return HM_OK;
}

}  // namespace

// H->rank_of, node_of and rank_bounds, on first use.
int ensure_ranks(hm_graph* H, hipStream_t st) {
  if (H->rank_of) return HM_OK;
  HM_TRY(refuse_capture(st));
  note_use(H, st);
  const uint32_t n = H->n_nodes;
  Scratch tmp(st);
  uint32_t *keys = nullptr, *keys_tmp = nullptr;
  HM_TRY(tmp.get(&keys, n));
  HM_TRY(tmp.get(&keys_tmp, n));
  // (handed over to the graph once the launches are in; the sort's one pass
  // leaves the order in the second buffer, which becomes node_of)
  Scratch kept(st);
  uint32_t *rank_of = nullptr, *node_of = nullptr, *vals_tmp = nullptr, *bounds = nullptr;
  HM_TRY(kept.get(&rank_of, n));
  HM_TRY(kept.get(&node_of, n));
  HM_TRY(kept.get(&vals_tmp, n));
  HM_TRY(kept.get(&bounds, 3));
  k_rank_keys<<<grid_of(n, 256, 2048), 256, 0, st>>>(H->g2_off, n, keys, node_of, bounds);
  HM_HIP(hipGetLastError());
  HM_TRY(radix_sort_pairs(keys, node_of, keys_tmp, vals_tmp, n, kRankBits, st));
  k_rank_assign<<<grid_of(n, 256, 2048), 256, 0, st>>>(keys, node_of, n, rank_of, bounds);
  HM_HIP(hipGetLastError());
  kept.ptrs.assign(1, vals_tmp);   // (the other order buffer goes)
  H->rank_of = rank_of;
  H->node_of = node_of;
  H->rank_bounds = bounds;
  return HM_OK;
}

// Triangles of every pair of G2 (tri_e, n2 values) and, at order 4, the number
// of 4-cycles and of 4-cliques of G2 (non-induced; device words).
int wedge_counts(hm_graph* H, int k, uint32_t* tri_e, unsigned long long* n_cycles, unsigned long long* n_cliques,
                 hipStream_t st) {
  const uint64_t n2 = H->n_by_size[2];
  Scratch tmp(st);
  unsigned long long* copies = nullptr;
  HM_TRY(tmp.get(&copies, 2 * kAccCopies));
  HM_TRY(fill_u64(copies, 0, 2 * kAccCopies, st));
  HM_TRY(fill_u32(tri_e, 0, n2, st));
  Ranked g;
  uint32_t most = 0;
  HM_TRY(ranked_graph(H, st, tmp, &g, k == 4 ? &most : nullptr));
  WalkArgs a{};
  a.g = g;
  a.tri_e = tri_e;
  a.cycles = copies;
  Split sp;
  if (k == 3) return launch_walks<kTri>(a, n2, sp, "k_walk", st);
  HM_TRY(plan_split(g, n2, tmp, &sp, st));
  HM_TRY(launch_walks<kCycles>(a, n2, sp, "k_walk", st));
  HM_TRY(launch_cliques<false>(H, g, most, copies + kAccCopies, nullptr, st, tmp));
  k_sum_copies<<<1, kWave, 0, st>>>(copies, n_cycles);
  k_sum_copies<<<1, kWave, 0, st>>>(copies + kAccCopies, n_cliques);
  HM_HIP(hipGetLastError());
  return HM_OK;
}

__global__ void k_es_widen(const uint32_t* __restrict__ t32, uint64_t n, unsigned long long* __restrict__ t64) {
  for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += uint64_t(gridDim.x) * blockDim.x)
    t64[i] = t32[i];
}

// per core entry, its pair's triangles
__global__ void k_core_tri(const uint32_t* __restrict__ core_eid, const uint32_t* __restrict__ tri_e,
                           const uint32_t* __restrict__ facts, uint32_t* __restrict__ core_tri) {
  const uint32_t n = facts[kCoreEntries];
  for (uint64_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
    core_tri[i] = tri_e[core_eid[i]];
}

// The per-pair statistics of hm_graph::es (6 x n2).
int wedge_edge_stats(hm_graph* H, unsigned long long* es, hipStream_t st) {
  const uint64_t n2 = H->n_by_size[2];
  HM_TRY(fill_u64(es, 0, 6 * n2, st));
  if (!n2) return HM_OK;
  Scratch tmp(st);
  unsigned long long* copies = nullptr;
  uint32_t* tri_e = nullptr;
  HM_TRY(tmp.get(&copies, 2 * kAccCopies));
  HM_TRY(tmp.get(&tri_e, n2));
  HM_TRY(fill_u64(copies, 0, 2 * kAccCopies, st));
  HM_TRY(fill_u32(tri_e, 0, n2, st));
  Ranked g;
  uint32_t most = 0;
  HM_TRY(ranked_graph(H, st, tmp, &g, &most));
  WalkArgs a{};
  a.g = g;
  a.tri_e = tri_e;
  a.cycles = copies;
  a.c4e = es + 2 * n2;
  a.sum_a = es + 3 * n2;
  a.sum_b = es + 4 * n2;
  a.sum_d = es + 5 * n2;
  uint32_t* core_tri = nullptr;
  HM_TRY(tmp.get(&core_tri, 2 * n2));
  a.core_tri = core_tri;
  HM_TRY(tmp.get(&a.vals, uint64_t(256) * kBitWide));
  Split sp;
  HM_TRY(plan_split(g, n2, tmp, &sp, st));
  HM_TRY(launch_walks<kPairCycles>(a, n2, sp, "k_walk", st));
  k_es_widen<<<grid_of(n2, 256, 2048), 256, 0, st>>>(tri_e, n2, es);
  k_core_tri<<<grid_of(2 * n2, 256, 4096), 256, 0, st>>>(g.core_eid, tri_e, g.facts, core_tri);
  HM_TRY(launch_walks<kSums>(a, n2, sp, "k_walk_sums", st));
  HM_TRY(launch_cliques<true>(H, g, most, copies + kAccCopies, es + n2, st, tmp));
  return HM_OK;
}

}  // namespace hm
