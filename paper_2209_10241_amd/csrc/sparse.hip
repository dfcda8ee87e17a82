// Exact order-3 and order-4 counts on hypergraphs without adjacency bit rows
// (Algorithms 2 and 3, Section 4.2), sized for graphs with millions of
// hyperedges and heavy-tailed degrees.
//
// The generators and ownership rules are those of the bit-row path:
//   (a) every k-node hyperedge, classified by fill-in;
//   (b) order 4: the sets around 3-node hyperedges, counted by
//       inclusion-exclusion (triples.hip);
//   (c) sets connected through pairs only: never enumerated.  The number of
//       connected k-node sets of the pairwise graph G2 per induced shape
//       follows from non-induced subgraph counts: 3-stars sum C(d,3),
//       3-paths sum over edges (d_u-1)(d_v-1) - 3T, paws sum t_v (d_v-2),
//       diamonds sum over edges C(t_e,2), triangles, 4-cycles and 4-cliques
//       by degree-ordered walks (wedge.hip), inverted through the matrix of
//       how often each shape contains another; then the sets that (a) or (b)
//       own are subtracted by shape.
#include <algorithm>
#include <vector>

#include "hm_sparse.h"
#include "hm_wedge.h"

namespace hm {
namespace {

enum : int { kAccT3 = 0, kAccDiamond, kAccP4, kAccPaw2, kAccStar, kAccWedge, kAccC4, kAccK4, kAccN };

// sum of x over the workgroup, added to *out by one thread
__device__ inline void block_add(unsigned long long x, unsigned long long* out) {
  __shared__ unsigned long long part[kWavesPerBlock];
  x = wave_sum(x);
  const int wv = threadIdx.x / kWave;
  if ((threadIdx.x & (kWave - 1)) == 0) part[wv] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long s = 0;
    for (int i = 0; i < kWavesPerBlock; ++i) s += part[i];
    if (s) atomicAdd(out, s);
  }
  __syncthreads();
}

// Per pair {a, b} of G2, from its triangles t: t (3 x triangles), C(t, 2)
// (diamonds through their diagonal), (d_a - 1)(d_b - 1) (3-paths, plus 3 x
// triangles), t (d_a + d_b - 4) (twice the paws).
__global__ void __launch_bounds__(kThreads) k_sp_pairs(View v, uint64_t n2, const uint32_t* __restrict__ tri_e,
                                                       unsigned long long* __restrict__ acc) {
  unsigned long long st = 0, sd = 0, sp = 0, sw = 0;
  for (uint64_t e = uint64_t(blockIdx.x) * kThreads + threadIdx.x; e < n2; e += uint64_t(gridDim.x) * kThreads) {
    const unsigned long long t = tri_e[e];
    const unsigned long long da = deg2_of(v, v.e2[2 * e]), db = deg2_of(v, v.e2[2 * e + 1]);
    st += t;
    sd += t * (t - (t > 0)) / 2;
    sp += (da - 1) * (db - 1);
    if (t) sw += t * (da + db - 4);   // (then both degrees are at least 2)
  }
  block_add(st, acc + kAccT3);
  block_add(sd, acc + kAccDiamond);
  block_add(sp, acc + kAccP4);
  block_add(sw, acc + kAccPaw2);
}

// Triangles for order 3 (3 x, as the sum over the pairs) by probes: a wavefront
// takes kProbePairs pairs, lays the shorter row of each out flat, four positions
// per lane and round, and looks every entry up beside the pair's other node.
// One launch, where the walks of wedge.hip rank the nodes and copy the rows
// first; the probes go to memory, where the walks' lookups stay in LDS, so
// they are the better up to a number of pairs, and of pairs times degrees
// (probes_order3).  Order 3 on kept graphs, us by probes and by walks (a
// wavefront per pair in brackets): 5,000 pairs on 10,000 nodes 42, 80 (63);
// co-authorship recipe, 9,900, 201,000 and 609,000 pairs 46, 107 (109); 173,
// 250 (291); 433, 515 (612); 1.02 million 1046, 857 (1512).  Communication
// recipe, 199,000 pairs on 9,400 nodes 344, 414 (367); 356,000 on 16,450 556,
// 670 (576); 620,000 on 28,200 1253, 1095 (1225).  (4 or 64 pairs a wavefront:
// 303 and 829 at 199,000; 50 and 54 at 9,900; 274 and 134 at a million pairs
// of degree 2, where 8 take 200.)
constexpr uint32_t kProbePairs = 8;
bool probes_order3(uint64_t n2, uint64_t nodes) { return n2 < 3u << 18 && 2 * n2 * n2 / nodes <= 1u << 24; }

__global__ void __launch_bounds__(kThreads) k_sp_pair_probes(View v, uint64_t n2, unsigned long long* __restrict__ acc) {
  constexpr uint32_t L = 4, per = kProbePairs;
  __shared__ uint32_t s_pos[kWavesPerBlock][per + 1], s_row[kWavesPerBlock][per], s_other[kWavesPerBlock][per];
  const uint32_t lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
  uint32_t *pos = s_pos[wv], *row = s_row[wv], *other = s_other[wv];
  const uint64_t n_waves = uint64_t(gridDim.x) * kWavesPerBlock;
  unsigned long long hits = 0;
  for (uint64_t e0 = (uint64_t(blockIdx.x) * kWavesPerBlock + wv) * per; e0 < n2; e0 += n_waves * per) {
    uint32_t len = 0;
    if (lane < per && e0 + lane < n2) {
      const uint32_t a = v.e2[2 * (e0 + lane)], b = v.e2[2 * (e0 + lane) + 1];
      const uint32_t ab = v.g2_off[a], da = v.g2_off[a + 1] - ab, bb = v.g2_off[b], db = v.g2_off[b + 1] - bb;
      len = min(da, db);
      if (len < 2) len = 0;   // (the pair itself)
      row[lane] = da <= db ? ab : bb;
      other[lane] = da <= db ? b : a;
    }
    uint32_t total;
    const uint32_t at = wave_exclusive_scan(len, &total);
    if (lane < per) pos[lane] = at;
    if (lane == 0) pos[per] = total;
    wave_sync();
    for (uint64_t t0 = lane * L; t0 < total; t0 += kWave * L) {
      uint32_t lo = 0, hi = per;   // pos[lo] <= t0 < pos[hi]
      while (hi - lo > 1) {
        const uint32_t m = (lo + hi) >> 1;
        if (pos[m] <= t0) lo = m; else hi = m;
      }
      Probe64 pr[L];
      uint32_t z[L], o[L];
#pragma unroll
      for (uint32_t r = 0; r < L; ++r) {
        const uint32_t t = uint32_t(min<uint64_t>(t0 + r, total - 1));
        while (pos[lo + 1] <= t) ++lo;   // (pairs without a row)
        o[r] = other[lo];
        z[r] = v.g2_adj[row[lo] + (t - pos[lo])];
      }
#pragma unroll
      for (uint32_t r = 0; r < L; ++r) pr[r] = probe2_start(v.hs2, o[r], z[r]);
#pragma unroll
      for (uint32_t r = 0; r < L; ++r)
        if (probe64_end(v.hs2, pr[r]) && t0 + r < total) ++hits;
    }
    wave_sync();   // (the next pairs' rows)
  }
  block_add(hits, acc + kAccT3);
}

// Per node: C(d,3) (3-stars), C(d,2) (wedges).
__global__ void __launch_bounds__(kThreads) k_sp_nodes(View v, unsigned long long* __restrict__ acc) {
  unsigned long long s3 = 0, s2 = 0;
  for (uint64_t x = blockIdx.x * kThreads + threadIdx.x; x < v.N; x += gridDim.x * kThreads) {
    const unsigned long long d = v.g2_off[x + 1] - v.g2_off[x];
    if (d >= 2) s2 += d * (d - 1) / 2;
    if (d >= 3) s3 += d * (d - 1) / 2 * (d - 2) / 3;
  }
  block_add(s3, acc + kAccStar);
  block_add(s2, acc + kAccWedge);
}

// Induced shape counts from the non-induced ones, into the G2 region.
struct ShapeClasses {
  int k3_path, k3_triangle;
  int path, star, cycle, paw, diamond, clique;
};

__global__ void k_sp_shapes(const unsigned long long* __restrict__ acc, int k, ShapeClasses cls,
                            unsigned long long* __restrict__ hist) {
  if (threadIdx.x != 0) return;
  const unsigned long long T = acc[kAccT3] / 3;
  if (k == 3) {
    hist[kG2 + cls.k3_triangle] = T;
    hist[kG2 + cls.k3_path] = acc[kAccWedge] - 3 * T;
    return;
  }
  const unsigned long long k4 = acc[kAccK4];
  const unsigned long long dia = acc[kAccDiamond] - 6 * k4;
  const unsigned long long cyc = acc[kAccC4] - dia - 3 * k4;
  const unsigned long long paw = acc[kAccPaw2] / 2 - 4 * dia - 12 * k4;
  const unsigned long long star = acc[kAccStar] - paw - 2 * dia - 4 * k4;
  const unsigned long long path = (acc[kAccP4] - 3 * T) - 4 * cyc - 2 * paw - 6 * dia - 12 * k4;
  hist[kG2 + cls.clique] = k4;
  hist[kG2 + cls.diamond] = dia;
  hist[kG2 + cls.cycle] = cyc;
  hist[kG2 + cls.paw] = paw;
  hist[kG2 + cls.star] = star;
  hist[kG2 + cls.path] = path;
}

// Entries of the pair index: code 3i + s for 3-node hyperedge i = {a<b<c} and
// slot s, the pair {a,b} (third node c), {a,c} (b) or {b,c} (a).  The
// entries are sorted by third node, then stably by pair, so that each pair's
// run lists its third nodes in ascending order.
__device__ inline uint32_t pl_third_of(const uint32_t* e3, uint32_t code) {
  const uint64_t i = code / 3;
  const uint32_t s = code % 3;
  return e3[3 * i + 2 - s];
}

__global__ void k_pl_third_keys(const uint32_t* __restrict__ e3, uint64_t n, uint32_t* __restrict__ keys,
                                uint32_t* __restrict__ codes) {
  for (uint64_t p = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; p < n; p += uint64_t(gridDim.x) * blockDim.x) {
    keys[p] = pl_third_of(e3, uint32_t(p));
    codes[p] = uint32_t(p);
  }
}

// (packed to `bits` per node for the sort, which then needs 2 * bits of key,
// in 32 bits when they fit; k_pl_wide_keys widens them to (x << 32) | y)
template <typename K>
__global__ void k_pl_pair_keys(const uint32_t* __restrict__ e3, const uint32_t* __restrict__ codes, uint64_t n, int bits,
                               K* __restrict__ keys) {
  for (uint64_t p = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; p < n; p += uint64_t(gridDim.x) * blockDim.x) {
    const uint32_t code = codes[p];
    const uint64_t i = code / 3;
    const uint32_t s = code % 3;
    const K a = e3[3 * i], b = e3[3 * i + 1], c = e3[3 * i + 2];
    keys[p] = s == 0 ? ((a << bits) | b) : (s == 1 ? ((a << bits) | c) : ((b << bits) | c));
  }
}

template <typename K>
__global__ void k_pl_wide_keys(const K* __restrict__ packed, uint64_t n, int bits, unsigned long long* __restrict__ keys) {
  for (uint64_t p = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; p < n; p += uint64_t(gridDim.x) * blockDim.x) {
    const unsigned long long k = packed[p];
    keys[p] = ((k >> bits) << 32) | (k & ((1ull << bits) - 1));
  }
}

// Hash index over the runs of the sorted pair keys.  First pass: every run's
// first position claims a slot for its key (start << 32); second pass: its
// last position adds the count.
__global__ void k_pl_index_starts(const unsigned long long* __restrict__ keys, uint64_t n, unsigned long long* slot,
                                  unsigned long long mask) {
  for (uint64_t p = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; p < n; p += uint64_t(gridDim.x) * blockDim.x) {
    const unsigned long long key = keys[p];
    if (p > 0 && keys[p - 1] == key) continue;
    unsigned long long h = mix64(key) & mask;
    while (atomicCAS(&slot[2 * h], kEmpty64, key) != kEmpty64) h = (h + 1) & mask;
    slot[2 * h + 1] = (unsigned long long)p << 32;
  }
}

__global__ void k_pl_index_counts(const unsigned long long* __restrict__ keys, uint64_t n, unsigned long long* slot,
                                  unsigned long long mask) {
  for (uint64_t p = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; p < n; p += uint64_t(gridDim.x) * blockDim.x) {
    const unsigned long long key = keys[p];
    if (p + 1 < n && keys[p + 1] == key) continue;
    unsigned long long h = mix64(key) & mask;
    while (slot[2 * h] != key) h = (h + 1) & mask;
    const unsigned long long start = slot[2 * h + 1] >> 32;
    slot[2 * h + 1] = (start << 32) | (p + 1 - start);
  }
}

// Per pair entry: its 3-node hyperedge (the code, in place), the third node
// and that node's pairwise adjacency to the two nodes of the key.
__global__ void k_pl_third(const uint32_t* __restrict__ e3, const unsigned long long* __restrict__ keys,
                           uint32_t* __restrict__ edge, uint64_t n, Set64 hs2, uint32_t* __restrict__ third,
                           uint8_t* __restrict__ adj) {
  for (uint64_t p = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; p < n; p += uint64_t(gridDim.x) * blockDim.x) {
    const unsigned long long key = keys[p];
    const uint32_t x = uint32_t(key >> 32), y = uint32_t(key);
    const uint32_t code = edge[p];
    const uint32_t t = pl_third_of(e3, code);
    edge[p] = code / 3;
    third[p] = t;
    adj[p] = uint8_t(uint32_t(has2(hs2, x, t)) | (uint32_t(has2(hs2, y, t)) << 1));
  }
}

// Common pairwise neighbours of every distinct pair of the index, into the
// pair's slot: a workgroup takes 256 positions of the sorted keys; for each
// run that starts among them the shorter of the pair's two rows is walked,
// all rows laid out flat (four positions per thread and round), and tested
// against the other node's dense row, or probed.  (A wavefront per run left
// most lanes idle and probed every position: 2.8 ms on the communication
// graph, 1.3 on the co-authorship one.)
__global__ void __launch_bounds__(kThreads) k_pl_codeg(View v, const unsigned long long* __restrict__ keys, uint64_t n,
                                                       const unsigned long long* __restrict__ slot,
                                                       unsigned long long mask, const int32_t* __restrict__ hub_rank,
                                                       const uint32_t* __restrict__ hub_bits, uint32_t hub_w,
                                                       uint32_t* __restrict__ codeg) {
  constexpr uint32_t L = 4;
  __shared__ uint32_t pos[kThreads + 1], row[kThreads], other[kThreads], cnt[kThreads];
  __shared__ int hub[kThreads];
  __shared__ uint32_t wave_tot[kWavesPerBlock];
  const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
  for (uint64_t p0 = uint64_t(blockIdx.x) * kThreads; p0 < n; p0 += uint64_t(gridDim.x) * kThreads) {
    const uint64_t p = p0 + tid;
    unsigned long long key = 0;
    uint32_t len = 0;
    bool start = false;
    __syncthreads();   // the previous positions' arrays are no longer read
    if (p < n) {
      key = keys[p];
      start = p == 0 || keys[p - 1] != key;
      if (start) {
        const uint32_t x = uint32_t(key >> 32), y = uint32_t(key);
        const uint32_t xb = v.g2_off[x], xe = v.g2_off[x + 1], yb = v.g2_off[y], ye = v.g2_off[y + 1];
        const bool at_x = xe - xb <= ye - yb;
        len = at_x ? xe - xb : ye - yb;
        row[tid] = at_x ? xb : yb;
        other[tid] = at_x ? y : x;
        hub[tid] = hub_rank ? hub_rank[at_x ? y : x] : -1;
      }
    }
    cnt[tid] = 0;
    uint32_t tot;
    uint32_t at = wave_exclusive_scan(len, &tot);
    if (lane == 0) wave_tot[wv] = tot;
    __syncthreads();
    for (uint32_t q = 0; q < wv; ++q) at += wave_tot[q];
    pos[tid] = at;
    if (tid == kThreads - 1) pos[kThreads] = at + len;
    __syncthreads();
    const uint32_t total = pos[kThreads];
    for (uint32_t t0 = tid * L; t0 < total; t0 += kThreads * L) {
      uint32_t lo = 0, hi = kThreads;   // pos[lo] <= t0 < pos[hi]
      while (hi - lo > 1) {
        const uint32_t m = (lo + hi) >> 1;
        if (pos[m] <= t0) lo = m; else hi = m;
      }
      uint32_t k[L], z[L];
      Probe64 pr[L];
#pragma unroll
      for (uint32_t r = 0; r < L; ++r) {
        const uint32_t t = min(t0 + r, total - 1);
        while (pos[lo + 1] <= t) ++lo;   // (positions without a start have no row)
        k[r] = lo;
        z[r] = v.g2_adj[row[lo] + (t - pos[lo])];
      }
#pragma unroll
      for (uint32_t r = 0; r < L; ++r)
        if (hub[k[r]] < 0) pr[r] = probe2_start(v.hs2, other[k[r]], z[r]);
#pragma unroll
      for (uint32_t r = 0; r < L; ++r) {
        if (t0 + r >= total) continue;
        const int h = hub[k[r]];
        const bool hit = h >= 0 ? (hub_bits[uint64_t(h) * hub_w + (z[r] >> 5)] >> (z[r] & 31)) & 1u
                                : probe64_end(v.hs2, pr[r]);
        if (hit) atomicAdd(&cnt[k[r]], 1u);
      }
    }
    __syncthreads();
    if (start) {
      unsigned long long h = mix64(key) & mask;
      while (slot[2 * h] != key) h = (h + 1) & mask;
      codeg[h] = cnt[tid];
    }
  }
}

unsigned grid_cap(uint64_t items, uint64_t per_block, unsigned cap) {
  uint64_t g = (items + per_block - 1) / per_block;
  return unsigned(std::max<uint64_t>(1, std::min<uint64_t>(g, cap)));
}



// Per node, over its adjacency row: the sum of the neighbours' degrees, and
// of its pairs' triangles (twice the triangles at the node).  A wavefront
// takes 64 consecutive entries, sums them by row with a segmented scan, and
// each row's last lane adds once.
__global__ void k_ns_rows(View v, uint64_t m, const uint32_t* __restrict__ eid, const unsigned long long* __restrict__ tri_e,
                          unsigned long long* __restrict__ nbr, unsigned long long* __restrict__ tri2) {
  const uint32_t lane = threadIdx.x & (kWave - 1);
  for (uint64_t base = (uint64_t(blockIdx.x) * blockDim.x + threadIdx.x) & ~uint64_t(kWave - 1); base < m;
       base += uint64_t(gridDim.x) * blockDim.x) {
    const uint64_t i = base + lane;
    uint32_t owner = 0xFFFFFFFFu;
    unsigned long long d = 0, t = 0;
    if (i < m) {
      const uint32_t z = v.g2_adj[i];
      const uint64_t e = eid[i];
      owner = v.e2[2 * e] ^ v.e2[2 * e + 1] ^ z;
      d = deg2_of(v, z);
      t = tri_e[e];
    }
    for (int s = 1; s < kWave; s <<= 1) {
      const uint32_t o = uint32_t(__shfl_up(int(owner), s, kWave));
      const unsigned long long dd = __shfl_up(d, s, kWave), tt = __shfl_up(t, s, kWave);
      if (int(lane) >= s && o == owner) {   // (a row's entries are consecutive)
        d += dd;
        t += tt;
      }
    }
    const uint32_t after = uint32_t(__shfl_down(int(owner), 1, kWave));
    if (i < m && (lane == kWave - 1 || after != owner)) {
      atomicAdd(&nbr[owner], d);
      if (t) atomicAdd(&tri2[owner], t);
    }
  }
}

__global__ void k_ns_half(unsigned long long* __restrict__ tri, uint32_t n) {
  for (uint64_t x = blockIdx.x * blockDim.x + threadIdx.x; x < n; x += gridDim.x * blockDim.x) tri[x] /= 2;
}

// per 3-node hyperedge {a < b < c}: a ~ b, a ~ c, b ~ c (bits 0..2)
__global__ void k_e3_pat(View v, uint64_t n3, uint8_t* __restrict__ pat) {
  for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n3; i += uint64_t(gridDim.x) * blockDim.x) {
    const uint32_t a = v.e3[3 * i], b = v.e3[3 * i + 1], c = v.e3[3 * i + 2];
    const Probe64 pab = probe2_start(v.hs2, a, b), pac = probe2_start(v.hs2, a, c), pbc = probe2_start(v.hs2, b, c);
    pat[i] = uint8_t(uint32_t(probe64_end(v.hs2, pab)) | (uint32_t(probe64_end(v.hs2, pac)) << 1) |
                     (uint32_t(probe64_end(v.hs2, pbc)) << 2));
  }
}

// per node o, its 3-node hyperedges {o, y, z} (y < z) by (o~y, o~z, y~z).  A
// wavefront takes 64 consecutive incidence entries, adds their counts (eight
// of 8 bits) by row with a segmented scan, and each row's last lane adds them
// once: three atomics per hyperedge, most of them to few nodes, took 191 us
// for 381,000 hyperedges, this 58 and k_e3_pat 35.
__global__ void k_ns_h3(View v, uint64_t m, const uint8_t* __restrict__ pat, uint32_t* __restrict__ h3) {
  const uint32_t lane = threadIdx.x & (kWave - 1);
  for (uint64_t base = (uint64_t(blockIdx.x) * blockDim.x + threadIdx.x) & ~uint64_t(kWave - 1); base < m;
       base += uint64_t(gridDim.x) * blockDim.x) {
    const uint64_t p = base + lane;
    uint32_t o = 0xFFFFFFFFu;
    unsigned long long n = 0;
    if (p < m) {
      o = upper_bound(v.i3_off, 0, v.N + 1, uint32_t(p)) - 1;   // the last row that starts at or before p
      const uint32_t i = v.i3_idx[p], q = pat[i];
      const uint32_t ab = q & 1u, ac = (q >> 1) & 1u, bc = q >> 2;
      const uint32_t a = v.e3[3ull * i], b = v.e3[3ull * i + 1];
      const uint32_t w = o == a ? (ab | (ac << 1) | (bc << 2)) : (o == b ? (ab | (bc << 1) | (ac << 2))
                                                                         : (ac | (bc << 1) | (ab << 2)));
      n = 1ull << (8 * w);
    }
    for (int s = 1; s < kWave; s <<= 1) {
      const uint32_t before = uint32_t(__shfl_up(int(o), s, kWave));
      const unsigned long long k = __shfl_up(n, s, kWave);
      if (int(lane) >= s && before == o) n += k;   // (a row's entries are consecutive; at most 64 each)
    }
    const uint32_t after = uint32_t(__shfl_down(int(o), 1, kWave));
    if (p < m && (lane == kWave - 1 || after != o)) {
#pragma unroll
      for (uint32_t w = 0; w < 8; ++w) {
        const uint32_t k = uint32_t(n >> (8 * w)) & 255u;
        if (k) atomicAdd(&h3[8ull * o + w], k);
      }
    }
  }
}

}  // namespace

// HM_EUNSUPPORTED for a pairwise graph over more than 2^31 nodes at order 4.
static int within_node_range(const hm_graph* H) {
  if (H->n_nodes <= 1u << 31 || H->n_by_size[2] == 0) return HM_OK;
  set_error("order 4 supports at most 2^31 nodes with pairwise hyperedges, not %u", H->n_nodes);
  return HM_EUNSUPPORTED;
}

// Per-pair statistics of H for the pair sampler without bit rows (layout in
// hm_graph::es), built on first use.
int ensure_edge_stats(hm_graph* H, hipStream_t st) {
  note_use(H, st);
  if (H->es) return HM_OK;
  HM_TRY(within_node_range(H));
  HM_TRY(refuse_capture(st));
  void* es = nullptr;
  HM_TRY(dalloc(&es, 6 * std::max<uint64_t>(H->n_by_size[2], 1) * sizeof(unsigned long long)));
  const int rc = wedge_edge_stats(H, static_cast<unsigned long long*>(es), st);
  if (rc != HM_OK) {
    dfree_on(es, st);
    return rc;
  }
  H->es = static_cast<unsigned long long*>(es);
  return HM_OK;
}

// Per-node statistics of H for the pair samplers without bit rows, built on
// first use (after the per-pair ones): triangles at each node, the sum of its
// neighbours' degrees, and its 3-node hyperedges by pairwise pattern.
int ensure_node_stats(hm_graph* H, hipStream_t st) {
  note_use(H, st);
  if (H->ns_tri) return HM_OK;
  HM_TRY(refuse_capture(st));
  HM_TRY(ensure_edge_stats(H, st));
  const View v = view_of(H);
  const uint64_t n2 = H->n_by_size[2], n3 = H->n_by_size[3], N = H->n_nodes;
  void *p_tri = nullptr, *p_nbr = nullptr, *p_h3 = nullptr, *p_pat = nullptr;
  int rc = dalloc(&p_tri, N * sizeof(unsigned long long));
  if (rc == HM_OK) rc = dalloc(&p_nbr, N * sizeof(unsigned long long));
  if (rc == HM_OK) rc = dalloc(&p_h3, 8 * N * sizeof(uint32_t));
  if (rc == HM_OK) rc = dalloc(&p_pat, n3 + 1);
  auto* tri = static_cast<unsigned long long*>(p_tri);
  auto* nbr = static_cast<unsigned long long*>(p_nbr);
  auto* h3 = static_cast<uint32_t*>(p_h3);
  if (rc == HM_OK) rc = fill_u64(tri, 0, N, st);
  if (rc == HM_OK) rc = fill_u64(nbr, 0, N, st);
  if (rc == HM_OK) rc = fill_u32(h3, 0, 8 * N, st);
  if (rc == HM_OK) {
    if (n2) k_ns_rows<<<grid_cap(2 * n2, 256, 4096), 256, 0, st>>>(v, 2 * n2, H->g2_eid, H->es, nbr, tri);
    k_ns_half<<<grid_cap(N, 256, 1024), 256, 0, st>>>(tri, uint32_t(N));
    if (n3) {
      k_e3_pat<<<grid_cap(n3, 256, 4096), 256, 0, st>>>(v, n3, static_cast<uint8_t*>(p_pat));
      k_ns_h3<<<grid_cap(3 * n3, 256, 4096), 256, 0, st>>>(v, 3 * n3, static_cast<uint8_t*>(p_pat), h3);
    }
    if (hipGetLastError() != hipSuccess) {
      set_error("per-node statistics: kernel launch failed");
      rc = HM_EDEVICE;
    }
  }
  if (rc != HM_OK) {
    void* ps[] = {p_tri, p_nbr, p_h3, p_pat};
    dfree_on(ps, 4, st);
    return rc;
  }
  H->ns_tri = tri;
  H->ns_nbr = nbr;
  H->ns_h3 = h3;
  H->e3_pat = static_cast<uint8_t*>(p_pat);
  return HM_OK;
}

// Every 3-node subset of every 4-node hyperedge, packed as in quad_find, with
// the hyperedge's fourth node.
__global__ void k_quad_keys(const uint32_t* __restrict__ e4, uint64_t n4, int q, unsigned long long* __restrict__ keys,
                            uint32_t* __restrict__ fourth) {
  for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n4; i += uint64_t(gridDim.x) * blockDim.x) {
    const unsigned long long m[4] = {e4[4 * i], e4[4 * i + 1], e4[4 * i + 2], e4[4 * i + 3]};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const unsigned long long x = m[s == 0 ? 1 : 0], y = m[s <= 1 ? 2 : 1], z = m[s <= 2 ? 3 : 2];
      keys[4 * i + s] = (x << (2 * q)) | (y << q) | z;
      fourth[4 * i + s] = uint32_t(m[s]);
    }
  }
}

// Takes p (allocated in tmp) out of tmp: it stays with its new owner.
template <typename T>
T* keep(Scratch& tmp, T* p) {
  tmp.ptrs.erase(std::find(tmp.ptrs.begin(), tmp.ptrs.end(), static_cast<void*>(p)));
  return p;
}

// The 3-node subset -> 4-node hyperedge index (H->q_*), when the packed key
// fits 63 bits; otherwise none (q_bits = 0) and the incidence lists serve.
// Built on first use.
int ensure_quad_index(hm_graph* H, hipStream_t st) {
  note_use(H, st);
  if (H->q_done) return HM_OK;
  HM_TRY(refuse_capture(st));
  const uint64_t n4 = H->n_by_size[4];
  int bits = 1;
  while (bits < 32 && (1ull << bits) < H->n_nodes) ++bits;
  if (n4 == 0 || 3 * bits > 63) {
    H->q_done = true;
    return HM_OK;
  }
  const uint64_t n = 4 * n4;
  Scratch tmp(st);
  unsigned long long *k = nullptr, *kt = nullptr, *slots = nullptr;
  uint32_t *f = nullptr, *ft = nullptr;
  const unsigned long long cap = pow2_capacity(n);
  HM_TRY(tmp.get(&k, n));
  HM_TRY(tmp.get(&kt, n));
  HM_TRY(tmp.get(&f, n));
  HM_TRY(tmp.get(&ft, n));
  HM_TRY(tmp.get(&slots, 2 * cap));
  HM_TRY(fill_u64(slots, kEmpty64, 2 * cap, st));
  k_quad_keys<<<grid_cap(n4, 256, 4096), 256, 0, st>>>(H->e4, n4, bits, k, f);
  HM_HIP(hipGetLastError());
  HM_TRY(radix_sort_pairs(k, f, kt, ft, n, 3 * bits, st));
  const unsigned g = grid_cap(n, 256, 4096);
  k_pl_index_starts<<<g, 256, 0, st>>>(k, n, slots, cap - 1);
  k_pl_index_counts<<<g, 256, 0, st>>>(k, n, slots, cap - 1);
  HM_HIP(hipGetLastError());
  H->q_slot = keep(tmp, slots);
  H->q_mask = cap - 1;
  H->q_fourth = keep(tmp, f);
  H->q_bits = bits;
  H->q_done = true;
  return HM_OK;
}

// The entries' codes in *e (buffers *e and *et) into the order of their pairs,
// whose keys go to `keys`; packed keys of type K.
template <typename K>
int sort_by_pair(const hm_graph* H, uint64_t n, int bits, uint32_t*& e, uint32_t*& et, unsigned long long* keys,
                 hipStream_t st, Scratch& tmp) {
  K *k = nullptr, *kt = nullptr;
  HM_TRY(tmp.get(&k, n));
  HM_TRY(tmp.get(&kt, n));
  k_pl_pair_keys<K><<<grid_cap(n, 256, 4096), 256, 0, st>>>(H->e3, e, n, bits, k);
  HM_HIP(hipGetLastError());
  HM_TRY(radix_sort_pairs(k, e, kt, et, n, 2 * bits, st));
  k_pl_wide_keys<K><<<grid_cap(n, 256, 4096), 256, 0, st>>>(k, n, bits, keys);
  HM_HIP(hipGetLastError());
  return HM_OK;
}

// The pair -> 3-node hyperedge index of H, built on first use.
int ensure_pair_links(hm_graph* H, hipStream_t st) {
  note_use(H, st);
  if (H->pl_keys || H->n_by_size[3] == 0) return HM_OK;
  HM_TRY(refuse_capture(st));
  HM_TRY(ensure_hub_rows(H, st));
  const uint64_t n = 3 * H->n_by_size[3];
  int bits = 1;
  while (bits < 32 && (1ull << bits) < H->n_nodes) ++bits;
  // the index: at most n distinct keys, load at most 1/2
  const unsigned long long cap = pow2_capacity(n);
  Scratch tmp(st);
  unsigned long long *keys = nullptr, *slots = nullptr;
  uint32_t *t = nullptr, *tt = nullptr, *e = nullptr, *et = nullptr, *codeg = nullptr, *third = nullptr;
  uint8_t* adj = nullptr;
  HM_TRY(tmp.get(&keys, n));
  HM_TRY(tmp.get(&t, n));
  HM_TRY(tmp.get(&tt, n));
  HM_TRY(tmp.get(&e, n));
  HM_TRY(tmp.get(&et, n));
  HM_TRY(tmp.get(&slots, 2 * cap));
  HM_TRY(tmp.get(&codeg, cap));
  HM_TRY(tmp.get(&third, n));
  HM_TRY(tmp.get(&adj, n));
  const unsigned g = grid_cap(n, 256, 4096);
  k_pl_third_keys<<<g, 256, 0, st>>>(H->e3, n, t, e);
  HM_HIP(hipGetLastError());
  HM_TRY(radix_sort_pairs(t, e, tt, et, n, bits, st));
  if (2 * bits <= 32) HM_TRY(sort_by_pair<uint32_t>(H, n, bits, e, et, keys, st, tmp));
  else HM_TRY(sort_by_pair<unsigned long long>(H, n, bits, e, et, keys, st, tmp));
  HM_TRY(fill_u64(slots, kEmpty64, 2 * cap, st));
  k_pl_index_starts<<<g, 256, 0, st>>>(keys, n, slots, cap - 1);
  k_pl_index_counts<<<g, 256, 0, st>>>(keys, n, slots, cap - 1);
  k_pl_third<<<g, 256, 0, st>>>(H->e3, keys, e, n, H->hs2, third, adj);
  k_pl_codeg<<<grid_cap(n, kThreads, 8192), kThreads, 0, st>>>(view_of(H), keys, n, slots, cap - 1, H->hub_rank,
                                                               H->hub_bits, H->hub_words, codeg);
  HM_HIP(hipGetLastError());
  H->pl_edge = keep(tmp, e);
  H->pl_slot = keep(tmp, slots);
  H->pl_mask = cap - 1;
  H->pl_codeg = keep(tmp, codeg);
  H->pl_third = keep(tmp, third);
  H->pl_adj = keep(tmp, adj);
  H->pl_keys = keep(tmp, keys);
  return HM_OK;
}

PairLinks pair_links_of(const hm_graph* H) {
  PairLinks pl;
  pl.keys = H->pl_keys;
  pl.edge = H->pl_edge;
  pl.n = H->pl_keys ? 3 * H->n_by_size[3] : 0;
  pl.slot = reinterpret_cast<const ulonglong2*>(H->pl_slot);
  pl.mask = H->pl_mask;
  pl.codeg = H->pl_codeg;
  pl.third = H->pl_third;
  pl.adj = H->pl_adj;
  pl.q_slot = reinterpret_cast<const ulonglong2*>(H->q_slot);
  pl.q_mask = H->q_mask;
  pl.q_fourth = H->q_fourth;
  pl.q_bits = H->q_bits;
  pl.hub_rank = H->hub_rank;
  pl.hub_bits = H->hub_bits;
  pl.hub_w = H->hub_words;
  return pl;
}

// Dense rows: row i is that of the node of rank n - 1 - i, when it has at
// least min_deg pairwise neighbours.
__global__ void k_hub_ranks(const uint32_t* __restrict__ g2_off, const uint32_t* __restrict__ rank_of, uint32_t n,
                            uint32_t n_rows, uint32_t min_deg, int32_t* __restrict__ hub_rank) {
  for (uint64_t x = blockIdx.x * blockDim.x + threadIdx.x; x < n; x += gridDim.x * blockDim.x) {
    const uint32_t i = n - 1 - rank_of[x];
    hub_rank[x] = i < n_rows && g2_off[x + 1] - g2_off[x] >= min_deg ? int32_t(i) : -1;
  }
}

// One workgroup per dense row and range of kHubChunk words: the bits gather
// in LDS and go out once (an atomic per neighbour on device memory took 0.39
// ms for 363 rows of 2.3 MB, most of it the longest row).
constexpr uint32_t kHubChunk = 8192;
__global__ void __launch_bounds__(1024) k_hub_rows(const uint32_t* __restrict__ g2_off,
                                                   const uint32_t* __restrict__ g2_adj,
                                                   const uint32_t* __restrict__ node_of, uint32_t n, uint32_t n_rows,
                                                   uint32_t min_deg, uint32_t words, uint32_t chunks,
                                                   uint32_t* __restrict__ bits) {
  __shared__ uint32_t part[kHubChunk];
  for (uint64_t t = blockIdx.x; t < uint64_t(n_rows) * chunks; t += gridDim.x) {
    const uint32_t r = uint32_t(t / chunks), w0 = uint32_t(t % chunks) * kHubChunk;
    const uint32_t x = node_of[n - 1 - r], cnt = min(kHubChunk, words - w0);
    uint32_t b = g2_off[x], e = g2_off[x + 1];
    if (e - b < min_deg) continue;
    // the row's entries (ascending) in this range of words
    if (w0) b = upper_bound(g2_adj, b, e, w0 * 32 - 1);
    if (w0 + cnt < words) e = upper_bound(g2_adj, b, e, (w0 + cnt) * 32 - 1);
    __syncthreads();   // the previous part is written out
    for (uint32_t i = threadIdx.x; i < cnt; i += 1024) part[i] = 0;
    __syncthreads();
    for (uint32_t p = b + threadIdx.x; p < e; p += 1024) {
      const uint32_t z = g2_adj[p];
      atomicOr(&part[(z >> 5) - w0], 1u << (z & 31));
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < cnt; i += 1024) bits[uint64_t(r) * words + w0 + i] = part[i];
  }
}

// H->hub_rank and H->hub_bits: the nodes with at least hub_min_degree()
// pairwise neighbours, the highest ranks first (wedge.hip's order by degree),
// as many as fit in kHubRowBytes.  Built once per graph, without a host
// round trip.
int ensure_hub_rows(hm_graph* H, hipStream_t st) {
  note_use(H, st);
  if (H->hub_built) return HM_OK;
  HM_TRY(refuse_capture(st));
  const uint32_t n = H->n_nodes, min_deg = hub_min_degree();
  const uint32_t words = (n + 31) / 32;
  uint64_t rows = 0;
  if (n && min_deg && H->g2_off) {
    // at most 2 |E2| / min_deg nodes have that many neighbours
    rows = std::min<uint64_t>(kHubRowBytes / (uint64_t(words) * sizeof(uint32_t)), 2 * H->n_by_size[2] / min_deg);
    rows = std::min<uint64_t>(rows, n);
  }
  if (!rows) {
    H->hub_built = true;
    return HM_OK;
  }
  HM_TRY(ensure_ranks(H, st));
  Scratch kept(st);
  int32_t* rank = nullptr;
  uint32_t* bits = nullptr;
  HM_TRY(kept.get(&rank, n));
  HM_TRY(kept.get(&bits, rows * words));
  const uint32_t chunks = (words + kHubChunk - 1) / kHubChunk;
  k_hub_ranks<<<grid_cap(n, 256, 2048), 256, 0, st>>>(H->g2_off, H->rank_of, n, uint32_t(rows), min_deg, rank);
  k_hub_rows<<<grid_cap(rows * chunks, 1, 2048), 1024, 0, st>>>(H->g2_off, H->g2_adj, H->node_of, n, uint32_t(rows),
                                                                 min_deg, words, chunks, bits);
  HM_HIP(hipGetLastError());
  kept.ptrs.clear();
  H->hub_rank = rank;
  H->hub_bits = bits;
  H->hub_words = words;
  H->hub_built = true;
  return HM_OK;
}

// Fills the main, sub and G2 regions of H->hist (zeroed by the caller) except
// case (a), which the caller counts.
int count_sparse(const hm_graph* H, int k, hipStream_t st) {
  if (k == 4) HM_TRY(within_node_range(H));
  note_use(H, st);
  const uint8_t *lut4 = nullptr, *lut3 = nullptr;
  HM_TRY(device_luts(H->device, &lut4, &lut3));
  const View v = view_of(H);
  const uint64_t n2 = H->n_by_size[2];
  Scratch tmp(st);
  unsigned long long* acc = nullptr;
  uint32_t* tri_e = nullptr;
  HM_TRY(tmp.get(&acc, kAccN));
  HM_TRY(fill_u64(acc, 0, kAccN, st));
  if (n2 && k == 3 && probes_order3(n2, H->n_nodes)) {
    ProfileScope ps("k_sp_pair_probes", st);
    k_sp_pair_probes<<<grid_cap(n2, kWavesPerBlock * kProbePairs, 2048), kThreads, 0, st>>>(v, n2, acc);
  } else if (n2) {
    HM_TRY(tmp.get(&tri_e, n2));
    HM_TRY(wedge_counts(const_cast<hm_graph*>(H), k, tri_e, acc + kAccC4, acc + kAccK4, st));
    ProfileScope ps("k_sp_pairs", st);
    k_sp_pairs<<<grid_cap(n2, kThreads, 512), kThreads, 0, st>>>(v, n2, tri_e, acc);
  }
  {
    ProfileScope ps("k_sp_nodes", st);
    k_sp_nodes<<<grid_cap(H->n_nodes, kThreads, 512), kThreads, 0, st>>>(v, acc);
  }
  HM_HIP(hipGetLastError());
  const ClassTables& t = class_tables();
  ShapeClasses cls;
  // representative pair patterns (local nodes 0..3; bits: 01=0, 02=1, 12=2, 03=4, 13=5, 23=7)
  cls.k3_path = t.lut3[0x3];       // 01, 02
  cls.k3_triangle = t.lut3[0x7];   // 01, 02, 12
  cls.path = t.lut4[(1u << 0) | (1u << 2) | (1u << 7)];
  cls.star = t.lut4[(1u << 0) | (1u << 1) | (1u << 4)];
  cls.cycle = t.lut4[(1u << 0) | (1u << 2) | (1u << 7) | (1u << 4)];
  cls.paw = t.lut4[(1u << 0) | (1u << 1) | (1u << 2) | (1u << 4)];
  cls.diamond = t.lut4[(1u << 0) | (1u << 1) | (1u << 2) | (1u << 4) | (1u << 5)];
  cls.clique = t.lut4[kPairBits4];
  if (k == 4) HM_TRY(count_triples(H, st));
  k_sp_shapes<<<1, 64, 0, st>>>(acc, k, cls, H->hist);
  HM_HIP(hipGetLastError());
  return HM_OK;
}

}  // namespace hm
