// Neighbourhood of one 3-node hyperedge without adjacency bit rows, counted
// rather than enumerated (Algorithm 4's exploration around a sampled 3-node
// hyperedge), and the pair index that exact counting shares with it.
//
// For e = {a<b<c} the candidate sets are e u {v}.  A node v is *exceptional*
// when {a,b,v}, {a,c,v} or {b,c,v} is another 3-node hyperedge or {a,b,c,v}
// is a 4-node hyperedge; every other v has e as the only hyperedge of size
// >= 3 in e u {v}, so its class depends only on which of a, b, c it is
// paired with (the combination (av, bv, cv)).  The number of such v per
// combination follows from |N(a)|, |N(b)|, |N(c)|, the three pairwise and the
// triple intersection sizes (inclusion-exclusion, members of e excluded), less
// the exceptional v of that combination; exceptional v are classified one by
// one by fill-in, and every set whose largest hyperedge has 3 nodes counts.
#pragma once

#include "hm_items.h"

namespace hm {

// Pairs inside 3-node hyperedges, sorted: keys (x << 32) | y with x < y, and
// the position in e3 of the hyperedge each came from; a hash index (linear
// probing, slots of (key, start << 32 | count)) finds the run of one key.
struct PairLinks {
  const unsigned long long* keys;
  const uint32_t* edge;
  uint64_t n;
  const ulonglong2* slot;
  unsigned long long mask;
  const uint32_t* codeg;   // per slot: |N(x) n N(y)| in the pairwise graph
  // per entry: the third node t of its 3-node hyperedge, and t's pairwise
  // adjacency to the key's nodes (bit 0: x ~ t, bit 1: y ~ t)
  const uint32_t* third;
  const uint8_t* adj;
  // (the entries of a run are in ascending third node)
  // 4-node hyperedges by their 3-node subsets: for a < b < c, the run of the
  // key (a << 2q) | (b << q) | c (q = q_bits) in q_slot lists the fourth
  // nodes (q_fourth) of the 4-node hyperedges holding {a, b, c}; q_bits = 0
  // when not built (node ids too wide), and then the 4-node incidence list of
  // a member is walked instead
  const ulonglong2* q_slot;
  unsigned long long q_mask;
  const uint32_t* q_fourth;
  int q_bits;
  // dense adjacency rows of the highest-degree nodes: hub_rank[v] is v's row
  // (hub_w words at hub_bits + row * hub_w) or -1; hub_rank null: none
  const int32_t* hub_rank;
  const uint32_t* hub_bits;
  uint32_t hub_w;
};

// The dense adjacency row of x, or -1.
__device__ inline int hub_of(const PairLinks& pl, uint32_t x) { return pl.hub_rank ? pl.hub_rank[x] : -1; }
// Whether z is a pairwise neighbour of the node with dense row r.
__device__ inline uint32_t hub_adj(const PairLinks& pl, int r, uint32_t z) {
  return (pl.hub_bits[uint64_t(r) * pl.hub_w + (z >> 5)] >> (z & 31)) & 1u;
}

// Run [*lo, *lo + *len) of pl.keys holding `key` (empty when absent).
__device__ inline void pl_find(const PairLinks& pl, unsigned long long key, uint64_t* lo, uint32_t* len) {
  *lo = 0;
  *len = 0;
  if (!pl.n) return;
  unsigned long long h = mix64(key) & pl.mask;
  while (true) {
    const ulonglong2 s = pl.slot[h];
    if (s.x == key) {
      *lo = s.y >> 32;
      *len = uint32_t(s.y);
      return;
    }
    if (s.x == kEmpty64) return;
    h = (h + 1) & pl.mask;
  }
}

// Run [*lo, *lo + *len) of q_fourth: the fourth nodes of the 4-node
// hyperedges holding {a < b < c} (pl.q_bits != 0).
__device__ inline void quad_find(const PairLinks& pl, uint32_t a, uint32_t b, uint32_t c, uint64_t* lo,
                                 uint32_t* len) {
  const int q = pl.q_bits;
  const unsigned long long key = ((unsigned long long)a << (2 * q)) | ((unsigned long long)b << q) | c;
  *lo = 0;
  *len = 0;
  unsigned long long h = mix64(key) & pl.q_mask;
  while (true) {
    const ulonglong2 s = pl.q_slot[h];
    if (s.x == key) {
      *lo = s.y >> 32;
      *len = uint32_t(s.y);
      return;
    }
    if (s.x == kEmpty64) return;
    h = (h + 1) & pl.q_mask;
  }
}

// The number of common pairwise neighbours of x < y, a pair inside some
// 3-node hyperedge (so present in the index).
__device__ inline uint32_t pl_codeg(const PairLinks& pl, uint32_t x, uint32_t y) {
  const unsigned long long key = ((unsigned long long)x << 32) | y;
  unsigned long long h = mix64(key) & pl.mask;
  while (pl.slot[h].x != key) h = (h + 1) & pl.mask;
  return pl.codeg[h];
}

__device__ inline uint32_t deg2_of(const View& v, uint32_t x) { return v.g2_off[x + 1] - v.g2_off[x]; }

// The hyperedge e = {a<b<c} with its pairwise pattern and the ranges of its
// exceptional nodes: slot 0..2 the pair index entries of {a,b}, {a,c},
// {b,c}; slot 3 the fourth nodes of the 4-node hyperedges holding e (with
// pl.q_bits), else the 4-node hyperedges of the member with the fewest.
struct B4Ctx {
  uint32_t a, b, c, base_p;
  int ra, rb, rc;   // dense adjacency rows of a, b, c, or -1
  // named scalars, not arrays: a dynamically indexed array would live in scratch
  uint64_t lo0, lo1, lo2, lo3, len0, len1, len2, len3, total;
};

__device__ __forceinline__ uint64_t readlane_u64(uint64_t x, int lane) {
  return (uint64_t(uint32_t(__builtin_amdgcn_readlane(int(uint32_t(x >> 32)), lane))) << 32) |
         uint32_t(__builtin_amdgcn_readlane(int(uint32_t(x)), lane));
}

// Every lane of the wavefront calls this.  The ten lookups e needs are spread
// over lanes 0..9, which run the same probe loop each on its own table, so
// that they take one round of memory latency rather than ten in a row; the
// results are then read from those lanes.  Lanes 0..2: the pair index runs of
// {a,b}, {a,c}, {b,c}; 3..5: the pairs' membership in the pair set; 6: the
// run of e in the 4-node index; 7..9: the dense rows of a, b, c.
__device__ __forceinline__ B4Ctx b4_ctx(const View& v, const PairLinks& pl, uint32_t a, uint32_t b, uint32_t c) {
  const int lane = threadIdx.x & (kWave - 1);
  B4Ctx x;
  x.a = a;
  x.b = b;
  x.c = c;
  const unsigned long long* base = nullptr;
  unsigned long long key = 0, mask = 0;
  uint32_t stride = 2;   // 64-bit words per slot: key, then value
  if (lane < 3 && pl.n) {
    const uint32_t u = lane == 2 ? b : a, w = lane == 0 ? b : c;
    key = ((unsigned long long)u << 32) | w;
    base = reinterpret_cast<const unsigned long long*>(pl.slot);
    mask = pl.mask;
  } else if (lane >= 3 && lane < 6) {
    const uint32_t u = lane == 5 ? b : a, w = lane == 3 ? b : c;
    key = key2(u, w);
    base = v.hs2.slot;
    mask = v.hs2.mask;
    stride = 1;
  } else if (lane == 6 && pl.q_bits) {
    const int q = pl.q_bits;
    key = ((unsigned long long)a << (2 * q)) | ((unsigned long long)b << q) | c;
    base = reinterpret_cast<const unsigned long long*>(pl.q_slot);
    mask = pl.q_mask;
  }
  unsigned long long val = 0;
  if (base) {
    unsigned long long h = mix64(key) & mask;
    while (true) {
      const unsigned long long k = base[stride * h];
      if (k == key) {
        val = stride == 2 ? base[2 * h + 1] : 1ull;
        break;
      }
      if (k == kEmpty64) break;
      h = (h + 1) & mask;
    }
  } else if (lane >= 7 && lane < 10) {
    val = uint32_t(hub_of(pl, lane == 7 ? a : (lane == 8 ? b : c)));
  }
  // the same in every lane: kept in scalar registers
  const uint64_t r0 = readlane_u64(val, 0), r1 = readlane_u64(val, 1), r2 = readlane_u64(val, 2);
  x.lo0 = r0 >> 32;
  x.len0 = uint32_t(r0);
  x.lo1 = r1 >> 32;
  x.len1 = uint32_t(r1);
  x.lo2 = r2 >> 32;
  x.len2 = uint32_t(r2);
  x.base_p = uint32_t(__builtin_amdgcn_readlane(int(val), 3)) | (uint32_t(__builtin_amdgcn_readlane(int(val), 4)) << 1) |
             (uint32_t(__builtin_amdgcn_readlane(int(val), 5)) << 2) | (1u << 3);
  x.ra = __builtin_amdgcn_readlane(int(val), 7);
  x.rb = __builtin_amdgcn_readlane(int(val), 8);
  x.rc = __builtin_amdgcn_readlane(int(val), 9);
  if (pl.q_bits) {
    const uint64_t r6 = readlane_u64(val, 6);
    x.lo3 = r6 >> 32;
    x.len3 = uint32_t(r6);
  } else {
    const uint32_t fa = v.i4_off[a + 1] - v.i4_off[a], fb = v.i4_off[b + 1] - v.i4_off[b],
                   fc = v.i4_off[c + 1] - v.i4_off[c];
    const uint32_t m4 = (fa <= fb && fa <= fc) ? a : (fb <= fc ? b : c);
    x.lo3 = uniform_u64(v.i4_off[m4]);
    x.len3 = uniform_u64(v.i4_off[m4 + 1] - v.i4_off[m4]);
  }
  x.total = x.len0 + x.len1 + x.len2 + x.len3;
  return x;
}

// Number of nodes v outside e per pairwise combination (av | bv<<1 | cv<<2),
// exceptional ones included, valid in every lane: the smallest row walked
// against the other two members, the common neighbours of those two from
// the pair index; inclusion-exclusion with the members of e removed.
__device__ __forceinline__ void b4_combo_counts(const View& v, const PairLinks& pl, const B4Ctx& x, uint32_t n[8]) {
  const int lane = threadIdx.x & (kWave - 1);
  const uint32_t a = x.a, b = x.b, c = x.c;
  const uint32_t pab = x.base_p & 1u, pac = (x.base_p >> 1) & 1u, pbc = (x.base_p >> 2) & 1u;
  const uint32_t da = deg2_of(v, a), db = deg2_of(v, b), dc = deg2_of(v, c);
  uint32_t r1, x1, y1, r2, x2;   // rows walked and the members they are probed against
  if (da <= db && da <= dc) {
    r1 = a; x1 = b; y1 = c;
    r2 = db <= dc ? b : c; x2 = db <= dc ? c : b;
  } else if (db <= dc) {
    r1 = b; x1 = a; y1 = c;
    r2 = da <= dc ? a : c; x2 = da <= dc ? c : a;
  } else {
    r1 = c; x1 = a; y1 = b;
    r2 = da <= db ? a : b; x2 = da <= db ? b : a;
  }
  uint32_t n1x = 0, n1y = 0, n1xy = 0;
  const uint32_t b1 = v.g2_off[r1], l1 = v.g2_off[r1 + 1] - b1;
  const int ra = x.ra, rb = x.rb, rc = x.rc;
  const int hx1 = x1 == a ? ra : (x1 == b ? rb : rc), hy1 = y1 == a ? ra : (y1 == b ? rb : rc);
  for (uint32_t t = lane; t < l1; t += kWave) {
    const uint32_t z = v.g2_adj[b1 + t];
    Probe64 px, py;
    if (hx1 < 0) px = probe2_start(v.hs2, x1, z);
    if (hy1 < 0) py = probe2_start(v.hs2, y1, z);
    const uint32_t hx = hx1 >= 0 ? hub_adj(pl, hx1, z) : uint32_t(probe64_end(v.hs2, px));
    const uint32_t hy = hy1 >= 0 ? hub_adj(pl, hy1, z) : uint32_t(probe64_end(v.hs2, py));
    n1x += hx;
    n1y += hy;
    n1xy += hx & hy;
  }
  n1x = wave_sum_u32(n1x);
  n1y = wave_sum_u32(n1y);
  n1xy = wave_sum_u32(n1xy);
  const uint32_t n2x = pl_codeg(pl, min(r2, x2), max(r2, x2));
  const uint32_t tri = n1xy;
  uint32_t cab, cac, cbc;
  if (r1 == a) { cab = n1x; cac = n1y; cbc = n2x; }
  else if (r1 == b) { cab = n1x; cbc = n1y; cac = n2x; }
  else { cac = n1x; cbc = n1y; cab = n2x; }
  const uint32_t sa = da - pab - pac, sb = db - pab - pbc, sc = dc - pac - pbc;
  const uint32_t iab = cab - pac * pbc, iac = cac - pab * pbc, ibc = cbc - pab * pac;
  n[0] = 0;
  n[7] = tri;
  n[3] = iab - tri;
  n[5] = iac - tri;
  n[6] = ibc - tri;
  n[1] = sa - n[3] - n[5] - n[7];
  n[2] = sb - n[3] - n[6] - n[7];
  n[4] = sc - n[5] - n[6] - n[7];
}

// The exceptional node at flat position t of the ranges of x, each node
// once (by the first hyperedge that makes it exceptional).  Returns 0 when the
// position holds none; else bit 4 set, its pairwise combination in bits 0..2,
// bit 3 set when its set counts (not a 4-node hyperedge), with the set's
// pattern in *pat.
//
// b4_exception_node takes the node itself: y with its slot (0..2: the third
// node of a 3-node hyperedge on pair {a,b}, {a,c} or {b,c} of e, pair_adj its
// pairwise adjacency to that pair's lower and higher node in bits 0 and 1;
// 3: the fourth node of a 4-node hyperedge holding e, pair_adj unused).
__device__ __forceinline__ uint32_t b4_exception_node(const View& v, const PairLinks& pl, const B4Ctx& x, int slot,
                                                      uint32_t y, uint32_t pair_adj, uint32_t* pat) {
  const uint32_t a = x.a, b = x.b, c = x.c;
  const int ra = x.ra, rb = x.rb, rc = x.rc;
  if (slot < 3 && (y == a || y == b || y == c)) return 0;   // e itself
  // Every membership test the set e u {y} needs, issued together: the
  // 3-node sets through y not already known from the slot, the 4-node set
  // (unless the slot is the 4-node hyperedges'), y's pairs with a, b, c.
  Probe128 pab, pac, pbc, pq;
  if (slot != 0) pab = probe3_start(v.hs3, a, b, y);
  if (slot != 1) pac = probe3_start(v.hs3, a, c, y);
  if (slot != 2) pbc = probe3_start(v.hs3, b, c, y);
  if (slot < 3) {
    uint32_t s0 = a, s1 = b, s2 = c, s3 = y;
    // ascending 4-tuple for the 4-node probe
    if (s3 < s2) { const uint32_t tt = s2; s2 = s3; s3 = tt; }
    if (s2 < s1) { const uint32_t tt = s1; s1 = s2; s2 = tt; }
    if (s1 < s0) { const uint32_t tt = s0; s0 = s1; s1 = tt; }
    pq = probe128_start(v.hs4, key4(s0, s1, s2, s3));
  }
  // y's pairs with the two members of the slot's pair come with the entry
  Probe64 pa, pb, pc;
  if ((slot == 2 || slot == 3) && ra < 0) pa = probe2_start(v.hs2, a, y);
  if ((slot == 1 || slot == 3) && rb < 0) pb = probe2_start(v.hs2, b, y);
  if ((slot == 0 || slot == 3) && rc < 0) pc = probe2_start(v.hs2, c, y);
  const uint32_t abv = slot == 0 ? 1u : uint32_t(probe128_end(v.hs3, pab));
  const uint32_t acv = slot == 1 ? 1u : uint32_t(probe128_end(v.hs3, pac));
  const uint32_t bcv = slot == 2 ? 1u : uint32_t(probe128_end(v.hs3, pbc));
  // each exceptional node once: a 3-node hyperedge of an earlier slot takes it
  if (slot == 1 && abv) return 0;
  if (slot == 2 && (abv || acv)) return 0;
  if (slot == 3 && (abv || acv || bcv)) return 0;
  const uint32_t quad = slot == 3 ? 1u : uint32_t(probe128_end(v.hs4, pq));
  const uint32_t av = slot == 0 || slot == 1 ? (pair_adj & 1u)
                                             : (ra >= 0 ? hub_adj(pl, ra, y) : uint32_t(probe64_end(v.hs2, pa)));
  const uint32_t bv = slot == 0 ? (pair_adj >> 1)
                                : (slot == 2 ? (pair_adj & 1u)
                                             : (rb >= 0 ? hub_adj(pl, rb, y) : uint32_t(probe64_end(v.hs2, pb))));
  const uint32_t cv = slot == 1 || slot == 2 ? (pair_adj >> 1)
                                             : (rc >= 0 ? hub_adj(pl, rc, y) : uint32_t(probe64_end(v.hs2, pc)));
  const uint32_t combo = av | (bv << 1) | (cv << 2);
  *pat = x.base_p | (av << 4) | (bv << 5) | (abv << 6) | (cv << 7) | (acv << 8) | (bcv << 9);
  // (a 4-node hyperedge is larger than the sampled 3-node one)
  return 16u | (quad ? 0u : 8u) | combo;
}

__device__ __forceinline__ uint32_t b4_exception(const View& v, const PairLinks& pl, const B4Ctx& x, uint64_t t,
                                                 uint32_t* pat) {
  // slot and offset of t, with constant indices only (registers)
  if (t < x.len0) {
    const uint64_t p = x.lo0 + t;
    return b4_exception_node(v, pl, x, 0, pl.third[p], pl.adj[p], pat);
  }
  if (t < x.len0 + x.len1) {
    const uint64_t p = x.lo1 + (t - x.len0);
    return b4_exception_node(v, pl, x, 1, pl.third[p], pl.adj[p], pat);
  }
  if (t < x.len0 + x.len1 + x.len2) {
    const uint64_t p = x.lo2 + (t - x.len0 - x.len1);
    return b4_exception_node(v, pl, x, 2, pl.third[p], pl.adj[p], pat);
  }
  if (pl.q_bits)
    return b4_exception_node(v, pl, x, 3, pl.q_fourth[x.lo3 + (t - x.len0 - x.len1 - x.len2)], 0u, pat);
  const uint32_t* f = v.e4 + 4ull * v.i4_idx[x.lo3 + (t - x.len0 - x.len1 - x.len2)];
  const uint32_t f0 = f[0], f1 = f[1], f2 = f[2], f3 = f[3];
  const uint32_t a = x.a, b = x.b, c = x.c;
  const uint32_t hit = uint32_t(f0 == a || f0 == b || f0 == c) + uint32_t(f1 == a || f1 == b || f1 == c) +
                       uint32_t(f2 == a || f2 == b || f2 == c) + uint32_t(f3 == a || f3 == b || f3 == c);
  if (hit != 3) return 0;
  return b4_exception_node(v, pl, x, 3, f0 ^ f1 ^ f2 ^ f3 ^ a ^ b ^ c, 0u, pat);
}

// The combination pattern of e u {v} for a non-exceptional v.
__device__ inline uint32_t b4_combo_pattern(const B4Ctx& x, uint32_t cmb) {
  return x.base_p | ((cmb & 1u) << 4) | (((cmb >> 1) & 1u) << 5) | ((cmb >> 2) << 7);
}

// Position of node z among the third nodes of the run [lo, lo + len) (sorted),
// or ~0 when absent.
__device__ inline uint64_t run_find(const PairLinks& pl, uint64_t lo, uint32_t len, uint32_t z) {
  uint64_t l = lo, h = lo + len;   // pl.third[l..h) may hold z
  while (h > l) {
    const uint64_t m = l + ((h - l) >> 1);
    const uint32_t y = pl.third[m];
    if (y == z) return m;
    if (y < z) l = m + 1; else h = m;
  }
  return ~0ull;
}

// (sparse.hip; the indices that are not built yet are left out)
PairLinks pair_links_of(const hm_graph* H);
// triples.hip: the sets around 3-node hyperedges, added to H->hist
int count_triples(const hm_graph* H, hipStream_t st);

}  // namespace hm
