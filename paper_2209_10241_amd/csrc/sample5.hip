// Sampled counting of order-5 higher-order motifs (Section 6.4 applies the
// sampling algorithm of Section 5 at order 5, where exact counting does not
// reach).
//
// Algorithm 4 at order 5: every sampled hyperedge e of size j (j = 2..5)
// takes every 5-node set V containing e whose induced sub-hypergraph is
// connected and holds no hyperedge larger than e; such a V lies within
// 5 - j hops of e through hyperedges of size at most j.  One workgroup per
// sample lists that ball in LDS (a hash set and a list), then its threads
// stride over the C(|ball|, 5 - j) choices of the other nodes, fill each set
// in (26 subsets: pairs, triples, quadruples and the set itself, Section 4.3)
// and classify it.
//
// That is the general path.  Hypergraphs of at most kDense5MaxNodes nodes
// with adjacency bit rows take the dense path instead (k_dense5), unless a call's
// samples can meet few sets (dense5_pays): with the
// 3-node hyperedges also kept as bit rows, one row of z per node pair, the
// sets around a sampled pair are counted 32 at a time by popcounts.
//
// At order 5 there are 2^26 patterns, too many for a lookup table in LDS:
// counts gather by pattern (of any labelling of the five nodes), in LDS per
// workgroup and then in a device hash table; one launch then puts each
// distinct pattern in canonical form, its smallest value over the 120
// relabellings, and adds it to the class table.  Classes are reported in
// ascending canonical order, scaled: est = raw |E_j| / (S_j countmax), j the
// class's largest hyperedge size and countmax the number of its hyperedges
// of that size.
#include <algorithm>
#include <cmath>
#include <vector>

#include "hm_items.h"

namespace hm {

int sample_sizes(const hm_graph* H, int k, double fraction, int allocation, uint64_t* S);

namespace {

constexpr int kSub5 = 26;
constexpr uint32_t kBallCap = 4096;           // ball nodes per sample
constexpr uint32_t kLocalCap = 1024;          // classes cached per workgroup
constexpr uint32_t kThreads5 = 256;
constexpr uint64_t kMaxCandidates = 1ull << 32;   // per sample
constexpr uint32_t kErrBall = 1u, kErrWork = 2u, kErrTable = 4u;
// slots of the pattern table: a pattern that finds no room goes to the class
// table at once, in canonical form
constexpr uint32_t kRawSlots = 1u << 19;

struct Tables5 {
  uint8_t sub_mask[kSub5];       // subset masks of {0..4} with >= 2 members, ascending
  int8_t bit_of_mask[32];
  uint8_t perm[120][5];
};

Tables5 make_tables5() {
  Tables5 t{};
  int n = 0;
  for (int m = 0; m < 32; ++m) {
    t.bit_of_mask[m] = -1;
    if (__builtin_popcount(m) >= 2) {
      t.bit_of_mask[m] = int8_t(n);
      t.sub_mask[n++] = uint8_t(m);
    }
  }
  uint8_t p[5] = {0, 1, 2, 3, 4};
  int q = 0;
  do {
    for (int i = 0; i < 5; ++i) t.perm[q][i] = p[i];
    ++q;
  } while (std::next_permutation(p, p + 5));
  return t;
}

// ------------------------------------------------------------------ 5-node hyperedges
__device__ inline unsigned long long hash5(const uint32_t* m) {
  unsigned long long h = 0x6a09e667f3bcc909ull;
  for (int i = 0; i < 5; ++i) h = mix64(h ^ (m[i] + 0x9e3779b97f4a7c15ull * uint64_t(i + 1)));
  return h;
}

// every unique hyperedge of size 5 of the all-hyperedges list: flags
__global__ void k_e5_flags(const unsigned long long* __restrict__ off, uint64_t n, uint32_t* __restrict__ flag) {
  for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += uint64_t(gridDim.x) * blockDim.x)
    flag[i] = off[i + 1] - off[i] == 5 ? 1u : 0u;
}

__global__ void k_e5_gather(const unsigned long long* __restrict__ off, const uint32_t* __restrict__ members, uint64_t n,
                            const uint32_t* __restrict__ flag, const uint32_t* __restrict__ pos, uint32_t* __restrict__ e5) {
  for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += uint64_t(gridDim.x) * blockDim.x)
    if (flag[i])
      for (int j = 0; j < 5; ++j) e5[5ull * pos[i] + j] = members[off[i] + j];
}

__global__ void k_e5_insert(const uint32_t* __restrict__ e5, uint64_t n5, uint32_t* slots, unsigned long long mask) {
  for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n5; i += uint64_t(gridDim.x) * blockDim.x) {
    unsigned long long h = hash5(e5 + 5 * i) & mask;
    while (atomicCAS(&slots[h], 0u, uint32_t(i + 1)) != 0u) h = (h + 1) & mask;
  }
}

__device__ inline bool has5(const uint32_t* __restrict__ e5, const uint32_t* __restrict__ slots, unsigned long long mask,
                            const uint32_t* m) {
  if (!slots) return false;
  unsigned long long h = hash5(m) & mask;
  for (;;) {
    const uint32_t s = slots[h];
    if (s == 0u) return false;
    const uint32_t* r = e5 + 5ull * (s - 1);
    if (r[0] == m[0] && r[1] == m[1] && r[2] == m[2] && r[3] == m[3] && r[4] == m[4]) return true;
    h = (h + 1) & mask;
  }
}

// ------------------------------------------------------------------ the counting kernel
struct Sampled5Args {
  View v;
  const uint32_t* e5;
  const uint32_t* hs5;
  unsigned long long hs5_mask;
  const uint32_t* idx[6];       // explicit draws per stratum, or null: drawn here
  uint64_t S[6];                // draws per stratum
  uint64_t n[6];                // |E_j|
  uint64_t seed;
  // device pattern table: key = pattern + 1 (0 empty), count
  uint32_t* raw_keys;
  unsigned long long* raw_counts;
  // device class table: key = canonical + 1 (0 empty), count
  uint32_t* keys;
  unsigned long long* counts;
  unsigned long long mask;
  uint32_t* err;
};

__device__ inline const uint32_t* edge_row(const Sampled5Args& a, int j, uint64_t i) {
  return j == 2 ? a.v.e2 + 2 * i : j == 3 ? a.v.e3 + 3 * i : j == 4 ? a.v.e4 + 4 * i : a.e5 + 5 * i;
}

// (The key is looked for with a plain load first: an atomic that returns a
// value to many workgroups from one address is served one at a time.)
__device__ inline void add_global(const Sampled5Args& a, uint32_t canon, unsigned long long cnt) {
  const uint32_t key = canon + 1u;
  unsigned long long h = mix64(canon) & a.mask;
  for (uint64_t probes = 0; probes <= a.mask; ++probes) {
    uint32_t cur = __hip_atomic_load(&a.keys[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (cur == 0u) cur = atomicCAS(&a.keys[h], 0u, key);
    if (cur == 0u || cur == key) {
      atomicAdd(&a.counts[h], cnt);
      return;
    }
    h = (h + 1) & a.mask;
  }
  atomicOr(a.err, kErrTable);
}

// fill-in of the 5-node set V (ascending): bit b for the b-th subset
// The subsets of the five local positions with at least two members, in
// ascending mask order (the order of Tables5::sub_mask and of the pattern's
// bits), as constants so that fill5's loops unroll to fixed subsets.
constexpr uint8_t kSubMask5[kSub5] = {3,  5,  6,  7,  9,  10, 11, 12, 13, 14, 15, 17, 18,
                                      19, 20, 21, 22, 23, 24, 25, 26, 27, 28, 29, 30, 31};

// The 26-bit pattern of the ascending 5-node set V: bit b set when subset b
// of V is a hyperedge.  The home slots of the ten 3-node and five 4-node
// subsets are loaded before any probe is resolved, so that their latencies
// overlap; a probe that meets another key continues from there.
__device__ inline uint32_t fill5(const Sampled5Args& a, const Tables5& T, const uint32_t* V) {
  (void)T;
  uint32_t p = 0;
  ulonglong2 home[kSub5];
#pragma unroll
  for (int b = 0; b < kSub5; ++b) {
    const uint32_t m = kSubMask5[b];
    const int n = __builtin_popcount(m);
    uint32_t x[5];
    int k = 0;
#pragma unroll
    for (int i = 0; i < 5; ++i)
      if ((m >> i) & 1u) x[k++] = V[i];
    if (n == 2) {
      p |= pair_bit(a.v.hs2, a.v.bits, a.v.W, x[0], x[1]) << b;
    } else if (n == 3 || n == 4) {
      const Key128 key = n == 3 ? key3(x[0], x[1], x[2]) : key4(x[0], x[1], x[2], x[3]);
      const Set128& set = n == 3 ? a.v.hs3 : a.v.hs4;
      home[b] = *reinterpret_cast<const ulonglong2*>(set.slot + 2 * (hash128(key) & set.mask));
    }
  }
#pragma unroll
  for (int b = 0; b < kSub5; ++b) {
    const uint32_t m = kSubMask5[b];
    const int n = __builtin_popcount(m);
    uint32_t x[5];
    int k = 0;
#pragma unroll
    for (int i = 0; i < 5; ++i)
      if ((m >> i) & 1u) x[k++] = V[i];
    if (n == 3 || n == 4) {
      const Key128 key = n == 3 ? key3(x[0], x[1], x[2]) : key4(x[0], x[1], x[2], x[3]);
      const Set128& set = n == 3 ? a.v.hs3 : a.v.hs4;
      bool has = false;
      ulonglong2 v = home[b];
      if (v.x == key.hi && v.y == key.lo) {
        has = true;
      } else if (v.x != kEmpty64) {
        Probe128 pr;
        pr.key = key;
        pr.pos = ((hash128(key) & set.mask) + 1) & set.mask;
        pr.v = *reinterpret_cast<const ulonglong2*>(set.slot + 2 * pr.pos);
        has = probe128_end(set, pr);
      }
      p |= uint32_t(has) << b;
    } else if (n == 5) {
      p |= uint32_t(has5(a.e5, a.hs5, a.hs5_mask, x)) << b;
    }
  }
  return p;
}

__device__ inline bool connected5(const Tables5& T, uint32_t p) {
  uint32_t adj[5] = {0, 0, 0, 0, 0};
  uint32_t covered = 0;
  for (int b = 0; b < kSub5; ++b)
    if ((p >> b) & 1u) {
      const uint32_t m = T.sub_mask[b];
      covered |= m;
      for (int i = 0; i < 5; ++i)
        if ((m >> i) & 1u) adj[i] |= m;
    }
  if (covered != 31u) return false;
  uint32_t reach = 1u, prev = 0u;
  while (reach != prev) {
    prev = reach;
    for (int i = 0; i < 5; ++i)
      if ((reach >> i) & 1u) reach |= adj[i];
  }
  return reach == 31u;
}

__device__ inline int maxcard5(const Tables5& T, uint32_t p) {
  int mc = 0;
  for (int b = 0; b < kSub5; ++b)
    if ((p >> b) & 1u) mc = max(mc, __popc(T.sub_mask[b]));
  return mc;
}

__device__ inline uint32_t canonical5(const Tables5& T, uint32_t p) {
  uint32_t best = 0xFFFFFFFFu;
  for (int g = 0; g < 120; ++g) {
    uint32_t q = 0;
    for (uint32_t r = p; r; r &= r - 1) {
      const uint32_t m = T.sub_mask[__ffs(r) - 1];
      uint32_t img = 0;
      for (int i = 0; i < 5; ++i)
        if ((m >> i) & 1u) img |= 1u << T.perm[g][i];
      q |= 1u << T.bit_of_mask[img];
    }
    best = min(best, q);
  }
  return best;
}

// cnt sets of pattern p (the key looked for as in add_global).
__device__ inline void add_raw(const Tables5& T, const Sampled5Args& a, uint32_t p, unsigned long long cnt) {
  const uint32_t key = p + 1u;
  uint32_t h = uint32_t(mix64(key)) & (kRawSlots - 1);
  for (int probes = 0; probes < 64; ++probes) {
    uint32_t cur = __hip_atomic_load(&a.raw_keys[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (cur == 0u) cur = atomicCAS(&a.raw_keys[h], 0u, key);
    if (cur == 0u || cur == key) {
      atomicAdd(&a.raw_counts[h], cnt);
      return;
    }
    h = (h + 1) & (kRawSlots - 1);
  }
  add_global(a, canonical5(T, p), cnt);
}

// largest k with C(k, r) <= t (r = 1, 2, 3), k >= r - 1
__device__ inline uint64_t binom(uint64_t n, int r) {
  return r == 1 ? n : r == 2 ? n * (n - 1) / 2 : n * (n - 1) * (n - 2) / 6;
}

__device__ inline uint64_t colex_top(uint64_t t, int r) {
  double x = r == 1 ? double(t) : r == 2 ? sqrt(2.0 * double(t)) : cbrt(6.0 * double(t));
  uint64_t k = uint64_t(x) + 2;
  while (k > uint64_t(r - 1) && binom(k, r) > t) --k;
  while (binom(k + 1, r) <= t) ++k;
  return k;
}

// LDS of a workgroup
struct Lds5 {
  Tables5 T;
  uint32_t set[2 * kBallCap];     // open addressing, node + 1 (0 empty)
  uint32_t ball[kBallCap];
  uint32_t n_ball;
  uint32_t overflow;
  uint32_t lkeys[kLocalCap];      // pattern + 1 (add_local)
  unsigned long long lcount[kLocalCap];
};

__device__ inline bool ball_insert(Lds5& L, uint32_t node) {
  uint32_t h = uint32_t(mix64(node)) & (2 * kBallCap - 1);
  for (uint32_t probes = 0; probes < 2 * kBallCap; ++probes) {
    const uint32_t cur = atomicCAS(&L.set[h], 0u, node + 1u);
    if (cur == 0u) return true;
    if (cur == node + 1u) return false;
    h = (h + 1) & (2 * kBallCap - 1);
  }
  return false;
}

// The workgroup's counts are kept by pattern (key p + 1, 0 empty), since
// patterns repeat across a sample's candidate sets; a set that finds no room
// goes to the pattern table at once.
template <typename Lds>
__device__ inline void add_local(Lds& L, const Sampled5Args& a, uint32_t p) {
  const uint32_t key = p + 1u;
  uint32_t h = uint32_t(mix64(key)) & (kLocalCap - 1);
  for (int probes = 0; probes < 16; ++probes) {
    const uint32_t cur = atomicCAS(&L.lkeys[h], 0u, key);
    if (cur == 0u || cur == key) {
      atomicAdd(&L.lcount[h], 1ull);
      return;
    }
    h = (h + 1) & (kLocalCap - 1);
  }
  add_raw(L.T, a, p, 1ull);
}

template <typename Lds>
__device__ inline void clear_local(Lds& L) {
  for (uint32_t i = threadIdx.x; i < kLocalCap; i += blockDim.x) {
    L.lkeys[i] = 0u;
    L.lcount[i] = 0ull;
  }
}

template <typename Lds>
__device__ inline void flush_local(const Lds& L, const Sampled5Args& a) {
  for (uint32_t x = threadIdx.x; x < kLocalCap; x += blockDim.x)
    if (L.lkeys[x]) add_raw(L.T, a, L.lkeys[x] - 1u, L.lcount[x]);
}

// Sample s of the launch: its stratum j and the position i of its hyperedge
// in that stratum (explicit, or drawn from the seed).
__device__ inline void sample_of(const Sampled5Args& a, uint64_t s, int* j_out, uint64_t* i_out) {
  int j = 2;
  uint64_t r = s;
  while (r >= a.S[j]) r -= a.S[j++];
  *j_out = j;
  *i_out = a.idx[j] ? a.idx[j][r]
                    : bounded64(philox4x64_10(r, 0, 0, 0, a.seed, (kDomainSample << 32) | uint64_t(j)).v[0], a.n[j]);
}

// The ball of a sampled hyperedge e (j nodes): every node within 5 - j hops
// of e through hyperedges of size 2..4 (and, for j = 5, none), e's own
// nodes left out, in L.ball[0 .. L.n_ball) in ascending node order, so that
// every workgroup that builds it enumerates the same candidate sets in the
// same order.  Returns false (L.overflow set) when it holds more than
// kBallCap nodes.  Every thread of the workgroup calls this.
__device__ bool ball5(Lds5& L, const Sampled5Args& a, const uint32_t* e, int j) {
  const int need = 5 - j;
  __syncthreads();   // the previous ball is no longer read
  for (uint32_t x = threadIdx.x; x < 2 * kBallCap; x += blockDim.x) L.set[x] = 0u;
  if (threadIdx.x == 0) {
    L.n_ball = 0;
    L.overflow = 0;
  }
  __syncthreads();
  if (threadIdx.x < uint32_t(j)) ball_insert(L, e[threadIdx.x]);
  __syncthreads();
  // breadth-first: hop h takes the nodes added by hop h - 1 (e itself first)
  uint32_t f0 = 0, f1 = 0;
  for (int h = 0; h < need; ++h) {
    const uint32_t nf = h == 0 ? uint32_t(j) : f1 - f0;
    const int wv = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
    for (uint32_t q = wv; q < nf; q += kThreads5 / kWave) {
      const uint32_t u = h == 0 ? e[q] : L.ball[f0 + q];
      // pairs
      for (uint32_t t = a.v.g2_off[u] + lane; t < a.v.g2_off[u + 1]; t += kWave) {
        const uint32_t w = a.v.g2_adj[t];
        if (ball_insert(L, w)) {
          const uint32_t at = atomicAdd(&L.n_ball, 1u);
          if (at < kBallCap) L.ball[at] = w; else L.overflow = 1u;
        }
      }
      for (int fs = 3; fs <= j && fs <= 4; ++fs) {
        const uint32_t* off = fs == 3 ? a.v.i3_off : a.v.i4_off;
        const uint32_t* idx = fs == 3 ? a.v.i3_idx : a.v.i4_idx;
        const uint32_t* rows = fs == 3 ? a.v.e3 : a.v.e4;
        for (uint32_t t = off[u] + lane; t < off[u + 1]; t += kWave) {
          const uint32_t* f = rows + uint64_t(fs) * idx[t];
          for (int m = 0; m < fs; ++m)
            if (ball_insert(L, f[m])) {
              const uint32_t at = atomicAdd(&L.n_ball, 1u);
              if (at < kBallCap) L.ball[at] = f[m]; else L.overflow = 1u;
            }
        }
      }
    }
    __syncthreads();
    f0 = h == 0 ? 0u : f1;
    f1 = min(L.n_ball, kBallCap);
    if (L.overflow) break;
  }
  if (L.overflow) return false;
  // ascending order (bitonic sort in LDS, padded with ~0 to a power of two)
  const uint32_t nb = L.n_ball;
  uint32_t pad = 1;
  while (pad < nb) pad <<= 1;
  for (uint32_t x = nb + threadIdx.x; x < pad; x += blockDim.x) L.ball[x] = 0xFFFFFFFFu;
  __syncthreads();
  for (uint32_t k = 2; k <= pad; k <<= 1)
    for (uint32_t d = k >> 1; d > 0; d >>= 1) {
      for (uint32_t x = threadIdx.x; x < pad; x += blockDim.x) {
        const uint32_t y = x ^ d;
        if (y <= x) continue;
        const uint32_t vx = L.ball[x], vy = L.ball[y];
        if ((vx > vy) == ((x & k) == 0)) {
          L.ball[x] = vy;
          L.ball[y] = vx;
        }
      }
      __syncthreads();
    }
  return true;
}

// Candidate sets of a sample: the choices of 5 - j ball nodes (one set, e
// itself, when j = 5).
__device__ inline uint64_t candidates5(uint32_t nb, int j) {
  const int need = 5 - j;
  return need ? (nb >= uint64_t(need) ? binom(nb, need) : 0) : 1;
}

// Pass 1: every sample's number of candidate chunks (kChunk5 candidate sets
// each; 0 when its ball or its candidates are too many, with the error bit
// set).  One workgroup per sample.
constexpr uint64_t kChunk5 = 1ull << 16;
__global__ void __launch_bounds__(kThreads5) k_chunks5(Sampled5Args a, uint64_t total, uint32_t* __restrict__ chunks) {
  __shared__ Lds5 L;
  for (uint64_t s = blockIdx.x; s < total; s += gridDim.x) {
    int j;
    uint64_t i;
    sample_of(a, s, &j, &i);
    const uint32_t* e = edge_row(a, j, i);
    uint32_t c = 0;
    if (!ball5(L, a, e, j)) {
      if (threadIdx.x == 0) atomicOr(a.err, kErrBall);
    } else {
      const uint64_t cand = candidates5(L.n_ball, j);
      if (cand >= kMaxCandidates) {
        if (threadIdx.x == 0) atomicOr(a.err, kErrWork);
      } else {
        c = uint32_t((cand + kChunk5 - 1) / kChunk5);
      }
    }
    if (threadIdx.x == 0) chunks[s] = c;
  }
}

// Pass 2: the tasks (sample, chunk), tasks [first[s], first[s + 1]) being
// sample s's chunks (first: exclusive scan of the chunk counts, first[total]
// their sum).  A workgroup takes tasks in turn, rebuilds the task's ball and
// classifies the task's candidate sets: with the ball in ascending order,
// candidate t is the t-th choice of 5 - j ball nodes in colex order.
__global__ void __launch_bounds__(kThreads5) k_sampled5(Sampled5Args a, Tables5 tables, uint64_t total,
                                                        const uint32_t* __restrict__ first) {
  __shared__ Lds5 L;
  clear_local(L);
  if (threadIdx.x == 0) L.T = tables;
  const uint32_t n_tasks = first[total];
  for (uint32_t task = blockIdx.x; task < n_tasks; task += gridDim.x) {
    // the sample whose task range holds `task`
    uint64_t lo = 0, hi = total;   // first[lo] <= task < first[hi]
    while (hi - lo > 1) {
      const uint64_t mid = (lo + hi) >> 1;
      if (first[mid] <= task) lo = mid; else hi = mid;
    }
    const uint64_t s = lo;
    int j;
    uint64_t i;
    sample_of(a, s, &j, &i);
    const uint32_t* e = edge_row(a, j, i);
    const int need = 5 - j;
    if (!ball5(L, a, e, j)) continue;   // (pass 1 gave it no task)
    const uint64_t cand = candidates5(L.n_ball, j);
    const uint64_t c0 = uint64_t(task - first[s]) * kChunk5, c1 = min(cand, c0 + kChunk5);
    for (uint64_t t = c0 + threadIdx.x; t < c1; t += blockDim.x) {
      uint32_t V[5];
      for (int m = 0; m < j; ++m) V[m] = e[m];
      // the t-th choice of `need` ball nodes, colex order
      uint64_t rest = t;
      for (int rr = need; rr >= 1; --rr) {
        const uint64_t top = colex_top(rest, rr);
        rest -= binom(top, rr);
        V[j + need - rr] = L.ball[top];
      }
      for (int x = 1; x < 5; ++x) {   // ascending node ids
        const uint32_t y = V[x];
        int z = x - 1;
        while (z >= 0 && V[z] > y) {
          V[z + 1] = V[z];
          --z;
        }
        V[z + 1] = y;
      }
      const uint32_t p = fill5(a, L.T, V);
      if (maxcard5(L.T, p) != j || !connected5(L.T, p)) continue;
      add_local(L, a, p);
    }
  }
  __syncthreads();
  flush_local(L, a);
}

// ------------------------------------------------------------------ the dense path
// Bit tensors over node pairs: row (p, q) of N bits (W words).  t3: the nodes
// z with {p, q, z} a 3-node hyperedge.  f4 and f5: the nodes z such that some
// 4-node (5-node) hyperedge holds p, q and z, a necessary condition that
// spares nearly every probe of the hash sets for the larger hyperedges.
struct Dense5 {
  uint32_t *t3, *f4, *f5;
};
// 3 N^2 W words: 3.4 MB at N = 200, 402 MB at the limit, kept with the graph
// (see dense5_pays).
constexpr uint32_t kDense5MaxNodes = 1024;
constexpr uint32_t kDense5MaxWords = kDense5MaxNodes / 32;

template <int S>
__device__ inline void dense_mark(const uint32_t* __restrict__ m, uint32_t N, uint32_t W, uint32_t* __restrict__ t) {
#pragma unroll
  for (int i = 0; i < S; ++i)
#pragma unroll
    for (int j = 0; j < S; ++j)
#pragma unroll
      for (int k = 0; k < S; ++k)
        if (i != j && i != k && j != k)
          atomicOr(&t[(uint64_t(m[i]) * N + m[j]) * W + (m[k] >> 5)], 1u << (m[k] & 31));
}

__global__ void k_dense5_build(const uint32_t* __restrict__ e3, uint64_t n3, const uint32_t* __restrict__ e4,
                               uint64_t n4, const uint32_t* __restrict__ e5, uint64_t n5, uint32_t N, uint32_t W,
                               Dense5 d) {
  for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n3 + n4 + n5;
       i += uint64_t(gridDim.x) * blockDim.x) {
    if (i < n3) dense_mark<3>(e3 + 3 * i, N, W, d.t3);
    else if (i < n3 + n4) dense_mark<4>(e4 + 4 * (i - n3), N, W, d.f4);
    else dense_mark<5>(e5 + 5 * (i - n3 - n4), N, W, d.f5);
  }
}

// Pattern bits by position masks; positions: the sample's nodes first, then
// the chosen ones in ascending order, the last chosen node being 4.
constexpr uint32_t bit5(uint32_t mask) {
  uint32_t b = 0;
  for (uint32_t i = 0; i < uint32_t(kSub5); ++i)
    if (kSubMask5[i] == mask) b = i;
  return b;
}

__device__ inline bool row_bit(const uint32_t* __restrict__ row, uint32_t z) { return (row[z >> 5] >> (z & 31)) & 1u; }

__device__ inline bool has4_any(const View& v, uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  sort3(a, b, c);
  uint32_t t;
  if (d < c) { t = c; c = d; d = t; }
  if (c < b) { t = b; b = c; c = t; }
  if (b < a) { t = a; a = b; b = t; }
  return set128_has(v.hs4, key4(a, b, c, d));
}

__device__ inline bool has5_any(const Sampled5Args& a, uint32_t p, uint32_t q, uint32_t r, uint32_t s, uint32_t t) {
  uint32_t V[5] = {p, q, r, s, t};
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4 - i; ++j) {
      const uint32_t lo = min(V[j], V[j + 1]), hi = max(V[j], V[j + 1]);
      V[j] = lo;
      V[j + 1] = hi;
    }
  return has5(a.e5, a.hs5, a.hs5_mask, V);
}

// Counters of the sets around sampled pairs: 32 patterns of the pairs (ax,
// bx, ay, by, xy) times 16 of z's pairs (az, bz, xz, yz).
constexpr uint32_t kPairBins5 = 512;
constexpr uint32_t kPairCopies5 = 16;   // device copies (workgroup b adds to copy b mod 16)

struct LdsDense5 {
  Tables5 T;
  unsigned long long bins[kPairBins5];
  uint32_t lkeys[kLocalCap];
  unsigned long long lcount[kLocalCap];
  uint32_t seen[kDense5MaxWords], front[kDense5MaxWords], next[kDense5MaxWords];
  uint32_t list[kDense5MaxNodes];   // ball nodes of a pair; node profiles of a 3-node hyperedge
  uint32_t n_list;
};

// The nodes within three hops of {p, q} through pairs, p and q left out:
// bitmap in L.seen, ascending list in L.list.  Every thread calls this.
__device__ void pair_ball5(LdsDense5& L, const View& v, uint32_t p, uint32_t q) {
  const uint32_t W = v.W, N = v.N;
  __syncthreads();   // the previous task's lists are no longer read
  if (threadIdx.x < W) {
    const uint32_t w = threadIdx.x;
    uint32_t self = 0;
    if ((p >> 5) == w) self |= 1u << (p & 31);
    if ((q >> 5) == w) self |= 1u << (q & 31);
    const uint32_t nb = (v.bits[uint64_t(p) * W + w] | v.bits[uint64_t(q) * W + w]) & ~self;
    L.seen[w] = nb | self;
    L.front[w] = nb;
  }
  for (int hop = 1; hop < 3; ++hop) {
    if (threadIdx.x < W) L.next[threadIdx.x] = 0u;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < N * W; i += blockDim.x) {
      const uint32_t u = i / W, w = i - u * W;
      if ((L.front[u >> 5] >> (u & 31)) & 1u) {
        const uint32_t x = v.bits[i] & ~L.seen[w];
        if (x) atomicOr(&L.next[w], x);
      }
    }
    __syncthreads();
    if (threadIdx.x < W) {
      L.front[threadIdx.x] = L.next[threadIdx.x];
      L.seen[threadIdx.x] |= L.next[threadIdx.x];
    }
  }
  __syncthreads();
  if (threadIdx.x < uint32_t(kWave)) {   // W <= 32 words, one per lane
    const uint32_t w = threadIdx.x;
    uint32_t word = 0;
    if (w < W) {
      word = L.seen[w];
      if ((p >> 5) == w) word &= ~(1u << (p & 31));
      if ((q >> 5) == w) word &= ~(1u << (q & 31));
      L.seen[w] = word;
    }
    uint32_t total;
    uint32_t at = wave_exclusive_scan(__popc(word), &total);
    for (; word; word &= word - 1) L.list[at++] = (w << 5) | uint32_t(__ffs(word) - 1);
    if (w == 0) L.n_list = total;
  }
  __syncthreads();
}

// Share c of nc of the sets {a, b, x, y, z} (x < y < z in the ball) around
// the sampled pair {a, b}: connected through pairs and holding no larger
// hyperedge.  A thread takes a pair x < y; for each word of z the rows of the
// six node pairs without z leave the z that complete no 3-node hyperedge, and
// the rows of a, b, x and y split them by z's pairs into 15 patterns, counted
// by popcounts (z with none of the pairs belongs to no connected set).
__device__ void pair_sets5(LdsDense5& L, const Sampled5Args& s, const Dense5& d, uint32_t a, uint32_t b, uint32_t c,
                           uint32_t nc) {
  const View& v = s.v;
  const uint32_t N = v.N, W = v.W;
  pair_ball5(L, v, a, b);
  const uint32_t n = L.n_list;
  if (n < 3) return;
  auto row = [&](const uint32_t* t, uint32_t p, uint32_t q) { return t + (uint64_t(p) * N + q) * W; };
  const uint32_t *t_ab = row(d.t3, a, b), *f_ab = row(d.f4, a, b), *g_ab = row(d.f5, a, b);
  const uint32_t *r_a = v.bits + uint64_t(a) * W, *r_b = v.bits + uint64_t(b) * W;
  // rows i and n - 2 - i of the triangle of pairs (i < j) hold n pairs together
  const uint32_t folded = (n / 2) * n;   // ceil((n - 1) / 2) rows of n
  for (uint32_t t = c * kThreads5 + threadIdx.x; t < folded; t += nc * kThreads5) {
    const uint32_t r = t / n, q = t - r * n;
    uint32_t i = r, j = r + 1 + q;
    if (q >= n - 1 - r) {
      i = n - 2 - r;
      if (i == r) continue;
      j = i + 1 + (q - (n - 1 - r));
    }
    const uint32_t x = L.list[i], y = L.list[j];
    const uint32_t *t_ax = row(d.t3, a, x), *t_bx = row(d.t3, b, x);
    if (row_bit(t_ab, x) | row_bit(t_ab, y) | row_bit(t_ax, y) | row_bit(t_bx, y)) continue;
    const uint32_t *f_ax = row(d.f4, a, x), *f_bx = row(d.f4, b, x);
    const bool f_abx = row_bit(f_ab, x), f_aby = row_bit(f_ab, y), f_axy = row_bit(f_ax, y), f_bxy = row_bit(f_bx, y);
    if (f_abx && f_aby && f_axy && f_bxy && has4_any(v, a, b, x, y)) continue;
    const uint32_t *g_ax = row(d.f5, a, x), *g_bx = row(d.f5, b, x);
    const bool g5 = row_bit(g_ab, x) & row_bit(g_ab, y) & row_bit(g_ax, y) & row_bit(g_bx, y);
    const bool larger = f_abx | f_aby | f_axy | f_bxy | g5;
    const uint32_t *t_ay = row(d.t3, a, y), *t_by = row(d.t3, b, y), *t_xy = row(d.t3, x, y);
    const uint32_t *r_x = v.bits + uint64_t(x) * W, *r_y = v.bits + uint64_t(y) * W;
    const uint32_t fixed = uint32_t(row_bit(r_a, x)) | (uint32_t(row_bit(r_b, x)) << 1) |
                           (uint32_t(row_bit(r_a, y)) << 2) | (uint32_t(row_bit(r_b, y)) << 3) |
                           (uint32_t(row_bit(r_x, y)) << 4);
    uint32_t cnt[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) cnt[k] = 0;
    for (uint32_t w = y >> 5; w < W; ++w) {
      uint32_t m = mask_gt(y, w) & L.seen[w] & ~(t_ab[w] | t_ax[w] | t_bx[w] | t_ay[w] | t_by[w] | t_xy[w]);
      if (larger && m) {
        const uint32_t *f_ay = row(d.f4, a, y), *f_by = row(d.f4, b, y), *f_xy = row(d.f4, x, y);
        const uint32_t abx = f_abx ? f_ab[w] & f_ax[w] & f_bx[w] : 0u, aby = f_aby ? f_ab[w] & f_ay[w] & f_by[w] : 0u;
        const uint32_t axy = f_axy ? f_ax[w] & f_ay[w] & f_xy[w] : 0u, bxy = f_bxy ? f_bx[w] & f_by[w] & f_xy[w] : 0u;
        const uint32_t all = g5 ? g_ab[w] & g_ax[w] & g_bx[w] & row(d.f5, a, y)[w] & row(d.f5, b, y)[w] &
                                      row(d.f5, x, y)[w]
                                : 0u;
        for (uint32_t rest = m & (abx | aby | axy | bxy | all); rest; rest &= rest - 1) {
          const uint32_t bit = rest & (0u - rest), z = (w << 5) | uint32_t(__ffs(rest) - 1);
          if (((abx & bit) && has4_any(v, a, b, x, z)) || ((aby & bit) && has4_any(v, a, b, y, z)) ||
              ((axy & bit) && has4_any(v, a, x, y, z)) || ((bxy & bit) && has4_any(v, b, x, y, z)) ||
              ((all & bit) && has5_any(s, a, b, x, y, z)))
            m &= ~bit;
        }
      }
      const uint32_t A = r_a[w], B = r_b[w], X = r_x[w], Y = r_y[w];
      const uint32_t ab[4] = {m & ~A & ~B, m & A & ~B, m & ~A & B, m & A & B};
      const uint32_t xy[4] = {~X & ~Y, X & ~Y, ~X & Y, X & Y};
#pragma unroll
      for (int k = 1; k < 16; ++k) cnt[k] += __popc(ab[k & 3] & xy[k >> 2]);
    }
#pragma unroll
    for (uint32_t k = 1; k < 16; ++k)
      if (cnt[k]) atomicAdd(&L.bins[fixed * 16 + k], (unsigned long long)cnt[k]);
  }
}

// The pattern of counter k of the sets around pairs (a, b, x, y, z at
// positions 0..4).
__device__ inline uint32_t pair_bin_pattern5(uint32_t k) {
  const uint32_t f = k >> 4, z = k & 15u;
  return (1u << bit5(3)) | ((f & 1u) << bit5(5)) | (((f >> 1) & 1u) << bit5(6)) | (((f >> 2) & 1u) << bit5(9)) |
         (((f >> 3) & 1u) << bit5(10)) | ((f >> 4) << bit5(12)) | ((z & 1u) << bit5(17)) |
         (((z >> 1) & 1u) << bit5(18)) | (((z >> 2) & 1u) << bit5(20)) | ((z >> 3) << bit5(24));
}

// The sets {a, b, c, y, z} (y < z) around the sampled 3-node hyperedge
// {a, b, c}: connected, no larger hyperedge.  Per node, its three pairs and
// three 3-node hyperedges with the sample are kept in LDS; a thread takes a
// (y, word of z) and walks the z that its rows leave connected.  This is share
// `share` of `shares` of the sample's (y, word) items.
__device__ void triple_sets5(LdsDense5& L, const Sampled5Args& s, const Dense5& d, uint32_t a, uint32_t b, uint32_t c,
                             uint32_t share, uint32_t shares) {
  const View& v = s.v;
  const uint32_t N = v.N, W = v.W;
  auto row = [&](const uint32_t* t, uint32_t p, uint32_t q) { return t + (uint64_t(p) * N + q) * W; };
  const uint32_t *t_ab = row(d.t3, a, b), *t_ac = row(d.t3, a, c), *t_bc = row(d.t3, b, c);
  const uint32_t *f_ab = row(d.f4, a, b), *f_ac = row(d.f4, a, c), *f_bc = row(d.f4, b, c);
  const uint32_t *g_ab = row(d.f5, a, b), *g_ac = row(d.f5, a, c), *g_bc = row(d.f5, b, c);
  const uint32_t *r_a = v.bits + uint64_t(a) * W, *r_b = v.bits + uint64_t(b) * W, *r_c = v.bits + uint64_t(c) * W;
  __syncthreads();   // the previous task's lists are no longer read
  // L.list: the node's pattern bits with the sample (as y); L.seen: the nodes
  // that may be chosen; L.front: those of them that touch the sample
  for (uint32_t y0 = 0; y0 < W * 32; y0 += kThreads5) {
    const uint32_t y = y0 + threadIdx.x;
    bool allowed = y < N && y != a && y != b && y != c;
    uint32_t p = 0;
    if (allowed) {
      if (row_bit(f_ab, y) & row_bit(f_ac, y) & row_bit(f_bc, y)) allowed = !has4_any(v, a, b, c, y);
      p = (uint32_t(row_bit(r_a, y)) << bit5(9)) | (uint32_t(row_bit(r_b, y)) << bit5(10)) |
          (uint32_t(row_bit(r_c, y)) << bit5(12)) | (uint32_t(row_bit(t_ab, y)) << bit5(11)) |
          (uint32_t(row_bit(t_ac, y)) << bit5(13)) | (uint32_t(row_bit(t_bc, y)) << bit5(14));
    }
    const unsigned long long on = __ballot(allowed), touch = __ballot(allowed && p);
    if (y < N) L.list[y] = p;
    const uint32_t lane = threadIdx.x & (kWave - 1), w = y >> 5;
    if ((lane & 31) == 0 && w < W) {
      L.seen[w] = uint32_t(on >> (lane & 32));
      L.front[w] = uint32_t(touch >> (lane & 32));
    }
  }
  __syncthreads();
  const uint32_t base = (1u << bit5(7)) | (uint32_t(row_bit(r_a, b)) << bit5(3)) |
                        (uint32_t(row_bit(r_a, c)) << bit5(5)) | (uint32_t(row_bit(r_b, c)) << bit5(6));
  for (uint32_t t = share * kThreads5 + threadIdx.x; t < N * W; t += shares * kThreads5) {
    const uint32_t y = t / W, w = t - y * W;
    if (w < (y >> 5) || !((L.seen[y >> 5] >> (y & 31)) & 1u)) continue;
    const uint32_t py = L.list[y];
    const uint32_t yz = v.bits[t], ta = row(d.t3, a, y)[w], tb = row(d.t3, b, y)[w], tc = row(d.t3, c, y)[w];
    const uint32_t touch = L.front[w];
    uint32_t cand = mask_gt(y, w) & L.seen[w] & (ta | tb | tc | (py ? (yz | touch) : (yz & touch)));
    if (!cand) continue;
    uint32_t aby = 0, acy = 0, bcy = 0, all = 0;
    const bool fab = row_bit(f_ab, y), fac = row_bit(f_ac, y), fbc = row_bit(f_bc, y);
    if (fab | fac | fbc) {
      const uint32_t fa = row(d.f4, a, y)[w], fb = row(d.f4, b, y)[w], fc = row(d.f4, c, y)[w];
      if (fab) aby = f_ab[w] & fa & fb;
      if (fac) acy = f_ac[w] & fa & fc;
      if (fbc) bcy = f_bc[w] & fb & fc;
    }
    if (row_bit(g_ab, y) & row_bit(g_ac, y) & row_bit(g_bc, y))
      all = g_ab[w] & g_ac[w] & g_bc[w] & row(d.f5, a, y)[w] & row(d.f5, b, y)[w] & row(d.f5, c, y)[w];
    for (uint32_t rest = cand & (aby | acy | bcy | all); rest; rest &= rest - 1) {
      const uint32_t bit = rest & (0u - rest), z = (w << 5) | uint32_t(__ffs(rest) - 1);
      if (((aby & bit) && has4_any(v, a, b, y, z)) || ((acy & bit) && has4_any(v, a, c, y, z)) ||
          ((bcy & bit) && has4_any(v, b, c, y, z)) || ((all & bit) && has5_any(s, a, b, c, y, z)))
        cand &= ~bit;
    }
    for (; cand; cand &= cand - 1) {
      const uint32_t zb = uint32_t(__ffs(cand) - 1), z = (w << 5) | zb, pz = L.list[z];
      // z's bits with the sample, moved from position 3 to position 4
      const uint32_t zp = (((pz >> bit5(9)) & 1u) << bit5(17)) | (((pz >> bit5(10)) & 1u) << bit5(18)) |
                          (((pz >> bit5(12)) & 1u) << bit5(20)) | (((pz >> bit5(11)) & 1u) << bit5(19)) |
                          (((pz >> bit5(13)) & 1u) << bit5(21)) | (((pz >> bit5(14)) & 1u) << bit5(22));
      add_local(L, s,
                base | py | zp | (((yz >> zb) & 1u) << bit5(24)) | (((ta >> zb) & 1u) << bit5(25)) |
                    (((tb >> zb) & 1u) << bit5(26)) | (((tc >> zb) & 1u) << bit5(28)));
    }
  }
}

// The sets {a, b, c, d, z} around the sampled 4-node hyperedge m: no 5-node
// hyperedge, z touching the sample; a thread takes a z.
__device__ void quad_sets5(LdsDense5& L, const Sampled5Args& s, const Dense5& d, const uint32_t* m) {
  const View& v = s.v;
  const uint32_t N = v.N, W = v.W;
  const uint32_t e[4] = {m[0], m[1], m[2], m[3]};
  for (uint32_t z = threadIdx.x; z < N; z += kThreads5) {
    if (z == e[0] || z == e[1] || z == e[2] || z == e[3]) continue;
    uint32_t base = 1u << bit5(15), p = 0, f4 = 0, f5 = 0;   // f4, f5: position masks of pairs held with z
    int q = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) p |= uint32_t(row_bit(v.bits + uint64_t(e[i]) * W, z)) << bit5((1u << i) | 16u);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = i + 1; j < 4; ++j) {
        const uint64_t at = (uint64_t(e[i]) * N + e[j]) * W;
        base |= uint32_t(row_bit(v.bits + uint64_t(e[i]) * W, e[j])) << bit5((1u << i) | (1u << j));
        p |= uint32_t(row_bit(d.t3 + at, z)) << bit5((1u << i) | (1u << j) | 16u);
#pragma unroll
        for (int k = j + 1; k < 4; ++k)
          base |= uint32_t(row_bit(d.t3 + at, e[k])) << bit5((1u << i) | (1u << j) | (1u << k));
        f4 |= uint32_t(row_bit(d.f4 + at, z)) << q;
        f5 |= uint32_t(row_bit(d.f5 + at, z)) << q;
        ++q;
      }
    // pair bits of f4: 01 = 0, 02 = 1, 03 = 2, 12 = 3, 13 = 4, 23 = 5
    if ((f4 & 0x0Bu) == 0x0Bu) p |= uint32_t(has4_any(v, e[0], e[1], e[2], z)) << bit5(23);
    if ((f4 & 0x15u) == 0x15u) p |= uint32_t(has4_any(v, e[0], e[1], e[3], z)) << bit5(27);
    if ((f4 & 0x26u) == 0x26u) p |= uint32_t(has4_any(v, e[0], e[2], e[3], z)) << bit5(29);
    if ((f4 & 0x38u) == 0x38u) p |= uint32_t(has4_any(v, e[1], e[2], e[3], z)) << bit5(30);
    if (!p) continue;
    if (f5 == 0x3Fu && has5_any(s, e[0], e[1], e[2], e[3], z)) continue;
    add_local(L, s, base | p);
  }
}

// Every sample of the call.  Tasks: the 3-node samples in nc3 shares each,
// the pair samples in nc2, then one per 4-node sample, then the 5-node
// samples 256 at a time.  A pair sample is N^2/2 node pairs of W words at about 75
// operations a word.  On the communication recipe at N = 200 (1.3e6 candidate
// sets a pair sample, 5% of every stratum drawn) this launch takes 0.21 ms where
// the general path's k_sampled5, which fills in and classifies every set, took
// 53.3 ms; the 3-node samples' shares come first, since one workgroup a sample
// left a tail (0.40 ms).  What bounds it is latency with few wavefronts in
// flight, six a CU: 60% of their cycles wait, 29% of the VALU issue rate is
// used.
__global__ void __launch_bounds__(kThreads5) k_dense5(Sampled5Args a, Dense5 d, Tables5 tables, uint32_t nc2,
                                                      uint32_t nc3,
                                                      unsigned long long* __restrict__ pair_bins) {
  __shared__ LdsDense5 L;
  clear_local(L);
  for (uint32_t i = threadIdx.x; i < kPairBins5; i += kThreads5) L.bins[i] = 0ull;
  if (threadIdx.x == 0) L.T = tables;
  __syncthreads();
  const uint64_t n3 = a.S[3] * nc3, n23 = n3 + a.S[2] * nc2, n234 = n23 + a.S[4];
  const uint64_t tasks = n234 + (a.S[5] + kThreads5 - 1) / kThreads5;
  for (uint64_t t = blockIdx.x; t < tasks; t += gridDim.x) {
    int j;
    uint64_t i;
    if (t < n3) {
      sample_of(a, a.S[2] + t / nc3, &j, &i);
      triple_sets5(L, a, d, a.v.e3[3 * i], a.v.e3[3 * i + 1], a.v.e3[3 * i + 2], uint32_t(t % nc3), nc3);
    } else if (t < n23) {
      sample_of(a, (t - n3) / nc2, &j, &i);
      pair_sets5(L, a, d, a.v.e2[2 * i], a.v.e2[2 * i + 1], uint32_t((t - n3) % nc2), nc2);
    } else if (t < n234) {
      sample_of(a, a.S[2] + a.S[3] + (t - n23), &j, &i);
      quad_sets5(L, a, d, a.v.e4 + 4 * i);
    } else {
      const uint64_t r = (t - n234) * kThreads5 + threadIdx.x;
      if (r < a.S[5]) {
        sample_of(a, a.S[2] + a.S[3] + a.S[4] + r, &j, &i);
        uint32_t V[5];
        for (int m = 0; m < 5; ++m) V[m] = a.e5[5 * i + m];
        add_local(L, a, fill5(a, L.T, V));
      }
    }
  }
  __syncthreads();
  unsigned long long* out = pair_bins + (blockIdx.x % kPairCopies5) * kPairBins5;
  for (uint32_t i = threadIdx.x; i < kPairBins5; i += kThreads5)
    if (L.bins[i]) atomicAdd(&out[i], L.bins[i]);
  flush_local(L, a);
}

// ------------------------------------------------------------------ classes
// Clear the tables of one call: n_words words of the pattern and class
// tables' keys and counts, laid out as one block.
__global__ void k_clear5(uint4* __restrict__ p, uint64_t n) {
  for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += uint64_t(gridDim.x) * blockDim.x)
    p[i] = make_uint4(0u, 0u, 0u, 0u);
}

// Each distinct pattern (the pair counters first, when there are any, then
// the pattern table) in canonical form, added to the class table.  A
// wavefront takes 64 entries and each occupied one in turn, its lanes the
// relabellings, whose images of the 26 subsets are in LDS.
__global__ void __launch_bounds__(256) k_canon5(Sampled5Args a, Tables5 T, const unsigned long long* __restrict__ pair_bins) {
  __shared__ uint8_t img[kSub5][128];
  for (uint32_t x = threadIdx.x; x < kSub5 * 120; x += 256) {
    const uint32_t b = x / 120, g = x % 120, m = T.sub_mask[b];
    uint32_t to = 0;
    for (int i = 0; i < 5; ++i)
      if ((m >> i) & 1u) to |= 1u << T.perm[g][i];
    img[b][g] = uint8_t(T.bit_of_mask[to]);
  }
  __syncthreads();
  const uint32_t lane = threadIdx.x & (kWave - 1);
  const uint32_t n_bins = pair_bins ? kPairBins5 : 0u, n = n_bins + kRawSlots;
  for (uint32_t base = (blockIdx.x * 256 + threadIdx.x) & ~uint32_t(kWave - 1); base < n; base += gridDim.x * 256) {
    const uint32_t i = base + lane;
    uint32_t p = 0;
    unsigned long long cnt = 0;
    if (i < n_bins) {
      for (uint32_t q = 0; q < kPairCopies5; ++q) cnt += pair_bins[q * kPairBins5 + i];
      p = pair_bin_pattern5(i);
      if (cnt && !connected5(T, p)) cnt = 0;
    } else if (i < n) {
      const uint32_t key = a.raw_keys[i - n_bins];
      p = key - 1u;
      if (key) cnt = a.raw_counts[i - n_bins];
    }
    for (unsigned long long m = __ballot(cnt != 0); m; m &= m - 1) {
      const int l = __ffsll(m) - 1;
      const uint32_t pat = uint32_t(__builtin_amdgcn_readlane(int(p), l));
      uint32_t q0 = 0, q1 = 0;
      for (uint32_t r = pat; r; r &= r - 1) {
        const uint8_t* to = img[__ffs(r) - 1];
        q0 |= 1u << to[lane];
        q1 |= 1u << (lane < 56 ? to[64 + lane] : to[lane]);
      }
      uint32_t best = min(q0, q1);
      for (int o = kWave / 2; o > 0; o >>= 1) best = min(best, uint32_t(__shfl_xor(int(best), o, kWave)));
      if (lane == uint32_t(l)) add_global(a, best, cnt);
    }
  }
}

// Compact the device class table in two launches: the classes of each
// workgroup's share (kCompact5 slots), then each share written after those
// before it (every workgroup sums their counts) and the total by the last.
constexpr uint32_t kCompact5 = 8192;
__device__ inline uint32_t block_sum256(uint32_t x, uint32_t* wsum) {
  x = wave_sum_u32(x);
  if ((threadIdx.x & (kWave - 1)) == 0) wsum[threadIdx.x / kWave] = x;
  __syncthreads();
  const uint32_t s = wsum[0] + wsum[1] + wsum[2] + wsum[3];
  __syncthreads();
  return s;
}

__global__ void __launch_bounds__(256) k_class_count(const uint32_t* __restrict__ keys, uint64_t n,
                                                     uint32_t* __restrict__ counts) {
  __shared__ uint32_t wsum[4];
  const uint64_t base = uint64_t(blockIdx.x) * kCompact5;
  uint32_t c = 0;
#pragma unroll
  for (uint32_t r = 0; r < kCompact5 / 256; ++r) {
    const uint64_t i = base + r * 256 + threadIdx.x;
    c += i < n && keys[i] != 0u;
  }
  c = block_sum256(c, wsum);
  if (threadIdx.x == 0) counts[blockIdx.x] = c;
}

__global__ void __launch_bounds__(256) k_class_compact(const uint32_t* __restrict__ keys,
                                                       const unsigned long long* __restrict__ counts, uint64_t n,
                                                       const uint32_t* __restrict__ share, uint64_t capacity,
                                                       unsigned long long* __restrict__ canon_out,
                                                       uint32_t* __restrict__ order_out,
                                                       unsigned long long* __restrict__ cnt_out,
                                                       uint32_t* __restrict__ total) {
  __shared__ uint32_t wsum[4];
  uint32_t before = 0;
  for (uint32_t i = threadIdx.x; i < blockIdx.x; i += 256) before += share[i];
  before = block_sum256(before, wsum);
  const uint32_t mine = share[blockIdx.x];
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) total[0] = before + mine;
  if (!mine) return;
  const uint64_t base = uint64_t(blockIdx.x) * kCompact5;
  for (uint32_t r = 0; r < kCompact5 / 256; ++r) {
    const uint64_t i = base + r * 256 + threadIdx.x;
    const uint32_t key = i < n ? keys[i] : 0u;
    const unsigned long long m = __ballot(key != 0u);
    const uint32_t wv = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
    if (lane == 0) wsum[wv] = uint32_t(__popcll(m));
    __syncthreads();
    uint32_t at = before + uint32_t(__popcll(m & ((1ull << lane) - 1ull)));
    for (uint32_t q = 0; q < wv; ++q) at += wsum[q];
    before += wsum[0] + wsum[1] + wsum[2] + wsum[3];
    if (key && at < capacity) {   // (more classes than the outputs hold: an error, only their number is used)
      canon_out[at] = key - 1u;
      order_out[at] = at;
      cnt_out[at] = counts[i];
    }
    __syncthreads();
  }
}

struct Scale5 {
  double n[6];
  double s[6];
};

// Class c with raw count r at place i of the outputs: canonical, raw count,
// estimate (Algorithm 4's correction, fp64 rounded once to fp32).
__device__ inline void write_class5(uint64_t i, uint32_t c, unsigned long long r, const Scale5& sc,
                                    uint32_t* __restrict__ canon_out, int64_t* __restrict__ raw_out,
                                    float* __restrict__ est_out) {
  int mc = 0, cm = 0;
#pragma unroll
  for (int b = 0; b < kSub5; ++b)
    if ((c >> b) & 1u) {
      const int sz = __builtin_popcount(kSubMask5[b]);
      if (sz > mc) {
        mc = sz;
        cm = 1;
      } else if (sz == mc) {
        ++cm;
      }
    }
  canon_out[i] = c;
  raw_out[i] = int64_t(r);
  est_out[i] = sc.s[mc] > 0.0 ? float(double(r) * sc.n[mc] / (sc.s[mc] * double(cm))) : 0.f;
}

// classes in canonical order from the sorted keys
__global__ void k_finish5(const unsigned long long* __restrict__ sorted_canon, const uint32_t* __restrict__ order,
                          const unsigned long long* __restrict__ cnt, uint64_t n, Scale5 sc,
                          uint32_t* __restrict__ canon_out, int64_t* __restrict__ raw_out, float* __restrict__ est_out) {
  for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += uint64_t(gridDim.x) * blockDim.x)
    write_class5(i, uint32_t(sorted_canon[i]), cnt[order[i]], sc, canon_out, raw_out, est_out);
}

// The same for at most kRankMax classes in any order: a class's place is the
// number of smaller canonical values.  Sixteen threads share a class's
// comparisons (canonical values are distinct): one launch of 45 us at 2,780
// classes, where four radix passes took twelve launches and 0.2 ms.
constexpr uint64_t kRankMax = 16384;
constexpr uint32_t kRankLanes = 16;
__global__ void __launch_bounds__(256) k_rank5(const unsigned long long* __restrict__ canon,
                                               const unsigned long long* __restrict__ cnt, uint32_t n, Scale5 sc,
                                               uint32_t* __restrict__ canon_out, int64_t* __restrict__ raw_out,
                                               float* __restrict__ est_out) {
  const uint32_t i = (blockIdx.x * 256 + threadIdx.x) / kRankLanes, part = threadIdx.x % kRankLanes;
  const uint32_t c = i < n ? uint32_t(canon[i]) : 0u;
  uint32_t below = 0;
  // (eight loads in flight: the loop is a chain of them otherwise)
  for (uint32_t k0 = part; k0 < n; k0 += 8 * kRankLanes) {
#pragma unroll
    for (uint32_t r = 0; r < 8; ++r) {
      const uint32_t k = k0 + r * kRankLanes;
      below += k < n && uint32_t(canon[k]) < c;
    }
  }
#pragma unroll
  for (uint32_t d = 1; d < kRankLanes; d <<= 1) below += uint32_t(__shfl_xor(int(below), int(d), kWave));
  if (i < n && part == 0) write_class5(below, c, cnt[i], sc, canon_out, raw_out, est_out);
}

unsigned grid5(uint64_t n) {
  uint64_t g = (n + 255) / 256;
  return unsigned(std::max<uint64_t>(1, std::min<uint64_t>(g, 4096)));
}

}  // namespace

// E_5 and its hash set, on first use.
int ensure_order5(hm_graph* H, hipStream_t st) {
  if (H->order5_built) return HM_OK;
  HM_TRY(refuse_capture(st));
  note_use(H, st);
  const uint64_t n = H->n_unique;
  std::vector<void*> tmp;
  struct Free {
    std::vector<void*>& t;
    hipStream_t st;
    ~Free() { dfree_on(t.data(), t.size(), st); }
  } release{tmp, st};
  auto get = [&](void** p, size_t bytes) {
    int rc = dalloc(p, bytes ? bytes : 4);
    if (rc == HM_OK) tmp.push_back(*p);
    return rc;
  };
  void *flag = nullptr, *pos = nullptr, *tot = nullptr;
  HM_TRY(get(&flag, (n + 1) * 4));
  HM_TRY(get(&pos, (n + 1) * 4));
  HM_TRY(get(&tot, 8));
  uint32_t n5 = 0;
  if (n) {
    k_e5_flags<<<grid5(n), 256, 0, st>>>(H->all_off, n, static_cast<uint32_t*>(flag));
    HM_HIP(hipGetLastError());
    HM_TRY(scan_exclusive_u32(static_cast<uint32_t*>(flag), static_cast<uint32_t*>(pos), n,
                              static_cast<uint32_t*>(tot), st));
    HM_HIP(hipMemcpyAsync(&n5, tot, 4, hipMemcpyDeviceToHost, st));
    HM_HIP(hipStreamSynchronize(st));
  }
  void *e5 = nullptr, *slots = nullptr;
  const unsigned long long cap = pow2_capacity(n5);
  HM_TRY(dalloc(&e5, size_t(n5 ? n5 : 1) * 5 * 4));
  int rc = dalloc(&slots, size_t(cap) * 4);
  if (rc != HM_OK) {
    dfree(e5);
    return rc;
  }
  rc = fill_u32(static_cast<uint32_t*>(slots), 0u, cap, st);
  if (rc == HM_OK && n5) {
    k_e5_gather<<<grid5(n), 256, 0, st>>>(H->all_off, H->all_members, n, static_cast<uint32_t*>(flag),
                                          static_cast<uint32_t*>(pos), static_cast<uint32_t*>(e5));
    k_e5_insert<<<grid5(n5), 256, 0, st>>>(static_cast<uint32_t*>(e5), n5, static_cast<uint32_t*>(slots), cap - 1);
    if (hipGetLastError() != hipSuccess) rc = HM_EDEVICE;
  }
  if (rc == HM_OK && hipStreamSynchronize(st) != hipSuccess) rc = HM_EDEVICE;
  if (rc != HM_OK) {
    dfree(e5);
    dfree(slots);
    return rc;
  }
  H->e5 = static_cast<uint32_t*>(e5);
  H->hs5 = static_cast<uint32_t*>(slots);
  H->hs5_mask = cap - 1;
  H->n5 = n5;
  H->order5_built = true;
  return HM_OK;
}

// Whether a call's samples S[2..5] are worth the dense path's bit tensors on a
// graph that has none yet.  Clearing them costs what the general path needs for
// about a candidate set per 96 words (some 10^10 sets a second, 0.08 ms for the
// 10^8 words of 1,024 nodes).  The sets are bounded by the choices among the
// nodes that any pair (or 3- or 4-node hyperedge) could bring within reach: far
// too many mostly, so that the general path is left to samples of hypergraphs
// with a few hyperedges among many nodes.  First calls there, 1,024 nodes, one
// sample: 50 pairs 143 us by the general path, 220 with the tensors; 50 4-node
// hyperedges 148 and 195; but 400 pairs and 50 3-node hyperedges, 23 samples,
// 661 and 558; 2,000 and 100, 2 samples, 3,160 and 340.
bool dense5_pays(const hm_graph* H, const uint64_t S[6]) {
  const double N = H->n_nodes, words = 3.0 * N * N * H->words;
  const double r2 = std::min(N, 2.0 * H->n_by_size[2]), r3 = std::min(N, r2 + 3.0 * H->n_by_size[3]),
               r4 = std::min(N, r3 + 4.0 * H->n_by_size[4]);
  const double sets = double(S[2]) * r2 * r2 * r2 / 6 + double(S[3]) * r3 * r3 / 2 + double(S[4]) * r4;
  return 96 * sets >= words;
}

// The dense path's bit tensors, on first use; H->dense5 stays null when the
// hypergraph does not take that path or the memory is not there.
int ensure_dense5(hm_graph* H, const uint64_t S[6], hipStream_t st) {
  if (H->dense5 || !H->bits || H->n_nodes > kDense5MaxNodes || !dense5_pays(H, S)) return HM_OK;
  HM_TRY(refuse_capture(st));
  const uint64_t words = uint64_t(H->n_nodes) * H->n_nodes * H->words;
  void* p = nullptr;
  if (dalloc(&p, 3 * words * sizeof(uint32_t)) != HM_OK) return HM_OK;
  uint32_t* t = static_cast<uint32_t*>(p);
  int rc = fill_u32(t, 0u, 3 * words, st);
  const uint64_t n3 = H->n_by_size[3], n4 = H->n_by_size[4], n5 = H->n5;
  if (rc == HM_OK && n3 + n4 + n5) {
    k_dense5_build<<<grid5(n3 + n4 + n5), 256, 0, st>>>(H->e3, n3, H->e4, n4, H->e5, n5, H->n_nodes, H->words,
                                                        Dense5{t, t + words, t + 2 * words});
    if (hipGetLastError() != hipSuccess) {
      set_error("order 5: kernel launch failed");
      rc = HM_EDEVICE;
    }
  }
  if (rc != HM_OK) {
    dfree_on(p, st);
    return rc;
  }
  H->dense5 = t;
  return HM_OK;
}

// Algorithm 4 at order 5 for the draws S[j] (idx[j] explicit, or drawn from
// seed); synchronous.
int sampled5(hm_graph* H, const uint32_t* const idx[6], const uint64_t S[6], uint64_t seed, uint64_t capacity,
             uint32_t* canon, int64_t* raw, float* est, uint64_t* n_classes, hipStream_t st) {
  HM_TRY(ensure_order5(H, st));
  note_use(H, st);
  Sampled5Args a{};
  a.v = view_of(H);
  a.e5 = H->e5;
  a.hs5 = H->n5 ? H->hs5 : nullptr;
  a.hs5_mask = H->hs5_mask;
  const uint64_t nj[6] = {0, 0, H->n_by_size[2], H->n_by_size[3], H->n_by_size[4], H->n5};
  uint64_t total = 0;
  for (int j = 0; j < 6; ++j) {
    a.idx[j] = j >= 2 ? idx[j] : nullptr;
    a.n[j] = nj[j];
    a.S[j] = (j >= 2 && nj[j]) ? S[j] : 0;
    total += a.S[j];
  }
  a.seed = seed;
  if (total) HM_TRY(ensure_dense5(H, a.S, st));
  // the device class table: at most one class per candidate set, bounded by
  // the 2^26 patterns; sized for the output capacity at load 1/2
  const unsigned long long tcap = pow2_capacity(std::min<uint64_t>(std::max<uint64_t>(capacity, 1024), 1ull << 26));
  std::vector<void*> tmp;
  struct Free {
    std::vector<void*>& t;
    hipStream_t st;
    ~Free() { dfree_on(t.data(), t.size(), st); }
  } release{tmp, st};
  auto get = [&](void** p, size_t bytes) {
    int rc = dalloc(p, bytes ? bytes : 8);
    if (rc == HM_OK) tmp.push_back(*p);
    return rc;
  };
  // the pattern table, the class table, the pair counters and the error word
  // in one block, cleared by one launch
  constexpr uint64_t kBinWords = uint64_t(kPairCopies5) * kPairBins5;
  const uint64_t words64 = kRawSlots + tcap + kBinWords;
  const uint64_t words32 = kRawSlots + tcap + 4;
  void* tables = nullptr;
  HM_TRY(get(&tables, words64 * 8 + words32 * 4));
  a.raw_counts = static_cast<unsigned long long*>(tables);
  a.counts = a.raw_counts + kRawSlots;
  unsigned long long* pair_bins = a.counts + tcap;
  a.raw_keys = reinterpret_cast<uint32_t*>(pair_bins + kBinWords);
  a.keys = a.raw_keys + kRawSlots;
  a.err = a.keys + tcap;
  a.mask = tcap - 1;
  const uint64_t quads = (words64 * 8 + words32 * 4) / 16;   // every part is a multiple of 16 bytes
  k_clear5<<<grid5(quads), 256, 0, st>>>(static_cast<uint4*>(tables), quads);
  HM_HIP(hipGetLastError());
  const Tables5 T = make_tables5();
  const bool dense = H->dense5 != nullptr;
  if (total && dense) {
    const uint64_t words = uint64_t(H->n_nodes) * H->n_nodes * H->words;
    const Dense5 d{H->dense5, H->dense5 + words, H->dense5 + 2 * words};
    // shares of a sample: enough tasks to fill the chip, each of at least
    // about 2,048 node pairs (eight rounds of a workgroup, against the two
    // hops that every share of a pair sample walks again), or 256 (y, word of
    // z) items of a 3-node sample
    auto shares_of = [](uint64_t most, uint64_t samples) {
      return uint32_t(std::max<uint64_t>(1, std::min<uint64_t>(most, 4096 / std::max<uint64_t>(samples, 1))));
    };
    const uint32_t nc2 = shares_of((uint64_t(H->n_nodes) * H->n_nodes / 2 + 2047) / 2048, a.S[2]);
    const uint32_t nc3 = shares_of((uint64_t(H->n_nodes) * H->words + 255) / 256, a.S[3]);
    const uint64_t tasks = a.S[2] * nc2 + a.S[3] * nc3 + a.S[4] + (a.S[5] + kThreads5 - 1) / kThreads5;
    ProfileScope ps("k_dense5", st);
    k_dense5<<<unsigned(std::min<uint64_t>(tasks, 2048)), kThreads5, 0, st>>>(a, d, T, nc2, nc3, pair_bins);
    HM_HIP(hipGetLastError());
  } else if (total) {
    // pass 1: candidate chunks per sample; pass 2: the (sample, chunk) tasks
    void *chunks = nullptr, *first = nullptr;
    HM_TRY(get(&chunks, total * 4));
    HM_TRY(get(&first, (total + 1) * 4));
    k_chunks5<<<unsigned(std::min<uint64_t>(total, 4096)), kThreads5, 0, st>>>(a, total,
                                                                               static_cast<uint32_t*>(chunks));
    HM_HIP(hipGetLastError());
    HM_TRY(scan_exclusive_u32(static_cast<uint32_t*>(chunks), static_cast<uint32_t*>(first), total,
                              static_cast<uint32_t*>(first) + total, st));
    ProfileScope ps("k_sampled5", st);
    k_sampled5<<<4096, kThreads5, 0, st>>>(a, T, total, static_cast<const uint32_t*>(first));
    HM_HIP(hipGetLastError());
  }
  // the distinct patterns to classes, and the classes compacted
  const unsigned shares = unsigned((tcap + kCompact5 - 1) / kCompact5);
  const uint64_t most = std::min<uint64_t>(capacity, tcap);
  void *sk = nullptr, *sv = nullptr, *cnt = nullptr, *share = nullptr;
  HM_TRY(get(&sk, size_t(most) * 8));
  HM_TRY(get(&sv, size_t(most) * 4));
  HM_TRY(get(&cnt, size_t(most) * 8));
  HM_TRY(get(&share, size_t(shares + 1) * 4));
  uint32_t* nc_dev = static_cast<uint32_t*>(share) + shares;
  if (total) {
    k_canon5<<<(kRawSlots + kPairBins5 + 255) / 256, 256, 0, st>>>(a, T, dense ? pair_bins : nullptr);
    HM_HIP(hipGetLastError());
  }
  k_class_count<<<shares, 256, 0, st>>>(a.keys, tcap, static_cast<uint32_t*>(share));
  k_class_compact<<<shares, 256, 0, st>>>(a.keys, a.counts, tcap, static_cast<const uint32_t*>(share), most,
                                          static_cast<unsigned long long*>(sk), static_cast<uint32_t*>(sv),
                                          static_cast<unsigned long long*>(cnt), nc_dev);
  HM_HIP(hipGetLastError());
  uint32_t host_err = 0, nc = 0;
  HM_HIP(hipMemcpyAsync(&host_err, a.err, 4, hipMemcpyDeviceToHost, st));
  HM_HIP(hipMemcpyAsync(&nc, nc_dev, 4, hipMemcpyDeviceToHost, st));
  HM_HIP(hipStreamSynchronize(st));
  if (host_err & kErrBall) {
    set_error("order 5: a sampled hyperedge has more than %u nodes within reach", kBallCap);
    return HM_EUNSUPPORTED;
  }
  if (host_err & kErrWork) {
    set_error("order 5: a sampled hyperedge has 2^32 or more candidate node sets");
    return HM_EUNSUPPORTED;
  }
  if (host_err & kErrTable) {
    set_error("order 5: more classes than the class table holds (raise the capacity)");
    return HM_EINVAL;
  }
  *n_classes = nc;
  if (nc > capacity) {
    set_error("order 5: %u classes found, the output holds %llu", nc, (unsigned long long)capacity);
    return HM_EINVAL;
  }
  if (!nc) return HM_OK;
  Scale5 sc{};
  for (int j = 2; j <= 5; ++j) {
    sc.n[j] = double(nj[j]);
    sc.s[j] = double(a.S[j]);
  }
  auto* canon64 = static_cast<unsigned long long*>(sk);
  if (nc <= kRankMax) {
    k_rank5<<<unsigned((uint64_t(nc) * kRankLanes + 255) / 256), 256, 0, st>>>(
        canon64, static_cast<unsigned long long*>(cnt), nc, sc, canon, raw, est);
  } else {
    void *skt = nullptr, *svt = nullptr;
    HM_TRY(get(&skt, size_t(nc) * 8));
    HM_TRY(get(&svt, size_t(nc) * 4));
    auto *order = static_cast<uint32_t*>(sv), *order_tmp = static_cast<uint32_t*>(svt);
    auto* canon_tmp = static_cast<unsigned long long*>(skt);
    HM_TRY(radix_sort_pairs(canon64, order, canon_tmp, order_tmp, nc, 26, st));
    k_finish5<<<grid5(nc), 256, 0, st>>>(canon64, order, static_cast<unsigned long long*>(cnt), nc, sc, canon, raw, est);
  }
  HM_HIP(hipGetLastError());
  HM_HIP(hipStreamSynchronize(st));
  return HM_OK;
}

}  // namespace hm

extern "C" {

int hm_order5_sizes(const hm_graph* H, uint64_t* n_by_size4, void* stream) {
  try {
    if (!H || !n_by_size4) {
      hm::set_error("NULL argument to hm_order5_sizes");
      return HM_EINVAL;
    }
    HM_TRY(hm::ensure_order5(const_cast<hm_graph*>(H), static_cast<hipStream_t>(stream)));
    n_by_size4[0] = H->n_by_size[2];
    n_by_size4[1] = H->n_by_size[3];
    n_by_size4[2] = H->n_by_size[4];
    n_by_size4[3] = H->n5;
    return HM_OK;
  } catch (...) {
    return hm::api_failure();
  }
}

int count_sampled5(const hm_graph* H, double fraction, uint64_t seed, uint64_t capacity, uint32_t* canon, int64_t* raw,
                   float* est, uint64_t* n_classes, void* stream) {
  try {
    if (!H || !canon || !raw || !est || !n_classes) {
      hm::set_error("NULL argument to count_sampled5");
      return HM_EINVAL;
    }
    if (!(fraction > 0.0 && fraction <= 1.0)) {
      hm::set_error("fraction must be in (0, 1]");
      return HM_EINVAL;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    HM_TRY(hm::ensure_order5(const_cast<hm_graph*>(H), st));
    const uint64_t nj[6] = {0, 0, H->n_by_size[2], H->n_by_size[3], H->n_by_size[4], H->n5};
    uint64_t S[6] = {0, 0, 0, 0, 0, 0};
    for (int j = 2; j <= 5; ++j) S[j] = uint64_t(std::ceil(fraction * double(nj[j])));
    const uint32_t* idx[6] = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
    return hm::sampled5(const_cast<hm_graph*>(H), idx, S, seed, capacity, canon, raw, est, n_classes, st);
  } catch (...) {
    return hm::api_failure();
  }
}

int count_sampled5_indices(const hm_graph* H, const uint32_t* idx2, uint64_t s2, const uint32_t* idx3, uint64_t s3,
                           const uint32_t* idx4, uint64_t s4, const uint32_t* idx5, uint64_t s5, uint64_t capacity,
                           uint32_t* canon, int64_t* raw, float* est, uint64_t* n_classes, void* stream) {
  try {
    if (!H || !canon || !raw || !est || !n_classes) {
      hm::set_error("NULL argument to count_sampled5_indices");
      return HM_EINVAL;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    HM_TRY(hm::ensure_order5(const_cast<hm_graph*>(H), st));
    const uint32_t* idx[6] = {nullptr, nullptr, idx2, idx3, idx4, idx5};
    const uint64_t S[6] = {0, 0, s2, s3, s4, s5};
    const uint64_t nj[6] = {0, 0, H->n_by_size[2], H->n_by_size[3], H->n_by_size[4], H->n5};
    for (int j = 2; j <= 5; ++j)
      if (S[j] && (!idx[j] || !nj[j])) {
        hm::set_error("stratum %d: draws without an index array or from an empty stratum", j);
        return HM_EINVAL;
      }
    // every index must lie in its stratum (checked on the host copy)
    for (int j = 2; j <= 5; ++j) {
      if (!S[j]) continue;
      std::vector<uint32_t> h(S[j]);
      HM_HIP(hipMemcpy(h.data(), idx[j], S[j] * 4, hipMemcpyDeviceToHost));
      for (uint32_t x : h)
        if (x >= nj[j]) {
          hm::set_error("a sample index lies outside its stratum");
          return HM_EINVAL;
        }
    }
    return hm::sampled5(const_cast<hm_graph*>(H), idx, S, 0, capacity, canon, raw, est, n_classes, st);
  } catch (...) {
    return hm::api_failure();
  }
}

}  // extern "C"
