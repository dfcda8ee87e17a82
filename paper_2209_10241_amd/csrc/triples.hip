// Exact order-4 counts around the 3-node hyperedges on hypergraphs without
// adjacency bit rows (case (b) of Algorithm 3, Section 4.2).
//
// What is wanted: every connected 4-node set S that holds 3-node hyperedges
// T(S) and is no 4-node hyperedge, counted once in the class of its pairs and
// T(S), and once in the pairwise shape of its pairs (when they connect it).
// Written as a sum of terms that need no set to be looked at twice:
//
//   (1) every e in T(S) counts S as if e were its only 3-node hyperedge: the
//       nodes v outside e by which of e's members they are paired with, from
//       degrees, the common neighbours of e's three pairs (kept in the pair
//       index) and of all three members (k_tri_items).  Sets where v is
//       paired with no member are in no such term.
//   (2) a set with two or more 3-node hyperedges takes those terms back and
//       counts its class once.  It is found at the pair {x, y} that two of
//       them share: {x, y, t} and {x, y, z} are entries t < z of the run of
//       {x, y} in the pair index.  The two smallest 3-node hyperedges of S
//       decide (the others only undo (3)).
//   (3) most t, z of a run have nothing else between them: not a pair, and
//       neither {x, t, z} nor {y, t, z} a 3-node hyperedge.  What such a set
//       adds depends only on how t and z are paired with x and y, so the
//       run's counts of its entries by that (four classes) give all of them
//       in closed form (k_run_plan); k_run_items replaces the closed form
//       where t and z are related.
//   (4) 4-node hyperedges are not looked at: where one holds 3-node
//       hyperedges, what (1) to (3) counted for it is one set of its pairs
//       and T(S), which case (a) subtracts when it classifies it.
//
// The related t, z of an entry t are found by testing the later entries of its
// run, or from t's side (its pairwise row and the runs of {x, t} and {y, t},
// above t), whichever is shorter.  Both kinds of work are lists of very
// uneven lengths (an entry or a hyperedge has from none to tens of thousands
// of items), so their lengths are scanned and every thread takes items of the
// concatenated list, finding an item's owner in a window of the scan held in
// LDS.
//
// What bounds the item kernels is the latency of their dependent loads (a node,
// two or three memberships): (1) runs two items of a thread at once with eight
// wavefronts per SIMD, (2) one item with six (it then needs no scratch; two
// items with five took 0.96 ms).  808,000 3-node hyperedges on 50,000 nodes
// (heavy-tailed; 2.4 million entries, runs of up to 7,490): 163 million items
// in 0.50 ms (1) and 45 million in 0.88 (2), 0.14 ms each for the plans.  A
// wavefront per hyperedge and then per entry, which looked at every set from
// each of its 3-node hyperedges, took 2.06 and 6.33 ms, and needed an index of
// the 4-node hyperedges (0.55 ms).
#include <algorithm>

#include "hm_sparse.h"

namespace hm {
namespace {

// Owners whose records are planned at once (bounds the planning memory, 64
// bytes each).
constexpr uint64_t kPlanChunk = 1ull << 25;
constexpr uint32_t kTriUnit = 16384, kRunUnit = 2048;   // items a workgroup takes at a time
constexpr uint32_t kWindow = kThreads;   // owners of a unit looked at together
// units after which a workgroup's 32-bit counters are emptied
constexpr uint32_t kUnitsPerFlush = 1u << 16;

unsigned grid_cap(uint64_t items, uint64_t per_block, unsigned cap) {
  const uint64_t g = (items + per_block - 1) / per_block;
  return unsigned(std::max<uint64_t>(1, std::min<uint64_t>(g, cap)));
}

// The last p in [l, h) with pre[p] <= cur, given pre[l] <= cur < pre[h]; the
// wavefront's lanes take 64 probes a step and all return it.
__device__ __forceinline__ uint64_t owner_of(const unsigned long long* __restrict__ pre, uint64_t l, uint64_t h,
                                             unsigned long long cur) {
  const uint32_t lane = threadIdx.x & (kWave - 1);
  while (h - l > 1) {
    const uint64_t step = (h - l + kWave - 1) / kWave;
    const uint64_t q = l + step * lane;
    const bool le = q < h && pre[q] <= cur;
    l += step * (uint32_t(__popcll(__ballot(le))) - 1u);
    h = min(h, l + step);
  }
  return l;
}

// Hands out item k of every owner of [0, m), pre being the exclusive scan of
// the owners' item counts (pre[m] the total), over the whole grid; every
// thread of the workgroup calls this.  stage(slot, p) puts what owner p needs
// into slot of LDS, and items(slot, k, live) takes B items at once (slot[b],
// k[b] meaningful when live[b]), so that the loads of a thread's items go out
// together.  flush() is called by every thread after kUnitsPerFlush units and
// at the end.  s_pre: LDS of kWindow + 1 words.
//
// A workgroup claims units of kUnit items, the first one by its number, fewer
// items when there are not enough for the grid.  (In shares fixed beforehand
// k_tri_items took 0.75 ms and k_run_items 1.15 where claims took 0.57 and
// 0.87.)  Units whose owners fit in a few windows of kWindow find an item's
// owner in LDS; where most owners have no items, every thread searches the
// scan itself and stages its own owner (220,000 items of 1.1 million owners in
// k_run_items: 372 us by windows in units of 1,024, 131 in small ones, 43 so).
template <uint32_t B, uint32_t kUnit, typename Stage, typename Items, typename Flush>
__device__ __forceinline__ void flat_items(const unsigned long long* __restrict__ pre, uint64_t m,
                                           unsigned long long* __restrict__ next, uint32_t* s_pre,
                                           Stage stage, Items items, Flush flush) {
  static_assert(kUnit % (kThreads * B) == 0, "whole batches");
  static_assert(kWindow == uint32_t(kThreads), "an owner per thread");
  __shared__ uint64_t s_first, s_last;
  __shared__ unsigned long long s_unit;
  const uint32_t tid = threadIdx.x;
  const unsigned long long total = pre[m];
  const uint32_t unit = uint32_t(min<unsigned long long>(kUnit, max<unsigned long long>(kWave, total / gridDim.x + 1)));
  const unsigned long long n_units = (total + unit - 1) / unit;
  uint32_t done = 0;
  for (unsigned long long u = blockIdx.x; u < n_units;) {
    unsigned long long cur = u * unit;
    const unsigned long long end = min(total, cur + unit);
    while (cur < end) {
      if (tid < uint32_t(kWave)) {
        const uint64_t p = owner_of(pre, 0, m, cur);
        if (tid == 0) s_first = p;
      } else if (tid < 2 * uint32_t(kWave)) {
        const uint64_t p = owner_of(pre, 0, m, end - 1);
        if (tid == uint32_t(kWave)) s_last = p;
      }
      __syncthreads();
      const uint64_t p0 = s_first, p1 = s_last;
      const bool sparse = p1 - p0 >= 4 * kWindow;
      uint32_t n = uint32_t(end - cur), skipped = 0;
      if (!sparse) {
        const uint64_t p = p0 + tid;
        const unsigned long long a = pre[min(p, m)], b = pre[min(p + 1, m)];
        skipped = uint32_t(cur - pre[p0]);   // items of the first owner before cur
        s_pre[tid] = a <= cur ? 0u : uint32_t(min<unsigned long long>(a - cur, kUnit));
        if (tid == kThreads - 1) s_pre[kWindow] = uint32_t(min<unsigned long long>(b - cur, kUnit));
        if (a < b && a < end) stage(tid, p);
        __syncthreads();
        n = min(n, s_pre[kWindow]);
      }
      for (uint32_t i0 = 0; i0 < n; i0 += sparse ? uint32_t(kThreads) : kThreads * B) {
        uint32_t j[B], k[B];
        bool live[B];
#pragma unroll
        for (uint32_t b = 0; b < B; ++b) {
          j[b] = k[b] = 0;
          live[b] = false;
        }
        if (sparse) {
          live[0] = i0 + tid < n;
          if (live[0]) {
            uint64_t l = p0, h = p1 + 1;
            while (h - l > 1) {
              const uint64_t mid = (l + h) >> 1;
              if (pre[mid] <= cur + i0 + tid) l = mid;
              else h = mid;
            }
            j[0] = tid;
            k[0] = uint32_t(cur + i0 + tid - pre[l]);
            stage(tid, l);
          }
        } else {
#pragma unroll
          for (uint32_t s = kWindow / 2; s; s >>= 1) {
#pragma unroll
            for (uint32_t b = 0; b < B; ++b)
              if (s_pre[j[b] + s] <= i0 + b * kThreads + tid) j[b] += s;
          }
#pragma unroll
          for (uint32_t b = 0; b < B; ++b) {
            const uint32_t i = i0 + b * kThreads + tid;
            live[b] = i < n;
            k[b] = i - s_pre[j[b]] + (j[b] == 0 ? skipped : 0u);
          }
        }
        items(j, k, live);
      }
      __syncthreads();
      cur += n;
    }
    if (++done == kUnitsPerFlush) {
      done = 0;
      flush();
    }
    if (n_units <= gridDim.x) break;
    if (tid == 0) s_unit = gridDim.x + atomicAdd(next, 1ull);
    __syncthreads();
    u = s_unit;
  }
  flush();
}

// Whether z is among the ascending l[0, n).
__device__ inline uint32_t holds(const uint32_t* __restrict__ l, uint32_t n, uint32_t z) {
  uint32_t at = 0;   // entries before at are <= z
  while (n > 1) {
    const uint32_t half = n >> 1;
    at += l[at + half] <= z ? half : 0u;
    n -= half;
  }
  return n && l[at] == z;
}

__device__ inline void swap2(uint32_t& a, uint32_t& b) { const uint32_t t = a; a = b; b = t; }
__device__ inline void swap2(int& a, int& b) { const int t = a; a = b; b = t; }

__device__ inline void add_class(const uint8_t* lut, unsigned long long* h, uint32_t pattern, unsigned long long n) {
  const uint8_t c = lut[pattern];
  if (c != 0xFF) atomicAdd(&h[c], n);
}

// ---------------------------------------------------------------- (1)
// n nodes v outside hyperedges with pairwise pattern base (bits ab, ac, bc),
// paired with the members in cmb (bits a, b, c).
__device__ inline void add_combo(const uint8_t* lut, unsigned long long* h_main, unsigned long long* h_sub,
                                 uint32_t base, uint32_t cmb, unsigned long long n) {
  const uint32_t pairs = base | ((cmb & 1u) << 4) | (((cmb >> 1) & 1u) << 5) | ((cmb >> 2) << 7);
  add_class(lut, h_main, pairs | (1u << 3), n);
  add_class(lut, h_sub, pairs, n);
}

// The common neighbours of e's members: the entries z of the shortest of
// their rows are tested against the other two (x first), or, when all three
// have dense rows of fewer words than that, the rows' words are combined.
struct TriRec {
  uint32_t row;      // the first entry of the row, or its dense row
  uint32_t x, y;
  int32_t hx, hy;    // dense rows of x and y, or -1
  uint32_t flags;    // bits 0..2: e's pairwise pattern; bit 3: dense rows combined
};

constexpr uint32_t kTriCopies = 16;   // copies of the 64 counters (lanes of a wavefront add to like ones)

__global__ void __launch_bounds__(kThreads) k_tri_plan(View v, PairLinks pl, uint64_t first, uint64_t m,
                                                       TriRec* __restrict__ rec, unsigned long long* __restrict__ cnt,
                                                       unsigned long long* __restrict__ next,
                                                       const uint8_t* __restrict__ lut_g,
                                                       unsigned long long* __restrict__ hist) {
  __shared__ uint8_t lut[2048];
  __shared__ unsigned long long h_main[256], h_sub[256];
  __shared__ unsigned long long bins[64][kTriCopies];
  load_lut(lut, lut_g, 2048);
  h_main[threadIdx.x] = 0;
  h_sub[threadIdx.x] = 0;
  for (uint32_t i = threadIdx.x; i < 64 * kTriCopies; i += kThreads) (&bins[0][0])[i] = 0;
  __syncthreads();
  const uint32_t copy = threadIdx.x & (kTriCopies - 1);
  if (blockIdx.x == 0 && threadIdx.x == 0) *next = 0;
  for (uint64_t i = uint64_t(blockIdx.x) * kThreads + threadIdx.x; i <= m; i += uint64_t(gridDim.x) * kThreads) {
    unsigned long long items = 0;
    if (i < m) {
      const uint32_t* e = v.e3 + 3 * (first + i);
      const uint32_t a = e[0], b = e[1], c = e[2];
      const Probe64 qab = probe2_start(v.hs2, a, b), qac = probe2_start(v.hs2, a, c), qbc = probe2_start(v.hs2, b, c);
      const uint32_t cab = pl_codeg(pl, a, b), cac = pl_codeg(pl, a, c), cbc = pl_codeg(pl, b, c);
      const uint32_t da = deg2_of(v, a), db = deg2_of(v, b), dc = deg2_of(v, c);
      const uint32_t pab = probe64_end(v.hs2, qab), pac = probe64_end(v.hs2, qac), pbc = probe64_end(v.hs2, qbc);
      const uint32_t base = pab | (pac << 1) | (pbc << 2);
      // (differences may be negative before the common neighbours of all
      // three are added: sums modulo 2^64)
      const unsigned long long iab = cab - pac * pbc, iac = cac - pab * pbc, ibc = cbc - pab * pac;
      const unsigned long long sa = da - pab - pac, sb = db - pab - pbc, sc = dc - pac - pbc;
      const unsigned long long n[8] = {0, sa - iab - iac, sb - iab - ibc, iab, sc - iac - ibc, iac, ibc, 0};
#pragma unroll
      for (uint32_t cmb = 1; cmb < 7; ++cmb)
        if (n[cmb]) atomicAdd(&bins[base * 8 + cmb][copy], n[cmb]);
      if (cab && cac && cbc) {
        uint32_t r = a, x = b, y = c, dr = da, dx = db, dy = dc;
        if (dx < dr) { swap2(r, x); swap2(dr, dx); }
        if (dy < dr) { swap2(r, y); swap2(dr, dy); }
        if (dy < dx) { swap2(x, y); swap2(dx, dy); }
        // (the smaller row as x, tested first: fewer z pass it; but a dense
        // row before a hash table)
        int hx = hub_of(pl, x), hy = hub_of(pl, y);
        if (hx < 0 && hy >= 0) { swap2(x, y); swap2(hx, hy); }
        const int hr = hub_of(pl, r);
        const bool dense = hr >= 0 && hx >= 0 && hy >= 0 && dr > pl.hub_w;
        items = dense ? pl.hub_w : dr;
        TriRec t;
        t.row = dense ? uint32_t(hr) : v.g2_off[r];
        t.x = x;
        t.y = y;
        t.hx = hx;
        t.hy = hy;
        t.flags = base | (uint32_t(dense) << 3);
        rec[i] = t;
      }
    }
    cnt[i] = items;
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    unsigned long long n = 0;
    for (uint32_t k = 0; k < kTriCopies; ++k) n += bins[threadIdx.x][k];
    if (n) add_combo(lut, h_main, h_sub, threadIdx.x >> 3, threadIdx.x & 7u, n);
  }
  __syncthreads();
  unsigned long long* hc = hist_copy(hist, kExactHistStride);
  flush(h_main, hc + kMain, 256);
  flush(h_sub, hc + kSub, 256);
}

__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(8,8))) k_tri_items(View v, PairLinks pl, uint64_t m,
                                                        const TriRec* __restrict__ rec,
                                                        const unsigned long long* __restrict__ pre,
                                                        unsigned long long* __restrict__ next,
                                                        const uint8_t* __restrict__ lut_g,
                                                        unsigned long long* __restrict__ hist) {
  constexpr uint32_t kCopies = 32;
  __shared__ uint8_t lut[2048];
  __shared__ unsigned long long h_main[256], h_sub[256];
  __shared__ uint32_t bins[8][kCopies];
  __shared__ uint32_t s_pre[kWindow + 1];
  __shared__ TriRec s_rec[kWindow];
  load_lut(lut, lut_g, 2048);
  h_main[threadIdx.x] = 0;
  h_sub[threadIdx.x] = 0;
  bins[threadIdx.x / kCopies][threadIdx.x % kCopies] = 0;
  __syncthreads();
  const uint32_t copy = threadIdx.x % kCopies;
  flat_items<2, kTriUnit>(
      pre, m, next, s_pre,
      [&](uint32_t slot, uint64_t p) { s_rec[slot] = rec[p]; },
      [&](const uint32_t (&slot)[2], const uint32_t (&k)[2], const bool (&live)[2]) {
        TriRec t[2];
        uint32_t z[2], hits[2];
        Probe64 q[2];
#pragma unroll
        for (int b = 0; b < 2; ++b)
          if (live[b]) t[b] = s_rec[slot[b]];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          z[b] = 0;
          if (!live[b]) continue;
          if (t[b].flags & 8u)
            z[b] = pl.hub_bits[uint64_t(t[b].row) * pl.hub_w + k[b]] & pl.hub_bits[uint64_t(t[b].hx) * pl.hub_w + k[b]] &
                   pl.hub_bits[uint64_t(t[b].hy) * pl.hub_w + k[b]];
          else
            z[b] = v.g2_adj[t[b].row + k[b]];
        }
        // (the first slot of a hash table and the word of a dense row alike)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          hits[b] = 0;
          if (!live[b]) continue;
          if (t[b].flags & 8u) hits[b] = uint32_t(__popc(z[b]));
          else if (t[b].hx >= 0) hits[b] = hub_adj(pl, t[b].hx, z[b]);
          else q[b] = probe2_start(v.hs2, t[b].x, z[b]);
        }
#pragma unroll
        for (int b = 0; b < 2; ++b)
          if (live[b] && !(t[b].flags & 8u) && t[b].hx < 0) hits[b] = uint32_t(probe64_end(v.hs2, q[b]));
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          if (!hits[b] || (t[b].flags & 8u)) continue;
          if (t[b].hy >= 0) hits[b] = hub_adj(pl, t[b].hy, z[b]);
          else q[b] = probe2_start(v.hs2, t[b].y, z[b]);
        }
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          if (!hits[b]) continue;
          if (!(t[b].flags & 8u) && t[b].hy < 0) hits[b] = uint32_t(probe64_end(v.hs2, q[b]));
          if (hits[b]) atomicAdd(&bins[t[b].flags & 7u][copy], hits[b]);
        }
      },
      [&]() {
        // one common neighbour of all three members moves one node between
        // the combinations by inclusion-exclusion
        __syncthreads();
        if (threadIdx.x < 64) {
          const uint32_t base = threadIdx.x >> 3, cmb = threadIdx.x & 7u;
          unsigned long long n = 0;
          for (uint32_t k = 0; k < kCopies; ++k) n += bins[base][k];
          if (cmb == 3 || cmb == 5 || cmb == 6) n = 0ull - n;
          if (n && cmb) add_combo(lut, h_main, h_sub, base, cmb, n);
        }
        __syncthreads();
        bins[threadIdx.x / kCopies][threadIdx.x % kCopies] = 0;
        __syncthreads();
      });
  unsigned long long* hc = hist_copy(hist, kExactHistStride);
  flush(h_main, hc + kMain, 256);
  flush(h_sub, hc + kSub, 256);
}

// ---------------------------------------------------------------- (2), (3)
// A set {x, y, t, z} whose 3-node hyperedges {x, y, t} and {x, y, z} meet at
// an index run: x ~ y, how t and z are paired with x and y (bit 0: x, bit 1:
// y), t ~ z, {x, t, z}, {y, t, z}.  n such sets take back the terms (1) of
// their 3-node hyperedges and count once.
__device__ inline void add_run_set(const uint8_t* lut, unsigned long long* h_main, unsigned long long* h_sub,
                                   uint32_t xy, uint32_t ct, uint32_t cz, uint32_t tz, uint32_t xtz, uint32_t ytz,
                                   unsigned long long n) {
  // local nodes x, y, t, z = 0, 1, 2, 3
  const uint32_t pairs = xy | (ct << 1) | (cz << 4) | (tz << 7);
  add_class(lut, h_main, pairs | (1u << 3) | (1u << 6) | (xtz << 8) | (ytz << 9), n);
  if (cz | tz) add_class(lut, h_main, pairs | (1u << 3), 0ull - n);
  if (ct | tz) add_class(lut, h_main, pairs | (1u << 6), 0ull - n);
  if (xtz && (xy | (ct >> 1) | (cz >> 1))) add_class(lut, h_main, pairs | (1u << 8), 0ull - n);
  if (ytz && (xy | (ct & 1u) | (cz & 1u))) add_class(lut, h_main, pairs | (1u << 9), 0ull - n);
  // (pairs that connect the set connect each of its nodes to the others)
  add_class(lut, h_sub, pairs, 0ull - (1u + xtz + ytz) * n);
}

// Prefix counts of the entries by adjacency class: the four classes' counts of
// each tile of kClassTile entries (class-major, so that one scan serves all
// four), then within each tile.  pre[c * (n + 1) + p] is the number of entries
// before position p of class c.
constexpr uint32_t kClassTile = 2048;
__global__ void __launch_bounds__(kThreads) k_pl_class_count(const uint8_t* __restrict__ adj, uint64_t n,
                                                             uint32_t* __restrict__ counts) {
  __shared__ uint32_t c[4];
  if (threadIdx.x < 4) c[threadIdx.x] = 0;
  __syncthreads();
  const uint64_t base = uint64_t(blockIdx.x) * kClassTile;
#pragma unroll
  for (uint32_t r = 0; r < kClassTile / kThreads; ++r) {
    const uint64_t p = base + r * kThreads + threadIdx.x;
    const uint32_t a = p < n ? adj[p] : 4u;
#pragma unroll
    for (uint32_t cl = 0; cl < 4; ++cl) {
      const uint32_t k = uint32_t(__popcll(__ballot(a == cl)));
      if ((threadIdx.x & (kWave - 1)) == 0 && k) atomicAdd(&c[cl], k);
    }
  }
  __syncthreads();
  if (threadIdx.x < 4) counts[uint64_t(threadIdx.x) * gridDim.x + blockIdx.x] = c[threadIdx.x];
}

__global__ void __launch_bounds__(kThreads) k_pl_class_prefix(const uint8_t* __restrict__ adj, uint64_t n,
                                                              const uint32_t* __restrict__ before,
                                                              uint32_t* __restrict__ pre) {
  __shared__ uint32_t part[2][4][kWavesPerBlock];
  const uint32_t lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
  const unsigned long long below = (1ull << lane) - 1ull;
  const uint64_t base = uint64_t(blockIdx.x) * kClassTile;
  uint32_t at[4];
#pragma unroll
  for (uint32_t cl = 0; cl < 4; ++cl)
    at[cl] = before[uint64_t(cl) * gridDim.x + blockIdx.x] - before[uint64_t(cl) * gridDim.x];
  for (uint32_t r = 0; r < kClassTile / kThreads; ++r) {
    const uint64_t p = base + r * kThreads + threadIdx.x;
    const uint32_t a = p < n ? adj[p] : 4u;
    uint32_t mine[4];
#pragma unroll
    for (uint32_t cl = 0; cl < 4; ++cl) {
      const unsigned long long m = __ballot(a == cl);
      mine[cl] = uint32_t(__popcll(m & below));
      if (lane == 0) part[r & 1][cl][wv] = uint32_t(__popcll(m));
    }
    __syncthreads();
#pragma unroll
    for (uint32_t cl = 0; cl < 4; ++cl) {
      uint32_t x = at[cl] + mine[cl];
      for (uint32_t q = 0; q < uint32_t(kWavesPerBlock); ++q) {
        const uint32_t k = part[r & 1][cl][q];
        if (q < wv) x += k;
        at[cl] += k;
      }
      if (p < n) pre[cl * (n + 1) + p] = x;
      if (p + 1 == n) pre[cl * (n + 1) + n] = x + (a == cl);
    }
  }
}

// What entry t (position p of the index) of the run of {x, y} looks at.  Bit 0 of flags set: the later
// entries of the run, each tested against t's pairwise row (n0 entries from
// a0) and the runs of {x, t} (n1 from a1) and {y, t} (n2 from a2).  Otherwise
// the entries above t of those three lists (n0, n1 and n2 of them), searched
// for in the run of {x, y}, which ends at end.  flags: bits 1, 2 how t is
// paired with x and y; bit 3: x ~ y; from bit 4: t's dense row plus one, or 0.
struct RunRec {
  uint32_t x, y, t, flags, a0, n0, a1, n1, a2, n2, p, end;
};
// t's related nodes in short lists are searched for there (the lists are
// shared by an entry's items and stay in the L1), in longer ones by a probe of
// the hash sets.
constexpr uint32_t kSearchMax = 256;

__global__ void __launch_bounds__(kThreads) k_run_plan(View v, PairLinks pl, const uint32_t* __restrict__ pre,
                                                       uint64_t first, uint64_t m, RunRec* __restrict__ rec,
                                                       unsigned long long* __restrict__ cnt,
                                                       unsigned long long* __restrict__ next,
                                                       const uint8_t* __restrict__ lut_g,
                                                       unsigned long long* __restrict__ hist) {
  __shared__ uint8_t lut[2048];
  __shared__ unsigned long long h_main[256], h_sub[256];
  __shared__ unsigned long long closed[32];   // sets by x ~ y, class of t, class of z
  load_lut(lut, lut_g, 2048);
  h_main[threadIdx.x] = 0;
  h_sub[threadIdx.x] = 0;
  if (threadIdx.x < 32) closed[threadIdx.x] = 0;
  __syncthreads();
  if (blockIdx.x == 0 && threadIdx.x == 0) *next = 0;
  for (uint64_t i = uint64_t(blockIdx.x) * kThreads + threadIdx.x; i <= m; i += uint64_t(gridDim.x) * kThreads) {
    unsigned long long items = 0;
    const uint64_t p = first + i;
    const unsigned long long key = i < m ? pl.keys[p] : 0;
    const bool begins = i < m && (p == 0 || pl.keys[p - 1] != key);
    const bool ends = i == m || p + 1 == pl.n || pl.keys[p + 1] != key;
    if (i < m && !ends) {   // (an entry that ends its run has no later one)
      const uint32_t x = uint32_t(key >> 32), y = uint32_t(key), t = pl.third[p];
      uint64_t lo, lo_xt, lo_yt;
      uint32_t L, len_xt, len_yt;
      const uint32_t xy = uint32_t(has2(v.hs2, x, y));
      pl_find(pl, key, &lo, &L);
      if (begins) {
        unsigned long long n[4];
#pragma unroll
        for (uint32_t c = 0; c < 4; ++c) n[c] = pre[c * (pl.n + 1) + lo + L] - pre[c * (pl.n + 1) + lo];
#pragma unroll
        for (uint32_t c = 0; c < 4; ++c) {
          if (n[c] > 1) atomicAdd(&closed[xy * 16 + c * 5], n[c] * (n[c] - 1) / 2);
#pragma unroll
          for (uint32_t d = c + 1; d < 4; ++d)
            if (n[c] && n[d]) atomicAdd(&closed[xy * 16 + c * 4 + d], n[c] * n[d]);
        }
      }
      pl_find(pl, ((unsigned long long)min(x, t) << 32) | max(x, t), &lo_xt, &len_xt);
      pl_find(pl, ((unsigned long long)min(y, t) << 32) | max(y, t), &lo_yt, &len_yt);
      const uint32_t row = v.g2_off[t], dt = v.g2_off[t + 1] - row;
      const uint32_t end = uint32_t(lo) + L, later = end - uint32_t(p) - 1;
      if (dt || len_xt > 1 || len_yt > 1) {   // (else nothing is related to t)
        RunRec r;
        r.x = x;
        r.y = y;
        r.t = t;
        r.flags = 1u | (uint32_t(pl.adj[p]) << 1) | (xy << 3) | (uint32_t(hub_of(pl, t) + 1) << 4);
        r.a0 = row;
        r.n0 = dt;
        r.a1 = uint32_t(lo_xt);
        r.n1 = len_xt;
        r.a2 = uint32_t(lo_yt);
        r.n2 = len_yt;
        r.end = end;
        r.p = uint32_t(p);
        items = later;
        if (later > uint64_t(dt) + len_xt + len_yt) {
          r.flags &= ~1u;
          r.a0 = upper_bound(v.g2_adj, row, row + dt, t);
          r.n0 = row + dt - r.a0;
          r.a1 = upper_bound(pl.third, r.a1, r.a1 + len_xt, t);
          r.n1 = uint32_t(lo_xt) + len_xt - r.a1;
          r.a2 = upper_bound(pl.third, r.a2, r.a2 + len_yt, t);
          r.n2 = uint32_t(lo_yt) + len_yt - r.a2;
          items = uint64_t(r.n0) + r.n1 + r.n2;
        }
        if (items) rec[i] = r;
      }
    }
    cnt[i] = items;
  }
  __syncthreads();
  if (threadIdx.x < 32) {
    const uint32_t b = threadIdx.x;
    if (closed[b]) add_run_set(lut, h_main, h_sub, b >> 4, (b >> 2) & 3u, b & 3u, 0, 0, 0, closed[b]);
  }
  __syncthreads();
  unsigned long long* hc = hist_copy(hist, kExactHistStride);
  flush(h_main, hc + kMain, 256);
  flush(h_sub, hc + kSub, 256);
}

// The related t, z are counted by their nine bits (x ~ y, class of t, class
// of z, t ~ z, {x, t, z}, {y, t, z}, whether {x, y, t} and {x, y, z} are the
// two smallest 3-node hyperedges of the set), in two sets of counters that the
// wavefronts share by pairs, which become class counts at the end.
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(6,6))) k_run_items(View v, PairLinks pl, uint64_t m,
                                                        const RunRec* __restrict__ rec,
                                                        const unsigned long long* __restrict__ pre,
                                                        unsigned long long* __restrict__ next,
                                                        const uint8_t* __restrict__ lut_g,
                                                        unsigned long long* __restrict__ hist) {
  __shared__ uint8_t lut[2048];
  __shared__ unsigned long long h_main[256], h_sub[256];
  __shared__ uint32_t bins[2][512];
  __shared__ uint32_t s_pre[kWindow + 1];
  __shared__ RunRec s_rec[kWindow];
  load_lut(lut, lut_g, 2048);
  h_main[threadIdx.x] = 0;
  h_sub[threadIdx.x] = 0;
  for (uint32_t i = threadIdx.x; i < 2 * 512; i += kThreads) (&bins[0][0])[i] = 0;
  __syncthreads();
  uint32_t* mine = bins[(threadIdx.x / kWave) & 1];
  flat_items<1, kRunUnit>(
      pre, m, next, s_pre,
      [&](uint32_t slot, uint64_t p) { s_rec[slot] = rec[p]; },
      [&](const uint32_t (&slot)[1], const uint32_t (&item)[1], const bool (&live)[1]) {
        if (!live[0]) return;
        const RunRec& r = s_rec[slot[0]];
        const uint32_t k = item[0], p = r.p, x = r.x, y = r.y, t = r.t;
        const int rt = int(r.flags >> 4) - 1;
        uint32_t z, cz, tz, xtz, ytz;
        if (r.flags & 1u) {
          z = pl.third[p + 1 + k];
          cz = pl.adj[p + 1 + k];
          Probe64 q2;
          Probe128 qx, qy;
          if (rt < 0 && r.n0 > kSearchMax) q2 = probe2_start(v.hs2, t, z);
          if (r.n1 > kSearchMax) qx = probe3_start(v.hs3, x, t, z);
          if (r.n2 > kSearchMax) qy = probe3_start(v.hs3, y, t, z);
          tz = rt >= 0 ? hub_adj(pl, rt, z)
                       : (r.n0 > kSearchMax ? uint32_t(probe64_end(v.hs2, q2)) : holds(v.g2_adj + r.a0, r.n0, z));
          xtz = r.n1 > kSearchMax ? uint32_t(probe128_end(v.hs3, qx))
                                  : (r.n1 > 1 ? holds(pl.third + r.a1, r.n1, z) : 0u);
          ytz = r.n2 > kSearchMax ? uint32_t(probe128_end(v.hs3, qy))
                                  : (r.n2 > 1 ? holds(pl.third + r.a2, r.n2, z) : 0u);
          if (!(tz | xtz | ytz)) return;
        } else {
          // each related z once, from the first list that holds it
          const int from = k < r.n0 ? 0 : (k < r.n0 + r.n1 ? 1 : 2);
          z = from == 0 ? v.g2_adj[r.a0 + k] : pl.third[from == 1 ? r.a1 + (k - r.n0) : r.a2 + (k - r.n0 - r.n1)];
          const uint64_t at = run_find(pl, p + 1, r.end - p - 1, z);
          if (at == ~0ull) return;   // {x, y, z} is not a 3-node hyperedge
          tz = 1;
          if (from)
            tz = rt >= 0 ? hub_adj(pl, rt, z)
                         : (r.n0 > kSearchMax ? uint32_t(has2(v.hs2, t, z)) : holds(v.g2_adj + r.a0, r.n0, z));
          if (from && tz) return;
          xtz = from == 1 ? 1u : 0u;
          if (from != 1)
            xtz = r.n1 > kSearchMax ? uint32_t(probe128_end(v.hs3, probe3_start(v.hs3, x, t, z)))
                                    : holds(pl.third + r.a1, r.n1, z);
          if (from == 2 && xtz) return;
          ytz = from == 2 ? 1u : 0u;
          if (from != 2)
            ytz = r.n2 > kSearchMax ? uint32_t(probe128_end(v.hs3, probe3_start(v.hs3, y, t, z)))
                                    : holds(pl.third + r.a2, r.n2, z);
          cz = pl.adj[at];
        }
        // the smaller of two 3-node hyperedges of a set leaves out the larger node
        const uint32_t own = uint32_t((!xtz || y < t) && (!ytz || x < t));
        const uint32_t xy = (r.flags >> 3) & 1u, ct = (r.flags >> 1) & 3u;
        atomicAdd(&mine[xy | (ct << 1) | (cz << 3) | (tz << 5) | (xtz << 6) | (ytz << 7) | (own << 8)], 1u);
      },
      [&]() {
        __syncthreads();
        for (uint32_t b = threadIdx.x; b < 512; b += kThreads) {
          unsigned long long n = 0;
#pragma unroll
          for (uint32_t w = 0; w < 2u; ++w) {
            n += bins[w][b];
            bins[w][b] = 0;
          }
          if (!n) continue;
          const uint32_t xy = b & 1u, ct = (b >> 1) & 3u, cz = (b >> 3) & 3u;
          add_run_set(lut, h_main, h_sub, xy, ct, cz, 0, 0, 0, 0ull - n);
          if (b >> 8) add_run_set(lut, h_main, h_sub, xy, ct, cz, (b >> 5) & 1u, (b >> 6) & 1u, (b >> 7) & 1u, n);
        }
        __syncthreads();
      });
  unsigned long long* hc = hist_copy(hist, kExactHistStride);
  flush(h_main, hc + kMain, 256);
  flush(h_sub, hc + kSub, 256);
}

// Workgroups of the item kernels: enough to fill the chip, as units are short.
constexpr unsigned kItemGrid = 2048;

}  // namespace

// Adds (1) to (3) to H->hist (4: see k_case_a4).
int count_triples(const hm_graph* H, hipStream_t st) {
  const uint64_t n3 = H->n_by_size[3], n = 3 * n3;
  if (!n3) return HM_OK;
  HM_TRY(ensure_pair_links(const_cast<hm_graph*>(H), st));
  HM_TRY(ensure_hub_rows(const_cast<hm_graph*>(H), st));
  const uint8_t *lut4 = nullptr, *lut3 = nullptr;
  HM_TRY(device_luts(H->device, &lut4, &lut3));
  const View v = view_of(H);
  const PairLinks pl = pair_links_of(H);
  Scratch tmp(st);
  const uint64_t chunk = std::min(n, kPlanChunk), tiles = (n + kClassTile - 1) / kClassTile;
  static_assert(sizeof(RunRec) >= sizeof(TriRec) && sizeof(RunRec) == 48, "one buffer serves both");
  unsigned long long *cnt = nullptr, *at = nullptr;
  RunRec* rec = nullptr;
  uint32_t *pre = nullptr, *counts = nullptr, *before = nullptr;
  HM_TRY(tmp.get(&cnt, chunk + 1));
  HM_TRY(tmp.get(&at, chunk + 2));
  unsigned long long* next = at + chunk + 1;   // units claimed
  HM_TRY(tmp.get(&rec, chunk));
  HM_TRY(tmp.get(&pre, 4 * (n + 1)));
  HM_TRY(tmp.get(&counts, 4 * tiles));
  HM_TRY(tmp.get(&before, 4 * tiles));
  TriRec* tri = reinterpret_cast<TriRec*>(rec);
  for (uint64_t i = 0; i < n3; i += chunk) {
    const uint64_t m = std::min(chunk, n3 - i);
    k_tri_plan<<<grid_cap(m + 1, kThreads, 2048), kThreads, 0, st>>>(v, pl, i, m, tri, cnt, next, lut4, H->hist);
    HM_HIP(hipGetLastError());
    HM_TRY(scan_exclusive_u64(cnt, at, m + 1, st));
    ProfileScope ps("k_tri_items", st);
    k_tri_items<<<kItemGrid, kThreads, 0, st>>>(v, pl, m, tri, at, next, lut4, H->hist);
    HM_HIP(hipGetLastError());
  }
  k_pl_class_count<<<unsigned(tiles), kThreads, 0, st>>>(pl.adj, n, counts);
  HM_HIP(hipGetLastError());
  HM_TRY(scan_exclusive_u32(counts, before, 4 * tiles, nullptr, st));
  k_pl_class_prefix<<<unsigned(tiles), kThreads, 0, st>>>(pl.adj, n, before, pre);
  HM_HIP(hipGetLastError());
  for (uint64_t p = 0; p < n; p += chunk) {
    const uint64_t m = std::min(chunk, n - p);
    k_run_plan<<<grid_cap(m + 1, kThreads, 2048), kThreads, 0, st>>>(v, pl, pre, p, m, rec, cnt, next, lut4, H->hist);
    HM_HIP(hipGetLastError());
    HM_TRY(scan_exclusive_u64(cnt, at, m + 1, st));
    ProfileScope ps("k_run_items", st);
    k_run_items<<<kItemGrid, kThreads, 0, st>>>(v, pl, m, rec, at, next, lut4, H->hist);
    HM_HIP(hipGetLastError());
  }
  return HM_OK;
}

}  // namespace hm
