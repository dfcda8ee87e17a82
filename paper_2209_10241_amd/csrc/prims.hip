// Device primitives used while building graphs: exclusive scans, a stable
// LSD radix sort of (64-bit key, 32-bit value) pairs and fills.
#include <algorithm>

#include "hm_device.h"

namespace hm {
namespace {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;

template <typename T>
__device__ T block_exclusive_scan(T v, T* wave_sums, T* total) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  const T x = wave_inclusive_scan(v);
  if (lane == kWave - 1) wave_sums[wave] = x;
  __syncthreads();
  T before = 0, all = 0;
  for (int w = 0; w < kScanThreads / kWave; ++w) {
    T s = wave_sums[w];
    if (w < wave) before += s;
    all += s;
  }
  __syncthreads();
  *total = all;
  return before + x - v;
}

// (item i of a tile is kept at i + i / 8: a thread's eight consecutive items
// and a wavefront's 64 both then spread over the LDS banks)
__device__ inline int scan_slot(int i) { return i + (i >> 3); }

template <typename T>
__global__ void __launch_bounds__(kScanThreads) k_scan_tile(const T* __restrict__ in, T* __restrict__ out,
                                                            T* __restrict__ sums, uint64_t n) {
  __shared__ T tile[kScanTile + kScanTile / 8];
  __shared__ T wave_sums[kScanThreads / kWave];
  const uint64_t base = uint64_t(blockIdx.x) * kScanTile;
  // (all of the thread's loads before its LDS stores, so that they go out
  // together)
  T v[kScanItems];
#pragma unroll
  for (int r = 0; r < kScanItems; ++r) {
    const uint64_t g = base + uint64_t(r) * kScanThreads + threadIdx.x;
    v[r] = g < n ? in[g] : T(0);
  }
#pragma unroll
  for (int r = 0; r < kScanItems; ++r) tile[scan_slot(r * kScanThreads + threadIdx.x)] = v[r];
  __syncthreads();
  T local[kScanItems];
  T s = 0;
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) {
    local[j] = tile[scan_slot(threadIdx.x * kScanItems + j)];
    s += local[j];
  }
  T total;
  T off = block_exclusive_scan(s, wave_sums, &total);
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) {
    tile[scan_slot(threadIdx.x * kScanItems + j)] = off;
    off += local[j];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kScanTile; i += kScanThreads) {
    uint64_t g = base + i;
    if (g < n) out[g] = tile[scan_slot(i)];
  }
  if (threadIdx.x == 0 && sums) sums[blockIdx.x] = total;
}

template <typename T>
__global__ void k_scan_add(T* __restrict__ out, const T* __restrict__ offs, uint64_t n) {
  uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) out[i] += offs[i / kScanTile];
}

template <typename T>
__global__ void k_scan_total(const T* in, const T* out, uint64_t n, T* total) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *total = n ? out[n - 1] + in[n - 1] : T(0);
}

// Multi-level exclusive scan of n values: level l scans the block sums of
// level l-1, in ws (scan_ws_count(n) values).  No allocation and no host
// synchronisation.
uint64_t scan_ws_count(uint64_t n) {
  uint64_t count = 0;
  while (n > uint64_t(kScanTile)) {
    n = (n + kScanTile - 1) / kScanTile;
    count += 2 * n;    // block sums and their scan
  }
  return count + 1;
}

template <typename T>
int scan_ws(const T* in, T* out, uint64_t n, T* ws, hipStream_t st) {
  if (n == 0) return HM_OK;
  const uint64_t nb = (n + kScanTile - 1) / kScanTile;
  if (nb == 1) {
    k_scan_tile<T><<<1, kScanThreads, 0, st>>>(in, out, nullptr, n);
  } else {
    T *sums = ws, *sums_scan = ws + nb;
    k_scan_tile<T><<<unsigned(nb), kScanThreads, 0, st>>>(in, out, sums, n);
    HM_HIP(hipGetLastError());
    HM_TRY(scan_ws<T>(sums, sums_scan, nb, ws + 2 * nb, st));
    k_scan_add<T><<<unsigned((n + 255) / 256), 256, 0, st>>>(out, sums_scan, n);
  }
  HM_HIP(hipGetLastError());
  return HM_OK;
}

// The same with a workspace of its own, released in stream order.
template <typename T>
int scan_impl(const T* in, T* out, uint64_t n, hipStream_t st) {
  Scratch tmp(st);
  T* ws = nullptr;
  if (n > uint64_t(kScanTile)) HM_TRY(tmp.get(&ws, scan_ws_count(n)));
  return scan_ws<T>(in, out, n, ws, st);
}

// ------------------------------------------------------------------ radix sort
constexpr int kSortThreads = 256;
constexpr int kSortItems = 16;
constexpr int kSortTile = kSortThreads * kSortItems;
constexpr int kSortWaves = kSortThreads / kWave;

constexpr int kSortWaveItems = kSortItems * kWave;   // consecutive items a wavefront takes

// Digit counts of each tile, digit-major; a wavefront counts in a copy of its
// own.
template <typename K>
__global__ void __launch_bounds__(kSortThreads) k_sort_hist(const K* __restrict__ keys, uint64_t n, int shift,
                                                            uint32_t digit_mask, uint32_t* __restrict__ hist,
                                                            uint32_t nb) {
  __shared__ uint32_t counts[kSortWaves][256];
  const int wave = threadIdx.x / kWave;
#pragma unroll
  for (int w = 0; w < kSortWaves; ++w) counts[w][threadIdx.x] = 0;
  __syncthreads();
  const uint64_t base = uint64_t(blockIdx.x) * kSortTile;
  // every key of the thread loaded before any is counted (the loads go out
  // together rather than each behind the previous count)
  uint32_t d[kSortItems];
#pragma unroll
  for (int r = 0; r < kSortItems; ++r) {
    const uint64_t i = base + uint64_t(r) * kSortThreads + threadIdx.x;
    d[r] = i < n ? uint32_t(keys[i] >> shift) & digit_mask : 0xFFFFFFFFu;
  }
#pragma unroll
  for (int r = 0; r < kSortItems; ++r)
    if (d[r] != 0xFFFFFFFFu) atomicAdd(&counts[wave][d[r]], 1u);
  __syncthreads();
  uint32_t c = 0;
#pragma unroll
  for (int w = 0; w < kSortWaves; ++w) c += counts[w][threadIdx.x];
  hist[uint64_t(threadIdx.x) * nb + blockIdx.x] = c;
}

// Stable scatter.  A wavefront takes 1,024 consecutive items of the tile, 64
// a round, and counts its digits in LDS of its own, so that the rounds need no
// barrier: an item's rank is its wavefront's count so far plus its place among
// the round's equal digits (ballots over the digit bits).  Then the tile's
// order by digit is formed in LDS (keys, then values through the same space)
// and thread t writes the tile's t-th item in that order to its digit's
// global range, so that each digit's items of the tile go out as one
// contiguous run.  (`offsets` is scanned per tile of kScanTile counters;
// `above` holds the sums before each, null when there is one.)  A version
// with three barriers a round and both arrays in LDS (two workgroups a CU)
// took 38 us a pass over 2e6 to 3.8e6 items of 8-byte keys, this one 23.
template <typename K>
__global__ void __launch_bounds__(kSortThreads) k_sort_scatter(
    const K* __restrict__ keys, const uint32_t* __restrict__ vals, K* __restrict__ out_keys,
    uint32_t* __restrict__ out_vals, uint64_t n, int shift, int digit_bits, const uint32_t* __restrict__ hist,
    const uint32_t* __restrict__ offsets, const uint32_t* __restrict__ above, uint32_t nb) {
  __shared__ K s_keys[kSortTile];
  __shared__ uint32_t tile_off[256], global_off[256];
  __shared__ uint32_t cnt[kSortWaves][256];
  __shared__ uint32_t wave_sums[kSortWaves];
  uint32_t* s_vals = reinterpret_cast<uint32_t*>(s_keys);
  const uint32_t digit_mask = (1u << digit_bits) - 1u;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  const uint64_t base = uint64_t(blockIdx.x) * kSortTile;
  // the wavefront's items, all loads issued before the first is needed
  const uint64_t first = base + uint64_t(wave) * kSortWaveItems + lane;
  K rk[kSortItems];
  uint32_t rv[kSortItems], at[kSortItems];
#pragma unroll
  for (int r = 0; r < kSortItems; ++r) {
    const uint64_t i = first + uint64_t(r) * kWave;
    rk[r] = i < n ? keys[i] : K(0);
    rv[r] = i < n ? vals[i] : 0u;
  }
  {
    const uint64_t slot = uint64_t(threadIdx.x) * nb + blockIdx.x;
    const uint32_t c = hist[slot];
    const uint32_t g = offsets[slot] + (above ? above[slot / kScanTile] : 0u);
    uint32_t total;
    tile_off[threadIdx.x] = block_exclusive_scan(c, wave_sums, &total);
    global_off[threadIdx.x] = g;
  }
#pragma unroll
  for (int w = 0; w < kSortWaves; ++w) cnt[w][threadIdx.x] = 0;
  __syncthreads();
  const unsigned long long lt_mask = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
#pragma unroll
  for (int r = 0; r < kSortItems; ++r) {
    const bool valid = first + uint64_t(r) * kWave < n;
    const uint32_t d = valid ? uint32_t(rk[r] >> shift) & digit_mask : 0u;
    unsigned long long peers = __ballot(valid);
    for (int b = 0; b < digit_bits; ++b) {
      const bool bit = (d >> b) & 1u;
      const unsigned long long bal = __ballot(valid && bit);
      peers &= bit ? bal : ~bal;
    }
    const uint32_t before = cnt[wave][d], rank = __popcll(peers & lt_mask);
    at[r] = before + rank;
    wave_sync();   // (every lane has read the count)
    if (valid && rank == 0) cnt[wave][d] = before + uint32_t(__popcll(peers));
    wave_sync();
  }
  __syncthreads();
  {
    uint32_t running = tile_off[threadIdx.x];
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) {
      const uint32_t c = cnt[w][threadIdx.x];
      cnt[w][threadIdx.x] = running;
      running += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSortItems; ++r)
    if (first + uint64_t(r) * kWave < n) {
      at[r] += cnt[wave][uint32_t(rk[r] >> shift) & digit_mask];
      s_keys[at[r]] = rk[r];
    }
  __syncthreads();
  const uint32_t tile_n = uint32_t(min<uint64_t>(uint64_t(kSortTile), n - base));
  uint32_t to[kSortItems];
#pragma unroll
  for (int r = 0; r < kSortItems; ++r) {
    const uint32_t j = r * kSortThreads + threadIdx.x;
    if (j < tile_n) {
      const K key = s_keys[j];
      const uint32_t d = uint32_t(key >> shift) & digit_mask;
      to[r] = global_off[d] + (j - tile_off[d]);
      out_keys[to[r]] = key;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSortItems; ++r)
    if (first + uint64_t(r) * kWave < n) s_vals[at[r]] = rv[r];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSortItems; ++r) {
    const uint32_t j = r * kSortThreads + threadIdx.x;
    if (j < tile_n) out_vals[to[r]] = s_vals[j];
  }
}

template <typename T>
__global__ void k_fill(T* p, T value, uint64_t n) {
  for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += uint64_t(gridDim.x) * blockDim.x)
    p[i] = value;
}

template <typename T>
int fill_impl(T* p, T value, uint64_t n, hipStream_t st) {
  if (n == 0) return HM_OK;
  uint64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  k_fill<T><<<unsigned(blocks), 256, 0, st>>>(p, value, n);
  HM_HIP(hipGetLastError());
  return HM_OK;
}

template <typename T>
__global__ void k_copy(const T* __restrict__ src, T* __restrict__ dst, uint64_t n) {
  for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += uint64_t(gridDim.x) * blockDim.x)
    dst[i] = src[i];
}

}  // namespace

// ------------------------------------------------------------------ planned (workspace) variants
uint64_t scan_ws_words(uint64_t n) { return scan_ws_count(n); }

int scan_u32_ws(const uint32_t* in, uint32_t* out, uint64_t n, uint32_t* total_dev, uint32_t* ws, hipStream_t st) {
  if (n == 0) {
    if (total_dev) HM_TRY(fill_u32(total_dev, 0, 1, st));
    return HM_OK;
  }
  HM_TRY(scan_ws<uint32_t>(in, out, n, ws, st));
  if (total_dev) {
    k_scan_total<uint32_t><<<1, 1, 0, st>>>(in, out, n, total_dev);
    HM_HIP(hipGetLastError());
  }
  return HM_OK;
}

uint64_t radix_ws_words(uint64_t n) {
  const uint64_t nb = (n + kSortTile - 1) / kSortTile;
  return 2 * 256 * nb + scan_ws_words(256 * nb) + 16;
}

namespace {

template <typename K>
int radix_sort_impl(K* k0, uint32_t* v0, K* k1, uint32_t* v1, uint64_t n, int bits, uint32_t* ws, hipStream_t st) {
  if (n == 0) return HM_OK;
  const uint64_t nb64 = (n + kSortTile - 1) / kSortTile;
  if (nb64 > 0xFFFFFFull) {
    set_error("radix sort of %llu items is too large", (unsigned long long)n);
    return HM_EUNSUPPORTED;
  }
  const uint32_t nb = uint32_t(nb64);
  const uint64_t counters = uint64_t(256) * nb, tiles = (counters + kScanTile - 1) / kScanTile;
  uint32_t *hist = ws, *offs = ws + counters, *sums = ws + 2 * counters, *above = sums + tiles;
  K *src_k = k0, *dst_k = k1;
  uint32_t *src_v = v0, *dst_v = v1;
  for (int shift = 0; shift < bits; shift += 8) {
    const int db = (bits - shift) < 8 ? (bits - shift) : 8;
    k_sort_hist<K><<<nb, kSortThreads, 0, st>>>(src_k, n, shift, (1u << db) - 1u, hist, nb);
    // (the scan's last step, adding the sums before each tile, is the
    // scatter's)
    k_scan_tile<uint32_t><<<unsigned(tiles), kScanThreads, 0, st>>>(hist, offs, tiles > 1 ? sums : nullptr, counters);
    HM_HIP(hipGetLastError());
    if (tiles > 1) HM_TRY(scan_ws<uint32_t>(sums, above, tiles, above + tiles, st));
    k_sort_scatter<K><<<nb, kSortThreads, 0, st>>>(src_k, src_v, dst_k, dst_v, n, shift, db, hist, offs,
                                                   tiles > 1 ? above : nullptr, nb);
    HM_HIP(hipGetLastError());
    std::swap(src_k, dst_k);
    std::swap(src_v, dst_v);
  }
  return HM_OK;
}

}  // namespace

int radix_sort_ws(unsigned long long* k0, uint32_t* v0, unsigned long long* k1, uint32_t* v1, uint64_t n, int bits,
                  uint32_t* ws, hipStream_t st) {
  return radix_sort_impl(k0, v0, k1, v1, n, bits, ws, st);
}

int copy_u32(const uint32_t* src, uint32_t* dst, uint64_t n, hipStream_t st) {
  if (!n) return HM_OK;
  k_copy<uint32_t><<<unsigned(std::min<uint64_t>((n + 255) / 256, 16384)), 256, 0, st>>>(src, dst, n);
  HM_HIP(hipGetLastError());
  return HM_OK;
}

int copy_u64(const unsigned long long* src, unsigned long long* dst, uint64_t n, hipStream_t st) {
  if (!n) return HM_OK;
  k_copy<unsigned long long><<<unsigned(std::min<uint64_t>((n + 255) / 256, 16384)), 256, 0, st>>>(src, dst, n);
  HM_HIP(hipGetLastError());
  return HM_OK;
}

int scan_exclusive_u32(const uint32_t* in, uint32_t* out, uint64_t n, uint32_t* total_dev, hipStream_t st) {
  HM_TRY(scan_impl<uint32_t>(in, out, n, st));
  if (total_dev) {
    k_scan_total<uint32_t><<<1, 1, 0, st>>>(in, out, n, total_dev);
    HM_HIP(hipGetLastError());
  }
  return HM_OK;
}

int scan_exclusive_u64(const unsigned long long* in, unsigned long long* out, uint64_t n, hipStream_t st) {
  return scan_impl<unsigned long long>(in, out, n, st);
}

template <typename K>
int radix_sort_pairs(K*& keys, uint32_t*& vals, K*& keys_tmp, uint32_t*& vals_tmp, uint64_t n, int bits,
                     hipStream_t st) {
  Scratch tmp(st);
  uint32_t* ws = nullptr;
  HM_TRY(tmp.get(&ws, radix_ws_words(n)));
  HM_TRY(radix_sort_impl(keys, vals, keys_tmp, vals_tmp, n, bits, ws, st));
  if (radix_passes(bits) & 1) {
    std::swap(keys, keys_tmp);
    std::swap(vals, vals_tmp);
  }
  return HM_OK;
}
template int radix_sort_pairs(unsigned long long*&, uint32_t*&, unsigned long long*&, uint32_t*&, uint64_t, int,
                              hipStream_t);
template int radix_sort_pairs(uint32_t*&, uint32_t*&, uint32_t*&, uint32_t*&, uint64_t, int, hipStream_t);

int fill_u32(uint32_t* p, uint32_t value, uint64_t n, hipStream_t st) { return fill_impl<uint32_t>(p, value, n, st); }

int fill_u64(unsigned long long* p, unsigned long long value, uint64_t n, hipStream_t st) {
  return fill_impl<unsigned long long>(p, value, n, st);
}

}  // namespace hm
