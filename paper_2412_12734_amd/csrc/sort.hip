// Device-wide exclusive scan and stable LSD radix sort of (uint32 key, uint32 value) pairs.
//
// Scan: reduce per 4096-element tile -> scan of tile sums in one workgroup -> per-tile scan.
// Radix pass (a digit of at most 8 bits; a key of b bits takes ceil(b/8) passes with the bits
// spread evenly over them), three launches: per-tile digit histogram, which also adds each
// digit's count to the pass's digit totals -> one workgroup per digit turns its row of the
// digit-major [digit][tile] counts into output offsets (the totals of the smaller digits
// give the row's base) -> scatter. The totals are kept in kTotCopies copies (workgroup b adds
// to copy b mod kTotCopies): device-wide atomics on one address are served one at a time,
// about 55 ns each, so 2048 workgroups adding to a single copy took 35 us. With few tiles the
// scatter works out its offsets itself (two launches; 100k records, four passes 76 -> 58 us), with
// very few its counts too (one launch). The scatter ranks each element stably among equal digits
// of its tile: each wave takes a contiguous part of the tile in rounds of 64; lanes with
// the same digit are found with one ballot per digit bit and counted against the wave's
// running per-digit counters in LDS. Wave offsets and digit starts then place every element
// in LDS in digit order, and the tile is written out so that consecutive lanes store
// consecutive addresses of one digit run.
#include "device_util.h"
#include "gbb_internal.h"

namespace gbb {

namespace {

constexpr int kThreads = 256;
constexpr int kItems = kScanTile / kThreads;  // 16

// Inclusive scan of v over the threads of the block; returns the inclusive value and
// writes the block total to *total. `wave_tot` is LDS scratch of one entry per wave.
template <int THREADS = kThreads>
__device__ __forceinline__ uint32_t block_inclusive_scan(uint32_t v, uint32_t* wave_tot,
                                                         uint32_t* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    uint32_t t = __shfl_up(v, d, 64);
    if (lane >= d) v += t;
  }
  if (lane == 63) wave_tot[w] = v;
  __syncthreads();
  uint32_t add = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < THREADS / 64; ++i) {
    uint32_t t = wave_tot[i];
    if (i < w) add += t;
    tot += t;
  }
  __syncthreads();
  *total = tot;
  return v + add;
}

template <bool GATHER>
__device__ __forceinline__ uint32_t scan_load(const uint32_t* in, const uint32_t* gather,
                                              int64_t i) {
  if (GATHER) return in[gather[i]];
  return in[i];
}

__device__ __forceinline__ int64_t scan_len(int64_t n, const ScanLen& L) {
  if (!L.d_count) return n;
  const int64_t m = ((int64_t)*L.d_count + L.per - 1) / L.per * L.mult;
  return m < n ? m : n;
}

template <bool GATHER>
__global__ void __launch_bounds__(kThreads)
scan_reduce_kernel(const uint32_t* __restrict__ in, const uint32_t* __restrict__ gather,
                   int64_t n_cap, ScanLen L, uint32_t* __restrict__ gathered,
                   uint32_t* __restrict__ partials,
                   unsigned long long* __restrict__ partials64) {
  __shared__ uint32_t wave_tot[4];
  __shared__ unsigned long long wave_tot64[4];
  const int64_t n = scan_len(n_cap, L);
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  if (base >= n && base > 0) return;
  uint32_t s = 0;
  unsigned long long s64 = 0;
#pragma unroll 4
  for (int k = 0; k < kItems; ++k) {
    int64_t i = base + k * kThreads + threadIdx.x;
    if (i < n) {
      const uint32_t x = scan_load<GATHER>(in, gather, i);
      if (GATHER) gathered[i] = x;
      s += x;
      s64 += x;
    }
  }
  if (partials64) {
    // exact block sum in 64 bits (the partials kernel adds the blocks up)
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) s64 += __shfl_xor(s64, d, 64);
    if ((threadIdx.x & 63) == 0) wave_tot64[threadIdx.x >> 6] = s64;
  }
  uint32_t total;
  block_inclusive_scan(s, wave_tot, &total);  // its barriers also publish wave_tot64
  if (threadIdx.x == 0) {
    partials[blockIdx.x] = total;
    if (partials64)
      partials64[blockIdx.x] = (wave_tot64[0] + wave_tot64[1]) + (wave_tot64[2] + wave_tot64[3]);
  }
}

// One workgroup: exclusive scan of partials[0..nb) in place, total to partials[nb] and *total.
__global__ void __launch_bounds__(1024)
scan_partials_kernel(uint32_t* __restrict__ partials, int64_t n_cap, ScanLen L,
                     uint32_t* __restrict__ total,
                     const unsigned long long* __restrict__ partials64,
                     unsigned long long* __restrict__ total64) {
  __shared__ uint32_t wave_tot[16];
  __shared__ uint32_t carry_s;
  __shared__ unsigned long long wave_sum64[16];
  const int64_t n = scan_len(n_cap, L);
  const int64_t nb = n > 0 ? (n + kScanTile - 1) / kScanTile : 1;
  if (total64) {
    unsigned long long s64 = 0;
    for (int64_t i = threadIdx.x; i < nb; i += 1024) s64 += partials64[i];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) s64 += __shfl_xor(s64, d, 64);
    if ((threadIdx.x & 63) == 0) wave_sum64[threadIdx.x >> 6] = s64;
    __syncthreads();
    if (threadIdx.x == 0) {
      unsigned long long t = 0;
      for (int k = 0; k < 16; ++k) t += wave_sum64[k];
      *total64 = t;
    }
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (threadIdx.x == 0) carry_s = 0;
  __syncthreads();
  for (int64_t start = 0; start < nb; start += 1024) {
    int64_t i = start + threadIdx.x;
    uint32_t x = i < nb ? partials[i] : 0u;
    uint32_t v = x;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      uint32_t t = __shfl_up(v, d, 64);
      if (lane >= d) v += t;
    }
    if (lane == 63) wave_tot[w] = v;
    __syncthreads();
    uint32_t add = 0, tot = 0;
    for (int k = 0; k < 16; ++k) {
      uint32_t t = wave_tot[k];
      if (k < w) add += t;
      tot += t;
    }
    const uint32_t carry = carry_s;
    if (i < nb) partials[i] = carry + add + v - x;
    __syncthreads();
    if (threadIdx.x == 0) carry_s = carry + tot;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    partials[nb] = carry_s;
    if (total) *total = carry_s;
  }
}

// LDS index with one pad word per 32 so that both the striped and the blocked access
// patterns below are free of bank conflicts.
__device__ __forceinline__ int pad_idx(int i) { return i + (i >> 5); }

// With chunk_owner, element i with value x > 0 and exclusive prefix o also records itself as
// the owner of every chunk of kChunkSlots slots that starts inside [o, o + x) (chunk indices
// below n_chunks).
// `in` may be `out`: a workgroup has read its elements before it writes them.
__global__ void __launch_bounds__(kThreads)
scan_down_kernel(const uint32_t* in, int64_t n_cap, ScanLen L,
                 const uint32_t* __restrict__ partials, uint32_t* out,
                 uint32_t* __restrict__ chunk_owner, int64_t n_chunks) {
  __shared__ uint32_t tile[kScanTile + kScanTile / 32];
  __shared__ uint32_t wave_tot[4];
  const int64_t n = scan_len(n_cap, L);
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  if (base >= n) return;
  // coalesced load into LDS, then each thread owns 16 consecutive elements
#pragma unroll 4
  for (int k = 0; k < kItems; ++k) {
    int64_t i = base + k * kThreads + threadIdx.x;
    tile[pad_idx(k * kThreads + threadIdx.x)] = i < n ? in[i] : 0u;
  }
  __syncthreads();
  uint32_t loc[kItems];
  uint32_t s = 0;
#pragma unroll
  for (int k = 0; k < kItems; ++k) loc[k] = tile[pad_idx(threadIdx.x * kItems + k)];
#pragma unroll
  for (int k = 0; k < kItems; ++k) s += loc[k];
  uint32_t total;
  uint32_t incl = block_inclusive_scan(s, wave_tot, &total);
  uint32_t run = partials[blockIdx.x] + incl - s;
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    uint32_t x = loc[k];
    loc[k] = run;
    if (chunk_owner && x > 0) {
      const int64_t i = base + threadIdx.x * kItems + k;
      const uint64_t o = run, e = (uint64_t)run + x;
      for (uint64_t c = (o + kChunkSlots - 1) / kChunkSlots;
           c * kChunkSlots < e && (int64_t)c < n_chunks; ++c)
        chunk_owner[c] = (uint32_t)i;
    }
    run += x;
  }
#pragma unroll
  for (int k = 0; k < kItems; ++k) tile[pad_idx(threadIdx.x * kItems + k)] = loc[k];
  __syncthreads();
#pragma unroll 4
  for (int k = 0; k < kItems; ++k) {
    int64_t i = base + k * kThreads + threadIdx.x;
    if (i < n) out[i] = tile[pad_idx(k * kThreads + threadIdx.x)];
  }
}

// ---- radix sort --------------------------------------------------------------------------
// A pass works on tiles of kRadixTile elements; the tile count follows the device-side
// element count, and workgroups take tiles in turn (at most kRadixGrid workgroups), so a
// short sort in a large buffer costs what its elements cost. Digit counts are stored
// digit-major, one column per tile.
constexpr int kRadixGrid = 2048;

__device__ __forceinline__ int64_t sort_count(const uint32_t* d_n, int64_t n_cap) {
  if (!d_n) return n_cap;
  int64_t n = (int64_t)(*d_n);
  return n < n_cap ? n : n_cap;
}

// Digit counts of one tile. Each wave counts into its own LDS histogram with plain LDS
// atomics (lanes that hit one bin are served one after another by the LDS, which is cheaper
// than grouping equal digits with ballots); each lane loads four consecutive keys at a time.
template <int NBITS>
__global__ void __launch_bounds__(kRadixThreads)
radix_hist_kernel(const uint32_t* __restrict__ keys, const uint32_t* __restrict__ d_n,
                  int64_t n_cap, int shift, uint32_t* __restrict__ hist,
                  uint32_t* __restrict__ digit_tot) {
  constexpr int kBins = 1 << NBITS;
  constexpr uint32_t kMask = (uint32_t)kBins - 1u;
  constexpr int kWaves = kRadixThreads / 64;
  __shared__ uint32_t h[kWaves][kBins];
  const int64_t n = sort_count(d_n, n_cap);
  const int64_t nb = (n + kRadixTile - 1) / kRadixTile;
  const int w = threadIdx.x >> 6;
  static_assert(kBins <= kRadixThreads, "one digit per thread");
  uint32_t acc = 0;  // this thread's digit, summed over the workgroup's tiles
  for (int64_t tile = blockIdx.x; tile < nb; tile += gridDim.x) {
    for (int i = threadIdx.x; i < kWaves * kBins; i += kRadixThreads) (&h[0][0])[i] = 0;
    __syncthreads();
    const int64_t base = tile * kRadixTile;
    {
      const int nvalid = (int)((n - base) < kRadixTile ? (n - base) : kRadixTile);
      const uint32_t* kt = keys + base;
      uint4 q[kRadixItems / 4];
#pragma unroll
      for (int k = 0; k < kRadixItems / 4; ++k) {
        const int i = 4 * (k * kRadixThreads + threadIdx.x);
        if (i + 3 < nvalid) {
          q[k] = *reinterpret_cast<const uint4*>(kt + i);
        } else {
          q[k].x = i < nvalid ? kt[i] : 0u;
          q[k].y = i + 1 < nvalid ? kt[i + 1] : 0u;
          q[k].z = i + 2 < nvalid ? kt[i + 2] : 0u;
          q[k].w = 0u;
        }
      }
#pragma unroll
      for (int k = 0; k < kRadixItems / 4; ++k) {
        const int i = 4 * (k * kRadixThreads + threadIdx.x);
        if (i < nvalid) atomicAdd(&h[w][(q[k].x >> shift) & kMask], 1u);
        if (i + 1 < nvalid) atomicAdd(&h[w][(q[k].y >> shift) & kMask], 1u);
        if (i + 2 < nvalid) atomicAdd(&h[w][(q[k].z >> shift) & kMask], 1u);
        if (i + 3 < nvalid) atomicAdd(&h[w][(q[k].w >> shift) & kMask], 1u);
      }
    }
    __syncthreads();
    const int d = threadIdx.x;
    if (d < kBins) {
      uint32_t c = 0;
#pragma unroll
      for (int ww = 0; ww < kWaves; ++ww) c += h[ww][d];
      hist[(int64_t)d * nb + tile] = c;
      acc += c;
    }
    __syncthreads();  // the next tile reuses the LDS histograms
  }
  if (digit_tot && threadIdx.x < kBins && acc != 0)
    atomicAdd(&digit_tot[(blockIdx.x % kTotCopies) * 256 + threadIdx.x], acc);
}

// Output offsets of one digit (the workgroup's): its row of the [digit][tile] counts becomes
// the exclusive prefix over tiles plus the number of elements with a smaller digit. Each
// thread takes kItems consecutive entries of a chunk.
template <int NBITS>
__global__ void __launch_bounds__(kThreads)
radix_offsets_kernel(const uint32_t* __restrict__ d_n, int64_t n_cap,
                     const uint32_t* __restrict__ digit_tot, uint32_t* __restrict__ hist) {
  static_assert((1 << NBITS) <= kThreads, "one smaller digit per thread");
  __shared__ uint32_t wave_tot[kThreads / 64];
  const int64_t n = sort_count(d_n, n_cap);
  const int64_t nb = (n + kRadixTile - 1) / kRadixTile;
  const int d = blockIdx.x, tid = threadIdx.x;
  uint32_t smaller = 0;  // elements whose digit is tid (< d)
  if (tid < d) {
#pragma unroll 16
    for (int c = 0; c < kTotCopies; ++c) smaller += digit_tot[c * 256 + tid];
  }
  uint32_t base;
  block_inclusive_scan(smaller, wave_tot, &base);
  uint32_t* __restrict__ row = hist + (int64_t)d * nb;
  for (int64_t c0 = 0; c0 < nb; c0 += (int64_t)kThreads * kItems) {
    const int64_t i0 = c0 + (int64_t)tid * kItems;
    uint32_t v[kItems], sum = 0;
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      v[k] = i0 + k < nb ? row[i0 + k] : 0u;
      sum += v[k];
    }
    uint32_t tot;
    uint32_t run = base + block_inclusive_scan(sum, wave_tot, &tot) - sum;
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      if (i0 + k < nb) row[i0 + k] = run;
      run += v[k];
    }
    base += tot;
  }
}

// Threads of a scatter workgroup: eight elements each (with 16 a thread took 160 registers and a
// SIMD held three waves); the reordered tile passes through LDS twice, keys and then values, which
// halves what a workgroup takes of it. Bound by the writes, runs of a digit 64 bytes long on average
// with 8-bit digits. Mean of a pass, with the XCD order below: 16M records and 60M and 19M pairs 160
// -> 126 us (2.8 -> 3.5 TB/s); 1M records 11.6 -> 10.5, 8.4M pairs 21.3 -> 19.1.
constexpr int kScatterThreads = 512;
constexpr int kScatterItems = kRadixTile / kScatterThreads;

// Places one tile's elements (from `base`, up to n): gstart is the output index of the tile's first
// element of digit threadIdx.x (threads below the number of digits). All threads take part.
template <int NBITS>
__device__ __forceinline__ void scatter_tile(const uint32_t* __restrict__ keys_in,
                                             const uint32_t* __restrict__ vals_in,
                                             uint32_t* __restrict__ keys_out,
                                             uint32_t* __restrict__ vals_out, int64_t n,
                                             int64_t base, int shift, uint32_t gstart) {
  constexpr int kBins = 1 << NBITS;
  constexpr uint32_t kMask = (uint32_t)kBins - 1u;
  constexpr int kWaves = kScatterThreads / 64;
  constexpr int kPerWave = kRadixTile / kWaves;  // contiguous elements ranked by one wave
  __shared__ uint32_t s_buf[kRadixTile];  // the tile's keys in digit order, then its values
  __shared__ uint32_t s_cnt[kWaves][kBins];  // running per-wave digit counts, then wave offsets
  __shared__ uint32_t s_gofs[kBins];  // output index of the tile's element 0 of each digit
  __shared__ uint32_t wave_tot[kWaves];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int nvalid = (int)((n - base) < kRadixTile ? (n - base) : kRadixTile);
  keys_in += base;
  vals_in += base;
#pragma unroll
  for (int k = 0; k < kBins; k += 64)
    if (k + lane < kBins) s_cnt[w][k + lane] = 0;
  __builtin_amdgcn_wave_barrier();
  // Each wave ranks its own contiguous part of the tile in rounds of 64 elements; program
  // order inside the wave keeps equal digits in index order.
  uint32_t key_r[kScatterItems], val_r[kScatterItems], place[kScatterItems];
  // all loads first (memory-level parallelism)
#pragma unroll
  for (int r = 0; r < kScatterItems; ++r) {
    const int i = w * kPerWave + r * 64 + lane;
    const bool valid = i < nvalid;
    key_r[r] = valid ? keys_in[i] : 0u;
    val_r[r] = valid ? vals_in[i] : 0u;
  }
#pragma unroll
  for (int r = 0; r < kScatterItems; ++r) {
    const int i = w * kPerWave + r * 64 + lane;
    const bool valid = i < nvalid;
    const uint32_t d = (key_r[r] >> shift) & kMask;
    // lanes holding the same digit: one ballot per digit bit
    uint64_t m = ballot(valid);
#pragma unroll
    for (int bit = 0; bit < NBITS; ++bit) {
      const bool set = (d >> bit) & 1u;
      const uint64_t b = ballot(set);
      m &= set ? b : ~b;
    }
    const uint32_t below = mbcnt(m);
    const uint32_t cnt = s_cnt[w][d];
    __builtin_amdgcn_wave_barrier();
    if (valid && below == 0) s_cnt[w][d] = cnt + popc64(m);
    __builtin_amdgcn_wave_barrier();
    place[r] = cnt + below;
  }
  __syncthreads();
  // digit totals of the tile, digit starts, and from both where each wave's part of a digit starts
  uint32_t c[kWaves], tot = 0;
  if (tid < kBins) {
#pragma unroll
    for (int ww = 0; ww < kWaves; ++ww) c[ww] = s_cnt[ww][tid];
#pragma unroll
    for (int ww = 0; ww < kWaves; ++ww) tot += c[ww];
  }
  uint32_t total;
  uint32_t start = block_inclusive_scan<kScatterThreads>(tot, wave_tot, &total) - tot;
  if (tid < kBins) {
    s_gofs[tid] = gstart - start;  // element counts fit in 32 bits, so output indices do too
#pragma unroll
    for (int ww = 0; ww < kWaves; ++ww) {
      s_cnt[ww][tid] = start;
      start += c[ww];
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kScatterItems; ++r) {
    const int i = w * kPerWave + r * 64 + lane;
    place[r] += s_cnt[w][(key_r[r] >> shift) & kMask];
    if (i < nvalid) s_buf[place[r]] = key_r[r];
  }
  __syncthreads();
  uint32_t gpos[kScatterItems];
#pragma unroll
  for (int r = 0; r < kScatterItems; ++r) {
    const int i = r * kScatterThreads + tid;
    if (i < nvalid) {
      const uint32_t key = s_buf[i];
      gpos[r] = s_gofs[(key >> shift) & kMask] + (uint32_t)i;
      keys_out[gpos[r]] = key;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kScatterItems; ++r) {
    const int i = w * kPerWave + r * 64 + lane;
    if (i < nvalid) s_buf[place[r]] = val_r[r];
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kScatterItems; ++r) {
    const int i = r * kScatterThreads + tid;
    if (i < nvalid) vals_out[gpos[r]] = s_buf[i];
  }
  __syncthreads();  // the next tile reuses the LDS
}

// OWN: the workgroup works out its output offsets itself from the tiles' raw counts (few tiles, see
// kOwnOffsetTiles) where otherwise radix_offsets_kernel has left them in `hist`.
template <int NBITS, bool OWN>
__global__ void __launch_bounds__(kScatterThreads)
radix_scatter_kernel(const uint32_t* __restrict__ keys_in, const uint32_t* __restrict__ vals_in,
                     uint32_t* __restrict__ keys_out, uint32_t* __restrict__ vals_out,
                     const uint32_t* __restrict__ d_n, int64_t n_cap, int shift,
                     const uint32_t* __restrict__ hist, uint32_t* __restrict__ digit_tot) {
  const int64_t n = sort_count(d_n, n_cap);
  const int64_t nb = (n + kRadixTile - 1) / kRadixTile;
  const int tid = threadIdx.x;
  if constexpr (OWN) {
    // one tile per workgroup: this thread's digit, over all tiles and over those before
    __shared__ uint32_t own_tot[kScatterThreads / 64];
    const int64_t tile = blockIdx.x;
    if (tile >= nb) return;
    uint32_t all = 0, before = 0;
    if (tid < (1 << NBITS)) {
      const uint32_t* __restrict__ row = hist + (int64_t)tid * nb;
#pragma unroll 8
      for (int64_t t = 0; t < nb; ++t) {
        const uint32_t c = row[t];
        all += c;
        before += t < tile ? c : 0u;
      }
    }
    uint32_t total;
    const uint32_t first = block_inclusive_scan<kScatterThreads>(all, own_tot, &total) - all;
    scatter_tile<NBITS>(keys_in, vals_in, keys_out, vals_out, n, tile * kRadixTile, shift,
                        first + before);
    return;
  }
  // the offsets launch has read this pass's digit totals: leave them zero for the next sort
  for (int c = blockIdx.x; c < kTotCopies; c += gridDim.x)
    if (tid < 256) digit_tot[c * 256 + tid] = 0u;
  // Workgroups go to the eight XCDs in turn: each XCD takes a contiguous eighth of the tiles, so
  // that neighbouring tiles, whose runs of a digit follow one another in the output, meet in one L2
  // and fill its lines together.
  const int64_t per_xcd = (nb + 7) / 8;
  for (int64_t v = blockIdx.x; v < 8 * per_xcd; v += gridDim.x) {
    const int64_t tile = (v & 7) * per_xcd + (v >> 3);
    if (tile >= nb) continue;
    // where each digit of this tile starts in the output (loaded early, used at the end)
    const uint32_t gstart = tid < (1 << NBITS) ? hist[(int64_t)tid * nb + tile] : 0u;
    scatter_tile<NBITS>(keys_in, vals_in, keys_out, vals_out, n, tile * kRadixTile, shift, gstart);
  }
}

// One pass of a short sort (at most kDirectTiles radix tiles) in one launch: instead of a histogram
// launch and an offsets launch, every workgroup counts the digits of all elements itself, those of
// the tiles before its own apart from the rest. With `ranges` (a sort of one pass: a digit is a
// tile of the image) the first workgroup also writes each digit's run as [first, end). Bound by
// launches, which each cost 4 to 5 us whatever they do: 5000 pairs in 64 tiles of an image, sort
// and ranges 28 -> 9 us.
template <int NBITS>
__global__ void __launch_bounds__(kScatterThreads)
radix_direct_kernel(const uint32_t* __restrict__ keys_in, const uint32_t* __restrict__ vals_in,
                    uint32_t* __restrict__ keys_out, uint32_t* __restrict__ vals_out,
                    const uint32_t* __restrict__ d_n, int64_t n_cap, int shift,
                    uint32_t* __restrict__ ranges) {
  constexpr int kBins = 1 << NBITS;
  constexpr uint32_t kMask = (uint32_t)kBins - 1u;
  __shared__ uint32_t s_before[kBins], s_after[kBins];
  __shared__ uint32_t own_tot[kScatterThreads / 64];
  const int n = (int)sort_count(d_n, n_cap);
  const int tid = threadIdx.x;
  const int base = (int)blockIdx.x * kRadixTile;
  if (base >= n) return;
  if (tid < kBins) s_before[tid] = s_after[tid] = 0u;
  __syncthreads();
#pragma unroll 4
  for (int i = tid; i < n; i += kScatterThreads)
    atomicAdd(&(i < base ? s_before : s_after)[(keys_in[i] >> shift) & kMask], 1u);
  __syncthreads();
  const uint32_t before = tid < kBins ? s_before[tid] : 0u;
  const uint32_t all = tid < kBins ? before + s_after[tid] : 0u;
  uint32_t total;
  const uint32_t first = block_inclusive_scan<kScatterThreads>(all, own_tot, &total) - all;
  if (ranges && blockIdx.x == 0 && all != 0u) {
    ranges[2 * tid] = first;
    ranges[2 * tid + 1] = first + all;
  }
  scatter_tile<NBITS>(keys_in, vals_in, keys_out, vals_out, n, base, shift, first + before);
}

// Depth order of few records in one launch: the rank of a record is the number of records with a
// smaller key, or an equal one and a smaller index. A workgroup ranks 64 records, one per lane;
// its 16 waves count over every 16th chunk of 64 keys each, read through the scalar cache (two
// vector instructions per key and wave). The work grows with n^2, the launches of a radix sort
// (12, 70 us) do not shrink with n.
constexpr int kRankThreads = 1024;

__global__ void __launch_bounds__(kRankThreads)
rank_order_kernel(const uint32_t* __restrict__ keys, int n, uint32_t* __restrict__ order) {
  __shared__ uint32_t s_rank[64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int own = (int)blockIdx.x, i = own * 64 + lane;
  const uint32_t key = i < n ? keys[i] : 0xffffffffu;
  if (tid < 64) s_rank[tid] = 0u;
  __syncthreads();
  uint32_t below = 0;
  const int chunks = (n + 63) / 64;
  for (int c = w; c < chunks; c += kRankThreads / 64) {
    const uint32_t* __restrict__ k = keys + c * 64;
    const int m = n - c * 64 < 64 ? n - c * 64 : 64;
    if (c == own) {
      for (int j = 0; j < m; ++j) below += (k[j] < key || (k[j] == key && j < lane)) ? 1u : 0u;
    } else if (c < own) {
#pragma unroll
      for (int j = 0; j < 64; ++j) below += k[j] <= key ? 1u : 0u;
    } else if (m == 64) {
#pragma unroll
      for (int j = 0; j < 64; ++j) below += k[j] < key ? 1u : 0u;
    } else {
      for (int j = 0; j < m; ++j) below += k[j] < key ? 1u : 0u;
    }
  }
  atomicAdd(&s_rank[lane], below);
  __syncthreads();
  if (tid < 64 && i < n) order[s_rank[tid]] = (uint32_t)i;
}

__global__ void fill_u32_kernel(uint32_t* __restrict__ p, uint32_t value, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = value;
}

// The same fill for a 16-byte aligned array: 16-byte stores for the n / 4 full quads, then the
// n % 4 trailing words.
__global__ void fill_u32x4_kernel(uint32_t* __restrict__ p, uint32_t value, int64_t n) {
  const int64_t n4 = n >> 2;
  const uint4 v = make_uint4(value, value, value, value);
  uint4* __restrict__ q = reinterpret_cast<uint4*>(p);
  const int64_t first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int64_t i = first; i < n4; i += (int64_t)gridDim.x * blockDim.x) q[i] = v;
  if (first < (n & 3)) p[4 * n4 + first] = value;
}

unsigned grid_for(int64_t n, int threads) {
  int64_t b = (n + threads - 1) / threads;
  if (b > 65536) b = 65536;
  if (b < 1) b = 1;
  return (unsigned)b;
}

}  // namespace

hipError_t launch_fill_u32(uint32_t* p, uint32_t value, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if ((reinterpret_cast<uintptr_t>(p) & 15) == 0 && n >= 64) {
    hipLaunchKernelGGL(fill_u32x4_kernel, dim3(grid_for((n + 3) / 4, 256)), dim3(256), 0, s, p,
                       value, n);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(fill_u32_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, p, value, n);
  return hipGetLastError();
}

hipError_t launch_scan_u32(const uint32_t* in, const uint32_t* gather, uint32_t* out, int64_t n,
                           uint32_t* partials, uint32_t* total, unsigned long long* total64,
                           unsigned long long* partials64, hipStream_t s,
                           uint32_t* chunk_owner, int64_t n_chunks, ScanLen len) {
  const int64_t nb = (n + kScanTile - 1) / kScanTile;
  if (nb == 0) return hipSuccess;
  if (!total64) partials64 = nullptr;
  if (total64 && !partials64) return hipErrorInvalidValue;
  // gathered values are kept in `out` by the first pass: the second then reads them in order (a
  // second gather took as long as the first; 16M records: 493 -> 300 us)
  if (gather)
    hipLaunchKernelGGL(scan_reduce_kernel<true>, dim3((unsigned)nb), dim3(kThreads), 0, s, in,
                       gather, n, len, out, partials, partials64);
  else
    hipLaunchKernelGGL(scan_reduce_kernel<false>, dim3((unsigned)nb), dim3(kThreads), 0, s, in,
                       gather, n, len, nullptr, partials, partials64);
  hipLaunchKernelGGL(scan_partials_kernel, dim3(1), dim3(1024), 0, s, partials, n, len, total,
                     partials64, total64);
  hipLaunchKernelGGL(scan_down_kernel, dim3((unsigned)nb), dim3(kThreads), 0, s,
                     gather ? out : in, n, len, partials, out, chunk_owner, n_chunks);
  return hipGetLastError();
}

// Radix tiles of a sort whose passes are one launch each: a workgroup reads every key, which costs
// about 1 us per tile and pass, against 4 to 5 for each of the two launches saved.
constexpr int64_t kDirectTiles = 4;

// Radix tiles up to which a pass leaves out the offsets launch: every workgroup then reads all
// tiles' counts, 1 KB per tile.
constexpr int64_t kOwnOffsetTiles = 128;

template <int NBITS>
hipError_t radix_pass(const uint32_t* ki, const uint32_t* vi, uint32_t* ko, uint32_t* vo,
                      const uint32_t* d_n, int64_t n_cap, int shift, int64_t nb, uint32_t* hist,
                      uint32_t* digit_tot, uint32_t* ranges, hipStream_t s) {
  if (nb <= kDirectTiles) {
    hipLaunchKernelGGL(radix_direct_kernel<NBITS>, dim3((unsigned)nb), dim3(kScatterThreads), 0,
                       s, ki, vi, ko, vo, d_n, n_cap, shift, ranges);
    return hipGetLastError();
  }
  const unsigned grid = (unsigned)(nb < kRadixGrid ? nb : kRadixGrid);
  const unsigned grid8 = (grid + 7) / 8 * 8;  // whole rounds over the XCDs
  if (nb <= kOwnOffsetTiles) {
    hipLaunchKernelGGL(radix_hist_kernel<NBITS>, dim3(grid), dim3(kRadixThreads), 0, s, ki, d_n,
                       n_cap, shift, hist, nullptr);
    hipLaunchKernelGGL((radix_scatter_kernel<NBITS, true>), dim3(grid), dim3(kScatterThreads), 0, s,
                       ki, vi, ko, vo, d_n, n_cap, shift, hist, nullptr);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(radix_hist_kernel<NBITS>, dim3(grid), dim3(kRadixThreads), 0, s, ki, d_n,
                     n_cap, shift, hist, digit_tot);
  hipLaunchKernelGGL(radix_offsets_kernel<NBITS>, dim3(1u << NBITS), dim3(kThreads), 0, s, d_n,
                     n_cap, digit_tot, hist);
  hipLaunchKernelGGL((radix_scatter_kernel<NBITS, false>), dim3(grid8), dim3(kScatterThreads), 0, s, ki, vi,
                     ko, vo, d_n, n_cap, shift, hist, digit_tot);
  return hipGetLastError();
}

// The fewest 8-bit-or-narrower passes (the key bits are spread evenly over them).
int radix_passes(int bits) { return (bits + 7) / 8; }

hipError_t launch_radix_sort(uint32_t* keys, uint32_t* vals, uint32_t* keys_alt,
                             uint32_t* vals_alt, const uint32_t* d_n, int64_t n_cap, int bits,
                             uint32_t* hist, uint32_t* digit_tot, uint32_t* ranges,
                             bool* ranges_written, hipStream_t s) {
  const int64_t nb = (n_cap + kRadixTile - 1) / kRadixTile;
  if (ranges_written) *ranges_written = false;
  if (nb == 0 || bits <= 0) return hipSuccess;
  if (bits > 32) return hipErrorInvalidValue;
  const int passes = radix_passes(bits);
  if (passes != 1 || nb > kDirectTiles) ranges = nullptr;
  if (ranges_written) *ranges_written = ranges != nullptr;
  hipError_t e = hipSuccess;
  uint32_t *ki = keys, *vi = vals, *ko = keys_alt, *vo = vals_alt;
  if (passes & 1) {  // the input is in the alternate arrays
    ki = keys_alt;
    vi = vals_alt;
    ko = keys;
    vo = vals;
  }
  int shift = 0;
  for (int p = 0; p < passes; ++p) {
    const int nbits = bits / passes + (p < bits % passes ? 1 : 0);
    uint32_t* const tot = digit_tot + (int64_t)kTotCopies * 256 * p;
#define GBB_PASS(B) \
  e = radix_pass<B>(ki, vi, ko, vo, d_n, n_cap, shift, nb, hist, tot, ranges, s)
    switch (nbits) {
      case 1: GBB_PASS(1); break;
      case 2: GBB_PASS(2); break;
      case 3: GBB_PASS(3); break;
      case 4: GBB_PASS(4); break;
      case 5: GBB_PASS(5); break;
      case 6: GBB_PASS(6); break;
      case 7: GBB_PASS(7); break;
      default: GBB_PASS(8); break;
    }
#undef GBB_PASS
    if (e != hipSuccess) return e;
    shift += nbits;
    uint32_t* t = ki;
    ki = ko;
    ko = t;
    t = vi;
    vi = vo;
    vo = t;
  }
  return hipGetLastError();
}

hipError_t launch_rank_order(const uint32_t* keys, int64_t n, uint32_t* order, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (n > kRankMax) return hipErrorInvalidValue;
  hipLaunchKernelGGL(rank_order_kernel, dim3((unsigned)((n + 63) / 64)), dim3(kRankThreads), 0, s,
                     keys, (int)n, order);
  return hipGetLastError();
}

}  // namespace gbb
