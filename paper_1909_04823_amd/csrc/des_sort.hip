// Device-wide exclusive scan and stable LSD radix sort for gfx950 (wave64).
//
// Both are plain multi-kernel primitives without inter-workgroup waiting: every kernel's
// workgroups are independent, so every wave reaches its exit whatever the dispatch order.
#include <type_traits>
#include "des_internal.h"

namespace des {

namespace {

constexpr int kScanItems = 8;                       // items per thread in the scan kernels
constexpr int kScanTile = kBlock * kScanItems;
constexpr int kSortItems = 16;                      // items per thread in the sort kernels
constexpr int kSortTile = kBlock * kSortItems;
constexpr int kFewSortItems = 4;                    // ... of a batch of up to kFewSort items
constexpr int kFewSortTile = kBlock * kFewSortItems;
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kMaxDigitBits = 9;                    // widest radix digit of one pass
constexpr int kMaxRadix = 1 << kMaxDigitBits;
constexpr int kFewItemsBits = 6;                    // widest digit for fewer than kSortTotals items, whose callers have 256 bytes of `totals`
static_assert(kMaxRadix <= kSortTotals && (1 << kFewItemsBits) * 4 <= 256, "the totals of a digit fit");

template <typename T>
__device__ inline T wave_inclusive_scan(T v) {
  const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    T o = __shfl_up(v, off, kWave);
    if (lane >= off) v += o;
  }
  return v;
}

// Exclusive prefix of v over the workgroup (thread order); total = sum over the workgroup.
template <typename T>
__device__ inline T block_exclusive_scan(T v, T *lds /*[kWavesPerBlock]*/, T &total) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  T inc = wave_inclusive_scan(v);
  if (lane == kWave - 1) lds[wave] = inc;
  __syncthreads();
  T base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kWavesPerBlock; ++w) {
    T x = lds[w];
    if (w < wave) base += x;
    tot += x;
  }
  __syncthreads();
  total = tot;
  return base + inc - v;
}

// The thread's kScanItems consecutive values in 16-byte accesses when they all exist (the arrays scanned here are
// the library's own, 256-byte aligned); values past n read as zero.
template <typename T>
__device__ inline void load_items(const T *__restrict__ data, int64_t base, int64_t n, T (&item)[kScanItems]) {
  constexpr int kPer = 16 / sizeof(T);
  static_assert(kScanItems % kPer == 0, "whole 16-byte accesses");
  if (base + kScanItems <= n) {
#pragma unroll
    for (int q = 0; q < kScanItems / kPer; ++q) {
      const uint4 raw = *reinterpret_cast<const uint4 *>(data + base + q * kPer);
      const T *t = reinterpret_cast<const T *>(&raw);
#pragma unroll
      for (int j = 0; j < kPer; ++j) item[q * kPer + j] = t[j];
    }
  } else {
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) item[i] = base + i < n ? data[base + i] : (T)0;
  }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_scan_reduce(const T *__restrict__ data, int64_t n, T *__restrict__ sums) {
  __shared__ T lds[kWavesPerBlock];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  T v = 0;
  T item[kScanItems];
  load_items(data, base, n, item);
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) v += item[i];
  T total;
  block_exclusive_scan(v, lds, total);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// One workgroup scans the per-tile sums in place (exclusive) and stores the grand total.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_scan_sums(T *__restrict__ sums, int64_t nb, T *__restrict__ total_out) {
  __shared__ T lds[kWavesPerBlock];
  T carry = 0;
  for (int64_t base = 0; base < nb; base += kBlock) {
    const int64_t i = base + threadIdx.x;
    T v = i < nb ? sums[i] : (T)0;
    T total;
    T ex = block_exclusive_scan(v, lds, total);
    if (i < nb) sums[i] = carry + ex;
    carry += total;
  }
  if (threadIdx.x == 0 && total_out) *total_out = carry;
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_scan_apply(T *__restrict__ data, int64_t n, const T *__restrict__ sums) {
  __shared__ T lds[kWavesPerBlock];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  T item[kScanItems];
  T v = 0;
  load_items(data, base, n, item);
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) v += item[i];
  T total;
  T run = sums[blockIdx.x] + block_exclusive_scan(v, lds, total);
  if (base + kScanItems <= n) {
    constexpr int kPer = 16 / sizeof(T);
#pragma unroll
    for (int q = 0; q < kScanItems / kPer; ++q) {
      uint4 raw;
      T *t = reinterpret_cast<T *>(&raw);
#pragma unroll
      for (int j = 0; j < kPer; ++j) { t[j] = run; run += item[q * kPer + j]; }
      *reinterpret_cast<uint4 *>(data + base + q * kPer) = raw;
    }
  } else {
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
      if (base + i < n) data[base + i] = run;
      run += item[i];
    }
  }
}

template <typename T>
void exclusive_scan(T *data, int64_t n, T *total_out, void *scratch, hipStream_t s) {
  if (n <= 0) return;
  const int64_t nb = (n + kScanTile - 1) / kScanTile;
  T *sums = (T *)scratch;
  hipLaunchKernelGGL(k_scan_reduce<T>, dim3((unsigned)nb), dim3(kBlock), 0, s, data, n, sums);
  hipLaunchKernelGGL(k_scan_sums<T>, dim3(1), dim3(kBlock), 0, s, sums, nb, total_out);
  hipLaunchKernelGGL(k_scan_apply<T>, dim3((unsigned)nb), dim3(kBlock), 0, s, data, n, sums);
}

// ---------------------------------------------------------------------------------------
// Radix sort.  One workgroup owns a tile of kBlock * kItems consecutive items; wave w owns the w-th
// quarter of the tile and walks it in rounds of 64, so "wave, round, lane" is item order.  Large tiles write longer runs; up to
// kFewSort items they would leave a CU one workgroup or none, whose sixteen rounds nobody overlaps (three passes over
// 1.0e6 / 3.7e5 items, the scatter kernels alone: 49 -> 32 / 45 -> 25 us).

// Digit counts of one tile per workgroup, one row of `hist`, written here and read by the scatter pass side by side.
// Neighbouring lanes count into kCopies different counters of a digit: a hot row (18 % of a skewed batch) brings ten
// equal digits per wave, and LDS adds to equal addresses run one after the other.  Three passes over 8.2e6 keys, Zipf(1.2):
// 73 -> 36 us with four copies (82 with counts in one row per digit); 1.05e8 keys, half of them uniform: 516 -> 341 us.
constexpr int kCopies = 4;
__device__ inline uint32_t csr_key(const SortCsr &csr, uint32_t row) { return (int32_t)row >= 0 ? row : csr.missing; }
// kCsr: the keys are the rows of a CSR batch, and the workgroups also note the bag of every tile's first entry, each for a share of
// the bags, and behind them the bag of the last entry.
template <typename KeyT, int kItems, bool kCsr>
__global__ __launch_bounds__(kBlock) void k_radix_hist(const KeyT *__restrict__ keys, int64_t n, int shift, int bits,
                                                        uint32_t *__restrict__ hist, const SortCsr csr) {
  __shared__ uint4 cnt[kMaxRadix];
  static_assert(kCopies == 4, "one uint4 per digit");
  const int radix = 1 << bits;
  const uint32_t mask = (1u << bits) - 1u, copy = threadIdx.x % kCopies;
  const int64_t base = (int64_t)blockIdx.x * (kBlock * kItems);
  KeyT key[kItems];
  // the keys are requested before the counters are cleared, so that the barrier is passed while they travel
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    const int64_t idx = base + (int64_t)i * kBlock + threadIdx.x;
    key[i] = idx < n ? (kCsr ? (KeyT)csr.rows[idx] : keys[idx]) : (KeyT)0;
  }
  if (kCsr) {
    constexpr int kTile = kBlock * kItems;
    const int64_t share = (csr.nbags + gridDim.x - 1) / gridDim.x, b1 = min(csr.nbags, (blockIdx.x + 1) * share);
    for (int64_t b = blockIdx.x * share + threadIdx.x; b < b1; b += kBlock) {
      const int64_t e0 = csr.offsets[b], e1 = csr.offsets[b + 1];
      for (int64_t t = (e0 + kTile - 1) / kTile; t * kTile < min(e1, n); ++t) csr.tile_bag[t] = (uint32_t)b;
      if (e0 < n && e1 >= n) csr.tile_bag[gridDim.x] = (uint32_t)b;
    }
  }
  for (int d = threadIdx.x; d < radix; d += kBlock) cnt[d] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  uint32_t *counters = reinterpret_cast<uint32_t *>(cnt);
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    const int64_t idx = base + (int64_t)i * kBlock + threadIdx.x;
    if (kCsr) key[i] = csr_key(csr, key[i]);
    if (idx < n) atomicAdd(&counters[((uint32_t)(key[i] >> shift) & mask) * kCopies + copy], 1u);
  }
  __syncthreads();
  for (int d = threadIdx.x; d < radix; d += kBlock) {
    const uint4 c = cnt[d];
    hist[(size_t)blockIdx.x * radix + d] = (c.x + c.y) + (c.z + c.w);
  }
}

// Turns the counts into each tile's offset inside its digit (exclusive sum over the tiles before it, in place) and leaves the
// digits' totals.  A workgroup takes kScanDigits digits of one stretch of kScanStretch tiles; its kScanGroups groups of as
// many lanes take consecutive runs of tiles, twice: once for their sums, which a wave per digit scans, once to write the
// offsets.  With several stretches k_radix_stretch has left the stretches' sums.
constexpr int kScanDigits = 16;
constexpr int kScanBlock = 1024;
constexpr int kScanGroups = kScanBlock / kScanDigits;
constexpr int kScanFlight = 16;                        // rows a thread requests together
constexpr int kScanStretch = kScanGroups * kScanFlight;

__device__ inline uint32_t scan_load(const uint32_t *p, int lo, int hi, int radix, uint32_t (&v)[kScanFlight]) {
  uint32_t sum = 0;
#pragma unroll
  for (int j = 0; j < kScanFlight; ++j) v[j] = lo + j < hi ? p[(size_t)(lo + j) * radix] : 0u;
#pragma unroll
  for (int j = 0; j < kScanFlight; ++j) sum += v[j];
  return sum;
}

// sums of the stretches: grid (digit groups, stretches)
__global__ __launch_bounds__(kScanBlock) void k_radix_stretch(const uint32_t *__restrict__ hist, int nblocks, int radix,
                                                               uint32_t *__restrict__ stretch_sums) {
  __shared__ uint32_t total[kScanDigits];
  const int col = threadIdx.x % kScanDigits, grp = threadIdx.x / kScanDigits, d = blockIdx.x * kScanDigits + col;
  if (threadIdx.x < kScanDigits) total[threadIdx.x] = 0;
  __syncthreads();
  const int lo = blockIdx.y * kScanStretch + grp * kScanFlight;
  uint32_t v[kScanFlight];
  if (d < radix) atomicAdd(&total[col], scan_load(hist + d, lo, nblocks, radix, v));
  __syncthreads();
  if (grp == 0 && d < radix) stretch_sums[(size_t)blockIdx.y * radix + d] = total[col];
}

__global__ __launch_bounds__(kScanBlock) void k_radix_scan(uint32_t *__restrict__ hist, int nblocks, int radix,
                                                            const uint32_t *__restrict__ stretch_sums,
                                                            uint32_t *__restrict__ totals) {
  __shared__ uint32_t sums[kScanDigits][kScanGroups + 1];
  static_assert(kScanGroups == kWave && kScanDigits == kScanBlock / kWave, "one wave scans one digit's groups");
  const int col = threadIdx.x % kScanDigits, grp = threadIdx.x / kScanDigits, d = blockIdx.x * kScanDigits + col;
  const bool live = d < radix;
  uint32_t *p = hist + (live ? d : 0);
  const int lo = blockIdx.y * kScanStretch + grp * kScanFlight;
  uint32_t v[kScanFlight];
  sums[col][grp] = scan_load(p, lo, nblocks, radix, v);
  __syncthreads();
  {
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, dw = blockIdx.x * kScanDigits + wave;
    uint32_t before = 0;                               // the digit's items in earlier stretches
    if (dw < radix)
      for (int st = lane; st < (int)blockIdx.y; st += kWave) before += stretch_sums[(size_t)st * radix + dw];
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) before += __shfl_xor(before, o, kWave);
    const uint32_t mine = sums[wave][lane], inc = wave_inclusive_scan(mine) + before;
    __builtin_amdgcn_wave_barrier();
    sums[wave][lane] = inc - mine;
    if (lane == kWave - 1 && dw < radix && blockIdx.y == gridDim.y - 1) totals[dw] = inc;
  }
  __syncthreads();
  uint32_t run = sums[col][grp];
  if (!live) return;
#pragma unroll
  for (int j = 0; j < kScanFlight; ++j) {
    if (lo + j < nblocks) p[(size_t)(lo + j) * radix] = run;
    run += v[j];
  }
}

// Lanes (of `live`) that hold the same `bits` low bits of d.
template <int kBits>
__device__ inline unsigned long long same_digit(uint32_t d, int bits, unsigned long long live) {
  uint32_t lo = (uint32_t)live, hi = (uint32_t)(live >> 32);
  const auto step = [&](int bit) {
    const uint32_t mine = (uint32_t)((int32_t)(d << (31 - bit)) >> 31);      // all ones where the bit is set
    const unsigned long long set = __ballot(mine != 0u);
    lo = __builtin_amdgcn_bitop3_b32(lo, mine, (uint32_t)set, 0x90);         // lo & ~(mine ^ set)
    hi = __builtin_amdgcn_bitop3_b32(hi, mine, (uint32_t)(set >> 32), 0x90);
  };
  if (kBits) {
#pragma unroll
    for (int bit = 0; bit < kBits; ++bit) step(bit);
  } else {
    for (int bit = 0; bit < bits; ++bit) step(bit);
  }
  return ((unsigned long long)hi << 32) | lo;
}

// Scatter of one pass.  The tile is first put in digit order inside LDS (rank of an item = items of
// smaller digits in the tile + items of its digit in earlier waves + earlier rounds of its wave +
// lower lanes of its round, which is item order, so the pass is stable); then consecutive threads
// write consecutive sorted items, so the items of one digit leave as one contiguous run instead of
// one 4-byte store per lane.  A tile's run of a digit is some 32 bytes long and the next tile's run follows it: in large
// batches a die takes consecutive tiles, so that its L2 puts the lines together (three passes over 1.05e8 pairs 2146 -> 1459 us,
// 8.2e6 121 -> 103; the tiles of up to kFewSort items all run at once, where it gives nothing: 29.8 and 32.1 us at 1.0e6).
// kBits: width of the digit where it is known here, else 0 (unrolled ballots: 145 -> 121 us at 8.2e6, the passes of smaller
// batches 32.6 -> 29.8 us at 1.0e6).
// kCsr (first pass over a CSR batch): an entry's bag is the one that the last bag start up to it belongs to.  The tile's starts are
// marked in LDS, as a bit per entry and the bag's number where the sorted keys come later; a wave holds the words of bits, one
// per lane, with the last start before each of them.  Without the pass that wrote (row, bag) pairs first the kernels up to here
// take, at 3.7e5 / 1.0e6 / 8.2e6 / 1.05e8 entries, 33 -> 29, 48 -> 37, 169 -> 145 and 2204 -> 1863 us.  (Three waves per SIMD instead
// of four, which spill 16 bytes: 46 against 43 us at 8.0e6.)
// kCounts: `offsets` holds the tiles' counts as they are and every workgroup adds up what it needs of them by itself, which while they
// are few is shorter than the launch of a scan: backward pass of 1.6e4 entries, three passes of 8 bits 68 -> 60 us, two of 9 and 8 61 -> 53;
// 6.4e4 (63 tiles) 70 -> 65 and, of 9 and 8, 61 -> 62; 1.3e5 81 -> 81 and 64 -> 71.
constexpr int kCountsAdded = 16384, kCountFlight = 16;   // counts; tiles whose counts a thread requests together
constexpr uint32_t kWideTile = 16;       // bags per entry of a tile from which a binary search per entry takes no longer than walking them
template <typename KeyT, bool kHasPayload, int kItems, int kBits, bool kCsr, bool kCounts>
__global__ __launch_bounds__(kBlock, kItems == kSortItems ? 4 : 8) void k_radix_scatter(const KeyT *__restrict__ keys_in,
                                                           const uint32_t *__restrict__ pay_in,
                                                           KeyT *__restrict__ keys_out, uint32_t *__restrict__ pay_out,
                                                           int64_t n, int shift, int any_bits,
                                                           const uint32_t *__restrict__ offsets,
                                                           const uint32_t *__restrict__ totals, const SortCsr csr) {
  constexpr int kTile = kBlock * kItems;
  constexpr int kWords = kTile / kWave;
  static_assert(!kCsr || (kHasPayload && kWords <= kWave && kItems <= kWave), "a lane per word of starts");
  __shared__ uint32_t starts[kCsr ? kWords * 2 : 1];    // bit per entry: a bag starts there
  __shared__ uint32_t cnt[kWavesPerBlock][kMaxRadix];   // per wave and digit: count, then start inside the digit's run
  __shared__ uint32_t dig_base[kMaxRadix];              // first sorted index of the digit inside the tile
  __shared__ uint32_t gofs[kMaxRadix];                  // where the tile's run of the digit starts in the output
  __shared__ unsigned long long scan_lds[kWavesPerBlock];
  __shared__ KeyT skey[kTile];                      // the sorted keys; afterwards reused for the payloads
  static_assert(sizeof(KeyT) >= sizeof(uint32_t), "payloads are staged in the key buffer");
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int bits = kBits ? kBits : any_bits;
  const uint32_t tile_no = kItems == kSortItems ? die_contiguous(blockIdx.x, gridDim.x) : blockIdx.x;
  const int64_t tile = (int64_t)tile_no * kTile;
  const int tile_n = (int)min((int64_t)kTile, n - tile);
  const int radix = 1 << bits;
  const uint32_t mask = (1u << bits) - 1u;
  const unsigned long long lane_lt = (1ull << lane) - 1ull;
  const int64_t wbase = tile + (int64_t)wave * (kItems * kWave);
  KeyT key[kItems];
  uint32_t pay[kItems];
  uint32_t rank[kItems];
  // the tile's items are requested first, so that their latency overlaps the fetch of the run offsets
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const int64_t idx = wbase + r * kWave + lane;
    const bool live = idx < n;
    key[r] = live ? (kCsr ? (KeyT)csr.rows[idx] : keys_in[idx]) : (KeyT)0;
    if (kHasPayload && !kCsr) pay[r] = live ? pay_in[idx] : 0u;
  }
  if (kCsr && threadIdx.x < kWords * 2) starts[threadIdx.x] = 0u;
  // kCounts: the sums over the tiles before this one and over all of them, of two digits per thread and as many tiles at a time as there are
  // threads for
  uint32_t *const before = dig_base, *const all = gofs;   // written in earnest only behind the ranking
  if (kCounts) {
    const int pairs = radix / 2 > 0 ? radix / 2 : 1, groups = kBlock / pairs, grp = threadIdx.x / pairs, d = (int)(threadIdx.x % pairs) * 2;
    for (int i = threadIdx.x; i < radix; i += kBlock) before[i] = all[i] = 0u;
    uint32_t sum[2] = {0u, 0u}, lower[2] = {0u, 0u};
    const auto row = [&](int t) { return *reinterpret_cast<const uint2 *>(offsets + (size_t)t * radix + d); };
    if (grp < groups) {
      for (int t0 = grp; t0 < (int)gridDim.x; t0 += groups * kCountFlight) {
        uint2 c[kCountFlight];
#pragma unroll
        for (int j = 0; j < kCountFlight; ++j) c[j] = row(min(t0 + j * groups, (int)gridDim.x - 1));
#pragma unroll
        for (int j = 0; j < kCountFlight; ++j) {
          const int t = t0 + j * groups;
          if (t >= (int)gridDim.x) c[j] = make_uint2(0u, 0u);
          sum[0] += c[j].x; sum[1] += c[j].y;
          if (t < (int)tile_no) { lower[0] += c[j].x; lower[1] += c[j].y; }
        }
      }
    }
    __syncthreads();
    if (grp < groups) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        atomicAdd(&before[d + j], lower[j]);
        atomicAdd(&all[d + j], sum[j]);
      }
    }
    __syncthreads();
  }
  // two digits per thread (kMaxRadix <= 2 * kBlock): the tile's offset inside the digit and the digit's total
  static_assert(kMaxRadix <= 2 * kBlock, "two digits per thread");
  uint32_t in_digit[2] = {0u, 0u};
  unsigned long long tot[2] = {0ull, 0ull};
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int d = threadIdx.x * 2 + j;
    if (d < radix) {
      in_digit[j] = kCounts ? before[d] : offsets[(size_t)tile_no * radix + d];
      tot[j] = (unsigned long long)(kCounts ? all[d] : totals[d]) << 32;
#pragma unroll
      for (int w = 0; w < kWavesPerBlock; ++w) cnt[w][d] = 0;
    }
  }
  __syncthreads();
  uint32_t *bag_at = reinterpret_cast<uint32_t *>(skey);  // bag that starts at the entry
  uint32_t first_bag = 0;                                // of the tile's first entry
  if (kCsr) {
    first_bag = csr.tile_bag[tile_no];
    const uint32_t last_bag = min(csr.tile_bag[tile_no + 1], (uint32_t)csr.nbags - 1u);
    if (last_bag - first_bag > kWideTile * kTile) {     // a long run of empty bags lies between: every entry looks its own bag up
      for (int at = threadIdx.x; at < tile_n; at += kBlock) {
        uint32_t lo = first_bag, hi = last_bag + 1;
        while (hi - lo > 1) {
          const uint32_t mid = (lo + hi) >> 1;
          if (csr.offsets[mid] <= tile + at) lo = mid; else hi = mid;
        }
        atomicOr(&starts[at >> 5], 1u << (at & 31));
        bag_at[at] = lo;
      }
    } else {
      for (uint32_t b = first_bag + 1 + threadIdx.x; b <= last_bag; b += kBlock) {
        const int64_t at = csr.offsets[b] - tile;
        if (at >= 0 && at < tile_n && csr.offsets[b + 1] - tile > at) {
          atomicOr(&starts[at >> 5], 1u << (at & 31));
          bag_at[at] = b;
        }
      }
    }
  }

#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const int64_t idx = wbase + r * kWave + lane;
    const bool live = idx < n;
    if (kCsr) key[r] = csr_key(csr, key[r]);
    const uint32_t d = (uint32_t)(key[r] >> shift) & mask;
    const unsigned long long peers = same_digit<kBits>(d, bits, __ballot(live));
    const uint32_t before = (uint32_t)__popcll(peers & lane_lt);
    uint32_t prev = 0;
    if (live) prev = cnt[wave][d];
    // every lane has read its counter before the group leaders below overwrite them:
    // the wave executes the load and the store as two instructions in program order
    __builtin_amdgcn_wave_barrier();
    if (live && before == 0) cnt[wave][d] = prev + (uint32_t)__popcll(peers);
    __builtin_amdgcn_wave_barrier();
    rank[r] = prev + before;
  }
  __syncthreads();
  if (kCsr) {                                           // done with the starts before the barriers ahead of the sorted keys
    uint32_t lo = 0, hi = 0;
    if (lane < kWords) { lo = starts[lane * 2]; hi = starts[lane * 2 + 1]; }
    int last = hi ? lane * kWave + 63 - __clz(hi) : lo ? lane * kWave + 31 - __clz(lo) : -1;
#pragma unroll
    for (int off = 1; off < kWords; off <<= 1) {
      const int o = __shfl_up(last, off, kWave);
      if (lane >= off) last = max(last, o);
    }
    last = __shfl_up(last, 1, kWave);
    if (lane == 0) last = -1;
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
      const int word = wave * kItems + r;
      const unsigned long long bits_r = ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane(hi, word) << 32) |
                                        (uint32_t)__builtin_amdgcn_readlane(lo, word);
      const unsigned long long upto = bits_r & (lane_lt | 1ull << lane);
      const int before = __builtin_amdgcn_readlane(last, word);  // not in a branch: the lane read from has to be active
      const int at = upto ? word * kWave + 63 - __clzll(upto) : before;
      const uint32_t bag = at >= 0 ? bag_at[at] : first_bag;
      const int64_t idx = wbase + r * kWave + lane;
      pay[r] = bag;
      if (csr.bag_of) {
        pay[r] = (uint32_t)idx;
        if (idx < n) csr.bag_of[idx] = (int32_t)bag;
      }
    }
  }
  // per digit: exclusive prefix over the waves; then one exclusive prefix over the digits of both the tile's counts (low
  // half) and the array's (high half): where the digit starts in the tile and where in the output
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int d = threadIdx.x * 2 + j;
    if (d < radix) {
      uint32_t run = 0;
#pragma unroll
      for (int w = 0; w < kWavesPerBlock; ++w) {
        const uint32_t c = cnt[w][d];
        cnt[w][d] = run;
        run += c;
      }
      tot[j] += run;
    }
  }
  unsigned long long total;
  unsigned long long ex = block_exclusive_scan<unsigned long long>(tot[0] + tot[1], scan_lds, total);
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int d = threadIdx.x * 2 + j;
    if (d < radix) {
      dig_base[d] = (uint32_t)ex;
      gofs[d] = (uint32_t)(ex >> 32) + in_digit[j];
    }
    ex += tot[j];
  }
  __syncthreads();
  uint32_t li[kItems];
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const int64_t idx = wbase + r * kWave + lane;
    li[r] = 0;
    if (idx < n) {
      const uint32_t d = (uint32_t)(key[r] >> shift) & mask;
      li[r] = dig_base[d] + cnt[wave][d] + rank[r];
      skey[li[r]] = key[r];
    }
  }
  __syncthreads();
  // keys out; every thread remembers where its sorted items went, for the payloads that follow
  constexpr int kOut = kTile / kBlock;
  uint32_t pos[kOut];
#pragma unroll
  for (int j = 0; j < kOut; ++j) {
    const int i = threadIdx.x + j * kBlock;
    pos[j] = 0;
    if (i < tile_n) {
      const KeyT k = skey[i];
      const uint32_t d = (uint32_t)(k >> shift) & mask;
      pos[j] = gofs[d] + ((uint32_t)i - dig_base[d]);
      keys_out[pos[j]] = k;
    }
  }
  if (kHasPayload) {
    uint32_t *spay = reinterpret_cast<uint32_t *>(skey);
    __syncthreads();                                   // all keys read before the buffer is overwritten
#pragma unroll
    for (int r = 0; r < kItems; ++r)
      if (wbase + r * kWave + lane < n) spay[li[r]] = pay[r];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kOut; ++j) {
      const int i = threadIdx.x + j * kBlock;
      if (i < tile_n) pay_out[pos[j]] = spay[i];
    }
  }
}

inline int64_t sort_blocks(int64_t n) { return (n + kSortTile - 1) / kSortTile; }

template <typename KeyT, bool kHasPayload, int kItems>
int radix_sort(SortBuffers buf, int64_t n, int bits, uint32_t *hist, uint32_t *stretch_sums, uint32_t *totals,
               const SortCsr *csr, hipStream_t s, int kid_hist, int kid_scan, int kid_scatter) {
  if (n <= 0 || bits <= 0) return 0;
  const int nblocks = (int)((n + kBlock * kItems - 1) / (kBlock * kItems));
  const int widest = n >= kSortTotals ? kMaxDigitBits : kFewItemsBits;
  const int npass = (bits + widest - 1) / widest;
  const int per = (bits + npass - 1) / npass;
  KeyT *kin = (KeyT *)buf.keys_a, *kout = (KeyT *)buf.keys_b;
  uint32_t *pin = buf.pay_a, *pout = buf.pay_b;
  int side = 0;
  for (int p = 0; p < npass; ++p) {
    const int shift = p * per;
    const int b = (bits - shift) < per ? (bits - shift) : per;
    const bool from_csr = csr && p == 0;
    {
      ProfScope ps(kid_hist, s);
      if (from_csr) hipLaunchKernelGGL((k_radix_hist<KeyT, kItems, true>), dim3(nblocks), dim3(kBlock), 0, s, kin, n, shift, b, hist, *csr);
      else hipLaunchKernelGGL((k_radix_hist<KeyT, kItems, false>), dim3(nblocks), dim3(kBlock), 0, s, kin, n, shift, b, hist, SortCsr{});
    }
    const bool counts = kItems == kFewSortItems && nblocks <= kCountsAdded >> b;
    if (!counts) {
      ProfScope ps(kid_scan, s);
      const dim3 grid(((1 << b) + kScanDigits - 1) / kScanDigits, (nblocks + kScanStretch - 1) / kScanStretch);
      if (grid.y > 1)
        hipLaunchKernelGGL(k_radix_stretch, dim3(grid.x, grid.y - 1), dim3(kScanBlock), 0, s, hist, nblocks, 1 << b, stretch_sums);
      hipLaunchKernelGGL(k_radix_scan, grid, dim3(kScanBlock), 0, s, hist, nblocks, 1 << b, stretch_sums, totals);
    }
    {
      ProfScope ps(kid_scatter, s);
      const auto scatter = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(nblocks), dim3(kBlock), 0, s, kin, pin, kout, pout, n, shift, b, hist, totals,
                           from_csr ? *csr : SortCsr{});
      };
      const auto of_width = [&](auto first, auto raw) {
        constexpr bool kCsr = decltype(first)::value, kCounts = decltype(raw)::value;
        if (b == 9) scatter(k_radix_scatter<KeyT, kHasPayload, kItems, 9, kCsr, kCounts>);
        else if (b == 8) scatter(k_radix_scatter<KeyT, kHasPayload, kItems, 8, kCsr, kCounts>);
        else if (b == 7) scatter(k_radix_scatter<KeyT, kHasPayload, kItems, 7, kCsr, kCounts>);
        else scatter(k_radix_scatter<KeyT, kHasPayload, kItems, 0, kCsr, kCounts>);
      };
      const auto of_first = [&](auto raw) { if (from_csr) of_width(std::true_type{}, raw); else of_width(std::false_type{}, raw); };
      if constexpr (kItems == kFewSortItems) {
        if (counts) of_first(std::true_type{}); else of_first(std::false_type{});
      } else {
        of_first(std::false_type{});
      }
    }
    KeyT *tk = kin; kin = kout; kout = tk;
    uint32_t *tp = pin; pin = pout; pout = tp;
    side ^= 1;
  }
  return side;
}

}  // namespace

size_t scan_scratch_bytes(int64_t n) {
  const int64_t nb = (n + kScanTile - 1) / kScanTile;
  return align_up((size_t)(nb + 1) * sizeof(unsigned long long), 256);
}

// One row of counts per tile, then either the sums of the stretches (kMaxRadix values per kScanStretch tiles, the last
// stretch left out: less than two bytes per tile) or the scratch of a device-wide scan, which the callers run after the sort.
size_t sort_scratch_bytes(int64_t n) {
  const int64_t nblocks = sort_blocks(n > 0 ? n : 1);
  static_assert(kMaxRadix * sizeof(uint32_t) * kScanTile <= kMaxRadix * sizeof(unsigned long long) * kScanStretch,
                "a stretch's row of sums fits where its tiles' counts would have their scan scratch");
  return align_up((size_t)kMaxRadix * nblocks * sizeof(uint32_t), 256) + scan_scratch_bytes(kMaxRadix * nblocks);
}

void exclusive_scan_u32(uint32_t *data, int64_t n, uint32_t *total_out, void *scratch, hipStream_t s) {
  exclusive_scan<uint32_t>(data, n, total_out, scratch, s);
}

void exclusive_scan_u64(unsigned long long *data, int64_t n, unsigned long long *total_out, void *scratch,
                        hipStream_t s) {
  exclusive_scan<unsigned long long>(data, n, total_out, scratch, s);
}

size_t csr_scratch_bytes(int64_t n) { return (size_t)((n + kFewSortTile - 1) / kFewSortTile + 1) * sizeof(uint32_t); }

size_t few_sort_scratch_bytes(int64_t n) {
  return (size_t)kMaxRadix * sizeof(uint32_t) * (size_t)((n + kFewSortTile - 1) / kFewSortTile);
}

int radix_sort_u32_pairs(SortBuffers buf, int64_t n, int bits, void *scratch, void *few_scratch, uint32_t *totals,
                         const SortCsr *csr, hipStream_t s) {
  static_assert(kFewSort <= (int64_t)kScanStretch * kFewSortTile, "one stretch: no sums of stretches");
  if (n <= kFewSort)
    return radix_sort<uint32_t, true, kFewSortItems>(buf, n, bits, (uint32_t *)few_scratch, nullptr, totals, csr, s, KID_SORT_HIST,
                                                     KID_SORT_SCAN, KID_SORT_SCATTER);
  // the sums of all stretches but the last lie behind the counts (see sort_scratch_bytes)
  uint32_t *stretch_sums = (uint32_t *)((char *)scratch + align_up((size_t)kMaxRadix * sort_blocks(n) * sizeof(uint32_t), 256));
  return radix_sort<uint32_t, true, kSortItems>(buf, n, bits, (uint32_t *)scratch, stretch_sums, totals, csr, s, KID_SORT_HIST,
                                                KID_SORT_SCAN, KID_SORT_SCATTER);
}

}  // namespace des
