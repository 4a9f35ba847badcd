// Backward of the sparse operators, duplicate-key merge and fused optimizer update.
//
// Section 3.2.2 (back-propagation phase): the gradient of each aggregate is handed unchanged to
// every shard's sub-operator, so the backward pass needs no exchange.  Section 5: the merged
// gradient of a weight is applied locally and the table row is updated.
//
// Steps: (1, 2) stable radix sort of the CSR batch's (row, bag) pairs by row, (3) mark
// segment heads and compact them (ascending row order), (4) one lane group per segment of up to
// kShortMax entries reduces its entries in registers and updates the row in the same kernel; longer
// segments are cut into chunks of 512 or 128 entries, one wave each: a segment that is a single chunk
// is updated by that wave, the others are combined and updated by one workgroup per segment.
// Steps (1)-(3) need the batch and its rows only and can be issued ahead of the gradients
// (des_backward_prepare).
//
// Per entry e of bag (b,f) with value x:  d/dw += x*g_lr[b],
//   d/dv += x*(g_fm[b]*A_sum[b,:] + g_pool[b,f,:]) - v * (x*x*g_fm[b])
// i.e. the row's own vector v enters only through one scalar per segment, so v is read once.
#include <math.h>
#include "des_index.h"
#include "des_internal.h"

namespace des {
namespace {

constexpr int kShortMax = 32;              // segments up to this many entries are reduced by one lane group
// Entries per chunk of a longer segment (one wave per chunk), as a power of two.  A wave reads its chunk in dependent steps of 4
// entries per lane group; a smaller batch has too few chunks of 512 to fill the chip, so those steps are all that is
// waited for.  k_long_partial, 512 -> 128, D = 64: 4.8e5 entries 50 -> 20 us, 1.9e6 58 -> 42, 3.8e6 84 -> 79, 7.7e6
// 179 -> 174, where k_long_final takes the gain back (17 -> 22).  64 or 256 are no better at 3.7e5.  (No batch has more chunks than n/33: a segment of L > 32 entries
// has at most ceil(L/128) <= L/33 of them.)
constexpr int kChunkShift = 9, kFewChunkShift = 7;
constexpr int64_t kFewEntries = 1 << 22;
inline int chunk_shift_for(int64_t n) { return n <= kFewEntries ? kFewChunkShift : kChunkShift; }
constexpr int kMidFan = 64;                // chunk partials that one wave pre-sums for segments of more chunks than this
constexpr int kShortGrid = 65536;          // most workgroups of the short-segment kernel (it strides over the segments)
constexpr int kHeadItems = 8;
constexpr int kHeadTile = kBlock * kHeadItems;
constexpr int64_t kHeadsSelfPrefix = 4096;  // up to this many tiles every workgroup sums the earlier tiles' head counts itself
constexpr int kWavesPerBlock = kBlock / kWave;

struct BwdArgs {
  // batch and upstream gradients
  const int32_t *offsets;
  const float *vals;
  const int32_t *rows;
  const float *g_lr, *g_fm, *A_sum, *g_pool;
  struct Take { const float *base; uint32_t mask; };   // an upstream array, or (mask 0) the table's first row in its place
  Take take_lr, take_fm, take_sum, take_pool;
  int64_t n;            // nnz
  int64_t nbags;
  int F;
  uint32_t missing;     // sort key of entries without a row (= capacity, sorts last)
  // table
  float *emb, *w, *acc_emb, *acc_w, *acc2_emb, *acc2_w;
  const uint64_t *row_keys;
  Ctrl *ctrl;
  // workspace
  uint32_t *key_sorted, *pay_sorted;
  int32_t *bag_of;      // entry -> bag, only with vals
  int32_t *seg_off;     // [n+1]
  int32_t *uniq_rows;   // [n]
  uint32_t *first_pay;  // [n]  payload of the first entry of each segment
  uint32_t *head_sums;
  int32_t *long_seg;    // segment index of long segment j
  uint32_t *long_c0;    // first chunk of long segment j
  // (the next three lie in the sorted keys, which nothing reads once the segments are cut)
  int32_t *multi_seg;   // long segment indices j of the segments with more than one chunk
  int32_t *group_seg;   // long segment index j of pre-summed group i (segments of more than kMidFan chunks)
  uint32_t *group_c;    // first chunk of that group
  int32_t *chunk_owner; // long segment index of chunk c
  int chunk_shift;      // log2 of the entries per chunk
  double *partials;     // [chunks][D+4]
  // optimizer (opt_emb == DES_OPT_NONE: merge only)
  int opt_emb, opt_w;
  float lr, eps;
  float b1, b2, c1, c2;   // Adam: decay rates and bias corrections 1/(1-b1^t), 1/(1-b2^t)
  float f_alpha, f_beta, f_l1, f_l2;
  // optional outputs
  int32_t *uniq_rows_out;
  uint64_t *uniq_keys_out;
  int32_t *counts_out;
  float *merged_out;
  int64_t *n_uniq_out;
};

__device__ inline int chunks_of(const BwdArgs &a, uint32_t len) { return (int)((len + (1u << a.chunk_shift) - 1u) >> a.chunk_shift); }

__device__ inline float4 ld4(const float *p) { return *reinterpret_cast<const float4 *>(p); }
__device__ inline void st4(float *p, float4 v) { *reinterpret_cast<float4 *>(p) = v; }
// Streaming variants for data that is touched once per call (table rows of one-entry segments,
// upstream gradient rows): they do not displace the reusable lines in the caches.
typedef float v4f __attribute__((ext_vector_type(4)));
__device__ inline float4 ld4_stream(const float *p) {
  const v4f r = __builtin_nontemporal_load(reinterpret_cast<const v4f *>(p));
  return make_float4(r.x, r.y, r.z, r.w);
}
__device__ inline void st4_stream(float *p, float4 v) {
  v4f r; r.x = v.x; r.y = v.y; r.z = v.z; r.w = v.w;
  __builtin_nontemporal_store(r, reinterpret_cast<v4f *>(p));
}
__device__ inline float4 f4zero() { return make_float4(0.f, 0.f, 0.f, 0.f); }
__device__ inline float4 f4add(float4 a, float4 b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); }

// (1) The first sorting pass takes rows and offsets as they are where bags are not many more than entries: its workgroups walk the bags
// of a tile of entries one step per 256 of them, which without a bound could be all of an almost empty batch's.  Row sort, segment
// heads and split with pairs written first / from the batch, at 0.5, 1, 2 and 4 bags per entry: 2e4 entries 46/44, 46/46, 45/47, 46/51 us;
// 1.0e6 70/64, 71/66, 72/69, 76/75; with the larger tiles 1.1e6 89/85, 88/91, 88/104, 92/132, 4.0e6 121/115, 126/122, 134/138, 151/171,
// 1.6e7 364/330, 388/362, 438/428, 527/590.  So up to one bag per entry, and three quarters of one while there are few large tiles.
inline bool bags_by_sort(int64_t n, int64_t nbags) {
  return n > kFewSort && n <= 4 * kFewSort ? nbags <= n - n / 4 : nbags <= n;
}

// Beyond that this kernel writes the pairs: sort key = row (or `missing`), payload = bag (or entry index with vals).  A workgroup takes
// kBlock consecutive bags, i.e. one contiguous range of entries, stages their offsets in LDS and
// walks the entries with consecutive threads (coalesced reads and writes); the bag of an entry
// is found by binary search in the staged offsets.
template <bool kHasVals>
__global__ __launch_bounds__(kBlock) void k_expand(const BwdArgs a, uint32_t *__restrict__ key_out,
                                                    uint32_t *__restrict__ pay_out) {
  __shared__ int offs[kBlock + 1];
  for (int64_t bag0 = (int64_t)blockIdx.x * kBlock; bag0 < a.nbags; bag0 += (int64_t)gridDim.x * kBlock) {
    const int nb = (int)min((int64_t)kBlock, a.nbags - bag0);
    __syncthreads();
    for (int i = threadIdx.x; i <= nb; i += kBlock) offs[i] = a.offsets[bag0 + i];
    __syncthreads();
    const uint32_t e0 = offs[0], e1 = offs[nb];
    for (uint32_t e = e0 + threadIdx.x; e < e1; e += kBlock) {
      int lo = 0, hi = nb;                              // largest i with offs[i] <= e
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if ((uint32_t)offs[mid] <= e) lo = mid; else hi = mid;
      }
      const int r = a.rows[e];
      key_out[e] = r >= 0 ? (uint32_t)r : a.missing;
      pay_out[e] = kHasVals ? e : (uint32_t)(bag0 + lo);
      if (kHasVals) a.bag_of[e] = (int32_t)(bag0 + lo);
    }
  }
}

// (3) segment heads.  flag(i) = key[i] is a row and differs from key[i-1].
__device__ inline uint32_t wave_incl_scan_u32(uint32_t v) {
  const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const uint32_t o = __shfl_up(v, off, kWave);
    if (lane >= off) v += o;
  }
  return v;
}

__device__ inline uint32_t block_excl_scan_u32(uint32_t v, uint32_t *lds, uint32_t &total) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const uint32_t inc = wave_incl_scan_u32(v);
  if (lane == kWave - 1) lds[wave] = inc;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kWavesPerBlock; ++w) {
    const uint32_t x = lds[w];
    if (w < wave) base += x;
    tot += x;
  }
  __syncthreads();
  total = tot;
  return base + inc - v;
}

// The thread's kHeadItems consecutive sorted keys (two 16-byte loads when they all exist); missing ones read as `fill`.
__device__ inline void load_head_keys(const uint32_t *__restrict__ keys, int64_t base, int64_t n, uint32_t fill,
                                      uint32_t (&k)[kHeadItems]) {
  static_assert(kHeadItems == 8, "two uint4 per thread");
  if (base + kHeadItems <= n) {
    const uint4 lo = *reinterpret_cast<const uint4 *>(keys + base);
    const uint4 hi = *reinterpret_cast<const uint4 *>(keys + base + 4);
    k[0] = lo.x; k[1] = lo.y; k[2] = lo.z; k[3] = lo.w; k[4] = hi.x; k[5] = hi.y; k[6] = hi.z; k[7] = hi.w;
  } else {
#pragma unroll
    for (int i = 0; i < kHeadItems; ++i) k[i] = base + i < n ? keys[base + i] : fill;
  }
}

__global__ __launch_bounds__(kBlock) void k_heads_count(const BwdArgs a) {
  __shared__ uint32_t lds[kWavesPerBlock];
  const int64_t n = a.n;
  const int64_t base = (int64_t)blockIdx.x * kHeadTile + (int64_t)threadIdx.x * kHeadItems;
  uint32_t cnt = 0;
  uint32_t prev = base > 0 && base <= n ? a.key_sorted[base - 1] : 0xFFFFFFFFu;
  uint32_t keys[kHeadItems];
  load_head_keys(a.key_sorted, base, n, a.missing, keys);
#pragma unroll
  for (int i = 0; i < kHeadItems; ++i) {
    if (base + i < n) {
      const uint32_t k = keys[i];
      cnt += (k != a.missing && (base + i == 0 || k != prev)) ? 1u : 0u;
      prev = k;
    }
  }
  uint32_t total;
  block_excl_scan_u32(cnt, lds, total);
  if (threadIdx.x == 0) a.head_sums[blockIdx.x] = total;
}

// Bookkeeping after a device-wide scan of the tile counts (many tiles): the scan left the total behind the counts.
__device__ inline void heads_bookkeeping(const BwdArgs &a, uint32_t n_uniq) {
  a.ctrl->n_uniq = n_uniq;
  a.ctrl->n_long = 0;
  a.ctrl->n_chunks = 0;
  a.ctrl->n_multi = 0;
  a.ctrl->n_groups = 0;
}

__global__ void k_heads_finish(const BwdArgs a, const uint32_t *total) { heads_bookkeeping(a, *total); }

// kSelfPrefix: head_sums still holds the tiles' counts and every workgroup adds up the counts of the tiles before
// its own (few tiles: cheaper than a launch that does it once); the last workgroup then also publishes the
// number of segments and resets the counters of the classify pass.
template <bool kSelfPrefix>
__global__ __launch_bounds__(kBlock) void k_heads_write(const BwdArgs a) {
  __shared__ uint32_t lds[kWavesPerBlock];
  __shared__ uint32_t l_key[kHeadTile];
  __shared__ int32_t l_idx[kHeadTile];
  const int64_t n = a.n;
  const int64_t base = (int64_t)blockIdx.x * kHeadTile + (int64_t)threadIdx.x * kHeadItems;
  uint32_t key[kHeadItems];
  bool flag[kHeadItems];
  uint32_t cnt = 0;
  uint32_t prev = base > 0 && base <= n ? a.key_sorted[base - 1] : 0xFFFFFFFFu;
  const uint32_t first_prev = prev;
  load_head_keys(a.key_sorted, base, n, a.missing, key);
#pragma unroll
  for (int i = 0; i < kHeadItems; ++i) {
    flag[i] = false;
    if (base + i < n) {
      flag[i] = key[i] != a.missing && (base + i == 0 || key[i] != prev);
      cnt += flag[i] ? 1u : 0u;
      prev = key[i];
    }
  }
  uint32_t total;
  uint32_t u0;                                          // heads before this tile
  if (kSelfPrefix) {
    uint32_t part = 0;
    for (uint32_t i = threadIdx.x; i < blockIdx.x; i += kBlock) part += a.head_sums[i];
    block_excl_scan_u32(part, lds, u0);
  } else {
    u0 = a.head_sums[blockIdx.x];
  }
  uint32_t loc = block_excl_scan_u32(cnt, lds, total);  // heads before this thread inside the tile
  if (kSelfPrefix && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) heads_bookkeeping(a, u0 + total);
  prev = first_prev;
#pragma unroll
  for (int i = 0; i < kHeadItems; ++i) {
    const int64_t idx = base + i;
    if (idx < n) {
      if (flag[i]) {
        l_key[loc] = key[i];
        l_idx[loc] = (int32_t)idx;
        ++loc;
      }
      // end of the last segment: first entry without a row, or the end of the array
      if (key[i] == a.missing && (idx == 0 || prev != a.missing)) a.seg_off[u0 + loc] = (int32_t)idx;
      if (idx == n - 1 && key[i] != a.missing) a.seg_off[u0 + loc] = (int32_t)n;
      prev = key[i];
    }
  }
  __syncthreads();
  // the tile's heads occupy consecutive output positions: write them with consecutive threads
  for (uint32_t j = threadIdx.x; j < total; j += kBlock) {
    const int32_t idx = l_idx[j];
    a.uniq_rows[u0 + j] = (int32_t)l_key[j];
    a.seg_off[u0 + j] = idx;
    a.first_pay[u0 + j] = a.pay_sorted[idx];
  }
}

// Long segments get a chunk range.  The order of the list is irrelevant to the results, so
// ranges are handed out with one atomic pair per workgroup.
__global__ __launch_bounds__(kBlock) void k_classify(const BwdArgs a) {
  __shared__ uint32_t lds[kWavesPerBlock];
  __shared__ unsigned long long base_long, base_chunk, base_multi, base_group;
  const long long U = a.ctrl->n_uniq;
  const int64_t tile0 = (int64_t)blockIdx.x * kHeadTile + (int64_t)threadIdx.x * kHeadItems;
  if ((int64_t)blockIdx.x * kHeadTile >= U) return;          // uniform per workgroup
  uint32_t nl = 0, nc = 0, nm = 0, ng = 0;
  int len[kHeadItems];
  if (tile0 + kHeadItems <= U) {                  // the thread's nine segment bounds: two 16-byte loads and one more
    const int4 lo = *reinterpret_cast<const int4 *>(a.seg_off + tile0);
    const int4 hi = *reinterpret_cast<const int4 *>(a.seg_off + tile0 + 4);
    const int last = a.seg_off[tile0 + kHeadItems];
    len[0] = lo.y - lo.x; len[1] = lo.z - lo.y; len[2] = lo.w - lo.z; len[3] = hi.x - lo.w;
    len[4] = hi.y - hi.x; len[5] = hi.z - hi.y; len[6] = hi.w - hi.z; len[7] = last - hi.w;
  } else {
#pragma unroll
    for (int i = 0; i < kHeadItems; ++i) {
      const int64_t u = tile0 + i;
      len[i] = u < U ? a.seg_off[u + 1] - a.seg_off[u] : 0;
    }
  }
#pragma unroll
  for (int i = 0; i < kHeadItems; ++i) {
    if (len[i] > kShortMax) {
      const uint32_t nch = (uint32_t)chunks_of(a, len[i]);
      ++nl; nc += nch;
      if (nch > 1) ++nm;
      if (nch > kMidFan) ng += (nch + kMidFan - 1) / kMidFan;
    }
  }
  uint32_t tot_l, tot_c, tot_m, tot_g;
  uint32_t ex_l = block_excl_scan_u32(nl, lds, tot_l);
  uint32_t ex_c = block_excl_scan_u32(nc, lds, tot_c);
  if (tot_l == 0) return;                                    // uniform: the scans synchronised the workgroup
  uint32_t ex_m = block_excl_scan_u32(nm, lds, tot_m);
  uint32_t ex_g = block_excl_scan_u32(ng, lds, tot_g);
  if (threadIdx.x == 0) {
    typedef unsigned long long ull;
    base_long = atomicAdd(reinterpret_cast<ull *>(&a.ctrl->n_long), (ull)tot_l);
    base_chunk = atomicAdd(reinterpret_cast<ull *>(&a.ctrl->n_chunks), (ull)tot_c);
    base_multi = tot_m ? atomicAdd(reinterpret_cast<ull *>(&a.ctrl->n_multi), (ull)tot_m) : 0ull;
    base_group = tot_g ? atomicAdd(reinterpret_cast<ull *>(&a.ctrl->n_groups), (ull)tot_g) : 0ull;
  }
  __syncthreads();
  uint32_t j = (uint32_t)base_long + ex_l, c0 = (uint32_t)base_chunk + ex_c;
  uint32_t jm = (uint32_t)base_multi + ex_m, gi = (uint32_t)base_group + ex_g;
#pragma unroll
  for (int i = 0; i < kHeadItems; ++i) {
    if (len[i] > kShortMax) {
      const uint32_t nch = (uint32_t)chunks_of(a, len[i]);
      a.long_seg[j] = (int32_t)(tile0 + i);
      a.long_c0[j] = c0;
      if (nch > 1) a.multi_seg[jm++] = (int32_t)j;           // what the per-segment combine has to visit
      if (nch > kMidFan)                                      // and the groups of chunk sums that are added up first
        for (uint32_t k = 0; k < nch; k += kMidFan) { a.group_seg[gi] = (int32_t)j; a.group_c[gi] = c0 + k; ++gi; }
      ++j;
      c0 += nch;
    }
  }
}

// one workgroup per long segment writes the owner of each of its chunks
__global__ __launch_bounds__(kBlock) void k_chunk_owner(const BwdArgs a) {
  const long long NL = a.ctrl->n_long;
  for (int64_t j = blockIdx.x; j < NL; j += gridDim.x) {
    const int u = a.long_seg[j];
    const int nch = chunks_of(a, a.seg_off[u + 1] - a.seg_off[u]);
    const uint32_t c0 = a.long_c0[j];
    for (int i = threadIdx.x; i < nch; i += blockDim.x) a.chunk_owner[c0 + i] = (int32_t)j;
  }
}

// Step (3) and the split for up to kFewHeads sorted entries in one workgroup, whose waves see all of it in LDS: one launch instead of
// four.  What it does is bound by a few dependent accesses; the passes over tiles, by the 2 to 4 us that each launch takes.  A thread's
// stretch of entries is consecutive for the count; the heads are then written with consecutive threads, eight of them in flight each,
// since up to 16 round trips in a row would be longer than the launches.  Backward pass with the four launches / this one: of 5e3 entries
// 49 / 39 us (1e5 rows, D = 16) and 58 / 45 (3e6, 32), of 9e3 52 / 43 and 59 / 50, of 1.6e4 53 / 45 and 59 / 52, with all entries on
// 40 rows 45 / 31.  The starts of twice the entries would not fit a workgroup's static 64 KB with the rest.
constexpr int64_t kFewHeads = 16384;
constexpr int kFewHeadsBlock = 1024, kFewHeadsItems = kFewHeads / kFewHeadsBlock;
__global__ __launch_bounds__(kFewHeadsBlock) void k_heads_few(const BwdArgs a) {
  constexpr int kWaves = kFewHeadsBlock / kWave, kItems = kFewHeadsItems;
  static_assert(kFewHeads <= 1 << 16, "positions in 16 bits");
  __shared__ uint16_t start[kFewHeads];
  __shared__ uint32_t sums[kWaves];
  __shared__ uint32_t n_long, n_chunks, n_multi, n_groups, end;
  const int n = (int)a.n, base = threadIdx.x * kItems, lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  uint32_t key[kItems];
  if (base + kItems <= n) {
#pragma unroll
    for (int q = 0; q < kItems / 4; ++q) {
      const uint4 v = *reinterpret_cast<const uint4 *>(a.key_sorted + base + q * 4);
      key[q * 4] = v.x; key[q * 4 + 1] = v.y; key[q * 4 + 2] = v.z; key[q * 4 + 3] = v.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < kItems; ++i) key[i] = base + i < n ? a.key_sorted[base + i] : a.missing;
  }
  uint32_t prev = base > 0 && base < n ? a.key_sorted[base - 1] : 0xFFFFFFFFu;
  if (threadIdx.x == 0) { n_long = n_chunks = n_multi = n_groups = 0; end = (uint32_t)n; }
  uint32_t heads = 0, with_row = 0;
  bool flag[kItems];
#pragma unroll
  for (int i = 0; i < kItems; ++i) {                       // entries past the end read as without a row
    flag[i] = key[i] != a.missing && (base + i == 0 || key[i] != prev);
    heads += flag[i] ? 1u : 0u;
    with_row += key[i] != a.missing ? 1u : 0u;
    prev = key[i];
  }
  const uint32_t inc = wave_incl_scan_u32(heads);
  if (lane == kWave - 1) sums[wave] = inc;
  __syncthreads();
  uint32_t u = inc - heads, U = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const uint32_t x = sums[w];
    if (w < wave) u += x;
    U += x;
  }
#pragma unroll
  for (int i = 0; i < kItems; ++i)
    if (flag[i]) start[u++] = (uint16_t)(base + i);
  if (with_row < kItems && base < n) atomicMin(&end, (uint32_t)(base + with_row));   // entries without a row sort last
  __syncthreads();
  const uint32_t stop = end;
  constexpr int kAtOnce = 8;                               // heads whose loads a thread has in flight
  for (uint32_t j0 = threadIdx.x; j0 < U; j0 += kAtOnce * kFewHeadsBlock) {
    uint32_t at[kAtOnce], row[kAtOnce], pay[kAtOnce];
#pragma unroll
    for (int i = 0; i < kAtOnce; ++i) {
      const uint32_t j = j0 + i * kFewHeadsBlock;
      at[i] = start[j < U ? j : 0];
      row[i] = a.key_sorted[at[i]];
      pay[i] = a.pay_sorted[at[i]];
    }
#pragma unroll
    for (int i = 0; i < kAtOnce; ++i) {
      const uint32_t j = j0 + i * kFewHeadsBlock;
      if (j < U) {
        a.uniq_rows[j] = (int32_t)row[i];
        a.seg_off[j] = (int32_t)at[i];
        a.first_pay[j] = pay[i];
      }
    }
  }
  if (threadIdx.x == 0) a.seg_off[U] = (int32_t)stop;
  __syncthreads();                                         // the keys have been read: the lists below take their place
  for (uint32_t j = threadIdx.x; j < U; j += kFewHeadsBlock) {
    const uint32_t len = (j + 1 < U ? start[j + 1] : stop) - start[j];
    if (len <= (uint32_t)kShortMax) continue;
    const uint32_t nch = (uint32_t)chunks_of(a, len), l = atomicAdd(&n_long, 1u), c0 = atomicAdd(&n_chunks, nch);
    a.long_seg[l] = (int32_t)j;
    a.long_c0[l] = c0;
    if (nch > 1) a.multi_seg[atomicAdd(&n_multi, 1u)] = (int32_t)l;
    if (nch > kMidFan) {
      uint32_t gi = atomicAdd(&n_groups, (nch + kMidFan - 1) / kMidFan);
      for (uint32_t k = 0; k < nch; k += kMidFan) { a.group_seg[gi] = (int32_t)l; a.group_c[gi] = c0 + k; ++gi; }
    }
    for (uint32_t k = 0; k < nch; ++k) a.chunk_owner[c0 + k] = (int32_t)l;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    a.ctrl->n_uniq = U;
    a.ctrl->n_long = n_long;
    a.ctrl->n_chunks = n_chunks;
    a.ctrl->n_multi = n_multi;
    a.ctrl->n_groups = n_groups;
  }
}

// Steps (1)-(3) and the split of long segments for a batch of up to kSmallSort entries, all in the LDS of one workgroup: such a
// batch is bound by launches (14 of them at 2560 entries, about 3.5 us each), not by work.  The sort is the same stable
// radix sort, eight bits a pass.
constexpr int kSmallSort = 4096;
constexpr int64_t kSmallBags = 65536;                // bags whose offsets one workgroup walks
constexpr int kSmallBlock = 1024;
constexpr int kSmallWaves = kSmallBlock / kWave;
constexpr int kSmallItems = kSmallSort / kSmallBlock;
constexpr int kSmallBits = 8;

// Exclusive scan over the workgroup's threads under `op` (sum or maximum, identity 0); total over all of them.
template <typename Op>
__device__ inline uint32_t small_excl_scan(uint32_t v, uint32_t *lds, uint32_t &total, Op op) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  uint32_t inc = v;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const uint32_t o = __shfl_up(inc, off, kWave);
    if (lane >= off) inc = op(inc, o);
  }
  uint32_t ex = __shfl_up(inc, 1, kWave);
  if (lane == 0) ex = 0;
  if (lane == kWave - 1) lds[wave] = inc;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kSmallWaves; w += 4) {                // 16-byte reads: every wave reads every sum
    const uint4 x = *reinterpret_cast<const uint4 *>(lds + w);
    base = op(base, w < wave ? x.x : 0u);
    base = op(base, w + 1 < wave ? x.y : 0u);
    base = op(base, w + 2 < wave ? x.z : 0u);
    base = op(base, w + 3 < wave ? x.w : 0u);
    tot = op(op(tot, x.x), op(op(x.y, x.z), x.w));
  }
  __syncthreads();
  total = tot;
  return op(base, ex);
}

template <bool kHasVals>
__global__ __launch_bounds__(kSmallBlock) void k_sort_small(const BwdArgs a, uint32_t *__restrict__ pay_out, int bits) {
  __shared__ __align__(16) uint32_t skey[kSmallSort + 4], spay[kSmallSort];
  __shared__ __align__(16) uint32_t cnt[kSmallWaves][1 << kSmallBits];
  __shared__ __align__(16) uint32_t scan_lds[kSmallWaves];
  static_assert(__alignof__(skey) >= 16 && __alignof__(spay) >= 16 && __alignof__(cnt) >= 16 && __alignof__(scan_lds) >= 16,
                "accessed 16 bytes at a time");
  __shared__ uint32_t n_long;
  const int n = (int)a.n;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const auto sum = [](uint32_t x, uint32_t y) { return x + y; };
  const auto largest = [](uint32_t x, uint32_t y) { return x > y ? x : y; };
  uint32_t total;
  if (tid == 0) n_long = 0;

  // (1) every bag that has entries leaves its number (plus one) at its first entry; the largest one up to an entry is its bag.
  // The rows and kSmallItems offsets per thread are requested together.
  int32_t row[kSmallItems];
#pragma unroll
  for (int j = 0; j < kSmallItems; ++j) row[j] = a.rows[min(tid * kSmallItems + j, n - 1)];
  static_assert(kSmallItems == 4, "a thread's items are one 16-byte LDS access");
  uint4 *const key4 = reinterpret_cast<uint4 *>(skey) + tid, *const pay4 = reinterpret_cast<uint4 *>(spay) + tid;
  *pay4 = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  for (int b0 = 0; b0 < (int)a.nbags; b0 += kSmallItems * kSmallBlock) {
    int e0[kSmallItems], e1[kSmallItems];
#pragma unroll
    for (int j = 0; j < kSmallItems; ++j) {
      const int b = min(b0 + j * kSmallBlock + tid, (int)a.nbags - 1);
      e0[j] = a.offsets[b];
      e1[j] = a.offsets[b + 1];
    }
#pragma unroll
    for (int j = 0; j < kSmallItems; ++j) {
      const int b = b0 + j * kSmallBlock + tid;
      if (b < (int)a.nbags && e0[j] < e1[j]) spay[e0[j]] = (uint32_t)b + 1u;
    }
  }
  __syncthreads();
  {
    const uint4 starts = *pay4;
    uint32_t bag[kSmallItems] = {starts.x, starts.y, starts.z, starts.w};
#pragma unroll
    for (int j = 1; j < kSmallItems; ++j) bag[j] = largest(bag[j], bag[j - 1]);
    const uint32_t before = small_excl_scan(bag[kSmallItems - 1], scan_lds, total, largest);
    uint32_t key[kSmallItems], pay[kSmallItems];
#pragma unroll
    for (int j = 0; j < kSmallItems; ++j) {
      const int e = tid * kSmallItems + j;
      bag[j] = largest(bag[j], before) - 1u;
      key[j] = row[j] >= 0 ? (uint32_t)row[j] : a.missing;
      pay[j] = kHasVals ? (uint32_t)e : bag[j];
      if (kHasVals && e < n) a.bag_of[e] = (int32_t)bag[j];
    }
    *key4 = make_uint4(key[0], key[1], key[2], key[3]);
    *pay4 = make_uint4(pay[0], pay[1], pay[2], pay[3]);
  }

  // (2) a wave owns `rounds` * 64 consecutive items and walks them in rounds of 64.  All sixteen waves share one CU, where an
  // instruction of each costs sixteen cycles, so the number of instructions is what counts: no more rounds than the batch needs,
  // four instructions per digit bit, digit counts read and written once, 16-byte LDS accesses (2560 entries, 14-bit rows: 13.7 -> 12.3 us,
  // of which some 5.5 are the two passes, 2.8 the bags, 2.2 the heads).
  const unsigned long long lane_lt = (1ull << lane) - 1ull;
  const int npass = (bits + kSmallBits - 1) / kSmallBits, per = (bits + npass - 1) / npass;
  const int rounds = (n + kSmallBlock - 1) / kSmallBlock, first = wave * rounds * kWave + lane;
  for (int p = 0; p < npass; ++p) {
    const int shift = p * per, b = min(per, bits - shift);
    const uint32_t radix = 1u << b, mask = radix - 1u;
    for (int i = tid; i < kSmallWaves << (kSmallBits - 2); i += kSmallBlock)
      reinterpret_cast<uint4 *>(&cnt[0][0])[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();                                 // the items are in place, the counters clear
    uint32_t key[kSmallItems], pay[kSmallItems], rank[kSmallItems];
#pragma unroll
    for (int r = 0; r < kSmallItems; ++r) {
      const int i = min(first + r * kWave, kSmallSort - 1);
      key[r] = skey[i];
      pay[r] = spay[i];
    }
#pragma unroll
    for (int r = 0; r < kSmallItems; ++r) {
      if (r >= rounds) break;
      const bool live = first + r * kWave < n;
      const uint32_t d = (key[r] >> shift) & mask;
      const unsigned long long alive = __ballot(live);
      uint32_t lo = (uint32_t)alive, hi = (uint32_t)(alive >> 32);
      for (int bit = 0; bit < b; ++bit) {
        const uint32_t mine = (uint32_t)((int32_t)(d << (31 - bit)) >> 31);     // all ones where the bit is set
        const unsigned long long set = __ballot(mine != 0u);
        lo = __builtin_amdgcn_bitop3_b32(lo, mine, (uint32_t)set, 0x90);        // lo & ~(mine ^ set)
        hi = __builtin_amdgcn_bitop3_b32(hi, mine, (uint32_t)(set >> 32), 0x90);
      }
      const unsigned long long peers = (unsigned long long)hi << 32 | lo;
      const uint32_t earlier = (uint32_t)__popcll(peers & lane_lt);
      uint32_t prev = 0;
      if (live) prev = cnt[wave][d];
      __builtin_amdgcn_wave_barrier();               // every lane has read its counter before the group leaders write
      if (live && earlier == 0) cnt[wave][d] = prev + (uint32_t)__popcll(peers);
      __builtin_amdgcn_wave_barrier();
      rank[r] = prev + earlier;
    }
    __syncthreads();
    uint32_t of_digit = 0, of_wave[kSmallWaves];     // thread d: the digit's items; its counters become starts in the sorted order
    if (tid < (int)radix) {
#pragma unroll
      for (int w = 0; w < kSmallWaves; ++w) {
        of_wave[w] = cnt[w][tid];
        of_digit += of_wave[w];
      }
    }
    uint32_t start = small_excl_scan(of_digit, scan_lds, total, sum);
    if (tid < (int)radix) {
#pragma unroll
      for (int w = 0; w < kSmallWaves; ++w) {
        cnt[w][tid] = start;
        start += of_wave[w];
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSmallItems; ++r) {
      const int i = first + r * kWave;
      if (r < rounds && i < n) {
        const uint32_t at = cnt[wave][(key[r] >> shift) & mask] + rank[r];
        skey[at] = key[r];
        spay[at] = pay[r];
      }
    }
    __syncthreads();
  }

  // (3) segment heads, in the order of the items
  uint32_t heads = 0;
  const int i0 = tid * kSmallItems;
  const uint4 k4 = *key4, p4 = *pay4;
  uint32_t key[kSmallItems] = {k4.x, k4.y, k4.z, k4.w};
  const uint32_t pay[kSmallItems] = {p4.x, p4.y, p4.z, p4.w};
  uint32_t prev = i0 > 0 ? skey[i0 - 1] : 0xFFFFFFFFu;
  const uint32_t first_prev = prev;
#pragma unroll
  for (int j = 0; j < kSmallItems; ++j) {
    if (i0 + j < n) pay_out[i0 + j] = pay[j];
    else key[j] = a.missing;
    heads += (key[j] != a.missing && (i0 + j == 0 || key[j] != prev)) ? 1u : 0u;
    prev = key[j];
  }
  uint32_t U;
  uint32_t u = small_excl_scan(heads, scan_lds, U, sum);   // ends with a barrier: every key is in registers, skey may go
  prev = first_prev;
#pragma unroll
  for (int j = 0; j < kSmallItems; ++j) {
    const int i = i0 + j;
    if (i < n) {
      if (key[j] != a.missing && (i == 0 || key[j] != prev)) {
        a.uniq_rows[u] = (int32_t)key[j];
        a.first_pay[u] = pay[j];
        a.seg_off[u] = i;
        skey[u] = (uint32_t)i;                       // and for the split below
        ++u;
      }
      // end of the last segment: first entry without a row, or the end of the array
      const bool end_here = key[j] == a.missing && (i == 0 || prev != a.missing), end_after = i == n - 1 && key[j] != a.missing;
      if (end_here || end_after) {
        const int end = end_here ? i : n;
        a.seg_off[U] = end;
        skey[U] = (uint32_t)end;
      }
      prev = key[j];
    }
  }
  __syncthreads();

  // long segments; their order is irrelevant to the results
  for (uint32_t v = tid; v < U; v += kSmallBlock)
    if (skey[v + 1] - skey[v] > (uint32_t)kShortMax) a.long_seg[atomicAdd(&n_long, 1u)] = (int32_t)v;
  __syncthreads();
  if (tid == 0) {
    heads_bookkeeping(a, U);
    a.ctrl->n_long = n_long;
  }
}

// Gradient sums of the sorted entries [i0, i1) seen by the lane holding columns 4*sub..4*sub+3:
//   s1 = sum x*(g_fm[b]*A_sum[b,:] + g_pool[bag,:]),  s2 = sum x*x*g_fm[b],  gw = sum x*g_lr[b]
// Accumulated in double: the first Adagrad step divides the merged gradient by |G| + eps, so a
// gradient that cancels to the order of eps must keep an absolute accuracy far below fp32's.
struct Acc {
  double v[4];
  double s2, gw;
};
__device__ inline Acc acc_zero() { Acc r; r.v[0] = r.v[1] = r.v[2] = r.v[3] = 0.0; r.s2 = 0.0; r.gw = 0.0; return r; }

// Upstream gradients of one entry.  Each is requested whether the caller passed that array or not (BwdArgs::take; an absent one
// reads the table's first row, and is then replaced by zeros): a load under a condition is waited for where the paths join,
// one after the other.
struct Upstream {
  float4 gp, as;
  float gf, gl;
};
template <int D, bool kStream = false>
__device__ inline Upstream request_upstream(const BwdArgs &a, uint32_t bag, int sub) {
  const uint32_t b = bag / (uint32_t)a.F;
  const float *gp = a.take_pool.base + (int64_t)(bag & a.take_pool.mask) * D + sub * 4;
  Upstream u;
  u.gp = kStream ? ld4_stream(gp) : ld4(gp);
  u.as = ld4(a.take_sum.base + (int64_t)(b & a.take_sum.mask) * D + sub * 4);
  u.gf = a.take_fm.base[b & a.take_fm.mask];
  u.gl = a.take_lr.base[b & a.take_lr.mask];
  return u;
}
// Waits for what was requested.
__device__ inline void arrive(Upstream &u) {
  asm volatile("" : "+v"(u.gp.x), "+v"(u.gp.y), "+v"(u.gp.z), "+v"(u.gp.w), "+v"(u.as.x), "+v"(u.as.y), "+v"(u.as.z), "+v"(u.as.w),
               "+v"(u.gf), "+v"(u.gl));
}
__device__ inline void drop_absent(const BwdArgs &a, Upstream &u) {
  if (!a.g_pool) u.gp = f4zero();
  if (!a.g_fm) { u.as = f4zero(); u.gf = 0.f; }
  if (!a.g_lr) u.gl = 0.f;
}
__device__ inline void add_upstream(const Upstream &u, float x, Acc &acc) {
  const double xd = (double)x;
  const double xg = xd * (double)u.gf;
  acc.v[0] += xd * (double)u.gp.x + xg * (double)u.as.x;
  acc.v[1] += xd * (double)u.gp.y + xg * (double)u.as.y;
  acc.v[2] += xd * (double)u.gp.z + xg * (double)u.as.z;
  acc.v[3] += xd * (double)u.gp.w + xg * (double)u.as.w;
  acc.s2 += xd * xg;
  acc.gw += xd * (double)u.gl;
}

// Adds the terms of up to U entries whose bags (and values) are already known (a dead entry has some valid bag): all their
// upstream gradient rows are requested before the first is used.
template <int D, int U>
__device__ inline void accumulate_batch(const BwdArgs &a, const uint32_t (&bag)[U], const bool (&live)[U],
                                        const float (&x)[U], int sub, Acc &acc) {
  Upstream u[U];
#pragma unroll
  for (int k = 0; k < U; ++k) u[k] = request_upstream<D>(a, bag[k], sub);
#pragma unroll
  for (int k = 0; k < U; ++k) arrive(u[k]);
#pragma unroll
  for (int k = 0; k < U; ++k) {
    if (!live[k]) continue;
    drop_absent(a, u[k]);
    add_upstream(u[k], x[k], acc);
  }
}

// Bags (and values) of the sorted entries i .. i+U-1, clipped at i1.
template <bool kHasVals, int U>
__device__ inline void load_batch_meta(const BwdArgs &a, uint32_t i, uint32_t i1, uint32_t (&bag)[U], bool (&live)[U], float (&x)[U]) {
#pragma unroll
  for (int k = 0; k < U; ++k) {
    live[k] = i + k < i1;                                     // unsigned, as where it is called from: see entry_ahead
    uint32_t p = live[k] ? a.pay_sorted[i + k] : 0u;
    x[k] = 1.f;
    if (kHasVals) {
      if (live[k]) x[k] = a.vals[p];
      p = live[k] ? (uint32_t)a.bag_of[p] : 0u;
    }
    bag[k] = p;
  }
}

// Sums over the sorted entries [i0, i1), U at a time; the payloads of the next U entries are requested
// before the gradient rows of the current ones, so a batch costs one memory round trip, not two.
template <int D, bool kHasVals, int U>
__device__ inline void reduce_entries(const BwdArgs &a, uint32_t i0, uint32_t i1, int sub, Acc &acc) {
  uint32_t nbag[U];
  bool nlive[U];
  float nx[U];
  if (i0 < i1) load_batch_meta<kHasVals, U>(a, i0, i1, nbag, nlive, nx);
  for (uint32_t i = i0; i < i1; i += U) {
    uint32_t bag[U];
    bool live[U];
    float x[U];
#pragma unroll
    for (int k = 0; k < U; ++k) { bag[k] = nbag[k]; live[k] = nlive[k]; x[k] = nx[k]; }
    if (i + U < i1) load_batch_meta<kHasVals, U>(a, i + U, i1, nbag, nlive, nx);
    accumulate_batch<D, U>(a, bag, live, x, sub, acc);
  }
}

// Pre-update state of one row as seen by the lane that owns columns 4*sub..4*sub+3 (sub 0 also
// owns the LR weight).  Loaded before the gradient reduction so that the row's memory latency
// overlaps the gathers of the upstream gradients.
struct RowState {
  float4 v, s, s2;      // latent columns and their first / second state arrays
  float w, aw, aw2;     // LR weight and its state
};

// kSecond = false: the caller knows that no second state array is in use (SGD, Adagrad), which frees its registers.
template <int D, bool kSecond = true>
__device__ inline RowState load_row(const BwdArgs &a, int row, int sub) {
  RowState st;
  st.v = ld4_stream(a.emb + (int64_t)row * D + sub * 4);
  st.s = f4zero();
  st.s2 = f4zero();
  st.w = st.aw = st.aw2 = 0.f;
  if (a.opt_emb == DES_OPT_ADAGRAD || a.opt_emb == DES_OPT_ADAM)
    st.s = ld4_stream(a.acc_emb + (int64_t)row * D + sub * 4);
  if (kSecond && a.opt_emb == DES_OPT_ADAM) st.s2 = ld4_stream(a.acc2_emb + (int64_t)row * D + sub * 4);
  if (sub == 0 && a.opt_w != DES_OPT_NONE) {
    st.w = a.w[row];
    if (a.opt_w != DES_OPT_SGD) st.aw = a.acc_w[row];
    if (kSecond && (a.opt_w == DES_OPT_ADAM || a.opt_w == DES_OPT_FTRL)) st.aw2 = a.acc2_w[row];
  }
  return st;
}

__device__ inline float adam_step(const BwdArgs &a, float g, float &m, float &v) {
  m = a.b1 * m + (1.f - a.b1) * g;
  v = a.b2 * v + (1.f - a.b2) * g * g;
  return a.lr * (m * a.c1) / (sqrtf(v * a.c2) + a.eps);
}

// Apply the merged gradient of one row.  The merged gradient is formed in double and rounded
// once; the optimizer arithmetic itself is well conditioned and runs in fp32 (FTRL, one scalar
// per row with a difference of square roots, in double).
template <int D, bool kSecond = true>
__device__ inline void apply_row(const BwdArgs &a, int64_t u, int row, int sub, const RowState &st, const Acc &acc) {
  const float4 v = st.v;
  const float4 G = make_float4((float)(acc.v[0] - (double)v.x * acc.s2), (float)(acc.v[1] - (double)v.y * acc.s2),
                               (float)(acc.v[2] - (double)v.z * acc.s2), (float)(acc.v[3] - (double)v.w * acc.s2));
  const float gw = (float)acc.gw;
  float *vp = a.emb + (int64_t)row * D + sub * 4;
  if (a.merged_out) {
    float *m = a.merged_out + u * (D + 1) + sub * 4;
    m[0] = G.x; m[1] = G.y; m[2] = G.z; m[3] = G.w;
    if (sub == 0) a.merged_out[u * (D + 1) + D] = gw;
  }
  if (a.opt_emb == DES_OPT_SGD) {
    st4_stream(vp, make_float4(v.x - a.lr * G.x, v.y - a.lr * G.y, v.z - a.lr * G.z, v.w - a.lr * G.w));
  } else if (a.opt_emb == DES_OPT_ADAGRAD) {
    float4 s = st.s;
    s.x += G.x * G.x; s.y += G.y * G.y; s.z += G.z * G.z; s.w += G.w * G.w;
    st4_stream(a.acc_emb + (int64_t)row * D + sub * 4, s);
    st4_stream(vp, make_float4(v.x - a.lr * G.x / (sqrtf(s.x) + a.eps), v.y - a.lr * G.y / (sqrtf(s.y) + a.eps),
                               v.z - a.lr * G.z / (sqrtf(s.z) + a.eps), v.w - a.lr * G.w / (sqrtf(s.w) + a.eps)));
  } else if (kSecond && a.opt_emb == DES_OPT_ADAM) {
    float4 m = st.s, q = st.s2;
    const float dx = adam_step(a, G.x, m.x, q.x), dy = adam_step(a, G.y, m.y, q.y);
    const float dz = adam_step(a, G.z, m.z, q.z), dw = adam_step(a, G.w, m.w, q.w);
    st4_stream(a.acc_emb + (int64_t)row * D + sub * 4, m);
    st4_stream(a.acc2_emb + (int64_t)row * D + sub * 4, q);
    st4_stream(vp, make_float4(v.x - dx, v.y - dy, v.z - dz, v.w - dw));
  }
  if (sub == 0) {
    if (a.opt_w == DES_OPT_SGD) {
      a.w[row] = st.w - a.lr * gw;
    } else if (a.opt_w == DES_OPT_ADAGRAD) {
      const float aw = st.aw + gw * gw;
      a.acc_w[row] = aw;
      a.w[row] = st.w - a.lr * gw / (sqrtf(aw) + a.eps);
    } else if (kSecond && a.opt_w == DES_OPT_ADAM) {
      float m = st.aw, q = st.aw2;
      const float d = adam_step(a, gw, m, q);
      a.acc_w[row] = m;
      a.acc2_w[row] = q;
      a.w[row] = st.w - d;
    } else if (kSecond && a.opt_w == DES_OPT_FTRL) {
      const double g = acc.gw, n0 = (double)st.aw, alpha = (double)a.f_alpha;
      const double n1 = n0 + g * g;
      const double sigma = (sqrt(n1) - sqrt(n0)) / alpha;
      const double z = (double)st.aw2 + g - sigma * (double)st.w;
      const double l1 = (double)a.f_l1;
      const double wn = fabs(z) <= l1 ? 0.0
                                      : -(z - (z > 0.0 ? l1 : -l1)) / (((double)a.f_beta + sqrt(n1)) / alpha + (double)a.f_l2);
      a.acc_w[row] = (float)n1;
      a.acc2_w[row] = (float)z;
      a.w[row] = (float)wn;
    }
  }
}

// (4a) one lane group per segment; long segments are left to the chunked path.  The segment's
// bounds, row and first payload arrive together; the row state and the first entry's upstream
// gradients are then fetched together, so a one-entry segment costs two memory round trips.
// All gathers are unconditional and waited for once per step, ahead of the row's stores: with a condition around each (an
// array the caller did not pass, an entry past the end) a step of two entries waited four times, and a segment's first
// accesses behind the previous one's stores.  8.0e6 entries of 64 floats, 1.0e6 short segments 387 -> 341 us (their 1.6 GB at
// 4.7 TB/s), 1.05e8 of 64 12.9 -> 11.5 ms, 8.2e6 of 32 128 -> 117 us, 3.7e5 of 32 with values and Adam 39.4 -> 28.5.  (Those 1.05e8 on a
// table of 6e7 rows; on one of 3e8 15.05 -> 14.86 ms: 104 GB then go through the fabric, at 7.0 TB/s, whatever waits for what.)
// Compiled for five waves per SIMD (up to 88 of 96 vector registers), two entries at a time: with six 395 us and 12.1 ms
// at those sizes, with four entries at a time 403 us and 13.1 ms, with four entries and four waves 341 us and 11.7 ms.
// The second state array's registers do
// not fit in 96, so those variants are compiled for four waves: D = 32, Adam, 4.8e5 / 1.9e6 / 7.7e6 entries
// 50.7 -> 45.4, 101 -> 90, 245 -> 224 us (before the gathers were freed of conditions, as the next).  Up to D = 16 they also have
// room for four entries at a time: FTRL with
// Adagrad, D = 16, same sizes: 54.7 -> 45.5, 110 -> 87, 270 -> 217 us (two at a time: 48.7, 90, 232; at D = 32 four lose).
// kSecond: an optimizer with a second state array (Adam, FTRL) may be in use.
template <int D, bool kHasVals, bool kSecond>
__device__ inline void update_short(const BwdArgs &a, uint32_t block, uint32_t blocks) {
  constexpr int G = D / 4;
  constexpr int U = kSecond && (D == 8 || D == 16) ? 4 : 2;
  const int64_t gid = (int64_t)block * kBlock + threadIdx.x;
  const int sub = (int)(gid % G);
  const int64_t ngroups = (int64_t)blocks * kBlock / G;
  const int64_t n_uniq = a.ctrl->n_uniq;
  if (gid == 0 && a.n_uniq_out) *a.n_uniq_out = n_uniq;
  // grid-stride over the segments: the grid is sized on the host for the chip, not for the (device-side) segment count.
  // The bounds, row and first payload of the lane group's next segment are requested while the current one is being
  // worked on, which takes one of the two dependent round trips per segment off the critical path.
  int64_t u = gid / G;
  int i0_n = 0, i1_n = 0, row_n = 0;
  uint32_t p0_n = 0;
  if (u < n_uniq) { i0_n = a.seg_off[u]; i1_n = a.seg_off[u + 1]; row_n = a.uniq_rows[u]; p0_n = a.first_pay[u]; }
  for (; u < n_uniq; u += ngroups) {
    const int i0 = i0_n, i1 = i1_n;
    const int row = row_n;
    const uint32_t p0 = p0_n;
    {
      const int64_t un = u + ngroups;
      if (un < n_uniq) { i0_n = a.seg_off[un]; i1_n = a.seg_off[un + 1]; row_n = a.uniq_rows[un]; p0_n = a.first_pay[un]; }
    }
    const int len = i1 - i0;
    if (len > kShortMax) continue;
    const int rest = i1 - 1;                               // the segment's last entry: what a dead lane or entry reads
    // The payloads of the next G entries are fetched lane by lane in the same round trip as the row state and
    // the first entry's gradients, so a segment of up to G+1 entries costs 2 + ceil((len-1)/U) round trips.
    uint32_t mine = G >= U ? a.pay_sorted[entry_ahead(i0, 1 + sub, rest)] : 0u;
    RowState st = load_row<D, kSecond>(a, row, sub);
    float x0 = 1.f;
    uint32_t bag0 = p0;
    if (kHasVals) { x0 = a.vals[p0]; bag0 = (uint32_t)a.bag_of[p0]; }
    Acc acc = acc_zero();
    {
      Upstream first = request_upstream<D, true>(a, bag0, sub);
      arrive(first);
      // and for all that was requested before it, so that nothing below waits behind this segment's stores
      asm volatile("" : "+v"(i0_n), "+v"(i1_n), "+v"(row_n), "+v"(p0_n), "+v"(mine));
      drop_absent(a, first);
      add_upstream(first, x0, acc);
    }
    if (G >= U) {
      float myx = 1.f;
      const int glane = (int)(threadIdx.x & (kWave - 1)) - sub;       // first lane of this group in the wave
      for (int base = 1; base < len; base += G) {
        if (base > 1) mine = a.pay_sorted[entry_ahead(i0, base + sub, rest)];
        if (kHasVals) {
          myx = a.vals[mine];
          mine = (uint32_t)a.bag_of[mine];
        }
        const int cnt = min(G, len - base);
        for (int j0 = 0; j0 < cnt; j0 += U) {
          uint32_t bag[U];
          bool live[U];
          float x[U];
#pragma unroll
          for (int k = 0; k < U; ++k) {
            live[k] = j0 + k < cnt;
            bag[k] = __shfl(mine, glane + ((j0 + k) & (G - 1)), kWave);
            x[k] = kHasVals ? __shfl(myx, glane + ((j0 + k) & (G - 1)), kWave) : 1.f;
          }
          accumulate_batch<D, U>(a, bag, live, x, sub, acc);
        }
      }
    } else {
      reduce_entries<D, kHasVals, U>(a, i0 + 1, i1, sub, acc);
    }
    apply_row<D, kSecond>(a, u, row, sub, st, acc);
  }
}

// What one wave needs to walk a stretch of a long segment: the lane groups take equal runs of a batch of kBatch entries.
template <int D>
struct Walk {
  static constexpr int G = D / 4, NG = kWave / G;
  static constexpr int U = 4;                                 // gradient rows in flight per lane
  static constexpr int kBatch = NG * (G > U ? G : U), kLoads = kBatch / kWave;
  uint2 bag[kBatch];                                          // (bag, sample) of a batch's entries
  float2 x[kBatch];                                           // their (value, g_fm)
};

// Sums over the sorted entries [lo, hi) (at least one), the same in every lane group.
// A lane loads, divides and adds up what an entry needs once (bag, sample, value, g_fm,
// g_lr) and leaves the rest to read in LDS; no gather is under a condition, so a step of U entries is waited for once: 8.2e6
// entries of 32 floats 165 -> 150 us, 3.7e5 of 32 with values 17.3 -> 14.4, 8.0e6 of 64 366 -> 359.  U = 2 / 8 (150 / 162,
// 15.2 / 14.9, 358 / 365) and six waves per SIMD (169, 20.8, 380) are no better.
template <int D, bool kHasVals>
__device__ inline Acc walk_entries(const BwdArgs &a, uint32_t lo, uint32_t hi, Walk<D> &lds) {
  constexpr int G = Walk<D>::G, NG = Walk<D>::NG, U = Walk<D>::U, kBatch = Walk<D>::kBatch, kLoads = Walk<D>::kLoads;
  uint2 (&l_bag)[kBatch] = lds.bag;
  float2 (&l_x)[kBatch] = lds.x;
  const int lane = threadIdx.x & (kWave - 1), g = lane / G, sub = lane % G;
  Acc acc = acc_zero();
  // payloads of the lane's entries of the first batch and of the one after (an index past the end reads the last entry)
  uint32_t bag[kLoads], pay_n[kLoads];
  float x[kLoads];
#pragma unroll
  for (int q = 0; q < kLoads; ++q) {
    bag[q] = a.pay_sorted[entry_ahead(lo, q * kWave + lane, hi - 1)];
    pay_n[q] = a.pay_sorted[entry_ahead(lo, kBatch + q * kWave + lane, hi - 1)];
    x[q] = 1.f;
  }
  if (kHasVals) {
#pragma unroll
    for (int q = 0; q < kLoads; ++q) { x[q] = a.vals[bag[q]]; bag[q] = (uint32_t)a.bag_of[bag[q]]; }
  }
  for (uint32_t base = lo; base < hi; base += kBatch) {
    float gf[kLoads], gl[kLoads], xc[kLoads];
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
      const uint32_t b = bag[q] / (uint32_t)a.F;
      l_bag[q * kWave + lane] = make_uint2(bag[q] & a.take_pool.mask, b & a.take_sum.mask);
      gf[q] = a.take_fm.base[b & a.take_fm.mask];
      gl[q] = a.take_lr.base[b & a.take_lr.mask];
      xc[q] = x[q];
    }
    // the next batch's, and the payloads of the one after that
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
      bag[q] = pay_n[q];
      if (kHasVals) { x[q] = a.vals[pay_n[q]]; bag[q] = (uint32_t)a.bag_of[pay_n[q]]; }
      pay_n[q] = a.pay_sorted[entry_ahead(base, 2 * kBatch + q * kWave + lane, hi - 1)];
    }
    const int cnt = min(kBatch, (int)(hi - base)), per = (cnt + NG - 1) / NG;
    const int mine = g * per, upto = min(mine + per, cnt);    // this lane group's run of the batch
    for (int k0 = 0; k0 < per; k0 += U) {
      float4 gp[U], as[U];
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const uint2 id = l_bag[min(mine + k0 + k, cnt - 1)];
        gp[k] = ld4(a.take_pool.base + (int64_t)id.x * D + sub * 4);
        as[k] = ld4(a.take_sum.base + (int64_t)id.y * D + sub * 4);
      }
#pragma unroll
      for (int k = 0; k < U; ++k)
        asm volatile("" : "+v"(gp[k].x), "+v"(gp[k].y), "+v"(gp[k].z), "+v"(gp[k].w), "+v"(as[k].x), "+v"(as[k].y), "+v"(as[k].z),
                     "+v"(as[k].w));
      if (k0 == 0) {                                          // the scalars of the lane's own entries came in the same round trip
#pragma unroll
        for (int q = 0; q < kLoads; ++q) {
          if (!a.g_fm) gf[q] = 0.f;
          if (!a.g_lr) gl[q] = 0.f;
          if (q * kWave + lane < cnt) {
            const double xd = (double)xc[q];
            acc.s2 += xd * (xd * (double)gf[q]);
            acc.gw += xd * (double)gl[q];
          }
          l_x[q * kWave + lane] = make_float2(xc[q], gf[q]);
        }
      }
      float2 f[U];
#pragma unroll
      for (int k = 0; k < U; ++k) f[k] = l_x[min(mine + k0 + k, cnt - 1)];
#pragma unroll
      for (int k = 0; k < U; ++k) {
        if (mine + k0 + k >= upto) continue;
        const double xd = kHasVals ? (double)f[k].x : 1.0;
        const double xg = xd * (double)f[k].y;
        if (!a.g_pool) gp[k] = f4zero();
        if (!a.g_fm) as[k] = f4zero();
        acc.v[0] += xd * (double)gp[k].x + xg * (double)as[k].x;
        acc.v[1] += xd * (double)gp[k].y + xg * (double)as[k].y;
        acc.v[2] += xd * (double)gp[k].z + xg * (double)as[k].z;
        acc.v[3] += xd * (double)gp[k].w + xg * (double)as[k].w;
      }
    }
    __builtin_amdgcn_wave_barrier();                          // every lane has read its entries before the next batch's are left
  }
#pragma unroll
  for (int m = 1; m < kWave; m <<= 1) {
    acc.s2 += __shfl_xor(acc.s2, m, kWave);
    acc.gw += __shfl_xor(acc.gw, m, kWave);
    if (m < G) continue;
#pragma unroll
    for (int k = 0; k < 4; ++k) acc.v[k] += __shfl_xor(acc.v[k], m, kWave);
  }
  return acc;
}

// Which chunk of its segment wave `c` takes, where the segment has the waves c0 .. c0 + nch - 1: the waves of one die (workgroups
// go round the eight dies) take consecutive chunks.  A row's entries come in batch order, so a die then sees an eighth of the
// samples of every row with eight workgroups or more, and that eighth of A_sum stays in its L2: 8.0e6 entries of 64 floats
// 359 -> 346 us, 1.05e8 of 64 2.62 -> 2.51 ms, 8.2e6 of 32 150 -> 141 us.
__device__ inline uint32_t chunk_of_wave(uint32_t c, uint32_t c0, uint32_t nch) {
  constexpr uint32_t kDies = 8, kRound = kDies * kWavesPerBlock;
  const auto before = [](uint32_t w, uint32_t die) {          // waves of the die below w
    const int in = (int)(w % kRound) - (int)(die * kWavesPerBlock);
    return w / kRound * kWavesPerBlock + (uint32_t)min(max(in, 0), kWavesPerBlock);
  };
  const uint32_t mine = c / kWavesPerBlock % kDies;
  uint32_t k = before(c, mine) - before(c0, mine);
  for (uint32_t die = 0; die < mine; ++die) k += before(c0 + nch, die) - before(c0, die);
  return k;
}

// (4b) one wave per chunk of a long segment: the wave walks the chunk in batches, its lane groups take equal runs of a
// batch, the groups' sums are combined with cross-lane shuffles, and the wave writes
// partials[c] = (s1[D], s2, gw, 0, 0) in double -- or, when the segment has no other chunk (33 .. 512 or 128
// entries, most long segments), updates the row at once.
// Bound by the gradient rows and A_sum rows that come through the fabric: with consecutive chunks on one die 2.65 GB at 7.0 TB/s for 8.0e6
// entries of 64 floats (2.72 GB before), 15.8 GB at 6.8 for 1.05e8 (17.1), 0.91 GB at 6.3 for 8.2e6 of 32 (1.07); in smaller batches by
// the round trips.
template <int D, bool kHasVals, bool kSecond>
__device__ inline void update_chunk(const BwdArgs &a, uint32_t block, Walk<D> (&lds)[kWavesPerBlock]) {
  constexpr int G = D / 4;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const uint32_t wave_no = block * kWavesPerBlock + wave;
  if (wave_no >= a.ctrl->n_chunks) return;                    // uniform per wave
  const int g = lane / G, sub = lane % G;
  const int j = a.chunk_owner[wave_no];
  const int u = a.long_seg[j];
  const int seg_lo = a.seg_off[u], seg_hi = a.seg_off[u + 1];
  const uint32_t c0 = a.long_c0[j], k_seg = chunk_of_wave(wave_no, c0, (uint32_t)chunks_of(a, seg_hi - seg_lo));
  const uint32_t c_lo = seg_lo + (k_seg << a.chunk_shift);
  const Acc acc = walk_entries<D, kHasVals>(a, c_lo, entry_ahead(c_lo, 1u << a.chunk_shift, seg_hi), lds[wave]);
  if (g == 0) {
    if (seg_hi - seg_lo <= (1 << a.chunk_shift)) {
      // the segment is this one chunk: the wave holds its whole sum and updates the row itself
      const int row = a.uniq_rows[u];
      apply_row<D, kSecond>(a, u, row, sub, load_row<D, kSecond>(a, row, sub), acc);
    } else {
      double *p = a.partials + (int64_t)(c0 + k_seg) * (D + 4);
      *reinterpret_cast<double2 *>(p + sub * 4) = make_double2(acc.v[0], acc.v[1]);
      *reinterpret_cast<double2 *>(p + sub * 4 + 2) = make_double2(acc.v[2], acc.v[3]);
      if (sub == 0) *reinterpret_cast<double2 *>(p + D) = make_double2(acc.s2, acc.gw);
    }
  }
}

// (4a) and (4b) in one launch: they touch different rows, and while either waits (a short segment for its round trips, a chunk for the
// fabric) the other's waves find work, as long as neither fills the chip by itself.  Workgroups of chunks come first from D = 32 on;
// of narrow rows, whose lane groups hold one to four lanes, the segments, whose longest then take longer than a chunk.  Both at
// once / one after the other, whole backward pass: 8.0e3 to 1.3e5 entries of any width 62 / 70 us on average, 3.7e5 of 32 with values and
// Adam 100 / 107, 1.0e6 of 16 123 / 125, 1.2e6 of 8 111 / 124, 2.7e6 of 4 173 / 203, 4.0e6 of 8 240 / 252, 8.0e6 412 / 412; above 2^20 nothing
// from D = 16 on (3.7e6 of 16 240 / 231, 8.2e6 of 32 492 / 488, 8.0e6 of 64 917 / 917) nor with second state arrays, with which this is
// compiled for a wave per SIMD less than chunks alone (1.7e6 with Adam 205 / 199).
inline bool update_at_once(int D, int64_t n, bool second) { return n <= kFewSort || (D <= 8 && !second && n <= kFewEntries); }
template <int D, bool kHasVals, bool kSecond>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kSecond || D == 4 ? 4 : 5, kSecond || D == 4 ? 4 : 5))) void k_update(
    const BwdArgs a, uint32_t n_short, uint32_t n_chunk) {
  __shared__ Walk<D> lds[kWavesPerBlock];
  if constexpr (D <= 16) {
    if (blockIdx.x < n_short) update_short<D, kHasVals, kSecond>(a, blockIdx.x, n_short);
    else update_chunk<D, kHasVals, kSecond>(a, blockIdx.x - n_short, lds);
  } else {
    if (blockIdx.x < n_chunk) update_chunk<D, kHasVals, kSecond>(a, blockIdx.x, lds);
    else update_short<D, kHasVals, kSecond>(a, blockIdx.x - n_chunk, n_short);
  }
}

template <int D, bool kHasVals, bool kSecond>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kSecond ? 4 : 5, kSecond ? 4 : 5))) void k_short_update(const BwdArgs a) {
  update_short<D, kHasVals, kSecond>(a, blockIdx.x, gridDim.x);
}

template <int D, bool kHasVals>
__global__ __launch_bounds__(kBlock, D == 4 ? 4 : 5) void k_long_partial(const BwdArgs a) {
  __shared__ Walk<D> lds[kWavesPerBlock];
  update_chunk<D, kHasVals, true>(a, blockIdx.x, lds);
}

// (4b, c) for a batch of up to kSmallSort entries: one workgroup per long segment, whose waves take equal stretches; their sums are
// added in wave order: one launch instead of two (3.4 -> 1.6 us where no segment is long).
template <int D>
constexpr int kLongSmallWaves = D == 4 ? 8 : 16;              // the waves' batches fit the LDS
template <int D, bool kHasVals>
__global__ __launch_bounds__(kLongSmallWaves<D> * kWave) void k_long_small(const BwdArgs a) {
  constexpr int G = D / 4, kWaves = kLongSmallWaves<D>;
  __shared__ Walk<D> lds[kWaves];
  __shared__ double red[kWaves][D + 2];
  const int64_t j = blockIdx.x;
  if (j >= a.ctrl->n_long) return;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, sub = lane % G;
  const int u = a.long_seg[j];
  const int seg_lo = a.seg_off[u], seg_hi = a.seg_off[u + 1], per = (seg_hi - seg_lo + kWaves - 1) / kWaves;
  const int lo = min(seg_lo + wave * per, seg_hi), hi = min(lo + per, seg_hi);
  Acc acc = acc_zero();
  if (lo < hi) acc = walk_entries<D, kHasVals>(a, lo, hi, lds[wave]);
  if (lane < G) {
#pragma unroll
    for (int k = 0; k < 4; ++k) red[wave][sub * 4 + k] = acc.v[k];
    if (sub == 0) { red[wave][D] = acc.s2; red[wave][D + 1] = acc.gw; }
  }
  __syncthreads();
  if (threadIdx.x >= G) return;
  acc = acc_zero();
#pragma unroll 2
  for (int w = 0; w < kWaves; ++w) {
#pragma unroll
    for (int k = 0; k < 4; ++k) acc.v[k] += red[w][sub * 4 + k];
    acc.s2 += red[w][D];
    acc.gw += red[w][D + 1];
  }
  const int row = a.uniq_rows[u];
  apply_row<D>(a, u, row, sub, load_row<D>(a, row, sub), acc);
}

// (4b') Segments of more than kMidFan chunks (rows that take a sizeable share of a skewed batch): one wave per
// group of kMidFan consecutive chunk partials adds them up in place, into the group's first slot, so that the
// per-segment combine below walks nch / kMidFan terms instead of nch.  Lane groups take the group's partials
// in strides and are combined by the same xor tree as in k_long_partial.
template <int D>
__global__ __launch_bounds__(kBlock) void k_long_mid(const BwdArgs a) {
  constexpr int G = D / 4;
  constexpr int NG = kWave / G;
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t gi = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
  if (gi >= a.ctrl->n_groups) return;                         // uniform per wave
  const int j = a.group_seg[gi];
  const int u = a.long_seg[j];
  const int nch = chunks_of(a, a.seg_off[u + 1] - a.seg_off[u]);
  const int64_t c = a.group_c[gi];
  const int rel = (int)(c - a.long_c0[j]);
  const int cnt = min(kMidFan, nch - rel);
  const int g = lane / G, sub = lane % G;
  Acc acc = acc_zero();
  for (int k = g; k < cnt; k += NG) {
    const double *p = a.partials + (c + k) * (D + 4);
    const double2 lo = *reinterpret_cast<const double2 *>(p + sub * 4);
    const double2 hi = *reinterpret_cast<const double2 *>(p + sub * 4 + 2);
    const double2 t = *reinterpret_cast<const double2 *>(p + D);
    acc.v[0] += lo.x; acc.v[1] += lo.y; acc.v[2] += hi.x; acc.v[3] += hi.y;
    acc.s2 += t.x; acc.gw += t.y;                             // the same two values in every lane group's sub lanes
  }
#pragma unroll
  for (int m = G; m < kWave; m <<= 1) {
#pragma unroll
    for (int k = 0; k < 4; ++k) acc.v[k] += __shfl_xor(acc.v[k], m, kWave);
    acc.s2 += __shfl_xor(acc.s2, m, kWave);
    acc.gw += __shfl_xor(acc.gw, m, kWave);
  }
  // every partial of the group has been read by this wave's loads above (the shuffles waited for them)
  if (g == 0) {
    double *p = a.partials + c * (D + 4);
    *reinterpret_cast<double2 *>(p + sub * 4) = make_double2(acc.v[0], acc.v[1]);
    *reinterpret_cast<double2 *>(p + sub * 4 + 2) = make_double2(acc.v[2], acc.v[3]);
    if (sub == 0) *reinterpret_cast<double2 *>(p + D) = make_double2(acc.s2, acc.gw);
  }
}

// (4c) one workgroup per long segment of several chunks: lane groups stride over the chunk partials, an
// LDS tree combines the groups, group 0 updates the row
template <int D>
__global__ __launch_bounds__(kBlock) void k_long_final(const BwdArgs a) {
  constexpr int G = D / 4;
  constexpr int NGB = kBlock / G;           // lane groups per workgroup
  __shared__ double red[NGB][D + 4];
  const int grp = threadIdx.x / G, sub = threadIdx.x % G;
  const long long NM = a.ctrl->n_multi;      // one-chunk segments were updated by the wave that reduced their chunk
  for (int64_t jj = blockIdx.x; jj < NM; jj += gridDim.x) {
    const int j = a.multi_seg[jj];
    const int u = a.long_seg[j];
    const int nch = chunks_of(a, a.seg_off[u + 1] - a.seg_off[u]);
    const double *p0 = a.partials + (int64_t)a.long_c0[j] * (D + 4);
    const int step = nch > kMidFan ? kMidFan : 1;      // k_long_mid left one sum per kMidFan chunks
    Acc acc = acc_zero();
    for (int c = grp * step; c < nch; c += NGB * step) {
      const double *p = p0 + (int64_t)c * (D + 4);
      const double2 lo = *reinterpret_cast<const double2 *>(p + sub * 4);
      const double2 hi = *reinterpret_cast<const double2 *>(p + sub * 4 + 2);
      acc.v[0] += lo.x; acc.v[1] += lo.y; acc.v[2] += hi.x; acc.v[3] += hi.y;
      if (sub == 0) {
        const double2 t = *reinterpret_cast<const double2 *>(p + D);
        acc.s2 += t.x; acc.gw += t.y;
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) red[grp][sub * 4 + k] = acc.v[k];
    if (sub == 0) { red[grp][D] = acc.s2; red[grp][D + 1] = acc.gw; }
    __syncthreads();
    for (int h = NGB / 2; h >= 1; h >>= 1) {
      if (grp < h) {
#pragma unroll
        for (int k = 0; k < 4; ++k) red[grp][sub * 4 + k] += red[grp + h][sub * 4 + k];
        if (sub == 0) { red[grp][D] += red[grp + h][D]; red[grp][D + 1] += red[grp + h][D + 1]; }
      }
      __syncthreads();
    }
    if (grp == 0) {
      Acc tot;
#pragma unroll
      for (int k = 0; k < 4; ++k) tot.v[k] = red[0][sub * 4 + k];
      tot.s2 = red[0][D];
      tot.gw = red[0][D + 1];
      const int row = a.uniq_rows[u];
      apply_row<D>(a, u, row, sub, load_row<D>(a, row, sub), tot);
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(kBlock) void k_export(const BwdArgs a) {
  const long long U = a.ctrl->n_uniq;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < U; u += stride) {
    const int row = a.uniq_rows[u];
    if (a.uniq_rows_out) a.uniq_rows_out[u] = row;
    if (a.uniq_keys_out) a.uniq_keys_out[u] = a.row_keys[row];
    if (a.counts_out) a.counts_out[u] = a.seg_off[u + 1] - a.seg_off[u];
  }
}

__global__ void k_set_i64(int64_t *p, int64_t v) { *p = v; }

inline unsigned blocks_for(int64_t threads, int64_t cap = 1ll << 30) {
  int64_t g = (threads + kBlock - 1) / kBlock;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (unsigned)g;
}

template <int D, bool kHasVals>
void launch_update(const BwdArgs &a, hipStream_t s) {
  constexpr int G = D / 4;
  const int64_t max_long = a.n / (kShortMax + 1) + 1;
  const int64_t max_chunks = (a.n >> a.chunk_shift) + max_long + 1;
  const bool second = a.opt_emb == DES_OPT_ADAM || a.opt_w == DES_OPT_ADAM || a.opt_w == DES_OPT_FTRL;
  // multiples of eight: consecutive workgroups go round the dies, on which chunk_of_wave counts
  const auto eights = [](unsigned blocks) { return (blocks + 7) / 8 * 8; };
  const unsigned n_short = eights(blocks_for(a.n * G, kShortGrid)), n_chunk = eights(blocks_for(max_chunks * kWave));
  const dim3 block(kBlock);
  if (a.n > kSmallSort && update_at_once(D, a.n, second)) {
    ProfScope ps(KID_UPDATE, s);
    if (second) hipLaunchKernelGGL((k_update<D, kHasVals, true>), dim3(n_short + n_chunk), block, 0, s, a, n_short, n_chunk);
    else hipLaunchKernelGGL((k_update<D, kHasVals, false>), dim3(n_short + n_chunk), block, 0, s, a, n_short, n_chunk);
  } else {
    {
      ProfScope ps(KID_SHORT_UPDATE, s);
      if (second) hipLaunchKernelGGL((k_short_update<D, kHasVals, true>), dim3(n_short), block, 0, s, a);
      else hipLaunchKernelGGL((k_short_update<D, kHasVals, false>), dim3(n_short), block, 0, s, a);
    }
    ProfScope ps(KID_LONG_PARTIAL, s);
    if (a.n <= kSmallSort) {
      hipLaunchKernelGGL((k_long_small<D, kHasVals>), dim3((unsigned)max_long), dim3(kLongSmallWaves<D> * kWave), 0, s, a);
      return;
    }
    hipLaunchKernelGGL((k_long_partial<D, kHasVals>), dim3(n_chunk), block, 0, s, a);
  }
  {
    ProfScope ps(KID_LONG_FINAL, s);
    const int64_t chunk = 1ll << a.chunk_shift, max_multi = a.n / (chunk + 1) + 1;
    const int64_t max_groups = 3 * (a.n / (chunk * kMidFan)) + 4;   // sum of ceil(chunks / kMidFan) over those segments
    if (a.n > chunk * kMidFan)          // a smaller batch cannot hold a segment of that many chunks
      hipLaunchKernelGGL(k_long_mid<D>, dim3(blocks_for(max_groups * kWave)), dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL(k_long_final<D>, dim3((unsigned)(max_multi < 8192 ? max_multi : 8192)), dim3(kBlock), 0, s, a);
  }
}

template <int D>
void launch_update_v(const BwdArgs &a, hipStream_t s) {
  if (a.vals) launch_update<D, true>(a, s); else launch_update<D, false>(a, s);
}

struct Layout {
  size_t key_a, key_b, pay_a, pay_b, bag_of, seg_off, uniq_rows, first_pay, head_sums, long_seg, long_c0, chunk_owner, partials, sort_scratch, total;
};

Layout layout_for(int D, int64_t n) {
  const size_t m = (size_t)(n > 0 ? n : 1);
  const size_t max_long = m / (kShortMax + 1) + 1, max_chunks = (m >> kChunkShift) + max_long + 1;
  Layout L;
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o += align_up(bytes, 256); return at; };
  L.key_a = take(m * 4); L.key_b = take(m * 4); L.pay_a = take(m * 4); L.pay_b = take(m * 4);
  L.bag_of = take(m * 4);
  L.seg_off = take((m + 1) * 4); L.uniq_rows = take(m * 4); L.first_pay = take(m * 4 > csr_scratch_bytes(n) ? m * 4 : csr_scratch_bytes(n));
  L.head_sums = take(((m + kHeadTile - 1) / kHeadTile + 1) * 4);
  L.long_seg = take(max_long * 4); L.long_c0 = take(max_long * 4);
  L.chunk_owner = take(max_chunks * 4);
  L.partials = take(max_chunks * (size_t)(D + 4) * 8);
  L.sort_scratch = take(sort_scratch_bytes(n));       // right behind the partials, see sort_stage
  // Room for the lists of segments that now lie in the sorted keys: the workspace also bounds how many rows
  // des_table_compact takes, which is to stay what it was.
  constexpr size_t kChunk = (size_t)1 << kChunkShift;
  take((m / (kChunk + 1) + 1) * 4);
  for (int i = 0; i < 2; ++i) take((3 * (m / (kChunk * kMidFan)) + 4) * 4);
  L.total = o;
  return L;
}

int bits_for(uint64_t max_value) {
  int b = 1;
  while (b < 32 && (max_value >> b) != 0) ++b;
  return b;
}

// Row-sorting half of the backward pass: CSR -> (row, bag) pairs, sort by row, segment heads, split into
// short and long segments.  Needs the batch and its rows only, not the gradients.  Returns which sort
// buffer holds the sorted pairs.
// The sorted keys' buffer, and in it the lists that the split of long segments leaves once the keys have served: up to n/129
// segments of several chunks, and 3n/8192 + 4 groups in batches of more than 8192 entries.
void set_sorted_keys(BwdArgs &a, uint32_t *keys) {
  a.key_sorted = keys;
  a.multi_seg = (int32_t *)keys;
  a.group_seg = (int32_t *)(keys + a.n / 2);
  a.group_c = keys + a.n / 4 * 3;
}

int sort_stage(des_table *t, BwdArgs &a, const Layout &L, hipStream_t s) {
  char *ws = t->ws;
  const int64_t n = a.n;
  uint32_t *key_a = (uint32_t *)(ws + L.key_a), *pay_a = (uint32_t *)(ws + L.pay_a);
  const int bits = bits_for((uint64_t)t->cfg.capacity_rows);
  if (n <= kSmallSort && a.nbags <= kSmallBags) {
    ProfScope ps(KID_SORT_SCATTER, s);
    a.pay_sorted = pay_a;
    set_sorted_keys(a, key_a);
    if (a.vals) hipLaunchKernelGGL(k_sort_small<true>, dim3(1), dim3(kSmallBlock), 0, s, a, pay_a, bits);
    else hipLaunchKernelGGL(k_sort_small<false>, dim3(1), dim3(kSmallBlock), 0, s, a, pay_a, bits);
    return 0;
  }
  // the tiles' first bags lie where the segments' first payloads come later
  const SortCsr csr{a.rows, a.offsets, a.nbags, a.missing, (uint32_t *)(ws + L.first_pay), a.vals ? a.bag_of : nullptr};
  const bool from_csr = bags_by_sort(n, a.nbags);
  if (!from_csr) {
    ProfScope ps(KID_EXPAND, s);
    const dim3 grid(blocks_for(a.nbags, 1 << 20)), block(kBlock);     // one workgroup per kBlock bags
    if (a.vals) hipLaunchKernelGGL(k_expand<true>, grid, block, 0, s, a, key_a, pay_a);
    else hipLaunchKernelGGL(k_expand<false>, grid, block, 0, s, a, key_a, pay_a);
  }
  SortBuffers sb{key_a, (uint32_t *)(ws + L.key_b), pay_a, (uint32_t *)(ws + L.pay_b)};
  // what the later steps fill serves as scratch here: the unique rows for the digits' totals, the chunk sums, with the sort
  // scratch right behind them, for the finer tile counts of a small batch (2 bytes per entry; the chunk sums alone are
  // 8*(D+4)*(1/33 + 1/512) >= 2.06 bytes per entry)
  const int side = radix_sort_u32_pairs(sb, n, bits, ws + L.sort_scratch, ws + L.partials, (uint32_t *)(ws + L.uniq_rows),
                                        from_csr ? &csr : nullptr, s);
  set_sorted_keys(a, (uint32_t *)(ws + (side ? L.key_b : L.key_a)));
  a.pay_sorted = (uint32_t *)(ws + (side ? L.pay_b : L.pay_a));
  if (n <= kFewHeads) {
    ProfScope ps(KID_HEADS, s);
    hipLaunchKernelGGL(k_heads_few, dim3(1), dim3(kFewHeadsBlock), 0, s, a);
    return side;
  }
  {
    ProfScope ps(KID_HEADS, s);
    const int64_t nb = (n + kHeadTile - 1) / kHeadTile;
    hipLaunchKernelGGL(k_heads_count, dim3((unsigned)nb), dim3(kBlock), 0, s, a);
    if (nb > kHeadsSelfPrefix) {                  // many tiles: one device-wide scan of the counts
      exclusive_scan_u32(a.head_sums, nb, a.head_sums + nb, ws + L.sort_scratch, s);
      hipLaunchKernelGGL(k_heads_finish, dim3(1), dim3(1), 0, s, a, (const uint32_t *)(a.head_sums + nb));
      hipLaunchKernelGGL(k_heads_write<false>, dim3((unsigned)nb), dim3(kBlock), 0, s, a);
    } else {
      hipLaunchKernelGGL(k_heads_write<true>, dim3((unsigned)nb), dim3(kBlock), 0, s, a);
    }
  }
  {
    ProfScope ps(KID_CLASSIFY, s);
    hipLaunchKernelGGL(k_classify, dim3((unsigned)((n + kHeadTile - 1) / kHeadTile)), dim3(kBlock), 0, s, a);
    const int64_t max_long = n / (kShortMax + 1) + 1;
    // at most eight workgroups per CU: 65536 of them, nearly all without a segment, took 17 us to start and end
    hipLaunchKernelGGL(k_chunk_owner, dim3((unsigned)(max_long < 2048 ? max_long : 2048)), dim3(kBlock), 0, s, a);
  }
  return side;
}

void batch_args(des_table *t, const des_batch_t *b, const int32_t *rows, const Layout &L, BwdArgs &a) {
  char *ws = t->ws;
  a = BwdArgs{};
  a.offsets = b->offsets; a.vals = b->vals; a.rows = rows;
  a.n = b->nnz; a.nbags = b->B * (int64_t)b->F; a.F = b->F;
  a.missing = (uint32_t)t->cfg.capacity_rows;
  a.emb = t->cfg.emb; a.w = t->cfg.w; a.acc_emb = t->cfg.acc_emb; a.acc_w = t->cfg.acc_w;
  a.acc2_emb = t->cfg.acc2_emb; a.acc2_w = t->cfg.acc2_w;
  a.row_keys = t->cfg.row_keys; a.ctrl = t->ctrl;
  a.bag_of = (int32_t *)(ws + L.bag_of);
  a.seg_off = (int32_t *)(ws + L.seg_off); a.uniq_rows = (int32_t *)(ws + L.uniq_rows);
  a.first_pay = (uint32_t *)(ws + L.first_pay);
  a.head_sums = (uint32_t *)(ws + L.head_sums);
  a.long_seg = (int32_t *)(ws + L.long_seg); a.long_c0 = (uint32_t *)(ws + L.long_c0);
  a.chunk_shift = chunk_shift_for(b->nnz);
  a.chunk_owner = (int32_t *)(ws + L.chunk_owner); a.partials = (double *)(ws + L.partials);
}

}  // namespace

size_t backward_ws_bytes(int D, int64_t max_n) { return layout_for(D, max_n).total; }

des_status_t backward_prepare_launch(des_table *t, const des_batch_t *b, const int32_t *rows, hipStream_t s) {
  t->prep.valid = false;
  if (b->nnz == 0) return DES_OK;
  const Layout L = layout_for(t->cfg.dim, b->nnz);
  BwdArgs a;
  batch_args(t, b, rows, L, a);
  const int side = sort_stage(t, a, L, s);
  if (hipGetLastError() != hipSuccess) return DES_ERR_DEVICE;
  t->prep.valid = true;
  t->prep.offsets = b->offsets; t->prep.rows = rows; t->prep.vals = b->vals;
  t->prep.nnz = b->nnz; t->prep.B = b->B; t->prep.F = b->F; t->prep.side = side;
  return DES_OK;
}

des_status_t backward_launch(des_table *t, const des_batch_t *b, const int32_t *rows, const des_backward_io_t *io,
                             const des_optimizer_t *opt, hipStream_t s) {
  const int64_t n = b->nnz;
  const int D = t->cfg.dim;
  const bool prepared = t->prep.valid && t->prep.offsets == b->offsets && t->prep.rows == rows &&
                        t->prep.vals == b->vals && t->prep.nnz == n && t->prep.B == b->B && t->prep.F == b->F;
  t->prep.valid = false;                          // the update consumes the sorted form
  if (n == 0) {
    if (io->n_uniq_out) hipLaunchKernelGGL(k_set_i64, dim3(1), dim3(1), 0, s, io->n_uniq_out, (int64_t)0);
    return DES_OK;
  }
  const Layout L = layout_for(D, n);
  char *ws = t->ws;
  BwdArgs a;
  batch_args(t, b, rows, L, a);
  a.g_lr = io->g_lr; a.g_fm = io->g_fm; a.A_sum = io->A_sum; a.g_pool = io->g_pool;
  const auto take = [&](const float *p) { return p ? BwdArgs::Take{p, ~0u} : BwdArgs::Take{a.emb, 0u}; };
  a.take_lr = take(a.g_lr); a.take_fm = take(a.g_fm); a.take_sum = take(a.g_fm ? a.A_sum : nullptr); a.take_pool = take(a.g_pool);
  a.opt_emb = opt->opt_emb; a.opt_w = opt->opt_w; a.lr = opt->lr; a.eps = opt->eps;
  a.b1 = opt->beta1; a.b2 = opt->beta2;
  const double t_step = (double)(opt->step > 0 ? opt->step : 1);
  a.c1 = (float)(1.0 / (1.0 - pow((double)opt->beta1, t_step)));
  a.c2 = (float)(1.0 / (1.0 - pow((double)opt->beta2, t_step)));
  a.f_alpha = opt->ftrl_alpha; a.f_beta = opt->ftrl_beta; a.f_l1 = opt->ftrl_l1; a.f_l2 = opt->ftrl_l2;
  a.uniq_rows_out = io->uniq_rows_out; a.uniq_keys_out = io->uniq_keys_out; a.counts_out = io->counts_out;
  a.merged_out = io->merged_out; a.n_uniq_out = io->n_uniq_out;
  if (prepared) {
    set_sorted_keys(a, (uint32_t *)(ws + (t->prep.side ? L.key_b : L.key_a)));
    a.pay_sorted = (uint32_t *)(ws + (t->prep.side ? L.pay_b : L.pay_a));
  } else {
    sort_stage(t, a, L, s);
  }
  switch (D) {
    case 4: launch_update_v<4>(a, s); break;
    case 8: launch_update_v<8>(a, s); break;
    case 16: launch_update_v<16>(a, s); break;
    case 32: launch_update_v<32>(a, s); break;
    case 64: launch_update_v<64>(a, s); break;
    case 128: launch_update_v<128>(a, s); break;
    case 256: launch_update_v<256>(a, s); break;
    default: return DES_ERR_INVALID_ARG;
  }
  if (io->uniq_rows_out || io->uniq_keys_out || io->counts_out) {
    ProfScope ps(KID_EXPORT, s);
    hipLaunchKernelGGL(k_export, dim3(blocks_for(n, 1 << 16)), dim3(kBlock), 0, s, a);
  }
  return hipGetLastError() == hipSuccess ? DES_OK : DES_ERR_DEVICE;
}

}  // namespace des
