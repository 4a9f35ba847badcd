// Growth and eviction of a table (Section 1, "Dynamic Features": the parameter set of a streaming
// recommender changes and grows over time; Section 5: dynamic hash table).  The paper states the
// requirement, not a mechanism.  Here the rows to keep move, in ascending row order, into a second,
// empty table of any capacity that holds them, and that table's hash slots are built from the moved
// keys: flags -> exclusive prefix sum (new row numbers) -> coalesced row copy -> parallel re-insert.
// A maintenance operation, not part of the training step: it synchronises with the host twice to
// size its launches and to refuse a target that is too small before anything is written.
//
// des_table_compact is the same eviction inside one table, for tables too large for a second copy: the kept
// rows close up towards row 0.  A kept row never moves up, so the arrays are walked in ascending chunks of
// rows: the kept rows of a chunk are gathered into a staging buffer and then stored at their new place, which
// lies at or below the chunk and holds only rows that have already been moved or dropped.  Rows before the first
// dropped one keep their place; if no kept row lies behind it, nothing moves at all.
#include "des_internal.h"

namespace des {
namespace {

inline unsigned blocks_for(int64_t n, int64_t cap = 1 << 20) {
  int64_t g = (n + kBlock - 1) / kBlock;
  return (unsigned)(g < 1 ? 1 : (g > cap ? cap : g));
}

__global__ __launch_bounds__(kBlock) void k_keep_flags(const uint8_t *__restrict__ keep, int64_t n,
                                                        unsigned long long *__restrict__ flags) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += stride)
    flags[r] = (!keep || keep[r]) ? 1ull : 0ull;
}

struct MoveArgs {
  const uint64_t *src_keys; uint64_t *dst_keys;
  const float *src_vec[3]; float *dst_vec[3];     // emb, acc_emb, acc2_emb  ([rows, D])
  const float *src_sc[3]; float *dst_sc[3];       // w, acc_w, acc2_w        ([rows])
  const uint32_t *src_aux; uint32_t *dst_aux;     // optional caller array, one word per row
  const uint8_t *keep;
  const unsigned long long *new_row;              // exclusive prefix sum of the keep flags
  int64_t n;
  int D;
};

// One lane group of D/4 lanes per source row: 16-byte loads and stores of the three vector arrays,
// lane 0 of the group moves the key, the scalars and the caller's word.  A state array that only the
// target has is zeroed for the moved rows; one that only the source has is dropped.
__global__ __launch_bounds__(kBlock) void k_move_rows(const MoveArgs a) {
  const int G = a.D / 4;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t r = gid / G;
  const int sub = (int)(gid % G);
  if (r >= a.n) return;
  if (a.keep && !a.keep[r]) return;
  const int64_t d = (int64_t)a.new_row[r];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    if (!a.dst_vec[i]) continue;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (a.src_vec[i]) v = *reinterpret_cast<const float4 *>(a.src_vec[i] + r * a.D + sub * 4);
    *reinterpret_cast<float4 *>(a.dst_vec[i] + d * a.D + sub * 4) = v;
  }
  if (sub == 0) {
    a.dst_keys[d] = a.src_keys[r];
#pragma unroll
    for (int i = 0; i < 3; ++i)
      if (a.dst_sc[i]) a.dst_sc[i][d] = a.src_sc[i] ? a.src_sc[i][r] : 0.f;
    if (a.dst_aux) a.dst_aux[d] = a.src_aux ? a.src_aux[r] : 0u;
  }
}

// Re-insert: row d's key claims the first empty slot of its probe sequence.  All keys are distinct,
// so a claimed slot is never claimed twice; the row is stored after the claim (nothing reads the
// slots until the stream has drained this kernel).
__global__ __launch_bounds__(kBlock) void k_rehash(Slot *__restrict__ slots, uint64_t slot_mask,
                                                    const uint64_t *__restrict__ row_keys, int64_t n,
                                                    Ctrl *__restrict__ ctrl) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t d = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; d < n; d += stride) {
    const uint64_t key = row_keys[d];
    uint64_t idx = mix64(key) & slot_mask;
    bool placed = false;
    for (uint64_t probe = 0; probe <= slot_mask; ++probe) {
      const unsigned long long old =
          atomicCAS(reinterpret_cast<unsigned long long *>(&slots[idx].key), kEmptyKey, key);
      if (old == kEmptyKey) {
        slots[idx].row = (int32_t)d;
        placed = true;
        break;
      }
      idx = (idx + 1) & slot_mask;
    }
    if (!placed) atomicCAS(&ctrl->status, 0, (int)DES_ERR_FULL);
  }
}

__global__ void k_set_rows(Ctrl *ctrl, long long n) { ctrl->n_rows = n; }

// In-place compaction of one per-row array of `upr` units of type T per row, rows [c0, c1).
// new_row: exclusive prefix sum of the keep flags over all n rows, new_row[n] = number of kept rows.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_compact_gather(const T *__restrict__ arr, int upr,
                                                            const uint8_t *__restrict__ keep,
                                                            const unsigned long long *__restrict__ new_row, int64_t c0,
                                                            int64_t c1, T *__restrict__ staging) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t r = c0 + gid / upr;
  const int u = (int)(gid % upr);
  if (r >= c1 || !keep[r]) return;
  staging[(int64_t)(new_row[r] - new_row[c0]) * upr + u] = arr[r * upr + u];
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_compact_store(T *__restrict__ arr, int upr,
                                                           const unsigned long long *__restrict__ new_row, int64_t c0,
                                                           int64_t c1, const T *__restrict__ staging) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t i = gid / upr;
  const int u = (int)(gid % upr);
  const int64_t first = (int64_t)new_row[c0], kept = (int64_t)new_row[c1] - first;
  if (i >= kept) return;
  arr[(first + i) * upr + u] = staging[i * upr + u];
}

// Compaction, first look at the keep flags: rows kept per tile of kKeepTile rows, a thread's eight flags by one load where they
// are aligned.
constexpr int kKeepTile = 2048;
constexpr int kKeepItems = kKeepTile / kBlock;

__device__ inline uint32_t load_keep(const uint8_t *__restrict__ keep, int64_t r0, int64_t n) {   // bit i: row r0 + i is kept
  static_assert(kKeepItems == 8, "one 8-byte load per thread");
  uint32_t bits = 0;
  if (r0 + kKeepItems <= n && ((uintptr_t)keep & 7u) == 0) {
    const uint2 v = *reinterpret_cast<const uint2 *>(keep + r0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if ((v.x >> (8 * i)) & 0xFFu) bits |= 1u << i;
      if ((v.y >> (8 * i)) & 0xFFu) bits |= 16u << i;
    }
  } else {
#pragma unroll
    for (int i = 0; i < kKeepItems; ++i)
      if (r0 + i < n && keep[r0 + i]) bits |= 1u << i;
  }
  return bits;
}

// Sum of v over the workgroup's threads before this one (and over all of them).
__device__ inline uint32_t block_sum_before(uint32_t v, uint32_t *lds, uint32_t &total) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, waves = blockDim.x / kWave;
  uint32_t inc = v;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const uint32_t o = __shfl_up(inc, off, kWave);
    if (lane >= off) inc += o;
  }
  if (lane == kWave - 1) lds[wave] = inc;
  __syncthreads();
  uint32_t base = 0, tot = 0;
  for (int w = 0; w < waves; ++w) {
    const uint32_t x = lds[w];
    if (w < wave) base += x;
    tot += x;
  }
  __syncthreads();
  total = tot;
  return base + inc - v;
}

__global__ __launch_bounds__(kBlock) void k_keep_count(const uint8_t *__restrict__ keep, int64_t n, uint32_t *__restrict__ counts) {
  __shared__ uint32_t lds[kBlock / kWave];
  const int64_t r0 = (int64_t)blockIdx.x * kKeepTile + (int64_t)threadIdx.x * kKeepItems;
  uint32_t total;
  block_sum_before(__popc(load_keep(keep, r0, n)), lds, total);
  if (threadIdx.x == 0) counts[blockIdx.x] = total;
}

// The slots are rebuilt in place, tile by tile: under linear probing a key lies between its home slot and the next empty one, so
// the slots from one empty slot to the next hold the same keys whatever the order of insertion, and fewer keys need no others.
// A tile's region runs from its first empty slot to the next tile's, here noted (kSlotTile if it has none) before any
// region is changed.  One wave per tile; the first 64 slots nearly always answer.
constexpr int kSlotTile = 1024;
__global__ __launch_bounds__(kBlock) void k_slot_bounds(const Slot *__restrict__ slots, int64_t ntiles, uint32_t *__restrict__ first_empty) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t t = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
  if (t >= ntiles) return;                                    // uniform per wave
  uint32_t at = kSlotTile;
  for (int i = 0; i < kSlotTile; i += kWave) {
    const unsigned long long empty = __ballot(slots[t * kSlotTile + i + lane].key == kEmptyKey);
    if (empty) { at = (uint32_t)(i + __ffsll(empty) - 1); break; }
  }
  if (lane == 0) first_empty[t] = at;
}

// One workgroup: turns the tiles' counts into exclusive sums, sets the table's row count and leaves for the host what it decides
// by: {rows kept, first dropped row (n if none), whether a slot tile has no empty slot}.
constexpr int kTellBlock = 1024;
__global__ __launch_bounds__(kTellBlock) void k_keep_tell(Ctrl *ctrl, const uint8_t *__restrict__ keep, int64_t n,
                                                           uint32_t *__restrict__ counts, const uint32_t *__restrict__ first_empty,
                                                           int64_t ntiles, long long *__restrict__ out) {
  __shared__ uint32_t lds[kTellBlock / kWave];
  __shared__ unsigned int first_tile, full_tiles;
  __shared__ int first_row;
  const int64_t nb = (n + kKeepTile - 1) / kKeepTile;
  if (threadIdx.x == 0) { first_tile = 0xFFFFFFFFu; full_tiles = 0; first_row = kKeepTile; }
  __syncthreads();
  // Each thread takes consecutive tiles, whose counts it adds up, and, once it knows what lies before, replaces; rows are fewer than
  // 2^31.  All loads of a step are requested together.
  constexpr int U = 4, UB = 8;
  const int64_t per = (nb + kTellBlock - 1) / kTellBlock, i0 = min(threadIdx.x * per, nb), i1 = min(i0 + per, nb);
  uint32_t sum = 0, carry;
  for (int64_t i = i0; i < i1; i += U) {
    uint32_t c[U];
#pragma unroll
    for (int j = 0; j < U; ++j) c[j] = counts[min(i + j, i1 - 1)];
#pragma unroll
    for (int j = 0; j < U; ++j) sum += i + j < i1 ? c[j] : 0u;
  }
  bool full = false;
  for (int64_t t = threadIdx.x; t < ntiles; t += UB * kTellBlock) {
    uint32_t e[UB];
#pragma unroll
    for (int j = 0; j < UB; ++j) e[j] = first_empty[min(t + j * kTellBlock, ntiles - 1)];
#pragma unroll
    for (int j = 0; j < UB; ++j) full |= e[j] >= kSlotTile;
  }
  if (full) full_tiles = 1;
  uint32_t before = block_sum_before(sum, lds, carry), dropped = 0xFFFFFFFFu;   // the thread's first tile with a dropped row
  for (int64_t i = i0; i < i1; i += U) {
    uint32_t c[U];
#pragma unroll
    for (int j = 0; j < U; ++j) c[j] = counts[min(i + j, i1 - 1)];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      if (i + j >= i1) break;
      counts[i + j] = before;
      before += c[j];
      if (c[j] < (uint32_t)min((int64_t)kKeepTile, n - (i + j) * kKeepTile)) dropped = min(dropped, (uint32_t)(i + j));
    }
  }
  // Of a wave only the lowest lane that found one says so: LDS atomics on one address run one after the other (a tile's 2048 dropped
  // rows and 600 tiles with dropped ones: 17.9 -> 5.4 us).
  const auto lowest = [](bool found) {
    const unsigned long long lanes = __ballot(found);
    return found && (int)(threadIdx.x % kWave) == __ffsll(lanes) - 1;
  };
  if (lowest(dropped != 0xFFFFFFFFu)) atomicMin(&first_tile, dropped);
  __syncthreads();
  if (first_tile != 0xFFFFFFFFu) {                            // uniform
    const int64_t r0 = (int64_t)first_tile * kKeepTile;
    static_assert(kKeepTile % kTellBlock == 0, "whole waves");
    for (int i = threadIdx.x; i < kKeepTile; i += kTellBlock)
      if (lowest(r0 + i < n && !keep[r0 + i])) atomicMin(&first_row, i);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    out[0] = (long long)carry;
    out[1] = first_tile == 0xFFFFFFFFu ? n : (long long)first_tile * kKeepTile + first_row;
    out[2] = (long long)full_tiles;
    ctrl->n_rows = (long long)carry;
  }
}

// Exclusive prefix sum of the keep flags, where rows move: new_row[n] is the number of kept rows.
__global__ __launch_bounds__(kBlock) void k_keep_rows(const uint8_t *__restrict__ keep, int64_t n, const uint32_t *__restrict__ sums,
                                                       unsigned long long *__restrict__ new_row) {
  __shared__ uint32_t lds[kBlock / kWave];
  const int64_t r0 = (int64_t)blockIdx.x * kKeepTile + (int64_t)threadIdx.x * kKeepItems;
  const uint32_t bits = load_keep(keep, r0, n);
  uint32_t total;
  uint32_t run = sums[blockIdx.x] + block_sum_before(__popc(bits), lds, total);
#pragma unroll
  for (int i = 0; i < kKeepItems; ++i) {
    if (r0 + i < n) new_row[r0 + i] = run;
    run += (bits >> i) & 1u;
    if (r0 + i == n - 1) new_row[n] = run;
  }
}

// Rebuilds one tile's region in LDS (see k_slot_bounds): drops the keys whose rows go, renumbers the others.  Rows below `lo` keep
// their number, later ones take new_row, or go if that is null.  Bound by reading and writing the slots once; clearing them and
// claiming each kept key's slot by compare-and-swap took about 310 us for 4.0e6 rows in 8.4e6
// slots; with the first look at the flags, which wrote and scanned 8 bytes a row, the whole call's kernels 440 -> 136 us.
__global__ __launch_bounds__(kBlock) void k_rebuild_slots(Slot *__restrict__ slots, uint64_t n_slots, const uint32_t *__restrict__ first_empty,
                                                           const uint8_t *__restrict__ keep,
                                                           const unsigned long long *__restrict__ new_row, int64_t lo,
                                                           Ctrl *__restrict__ ctrl) {
  __shared__ unsigned long long keys[2 * kSlotTile];
  __shared__ int32_t rows[2 * kSlotTile];
  constexpr int kItems = 2 * kSlotTile / kBlock;
  const uint64_t mask = n_slots - 1, t = blockIdx.x, ntiles = n_slots / kSlotTile;
  const uint64_t start = t * kSlotTile + first_empty[t];
  const int len = (int)((t + 1) * kSlotTile + first_empty[t + 1 < ntiles ? t + 1 : 0] - start);   // 1 .. 2 * kSlotTile - 1
  unsigned long long key[kItems];
  int32_t row[kItems];
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int i = j * kBlock + threadIdx.x;
    key[j] = kEmptyKey;
    row[j] = -1;
    if (i < len) {
      const Slot s = slots[(start + i) & mask];
      key[j] = s.key;
      row[j] = s.row;
    }
    keys[i] = kEmptyKey;
    rows[i] = -1;
  }
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    if (row[j] >= lo) row[j] = new_row && keep[row[j]] ? (int32_t)new_row[row[j]] : -1;
    if (row[j] < 0) key[j] = kEmptyKey;                       // dropped, or a key that never got a row
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    if (key[j] == kEmptyKey) continue;
    bool placed = false;
    for (uint64_t at = ((mix64(key[j]) & mask) - start) & mask; at < (uint64_t)len; ++at) {
      if (atomicCAS(&keys[at], (unsigned long long)kEmptyKey, key[j]) == kEmptyKey) {
        rows[at] = row[j];
        placed = true;
        break;
      }
    }
    if (!placed) atomicCAS(&ctrl->status, 0, (int)DES_ERR_FULL);
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int i = j * kBlock + threadIdx.x;
    if (i < len) {
      Slot s;
      s.key = keys[i]; s.row = rows[i]; s.first = 0xFFFFFFFFu;
      slots[(start + i) & mask] = s;
    }
  }
}

// empty slot = all-ones key, row -1: one 16-byte pattern of 0xFF
__global__ __launch_bounds__(kBlock) void k_fill_slots(uint4 *__restrict__ p, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const uint4 ones = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = ones;
}

// moves the kept rows among [lo, hi)
template <typename T>
void compact_array(T *arr, int upr, const uint8_t *keep, const unsigned long long *new_row, int64_t lo, int64_t hi,
                   void *staging, size_t staging_bytes, hipStream_t s) {
  if (!arr) return;
  const int64_t chunk = (int64_t)(staging_bytes / ((size_t)upr * sizeof(T)));
  for (int64_t c0 = lo; c0 < hi; c0 += chunk) {
    const int64_t c1 = c0 + chunk < hi ? c0 + chunk : hi;
    const unsigned grid = (unsigned)(((c1 - c0) * upr + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(k_compact_gather<T>, dim3(grid), dim3(kBlock), 0, s, (const T *)arr, upr, keep, new_row, c0, c1,
                       (T *)staging);
    hipLaunchKernelGGL(k_compact_store<T>, dim3(grid), dim3(kBlock), 0, s, arr, upr, new_row, c0, c1, (const T *)staging);
  }
}

__global__ __launch_bounds__(kBlock) void k_mark_seen(const int32_t *__restrict__ rows, int64_t n, uint32_t stamp,
                                                       uint32_t *__restrict__ last_seen) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) {
    const int32_t r = rows[e];
    if (r >= 0) last_seen[r] = stamp;               // entries of one row all store the same value
  }
}

__global__ __launch_bounds__(kBlock) void k_select_recent(const uint32_t *__restrict__ last_seen, int64_t n,
                                                           uint32_t min_stamp, uint8_t *__restrict__ keep) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += stride)
    keep[r] = last_seen[r] >= min_stamp ? 1 : 0;
}

// Smallest index whose value breaks the batch contract (see des_batch_validate); kept with an atomic minimum.
__global__ __launch_bounds__(kBlock) void k_validate(const int32_t *__restrict__ offsets, int64_t nbags, int64_t nnz,
                                                      const int32_t *__restrict__ rows, const Ctrl *__restrict__ ctrl,
                                                      unsigned long long *__restrict__ first_bad) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t total = nbags + 1 + (rows ? nnz : 0);
  const long long n_rows = ctrl->n_rows;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
    bool bad;
    if (i <= nbags) {
      const int32_t o = offsets[i];
      bad = (i == 0 && o != 0) || (i == nbags && (int64_t)o != nnz) || (i > 0 && o < offsets[i - 1]) || o < 0 ||
            (int64_t)o > nnz;
    } else {
      const int32_t r = rows[i - nbags - 1];
      bad = r < -1 || (long long)r >= n_rows;
    }
    if (bad) atomicMin(first_bad, (unsigned long long)i);
  }
}

bool overlap(const void *a, size_t na, const void *b, size_t nb) {
  if (!a || !b) return false;
  const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  return x < y + nb && y < x + na;
}

}  // namespace
}  // namespace des

using namespace des;

extern "C" {

des_status_t des_table_migrate_bytes(int64_t n_rows, size_t *workspace_bytes) {
  if (!workspace_bytes || n_rows < 0) return DES_ERR_INVALID_ARG;
  *workspace_bytes = 256 + align_up((size_t)(n_rows > 0 ? n_rows : 1) * 8, 256) + scan_scratch_bytes(n_rows > 0 ? n_rows : 1);
  return DES_OK;
}

des_status_t des_table_migrate(des_table_t *src, const uint8_t *keep, des_table_t *dst, const uint32_t *src_aux,
                               uint32_t *dst_aux, int64_t *n_rows_out, void *stream) {
  if (!src || !dst || src == dst) return DES_ERR_INVALID_ARG;
  const des_table_config_t &sc = src->cfg, &dc = dst->cfg;
  if (sc.dim != dc.dim || ((uintptr_t)src_aux & 3u) || ((uintptr_t)dst_aux & 3u)) return DES_ERR_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  int64_t n = 0, n_dst = 0;
  des_status_t st = des_table_size(src, &n);
  if (st != DES_OK) return st;
  st = des_table_size(dst, &n_dst);
  if (st != DES_OK) return st;
  if (n_dst != 0 || blocking_status(dst) != DES_OK || blocking_status(src) != DES_OK) return DES_ERR_INVALID_ARG;
  const size_t row_bytes = (size_t)sc.dim * 4;
  if (overlap(sc.emb, (size_t)sc.capacity_rows * row_bytes, dc.emb, (size_t)dc.capacity_rows * row_bytes) ||
      overlap(sc.row_keys, (size_t)sc.capacity_rows * 8, dc.row_keys, (size_t)dc.capacity_rows * 8) ||
      overlap(sc.w, (size_t)sc.capacity_rows * 4, dc.w, (size_t)dc.capacity_rows * 4) ||
      overlap(sc.slots, sc.slots_bytes, dc.slots, dc.slots_bytes))
    return DES_ERR_INVALID_ARG;
  if (n_rows_out) *n_rows_out = 0;
  src->last_stream = s;
  dst->last_stream = s;
  dst->prep.valid = false;
  if (n == 0) return DES_OK;
  size_t need = 0;
  (void)des_table_migrate_bytes(n, &need);
  if (dst->ws_bytes + 256 < need) return DES_ERR_WORKSPACE;
  unsigned long long *flags = (unsigned long long *)dst->ws;
  void *scan_scratch = dst->ws + align_up((size_t)n * 8, 256);
  ProfScope ps(KID_MIGRATE, s);
  hipLaunchKernelGGL(k_keep_flags, dim3(blocks_for(n)), dim3(kBlock), 0, s, keep, n, flags);
  // the total lands in the target's row counter, which is exactly what it is
  exclusive_scan_u64(flags, n, (unsigned long long *)&dst->ctrl->n_rows, scan_scratch, s);
  long long kept = 0;
  if (hipMemcpyAsync(&kept, &dst->ctrl->n_rows, sizeof(kept), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    return DES_ERR_DEVICE;
  if (kept > dc.capacity_rows) {                       // refuse before anything is moved
    hipLaunchKernelGGL(k_set_rows, dim3(1), dim3(1), 0, s, dst->ctrl, 0ll);
    (void)hipStreamSynchronize(s);
    return DES_ERR_FULL;
  }
  MoveArgs a;
  a.src_keys = sc.row_keys; a.dst_keys = dc.row_keys;
  a.src_vec[0] = sc.emb; a.src_vec[1] = sc.acc_emb; a.src_vec[2] = sc.acc2_emb;
  a.dst_vec[0] = dc.emb; a.dst_vec[1] = dc.acc_emb; a.dst_vec[2] = dc.acc2_emb;
  a.src_sc[0] = sc.w; a.src_sc[1] = sc.acc_w; a.src_sc[2] = sc.acc2_w;
  a.dst_sc[0] = dc.w; a.dst_sc[1] = dc.acc_w; a.dst_sc[2] = dc.acc2_w;
  a.src_aux = src_aux; a.dst_aux = dst_aux;
  a.keep = keep; a.new_row = flags; a.n = n; a.D = sc.dim;
  const int64_t threads = n * (sc.dim / 4);
  hipLaunchKernelGGL(k_move_rows, dim3((unsigned)((threads + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, a);
  if (kept > 0)
    hipLaunchKernelGGL(k_rehash, dim3(blocks_for(kept, 1 << 16)), dim3(kBlock), 0, s, dst->slots, dst->n_slots - 1,
                       (const uint64_t *)dc.row_keys, (int64_t)kept, dst->ctrl);
  if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) return DES_ERR_DEVICE;
  if (n_rows_out) *n_rows_out = kept;
  return blocking_status(dst);
}

des_status_t des_table_compact(des_table_t *t, const uint8_t *keep, uint32_t *aux, void *staging, size_t staging_bytes,
                               int64_t *n_rows_out, void *stream) {
  if (!t || ((uintptr_t)aux & 3u)) return DES_ERR_INVALID_ARG;
  const des_table_config_t &c = t->cfg;
  hipStream_t s = (hipStream_t)stream;
  Ctrl ctrl;                                                // the row count and the status in one copy
  if (hipStreamSynchronize(t->last_stream) != hipSuccess ||
      hipMemcpy(&ctrl, t->ctrl, sizeof(ctrl), hipMemcpyDeviceToHost) != hipSuccess)
    return DES_ERR_DEVICE;
  const int64_t n = ctrl.n_rows;
  if (ctrl.status != DES_OK) return DES_ERR_INVALID_ARG;
  if (n_rows_out) *n_rows_out = n;
  t->last_stream = s;
  t->prep.valid = false;
  if (n == 0 || !keep) return DES_OK;                       // nothing to drop
  // the staging buffer holds at least 4096 rows of the widest array at a time
  if (!staging || ((uintptr_t)staging & 15u) || staging_bytes < (size_t)4096 * (size_t)c.dim * 4) return DES_ERR_WORKSPACE;
  const size_t flags_bytes = align_up((size_t)(n + 1) * 8, 256);
  if (t->ws_bytes < flags_bytes + scan_scratch_bytes(n + 1)) return DES_ERR_WORKSPACE;
  // the new row numbers, then three words for the host, the tiles' counts and, if there is room, the bounds of the slot tiles
  unsigned long long *flags = (unsigned long long *)t->ws;
  const unsigned nb = (unsigned)((n + kKeepTile - 1) / kKeepTile);
  long long *words = (long long *)(t->ws + flags_bytes);
  uint32_t *counts = (uint32_t *)(words + 4);
  const size_t bounds_at = flags_bytes + align_up(sizeof(long long) * 4 + (size_t)nb * 4, 256);
  static_assert(kKeepTile >= 2048, "the words and counts fit where the scratch of a scan of n + 1 values would lie");
  static_assert(kSlotTile <= 1024, "whole tiles: a table has at least 1024 slots, a power of two");
  const int64_t ntiles = t->ws_bytes >= bounds_at + t->n_slots / kSlotTile * 4 ? (int64_t)(t->n_slots / kSlotTile) : 0;
  uint32_t *bounds = (uint32_t *)(t->ws + bounds_at);
  ProfScope ps(KID_MIGRATE, s);
  hipLaunchKernelGGL(k_keep_count, dim3(nb), dim3(kBlock), 0, s, keep, n, counts);
  if (ntiles)
    hipLaunchKernelGGL(k_slot_bounds, dim3((unsigned)((ntiles * kWave + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, t->slots, ntiles, bounds);
  hipLaunchKernelGGL(k_keep_tell, dim3(1), dim3(kTellBlock), 0, s, t->ctrl, keep, n, counts, (const uint32_t *)bounds, ntiles, words);
  long long told[3] = {0, 0, 0};
  if (hipMemcpyAsync(told, words, sizeof(told), hipMemcpyDeviceToHost, s) != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
    return DES_ERR_DEVICE;
  const int64_t kept = told[0], lo = told[1];
  // As many kept rows as rows before the first drop: nothing moves.  Moving a row onto itself through the staging buffer costs
  // as much as any other move: 4.0e6 rows of 32 columns with their state in front of 1.2e6 dropped ones took 160 launches, 1.2 ms.
  const int64_t hi = kept > lo ? n : lo;
  if (hi > lo) hipLaunchKernelGGL(k_keep_rows, dim3(nb), dim3(kBlock), 0, s, keep, n, (const uint32_t *)counts, flags);
  compact_array<float4>((float4 *)c.emb, c.dim / 4, keep, flags, lo, hi, staging, staging_bytes, s);
  compact_array<float4>((float4 *)c.acc_emb, c.dim / 4, keep, flags, lo, hi, staging, staging_bytes, s);
  compact_array<float4>((float4 *)c.acc2_emb, c.dim / 4, keep, flags, lo, hi, staging, staging_bytes, s);
  compact_array<uint32_t>((uint32_t *)c.w, 1, keep, flags, lo, hi, staging, staging_bytes, s);
  compact_array<uint32_t>((uint32_t *)c.acc_w, 1, keep, flags, lo, hi, staging, staging_bytes, s);
  compact_array<uint32_t>((uint32_t *)c.acc2_w, 1, keep, flags, lo, hi, staging, staging_bytes, s);
  compact_array<uint32_t>(aux, 1, keep, flags, lo, hi, staging, staging_bytes, s);
  compact_array<unsigned long long>((unsigned long long *)c.row_keys, 1, keep, flags, lo, hi, staging, staging_bytes, s);
  // The slots: each tile by itself, unless one has no empty slot (a run of a thousand occupied ones) or the workspace has no
  // room for the tiles' bounds; then from nothing, by the kept keys.
  if (ntiles && told[2] == 0) {
    hipLaunchKernelGGL(k_rebuild_slots, dim3((unsigned)ntiles), dim3(kBlock), 0, s, t->slots, t->n_slots, (const uint32_t *)bounds, keep,
                       hi > lo ? (const unsigned long long *)flags : nullptr, lo, t->ctrl);
  } else {
    hipLaunchKernelGGL(k_fill_slots, dim3(blocks_for((int64_t)t->n_slots, 1 << 16)), dim3(kBlock), 0, s, (uint4 *)t->slots,
                       (int64_t)t->n_slots);
    if (kept > 0)
      hipLaunchKernelGGL(k_rehash, dim3(blocks_for(kept, 1 << 16)), dim3(kBlock), 0, s, t->slots, t->n_slots - 1,
                         (const uint64_t *)c.row_keys, (int64_t)kept, t->ctrl);
  }
  int status = 0;
  if (hipGetLastError() != hipSuccess || hipMemcpyAsync(&status, &t->ctrl->status, sizeof(status), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    return DES_ERR_DEVICE;
  if (n_rows_out) *n_rows_out = kept;
  return (des_status_t)status;
}

des_status_t des_batch_validate(des_table_t *t, const des_batch_t *batch, const int32_t *rows, int64_t *first_bad,
                                void *stream) {
  if (!t || !batch || batch->B < 0 || batch->F < 1 || batch->nnz < 0 || batch->nnz >= 2147483647ll ||
      batch->B * (int64_t)batch->F >= 2147483647ll || !batch->offsets || ((uintptr_t)batch->offsets & 3u) ||
      ((uintptr_t)rows & 3u))
    return DES_ERR_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  unsigned long long *word = &t->ctrl->first_bad;
  const unsigned long long none = ~0ull;
  unsigned long long got = none;
  const int64_t nbags = batch->B * (int64_t)batch->F, total = nbags + 1 + (rows ? batch->nnz : 0);
  if (hipMemcpyAsync(word, &none, sizeof(none), hipMemcpyHostToDevice, s) != hipSuccess) return DES_ERR_DEVICE;
  hipLaunchKernelGGL(k_validate, dim3(blocks_for(total, 1 << 16)), dim3(kBlock), 0, s, batch->offsets, nbags, batch->nnz,
                     rows, t->ctrl, word);
  if (hipMemcpyAsync(&got, word, sizeof(got), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess || hipGetLastError() != hipSuccess)
    return DES_ERR_DEVICE;
  if (first_bad) *first_bad = got == none ? -1 : (int64_t)got;
  return got == none ? DES_OK : DES_ERR_INVALID_ARG;
}

des_status_t des_table_mark_seen(const int32_t *rows, int64_t n, uint32_t stamp, uint32_t *last_seen, void *stream) {
  if (n < 0 || (n > 0 && (!rows || !last_seen)) || ((uintptr_t)rows & 3u) || ((uintptr_t)last_seen & 3u))
    return DES_ERR_INVALID_ARG;
  if (n == 0) return DES_OK;
  hipStream_t s = (hipStream_t)stream;
  ProfScope ps(KID_MIGRATE, s);
  hipLaunchKernelGGL(k_mark_seen, dim3(blocks_for(n)), dim3(kBlock), 0, s, rows, n, stamp, last_seen);
  return hipGetLastError() == hipSuccess ? DES_OK : DES_ERR_DEVICE;
}

des_status_t des_table_select_recent(const uint32_t *last_seen, int64_t n_rows, uint32_t min_stamp, uint8_t *keep,
                                     void *stream) {
  if (n_rows < 0 || (n_rows > 0 && (!last_seen || !keep)) || ((uintptr_t)last_seen & 3u)) return DES_ERR_INVALID_ARG;
  if (n_rows == 0) return DES_OK;
  hipStream_t s = (hipStream_t)stream;
  ProfScope ps(KID_MIGRATE, s);
  hipLaunchKernelGGL(k_select_recent, dim3(blocks_for(n_rows)), dim3(kBlock), 0, s, last_seen, n_rows, min_stamp, keep);
  return hipGetLastError() == hipSuccess ? DES_OK : DES_ERR_DEVICE;
}

}  // extern "C"
