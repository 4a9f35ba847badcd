// Forward sub-operators of every logical shard in one pass over the batch:
//   LR  M1 (Section 4.1, Eq. lr_m1), FM M1 and M2 (Section 4.2, Eq. fm_m1m2) and the per-field
//   pooled embeddings (Section 4.3).
//
// Mapping: 1, 2 or 4 wave64s per sample, or several samples of few fields per wave.  A row of D floats is read by G = D/4 adjacent lanes
// as one 16-byte load each, so a wave holds 64/G "lane groups" that each fetch a different row
// at the same time.  Every group owns a contiguous range of the sample's bags and walks its
// entries in CSR order in chunks of G: lane i of the group loads the metadata of entry i of
// the chunk (row, key -> shard, value, bag found in the sample's offsets staged in LDS) and
// publishes it in LDS, from where the group reads entry j with one broadcast read (groups inside a quad
// of lanes exchange it by DPP instead); the row
// gathers of a chunk are issued back to back.  The running bag sum stays in registers (the
// pooled output is written once per bag, at its last entry, already summed over shards).  The per-shard FM / LR
// partials of the sample live in LDS ([K][D+2] doubles per sample: D columns, then the sum of
// squares and the LR sum) and are updated with LDS atomics, because the entries of one shard are
// scattered over all groups; the two scalars of an entry by the lane that holds its metadata, once per chunk.
// A lane owns columns 4*sub..4*sub+3 of a row but the LDS copy is
// stored column-permuted (column 4*sub+k at k*G+sub) with a row pitch of D+2 doubles, so that the
// 64 lanes of one atomic instruction spread over the LDS banks instead of piling onto a few.
//
// What bounds it (8e6 entries): dependent accesses, at D = 32 beside an LDS pipe that is busy 73 % of the time (double additions for the most
// part; vector ALU 46 %), at D = 64 beside a vector ALU busy 40 % (LDS 39 %; the waves wait for 62 % of their time).
// Vector instructions: row addresses by one multiply-add, the sums of squares of up to four entries together, a remainder by a known
// reciprocal, sums that are set back without selecting, gathers whose four floats stay together: 80.6 -> 59.3 million of them for 8.2e6
// entries of 32 floats, whose 212 us hardly change (208), 1.0e6 of 16 26.0 -> 24.6 us, 8.0e6 of 64 627 -> 616, 9.9e5 of 128
// 98 -> 83; 40 shapes of all widths take 4 % less on average, none more.
// Vector memory operations complete in order and a wait can only be counted along straight code: with a gather under a
// condition, or the bag's store between a batch's gathers and their uses, each was waited for alone.  Gathers without
// conditions, all waited for at once ahead of the stores: 8.0e6 entries of 64 floats 694 -> 598 us, 1.05e8 of 64 7.50 -> 6.35 ms,
// 8.2e6 of 32 236 -> 218 us.
// Registers: U gathers of four floats each.  Four waves per SIMD need 128 registers (without the bound 131 at D = 128 with values:
// 91 -> 81 us for 8.1e5 entries); D = 32 without values fits six waves with four gathers in flight (8.2e6 entries 217 -> 207 us, with
// the scalars' additions below).  Narrower rows need no bound for six (at most 72 registers without values).  At D = 64 it depends on
// where the rows come from: 1.7e6 entries by Zipf's law 76.5 -> 72.4 us with six waves and four gathers, uniform 105 -> 110, so it stays.
//
// Accumulation is in double, inputs and outputs are fp32: a sample's sum of several hundred
// signed terms cancels, and fp32 accumulation alone would exceed the 1e-5 relative bound
// against an exact reference.
#include <type_traits>
#include "des_internal.h"

namespace des {
namespace {

constexpr int64_t kFillGroups = 512;      // two workgroups per CU
constexpr size_t kSixPerCu = 160 * 1024 / 6;     // LDS bytes of a workgroup of which a CU holds six

struct FwdArgs {
  const float *emb, *w;
  const uint64_t *keys;
  const int32_t *offsets;
  const float *vals;
  const int32_t *rows;
  float *P_lr, *P_sum, *P_sq, *pool;
  int64_t B;
  int F, K, policy;
  int pitch;            // LDS doubles from one shard's sums to the next's
  int acc_doubles;      // LDS doubles of one set of a sample's accumulators
  int sets;             // sets per sample: 1, which its waves share, or one for each of them
  int lds_per_sample;   // LDS doubles per sample in total (accumulators + staged offsets)
  uint32_t per_shard;   // floor(2^32 / K), at most 2^32 - 1
  int log_threads;      // log2 of the threads per sample: part of a wave (whole lane groups), or 1, 2 or 4 waves
};

__device__ inline float4 ld4(const float *p) { return *reinterpret_cast<const float4 *>(p); }
__device__ inline void st4(float *p, float4 v) { *reinterpret_cast<float4 *>(p) = v; }

// Cross-lane move of a double with a DPP control word (VALU, does not use the LDS pipe).
template <int kCtrl>
__device__ inline double dpp_f64(double v) {
  int lo = __double2loint(v), hi = __double2hiint(v);
  lo = __builtin_amdgcn_update_dpp(0, lo, kCtrl, 0xF, 0xF, true);
  hi = __builtin_amdgcn_update_dpp(0, hi, kCtrl, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}

// Four floats at `base` in row `row` of rows of `pitch` bytes.  The address is one multiply-add: `pitch` is opaque to the compiler, which
// would take four instructions for the shift that it makes of a known one.
typedef float v4f __attribute__((ext_vector_type(4)));
__device__ inline v4f ld4_row(const float *base, uint32_t row, uint32_t pitch) {
  const uint64_t at = reinterpret_cast<uint64_t>(base) + (uint64_t)row * pitch;
  return *reinterpret_cast<const __attribute__((address_space(1))) v4f *>(at);
}

// Sum of q over the G adjacent lanes of a lane group (every lane gets the total).
template <int G>
__device__ inline double group_sum(double q) {
  if (G >= 2) q += dpp_f64<0xB1>(q);     // quad_perm [1,0,3,2]
  if (G >= 4) q += dpp_f64<0x4E>(q);     // quad_perm [2,3,0,1]
  if (G >= 8) q += dpp_f64<0x141>(q);    // row_half_mirror: pairs the two quads of 8 lanes
  if (G >= 16) q += dpp_f64<0x140>(q);   // row_mirror: pairs the two halves of 16 lanes
#pragma unroll
  for (int m = 16; m < G; m <<= 1) q += __shfl_xor(q, m, kWave);
  return q;
}

// The sums of n = 1, 2 or 4 values over the lanes of a group, of which lane `sub` gets the one of value sub % n: a lane hands half of its
// values to its neighbour and takes the other half of the neighbour's, so that all sums together take hardly more instructions than one
// (n = 4, G = 8: 26 against 44).  odd0 and odd1: bits 0 and 1 of the lane's number, turned in every second quad, since the
// mirrored steps pair lanes of different quads whose numbers differ in these bits as well (kTurn: in the others instead, so that
// the lanes of the group's every second quad are the ones that hold sub % n).
template <int kCtrl, bool kTurn>
__device__ inline double exchange(double a, double b, bool odd) {
  const double keep = odd != kTurn ? b : a, give = odd != kTurn ? a : b;
  return keep + dpp_f64<kCtrl>(give);
}
template <int G, int N, bool kTurn>
__device__ inline double group_sums(const double (&p)[N], bool odd0, bool odd1) {
  static_assert(N == 1 || N == 2 || N == 4, "up to a quad");
  if constexpr (N == 1 || G < N) {
    return group_sum<G>(p[0]);
  } else {
    double q = exchange<0xB1, kTurn>(p[0], p[1], odd0);
    if constexpr (N == 4) {
      const double r = exchange<0xB1, kTurn>(p[2], p[3], odd0);
      q = exchange<0x4E, kTurn>(q, r, odd1);
    } else if constexpr (G >= 4) {
      q += dpp_f64<0x4E>(q);
    }
    if (G >= 8) q += dpp_f64<0x141>(q);
    if (G >= 16) q += dpp_f64<0x140>(q);
#pragma unroll
    for (int m = 16; m < G; m <<= 1) q += __shfl_xor(q, m, kWave);
    return q;
  }
}

// v of lane `src` of the caller's group of G = 1, 2 or 4 lanes (VALU, does not use the LDS pipe).
template <int G>
__device__ inline int group_lane(int v, int src) {
  static_assert(G <= 4, "inside a quad");
  if (G == 1) return v;
  if (G == 2) return src == 0 ? __builtin_amdgcn_mov_dpp(v, 0xA0, 0xF, 0xF, true) : __builtin_amdgcn_mov_dpp(v, 0xF5, 0xF, 0xF, true);
  if (src == 0) return __builtin_amdgcn_mov_dpp(v, 0x00, 0xF, 0xF, true);
  if (src == 1) return __builtin_amdgcn_mov_dpp(v, 0x55, 0xF, 0xF, true);
  if (src == 2) return __builtin_amdgcn_mov_dpp(v, 0xAA, 0xF, 0xF, true);
  return __builtin_amdgcn_mov_dpp(v, 0xFF, 0xF, 0xF, true);
}

// x mod K from floor(2^32 / K): the quotient that gives is the true one or one less.  (The compiler's own division corrects twice.)
__device__ inline uint32_t mod_shards(uint32_t x, uint32_t K, uint32_t per_shard) {
  const uint32_t r = x - __umulhi(x, per_shard) * K;
  return min(r, r - K);
}

// kByKey: shard of an entry = hash of its ID (entries of a bag scatter over the shards: one LDS update per
// entry).  Otherwise the field partition of Section 5: a bag belongs to shard f mod K as a whole, so its sums
// are formed in registers and the shard's accumulators take one update per bag.
// kHasVals: the batch carries feature values; without them every x is 1 and the products with x are left out.
// kFew: few entries per lane group, so that most of a batch of gathers would be of entries that are not there.  They are requested and
// waited for all the same, hence fewer at a time (and fewer registers): 2.0e5 samples of 10 one-entry bags, D = 64 (1.0e5) / 32 204 / 251 ->
// 159 / 225 us, 12 and more entries per group of D = 64 69 -> 72.
// Where accumulators leave LDS for no more than four workgroups per CU, registers saved are none gained and a batch of the usual size
// is one round trip less: there only while a batch of these few takes all entries (D = 64, K = 32 / 60,
// 24 / 50 bags a sample 119 / 114 -> 114 / 109 us, with the former kernel 110 / 105; D = 32 134 / 131 -> 131 / 128, 129 / 128).
constexpr int64_t kFewEntries = 12;
constexpr size_t kFewLds = 32 * 1024;
constexpr int few_gathers(int D) { return D >= 128 ? 4 : 2; }
template <int D, bool kByKey, bool kHasVals, bool kFew>
__global__ __launch_bounds__(kBlock, D == 32 && !kHasVals ? 6 : 4) void k_forward(const FwdArgs a) {
  extern __shared__ __align__(16) double lds[];
  constexpr int G = D / 4;                 // lanes per row = entries per chunk
  constexpr int U = kFew ? few_gathers(D) : G < 8 ? G : D == 32 && !kHasVals ? 4 : 8;         // row gathers in flight per lane (4 / 8: D = 64 625 -> 598 us, D = 32 with values 21.9 -> 21.4, without 218 -> 219)
  // Rows of one or two lanes: a wave's groups end their bags at up to 64 different steps, and stores among the steps are waited for with
  // the next gathers (loads and stores complete in order).  So the pooled stores of a group's last bag and of bags without entries
  // come behind its steps: 2.0e6 bags of 0 to 4 entries, 26 a sample, D = 4 / 8 125 / 114 -> 96 / 107 us, 60 a sample 126 -> 98 at D = 4.
  constexpr bool kBehind = G <= 2;
  constexpr bool kQuad = G <= 4;           // a group lies inside a quad: its lanes' metadata comes by DPP instead of through LDS
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int g = lane / G, sub = lane % G;
  const int K = a.K, F = a.F;
  const int local = threadIdx.x >> a.log_threads;         // sample in the workgroup
  const int nts = 1 << a.log_threads, tis = threadIdx.x & (nts - 1);   // threads per sample, thread in sample
  // LDS: one 16-byte metadata slot per thread, then per sample the accumulators and offsets
  int4 *meta = reinterpret_cast<int4 *>(lds) + wave * kWave;
  const int P = a.pitch;                                  // row pitch: D columns, sum of squares, LR sum (and none or some of no use)
  double *sums = lds + 2 * kBlock + (size_t)local * a.lds_per_sample;  // [sets][K][P]
  double *sum = a.sets > 1 ? sums + tis / kWave * a.acc_doubles : sums;  // the one this wave adds to
  int *offs = reinterpret_cast<int *>(sums + a.sets * a.acc_doubles);  // [F+1]
  const int64_t b = ((int64_t)blockIdx.x * kBlock >> a.log_threads) + local;
  const bool active = b < a.B;
  const bool need_fm = a.P_sum != nullptr, need_lr = a.P_lr != nullptr, need_pool = a.pool != nullptr;
  const bool hashed = kByKey && (need_fm || need_lr);
  const int row_mask = need_fm || need_pool ? -1 : 0;     // first-order terms alone need no rows
  const float *w_base = need_lr ? a.w : a.emb;
  const float *const emb = a.emb + sub * 4;
  uint32_t pitch = D * sizeof(float);
  asm("" : "+s"(pitch));
  const bool turned = G >= 8 && (sub & 4) != 0, odd0 = ((sub & 1) != 0) != turned, odd1 = ((sub & 2) != 0) != turned;

  for (int i = tis; i < a.sets * a.acc_doubles; i += nts) sums[i] = 0.0;
  if (active)
    for (int i = tis; i <= F; i += nts) offs[i] = a.offsets[b * F + i];
  __syncthreads();

  if (active) {
    const int gg = tis / G, ngt = nts / G;
    const int f0 = (int)(((int64_t)F * gg) / ngt), f1 = (int)(((int64_t)F * (gg + 1)) / ngt);
    const int first = offs[0];                            // the sample's entries start here
    const int e0 = offs[f0] - first, e1 = offs[f1] - first;
    const int32_t *rows = a.rows + first;
    const uint64_t *keys = a.keys + first;
    const float *vals = kHasVals ? a.vals + first : nullptr;
    float *pool = a.pool + (b * F) * (int64_t)D;
    if (need_pool && !kBehind)                            // bags without entries; the others are stored at their last entry
      for (int f = f0; f < f1; ++f)
        if (offs[f] == offs[f + 1]) st4(pool + (f * D + sub * 4), make_float4(0.f, 0.f, 0.f, 0.f));
    const int last_marked = need_pool || (!kByKey && need_fm) ? (kBehind ? e1 - 1 : e1) : 0;   // entries before it may end a bag
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    double bag_sq = 0.0;                                  // field partition: this lane's share of the bag's sum of squares
    int cur = f0;                                         // a bag that no entry to come lies before
    int cur_end = offs[min(f0 + 1, F)];                   // kQuad: where it ends
    int cur_sh = kQuad && !kByKey ? f0 % K : 0;           // ... and its shard

    // metadata of entry e0 + sub of the first chunk; later chunks are fetched one chunk ahead
    int r_n = -1;
    uint64_t key_n = 0;
    float x_n = 1.f;
    if (e0 + sub < e1) {
      r_n = rows[e0 + sub];
      if (hashed) key_n = keys[e0 + sub];
      if (kHasVals) x_n = vals[e0 + sub];
    }
    for (int e = e0; e < e1; e += G) {
      const int my = e + sub, at = my + first;
      const int r_l = r_n;
      const uint64_t key_l = key_n;
      const float x_l = x_n;
      r_n = -1;
      if (my + G < e1) {                                  // the next chunk's metadata
        r_n = rows[my + G];
        if (hashed) key_n = keys[my + G];
        if (kHasVals) x_n = vals[my + G];
      }
      // Bag of this lane's entry: the largest f with offs[f] <= its index, and where that bag ends.  A lane of a small group comes
      // back after few entries, mostly to the same bag or the next.  In larger groups the chunk starts at or shortly after the bag of
      // the one before: up to four bags on in one step (offsets ascend), then a binary search for the rare long run of short or
      // empty bags.
      int lo = cur, end = 0x7FFFFFFF;
      if (kQuad) {
        end = cur_end;
        if (my < e1 && end <= at)
          do {
            ++lo;
            end = offs[lo + 1];
            if (!kByKey) cur_sh = cur_sh + 1 == K ? 0 : cur_sh + 1;
          } while (end <= at);
        cur_end = end;
      } else {
        int ahead = 0;
#pragma unroll
        for (int k = 1; k <= 4; ++k) {
          const int o = offs[min(cur + k, f1)];
          ahead += o <= at ? 1 : 0;
          if (o > at) end = min(end, o);
        }
        lo += ahead;
        if (my < e1 && ahead == 4) {
          if (offs[lo + 1] <= at) {
            int hi = f1;
            ++lo;
            while (hi - lo > 1) {
              const int mid = (lo + hi) >> 1;
              if (offs[mid] <= at) lo = mid; else hi = mid;
            }
          }
          end = offs[lo + 1];
        }
      }
      const int bag_l = my < e1 ? lo : cur;
      cur = kQuad ? bag_l : __shfl(bag_l, lane - sub + min(G, e1 - e) - 1, kWave);
      const int sh_l = !need_fm && !need_lr ? 0 : kByKey ? (int)mod_shards((uint32_t)(mix64(key_l) >> 32), (uint32_t)K, a.per_shard) : kQuad ? cur_sh : bag_l % K;
      // what the group needs of this lane's entry: row (0 if absent), its shard's accumulators (negative: absent; by field their
      // complement, for the bag that ends there), its bag's pooled row if it is the bag's last entry (-1: it is not), its value
      const int row_l = max(r_l, 0) & row_mask;
      const int acc_l = r_l >= 0 ? sh_l * P : kByKey ? -1 : ~(sh_l * P);
      const int end_l = my < last_marked && at + 1 == end ? bag_l * D : -1;
      // read back with one broadcast LDS read per entry; same wave, program order: no barrier needed
      if (!kQuad) meta[lane] = make_int4(row_l, acc_l, end_l, __float_as_int(x_l));
      // The first-order weight of this lane's own entry: one gather per chunk for the whole group (without first-order terms of one
      // and the same element: without that a gather by row for nothing, 35 -> 29 us for the pooled sums alone of 4.3e6 entries of 4 floats).
      float w_l = w_base[need_lr ? max(r_l, 0) : 0];
      double q_l = 0.0;                                   // sum of squares of this lane's own entry
      const int cnt = min(G, e1 - e);
#pragma unroll
      for (int j0 = 0; j0 < G; j0 += U) {
        if (j0 == 0 || j0 < cnt) {
          int4 md[U];
          v4f v[U];
          // Every row is requested without a condition (an absent one reads row 0 and is left out below) and all of them,
          // with what was requested before them, are waited for here: loads under a condition, or waits between the pooled
          // stores, would be waited for one by one.
#pragma unroll
          for (int i = 0; i < U; ++i) {
            if constexpr (kQuad)
              md[i] = make_int4(group_lane<G>(row_l, j0 + i), group_lane<G>(acc_l, j0 + i), group_lane<G>(end_l, j0 + i),
                                kHasVals ? group_lane<G>(__float_as_int(x_l), j0 + i) : 0);
            else
              md[i] = meta[g * G + j0 + i];
            v[i] = ld4_row(emb, (uint32_t)md[i].x, pitch);
          }
#pragma unroll
          for (int i = 0; i < U; ++i) asm volatile("" : "+v"(v[i]));
          if (j0 == 0) {
            asm volatile("" : "+v"(w_l), "+v"(r_n));
            if (hashed) asm volatile("" : "+v"(key_n));
            if (kHasVals) asm volatile("" : "+v"(x_n));
          }
          double squares[U];
#pragma unroll
          for (int i = 0; i < U; ++i) {
            squares[i] = 0.0;
            if (md[i].y >= 0) {
              const double xd = kHasVals ? (double)__int_as_float(md[i].w) : 1.0;
              const double xv[4] = {kHasVals ? xd * (double)v[i].x : (double)v[i].x, kHasVals ? xd * (double)v[i].y : (double)v[i].y,
                                    kHasVals ? xd * (double)v[i].z : (double)v[i].z, kHasVals ? xd * (double)v[i].w : (double)v[i].w};
#pragma unroll
              for (int k = 0; k < 4; ++k) acc[k] += xv[k];
              if (need_fm) {
                const double p = xv[0] * xv[0] + xv[1] * xv[1] + xv[2] * xv[2] + xv[3] * xv[3];
                if (!kByKey) {
                  bag_sq += p;
                } else {
                  double *dst = sum + md[i].y + sub;
#pragma unroll
                  for (int k = 0; k < 4; ++k) atomicAdd(dst + k * G, xv[k]);
                  squares[i] = p;
                }
              }
            }
            // The bag ends: pooled sum out, and to its shard under the field partition.  (Where neither is asked for no entry is
            // marked as a last one: a condition less around the sums that are set back.)
            if (md[i].z >= 0) {
              if (kByKey || need_pool) st4(pool + (md[i].z + sub * 4), make_float4((float)acc[0], (float)acc[1], (float)acc[2], (float)acc[3]));
              if (!kByKey && need_fm) {
                double *const shard = sum + (md[i].y ^ (md[i].y >> 31)), *const dst = shard + sub;
#pragma unroll
                for (int k = 0; k < 4; ++k) atomicAdd(dst + k * G, acc[k]);
                const double q = group_sum<G>(bag_sq);
                if (sub == 0) atomicAdd(shard + D, q);
                bag_sq = 0.0;
              }
              acc[0] = acc[1] = acc[2] = acc[3] = 0.0;
            }
          }
          if (kByKey && need_fm) {                         // sums of squares, each to the lane that holds its entry's metadata
            constexpr int N = U < 4 ? U : 4;
#pragma unroll
            for (int i = 0; i < U; i += N) {
              double p[N];
#pragma unroll
              for (int k = 0; k < N; ++k) p[k] = squares[i + k];
              const double q = ((j0 + i) & 4) && G >= 8 ? group_sums<G, N, true>(p, odd0, odd1) : group_sums<G, N, false>(p, odd0, odd1);
              if (sub >= j0 + i && sub < j0 + i + N) q_l = q;
            }
          }
        }
      }
      if (r_l >= 0) {
        double *dst = sum + sh_l * P + D;
        const double l_l = kHasVals ? (double)x_l * (double)w_l : (double)w_l;
        // half of the lanes the other way round: with few shards the lanes' addresses are equal (K = 2: 7.2e6 entries of 8 floats
        // 149 -> 135 us, 6.9e6 of 16 207 -> 187)
        if (kByKey && need_fm && need_lr) {
          const bool odd = sub & 1;
          atomicAdd(dst + (odd ? 1 : 0), odd ? l_l : q_l);
          atomicAdd(dst + (odd ? 0 : 1), odd ? q_l : l_l);
        } else if (kByKey && need_fm) {
          atomicAdd(dst, q_l);
        } else if (need_lr) {
          atomicAdd(dst + 1, l_l);
        }
      }
    }
    if constexpr (kBehind) {
      if (need_pool || (!kByKey && need_fm)) {
        if (e0 < e1) {
          const int last = group_lane<G>(cur, (e1 - e0 - 1) & (G - 1));   // bag of the range's last entry
          if (need_pool) st4(pool + (last * D + sub * 4), make_float4((float)acc[0], (float)acc[1], (float)acc[2], (float)acc[3]));
          if (!kByKey && need_fm) {
            double *const shard = sum + group_lane<G>(cur_sh, (e1 - e0 - 1) & (G - 1)) * P, *const dst = shard + sub;
#pragma unroll
            for (int k = 0; k < 4; ++k) atomicAdd(dst + k * G, acc[k]);
            const double q = group_sum<G>(bag_sq);
            if (sub == 0) atomicAdd(shard + D, q);
          }
        }
        if (need_pool)
          for (int f = f0, start = offs[f0]; f < f1; ++f) {
            const int next = offs[f + 1];
            if (start == next) st4(pool + (f * D + sub * 4), make_float4(0.f, 0.f, 0.f, 0.f));
            start = next;
          }
      }
    }
  }
  __syncthreads();

  if (active) {
    const auto write = [&](auto sets_c) {
      constexpr int kSets = decltype(sets_c)::value;
      const auto total = [&](int i) {
        double v[kSets];
#pragma unroll
        for (int w = 0; w < kSets; ++w) v[w] = sums[w * a.acc_doubles + i];
#pragma unroll
        for (int w = 1; w < kSets; ++w) v[0] += v[w];
        return (float)v[0];
      };
      if (need_fm) {
        for (int idx = tis * 4; idx < K * D; idx += nts * 4) {
          const int s = idx / D, d = idx % D;               // d = 4*sub: columns d..d+3 sit at k*G + sub
          const int at = s * P + d / 4;
          st4(a.P_sum + ((int64_t)s * a.B + b) * D + d, make_float4(total(at), total(at + G), total(at + 2 * G), total(at + 3 * G)));
        }
        for (int s = tis; s < K; s += nts) a.P_sq[(int64_t)s * a.B + b] = total(s * P + D);
      }
      if (need_lr)
        for (int s = tis; s < K; s += nts) a.P_lr[(int64_t)s * a.B + b] = total(s * P + D + 1);
    };
    if (a.sets == 1) write(std::integral_constant<int, 1>{});
    else if (a.sets == 2) write(std::integral_constant<int, 2>{});
    else write(std::integral_constant<int, 4>{});
  }
}

// Per-shard pooled partials [K,B,F,D] (small shapes only): one lane group per bag, one pass
// over the bag per shard.
template <int D>
__global__ __launch_bounds__(kBlock) void k_pool_dense(const FwdArgs a, float *__restrict__ P_pool) {
  constexpr int G = D / 4;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t bag = gid / G;
  const int sub = (int)(gid % G);
  const int64_t nbags = a.B * a.F;
  if (bag >= nbags) return;
  const int f = (int)(bag % a.F);
  const int e0 = a.offsets[bag], e1 = a.offsets[bag + 1];
  for (int s = 0; s < a.K; ++s) {
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int e = e0; e < e1; ++e) {
      const int r = a.rows[e];
      if (r < 0) continue;
      const int sh = a.policy == DES_SHARD_KEY_HASH ? (int)((uint32_t)(mix64(a.keys[e]) >> 32) % (uint32_t)a.K)
                                                     : f % a.K;
      if (sh != s) continue;
      const double x = a.vals ? (double)a.vals[e] : 1.0;
      const float4 v = ld4(a.emb + (int64_t)r * D + sub * 4);
      acc[0] += x * (double)v.x; acc[1] += x * (double)v.y; acc[2] += x * (double)v.z; acc[3] += x * (double)v.w;
    }
    st4(P_pool + ((int64_t)s * nbags + bag) * D + sub * 4,
        make_float4((float)acc[0], (float)acc[1], (float)acc[2], (float)acc[3]));
  }
}

template <int D, bool kFew>
void launch_forward(bool by_key, bool has_vals, dim3 grid, dim3 block, size_t shmem, hipStream_t s, const FwdArgs &a) {
  if (by_key) {
    if (has_vals) hipLaunchKernelGGL((k_forward<D, true, true, kFew>), grid, block, shmem, s, a);
    else hipLaunchKernelGGL((k_forward<D, true, false, kFew>), grid, block, shmem, s, a);
  } else {
    if (has_vals) hipLaunchKernelGGL((k_forward<D, false, true, kFew>), grid, block, shmem, s, a);
    else hipLaunchKernelGGL((k_forward<D, false, false, kFew>), grid, block, shmem, s, a);
  }
}
template <int D>
void launch_forward(bool few, bool by_key, bool has_vals, dim3 grid, dim3 block, size_t shmem, hipStream_t s, const FwdArgs &a) {
  if constexpr (D >= 32) {
    if (few) return launch_forward<D, true>(by_key, has_vals, grid, block, shmem, s, a);
  }
  launch_forward<D, false>(by_key, has_vals, grid, block, shmem, s, a);
}

FwdArgs make_args(des_table *t, const des_batch_t *b, const int32_t *rows) {
  FwdArgs a;
  a.emb = t->cfg.emb; a.w = t->cfg.w;
  a.keys = b->keys; a.offsets = b->offsets; a.vals = b->vals; a.rows = rows;
  a.P_lr = a.P_sum = a.P_sq = a.pool = nullptr;
  a.B = b->B; a.F = b->F; a.K = t->cfg.num_shards; a.policy = t->cfg.shard_policy;
  a.pitch = 0;
  a.per_shard = a.K > 1 ? (uint32_t)((1ull << 32) / (uint32_t)a.K) : ~0u;
  a.acc_doubles = 0; a.sets = 1; a.lds_per_sample = 0; a.log_threads = 6;
  return a;
}

}  // namespace

des_status_t forward_launch(des_table *t, const des_batch_t *b, const int32_t *rows, float *P_lr, float *P_sum,
                            float *P_sq, float *pool, hipStream_t s) {
  if (b->B == 0) return DES_OK;
  FwdArgs a = make_args(t, b, rows);
  a.P_lr = P_lr; a.P_sum = P_sum; a.P_sq = P_sq; a.pool = pool;
  const int D = t->cfg.dim;
  // LDS per sample: K*(D+2) doubles of accumulators plus the sample's F+1 offsets.  Fewer
  // samples per workgroup (more waves per sample) when that is large, so that a CU still holds
  // several workgroups.
  int64_t acc_doubles = (int64_t)align_up((size_t)a.K * (D + 2), 2);
  const int64_t offs_doubles = ((int64_t)b->F + 2) / 2, per_sample = acc_doubles + offs_doubles;
  if (per_sample * 8 + 16 * kBlock > 65536) return DES_ERR_INVALID_ARG;   // K*(dim+2) doubles + F+1 ints + 4 KB must fit 64 KB of LDS
  a.pitch = D + 2;
  int wps = 1;
  while (wps < 4 && (kBlock / kWave / wps) * per_sample * 8 > 40 * 1024) wps *= 2;
  const int64_t entries_per_sample = b->nnz / (b->B > 0 ? b->B : 1);
  if (entries_per_sample >= 2048 && wps < 4) wps = 4;       // very long samples: spread over the workgroup
  // Small batches: more waves per sample while the chip has fewer than kFillGroups workgroups and the sample has bags for
  // them (a wave takes 64/(D/4) bags at a time; what a lane group walks one after the other is all that is waited for).
  // 48 x 26 bags of 16 columns: 10.9 -> 7.6 us, 100 / 1000 / 2000 x 100 bags of 32: 36.9 / 43.4 / 48.1 -> 14.5 / 22.9 / 35.5;
  // from 512 workgroups on there is nothing more to gain (37.3 at 1024 or 2048).
  // One wave adds to a sample's accumulators in program order.  Where several take its place, each has a set of its own and the
  // sets are added in the order of the waves, so that sums do not depend on scheduling there either; a workgroup needs no more
  // LDS for it than with four samples of one wave each.
  const int without = wps;
  while (wps < 4 && (b->B * wps + 3) / 4 < kFillGroups && b->F > wps * (kWave * 4 / D)) wps *= 2;
  // Few fields: a wave's lane groups beyond the sample's bags would idle, so it takes several samples, as long as every bag has a
  // group of its own and the chip stays full (D = 16: 73821 x 4 bags 85 -> 31 us; D = 4: 32762 x 2 51 -> 15 us).
  int threads = kWave * wps;
  while (threads <= kWave && b->F * (D / 4) <= threads / 2 && b->B * (threads / 2) / kBlock >= kFillGroups &&
         kBlock / (threads / 2) * per_sample * 8 <= 40 * 1024)
    threads /= 2;
  a.log_threads = __builtin_ctz((unsigned)threads);
  a.sets = without == 1 ? wps : 1;
  const int spb = kBlock / threads;
  // An addition of doubles takes 16 lanes at a time over 32 banks (64 consecutive doubles: 8 cycles).  At D = 32 those are two lane groups
  // of 16 banks each: with rows 16 banks apart they meet where both shards are odd or both even, with rows 4 apart nearly always
  // (8.2e6 entries, 16 shards 208 -> 202 us).  Only where a CU still holds the workgroups that its registers allow.
  if (D == 32 && a.policy == DES_SHARD_KEY_HASH) {
    const int64_t spread = (int64_t)a.K * 40;
    if ((size_t)(a.sets * spread + offs_doubles) * 8 * spb + 16 * kBlock <= kSixPerCu) { a.pitch = 40; acc_doubles = spread; }
  }
  a.lds_per_sample = (int)(a.sets * acc_doubles + offs_doubles);
  a.acc_doubles = (int)acc_doubles;
  const dim3 grid((unsigned)((b->B + spb - 1) / spb)), block(kBlock);
  const size_t shmem = 16 * (size_t)kBlock + (size_t)a.lds_per_sample * 8 * spb;
  const bool by_key = a.policy == DES_SHARD_KEY_HASH;
  const bool few = b->nnz <= (shmem > kFewLds ? few_gathers(D) : kFewEntries) * b->B * (threads / (D / 4));
  ProfScope ps(KID_FORWARD, s);
  switch (D) {
    case 4: launch_forward<4>(few, by_key, a.vals != nullptr, grid, block, shmem, s, a); break;
    case 8: launch_forward<8>(few, by_key, a.vals != nullptr, grid, block, shmem, s, a); break;
    case 16: launch_forward<16>(few, by_key, a.vals != nullptr, grid, block, shmem, s, a); break;
    case 32: launch_forward<32>(few, by_key, a.vals != nullptr, grid, block, shmem, s, a); break;
    case 64: launch_forward<64>(few, by_key, a.vals != nullptr, grid, block, shmem, s, a); break;
    case 128: launch_forward<128>(few, by_key, a.vals != nullptr, grid, block, shmem, s, a); break;
    case 256: launch_forward<256>(few, by_key, a.vals != nullptr, grid, block, shmem, s, a); break;
    default: return DES_ERR_INVALID_ARG;
  }
  return hipGetLastError() == hipSuccess ? DES_OK : DES_ERR_DEVICE;
}

des_status_t pool_dense_launch(des_table *t, const des_batch_t *b, const int32_t *rows, float *P_pool, hipStream_t s) {
  if (b->B == 0) return DES_OK;
  FwdArgs a = make_args(t, b, rows);
  const int D = t->cfg.dim;
  const int64_t threads = b->B * b->F * (D / 4);
  const dim3 grid((unsigned)((threads + kBlock - 1) / kBlock)), block(kBlock);
  ProfScope ps(KID_POOL_DENSE, s);
  switch (D) {
    case 4: hipLaunchKernelGGL(k_pool_dense<4>, grid, block, 0, s, a, P_pool); break;
    case 8: hipLaunchKernelGGL(k_pool_dense<8>, grid, block, 0, s, a, P_pool); break;
    case 16: hipLaunchKernelGGL(k_pool_dense<16>, grid, block, 0, s, a, P_pool); break;
    case 32: hipLaunchKernelGGL(k_pool_dense<32>, grid, block, 0, s, a, P_pool); break;
    case 64: hipLaunchKernelGGL(k_pool_dense<64>, grid, block, 0, s, a, P_pool); break;
    case 128: hipLaunchKernelGGL(k_pool_dense<128>, grid, block, 0, s, a, P_pool); break;
    case 256: hipLaunchKernelGGL(k_pool_dense<256>, grid, block, 0, s, a, P_pool); break;
    default: return DES_ERR_INVALID_ARG;
  }
  return hipGetLastError() == hipSuccess ? DES_OK : DES_ERR_DEVICE;
}

}  // namespace des
