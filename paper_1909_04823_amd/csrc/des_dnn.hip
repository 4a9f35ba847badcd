// First fully-connected layer of the DNN tower under DES (Section 4.3, Eq. dnn_bmm / dnn_des).
//
// The concatenated pooled embeddings V [B, F*D] and the layer weights W [F*D, H] are both cut
// along the field dimension; shard s owns the fields f with f mod K == s and its sub-operator is
// M1(V_s, W_s) = V_s^T W_s, a [B,H] partial that the aggregation sums over the shards.  Backward:
// the gradient dY of the aggregate reaches every shard unchanged (Section 3.2.2), each shard
// forms the gradient of its own field columns (dY W_s^T, which is the upstream gradient of the
// pooled embeddings) and of its own weight rows (V_s dY).
//
// This is the one dense contraction of the path, so it runs on the matrix cores.  128x128 output tile per workgroup (64x64
// where that leaves CUs idle), four waves in a 2x2 arrangement of 64x64 (32x32).  Three kernels:
//
// k_gemm_f32, the forward product: the fp32 matrix instruction (32x32x2, 64 cycles), 16 or 32 products deep per LDS tile, the
// next tile in registers meanwhile.  Bound by the matrix pipe, and by its writes where the shards are shallow.  The sum of an
// output element is one chain in ascending k (above 1024 products: of chains of forward_run products) whatever the tile,
// so results do not depend on the tile size.  It keeps the fp32 chain because a ReLU follows it: with a split (223 against
// 271 us at 16384 x 3200 x 256) a unit within 1e-8 of zero changes sides in one of six training steps at 4096 x 256 units, and
// its gradient with it.  A shard's fields are walked as one range (a field of 20 columns costs no padding).
//
// k_gemm_halves, the two gradient products: fp32 accuracy from the fp16 instruction (32x32x16, 32 cycles).  Every operand element,
// times a power of two that its row of the tile has, is cut into two fp16 parts, a = hi + lo, each the nearest to what is left (11 + 12
// significant bits with lo's sign: the cut is exact but for the last bit of every fourth element), and a product is three:
//   hi*hi + hi*lo + lo*hi
// so 16 products of depth take 3 x 32 instead of 8 x 64 cycles.  lo is kept times 2^11, in hi's range, and the last two terms in sums
// of their own: with one sum for all, lo would leave fp16's range 2^10 below the row's largest; so an element is cut in full
// down to 2^-14 of the row's unit and to the nearest multiple of 2^-36 below.  The unit is the power of two at or below the
// largest of the row's first 32 products, which leaves 2^16 above it; a later element beyond that, or a row whose first 32
// products are zeros and whose largest is then below 2^-10 of the unit it was given instead (the tile's), is computed again with
// the fp32 instruction, as is a sum that is not finite.
// A single product is off by 7e-8 on average (fp32 3e-8), but the sum is rounded once per 16 products instead of once per product, so that
// sums of 64 and more are closer than in fp32 or from three bf16 parts.  Error against 64 bits, 2-norm, fp32 / thirds / halves: sums of 64
// 1.45 / 1.1 / 0.97 e-7, 128 - / 1.6 / 1.1, 256 2.9 / 2.4 / 1.3, 512 - / 3.4 / 1.7; of 1648 in slices 1.8 (thirds) and 1.7.  Deep sums
// (above 1024) are taken 512 products at a time, which are added to the result in memory: registers for a second level are not left.
// Bound by the vector instructions of the cut (5 per element and tile) beside a matrix pipe busy a quarter of the time.  32 products per
// step in two LDS buffers; the next tile travels in registers, both its halves requested together, so that lines of 128 bytes
// along k are used when they come (16 per step: g_pool 152, dW 213 us).  16384 x 3200 x 256, thirds / halves: g_pool 181 / 138 us,
// dW 162 / 147; both 346 / 273; 131072 x 320 x 64 614 / 354; 65536 x 416 x 256 371 / 265; 4096 x 416 x 256 40 / 32.
//
// k_gemm_split, sums of fewer than 64 products: three bf16 parts, a = hi + mid + lo (the cut is exact: 3 x 8 significant bits), and
// six products:
//   hi*hi + hi*mid + mid*hi + hi*lo + lo*hi + mid*mid
// What is left out is at most 2^-24 of a*b (mid is up to 2^-8 of a, lo up to 2^-17): a single product can be off by 2^-23 where the
// fp32 instruction is by 2^-24, a sum is closer from three products on.  Error, split / fp32: sums of 1, 2, 3, 16 products
// 3.5 / 2.5, 3.3 / 3.1, 3.2 / 3.6, 3.4 / 7.3 e-8.  Two LDS buffers of 16 products, and two tiles under way in registers.
//
// The 16-bit instructions drop the bits of their sum that do not fit, towards minus infinity; over many runs that adds up (a mean
// of -3e-7 of the results' root mean square at 124623 samples), so every second run of kRun products is accumulated with the
// opposite sign.  A single run, or a last one without a partner, keeps its part: tiles (in k_gemm_halves blocks of 64 x 64 outputs) and
// slices begin with alternating signs, so that it has both signs in what a row of the table adds up over the samples and in a slice sum (of thirds, mean error /
// root mean square, all beginning with plus and so: g_pool of 128 hidden units, 4096 samples, -9.4e-9 and -2e-11; dW of 2048
// samples -2.9e-8 and 3e-10.  Signs by rows instead of tiles cost g_pool 4 %).
//
// Products through operand strides and a sliced k range:
//   forward   C_s[B,H]   = sum over the shard's fields of pool[:, f, :] x W[f*D:(f+1)*D, :]
//   g_pool    C[B,F*D]   = dY x W^T
//   dW        C_z[F*D,H] = pool[z-th slice of samples]^T x dY[slice]   (split over samples, summed after)
#include <type_traits>
#include "des_internal.h"

namespace des {
namespace {

constexpr int kRun = 128;                    // products per first-level run of a two-level sum
constexpr long long kTwoLevelDepth = 1024;
constexpr long long kHalvesDepth = 64;       // products from which a sum of fp16 halves is no less exact than one of bf16 thirds
constexpr int kDeepRun = 512;                // products of a deep sum of halves that are summed before they are added to the result
constexpr int kMinSlice = 16;                // samples a slice of dW has at least; slices are multiples of it
constexpr int kForwardGroup = 16;           // row tiles of the forward product whose shards are done together
constexpr int kShallowDepth = 64;           // products of the largest shard up to which the forward product is bound by its writes
constexpr long long kStreamBytes = 128ll << 20;
constexpr int kXcds = 8;                     // dies; consecutive workgroups are handed to them in turn
constexpr uint32_t kGridRow = 1u << 23;      // workgroups per row of a grid; a launch takes fewer than 2^32 threads along x

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

struct GemmArgs {
  const float *A, *B;
  float *C;
  // element (x, k) of an operand, x the row of A or the column of B: P[x*xs + kpos*ks]; one of xs, ks is 1
  uint32_t a_xs, a_ks, b_xs, b_ks;
  int M, N;
  long long c_rs;                     // C(m,n) = C[slice*c_slice + m*c_rs + n]
  long long c_slice;
  // Slice z sums over the positions kpos of the blocks [base, base + blk_len) for base = z*k_shift, += blk_stride,
  // below k_limit, at most k_max positions; the blocks are walked as one range, so a k tile may span several of them.
  uint32_t k_shift, k_limit, k_max, blk_stride, blk_len;
  int tiles_m, tiles_n, slices, m_group;
  bool in_turn = false;               // the dies take the n tiles of one row tile and slice each, in turn; else each an eighth of all tiles
  uint32_t die_run = 0;               // tiles in succession that a die takes, accordingly
  int run;                            // products per first-level run of a two-level sum with the fp32 instruction
  bool stream;                        // the result is larger than what caches keep for who reads it next
};

__device__ inline float4 ld4g(const float *p) { return *reinterpret_cast<const float4 *>(p); }

// Byte offset of 16-byte chunk `chunk` (eight bf16 along k) of row `row` in one plane of rows of 32 bytes.  The chunks of a row
// change places from one group of four rows to the next and the rows of a group turn every second group, so that the operand
// reads (one chunk of consecutive rows) and both kinds of stores spread over the banks.
__device__ inline int lds_offset(int row, int chunk) {
  return (((row & ~3) | ((row + (row >> 3)) & 3)) << 5) | ((chunk ^ ((row >> 2) & 1)) << 4);
}

// Two floats to their three bf16 parts, packed pairwise.  What the cut cannot represent shows in the low half of `odd`: bits
// of the last rest below bf16's smallest denormal (operands under 2^-110).
__device__ inline void split2(float a0, float a1, uint32_t &hi, uint32_t &mid, uint32_t &lo, uint32_t &odd) {
  hi = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){a0, a1}, bf16x2));
  const float r0 = a0 - __uint_as_float(hi << 16), r1 = a1 - __uint_as_float(hi & 0xFFFF0000u);
  mid = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){r0, r1}, bf16x2));
  const float l0 = r0 - __uint_as_float(mid << 16), l1 = r1 - __uint_as_float(mid & 0xFFFF0000u);
  lo = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){l0, l1}, bf16x2));
  odd |= __float_as_uint(l0) | __float_as_uint(l1);
}

// Two floats times `scale`, a power of two, to two fp16 parts: the nearest, and 2^11 times the nearest to the rest.
__device__ inline void halve2(float a0, float a1, float scale, uint32_t &hi, uint32_t &lo) {
  const f16x2 h = __builtin_convertvector((f32x2){a0 * scale, a1 * scale}, f16x2);
  const float up = scale * 2048.f;
  const float l0 = __builtin_fmaf((float)h.x, -2048.f, a0 * up), l1 = __builtin_fmaf((float)h.y, -2048.f, a1 * up);   // exact
  hi = __builtin_bit_cast(uint32_t, h);
  lo = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){l0, l1}, f16x2));
}

// The part of a T x BK operand tile that a thread stages, and its way there.
// kKContig: k is contiguous in memory; BK/4 threads read a row's products side by side, each thread the same four products
// of kUnits rows.  Else x is; a thread reads 4 rows x 4 products.
// Rows past the operand's end repeat its last ones: they only reach outputs that are not stored.
template <int T, int BK, bool kKContig>
struct Operand {
  static constexpr int kTotal = kKContig ? T * BK / 4 : T * BK / 16;    // units of the tile: float4s, 4x4 blocks
  static constexpr int kUnits = kTotal > kBlock ? kTotal / kBlock : 1;  // per thread
  static constexpr int kRowStep = T / kUnits;
  static constexpr int kVecs = kKContig ? kUnits : 4;
  const float *row[kUnits];        // k contiguous: the unit's row; else the unit's four columns
  uint32_t ks, last;               // stride of a position; last position that exists (of a float4 along k: its first)
  uint32_t pos, in_blk;            // position of the thread's products, relative to the first block; offset inside the current one
  int k_in, x0;
  bool active;

  // `t`: which of the tile's units (threads past the last one stay idle).  klen > 0.
  __device__ inline void start(const float *P, uint32_t xs, uint32_t ks_, int x_base, int X, int t, int klen, const GemmArgs &g) {
    ks = ks_;
    active = T == 128 || t < kTotal;               // the large tile keeps every thread busy
    t %= kBlock;
    if constexpr (kKContig) {
      k_in = t % (BK / 4) * 4;
      x0 = t / (BK / 4);
#pragma unroll
      for (int u = 0; u < kUnits; ++u) row[u] = P + (long long)min(x_base + x0 + u * kRowStep, X - 1) * xs;
    } else {
      constexpr int kPerWave = kWave / (BK / 4);   // a wave takes that many groups of four rows at all its products
      k_in = t % kWave / kPerWave * 4;
      x0 = (t / kWave * kPerWave + t % kPerWave) * 4;
      row[0] = P + min(x_base + x0, X - 4);
    }
    const uint32_t k_last = klen - (kKContig ? 4 : 1);
    last = k_last / g.blk_len * g.blk_stride + k_last % g.blk_len;
    const uint32_t q = (uint32_t)k_in / g.blk_len;
    in_blk = k_in - q * g.blk_len;
    pos = q * g.blk_stride + in_blk;
  }
  // Requests the next tile into v and moves on by BK products = `whole` blocks and `rest`.  Whole float4s exist or do
  // not: every extent that a float4 runs along is a multiple of four.  Past the last position it is read again (no
  // branch around a load: the wait for it would be a wait for all of them); blank() then takes that out.
  __device__ inline void load(float4 (&v)[kVecs], uint32_t whole, uint32_t rest, const GemmArgs &g) {
    if (T == 128 || active) {
#pragma unroll
      for (int i = 0; i < kVecs; ++i) {
        if constexpr (kKContig) v[i] = ld4g(row[i] + min(pos, last));
        else v[i] = ld4g(row[0] + (unsigned long long)min(pos + i, last) * ks);
      }
    }
    in_blk += rest;
    pos += whole * g.blk_stride + rest;
    if (in_blk >= g.blk_len) { in_blk -= g.blk_len; pos += g.blk_stride - g.blk_len; }
  }
  // zeros for the products of tile k0 that do not exist
  __device__ inline void blank(float4 (&v)[kVecs], int k0, int klen) const {
#pragma unroll
    for (int i = 0; i < kVecs; ++i)
      if (k0 + k_in + (kKContig ? 0 : i) >= klen) v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  static constexpr int kRows = kKContig ? kUnits : 4;      // rows of which a thread stages products
  // largest magnitude of the staged values of each of the thread's rows, and so far
  __device__ inline void largest(const float4 (&v)[kVecs], float (&top)[kRows]) const {
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
      const float x0 = kKContig ? v[i].x : reinterpret_cast<const float *>(&v[0])[i], x1 = kKContig ? v[i].y : reinterpret_cast<const float *>(&v[1])[i];
      const float x2 = kKContig ? v[i].z : reinterpret_cast<const float *>(&v[2])[i], x3 = kKContig ? v[i].w : reinterpret_cast<const float *>(&v[3])[i];
      top[i] = fmaxf(fmaxf(top[i], fabsf(x0)), fabsf(x1));
      top[i] = fmaxf(fmaxf(top[i], fabsf(x2)), fabsf(x3));
      asm volatile("" : "+v"(top[i]));             // now: done later, it would keep the values in registers that the next tile is loaded to
    }
  }
  // largest of each row over the BK/4 lanes that its products are spread over
  __device__ inline void row_tops(const float (&top)[kRows], float (&of_row)[kRows]) const {
    constexpr int kNext = kKContig ? 1 : kWave / (BK / 4);
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
      of_row[i] = top[i];
#pragma unroll
      for (int m = kNext; m < kNext * (BK / 4); m <<= 1) of_row[i] = fmaxf(of_row[i], __shfl_xor(of_row[i], m, kWave));
    }
  }
  __device__ inline int tile_row(int i) const { return kKContig ? x0 + i * kRowStep : x0 + i; }
  // the staged values times their rows' scales as fp16 parts into the two planes at `plane`
  __device__ inline void store_halves(const float4 (&v)[kVecs], char *plane, const float (&scale)[kRows]) const {
    static_assert(BK == 16, "two chunks per row");
    if (T != 128 && !active) return;
    const float *f = reinterpret_cast<const float *>(v);
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
      uint2 p[2];
      halve2(f[kKContig ? i * 4 : i], f[kKContig ? i * 4 + 1 : 4 + i], scale[i], p[0].x, p[1].x);
      halve2(f[kKContig ? i * 4 + 2 : 8 + i], f[kKContig ? i * 4 + 3 : 12 + i], scale[i], p[0].y, p[1].y);
      const int at = lds_offset(tile_row(i), k_in / 8) + (k_in & 4) * 2;
#pragma unroll
      for (int q = 0; q < 2; ++q) *reinterpret_cast<uint2 *>(plane + q * (T * 32) + at) = p[q];
    }
  }
  // cuts the staged values into the three planes at `plane` (T rows each), their signs flipped if `flip` is the sign bit
  template <bool kFlip>
  __device__ inline void store_split(const float4 (&v)[kVecs], char *plane, uint32_t flip, uint32_t &odd) const {
    static_assert(BK == 16, "two chunks per row");
    if (T != 128 && !active) return;
    float f[kVecs * 4];
#pragma unroll
    for (int i = 0; i < kVecs * 4; ++i) {
      const float x = reinterpret_cast<const float *>(v)[i];
      f[i] = kFlip ? __uint_as_float(__float_as_uint(x) ^ flip) : x;
    }
    if constexpr (kKContig) {
#pragma unroll
      for (int u = 0; u < kUnits; ++u) {
        uint2 p[3];
        split2(f[u * 4], f[u * 4 + 1], p[0].x, p[1].x, p[2].x, odd);
        split2(f[u * 4 + 2], f[u * 4 + 3], p[0].y, p[1].y, p[2].y, odd);
        const int at = lds_offset(x0 + u * kRowStep, k_in / 8) + (k_in & 4) * 2;
#pragma unroll
        for (int q = 0; q < 3; ++q) *reinterpret_cast<uint2 *>(plane + q * (T * 32) + at) = p[q];
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {                // transposed by picking registers
        uint2 p[3];
        split2(f[j], f[4 + j], p[0].x, p[1].x, p[2].x, odd);
        split2(f[8 + j], f[12 + j], p[0].y, p[1].y, p[2].y, odd);
        const int at = lds_offset(x0 + j, k_in / 8) + (k_in & 4) * 2;
#pragma unroll
        for (int q = 0; q < 3; ++q) *reinterpret_cast<uint2 *>(plane + q * (T * 32) + at) = p[q];
      }
    }
  }
};

// The same for the fp32 instruction: the part of a T x BK tile that a thread stages as it is, in memory order.  k contiguous: as
// above; else a thread reads a few successive products (1, 2 or 4, never of two blocks) of four neighbouring rows.
template <int T, int BK, bool kKContig>
struct Plain {
  static constexpr int kVecs = T * BK / 4 / kBlock;
  static constexpr int kRowStep = T / kVecs;
  static constexpr int kPitch = kKContig ? BK + 4 : T + 4;
  static constexpr int kFloats = (kKContig ? T : BK) * kPitch;
  const float *row[kKContig ? kVecs : 1];
  uint32_t ks, last, pos, in_blk;
  int k_in, x0;

  __device__ inline void start(const float *P, uint32_t xs, uint32_t ks_, int x_base, int X, int klen, const GemmArgs &g) {
    static_assert(4 % kVecs == 0 || kKContig, "a block is a multiple of four products");
    const int t = threadIdx.x;
    ks = ks_;
    if constexpr (kKContig) {
      k_in = t % (BK / 4) * 4;
      x0 = t / (BK / 4);
#pragma unroll
      for (int u = 0; u < kVecs; ++u) row[u] = P + (long long)min(x_base + x0 + u * kRowStep, X - 1) * xs;
    } else {
      k_in = t / (T / 4) * kVecs;
      x0 = t % (T / 4) * 4;
      row[0] = P + min(x_base + x0, X - 4);
    }
    const uint32_t k_last = klen - (kKContig ? 4 : 1);
    last = k_last / g.blk_len * g.blk_stride + k_last % g.blk_len;
    const uint32_t q = (uint32_t)k_in / g.blk_len;
    in_blk = k_in - q * g.blk_len;
    pos = q * g.blk_stride + in_blk;
  }
  __device__ inline void load(float4 (&v)[kVecs], uint32_t whole, uint32_t rest, const GemmArgs &g) {
#pragma unroll
    for (int i = 0; i < kVecs; ++i) {
      if constexpr (kKContig) v[i] = ld4g(row[i] + min(pos, last));
      else v[i] = ld4g(row[0] + (unsigned long long)min(pos + i, last) * ks);
    }
    in_blk += rest;
    pos += whole * g.blk_stride + rest;
    if (in_blk >= g.blk_len) { in_blk -= g.blk_len; pos += g.blk_stride - g.blk_len; }
  }
  // zeros for the products of tile k0 that do not exist
  __device__ inline void blank(float4 (&v)[kVecs], int k0, int klen) const {
#pragma unroll
    for (int i = 0; i < kVecs; ++i)
      if (k0 + k_in + (kKContig ? 0 : i) >= klen) v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  __device__ inline void store(const float4 (&v)[kVecs], float *tile) const {
#pragma unroll
    for (int i = 0; i < kVecs; ++i)
      *reinterpret_cast<float4 *>(tile + (kKContig ? (x0 + i * kRowStep) * kPitch + k_in : (k_in + i) * kPitch + x0)) = v[i];
  }
  static __device__ inline float at(const float *tile, int x, int k) { return kKContig ? tile[x * kPitch + k] : tile[k * kPitch + x]; }
};

// One workgroup's place: output tile, slice and the slice's products.
template <int T>
struct Place {
  int m0, n0, z, klen;
  int sign;                        // 1: the split product's first run is accumulated with the opposite sign
  uint32_t first;                  // position of the slice's first product
  bool ok;
  // kInTurn: g.in_turn may be set (the division tells in short products)
  template <bool kInTurn>
  __device__ inline Place(const GemmArgs &g, uint32_t block, std::integral_constant<bool, kInTurn>) {
    // Every die takes contiguous runs of tiles.  They are numbered n first, then m inside a group of m_group tiles, then
    // the slice, then the group: tiles that read the same rows of A follow each other, a slice's part of B is used by a
    // whole group, and the slices of a group (in the forward product: the shards' columns of the same rows of A) are
    // done together, before the next rows.
    const uint32_t total = (uint32_t)g.tiles_m * g.tiles_n * g.slices, turn = block / kXcds;
    uint32_t round = 0;
    if (kInTurn && g.in_turn) round = turn / g.die_run;
    const uint32_t tile = (round * kXcds + block % kXcds) * g.die_run + (turn - round * g.die_run);
    ok = tile < total;
    const uint32_t per_group = (uint32_t)g.tiles_n * g.m_group * g.slices, group = tile / per_group;
    const uint32_t in_group = min((uint32_t)g.m_group, g.tiles_m - group * g.m_group);
    const uint32_t mz = (tile - group * per_group) / g.tiles_n;
    n0 = (int)(tile - group * per_group - mz * g.tiles_n) * T;
    z = (int)(mz / in_group);
    m0 = (int)(group * g.m_group + mz % in_group) * T;
    sign = (m0 / T ^ n0 / T ^ z) & 1;
    const unsigned long long at = (unsigned long long)z * g.k_shift;      // may lie past the end: a shard without a field
    first = at < g.k_limit ? (uint32_t)at : g.k_limit;
    const uint32_t avail = g.k_limit - first, blocks = avail / g.blk_stride, tail = avail - blocks * g.blk_stride;
    klen = (int)min(blocks * g.blk_len + min(tail, g.blk_len), g.k_max);
  }
};

// Sums of a wave: NB x NB blocks of 32x32.  kTwoLevel (long contractions; the weight gradient sums over the whole batch):
// the matrix cores accumulate runs of kRun products from zero and each run is then added into `total`, so small
// products are never added to a large running sum.  Short contractions keep the single accumulator and the registers
// that saves.
template <int NB, bool kTwoLevel>
struct Sums {
  f32x16 acc[NB][NB], total[NB][NB];
  __device__ inline void clear() {
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) { acc[i][j][r] = 0.f; total[i][j][r] = 0.f; }
  }
  __device__ inline void flush() {
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        total[i][j] += acc[i][j];
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
      }
  }
  __device__ inline void negate() {                // a sum of zeros stays +0
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        // opaque, so that it stays where it is: the compiler would negate ahead of the branch around it, every other step
        asm volatile("" : "+v"(acc[i][j]));
        acc[i][j] = 0.f - acc[i][j];
      }
  }
  // The finished sum; flush() first if there are two levels.
  __device__ inline float value(int i, int j, int r) const { return kTwoLevel ? total[i][j][r] : acc[i][j][r]; }
  __device__ inline bool finite() const {
    float any = 0.f;                               // times zero: NaN for an infinity or NaN, else zero
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) any = __builtin_fmaf(value(i, j, r), 0.f, any);
    return any == 0.f;
  }
  // adds what store() left in the matrix, a block's sixteen values at a time
  __device__ inline void add_stored(const GemmArgs &g, int z, int m_wave, int n_wave) {
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        int row0 = m_wave + i * 32 + (lane >> 5) * 4;
        asm volatile("" : "+v"(row0));             // the addresses are made here: ahead of the loop around this they would all be kept
        const float *C = g.C + (long long)z * g.c_slice + min(n_wave + j * 32 + (lane & 31), g.N - 1);
        float old[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) old[r] = C[(long long)min(row0 + (r >> 2) * 8 + (r & 3), g.M - 1) * g.c_rs];
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] += old[r];
      }
  }
  // element r of a 32x32 block sits at row (r/4)*8 + (lane/32)*4 + r%4, column lane%32
  __device__ inline void store(const GemmArgs &g, int z, int m_wave, int n_wave) const {
    const int lane = threadIdx.x & (kWave - 1);
    float *C = g.C + (long long)z * g.c_slice;
    // a block inside the matrix: no comparisons, addresses by addition
    const auto inside = [&](auto put) {
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        float *row = C + (long long)(m_wave + i * 32 + (lane >> 5) * 4) * g.c_rs + n_wave + (lane & 31);
        asm volatile("" : "+v"(row));              // see add_stored
#pragma unroll
        for (int r = 0; r < 16; ++r) {
#pragma unroll
          for (int j = 0; j < NB; ++j) put(row + j * 32, value(i, j, r));
          row += (r & 3) == 3 ? 5 * g.c_rs : g.c_rs;
        }
      }
    };
    if (m_wave + NB * 32 <= g.M && n_wave + NB * 32 <= g.N) {     // uniform per wave
      if (g.stream) inside([](float *p, float v) { __builtin_nontemporal_store(v, p); });
      else inside([](float *p, float v) { *p = v; });
      return;
    }
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int col = n_wave + j * 32 + (lane & 31);
        int row0 = m_wave + i * 32 + (lane >> 5) * 4;
        asm volatile("" : "+v"(row0));             // see add_stored
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = row0 + (r >> 2) * 8 + (r & 3);
          if (row < g.M && col < g.N) C[(long long)row * g.c_rs + col] = value(i, j, r);
        }
      }
  }
};

// The whole contraction of one tile with the fp32 instruction.
constexpr int kPlainBK = 32;                      // ... of two-level sums and small tiles; see launch()
template <int T, int BK, bool kAKContig, bool kBKContig>
constexpr int plain_floats() { return Plain<T, BK, kAKContig>::kFloats + Plain<T, BK, kBKContig>::kFloats; }

template <int T, int BK, bool kAKContig, bool kBKContig, bool kTwoLevel>
__device__ inline void multiply_f32(const GemmArgs &g, const Place<T> &at, float *lds, Sums<T / 64, kTwoLevel> &sums) {
  constexpr int NB = T / 64;
  using OpA = Plain<T, BK, kAKContig>;
  using OpB = Plain<T, BK, kBKContig>;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int xa = (wave >> 1) * (T / 2) + (lane & 31), xb = (wave & 1) * (T / 2) + (lane & 31), lk = lane >> 5;
  const uint32_t whole = BK / g.blk_len, rest = BK - whole * g.blk_len;
  const int klen = at.klen;
  sums.clear();
  if (klen == 0) return;
  float *ta = lds, *tb = lds + OpA::kFloats;
  OpA oa;
  OpB ob;
  float4 va[OpA::kVecs], vb[OpB::kVecs];
  oa.start(g.A + (unsigned long long)at.first * g.a_ks, g.a_xs, g.a_ks, at.m0, g.M, klen, g);
  ob.start(g.B + (unsigned long long)at.first * g.b_ks, g.b_xs, g.b_ks, at.n0, g.N, klen, g);
  oa.load(va, whole, rest, g);
  ob.load(vb, whole, rest, g);
  int run = 0;
  for (int k0 = 0; k0 < klen; k0 += BK) {
    if (k0 + BK > klen) { oa.blank(va, k0, klen); ob.blank(vb, k0, klen); }
    __syncthreads();                              // previous tile fully consumed
    oa.store(va, ta);
    ob.store(vb, tb);
    __syncthreads();
    if (k0 + BK < klen) {                         // the next tile travels while this one is multiplied
      oa.load(va, whole, rest, g);
      ob.load(vb, whole, rest, g);
    }
    // operands of step kk+2 are read from LDS before the matrix instructions of step kk are issued
    float a[NB], b[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) { a[i] = OpA::at(ta, xa + i * 32, lk); b[i] = OpB::at(tb, xb + i * 32, lk); }
#pragma unroll
    for (int kk = 0; kk < BK; kk += 2) {
      if (kk == 16 && k0 + 16 >= klen) break;     // uniform: nothing but padding from here on
      float an[NB], bn[NB];
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        an[i] = bn[i] = 0.f;
        if (kk + 2 < BK) { an[i] = OpA::at(ta, xa + i * 32, kk + 2 + lk); bn[i] = OpB::at(tb, xb + i * 32, kk + 2 + lk); }
      }
      __builtin_amdgcn_sched_barrier(0);          // keep the reads above: the scheduler would sink them to their use
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) sums.acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], sums.acc[i][j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < NB; ++i) { a[i] = an[i]; b[i] = bn[i]; }
    }
    if (kTwoLevel && (run += BK) == g.run) { run = 0; sums.flush(); }
  }
  if (kTwoLevel) sums.flush();
}

template <int T, int BK, bool kAKContig, bool kBKContig, bool kTwoLevel>
__global__ __launch_bounds__(kBlock, 2) void k_gemm_f32(const GemmArgs g) {
  __shared__ __align__(16) float lds[plain_floats<T, BK, kAKContig, kBKContig>()];
  const Place<T> at(g, blockIdx.y * kGridRow + blockIdx.x, std::true_type{});
  if (!at.ok) return;                             // uniform per workgroup
  Sums<T / 64, kTwoLevel> sums;
  multiply_f32<T, BK, kAKContig, kBKContig, kTwoLevel>(g, at, lds, sums);
  const int wave = threadIdx.x / kWave;
  sums.store(g, at.z, at.m0 + (wave >> 1) * (T / 2), at.n0 + (wave & 1) * (T / 2));
}

// Staging of both operands' tiles as bf16 planes.  Where both need half of the threads or less, each thread stages one of the
// two (no branch, and one set of registers).
template <int T, int BK, bool kAKContig, bool kBKContig>
struct SplitStage {
  static constexpr int kOperandBytes = 3 * T * 32;
  static constexpr bool kShared = !kAKContig && !kBKContig;
  using OpA = Operand<T, BK, kAKContig>;
  using OpB = Operand<T, BK, kBKContig>;
  OpA oa;
  OpB ob;
  float4 va[2][OpA::kVecs], vb[2][OpB::kVecs];    // two tiles under way
  char *to;
  uint32_t flip;                                  // the sign bit for threads that stage A, in every second tile
  __device__ inline void start(const GemmArgs &g, const Place<T> &at, char *lds) {
    const float *A = g.A + (unsigned long long)at.first * g.a_ks, *B = g.B + (unsigned long long)at.first * g.b_ks;
    if constexpr (kShared) {
      constexpr int n = Operand<T, BK, false>::kTotal;
      const bool second = threadIdx.x / n == 1;   // threads past the second operand's units: idle
      to = lds + (second ? kOperandBytes : 0);
      flip = second || !at.sign ? 0u : 0x80000000u;
      oa.start(second ? B : A, 1, second ? g.b_ks : g.a_ks, second ? at.n0 : at.m0, second ? g.N : g.M,
               second ? threadIdx.x - n : threadIdx.x, at.klen, g);
    } else {
      to = lds;
      flip = at.sign ? 0x80000000u : 0u;
      oa.start(A, g.a_xs, g.a_ks, at.m0, g.M, threadIdx.x, at.klen, g);
      ob.start(B, g.b_xs, g.b_ks, at.n0, g.N, threadIdx.x ^ (kBlock / 2), at.klen, g);
    }
  }
  template <int kSet>
  __device__ inline void load(uint32_t whole, uint32_t rest, const GemmArgs &g) {
    oa.load(va[kSet], whole, rest, g);
    if constexpr (!kShared) ob.load(vb[kSet], whole, rest, g);
  }
  template <int kSet>
  __device__ inline void blank(int k0, int klen) {
    if (k0 + BK <= klen) return;                  // uniform
    oa.blank(va[kSet], k0, klen);
    if constexpr (!kShared) ob.blank(vb[kSet], k0, klen);
  }
  template <int kSet>
  __device__ inline void store(int buf, uint32_t &odd) {
    oa.template store_split<true>(va[kSet], to + buf, flip, odd);
    if constexpr (!kShared) ob.template store_split<false>(vb[kSet], to + buf + kOperandBytes, 0u, odd);
  }
};

constexpr int at_least(int bytes, int other) { return bytes > other ? bytes : other; }
template <int T, bool kAKContig, bool kBKContig>
constexpr int split_bytes() { return at_least(2 * 6 * T * 32, plain_floats<T, kPlainBK, kAKContig, kBKContig>() * 4); }
template <int T, bool kAKContig, bool kBKContig>
__device__ inline void multiply_split(const GemmArgs &g, uint32_t block, char *lds) {
  constexpr int NB = T / 64, BK = 16;
  constexpr int kPlane = T * 32, kBuffer = 6 * kPlane;      // bytes: one bf16 plane of one operand; both operands' planes
  const Place<T> at(g, block, std::false_type{});
  if (!at.ok) return;                             // uniform per workgroup
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int m_wave = (wave >> 1) * (T / 2), n_wave = (wave & 1) * (T / 2);
  const int ra = lds_offset(m_wave + (lane & 31), lane >> 5), rb = 3 * kPlane + lds_offset(n_wave + (lane & 31), lane >> 5);
  const uint32_t whole = BK / g.blk_len, rest = BK - whole * g.blk_len;
  const int klen = at.klen;
  Sums<NB, false> sums;
  sums.clear();
  uint32_t odd = 0;
  if (klen > 0) {
    SplitStage<T, BK, kAKContig, kBKContig> stage;
    stage.start(g, at, lds);
    stage.template load<0>(whole, rest, g);
    stage.template load<1>(whole, rest, g);
    stage.template blank<0>(0, klen);
    stage.template store<0>(0, odd);
    stage.template load<0>(whole, rest, g);
    // multiplies the tile at k0 out of buffer kBuf and, unless it is the last, cuts the next one into the other buffer and requests
    // the third one on
    auto step = [&](auto buf_c, auto last_c, int k0) {
      constexpr int kBuf = decltype(buf_c)::value, kNext = 1 - kBuf;
      constexpr bool kLast = decltype(last_c)::value;
      if constexpr (!kLast) stage.template blank<kNext>(k0 + BK, klen);
      __syncthreads();                            // the current tile is written, the other buffer fully read
      bf16x8 a[3][NB], b[3][NB];
#pragma unroll
      for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int i = 0; i < NB; ++i) {
          a[q][i] = *reinterpret_cast<const bf16x8 *>(lds + kBuf * kBuffer + q * kPlane + i * 1024 + ra);
          b[q][i] = *reinterpret_cast<const bf16x8 *>(lds + kBuf * kBuffer + q * kPlane + i * 1024 + rb);
        }
      if constexpr (!kLast) stage.template store<kNext>(kNext * kBuffer, odd);
      // smallest terms first
      constexpr int qa[6] = {2, 0, 1, 1, 0, 0}, qb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
      for (int p = 0; p < 6; ++p)
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j)
            sums.acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[qa[p]][i], b[qb[p]][j], sums.acc[i][j], 0, 0, 0);
      if constexpr (!kLast) stage.template load<kNext>(whole, rest, g);
    };
    const std::integral_constant<int, 0> even{};
    const std::integral_constant<int, 1> uneven{};
    const std::false_type more{};
    // The last tile by itself, so that nothing past the end is cut and requested: of a single tile that is half of the work
    // (131072 x 12800 outputs of 16 products: 1383 -> 1234 us; dW of 256 samples, 2048 x 1024: 28.7 -> 27.4 us).  The small tile
    // with both operands along k is slower so (64 x 2048 outputs of 1024 products: 33.0 -> 35.6 us).
    constexpr bool kPeel = T == 128 || !kAKContig;
    int k0 = 0;
    for (; kPeel ? k0 + 2 * BK < klen : k0 < klen; k0 += 2 * BK) {
      step(even, more, k0);
      if (kPeel || k0 + BK < klen) step(uneven, more, k0 + BK);
    }
    if constexpr (kPeel) {
      if (k0 + BK < klen) {
        step(even, more, k0);
        step(uneven, std::true_type{}, k0 + BK);
      } else {
        step(even, std::true_type{}, k0);
      }
    }
    if (at.sign) sums.negate();
  }
  // An infinity or NaN among the operands (times a zero part it makes a NaN of what should stay infinite), a product or sum past
  // fp32's range (its parts' products can be infinities of both signs, a NaN again): either leaves a sum that is not
  // finite.  Then, or if an operand was too small for three bf16 parts, the tile is computed again with the fp32 instruction.
  if (__syncthreads_or((odd & 0xFFFFu) != 0 || !sums.finite()))
    multiply_f32<T, kPlainBK, kAKContig, kBKContig, false>(g, at, reinterpret_cast<float *>(lds), sums);
  sums.store(g, at.z, at.m0 + m_wave, at.n0 + n_wave);
}

// Largest of a wave's values, none of them negative, in its last lane.
__device__ inline float wave_max(float v) {
  const auto step = [&](auto ctrl) {                 // lanes that a step does not reach take a zero
    v = fmaxf(v, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), decltype(ctrl)::value, 0xF, 0xF, true)));
  };
  step(std::integral_constant<int, 0x111>{});        // row_shr 1, 2, 4, 8: the last lane of every 16
  step(std::integral_constant<int, 0x112>{});
  step(std::integral_constant<int, 0x114>{});
  step(std::integral_constant<int, 0x118>{});
  step(std::integral_constant<int, 0x142>{});        // row_bcast 15 and 31
  step(std::integral_constant<int, 0x143>{});
  return v;
}

// Staging of both operands' tiles as planes of fp16 parts, and their rows' scales.
template <int T, int BK, bool kAKContig, bool kBKContig>
struct HalfStage {
  static constexpr int kOperandBytes = 2 * T * 32;
  static constexpr bool kShared = !kAKContig && !kBKContig;
  using OpA = Operand<T, BK, kAKContig>;
  using OpB = Operand<T, BK, kBKContig>;
  OpA oa;
  OpB ob;
  float4 va[2][OpA::kVecs], vb[2][OpB::kVecs];    // the two halves of the tile under way
  float top_a[OpA::kRows], top_b[OpB::kRows];
  char *to;
  float scale_a[OpA::kRows], scale_b[OpB::kRows]; // of the rows that the thread stages; A's take the sign of the current run
  bool second;                                    // kShared: the thread stages B
  // the products from k0 on, `len` of them
  __device__ inline void start(const GemmArgs &g, const Place<T> &at, char *lds, int k0, int len) {
    const float *A = g.A + (unsigned long long)(at.first + k0) * g.a_ks, *B = g.B + (unsigned long long)(at.first + k0) * g.b_ks;
    if constexpr (kShared) {
      constexpr int n = Operand<T, BK, false>::kTotal;
      second = threadIdx.x / n == 1;              // threads past the second operand's units: idle
      to = lds + (second ? kOperandBytes : 0);
      oa.start(second ? B : A, 1, second ? g.b_ks : g.a_ks, second ? at.n0 : at.m0, second ? g.N : g.M,
               second ? threadIdx.x - n : threadIdx.x, len, g);
    } else {
      second = false;
      to = lds;
      oa.start(A, g.a_xs, g.a_ks, at.m0, g.M, threadIdx.x, len, g);
      ob.start(B, g.b_xs, g.b_ks, at.n0, g.N, threadIdx.x ^ (kBlock / 2), len, g);
    }
  }
  __device__ inline void clear() {
#pragma unroll
    for (int i = 0; i < OpA::kRows; ++i) top_a[i] = 0.f;
#pragma unroll
    for (int i = 0; i < OpB::kRows; ++i) top_b[i] = 0.f;
  }
  // The rows' scales from the magnitudes of the first tile: a row's largest is brought to 1 .. 2, a row of zeros is taken for one with
  // the tile's largest.  Every second 64 rows (and slice of A) take the other sign, so that a result does not depend on the tile's size.
  // `tops`: LDS, a float per wave and operand; `inverse`: LDS, where each operand's T rows leave 1 / scale.
  __device__ inline void set_scales(float (*tops)[kBlock / kWave], float (*inverse)[T], const Place<T> &at) {
    float row_a[OpA::kRows], row_b[OpB::kRows], ta = 0.f, tb = 0.f;
    oa.largest(va[0], top_a);
    oa.largest(va[1], top_a);
    oa.row_tops(top_a, row_a);
#pragma unroll
    for (int i = 0; i < OpA::kRows; ++i) ta = fmaxf(ta, row_a[i]);
    if constexpr (!kShared) {
      ob.largest(vb[0], top_b);
      ob.largest(vb[1], top_b);
      ob.row_tops(top_b, row_b);
#pragma unroll
      for (int i = 0; i < OpB::kRows; ++i) tb = fmaxf(tb, row_b[i]);
    } else {
      tb = second ? ta : 0.f;
      ta = second ? 0.f : ta;
    }
    ta = wave_max(ta);
    tb = wave_max(tb);
    const int wave = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == kWave - 1) { tops[0][wave] = ta; tops[1][wave] = tb; }
    __syncthreads();
    ta = tb = 0.f;
#pragma unroll
    for (int w = 0; w < kBlock / kWave; ++w) { ta = fmaxf(ta, tops[0][w]); tb = fmaxf(tb, tops[1][w]); }
    const auto exponent = [](float row, float tile) { // of a power of two within 2^-60 .. 2^60, so that the product of two is one as well
      const float t = row == 0.f ? tile : row;
      return t == 0.f ? 0 : min(max(127 - (int)(__float_as_uint(t) >> 23), -60), 60);
    };
    const auto power = [](int e, int sign) { return __uint_as_float((uint32_t)(127 + e) << 23 | (uint32_t)sign << 31); };
    const bool b_too = kShared && second;
#pragma unroll
    for (int i = 0; i < OpA::kRows; ++i) {
      const int e = exponent(row_a[i], b_too ? tb : ta), row = oa.tile_row(i);
      const int sign = ((b_too ? (at.n0 + row) >> 6 : (at.m0 + row) >> 6 ^ at.z) & 1);
      scale_a[i] = power(e, sign);
      if (oa.k_in == 0 && (T == 128 || oa.active)) inverse[b_too ? 1 : 0][row] = power(-e, sign);
    }
    if constexpr (!kShared) {
#pragma unroll
      for (int i = 0; i < OpB::kRows; ++i) {
        const int e = exponent(row_b[i], tb), row = ob.tile_row(i), sign = (at.n0 + row) >> 6 & 1;
        scale_b[i] = power(e, sign);
        if (ob.k_in == 0 && (T == 128 || ob.active)) inverse[1][row] = power(-e, sign);
      }
    }
  }
  template <int kSet>
  __device__ inline void load(uint32_t whole, uint32_t rest, const GemmArgs &g) {
    oa.load(va[kSet], whole, rest, g);
    if constexpr (!kShared) ob.load(vb[kSet], whole, rest, g);
  }
  template <int kSet>
  __device__ inline void blank(int k0, int klen) {
    if (k0 + BK <= klen) return;                  // uniform
    oa.blank(va[kSet], k0, klen);
    if constexpr (!kShared) ob.blank(vb[kSet], k0, klen);
  }
  __device__ inline void turn() {                 // A's sign is the other one from here on
#pragma unroll
    for (int i = 0; i < OpA::kRows; ++i)
      if (!(kShared && second)) scale_a[i] = -scale_a[i];
  }
  template <int kSet>
  __device__ inline void store(int buf) {
    oa.largest(va[kSet], top_a);
    oa.store_halves(va[kSet], to + buf, scale_a);
    if constexpr (!kShared) {
      ob.largest(vb[kSet], top_b);
      ob.store_halves(vb[kSet], to + buf + kOperandBytes, scale_b);
    }
  }
  // Is one of the thread's rows, whose first products were zeros, so small that its parts hold less than fp32 does?
  __device__ inline bool too_small() const {
    float row_a[OpA::kRows];
    oa.row_tops(top_a, row_a);
    bool small = false;
#pragma unroll
    for (int i = 0; i < OpA::kRows; ++i) small |= row_a[i] != 0.f && row_a[i] * fabsf(scale_a[i]) < 0x1p-10f;
    small &= T == 128 || oa.active;
    if constexpr (!kShared) {
      float row_b[OpB::kRows];
      ob.row_tops(top_b, row_b);
      bool small_b = false;
#pragma unroll
      for (int i = 0; i < OpB::kRows; ++i) small_b |= row_b[i] != 0.f && row_b[i] * fabsf(scale_b[i]) < 0x1p-10f;
      small |= small_b && (T == 128 || ob.active);
    }
    return small;
  }
};

template <int T, bool kAKContig, bool kBKContig>
constexpr int halves_bytes() { return at_least(2 * 8 * T * 32, plain_floats<T, kPlainBK, kAKContig, kBKContig>() * 4) + 2 * T * 4 + 2 * (kBlock / kWave) * 4; }
template <int T, bool kAKContig, bool kBKContig, bool kDeep>
__device__ inline void multiply_halves(const GemmArgs &g, uint32_t block, char *lds) {
  constexpr int NB = T / 64, BK = 16, kStep = 2 * BK;
  constexpr int kPlane = T * 32, kHalf = 4 * kPlane, kBuffer = 2 * kHalf;   // bytes: one part of one operand's half tile; both operands'; both halves
  char *const behind = lds + at_least(2 * kBuffer, plain_floats<T, kPlainBK, kAKContig, kBKContig>() * 4);
  float(*const inverse)[T] = reinterpret_cast<float(*)[T]>(behind);
  float(*const tops)[kBlock / kWave] = reinterpret_cast<float(*)[kBlock / kWave]>(behind + 2 * T * 4);
  const Place<T> at(g, block, std::false_type{});
  if (!at.ok) return;                             // uniform per workgroup
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int m_wave = (wave >> 1) * (T / 2), n_wave = (wave & 1) * (T / 2);
  const int ra = lds_offset(m_wave + (lane & 31), lane >> 5), rb = 2 * kPlane + lds_offset(n_wave + (lane & 31), lane >> 5);
  const uint32_t whole = BK / g.blk_len, rest = BK - whole * g.blk_len;
  Sums<NB, false> sums, cross;                    // of the products of leading parts, and of those with one rest, times 2^11
  sums.clear();
  cross.clear();
  bool again = false;
  HalfStage<T, BK, kAKContig, kBKContig> stage;
  stage.clear();
  for (int done = 0; done < at.klen; done += kDeepRun) {       // once, unless kDeep
    const int len = kDeep ? min(at.klen - done, kDeepRun) : at.klen;
    stage.start(g, at, lds, done, len);
    const auto load = [&]() {
      stage.template load<0>(whole, rest, g);
      stage.template load<1>(whole, rest, g);
    };
    load();
    stage.template blank<0>(0, len);
    stage.template blank<1>(BK, len);
    if (done == 0) stage.set_scales(tops, inverse, at);
    else __syncthreads();                         // the last tile has been read
    stage.template store<0>(0);
    stage.template store<1>(kHalf);
    load();
    // multiplies a half of the tile in buffer `buf` and, unless it is the last tile, cuts that half of the next one into the other buffer
    auto half = [&](auto half_c, auto last_c, int buf) {
      constexpr int kSet = decltype(half_c)::value;
      f16x8 a[2][NB], b[2][NB];
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int i = 0; i < NB; ++i) {
          a[q][i] = *reinterpret_cast<const f16x8 *>(lds + buf + (kSet * kHalf + q * kPlane + i * 1024) + ra);
          b[q][i] = *reinterpret_cast<const f16x8 *>(lds + buf + (kSet * kHalf + q * kPlane + i * 1024) + rb);
        }
      if constexpr (!decltype(last_c)::value) stage.template store<kSet>((buf ^ kBuffer) + kSet * kHalf);
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          cross.acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[1][i], b[0][j], cross.acc[i][j], 0, 0, 0);
          sums.acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0][i], b[0][j], sums.acc[i][j], 0, 0, 0);
        }
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          cross.acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0][i], b[1][j], cross.acc[i][j], 0, 0, 0);
    };
    const std::integral_constant<int, 0> first{};
    const std::integral_constant<int, 1> second{};
    int k0 = 0, buf = 0;
    for (; k0 + kStep < len; k0 += kStep, buf ^= kBuffer) {
      stage.template blank<0>(k0 + kStep, len);
      stage.template blank<1>(k0 + kStep + BK, len);
      __syncthreads();                            // the current tile is written, the other buffer fully read
      const bool turn = (k0 + kStep) % kRun == 0;
      if (turn) stage.turn();
      half(first, std::false_type{}, buf);
      half(second, std::false_type{}, buf);
      load();
      if (turn) { sums.negate(); cross.negate(); }
    }
    __syncthreads();
    half(first, std::true_type{}, buf);
    if (k0 + BK < len) half(second, std::true_type{}, buf);
    // both sums to one, in the operands' own scale and with their sign
    const bool odd = ((len - 1) / kRun & 1) != 0;
    if (kDeep && odd) stage.turn();
    const float sign = odd ? -1.f : 1.f;
    float of_col[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) of_col[j] = sign * inverse[1][n_wave + j * 32 + (lane & 31)];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 of_row = *reinterpret_cast<const float4 *>(&inverse[0][m_wave + i * 32 + q * 8 + (lane >> 5) * 4]);
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) {           // (adding zero: a sum of zeros is +0)
            const float v = __builtin_fmaf(cross.acc[i][j][q * 4 + r], 0x1p-11f, sums.acc[i][j][q * 4 + r]);
            sums.acc[i][j][q * 4 + r] = __builtin_fmaf(v, reinterpret_cast<const float *>(&of_row)[r] * of_col[j], 0.f);
          }
      }
    if (!kDeep) break;
    if (done > 0) sums.add_stored(g, at.z, at.m0 + m_wave, at.n0 + n_wave);
    if (done + len < at.klen) {
      sums.store(g, at.z, at.m0 + m_wave, at.n0 + n_wave);
      sums.clear();
      cross.clear();
    }
  }
  again = at.klen > 0 && stage.too_small();
  if (__syncthreads_or(again || !sums.finite())) {
    Sums<NB, kDeep> plain;
    multiply_f32<T, kPlainBK, kAKContig, kBKContig, kDeep>(g, at, reinterpret_cast<float *>(lds), plain);
    plain.store(g, at.z, at.m0 + m_wave, at.n0 + n_wave);
  } else {
    sums.store(g, at.z, at.m0 + m_wave, at.n0 + n_wave);
  }
}

template <int T, bool kAKContig, bool kBKContig>
__global__ __launch_bounds__(kBlock, 2) void k_gemm_split(const GemmArgs g) {
  __shared__ __align__(16) char lds[split_bytes<T, kAKContig, kBKContig>()];
  multiply_split<T, kAKContig, kBKContig>(g, blockIdx.x, lds);
}

template <int T, bool kAKContig, bool kBKContig, bool kDeep>
__global__ __launch_bounds__(kBlock, 2) void k_gemm_halves(const GemmArgs g) {
  __shared__ __align__(16) char lds[halves_bytes<T, kAKContig, kBKContig>()];
  multiply_halves<T, kAKContig, kBKContig, kDeep>(g, blockIdx.x, lds);
}

// Both gradient products in one launch, where each by itself leaves most of the chip idle: the first n_w workgroups take dW's tiles,
// the others g_pool's.  kWHalves, kGHalves: from fp16 halves, else from bf16 thirds.
template <int T, bool kWHalves, bool kGHalves, bool kWDeep = false>
__global__ __launch_bounds__(kBlock, 2) void k_gemm_both(const GemmArgs w, const GemmArgs g, uint32_t n_w) {
  constexpr int kWBytes = kWHalves ? halves_bytes<T, false, false>() : split_bytes<T, false, false>();
  constexpr int kGBytes = kGHalves ? halves_bytes<T, true, true>() : split_bytes<T, true, true>();
  __shared__ __align__(16) char lds[at_least(kWBytes, kGBytes)];
  if (blockIdx.x < n_w) {
    if constexpr (kWHalves) multiply_halves<T, false, false, kWDeep>(w, blockIdx.x, lds);
    else multiply_split<T, false, false>(w, blockIdx.x, lds);
  } else {
    if constexpr (kGHalves) multiply_halves<T, true, true, false>(g, blockIdx.x - n_w, lds);
    else multiply_split<T, true, true>(g, blockIdx.x - n_w, lds);
  }
}

inline long long tiles_of(long long n, int T) { return (n + T - 1) / T; }

// Tile edge.  The large tile reads and cuts each operand element half as often; the small one gives four times as many
// workgroups and less padding.  Measured, large / small tile:
//   thirds, 16384 x 3200 x 256: 172 / 242 us (g_pool), 159 / 313 us (dW); 5003 x 540 x 300, 200 and 240 large tiles: 24.1 / 26.5 us
//   and 24.0 / 26.6 us; 4096 x 416 x 256, 128 large tiles: 34.9 / 32.6 us for the two g_pool of a model step
//   fp32 (results do not depend on the choice), 16384 x 3200 x 256, 16 shards: 311 / 321 us; 5003 x 540 x 300 with 7 shards, where
//   the large tile multiplies 21 % more padding: 36 / 30 us
constexpr long long kFewLarge = 192;
template <bool kSplit>
inline int tile_edge(long long M, long long N, long long slices) {
  const long long large = tiles_of(M, 128) * tiles_of(N, 128) * slices, small = tiles_of(M, 64) * tiles_of(N, 64) * slices;
  if (kSplit) return large >= kFewLarge ? 128 : 64;
  return large >= 384 && large * 40 <= small * 11 ? 128 : 64;    // at most 10 % more area
}

// Runs of the forward product's two-level sums: as many products as eight 16-deep tiles hold that never span two fields, in whole
// k tiles, so 128 only where the fields fill such tiles.  (Runs of 128 for every D: error against 64 bits, 2-norm, at F x D =
// 300 x 4 / 200 x 8 / 100 x 20 / 50 x 36 2.1e-7 / 2.1e-7 / 2.2e-7 / 2.2e-7; so
// 1.5e-7 / 1.7e-7 / 1.8e-7 / 1.9e-7, in the same time.)
inline int forward_run(int D) {
  const int run = 8 * D / ((D + 15) / 16) / kPlainBK * kPlainBK;
  return run < kPlainBK ? kPlainBK : run;
}

// `depth`: products summed per output element of one slice; above kTwoLevelDepth the two-level kernel runs.
struct Product {
  GemmArgs g;
  int T;                              // tile edge
  long long blocks, depth;
  bool two;
};
template <bool kSplit>
des_status_t plan(GemmArgs g, int slices, long long depth, Product &p, int T = 0) {
  if (T == 0) T = tile_edge<kSplit>(g.M, g.N, slices);
  g.tiles_m = (int)tiles_of(g.M, T); g.tiles_n = (int)tiles_of(g.N, T); g.slices = slices;
  if (g.m_group <= 0 || g.m_group > g.tiles_m) g.m_group = g.tiles_m;
  const long long total = (long long)g.tiles_m * g.tiles_n * slices;
  if (total >= 2147483647ll) return DES_ERR_INVALID_ARG;
  g.die_run = g.in_turn ? (uint32_t)g.tiles_n : (uint32_t)((total + kXcds - 1) / kXcds);
  const long long round = (long long)kXcds * g.die_run;
  const long long blocks = (total + round - 1) / round * round;
  // A product whose operands and result fit the card has fewer than 2^23 large tiles; only the forward product, whose tiles
  // are small where it has few columns and whose shards come on top, may need further rows.
  if (kSplit && blocks > (long long)kGridRow) return DES_ERR_INVALID_ARG;
  // Results that the caches cannot keep until they are read are stored past them, so that they do not take the place of the operands: forward /
  // g_pool of 16384 x 3200 x 256 (268 and 210 MB) 272 / 147 -> 261 / 131 us, 131072 x 320 x 64 (537 and 168 MB) 137 / 54 -> 118 / 53.
  // Smaller ones are slower to read afterwards: a layer of 4096 x 416 x 256 (33 MB of partials) 52 -> 54 us in all.
  g.stream = (long long)g.M * g.N * slices * 4 > kStreamBytes;
  p = Product{g, T, blocks, depth, depth > kTwoLevelDepth};
  return DES_OK;
}

template <bool kSplit, bool kAKContig, bool kBKContig>
des_status_t launch(const Product &p, int kid, hipStream_t s) {
  const GemmArgs &g = p.g;
  const dim3 grid((unsigned)(p.blocks < (long long)kGridRow ? p.blocks : kGridRow), (unsigned)((p.blocks + kGridRow - 1) / kGridRow));
  const dim3 block(kBlock);
  ProfScope ps(kid, s);
  // k tiles of the fp32 product: 16 deep for large tiles of one level, so that four workgroups fit a CU (116 registers; 32 deep
  // 137 and three; 65536 x 416 x 256: 118 / 142 us), and shards whose depth is no multiple of 32 have no half tile of padding
  // (65536 x 26 x 16, 8 shards, 256 columns: 183 / 212 us).  Two-level sums do not fit more than two either way (16384 x 3200 x 256
  // with one shard: 301 / 250 us), and small tiles, of which there are few, wait for their barriers (4096 x 256 x 128: 10.0 / 8.7 us).
#define DES_GEMM(EDGE, TWO)                                                                                               \
  do {                                                                                                                    \
    constexpr int kBK = EDGE == 128 && !TWO ? 16 : kPlainBK;                                                              \
    if constexpr (kSplit) {                                                                                               \
      if (p.depth >= kHalvesDepth) hipLaunchKernelGGL((k_gemm_halves<EDGE, kAKContig, kBKContig, TWO>), grid, block, 0, s, g); \
      else if constexpr (!TWO) hipLaunchKernelGGL((k_gemm_split<EDGE, kAKContig, kBKContig>), grid, block, 0, s, g);        \
    }                                                                                                                     \
    else hipLaunchKernelGGL((k_gemm_f32<EDGE, kBK, kAKContig, kBKContig, TWO>), grid, block, 0, s, g);                     \
  } while (0)
  if (p.T == 128) { if (p.two) DES_GEMM(128, true); else DES_GEMM(128, false); }
  else            { if (p.two) DES_GEMM(64, true);  else DES_GEMM(64, false); }
#undef DES_GEMM
  return hipGetLastError() == hipSuccess ? DES_OK : DES_ERR_DEVICE;
}

// Both gradient products at once: they share operands, and neither fills the chip's last round by itself.  Their tiles have to be alike;
// where the rule above chose differently for each, it is asked for both together.  Both at once / one after the other, 5003 x 540 x 300
// 32 / 45 us, 109 x 816 x 300 15 / 19, 64 x 32 x 16 6.2 / 9.7, 4096 x 416 x 256 25 / 32, 2048 x 6400 x 256 80 / 85, 9000 x 540 x 300 54 / 55;
// dW of several stretches per slice, whose few workgroups run long: 16384 x 3200 x 256 245 / 273, 65536 x 416 x 256 221 / 265.  Not with a tile that
// doubles one's padding: 131072 x 320 x 64 with large tiles for dW too 438 / 354.
bool launch_both(Product &w, Product &g, hipStream_t s) {
  if (g.two) return false;
  const bool wh = w.depth >= kHalvesDepth, gh = g.depth >= kHalvesDepth;
  if (w.T != g.T) {
    if (!wh || !gh) return false;
    const auto tiles = [](const Product &p, int T) { return tiles_of(p.g.M, T) * tiles_of(p.g.N, T) * p.g.slices; };
    const int T = tiles(w, 128) + tiles(g, 128) >= kFewLarge ? 128 : 64;
    const Product &small = w.T < g.T ? w : g;
    if (T == 128 && tiles(small, 128) * 4 > tiles(small, 64) * 5 / 4) return false;      // a quarter of padding more
    if (plan<true>(w.g, w.g.slices, w.depth, w, T) != DES_OK || plan<true>(g.g, 1, g.depth, g, T) != DES_OK) return false;
  }
  if (((w.T == 128 || w.two) && !(wh && gh)) || w.blocks + g.blocks > (long long)kGridRow) return false;
  const dim3 grid((unsigned)(w.blocks + g.blocks)), block(kBlock);
  const uint32_t n_w = (uint32_t)w.blocks;
  ProfScope ps(KID_DNN_BOTH, s);
  if (w.two && w.T == 128) hipLaunchKernelGGL((k_gemm_both<128, true, true, true>), grid, block, 0, s, w.g, g.g, n_w);
  else if (w.two) hipLaunchKernelGGL((k_gemm_both<64, true, true, true>), grid, block, 0, s, w.g, g.g, n_w);
  else if (w.T == 128) hipLaunchKernelGGL((k_gemm_both<128, true, true>), grid, block, 0, s, w.g, g.g, n_w);
  else if (wh && gh) hipLaunchKernelGGL((k_gemm_both<64, true, true>), grid, block, 0, s, w.g, g.g, n_w);
  else if (wh) hipLaunchKernelGGL((k_gemm_both<64, true, false>), grid, block, 0, s, w.g, g.g, n_w);
  else if (gh) hipLaunchKernelGGL((k_gemm_both<64, false, true>), grid, block, 0, s, w.g, g.g, n_w);
  else hipLaunchKernelGGL((k_gemm_both<64, false, false>), grid, block, 0, s, w.g, g.g, n_w);
  return true;
}

bool al16(const void *p) { return ((uintptr_t)p & 15u) == 0; }

}  // namespace
}  // namespace des

using namespace des;

extern "C" {

des_status_t des_dnn_partial_forward(const float *pool, const float *W, int64_t B, int32_t F, int32_t D, int32_t H,
                                     int32_t K, float *Y_partial, void *stream) {
  if (B < 0 || F < 1 || D < 4 || (D & 3) || H < 4 || (H & 3) || K < 1 || K > 256) return DES_ERR_INVALID_ARG;
  if (B == 0) return DES_OK;
  if (!pool || !W || !Y_partial) return DES_ERR_INVALID_ARG;
  if (B >= 2147483647ll || (int64_t)F * D >= 2147483647ll || !al16(pool) || !al16(W) || !al16(Y_partial))
    return DES_ERR_INVALID_ARG;
  GemmArgs g;
  g.A = pool; g.a_xs = (uint32_t)F * D; g.a_ks = 1;
  g.B = W; g.b_xs = 1; g.b_ks = H;
  g.C = Y_partial; g.M = (int)B; g.N = H; g.c_rs = H; g.c_slice = (long long)B * H;
  // shard s: fields s, s+K, ... = k blocks of length D starting at s*D, K*D apart
  const long long depth = (long long)((F + K - 1) / K) * D;        // of the largest shard
  // Shallow shards, whose partials are most of the traffic, one shard after the other: with the shards of a group of rows done
  // together the card writes K distant places at a time.  16384 x 60 x 16, 64 shards, 128 columns: 125 / 118 us.  Where the pooled rows
  // are as large, their lines, which hold several shards' columns, are better read once: 131072 x 39 x 8, 8 shards, 64
  // columns 116 / 139 us; and deep shards use all of W anew with every shard: 131072 x 200 x 64, 64 shards 7.72 / 7.89 ms.
  const bool shallow = depth <= kShallowDepth && (long long)K * H >= 2ll * F * D;
  g.m_group = shallow ? 0 : kForwardGroup;
  g.in_turn = shallow;
  g.run = forward_run(D);
  g.k_shift = g.blk_len = D; g.blk_stride = (uint32_t)(K < F ? K : F) * D; g.k_limit = g.k_max = (uint32_t)F * D;
  Product p;
  const des_status_t st = plan<false>(g, K, depth, p);
  return st != DES_OK ? st : launch<false, true, false>(p, KID_DNN_FORWARD, (hipStream_t)stream);
}

des_status_t des_dnn_backward_bytes(int64_t B, int32_t F, int32_t D, int32_t H, size_t *workspace_bytes) {
  if (!workspace_bytes || B < 0 || F < 1 || D < 4 || H < 4) return DES_ERR_INVALID_ARG;
  *workspace_bytes = (size_t)16 * F * D * H * sizeof(float);    // up to 16 sample slices of dW
  return DES_OK;
}

des_status_t des_dnn_backward(const float *pool, const float *W, const float *dY, int64_t B, int32_t F, int32_t D,
                              int32_t H, float *g_pool, float *dW, void *workspace, size_t workspace_bytes,
                              void *stream) {
  if (B < 0 || F < 1 || D < 4 || (D & 3) || H < 4 || (H & 3)) return DES_ERR_INVALID_ARG;
  if (!g_pool && !dW) return DES_ERR_INVALID_ARG;
  if (B == 0) return DES_OK;            // g_pool is empty; dW would be all zero and is left untouched
  if (!pool || !W || !dY) return DES_ERR_INVALID_ARG;
  if (B >= 2147483647ll || (int64_t)F * D >= 2147483647ll || !al16(pool) || !al16(W) || !al16(dY) ||
      (g_pool && !al16(g_pool)) || (dW && !al16(dW)) || !al16(workspace))
    return DES_ERR_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  const long long FD = (long long)F * D;
  Product pg, pw;
  if (g_pool) {                                   // g_pool[B, F*D] = dY[B,H] x W^T: B(k=h, n=j) = W[j*H + h]
    GemmArgs g;
    g.A = dY; g.a_xs = H; g.a_ks = 1;
    g.B = W; g.b_xs = H; g.b_ks = 1;
    g.C = g_pool; g.M = (int)B; g.N = (int)FD; g.c_rs = FD; g.c_slice = 0;
    g.m_group = 0;
    g.run = kRun;
    g.k_shift = 0; g.blk_len = g.blk_stride = g.k_limit = g.k_max = H;
    const des_status_t st = plan<true>(g, 1, H, pg);
    if (st != DES_OK) return st;
    if (!dW) return launch<true, true, true>(pg, KID_DNN_GPOOL, s);
  }
  if (dW) {                                       // dW[F*D, H] = pool^T x dY, split over slices of samples
    const long long tiles = tiles_of(FD, 128) * tiles_of(H, 128);
    // Slices of samples: enough workgroups to fill the chip, chosen so that the last round of resident
    // workgroups (two per CU, 256 CUs) is as full as possible; fewer slices win ties
    // (less partial-sum traffic).  At most 16 slices, at least kMinSlice samples each.
    int Z = 1;
    {
      const long long per_round = 2 * 256;
      double best = -1.0;
      for (int z = 1; z <= 16 && (long long)z * kMinSlice <= (B > kMinSlice ? B : kMinSlice); ++z) {
        const long long blocks = tiles * z, rounds = (blocks + per_round - 1) / per_round;
        const double fill = (double)blocks / (double)(rounds * per_round);
        if (fill > best + 0.02) { best = fill; Z = z; }
      }
    }
    long long chunk = ((B + Z - 1) / Z + kMinSlice - 1) / kMinSlice * kMinSlice;
    Z = (int)((B + chunk - 1) / chunk);
    if (Z > 1 && (!workspace || workspace_bytes < (size_t)Z * FD * H * sizeof(float))) {
      if (g_pool) (void)launch<true, true, true>(pg, KID_DNN_GPOOL, s);      // which needs none
      return DES_ERR_WORKSPACE;
    }
    GemmArgs g;
    g.A = pool; g.a_xs = 1; g.a_ks = (uint32_t)FD;          // A(m=j, k=b) = pool[b*FD + j]
    g.B = dY; g.b_xs = 1; g.b_ks = H;
    g.C = Z > 1 ? (float *)workspace : dW; g.M = (int)FD; g.N = H; g.c_rs = H; g.c_slice = FD * H;
    g.m_group = 0;
    g.run = kRun;
    g.k_shift = g.k_max = (uint32_t)chunk; g.blk_len = g.blk_stride = 1u << 31; g.k_limit = (uint32_t)B;
    // one or two samples: a single rounding is closer than the split's truncated sums (2-norm error 2.5e-8 against 3.5e-8 and
    // 3.1e-8 against 3.3e-8; from three samples on the split is, 3.2e-8 against 3.6e-8)
    des_status_t st = B < 3 ? plan<false>(g, Z, chunk, pw) : plan<true>(g, Z, chunk, pw);
    if (st != DES_OK) return st;
    if (!g_pool || B < 3 || !launch_both(pw, pg, s)) {
      if (g_pool) st = launch<true, true, true>(pg, KID_DNN_GPOOL, s);
      if (st == DES_OK) st = B < 3 ? launch<false, false, false>(pw, KID_DNN_DW, s) : launch<true, false, false>(pw, KID_DNN_DW, s);
      if (st != DES_OK) return st;
    }
    if (Z > 1) return des_aggregate_partials((const float *)workspace, Z, FD * H, dW, stream);
  }
  return DES_OK;
}

}  // extern "C"
