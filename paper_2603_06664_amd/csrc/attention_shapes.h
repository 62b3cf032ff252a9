// The two shapes of a wave in the attention kernel.  Both hold S^T = K . Q^T with keys as MFMA rows and queries as
// columns, so that a lane's scores belong to one query (per tile of queries); the same registers, rounded to
// bf16, are the B operand (P^T) of O^T += V^T . P^T; the key order inside an MFMA step is whatever the
// accumulator layout gives, and the V^T fragment is fetched in that same order with the transposing LDS read
// (ds_read_b64_tr_b16) from the row-major V tile.
//
// Wide: 64 queries, four columns of 16, v_mfma_f32_16x16x32_bf16, tiles of 128 keys; every fragment feeds four
//   MFMAs.  A full chip is limited by power, and this MFMA draws less of it than the 32x32x16 one (half the
//   accumulator traffic per flop): MFMAs alone reach 2.02 PFLOP/s against 1.73 (the loops of ceilings.hip), the
//   480P last chunk 627 us against 690.
// Narrow: 32 queries, one column of 32, v_mfma_f32_32x32x16_bf16, tiles of 64 keys, for calls that do not fill
//   the chip: power is no limit there, what counts is the time of one work-group, and half as many MFMAs are
//   fewer instructions for the wave to issue (128 queries x 32760 keys: 384 us, 418 in two columns of 16).
//
// Software pipeline over 32-key blocks.  Sub-iteration b holds three independent instruction
// streams in ONE basic block:
//   MFMA:  O^T += V_{b-2}^T . P_{b-2}^T, then S_b = K_b . Q^T
//   VALU:  P_{b-1} = exp2(S_{b-1} - reference), rounded to bf16, and its sums
//   LDS:   the fragments of K_b under the PV half, those of V_{b-1} under the S half, each half a
//          sub-iteration ahead of its use
// The program order IS the schedule, pinned by a sched_barrier behind every MFMA: per 32 matrix clocks one
// exponential, half a conversion, one addition (where the sum of the unrounded probabilities is wanted) and the
// fragment reads.  Fragment reads come first behind their MFMA: behind the vector instructions of the same
// slot they cost 3 to 8 clocks more (one work-group of 256 queries: 544 against 525 us).
//
// Interface of a shape:
//   load(a, q0, head, lane)            query fragments and lane constants
//   place(lds0, lane)                  LDS offsets of the K and V fragments, in the first tile buffers
//   sub_iteration<...>(...)            see there
//   score(u, i), lower(u, x)           scores of the block of parity 0, i < kScores; subtract x from them
//   set_seed(u, x)                     start value of a FOLDED block's scores
//   clear(), fence()                   O's zeros, pinned; wait states behind the last of O's MFMAs
//   o_above(u, limit)                  whether an element of O is above the limit, or no number
//   quad(u, j), channel(j)             four channels of O, j < kQuads, and the first one's number
//   across_max(x), across_sum(x)       over the lanes that hold one query
//   denominator(u), range_sum(u)       sum of the rounded probabilities; a sum of them that no other query touches
#pragma once
#include "attention_tiles.h"

namespace crope {
namespace {

template <bool B>
struct BoolTag {
  static constexpr bool value = B;
};

// O's MFMAs are inline assembly so that O lives in accumulation registers; nothing reads or
// writes those inside the loop except the next of these MFMAs on the same tuple.
// The compiler inserts no wait states around an instruction that it cannot see, and an MFMA needs two
// between a vector instruction that writes an operand and itself.  The A operand arrives by an LDS
// read, which the compiler waits for; the B operand was written at least three MFMAs earlier; O's
// zeros are pinned where they are written, ahead of the loop.  The assembly that the compiler makes of
// this file is checked for these distances by the tests.
__device__ __forceinline__ void mfma_o(f32x16_t& o, bf16x8_t a, bf16x8_t b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(o) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_o(f32x4_t& o, bf16x8_t a, bf16x8_t b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(o) : "v"(a), "v"(b));
}
__device__ __forceinline__ bf16x8_t read_k(int off) {
  return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<__attribute__((address_space(3))) const uint4*>(
                                          (lds_byte*)(uintptr_t)(uint32_t)off));
}
template <int ROWS>   // rows between the two halves of the fragment
__device__ __forceinline__ bf16x8_t read_v(int off) {
  const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s16x4_t*)((lds_byte*)(uintptr_t)(uint32_t)off));
  const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s16x4_t*)((lds_byte*)(uintptr_t)(uint32_t)(off + ROWS * kRowBytes)));
  const uint2 a = __builtin_bit_cast(uint2, lo), b = __builtin_bit_cast(uint2, hi);
  return __builtin_bit_cast(bf16x8_t, make_uint4(a.x, a.y, b.x, b.y));
}

// Wait until at most N LDS reads of this wave are in flight (gfx9 encoding of the counter: bits 11:8).  Four of
// these per sub-iteration, each for four fragments, make the compiler's own sixteen unnecessary.
template <int N>
__device__ __forceinline__ void wait_lds() {
  __builtin_amdgcn_s_waitcnt(0xC07F | N << 8);
}

// The denominator of O is summed from the bf16 probabilities that O is made of: only then does their
// rounding cancel where few keys dominate (4680 keys, K gain 3: relative error 2.04e-3, 2.35e-3 over the
// unrounded sum; flat softmax 2.36e-3 both ways).  One sparse MFMA with an operand of ones takes a lane's 16
// probabilities, 16 clocks (dense MFMAs with ones 32, eight v_dot2_f32_bf16 18 each under MFMA load).
// Of every four elements A's row picks either 0, 1 or 2, 3.
__device__ __forceinline__ void add_probabilities(f32x4_t& sum, const uint32_t (&p)[8], bf16x8_t ones, int pick) {
  struct Words { uint32_t w[8]; };
  const bf16x16_t b = __builtin_bit_cast(bf16x16_t, Words{{p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7]}});
  sum = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(ones, b, sum, pick, 0, 0);
}

struct Narrow {
  static constexpr int kTileKeys = 64;
  static constexpr int kTiles = 1, kTileQ = 32, kWaveQ = 32;   // query tiles, queries in each, and per wave
  static constexpr int kScores = 16;      // a lane's scores of a block and query tile
  static constexpr int kSlots = 16;       // places for a copy in a sub-iteration
  static constexpr int kQuads = 16;       // groups of four channels a lane holds of a query
  static constexpr int kVMask = 3;        // swizzle of the V tile: see Loader
  static constexpr int kK = 8, kV = 4;    // fragment offsets
  static constexpr bool kNeedsSum = true; // the denominator may fall back to the unrounded sum

  f32x16_t o[4];        // [32-channel block], accumulation registers
  f32x16_t s[2];        // [block parity]
  uint32_t p[2][8];     // [block parity] bf16 probabilities
  f32x16_t seed;        // FOLDED: minus the reference in every element, the S accumulators' start value
  float m_ref[1], mc[1];
  float l_run[1];       // sum of the lane's fp32 probabilities
  f32x4_t l_bf16;
  bf16x8_t q[8], kf[8], vf[8];
  bf16x8_t ones;
  int pick;
  int k_off[kK], v_off[kV];
  int n, g;             // query column; which half of each 8-key group this lane holds

  // lane holds query n, channels 16*ks + 8g .. +7
  __device__ __forceinline__ void load(const AttnArgs& a, int q0, int head, int lane) {
    n = lane & 31;
    g = lane >> 5;
    const int qrow = min(q0 + n, a.n_q - 1);
    const uint16_t* qp = a.q + (int64_t)qrow * a.q_tok + (int64_t)head * a.q_head + 8 * g;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) q[ks] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(qp + 16 * ks));
    // Lane l of the sum's B operand holds column l%16, so the queries n and n+16 share a column: their lanes are
    // the even and the odd of the four k groups.  Of A the low half of a lane's words meets the even groups
    // and the high half the odd ones; bit 1 of the row says which of them is one, bit 0 which pair it picks.
    // Elements 0+1 of the result are then the sum of query l%16, elements 2+3 that of query l%16 + 16.
    const uint32_t even = lane & 2 ? 0u : 0x3f803f80u, odd = lane & 2 ? 0x3f803f80u : 0u;
    ones = __builtin_bit_cast(bf16x8_t, make_uint4(even, even, odd, odd));
    pick = lane & 1 ? (int)0xeeeeeeee : 0x44444444;
  }
  __device__ __forceinline__ void place(int lds0, int lane) {
    // K row n, logical chunk 2*ks + g
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) k_off[ks] = lds0 + n * kRowBytes + (((2 * ks + g) ^ (n & 15)) << 4);
    // V (transposing read): 16-lane group G = lane/16 covers channel half mh = G&1 of key half g;
    // lane i of the group points at row 4g + i/4 (+ step offset), channels 16*(db + 4*mh) + 4*(i%4)
    const int i16 = lane & 15, mh = (lane >> 4) & 1;
    const int kk = i16 >> 2, cc = i16 & 3;
#pragma unroll
    for (int db = 0; db < 4; ++db)
      v_off[db] = lds0 + 2 * kTileKeys * kRowBytes + (4 * g + kk) * kRowBytes + (((db ^ kk) + 4 * mh) << 5) + cc * 8;
  }
  __device__ __forceinline__ float score(int, int i) const { return s[0][i]; }
  __device__ __forceinline__ void lower(int, float x) {
#pragma unroll
    for (int i = 0; i < 16; ++i) s[0][i] -= x;
  }
  __device__ __forceinline__ void set_seed(int, float x) {
#pragma unroll
    for (int i = 0; i < 16; ++i) seed[i] = x;
  }
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[db][i] = 0.f;
    // written here, tile loads and S MFMAs ahead of mfma_o: without this the compiler copies the zeros
    // into place right in front of the first mfma_o that reads them, inside its wait states
#pragma unroll
    for (int db = 0; db < 4; ++db) asm volatile("" : "+a"(o[db]));
    l_bf16 = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
  __device__ __forceinline__ void fence() {
    asm volatile("s_nop 15\n\ts_nop 15" : "+a"(o[0]), "+a"(o[1]), "+a"(o[2]), "+a"(o[3]));
  }
  __device__ __forceinline__ bool o_above(int, float limit) const {
    bool r = false;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) r |= !(fabsf(o[db][i]) <= limit);
    return r;
  }
  __device__ __forceinline__ f32x4_t quad(int, int j) const {
    const int db = j >> 2, i4 = 4 * (j & 3);
    return f32x4_t{o[db][i4], o[db][i4 + 1], o[db][i4 + 2], o[db][i4 + 3]};
  }
  __device__ __forceinline__ int channel(int j) const { return 16 * (j >> 2) + 64 * ((j >> 1) & 1) + 8 * (j & 1) + 4 * g; }
  static __device__ __forceinline__ float across_max(float x) {
    const u32x2_t r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  static __device__ __forceinline__ float across_sum(float x) {
    const u32x2_t r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  // The sum contains the other query's probabilities times zero: where those are not finite it is NaN, and the
  // query falls back to the unrounded sum.
  __device__ __forceinline__ float denominator(int) const {
    const float l = n < 16 ? l_bf16[0] + l_bf16[1] : l_bf16[2] + l_bf16[3];
    return l < INFINITY ? l : across_sum(l_run[0]);
  }
  __device__ __forceinline__ float range_sum(int) const { return across_sum(l_run[0]); }

  // k_blk, v_blk: byte offsets of K_b and V_{b-1} from k_off / v_off, which move on by k_flip (exclusive or: the K
  // tiles start at a multiple of twice their size) and v_shift behind their last use; key0: index of K_b's first key; lim: the lane's queries see keys [0, lim).
  // FOLDED: the queries already carry scale*log2(e), so the MFMA result is the exponent itself once the
  // accumulators start from minus the reference; otherwise scores are raw and each costs one fma.
  template <int PAR, bool DO_PV, bool DO_S, bool DO_SM, bool READ_V, bool MASK, bool FOLDED, bool SUM, class FEED>
  __device__ __forceinline__ void sub_iteration(int k_blk, int v_blk, int key0, const int (&lim)[kTiles], float c,
                                                FEED& feed, int slot0, int k_flip, int v_shift) {
    static_assert(SUM);
    constexpr bool kFull = DO_PV && DO_S && READ_V;   // every fragment is requested half a sub-iteration ahead
    const f32x16_t& s_in = s[1 - PAR];
    f32x16_t& s_new = s[PAR];
    uint32_t(&p_new)[8] = p[1 - PAR];
    bf16x8_t pb[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
      pb[j] = __builtin_bit_cast(bf16x8_t, make_uint4(p[PAR][4 * j], p[PAR][4 * j + 1], p[PAR][4 * j + 2], p[PAR][4 * j + 3]));
    float l_a, l_b;   // this block's share of l_run
    float e[4];
    auto finish_pair = [&](int x) {   // the exponentials x and x+1 (x even) of the 16
      const float a = e[x & 2], b = e[(x & 2) + 1];
      p_new[x >> 1] = pack_bf16x2(a, b);
      l_a = x ? l_a + a : a;
      l_b = x ? l_b + b : b;
      asm volatile("" : "+v"(p_new[x >> 1]), "+v"(l_a), "+v"(l_b));
    };
    // slot x of the sub-iteration: exponential x, and the pair of which the last one is an odd slot old
    auto softmax_slot = [&](int x) {
      if (!DO_SM) return;
      float v = FOLDED ? __builtin_amdgcn_exp2f(s_in[x]) : __builtin_amdgcn_exp2f(fmaf(s_in[x], c, -mc[0]));
      asm volatile("" : "+v"(v));   // the empty asm statements keep each piece at its slot
      e[x & 3] = v;
      if ((x & 1) && x > 1) finish_pair(x - 3);
    };
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (kFull && i == 0) wait_lds<8>();   // V fragments 0..3
      if (kFull && i == 4) wait_lds<4>();   // V fragments 4..7
      if (DO_PV) mfma_o(o[i & 3], vf[i], pb[i >> 2]);
      if (DO_PV && i == 2) add_probabilities(l_bf16, p[PAR], ones, pick);
      __builtin_amdgcn_sched_barrier(0);
      if (DO_S) {
        kf[i] = read_k(k_off[i] + k_blk);
        k_off[i] ^= k_flip;
      }
      __builtin_amdgcn_sched_barrier(0);
      softmax_slot(i);
      feed.slot(slot0 + i);
      __builtin_amdgcn_sched_barrier(0);
    }
    f32x16_t start;   // keys past the limit are masked by starting their scores from -inf
    int left = lim[0] - key0 - 4 * g;
    if (MASK) asm volatile("" : "+v"(left));   // formed here: hoisted comparands would fill the register file
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float base = FOLDED ? seed[i] : 0.f;
      start[i] = MASK && 8 * (i >> 2) + (i & 3) >= left ? -INFINITY : base;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (kFull && i == 0) wait_lds<4>();   // K fragments 0..3
      if (kFull && i == 4) wait_lds<8>();   // K fragments 4..7
      if (DO_S) s_new = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i], q[i], i ? s_new : start, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (READ_V) vf[i] = read_v<8>(v_off[i & 3] + v_blk + (i >> 2) * 16 * kRowBytes);
      __builtin_amdgcn_sched_barrier(0);
      if (READ_V && i >= 4) v_off[i & 3] += v_shift;
      softmax_slot(8 + i);
      feed.slot(slot0 + 8 + i);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (DO_SM) {
      finish_pair(14);
      l_run[0] += l_a + l_b;
    }
  }
};

struct Wide {
  static constexpr int kTileKeys = 128;
  static constexpr int kTiles = 4, kTileQ = 16, kWaveQ = 64;
  static constexpr int kScores = 8;
  static constexpr int kSlots = 32;
  static constexpr int kQuads = 8;
  static constexpr int kVMask = 7;
  static constexpr int kK = 4, kV = 8;
  static constexpr bool kNeedsSum = false;

  f32x4_t o[kTiles][8];       // [query tile][16-channel block], accumulation registers
  f32x4_t s[2][kTiles][2];    // [block parity][query tile][16-key half]
  uint32_t p[kTiles][8];      // [query tile] bf16 probabilities of the two newest blocks, words 4*parity .. +3
  f32x4_t seed[kTiles];
  float m_ref[kTiles], mc[kTiles];
  float l_run[kTiles];        // SUM: sum of the lane's fp32 probabilities
  f32x4_t l_bf16[kTiles];     // elements 0+1: sum of the query's bf16 probabilities
  bf16x8_t q[kTiles][4];
  bf16x8_t kf[8], vf[8];      // K_b: [32 channels][16-key half]; V: [16 channels]
  int pick;
  int k_off[kK], v_off[kV];
  int n, g;                   // query column inside a tile; which quarter of each 16-key half this lane holds

  // lane holds query n of each tile, channels 32*ks + 8g .. +7
  __device__ __forceinline__ void load(const AttnArgs& a, int q0, int head, int lane) {
    n = lane & 15;
    g = lane >> 4;
#pragma unroll
    for (int u = 0; u < kTiles; ++u) {
      const int qrow = min(q0 + 16 * u + n, a.n_q - 1);
      const uint16_t* qp = a.q + (int64_t)qrow * a.q_tok + (int64_t)head * a.q_head + 8 * g;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) q[u][ks] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(qp + 32 * ks));
    }
    // A's even rows pick elements 0, 1 of every four and its odd rows 2, 3, all times one: elements 0+1 of the
    // result are the sum over the keys of two blocks for query l%16, in every lane.
    pick = lane & 1 ? (int)0xeeeeeeee : 0x44444444;
  }
  __device__ __forceinline__ void place(int lds0, int) {
    // K row n (+16 for the second half), logical chunk 4*ks + g
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) k_off[ks] = lds0 + n * kRowBytes + (((4 * ks + g) ^ n) << 4);
    // V (transposing read): lane i of the 16-lane group g points at row 4g + i/4 (+16 for the second half),
    // channels 16*cb + 4*(i%4), and gets channel 16*cb + i of rows 4g .. 4g+3
    const int row = 4 * g + (n >> 2), cc = n & 3;
#pragma unroll
    for (int cb = 0; cb < 8; ++cb)
      v_off[cb] = lds0 + 2 * kTileKeys * kRowBytes + row * kRowBytes + ((cb ^ (row & 7)) << 5) + cc * 8;
  }
  __device__ __forceinline__ float score(int u, int i) const { return s[0][u][i >> 2][i & 3]; }
  __device__ __forceinline__ void lower(int u, float x) {
#pragma unroll
    for (int i = 0; i < 8; ++i) s[0][u][i >> 2][i & 3] -= x;
  }
  __device__ __forceinline__ void set_seed(int u, float x) { seed[u] = f32x4_t{x, x, x, x}; }
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int u = 0; u < kTiles; ++u) {
#pragma unroll
      for (int cb = 0; cb < 8; ++cb) o[u][cb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int cb = 0; cb < 8; ++cb) asm volatile("" : "+a"(o[u][cb]));   // see Narrow
      l_bf16[u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
  }
  __device__ __forceinline__ void fence() {
#pragma unroll
    for (int u = 0; u < kTiles; ++u)
      asm volatile("s_nop 15\n\ts_nop 15"
                   : "+a"(o[u][0]), "+a"(o[u][1]), "+a"(o[u][2]), "+a"(o[u][3]), "+a"(o[u][4]), "+a"(o[u][5]),
                     "+a"(o[u][6]), "+a"(o[u][7]));
  }
  __device__ __forceinline__ bool o_above(int u, float limit) const {
    bool r = false;
#pragma unroll
    for (int cb = 0; cb < 8; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) r |= !(fabsf(o[u][cb][i]) <= limit);
    return r;
  }
  __device__ __forceinline__ f32x4_t quad(int u, int j) const { return o[u][j]; }
  __device__ __forceinline__ int channel(int j) const { return 16 * j + 4 * g; }
  static __device__ __forceinline__ float across_max(float x) {   // lanes l, l^16, l^32, l^48
    u32x2_t r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  static __device__ __forceinline__ float across_sum(float x) {
    u32x2_t r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  __device__ __forceinline__ float denominator(int u) const { return l_bf16[u][0] + l_bf16[u][1]; }
  __device__ __forceinline__ float range_sum(int u) const { return denominator(u); }

  // As Narrow's; two MFMAs of 16 clocks stand where Narrow has one of 32.  The query tiles run forth under one fragment and
  // back under the next, and the two key halves of a 32-channel step follow one another, so that an MFMA keeps one operand
  // of the one before (all but the first of each half and the three that begin the scores' next 32 channels): the same products
  // and sums for less power (the large cases 0.6 to 1.0 %: 480P last chunk 708 -> 702 us, rolling window 331 -> 328, 960p 10526 -> 10446).
  template <int PAR, bool DO_PV, bool DO_S, bool DO_SM, bool READ_V, bool MASK, bool FOLDED, bool SUM, class FEED>
  __device__ __forceinline__ void sub_iteration(int k_blk, int v_blk, int key0, const int (&lim)[kTiles], float c,
                                                FEED& feed, int slot0, int k_flip, int v_shift) {
    constexpr bool kFull = DO_PV && DO_S && READ_V;   // every fragment is requested half a sub-iteration ahead
    constexpr bool kSum = DO_PV && PAR == 1;          // p holds two whole blocks that are not summed yet
    f32x4_t(*const s_in)[2] = s[1 - PAR];
    f32x4_t(*const s_new)[2] = s[PAR];
    const uint32_t one = 0x3f803f80u;
    const bf16x8_t ones = __builtin_bit_cast(bf16x8_t, make_uint4(one, one, one, one));
    bf16x8_t pb[kTiles];
#pragma unroll
    for (int u = 0; u < kTiles; ++u) {
      const uint32_t* w = p[u] + 4 * PAR;
      pb[u] = __builtin_bit_cast(bf16x8_t, make_uint4(w[0], w[1], w[2], w[3]));
    }
    float l_a[kTiles], l_b[kTiles];   // this block's share of l_run
    float e[4];
    auto convert = [&](int x) {   // the exponentials x and x+1 (x even) of the 8*kTiles
      uint32_t& w = p[x >> 3][4 * (1 - PAR) + ((x & 7) >> 1)];
      w = pack_bf16x2(e[x & 2], e[(x & 2) + 1]);
      asm volatile("" : "+v"(w));
    };
    auto add = [&](int x) {
      float& l = (x & 1 ? l_b : l_a)[x >> 3];
      l = (x & 7) < 2 ? e[x & 3] : l + e[x & 3];
      if ((x & 7) >= 2) asm volatile("" : "+v"(l));
    };
    // behind MFMA m of the sub-iteration: every other one an exponential, every fourth a conversion of the pair of
    // which the last one is two exponentials old
    auto softmax_slot = [&](int m) {
      if (!DO_SM) return;
      const int x = m >> 1;
      if (!(m & 1)) {
        const float sc = s_in[x >> 3][(x >> 2) & 1][x & 3];
        float v = FOLDED ? __builtin_amdgcn_exp2f(sc) : __builtin_amdgcn_exp2f(fmaf(sc, c, -mc[x >> 3]));
        asm volatile("" : "+v"(v));   // the empty asm statements keep each piece at its slot
        e[x & 3] = v;
      } else {
        if (SUM && x >= 2) add(x - 2);
        if ((x & 1) && x > 1) convert(x - 3);
      }
    };
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int u = 0; u < kTiles; ++u) {
        if (kFull && u == 0 && i == 0) wait_lds<8>();   // V fragments 0..3
        if (kFull && u == 0 && i == 4) wait_lds<4>();   // V fragments 4..7
        const int v = i & 1 ? kTiles - 1 - u : u;
        if (DO_PV) mfma_o(o[v][i], vf[i], pb[v]);
        if (kSum && u == 3 && !(i & 3)) add_probabilities(l_bf16[i >> 2], p[i >> 2], ones, pick);
        __builtin_amdgcn_sched_barrier(0);
        if (DO_S && u == 1) {
          kf[i] = read_k(k_off[i >> 1] + k_blk + (i & 1) * 16 * kRowBytes);
          if (i & 1) k_off[i >> 1] ^= k_flip;
        }
        __builtin_amdgcn_sched_barrier(0);
        softmax_slot(kTiles * i + u);
        if (u & 1) feed.slot(slot0 + (kTiles * i + u) / 2);
        __builtin_amdgcn_sched_barrier(0);
      }
    f32x4_t start[kTiles][2];
#pragma unroll
    for (int u = 0; u < kTiles; ++u) {   // keys past the limit are masked by starting their scores from -inf
      int left = lim[u] - key0 - 4 * g;
      if (MASK) asm volatile("" : "+v"(left));   // formed here: hoisted comparands would fill the register file
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float base = FOLDED ? seed[u][i] : 0.f;
          start[u][h][i] = MASK && 16 * h + i >= left ? -INFINITY : base;
        }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int u = 0; u < kTiles; ++u) {
        const int ks = i >> 1, h = i & 1, v = h ? kTiles - 1 - u : u;
        if (kFull && u == 0 && i == 0) wait_lds<4>();   // K fragments 0..3
        if (kFull && u == 0 && i == 4) wait_lds<8>();   // K fragments 4..7
        if (DO_S) s_new[v][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[i], q[v][ks], ks ? s_new[v][h] : start[v][h], 0, 0, 0);
        if (kSum && u == 3 && !(i & 3)) add_probabilities(l_bf16[2 + (i >> 2)], p[2 + (i >> 2)], ones, pick);
        __builtin_amdgcn_sched_barrier(0);
        if (READ_V && u == 1) {
          vf[i] = read_v<16>(v_off[i] + v_blk);
          v_off[i] += v_shift;
        }
        __builtin_amdgcn_sched_barrier(0);
        softmax_slot(8 * kTiles + kTiles * i + u);
        if (u & 1) feed.slot(slot0 + 4 * kTiles + (kTiles * i + u) / 2);
        __builtin_amdgcn_sched_barrier(0);
      }
    if (DO_SM) {
      if (SUM) {
        add(8 * kTiles - 2);
        add(8 * kTiles - 1);
#pragma unroll
        for (int u = 0; u < kTiles; ++u) l_run[u] += l_a[u] + l_b[u];
      }
      convert(8 * kTiles - 2);
    }
  }
};

}  // namespace
}  // namespace crope
