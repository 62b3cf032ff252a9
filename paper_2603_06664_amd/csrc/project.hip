// Local QKV projection with qk-RMSNorm, causal 3D RoPE and the KV-cache update applied in
// the GEMM's epilogue (Algorithm 3 steps 1, 2, 3 and 5 in one pass; the operator fusion of
// Section 3.4.1 item 3), bf16 MFMA on gfx950.
//
// y[token][o] = sum_c x[token][c] * w[o][c] + bias[o];  o in [0, HD) is q, [HD, 2HD) k,
// [2HD, 3HD) v.  Both operands have the reduction index contiguous, so both are MFMA
// fragments as they lie in memory.  The product is formed transposed, C^T = W . x^T
// (channels = MFMA rows, tokens = columns): an accumulator lane then holds 4 consecutive
// channels of ONE token, i.e. two whole rotation pairs, and the epilogue needs no cross-lane
// traffic for the rotation.
//
// A work-group is 8 waves of 64 channels x up to 128 tokens (v_mfma_f32_16x16x32_bf16, two waves per SIMD) and owns two
// heads of q, k or v x 256 or 192 tokens, or one head; project_tiles.h says which
// width when, and how many of which.  What bounds the loop is the way from the L2 to LDS: with all CUs copying it carries 24 TB/s (39 bytes per
// clock and CU) in requests of 128 bytes and 13.5 TB/s in requests of 64, whatever the stride of the rows.  Hence two heads per
// work-group (32 to 37 bytes per clock at full MFMA rate; one head 48 to 53), and reduction steps of 64, whose LDS
// rows are one 128-byte request each (a version with steps of 32 and two work-groups per CU, 4680 tokens x 12 heads, row-wide norm:
// 105 us where this took 92).
// Then latency: W and x have rings of their own in LDS, as deep as 160 KB allow (see Shape, half_step).
// Row-wide norm (norm per head), us: 4680 tokens x 12 heads, c_in 1536, 91 -> 83 (72 -> 63), 585 x 40, 5120, 123 -> 98 (113 -> 90),
// 1320 x 16, 2048, 56 -> 46 (46 -> 35), 24 x 2, 256, 14.0 -> 7.9 (10.2 -> 5.2), against one head per work-group in 32x32x16 MFMAs with a
// three-stage ring for both operands and the epilogue's tables and tile through LDS.
// LDS rows are 128 B; 16-byte chunk c of row r sits at slot c ^ ((r >> 1) & 7), which makes the fragment reads (16 rows x
// 16 B per quarter wave) conflict-free.
//
// RMSNorm over one head is local to the tile and fully fused.  RMSNorm over the token's
// whole H*128 vector needs every head's sum of squares: the rotation commutes with the
// per-token scalar, so the epilogue stores z = rotate(gain * y) and the per-head sums of
// squares, and a second, bandwidth-bound pass multiplies q and k rows by 1/rms.  z is kept
// as TWO bf16 numbers, hi = bf16(z) in the destination row and lo = bf16(z - hi) in the
// workspace (16 mantissa bits together), so that the second pass rounds (hi + lo) / rms to
// bf16 once: the stored result is the single rounding of the fp32 value up to 2^-17 relative.
#include "crope_internal.h"
#include "project_tiles.h"

namespace crope {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) uint8_t lds_byte;

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  f32x2_t f = {lo, hi};
  bf16x2_t h = __builtin_convertvector(f, bf16x2_t);
  return __builtin_bit_cast(uint32_t, h);
}
__device__ __forceinline__ float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }
// sum over the lanes l, l^16, l^32, l^48
__device__ __forceinline__ float sum_across_rows(float x) {
  u32x2_t r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

constexpr int kTileCh = 128;    // one head
constexpr int kStepK = 64;      // reduction elements per LDS stage
constexpr int kRowB = kStepK * 2;             // 128 B per LDS row
constexpr int kWaves = 8, kThreads = 64 * kWaves;

// A tile of 64*WC channels (one head or two) x 16*TT*(8/WC) tokens: 8 waves of 64 channels x 16*TT tokens.
template <int WC_, int TT_>
struct Shape {
  static constexpr int WC = WC_, TT = TT_, WT = kWaves / WC;
  static constexpr int kCh = 64 * WC, kWaveTok = 16 * TT, kTileTok = WT * kWaveTok;
  static constexpr int kStageA = kCh * kRowB, kStageB = kTileTok * kRowB;
  // places for W and, behind them, for x: as many as 160 KB hold; one head's tiles run alone on a CU or nearly so, where
  // latency is all that counts
  static constexpr int kAStages = WC == 4 ? 3 : 4, kBStages = WC == 4 ? 2 : kTileTok > 192 ? 3 : 4;
  static constexpr int kLds = kAStages * kStageA + kBStages * kStageB;
  static constexpr int kACopies = kCh / 64, kBCopies = kTileTok / 64;   // per wave and stage
  static constexpr int kMfmas = 4 * TT, kReads = 4 + TT;       // per wave and half step
  static_assert(kTileTok % 64 == 0, "copies are whole kilobytes of every wave");
  // W of step kt+kAStages-1 is requested in the first half of step kt, x of step kt+kBStages in the second.  Copies that may
  // be in flight in the middle of step kt, when those of step kt+1 have to have landed: what was requested, in halves of
  // steps, after the later one of W and x of step kt+1
  static constexpr int in_flight() {
    const int a1 = 2 * (2 - kAStages), b1 = 2 * (1 - kBStages) + 1, t = a1 > b1 ? a1 : b1;
    int n = 0;
    for (int h = t + 1; h <= 0; ++h) n += h % 2 == 0 ? kACopies : kBCopies;
    return n;
  }
};

template <class S>
struct TileLoader {   // scalars only
  u32x4_t a_buf;           // W from the tile's first channel row on
  u32x4_t b_buf;           // x from the tile's first token row on
  // per-lane byte offsets of the lane's chunk for load instruction t: row 8*wave + lane/8 + 64*t
  uint32_t a_off[S::kACopies];
  uint32_t b_off[S::kBCopies];
};

// Copy instruction t of wave w covers tile rows 8*(w + 8*t) .. +7 (1 KB of LDS): lane i carries
// the chunk that belongs at (row 8*(w + 8*t) + i/8, slot i%8).  ((row >> 1) & 7) = (i>>4) | 4*(w&1)
// does not depend on t.  Token rows past the end re-read the last token (clamped when the
// offsets are formed); their results are never stored.
// The copy is inline assembly, not the compiler's builtin: while a builtin copy is in flight
// the compiler turns every counted wait on an LDS read into a wait for all of them.  LDS
// address of lane i's 16 bytes: M0 + 16*i; M0 is an input operand bound to that register, the
// s_nop covers the wait state after its write.  Base and step are scalar (a buffer and its scalar offset), so that a
// copy costs no vector instruction and two scalar ones.  A vector instruction that wrote one of the
// buffer's words would need five wait states that the compiler does not insert here: the words are formed ahead
// of the loop, and the tests check the assembly.
__device__ __forceinline__ void copy16(u32x4_t buf, uint32_t lane_off, uint32_t k_off /* wave-uniform */,
                                       uint32_t lds_dst /* wave-uniform */) {
  const uint32_t m0 = __builtin_amdgcn_readfirstlane(lds_dst);
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
               :: "v"(lane_off), "s"(buf), "s"(k_off), "{m0}"(m0) : "memory");
}
// 2^32 - 1 bytes from `base` on: offsets stay below (255 rows of at most 2^23 bytes, and 2^21 bytes of reduction)
__device__ __forceinline__ u32x4_t raw_buffer(const uint8_t* base /* wave-uniform */) {
  const uint64_t a = (uint64_t)base;
  return u32x4_t{(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a),
                 (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32)), 0xffffffffu, 0x00020000u};
}

// copy i of the W tile, of the x tile, of reduction step kt; dst: the place + 1024 * wave
template <class S>
__device__ __forceinline__ void copy_a(const TileLoader<S>& L, int kt, uint32_t dst, int i) {
  copy16(L.a_buf, L.a_off[i], (uint32_t)kt * kRowB, dst + i * (kWaves * 1024));
}
template <class S>
__device__ __forceinline__ void copy_b(const TileLoader<S>& L, int kt, uint32_t dst, int i) {
  copy16(L.b_buf, L.b_off[i], (uint32_t)kt * kRowB, dst + i * (kWaves * 1024));
}

template <int TT>
struct Frags {
  bf16x8_t a[4], b[TT];
};

__device__ __forceinline__ bf16x8_t read16(int off) {
  return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<__attribute__((address_space(3))) const u32x4_t*>(
                                          (lds_byte*)(uintptr_t)(uint32_t)off));
}
// fragment i of a half step, in the order in which the MFMAs want them; a_at, b_at: the lane's place in the stage
template <int TT>
__device__ __forceinline__ void read_frag(Frags<TT>& f, int a_at, int b_at, int i) {
  if (i < 4) f.a[i] = read16(a_at + i * 16 * kRowB);
  else f.b[i - 4] = read16(b_at + (i - 4) * 16 * kRowB);
}

// Wait until at most VM copies of this wave are in flight and every LDS read has returned, then a
// barrier WITHOUT the memory fence of __syncthreads(): the fence would wait for every copy in
// flight, also the ones into stages that are not needed yet.  The wait is the s_waitcnt builtin
// (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8), which the compiler's
// own wait-count bookkeeping understands.
template <int VM>
__device__ __forceinline__ void wait_and_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((VM & 15) | ((VM >> 4) << 14) | (7 << 4));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// number of n things that stand in front of slot s, when they are spread over `percent` of the slots
constexpr int placed(int s, int n, int slots, int percent) {
  const int c = s * n * 100 / (slots * percent);
  return s >= slots || c > n ? n : c;
}

// Half of a reduction step: 4*TT MFMAs on the fragments f, behind which, one by one, stand the reads of the next half's.
// The second half starts with the step's barrier (behind eight MFMAs, four with one head): nobody reads stage kt any more, and
// stage kt+1 has landed.  Behind it stand the copies of x, in the first half those of W, in the first 60 % (x of two heads 45 %)
// of the slots: with two heads x has about one step to land, and one that is requested later, or waited for
// earlier, holds everybody up (585 rows x 40 heads, norm per head: W two steps ahead in the second half, too, 107 us; W three and x two 96; W
// moved to the first half and x requested early 94; barrier behind 0, 4, 8, 12 MFMAs 104, 94, 92, 93).
template <class S, bool SECOND, bool STEADY>   // STEADY: 0 < kt and the copies of this step are known to exist
__device__ __forceinline__ void half_step(f32x4_t (&acc)[4][S::TT], Frags<S::TT>& f, Frags<S::TT>& f_next, const TileLoader<S>& L,
                                          int kt, int n_kt, int a_at, int b_at, uint32_t ld) {
  constexpr int kFirst = !SECOND ? 0 : S::WC == 4 && S::kMfmas > 8 ? 8 : S::kMfmas > 4 ? 4 : 0;
  constexpr int kSlots = S::kMfmas - kFirst, kPercent = SECOND && S::WC == 4 ? 45 : 60;
  constexpr int kCopies = SECOND ? S::kBCopies : S::kACopies;
  constexpr int kAhead = SECOND ? S::kBStages : S::kAStages - 1;
  constexpr int kMost = S::kAStages > S::kBStages ? S::kAStages : S::kBStages;
  const bool more = !SECOND || STEADY || kt + 1 < n_kt;
  const bool copies = STEADY || (kt + kAhead < n_kt && (SECOND || kt > 0));   // kt = 0: W's places are full
#pragma unroll
  for (int m = 0; m < S::kMfmas; ++m) {
    if (SECOND && m == kFirst) {
      if (STEADY || kt + kMost - 1 < n_kt) wait_and_barrier<S::in_flight()>();
      else wait_and_barrier<0>();
      __builtin_amdgcn_sched_barrier(0);
    }
    acc[m & 3][m >> 2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a[m & 3], f.b[m >> 2], acc[m & 3][m >> 2], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    if (m >= kFirst) {
      const int s = m - kFirst;
      if (more) {
#pragma unroll
        for (int i = placed(s, S::kReads, kSlots, 100); i < placed(s + 1, S::kReads, kSlots, 100); ++i)
          read_frag<S::TT>(f_next, a_at, b_at, i);
      }
      if (copies) {
#pragma unroll
        for (int i = placed(s, kCopies, kSlots, kPercent); i < placed(s + 1, kCopies, kSlots, kPercent); ++i) {
          if (SECOND) copy_b<S>(L, kt + kAhead, ld, i);
          else copy_a<S>(L, kt + kAhead, ld, i);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

template <bool B>
struct BoolTag {
  static constexpr bool value = B;
};

// 16 channels of one token and two neighbouring 16-channel blocks c0, c1, as lane g of four holds them (channels
// 4g .. 4g+3 of each): exchanged so that every lane has 8 neighbouring channels, 16*(c0 + g%2) + 8*(g/2) ..
__device__ __forceinline__ uint4 join_quads(const uint32_t (&c0)[2], const uint32_t (&c1)[2]) {
  const u32x2_t lo = __builtin_amdgcn_permlane16_swap(c0[0], c1[0], false, false);
  const u32x2_t hi = __builtin_amdgcn_permlane16_swap(c0[1], c1[1], false, false);
  return make_uint4(lo[0], hi[0], lo[1], hi[1]);
}

template <class S, bool PER_HEAD>
__device__ __forceinline__ void project_tile(const ProjArgs& a, int ch_tile0, int tok0, uint8_t* lds) {
  constexpr int TT = S::TT, kTileTok = S::kTileTok, kWaveTok = S::kWaveTok;
  const int lds0 = (int)(uint32_t)(uintptr_t)(lds_byte*)lds;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, g = lane >> 4;
  const int wq = wave % S::WC, wt = wave / S::WC;   // 64 channels of the tile, token part
  const int wc = wq & 1, ch_tile = ch_tile0 + (wq >> 1);   // half of a head, which head

  TileLoader<S> L;
  {
    const int row = 8 * wave + (lane >> 3);
    const uint32_t chunk_bytes = (uint32_t)(((lane & 7) ^ ((lane >> 4) | ((wave & 1) << 2))) * 16);
    const int64_t a_row_bytes = (int64_t)a.c_in * 2, b_row_bytes = a.x_tok * 2;
    L.a_buf = raw_buffer(reinterpret_cast<const uint8_t*>(a.w) + (int64_t)ch_tile0 * kTileCh * a_row_bytes);
    L.b_buf = raw_buffer(reinterpret_cast<const uint8_t*>(a.x) + (int64_t)tok0 * b_row_bytes);
    const int last = a.n_tokens - 1 - tok0;   // >= 0
#pragma unroll
    for (int t = 0; t < S::kACopies; ++t) L.a_off[t] = (uint32_t)((row + 64 * t) * a_row_bytes) + chunk_bytes;
#pragma unroll
    for (int t = 0; t < S::kBCopies; ++t)
      L.b_off[t] = (uint32_t)(min(row + 64 * t, last) * b_row_bytes) + chunk_bytes;
  }
  // fragment read offsets: row (64*wq or 16*TT*wt, + n), 16-byte chunk 4*half + g -> slot (4*half + g) ^ ((n>>1)&7)
  const int slot = (g ^ (n >> 1)) << 4;
  const int a_lane = lds0 + (64 * wq + n) * kRowB + slot;
  const int b_lane = lds0 + S::kAStages * S::kStageA + (kWaveTok * wt + n) * kRowB + slot;
  const uint32_t dst_a = (uint32_t)(lds0 + wave * 1024), dst_b = dst_a + S::kAStages * S::kStageA;

  f32x4_t acc[4][TT];
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int t = 0; t < TT; ++t) acc[c][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int n_kt = a.c_in / kStepK;
  Frags<TT> f0, f1;
  constexpr int kMost = S::kAStages > S::kBStages ? S::kAStages : S::kBStages;
#pragma unroll
  for (int j = 0; j < kMost; ++j) {
    if (j < S::kAStages && j < n_kt) {
#pragma unroll
      for (int i = 0; i < S::kACopies; ++i) copy_a<S>(L, j, dst_a + j * S::kStageA, i);
    }
    if (j < S::kBStages && j < n_kt) {
#pragma unroll
      for (int i = 0; i < S::kBCopies; ++i) copy_b<S>(L, j, dst_b + j * S::kStageB, i);
    }
  }
  if (n_kt >= kMost) wait_and_barrier<(S::kAStages - 1) * S::kACopies + (S::kBStages - 1) * S::kBCopies>();
  else wait_and_barrier<0>();
#pragma unroll
  for (int i = 0; i < S::kReads; ++i) read_frag<TT>(f0, a_lane, b_lane, i);
  // lgkmcnt(0): enter the loop with nothing pending, so that the loop's own waits are counted
  // ones (a pending scalar load would make the compiler wait for every LDS read instead)
  __builtin_amdgcn_s_waitcnt(0xC07F);
  // stage kt's places; the lane's fragments stand there at a_lane, b_lane, those of the second half at an exclusive or of 64
  int kt = 0, sa = 0, sb = 0;
  auto one_step = [&](auto steady) {
    constexpr bool kSteady = decltype(steady)::value;
    const int sa_free = sa == 0 ? (S::kAStages - 1) * S::kStageA : sa - S::kStageA;
    const int sa1 = sa == (S::kAStages - 1) * S::kStageA ? 0 : sa + S::kStageA;
    const int sb1 = sb == (S::kBStages - 1) * S::kStageB ? 0 : sb + S::kStageB;
    half_step<S, false, kSteady>(acc, f0, f1, L, kt, n_kt, (a_lane + sa) ^ 64, (b_lane + sb) ^ 64, dst_a + sa_free);
    half_step<S, true, kSteady>(acc, f1, f0, L, kt, n_kt, a_lane + sa1, b_lane + sb1, dst_b + sb);
    sa = sa1;
    sb = sb1;
    ++kt;
  };
  constexpr int kFarthest = S::kAStages - 1 > S::kBStages ? S::kAStages - 1 : S::kBStages;
  one_step(BoolTag<false>{});
  while (kt + kFarthest < n_kt) one_step(BoolTag<true>{});
  while (kt < n_kt) one_step(BoolTag<false>{});   // the last steps

  // ------------------------------------------------------------------ epilogue
  // acc[c][t][i]: token tok0 + kWaveTok*wt + 16*t + n, channel 64*wc + 16*c + 4*g + i of the head: two rotation pairs of
  // one token.  The last step's barrier has passed: nobody reads or fills the stages any more.  (cos, sin) come straight
  // from the tables, 16 bytes a lane: the four lanes of a token read 64 neighbouring bytes.  Outputs leave
  // from registers, 16 bytes a lane.  All that crosses waves is the sum of squares of the other 64 channels.
  float* const ss_lds = reinterpret_cast<float*>(lds);   // [wq][token of the tile]
  const int which = ch_tile / a.n_heads;   // 0: q, 1: k, 2: v
  const int head = ch_tile - which * a.n_heads;
  const int tok_lane = tok0 + kWaveTok * wt + n;
  if (a.bias) {
    const float* bp = a.bias + (int64_t)ch_tile * kTileCh + 64 * wc + 4 * g;
    f32x4_t bv[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) bv[c] = *reinterpret_cast<const f32x4_t*>(bp + 16 * c);
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int t = 0; t < TT; ++t) acc[c][t] += bv[c];
  }
  uint16_t* base;
  int64_t tstride;
  if (which == 0) { base = a.q_out + (int64_t)head * a.qo_head; tstride = a.qo_tok; }
  else {
    base = (which == 1 ? a.k_cache : a.v_cache) + a.dst_token * a.c_tok + (int64_t)head * a.c_head;
    tstride = a.c_tok;
  }
  const int ch_store = 64 * wc + 16 * (g & 1) + 8 * (g >> 1);   // + 32 for the second two 16-channel blocks
  auto store_token = [&](uint16_t* row, const uint32_t (&w)[4][2]) {
#pragma unroll
    for (int c = 0; c < 4; c += 2) *reinterpret_cast<uint4*>(row + ch_store + 16 * c) = join_quads(w[c], w[c + 1]);
  };

  // v: one rounding.  No LDS, so no barrier: all waves of the work-group are here, since v starts at channel tile 2*n_heads, an even
  // one, and pairs of heads start at even ones, so that none holds k and v.
  if (which == 2) {
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      const int token = tok_lane + 16 * t;
      uint32_t w[4][2];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        w[c][0] = pack_bf16x2(acc[c][t][0], acc[c][t][1]);
        w[c][1] = pack_bf16x2(acc[c][t][2], acc[c][t][3]);
      }
      // (store_token's exchange between lanes stands inside the condition: the four lanes that exchange have the same token)
      if (token < a.n_tokens) store_token(base + (int64_t)token * tstride, w);
    }
    return;
  }

  const float* gp = (which == 0 ? a.gain_q : a.gain_k) + head * kHeadDim + 64 * wc + 4 * g;
  f32x4_t gv[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) gv[c] = *reinterpret_cast<const f32x4_t*>(gp + 16 * c);

  // The lane's pairs: 32*wc + 8*c + 2*g and the next one.  Table entry of pair j on each axis, as if j ran through that
  // axis' row.  Where the two lie on different axes the second is fetched by itself.
  const int p_t = a.tl.pairs_t, p_th = a.tl.pairs_t + a.tl.pairs_h;
  const float2* tab2 = reinterpret_cast<const float2*>(a.table);
  constexpr int kBatch = TT % 2 ? TT : TT / 2;
  f32x4_t cs[kBatch][4];
  auto fetch = [&](int t0) {
    int bt[kBatch], bh[kBatch], bw[kBatch];
#pragma unroll
    for (int t = 0; t < kBatch; ++t) {   // tokens past the end: the last token's position
      const uint32_t ig = (uint32_t)(a.token_offset + min(tok_lane + 16 * (t0 + t), a.n_tokens - 1));
      const uint32_t f = fastdiv(ig, a.div_hw);
      const uint32_t r = ig - f * a.div_hw.d;
      const uint32_t ph = fastdiv(r, a.div_w);
      const uint32_t pw = r - ph * a.div_w.d;
      bt[t] = (int)(a.tl.off_t / 2) + (a.start_frame + (int)f) * a.tl.pairs_t;
      bh[t] = (int)(a.tl.off_h / 2) + (int)ph * a.tl.pairs_h - p_t;
      bw[t] = (int)(a.tl.off_w / 2) + (int)pw * a.tl.pairs_w - p_th;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int j = 32 * wc + 8 * c + 2 * g;
      const bool on_t = j < p_t, on_h = j < p_th;
#pragma unroll
      for (int t = 0; t < kBatch; ++t)
        __builtin_memcpy(&cs[t][c], tab2 + (uint32_t)(j + (on_t ? bt[t] : on_h ? bh[t] : bw[t])), 16);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int j = 32 * wc + 8 * c + 2 * g + 1;
      const bool apart = j == p_t || j == p_th;
      if (__builtin_amdgcn_ballot_w64(apart) != 0) {
        const bool on_t = j < p_t, on_h = j < p_th;
#pragma unroll
        for (int t = 0; t < kBatch; ++t) {
          const float2 e = tab2[(uint32_t)(j + (on_t ? bt[t] : on_h ? bh[t] : bw[t]))];
          if (apart) { cs[t][c][2] = e.x; cs[t][c][3] = e.y; }
        }
      }
    }
  };
  fetch(0);

  // ---- sums of squares over the head: lane-local, the other lanes of the token, the other wave
  float tot[TT];
  {
    float ss[TT];
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      float sq = 0.f;
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) sq = fmaf(acc[c][t][i], acc[c][t][i], sq);
      ss[t] = sum_across_rows(sq);
    }
    if (g == 0) {
#pragma unroll
      for (int t = 0; t < TT; ++t) ss_lds[wq * kTileTok + kWaveTok * wt + 16 * t + n] = ss[t];
    }
    wait_and_barrier<63>();   // the table rows stay in flight
#pragma unroll
    for (int t = 0; t < TT; ++t)
      tot[t] = ss_lds[(wq - wc) * kTileTok + kWaveTok * wt + 16 * t + n] + ss_lds[(wq - wc + 1) * kTileTok + kWaveTok * wt + 16 * t + n];
  }
  float r[TT];
#pragma unroll
  for (int t = 0; t < TT; ++t) r[t] = PER_HEAD ? 1.0f / sqrtf(tot[t] * (1.0f / kHeadDim) + a.eps) : 1.0f;
  if (!PER_HEAD && wc == 0 && g == 0) {
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      const int token = tok_lane + 16 * t;
      if (token < a.n_tokens) a.sumsq[((int64_t)which * a.n_tokens + token) * a.n_heads + head] = tot[t];
    }
  }
  // ---- normalise, gain, rotate, store
#pragma unroll
  for (int t0 = 0; t0 < TT; t0 += kBatch) {
    if (t0) fetch(t0);
#pragma unroll
    for (int tb = 0; tb < kBatch; ++tb) {
      const int t = t0 + tb, token = tok_lane + 16 * t;
      uint32_t w[4][2], w_lo[4][2];   // w_lo: row-wide norm: bf16 of what the first rounding dropped
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const f32x4_t e = cs[tb][c];
        const float xa0 = acc[c][t][0] * r[t] * gv[c][0], xb0 = acc[c][t][1] * r[t] * gv[c][1];
        const float xa1 = acc[c][t][2] * r[t] * gv[c][2], xb1 = acc[c][t][3] * r[t] * gv[c][3];
        const float z0 = xa0 * e[0] - xb0 * e[1], z1 = xa0 * e[1] + xb0 * e[0];
        const float z2 = xa1 * e[2] - xb1 * e[3], z3 = xa1 * e[3] + xb1 * e[2];
        w[c][0] = pack_bf16x2(z0, z1);
        w[c][1] = pack_bf16x2(z2, z3);
        if (!PER_HEAD) {
          w_lo[c][0] = pack_bf16x2(z0 - bf16_lo(w[c][0]), z1 - bf16_hi(w[c][0]));
          w_lo[c][1] = pack_bf16x2(z2 - bf16_lo(w[c][1]), z3 - bf16_hi(w[c][1]));
        }
      }
      if (token < a.n_tokens) {
        store_token(base + (int64_t)token * tstride, w);
        if (!PER_HEAD)   // workspace rows [which][token][head][128]
          store_token(a.resid + (((int64_t)which * a.n_tokens + token) * a.n_heads + head) * kHeadDim, w_lo);
      }
    }
  }
}

template <int WC, int TOK, bool PER_HEAD>
__device__ __forceinline__ void project_ragged(const ProjArgs& a, int ch_tile, int tok0, uint8_t* lds) {
  constexpr int U = 16 * (kWaves / WC);   // the last tile of the tokens takes the narrowest body that holds them
  const int left = a.n_tokens - tok0;
  if (left <= 64) project_tile<Shape<WC, 64 / U>, PER_HEAD>(a, ch_tile, tok0, lds);
  else if (left <= 128) project_tile<Shape<WC, 128 / U>, PER_HEAD>(a, ch_tile, tok0, lds);
  else if (TOK > 192 && left <= 192) project_tile<Shape<WC, 192 / U>, PER_HEAD>(a, ch_tile, tok0, lds);
  else project_tile<Shape<WC, TOK / U>, PER_HEAD>(a, ch_tile, tok0, lds);
}

template <int TOK, bool PER_HEAD>
__global__ __attribute__((amdgpu_flat_work_group_size(kThreads, kThreads), amdgpu_waves_per_eu(2, 2)))
void qkv_project_kernel(ProjArgs a, ProjTiles pt) {
  __shared__ __attribute__((aligned(1024))) uint8_t lds[160 * 1024];
  const ProjWork w = project_work(pt, blockIdx.x);
  if (w.heads == 0) return;   // the whole work-group leaves together
  static_assert(Shape<4, TOK / 32>::kLds <= (int)sizeof(lds) && Shape<2, TOK / 64>::kLds <= (int)sizeof(lds), "LDS");
  // (without readfirstlane the compiler works the tile out again in every body)
  const int ch_tile = __builtin_amdgcn_readfirstlane(w.ch_tile), tok0 = __builtin_amdgcn_readfirstlane(w.tok_tile * TOK);
  if (w.heads == 2) project_ragged<4, TOK, PER_HEAD>(a, ch_tile, tok0, lds);
  else project_ragged<2, TOK, PER_HEAD>(a, ch_tile, tok0, lds);
}

// Second pass of the row-wide norm: one wave per (tensor, token) sums the per-head sums of
// squares in a fixed order, and replaces the stored high part of rotate(gain * y) by the bf16
// rounding of (high + low) / rms.
constexpr int kScaleWaves = 4;
__global__ __launch_bounds__(64 * kScaleWaves) void scale_rows_kernel(ProjArgs a) {
  const int lane = threadIdx.x & 63;
  const int tok = blockIdx.y * kScaleWaves + (threadIdx.x >> 6);
  if (tok >= a.n_tokens) return;
  const int which = blockIdx.x;   // 0: q, 1: k
  float s = lane < a.n_heads ? a.sumsq[((int64_t)which * a.n_tokens + tok) * a.n_heads + lane] : 0.f;
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m, 64);
  const float r = 1.0f / sqrtf(s * (1.0f / (float)(a.n_heads * kHeadDim)) + a.eps);
  uint16_t* row = which == 0 ? a.q_out + (int64_t)tok * a.qo_tok : a.k_cache + (a.dst_token + tok) * a.c_tok;
  const int64_t hstride = which == 0 ? a.qo_head : a.c_head;
  const uint16_t* lo_row = a.resid + ((int64_t)which * a.n_tokens + tok) * a.n_heads * kHeadDim;
  const int n_chunks = a.n_heads * 16;
  for (int c = lane; c < n_chunks; c += 64) {
    uint4* p = reinterpret_cast<uint4*>(row + (int64_t)(c >> 4) * hstride + (c & 15) * 8);
    uint4 u = *p;
    const uint4 w = *reinterpret_cast<const uint4*>(lo_row + (int64_t)c * 8);
    u.x = pack_bf16x2((bf16_lo(u.x) + bf16_lo(w.x)) * r, (bf16_hi(u.x) + bf16_hi(w.x)) * r);
    u.y = pack_bf16x2((bf16_lo(u.y) + bf16_lo(w.y)) * r, (bf16_hi(u.y) + bf16_hi(w.y)) * r);
    u.z = pack_bf16x2((bf16_lo(u.z) + bf16_lo(w.z)) * r, (bf16_hi(u.z) + bf16_hi(w.z)) * r);
    u.w = pack_bf16x2((bf16_lo(u.w) + bf16_lo(w.w)) * r, (bf16_hi(u.w) + bf16_hi(w.w)) * r);
    *p = u;
  }
}

}  // namespace

// fp32 sums of squares [2][tokens][heads], rounded up to 256 bytes, then the bf16 low parts
// [2][tokens][heads][128]
static size_t sumsq_bytes(int n_tokens, int n_heads) {
  return (((size_t)2 * n_tokens * n_heads * sizeof(float)) + 255) & ~(size_t)255;
}
size_t project_workspace_bytes(int n_tokens, int n_heads, bool per_head_norm) {
  if (per_head_norm || n_tokens <= 0) return 0;
  return sumsq_bytes(n_tokens, n_heads) + (size_t)2 * n_tokens * n_heads * kHeadDim * sizeof(uint16_t);
}

template <int TOK>
static void launch_tiles(const ProjArgs& a, hipStream_t st) {
  const ProjTiles pt = make_tiles(a.n_tokens, a.n_heads, TOK);
  const dim3 grid(project_blocks(pt)), block(kThreads);
  if (a.per_head_norm) hipLaunchKernelGGL((qkv_project_kernel<TOK, true>), grid, block, 0, st, a, pt);
  else hipLaunchKernelGGL((qkv_project_kernel<TOK, false>), grid, block, 0, st, a, pt);
}

int project_tile_tokens(int n_tokens, int n_heads, int c_in) { return project_tile_width(n_tokens, n_heads, c_in); }

hipError_t launch_project(const ProjArgs& a_in, hipStream_t st) {
  ProjArgs a = a_in;
  if (!a.per_head_norm)
    a.resid = reinterpret_cast<uint16_t*>(reinterpret_cast<uint8_t*>(a.sumsq) + sumsq_bytes(a.n_tokens, a.n_heads));
  if (project_tile_tokens(a.n_tokens, a.n_heads, a.c_in) == 256) launch_tiles<256>(a, st);
  else launch_tiles<192>(a, st);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.per_head_norm) return e;
  hipLaunchKernelGGL(scale_rows_kernel, dim3(2, (a.n_tokens + kScaleWaves - 1) / kScaleWaves),
                     dim3(64 * kScaleWaves), 0, st, a);
  return hipGetLastError();
}

}  // namespace crope
