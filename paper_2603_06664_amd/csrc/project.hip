// Local QKV projection with qk-RMSNorm, causal 3D RoPE and the KV-cache update applied in
// the GEMM's epilogue (Algorithm 3 steps 1, 2, 3 and 5 in one pass; the operator fusion of
// Section 3.4.1 item 3), bf16 MFMA on gfx950.
//
// y[token][o] = sum_c x[token][c] * w[o][c] + bias[o];  o in [0, HD) is q, [HD, 2HD) k,
// [2HD, 3HD) v.  Both operands have the reduction index contiguous, so both are MFMA
// fragments as they lie in memory.  The product is formed transposed, C^T = W . x^T
// (channels = MFMA rows, tokens = columns): an accumulator lane then holds 4 consecutive
// channels of ONE token, i.e. two whole rotation pairs, and the epilogue needs no cross-lane
// traffic for the rotation; the bf16 tile is then transposed through LDS and leaves in whole
// 256-byte (token, head) rows.
//
// A work-group owns 128 output channels (one head of q, k or v) x 256 tokens (8 waves of 64 x 64, two
// per SIMD) or x 192 tokens (4 waves of 64 x 96, one per SIMD); launch_project says which one when.
// What bounds a full chip is the 256-wide loop at 1.2 PFLOP/s (18720 x 1536 -> 4608, row-wide norm
// and all epilogues included 336 us = 0.79 PFLOP/s; 344 us before the copies and fragment reads were
// spread between the MFMAs one by one), and then the serial epilogue; what bounds a small call is how
// its tiles divide over 256 CUs.  The reduction runs in steps of
// 64 through three LDS stages filled by global_load_lds (16 B per lane, no registers), one
// barrier per step.  LDS rows are 128 B; 16-byte chunk c of row r sits at slot
// c ^ ((r >> 1) & 7), which makes the fragment reads (32 rows x 16 B per half wave)
// conflict-free.
//
// RMSNorm over one head is local to the tile and fully fused.  RMSNorm over the token's
// whole H*128 vector needs every head's sum of squares: the rotation commutes with the
// per-token scalar, so the epilogue stores z = rotate(gain * y) and the per-head sums of
// squares, and a second, bandwidth-bound pass multiplies q and k rows by 1/rms.  z is kept
// as TWO bf16 numbers, hi = bf16(z) in the destination row and lo = bf16(z - hi) in the
// workspace (16 mantissa bits together), so that the second pass rounds (hi + lo) / rms to
// bf16 once: the stored result is the single rounding of the fp32 value up to 2^-17 relative.
#include "crope_internal.h"

namespace crope {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));

#define LDS_ADDR(p) ((uint32_t)(uintptr_t)((__attribute__((address_space(3))) void*)(p)))

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  f32x2_t f = {lo, hi};
  bf16x2_t h = __builtin_convertvector(f, bf16x2_t);
  return __builtin_bit_cast(uint32_t, h);
}
__device__ __forceinline__ float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }
__device__ __forceinline__ float sum_across_halves(float x) {
  const u32x2_t r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

constexpr int kTileCh = 128;    // output channels per work-group: one head
constexpr int kStepK = 64;      // reduction elements per LDS stage
constexpr int kRowB = kStepK * 2;             // 128 B per LDS row
constexpr int kStageA = kTileCh * kRowB;      // 16 KB
constexpr int kOutRowB = kTileCh * 2 + 16;    // bf16 output tile row in LDS, padded against bank conflicts
constexpr int kAngRowB = 64 * 8 + 16;         // one token's 64 (cos, sin) pairs in LDS, padded (16-byte rows)
constexpr int kXcds = 8;
constexpr int kTokGroup = 4;    // token tiles walked together with 8 channel tiles by one XCD's CUs

struct ProjTiles {
  int ch_tiles, tok_tiles, total, per_xcd;
  int wgs_per_xcd;   // work-groups launched per XCD (at most its 32 CUs)
};

// Shape of a work-group: 2 (channel halves) x WT waves, each 64 channels x 32*TT tokens.
template <int WT_, int TT_>
struct Shape {
  static constexpr int WT = WT_, TT = TT_;
  static constexpr int kWaves = 2 * WT, kThreads = 64 * kWaves;
  static constexpr int kWaveTok = 32 * TT, kTileTok = kWaveTok * WT;
  static constexpr int kACopies = kTileCh / (8 * kWaves);   // copies per wave and stage of the W tile
  static constexpr int kCopies = kACopies + 2 * TT;         // and of the x tile behind it
  static constexpr int kStage = kStageA + kTileTok * kRowB;
};

template <class S>
struct TileLoader {   // scalars only
  u32x4_t a_buf;           // W from the tile's first channel row on
  u32x4_t b_buf;           // x from the tile's first token row on
  // per-lane byte offsets of the lane's chunk for load instruction t: row 8*wave + lane/8 + 8*waves*t
  uint32_t a_off[S::kACopies];
  uint32_t b_off[2 * S::TT];
  int lds_off;             // wave * 1024
};

// Copy instruction t of wave w covers tile rows 8*(w + waves*t) .. +7 (1 KB of LDS): lane i carries
// the chunk that belongs at (row 8*(w + waves*t) + i/8, slot i%8).  ((row >> 1) & 7) = (i>>4) | 4*(w&1)
// does not depend on t.  Token rows past the end re-read the last token (clamped when the
// offsets are formed); their results are never stored.
// The copy is inline assembly, not the compiler's builtin: while a builtin copy is in flight
// the compiler turns every counted wait on an LDS read into a wait for all of them.  LDS
// address of lane i's 16 bytes: M0 + 16*i; M0 is an input operand bound to that register, the
// s_nop covers the wait state after its write.  Base and step are scalar (a buffer and its scalar offset), so that a
// copy costs no vector instruction and two scalar ones (585 rows x 40 heads 106.9 -> 101.7 us, 600 x 8 17.7 -> 16.3,
// W in the last-level cache; with 64-bit bases and LDS addresses taken from pointers it were eight).  A vector instruction that wrote one of the
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

// copy i of reduction step kt: the W tile first, then the x tile behind it in the stage
template <class S>
__device__ __forceinline__ void load_copy(const TileLoader<S>& L, int kt, uint32_t stage, int i) {
  const uint32_t k_off = (uint32_t)kt * kRowB;
  if (i < S::kACopies) copy16(L.a_buf, L.a_off[i], k_off, stage + L.lds_off + i * (S::kWaves * 1024));
  else copy16(L.b_buf, L.b_off[i - S::kACopies], k_off, stage + L.lds_off + i * (S::kWaves * 1024));
}
template <class S>
__device__ __forceinline__ void load_stage(const TileLoader<S>& L, int kt, uint32_t stage) {
#pragma unroll
  for (int i = 0; i < S::kCopies; ++i) load_copy<S>(L, kt, stage, i);
}

template <int TT>
struct Frags {
  bf16x8_t a[2], b[TT];
};

// fragment i of sub-step kk, in the order in which the MFMAs want them
template <int TT>
__device__ __forceinline__ void read_frag(Frags<TT>& f, const uint8_t* stage, int a_off0, int b_off0, int kk, int i) {
  if (i < 2)
    f.a[i] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(stage + ((a_off0 ^ (kk << 5)) + i * 4096)));
  else
    f.b[i - 2] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(
                                                  stage + kStageA + ((b_off0 ^ (kk << 5)) + (i - 2) * 4096)));
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

// One reduction step: 4 sub-steps of 2*TT MFMAs.  On entry f0 holds the fragments of sub-step 0 of
// stage `rd`.  Behind every MFMA stands at most one fragment read of the next sub-step and one copy
// of the stage two steps ahead, in this order (a burst of copies would leave
// the matrix unit idle while the address unit works it off).  The last sub-step holds
// the step's barrier behind its first MFMA and reads the next stage's first fragments.
template <class S, bool STEADY>   // STEADY: kt + 2 < n_kt is known, no conditions in the step
__device__ __forceinline__ void step(f32x16_t (&acc)[2][S::TT], Frags<S::TT>& f0, Frags<S::TT>& f1,
                                     const TileLoader<S>& L, int kt, int n_kt, const uint8_t* rd, uint32_t ld, const uint8_t* nx, int a_off0,
                                     int b_off0) {
  constexpr int TT = S::TT, kMfmas = 2 * TT, kCopies = S::kCopies;
  const bool prefetch = STEADY || kt + 2 < n_kt;
  const bool more = STEADY || kt + 1 < n_kt;
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    Frags<TT>& f = kk & 1 ? f1 : f0;
    Frags<TT>& f_next = kk & 1 ? f0 : f1;
#pragma unroll
    for (int m = 0; m < kMfmas; ++m) {
      acc[m & 1][m >> 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[m & 1], f.b[m >> 1], acc[m & 1][m >> 1], 0, 0, 0);
      if (kk < 3) {
        if (m < 2 + TT) read_frag<TT>(f_next, rd, a_off0, b_off0, kk + 1, m);
        const int s = kk * kMfmas + m;
        const int i = s * kCopies / (3 * kMfmas);
        if (prefetch && (s + 1) * kCopies / (3 * kMfmas) > i) load_copy<S>(L, kt + 2, ld, i);
      } else if (m == 0) {
        // every read of stage rd has completed before any wave may overwrite it (next step), and the
        // next stage has landed
        if (prefetch) wait_and_barrier<kCopies>();
        else wait_and_barrier<0>();
        if (more && TT < 3) read_frag<TT>(f_next, nx, a_off0, b_off0, 0, 1 + TT);   // no slot left for it below
      } else if (more && m - 1 < (TT < 3 ? 1 + TT : 2 + TT)) {
        read_frag<TT>(f_next, nx, a_off0, b_off0, 0, m - 1);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// unit -> (channel tile, token tile).  Units are ordered so that 32 consecutive ones (what an
// XCD's 32 CUs hold at a time) form 8 channel tiles x 4 token tiles: their W and x tiles
// together stream through that XCD's L2 once.
__device__ __forceinline__ void unit_to_tile(const ProjTiles& pt, int unit, int& ch_tile, int& tok_tile) {
  const int per_group = kTokGroup * pt.ch_tiles;
  const int full_groups = pt.tok_tiles / kTokGroup;
  int grp = unit / per_group;
  int gs = kTokGroup;
  if (grp >= full_groups) { grp = full_groups; gs = pt.tok_tiles - kTokGroup * full_groups; }
  const int local = unit - grp * per_group;
  ch_tile = local / gs;
  tok_tile = kTokGroup * grp + local % gs;
}

template <class S, bool PER_HEAD>
__global__ __attribute__((amdgpu_flat_work_group_size(S::kThreads, S::kThreads), amdgpu_waves_per_eu(S::kWaves / 4, S::kWaves / 4)))
void qkv_project_kernel(ProjArgs a, ProjTiles pt) {
  constexpr int WT = S::WT, TT = S::TT, kWaves = S::kWaves, kThreads = S::kThreads;
  constexpr int kTileTok = S::kTileTok, kWaveTok = S::kWaveTok, kStage = S::kStage, kCopies = S::kCopies;
  constexpr int kAngBytes = kTileTok * kAngRowB;
  // three stages of (W tile 16 KB, x tile 4*WT*TT KB); the epilogue reuses the space
  constexpr int kLds = 3 * kStage;
  static_assert(kAngBytes + 2 * kTileTok * (int)sizeof(float) <= kLds && kTileTok * kOutRowB <= kLds, "epilogue in LDS");
  __shared__ __attribute__((aligned(1024))) uint8_t lds[kLds];
  uint8_t* const lds0 = lds;
  uint8_t* const lds1 = lds + kStage;
  uint8_t* const lds2 = lds + 2 * kStage;
  const uint32_t dst0 = LDS_ADDR(lds), dst1 = dst0 + kStage, dst2 = dst1 + kStage;   // the same, for the copies

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, g = lane >> 5;
  const int wc = wave & 1, wt = wave >> 1;   // channel half, token part of the tile

  // Persistent work-groups, one per CU: a work-group walks its XCD's run of the unit list in
  // strides of the XCD's CU count.  Not ending between tiles lets a tile's output stores drain
  // under the next tile's reduction instead of holding up the hand-over of the CU.
  for (int idx = (int)(blockIdx.x / kXcds); idx < pt.per_xcd; idx += pt.wgs_per_xcd) {
  const int unit = (int)(blockIdx.x % kXcds) * pt.per_xcd + idx;
  if (unit >= pt.total) break;   // wave-uniform; the whole work-group leaves together
  int ch_tile, tok_tile;
  unit_to_tile(pt, unit, ch_tile, tok_tile);
  const int tok0 = tok_tile * kTileTok;

  TileLoader<S> L;
  {
    const int l_row = lane >> 3, l_slot = lane & 7;
    const int f = (lane >> 4) | ((wave & 1) << 2);
    const uint32_t chunk_bytes = (uint32_t)((l_slot ^ f) * 16);
    const int row = 8 * wave + l_row;
    const int64_t a_row_bytes = (int64_t)a.c_in * 2, b_row_bytes = a.x_tok * 2;
    L.a_buf = raw_buffer(reinterpret_cast<const uint8_t*>(a.w) + (int64_t)ch_tile * kTileCh * a_row_bytes);
    L.b_buf = raw_buffer(reinterpret_cast<const uint8_t*>(a.x) + (int64_t)tok0 * b_row_bytes);
    const int last = a.n_tokens - 1 - tok0;   // >= 0
#pragma unroll
    for (int t = 0; t < S::kACopies; ++t) L.a_off[t] = (uint32_t)((row + 8 * kWaves * t) * a_row_bytes) + chunk_bytes;
#pragma unroll
    for (int t = 0; t < 2 * TT; ++t) L.b_off[t] = (uint32_t)(min(row + 8 * kWaves * t, last) * b_row_bytes) + chunk_bytes;
    L.lds_off = wave * 1024;
  }
  // fragment read offsets: row (64*wc or 32*TT*wt, + n), 16-byte chunk 2*kk + g -> slot ((2kk+g) ^ ((n>>1)&7))
  const int fl = (n >> 1) & 7;
  const int a_off0 = (64 * wc + n) * kRowB + ((g ^ fl) << 4);
  const int b_off0 = (kWaveTok * wt + n) * kRowB + ((g ^ fl) << 4);

  f32x16_t acc[2][TT];
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[c][t][i] = 0.f;

  const int n_kt = a.c_in / kStepK;
  Frags<TT> f0, f1;
  load_stage<S>(L, 0, dst0);
  if (n_kt > 1) {
    load_stage<S>(L, 1, dst1);
    wait_and_barrier<kCopies>();
  } else {
    wait_and_barrier<0>();
  }
#pragma unroll
  for (int i = 0; i < 2 + TT; ++i) read_frag<TT>(f0, lds0, a_off0, b_off0, 0, i);
  // lgkmcnt(0): enter the loop with nothing pending, so that the loop's own waits are counted
  // ones (a pending scalar load would make the compiler wait for every LDS read instead)
  __builtin_amdgcn_s_waitcnt(0xC07F);
  int kt = 0;
  for (; kt + 4 < n_kt; kt += 3) {   // steady state: every step prefetches two steps ahead
    step<S, true>(acc, f0, f1, L, kt, n_kt, lds0, dst2, lds1, a_off0, b_off0);
    step<S, true>(acc, f0, f1, L, kt + 1, n_kt, lds1, dst0, lds2, a_off0, b_off0);
    step<S, true>(acc, f0, f1, L, kt + 2, n_kt, lds2, dst1, lds0, a_off0, b_off0);
  }
  for (; kt < n_kt; kt += 3) {       // the last (up to four) steps
    step<S, false>(acc, f0, f1, L, kt, n_kt, lds0, dst2, lds1, a_off0, b_off0);
    if (kt + 1 >= n_kt) break;
    step<S, false>(acc, f0, f1, L, kt + 1, n_kt, lds1, dst0, lds2, a_off0, b_off0);
    if (kt + 2 >= n_kt) break;
    step<S, false>(acc, f0, f1, L, kt + 2, n_kt, lds2, dst1, lds0, a_off0, b_off0);
  }

  // ------------------------------------------------------------------ epilogue
  // acc[c][t][i]: token tok0 + 32*TT*wt + 32*t + n, channel 64*wc + 32*c + 8*(i/4) + 4*g + i%4 of the head.
  // The closing barrier of the last step has passed: every wave is done with the stages.  The
  // LDS now holds, in turn, the (cos, sin) rows of the tile's tokens (gathered with pairs
  // on the lane axis, where a token's position is wave-uniform and its 64 pairs are three
  // contiguous runs of the tables, then read back with tokens on the lane axis at constant
  // offsets), the sums of squares, and the bf16 output tile, which leaves in whole 256-byte
  // (token, head) rows.
  uint8_t* const out_lds = lds;                                     // [tile tokens][kOutRowB]
  uint8_t* const ang_lds = lds;                                     // [tile tokens][kAngRowB]: 64 x (cos, sin)
  float* const ss_lds = reinterpret_cast<float*>(lds + kAngBytes);  // [wc][wt][t][32]
  const int which = ch_tile / a.n_heads;   // 0: q, 1: k, 2: v
  const int head = ch_tile - which * a.n_heads;
  // bias and gain of the lane's 32 channels: all loads issued together, ahead of their use
  float4 gv[2][4];
  if (which != 2) {
    const float* gp = (which == 0 ? a.gain_q : a.gain_k) + head * kHeadDim + 64 * wc + 4 * g;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int b = 0; b < 4; ++b) gv[c][b] = *reinterpret_cast<const float4*>(gp + 32 * c + 8 * b);
  }
  if (a.bias) {
    const float* bp = a.bias + (int64_t)ch_tile * kTileCh + 64 * wc + 4 * g;
    float4 bv[2][4];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int b = 0; b < 4; ++b) bv[c][b] = *reinterpret_cast<const float4*>(bp + 32 * c + 8 * b);
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int t = 0; t < TT; ++t) {
          acc[c][t][4 * b + 0] += bv[c][b].x; acc[c][t][4 * b + 1] += bv[c][b].y;
          acc[c][t][4 * b + 2] += bv[c][b].z; acc[c][t][4 * b + 3] += bv[c][b].w;
        }
  }
  uint32_t packed[TT][2][4][2];      // [t][c][b][pair of the 4 channels]
  uint32_t packed_lo[TT][2][4][2];   // row-wide norm: bf16 of what the first rounding dropped

  if (which == 2) {   // v: one rounding
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          packed[t][c][b][0] = pack_bf16x2(acc[c][t][4 * b + 0], acc[c][t][4 * b + 1]);
          packed[t][c][b][1] = pack_bf16x2(acc[c][t][4 * b + 2], acc[c][t][4 * b + 3]);
        }
  } else {
    const int p_t = a.tl.pairs_t, p_h = a.tl.pairs_h, p_w = a.tl.pairs_w, p_th = p_t + p_h;
    const float2* tab2 = reinterpret_cast<const float2*>(a.table);
    // ---- gather: wave w fetches the rows of the tile's part w.  Positions are decoded
    // with tokens on the lane axis; for the fetch the lane axis is the pair index (a token's
    // 64 pairs are three contiguous runs of the tables) and token rr's table row offsets are
    // broadcast from lane rr.  Lane j needs exactly one of the three offsets.
    {
      constexpr int kGather = kTileTok / kWaves, kBatch = kGather / 2;
      const int last_tok = a.n_tokens - 1;
      const int ig = a.token_offset + min(tok0 + kGather * wave + min(lane, kGather - 1), last_tok);   // past the end: last token's position
      const int hw = a.grid_h * a.grid_w;
      const int pf = ig / hw;
      const int rem = ig - pf * hw;
      const int ph = rem / a.grid_w;
      const int pw = rem - ph * a.grid_w;
      const int row_t = (a.start_frame + pf) * p_t, row_h = ph * p_h, row_w = pw * p_w;
      const int j = lane;
      const bool is_t = j < p_t, is_h = !is_t && j < p_th;
      const int m_t = is_t ? -1 : 0, m_h = is_h ? -1 : 0, m_w = (is_t || is_h) ? 0 : -1;
      const int cb = is_t ? (int)(a.tl.off_t / 2) + j
                          : is_h ? (int)(a.tl.off_h / 2) + (j - p_t) : (int)(a.tl.off_w / 2) + (j - p_th);
      uint8_t* dst = ang_lds + (kGather * wave) * kAngRowB + lane * 8;
#pragma unroll
      for (int b0 = 0; b0 < kGather; b0 += kBatch) {
        float2 row[kBatch];
#pragma unroll
        for (int rr = 0; rr < kBatch; ++rr) {
          const int st = __builtin_amdgcn_readlane(row_t, b0 + rr), sh = __builtin_amdgcn_readlane(row_h, b0 + rr),
                    sw = __builtin_amdgcn_readlane(row_w, b0 + rr);
          row[rr] = tab2[cb + ((st & m_t) | (sh & m_h) | (sw & m_w))];
        }
#pragma unroll
        for (int rr = 0; rr < kBatch; ++rr) *reinterpret_cast<float2*>(dst + (b0 + rr) * kAngRowB) = row[rr];
      }
    }
    // ---- sums of squares over the head: lane-local, the other half of the wave, the other wave
    float tot[TT];
    {
      float ss[TT];
#pragma unroll
      for (int t = 0; t < TT; ++t) {
        float sq = 0.f;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int i = 0; i < 16; ++i) sq = fmaf(acc[c][t][i], acc[c][t][i], sq);
        ss[t] = sum_across_halves(sq);
      }
      if (g == 0) {
#pragma unroll
        for (int t = 0; t < TT; ++t) ss_lds[((wc * WT + wt) * TT + t) * 32 + n] = ss[t];
      }
      __syncthreads();
#pragma unroll
      for (int t = 0; t < TT; ++t)
        tot[t] = ss_lds[((0 * WT + wt) * TT + t) * 32 + n] + ss_lds[((1 * WT + wt) * TT + t) * 32 + n];
    }
    float r[TT];
    if (PER_HEAD) {
#pragma unroll
      for (int t = 0; t < TT; ++t) r[t] = 1.0f / sqrtf(tot[t] * (1.0f / kHeadDim) + a.eps);
    } else {
#pragma unroll
      for (int t = 0; t < TT; ++t) r[t] = 1.0f;
      if (wc == 0 && g == 0) {
#pragma unroll
        for (int t = 0; t < TT; ++t) {
          const int token = tok0 + kWaveTok * wt + 32 * t + n;
          if (token < a.n_tokens) a.sumsq[((int64_t)which * a.n_tokens + token) * a.n_heads + head] = tot[t];
        }
      }
    }
    // ---- normalise, gain, rotate; the lane's pairs are 32*wc + 2*g + (16*c + 4*b + e)
    const uint8_t* ang_lane = ang_lds + (kWaveTok * wt + n) * kAngRowB + (32 * wc + 2 * g) * 8;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int b = 0; b < 4; ++b) {
#pragma unroll
        for (int t = 0; t < TT; ++t) {
          const float4 cs = *reinterpret_cast<const float4*>(ang_lane + 32 * t * kAngRowB + (16 * c + 4 * b) * 8);
          const float xa0 = acc[c][t][4 * b + 0] * r[t] * gv[c][b].x, xb0 = acc[c][t][4 * b + 1] * r[t] * gv[c][b].y;
          const float xa1 = acc[c][t][4 * b + 2] * r[t] * gv[c][b].z, xb1 = acc[c][t][4 * b + 3] * r[t] * gv[c][b].w;
          const float z0 = xa0 * cs.x - xb0 * cs.y, z1 = xa0 * cs.y + xb0 * cs.x;
          const float z2 = xa1 * cs.z - xb1 * cs.w, z3 = xa1 * cs.w + xb1 * cs.z;
          const uint32_t h0 = pack_bf16x2(z0, z1), h1 = pack_bf16x2(z2, z3);
          packed[t][c][b][0] = h0;
          packed[t][c][b][1] = h1;
          if (!PER_HEAD) {
            packed_lo[t][c][b][0] = pack_bf16x2(z0 - bf16_lo(h0), z1 - bf16_hi(h0));
            packed_lo[t][c][b][1] = pack_bf16x2(z2 - bf16_lo(h1), z3 - bf16_hi(h1));
          }
        }
      }
    __syncthreads();   // every wave has read its angles: the output tile may overwrite them
  }

  // ---- the tile leaves in whole token rows: 16 lanes x 16 B = the 256 bytes of one (token, head)
  {
    uint8_t* out_lane = out_lds + (kWaveTok * wt + n) * kOutRowB + (64 * wc + 4 * g) * 2;
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int b = 0; b < 4; ++b)
          *reinterpret_cast<uint2*>(out_lane + 32 * t * kOutRowB + (32 * c + 8 * b) * 2) =
              make_uint2(packed[t][c][b][0], packed[t][c][b][1]);
  }
  __syncthreads();
  {
    uint16_t* base;
    int64_t tstride;
    if (which == 0) { base = a.q_out + (int64_t)head * a.qo_head; tstride = a.qo_tok; }
    else {
      base = (which == 1 ? a.k_cache : a.v_cache) + a.dst_token * a.c_tok + (int64_t)head * a.c_head;
      tstride = a.c_tok;
    }
    const int chunk = tid & 15;
#pragma unroll 8
    for (int it = 0; it < kTileTok / (kThreads / 16); ++it) {
      const int row = (tid >> 4) + (kThreads / 16) * it;
      const int token = tok0 + row;
      if (token < a.n_tokens)
        *reinterpret_cast<uint4*>(base + (int64_t)token * tstride + chunk * 8) =
            *reinterpret_cast<const uint4*>(out_lds + row * kOutRowB + chunk * 16);
    }
  }
  __syncthreads();   // the output tile has been read: the next tile's copies may overwrite it
  if (!PER_HEAD && which != 2) {
    // the low parts take the same way out, into the workspace rows [which][token][head][128]
    uint8_t* out_lane = out_lds + (kWaveTok * wt + n) * kOutRowB + (64 * wc + 4 * g) * 2;
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int b = 0; b < 4; ++b)
          *reinterpret_cast<uint2*>(out_lane + 32 * t * kOutRowB + (32 * c + 8 * b) * 2) =
              make_uint2(packed_lo[t][c][b][0], packed_lo[t][c][b][1]);
    __syncthreads();
    uint16_t* base = a.resid + ((int64_t)which * a.n_tokens * a.n_heads + head) * kHeadDim;
    const int64_t tstride = (int64_t)a.n_heads * kHeadDim;
    const int chunk = tid & 15;
#pragma unroll 8
    for (int it = 0; it < kTileTok / (kThreads / 16); ++it) {
      const int row = (tid >> 4) + (kThreads / 16) * it;
      const int token = tok0 + row;
      if (token < a.n_tokens)
        *reinterpret_cast<uint4*>(base + (int64_t)token * tstride + chunk * 8) =
            *reinterpret_cast<const uint4*>(out_lds + row * kOutRowB + chunk * 16);
    }
    __syncthreads();
  }
  }   // next unit
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

template <class S>
static ProjTiles make_tiles(int n_tokens, int n_heads) {
  ProjTiles pt;
  pt.ch_tiles = 3 * n_heads;
  pt.tok_tiles = (n_tokens + S::kTileTok - 1) / S::kTileTok;
  pt.total = pt.ch_tiles * pt.tok_tiles;
  pt.per_xcd = (pt.total + kXcds - 1) / kXcds;
  pt.wgs_per_xcd = pt.per_xcd < 32 ? pt.per_xcd : 32;
  return pt;
}
static int rounds(const ProjTiles& pt) { return (pt.per_xcd + pt.wgs_per_xcd - 1) / pt.wgs_per_xcd; }

template <class S>
static void launch_tiles(const ProjArgs& a, hipStream_t st) {
  const ProjTiles pt = make_tiles<S>(a.n_tokens, a.n_heads);
  const dim3 grid(pt.wgs_per_xcd * kXcds), block(S::kThreads);
  if (a.per_head_norm) hipLaunchKernelGGL((qkv_project_kernel<S, true>), grid, block, 0, st, a, pt);
  else hipLaunchKernelGGL((qkv_project_kernel<S, false>), grid, block, 0, st, a, pt);
}

// Two token widths of a tile.  256: two waves per SIMD, the cheaper one per row (18720 tokens x 12
// heads: 336 us, 380 us in tiles of 192).  192: one wave per SIMD, for calls whose rounds of 256-wide
// tiles over the 256 CUs end nearly empty or whose last tile is mostly padding.  A round of 192-wide
// tiles takes 0.85 to 0.89 of a round of 256-wide ones where both take two rounds (585 rows x 120 channel
// tiles: 108 against 122 us; 4680 x 15: 104 / 123; 1320 x 48 in half-filled rounds: 51 / 58) and 0.84 to
// 0.98 where both take one (us, 192 / 256: 384 rows x 120 channel tiles, c_in 5120: 57 / 67; 600 x 36, 1536:
// 29.4 / 30.7; 600 x 24, 1024: 17.1 / 17.4), so it is taken where its rounds at that price are cheaper.  At
// short reductions the epilogue, which 8 waves work off faster, is most of a tile, and 256 is never the
// slower one (us, 192 / 256: 600 x 6, c_in 256: 11.7 / 11.2; 600 x 9, 384: 12.4 / 12.2; equal at 512 and 640).
// Tiles of 128 were never the fastest (122, 122, 61 us where the first three calls take 108, 104, 51).
using Wide = Shape<4, 2>;
using Mid = Shape<2, 3>;
constexpr double kMidCost = 0.88;
constexpr int kShortReduction = 512;

template <class S>
static int rounds(int n_tokens, int n_heads) { return rounds(make_tiles<S>(n_tokens, n_heads)); }

int project_tile_tokens(int n_tokens, int n_heads, int c_in) {
  const double mid_cost = c_in <= kShortReduction ? 1.0 : kMidCost;
  return rounds<Wide>(n_tokens, n_heads) <= rounds<Mid>(n_tokens, n_heads) * mid_cost ? Wide::kTileTok : Mid::kTileTok;
}

hipError_t launch_project(const ProjArgs& a_in, hipStream_t st) {
  ProjArgs a = a_in;
  if (!a.per_head_norm)
    a.resid = reinterpret_cast<uint16_t*>(reinterpret_cast<uint8_t*>(a.sumsq) + sumsq_bytes(a.n_tokens, a.n_heads));
  if (project_tile_tokens(a.n_tokens, a.n_heads, a.c_in) == Wide::kTileTok) launch_tiles<Wide>(a, st);
  else launch_tiles<Mid>(a, st);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.per_head_norm) return e;
  hipLaunchKernelGGL(scale_rows_kernel, dim3(2, (a.n_tokens + kScaleWaves - 1) / kScaleWaves),
                     dim3(64 * kScaleWaves), 0, st, a);
  return hipGetLastError();
}

}  // namespace crope
