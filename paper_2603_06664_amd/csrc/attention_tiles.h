// Key and value tiles of the attention kernel: their copies from memory to LDS.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "crope_internal.h"

namespace crope {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x16_t __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) uint8_t lds_byte;

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  f32x2_t f = {lo, hi};
  bf16x2_t h = __builtin_convertvector(f, bf16x2_t);
  return __builtin_bit_cast(uint32_t, h);
}

constexpr int kRowBytes = kHeadDim * 2;  // 256 B per key row in LDS (swizzled, unpadded)
constexpr int kBlkBytes = 32 * kRowBytes;   // a block of 32 keys
constexpr int kWaves = 4;                // waves per work-group, one per SIMD
constexpr int kCopyRows = 4 * kWaves;    // tile rows one copy instruction of every wave moves

// HBM -> LDS tile copy by a work-group.  Load instruction t of wave w moves tile rows
// 16*t + 4*w .. +3: lane i carries one 16-byte chunk of row 16*t + 4*w + i/16 into LDS
// position (that row, chunk i%16); which global chunk it fetches implements the swizzle:
//   K: row r, 16-byte chunk c (8 channels) at r*256 + ((c ^ (r&15))*16)
//   V: row r, 32-byte pair slot p (16 channels) at r*256 + ((p ^ (r&mask))*32), mask by the shape of the wave
// The swizzle depends on the row only through 4*w + i/16 and ONE per-lane byte offset
// serves every t.  In a tile whose keys are consecutive cache rows (the common case) the lane's
// address advances by 16 rows from copy to copy.
struct Loader {     // scalars only, so that it is promoted to registers at once
  const uint8_t *k_head, *v_head;    // cache base of this head (bytes)
  int seg_end0, seg_end1, seg_end2;  // visible key index -> cache row: vk + base of its segment
  int seg_base3, d2, d1, d0;         // base3, base2-base3, base1-base2, base0-base1
  int64_t row_bytes;                 // c_tok * 2
  int row0;       // 4*wave + lane/16
  int key_first;  // first visible key of this work-group's split
  int key_end;    // one past its last
  uint32_t k_chunk, v_chunk;         // swizzled chunk offset inside the lane's row
  uint32_t k_lane_off, v_lane_off;   // row0 * row_bytes + chunk offset
};

// 16 bytes per lane, HBM -> LDS without passing through registers: lane i's data lands at
// LDS address lds_dst + 16*i.  The LDS base travels in M0, which the compiler loads itself
// (an input operand bound to that register); the s_nop covers the wait state the hardware
// wants between a write of M0 and a copy that uses it.  Written as inline assembly, not
// with the compiler's builtin: while a builtin copy is in flight the compiler's wait-count
// insertion turns every later "wait for this LDS read" into "wait for ALL LDS reads", which
// exposes the full LDS latency at each MFMA that consumes a fragment.  The copies are
// waited for explicitly (s_waitcnt vmcnt) before the barrier that publishes a tile.
// The address is a per-lane register pair on purpose: a scalar base that the compiler reloads
// from a spill (v_readlane) right in front of the assembly would need five wait states that it does
// not insert for instructions it cannot see.
__device__ __forceinline__ void copy16(const uint8_t* src, uint32_t lds_dst /* wave-uniform */) {
  const uint32_t m0 = __builtin_amdgcn_readfirstlane(lds_dst);
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off" :: "v"(src), "{m0}"(m0) : "memory");
}
// The same from a buffer: base and advance are scalar, the lane's share of the address never changes.  `off` moves
// on by `step` in front of the copy, which also is the wait state behind the write of M0.  The buffer's words
// are formed by scalar instructions ahead of the loop (a vector instruction that wrote one of them would need
// five wait states; the tests check the assembly for both distances).
__device__ __forceinline__ void copy16_step(uint32_t& off, uint32_t step, u32x4_t rsrc, uint32_t lane_off, uint32_t lds_dst) {
  const uint32_t m0 = __builtin_amdgcn_readfirstlane(lds_dst);
  asm volatile("s_add_u32 %0, %0, %1\n\tbuffer_load_dwordx4 %2, %3, %0 offen lds"
               : "+s"(off) : "s"(step), "v"(lane_off), "s"(rsrc), "{m0}"(m0) : "memory", "scc");
}
// A raw buffer without bounds that matter: base, 2^32 - 1 bytes, 32-bit elements.  Offsets stay inside: a tile
// spans 128 rows of at most 2^25 bytes.
__device__ __forceinline__ u32x4_t raw_buffer(const uint8_t* base /* wave-uniform */) {
  const uint64_t a = (uint64_t)base;
  return u32x4_t{(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a),
                 (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32)), 0xffffffffu, 0x00020000u};
}
__device__ __forceinline__ void advance(u32x4_t& r, int64_t bytes) {
  const uint64_t a = ((uint64_t)r[1] << 32 | r[0]) + (uint64_t)bytes;
  r[0] = (uint32_t)a;
  r[1] = (uint32_t)(a >> 32);
}

__device__ __forceinline__ int seg_row(const Loader& L, int vk) {
  // arithmetic select (no value select the compiler could turn into a table lookup)
  return vk + L.seg_base3 + (vk < L.seg_end2 ? L.d2 : 0) + (vk < L.seg_end1 ? L.d1 : 0) +
         (vk < L.seg_end0 ? L.d0 : 0);
}

// end of the segment that holds visible key vk
__device__ __forceinline__ int segment_end(const Loader& L, int vk) {
  return vk < L.seg_end0 ? L.seg_end0 : vk < L.seg_end1 ? L.seg_end1 : vk < L.seg_end2 ? L.seg_end2 : INT32_MAX;
}

// the BN keys from k0 on are all visible to this split and lie in one segment (consecutive cache rows)
template <int BN>
__device__ __forceinline__ bool plain_tile(const Loader& L, int k0) {
  const int k1 = k0 + BN - 1;
  return k1 < L.key_end && !((k0 < L.seg_end0 && k1 >= L.seg_end0) || (k0 < L.seg_end1 && k1 >= L.seg_end1) ||
                             (k0 < L.seg_end2 && k1 >= L.seg_end2));
}

// The whole tile at once, any rows: tiles that straddle a segment boundary or the end of the keys
// look their rows up per lane; rows past the end re-read the last key (their scores are masked).
template <bool IS_V, int BN>
__device__ __forceinline__ void load_tile(const Loader& L, int tile, uint32_t dst /* incl. wave * 1024 */) {
  const int k0 = L.key_first + tile * BN;   // wave-uniform
  const uint8_t* head = IS_V ? L.v_head : L.k_head;
  if (plain_tile<BN>(L, k0)) {
    const uint8_t* src = head + (int64_t)seg_row(L, k0) * L.row_bytes + (IS_V ? L.v_lane_off : L.k_lane_off);
#pragma unroll
    for (int t = 0; t < BN / kCopyRows; ++t, src += kCopyRows * L.row_bytes) copy16(src, dst + t * kCopyRows * kRowBytes);
  } else {
#pragma unroll 1
    for (int t = 0; t < BN / kCopyRows; ++t) {
      const int vk = min(k0 + L.row0 + kCopyRows * t, L.key_end - 1);
      copy16(head + (int64_t)seg_row(L, vk) * L.row_bytes + (IS_V ? L.v_chunk : L.k_chunk), dst + t * kCopyRows * kRowBytes);
    }
  }
}

// The copies of a plain tile, issued one by one between the MFMAs: all of K, then all of V.  Behind
// the barrier in one burst they kept every wave waiting for the address unit (64 lanes x 16 B take
// it 16 clocks): 762 against 722 us.  One per 3 slots: a slot is one MFMA of Narrow, whose last copy then leaves
// at slot 22 of 32 with 31 % of the tile's time to land, and two of Wide, whose last one leaves at slot 46 of 128 with 64 %.
template <int BN>
struct Feed {
  static constexpr int kCopies = BN / kCopyRows;   // per wave and tensor
  static constexpr int kEvery = 3;
  u32x4_t k, v;              // the tile's first row, as a buffer
  uint32_t lane_k, lane_v;   // per lane
  uint32_t off, step;
  uint32_t k_dst, v_dst;
  __device__ __forceinline__ void slot(int s) {   // s: slot inside the tile (of the shape's kSlots per block), compile-time
    if (s % kEvery != 1 || s / kEvery >= 2 * kCopies) return;
    const int i = s / kEvery;
    if (i == kCopies) off = 0u - step;
    const uint32_t dst = i < kCopies ? k_dst + i * kCopyRows * kRowBytes : v_dst + (i - kCopies) * kCopyRows * kRowBytes;
    copy16_step(off, step, i < kCopies ? k : v, i < kCopies ? lane_k : lane_v, dst);
  }
};
struct NoFeed {
  __device__ __forceinline__ void slot(int) {}
};

// Every copy of this wave has landed, then the work-group's barrier (without the fence of
// __syncthreads(), which would also wait for the fragment reads in flight).
__device__ __forceinline__ void publish_tiles() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

}  // namespace
}  // namespace crope
