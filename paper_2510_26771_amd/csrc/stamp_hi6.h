// The 8-bit rows on the FP6 matrix pipeline (stamp_hi6.hip): layout and conversion of the operand.
//
// An 8-bit code c is 16 h + l with l in [-8, 7], h in [-8, 8]: two FP6 rows (E2M3 numbers h / 8, l / 8), whose sums over
// 4-bit weights are exact, and 16 times the one plus the other is the integer sum of the 8-bit row.  Rows are kept in groups
// of 32 * np (np = 1 or 2): [group][K step][2 np blocks: h and l of rows 0..31, h and l of rows 32..63][3 KB], a block as
// in stamp_gemm6.hip.
#ifndef STAMP_HI6_H_
#define STAMP_HI6_H_

#include "stamp_fp6.h"

namespace stamp_gemm {

// a lane's 48 bytes of a block: the operands of its two tiles of 16 rows (per-block scales: of the two halves of the K step).  (The middle
// part read as two 8-byte halves, which would save the moves: every line of it is touched twice, 17.4 us become 20.3.)
struct Frag6 {
  u4 p0, p1, p2;
  __device__ __forceinline__ void load(const uint8_t* q /* wave-uniform */, uint32_t lane16) {
    p0 = *reinterpret_cast<const u4*>(q + lane16);
    p1 = *reinterpret_cast<const u4*>(q + kPart + lane16);
    p2 = *reinterpret_cast<const u4*>(q + 2 * kPart + lane16);
  }
  // the builtin's operand has 8 registers, of which the instruction reads 6
  __device__ __forceinline__ v8i h0() const { return (v8i)__builtin_shufflevector(p0, p1, 0, 1, 2, 3, 4, 5, -1, -1); }
  __device__ __forceinline__ v8i h1() const { return (v8i)__builtin_shufflevector(p1, p2, 2, 3, 4, 5, 6, 7, -1, -1); }
};

// 32 codes (bytes) -> floats, channels 2 i in ev[i], 2 i + 1 in od[i]
__device__ __forceinline__ void codes32(const u4 (&w)[2], f16v& ev, f16v& od) {
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const uint32_t x = w[i >> 3][(i >> 1) & 3] << (16 - 16 * (i & 1));
    ev[i] = (float)((int)(x << 8) >> 24);
    od[i] = (float)((int)x >> 24);
  }
}

// one thread = 32 channels of a row, or of a place in the tiles of the 4-bit rows
__device__ __forceinline__ void hi6_pack(const StampHi6Pack& hp, int i) {
  if (i >= hp.threads) return;
  const StampHiOut& o = hp.out;
  const int nf = hp.KT * 4, m = i / nf, frag = i - m * nf, kt = frag >> 2, f = frag & 3;
  int row;
  uint8_t* dst;
  bool hf = false;
  if (o.ht.on) {
    int b, slot, tile, place, n;
    if (hp.places == 0) {
      b = m / o.seq;
      slot = m - b * o.seq;
      stamp_hi_places(o.ht, b, slot, &tile, &n, &place);
    } else {
      tile = m / hp.places;
      place = m - tile * hp.places;
      slot = stamp_hi_slot_of_place(o.ht, hp.nseq, tile, place, &b, &n);
      if (slot < 0) return;  // (a place without a row may hold anything)
    }
    row = b * hp.seq_rows + slot;
    dst = o.p + ((size_t)tile * hp.KT + kt) * kBlock6 + f * 256 + place * 16;
  } else {
    const int gr = 32 * o.np, grp = m / gr, r = m - grp * gr;
    row = m < hp.M ? m + (m / o.seq) * (hp.seq_rows - o.seq) : -1;
    dst = o.p + ((size_t)grp * hp.KT + kt) * (2 * o.np * kBlock6) + (r >> 5) * (2 * kBlock6) + f * 256 + row_lane6((uint32_t)r & 31);
    hf = hi_half6((uint32_t)r);
  }
  u4 w[2] = {};
  if (row >= 0 && frag * 32 < hp.d) {  // d is a multiple of 32
    const u4* src = reinterpret_cast<const u4*>(hp.q_hi + (size_t)row * hp.d + frag * 32);
    w[0] = src[0];
    w[1] = src[1];
  }
  // (field by field, some 1500 instructions in place of these 200: q_hi and q_lo of 2 x 1024 x 4096 in 6.4 us, now 6.0)
  f16v ev, od;
  codes32(w, ev, od);
  u6v hh, ll;
  split_hi(ev, od, hh, ll);
  store24(dst, hh, !o.ht.on && hf);
  store24(dst + (o.ht.on ? 0 : kBlock6), ll, o.ht.on || hf);
}

// 32 packed codes each of two rows (repack6_dist apart) -> a lane's 48 bytes of a block
__device__ __forceinline__ void repack6_store(uint8_t* dst, u4 w0, u4 w1) {
  uint64_t lo[3], hi[3];
  chunk_to_e2m3(w0, lo);
  chunk_to_e2m3(w1, hi);
  typedef uint64_t ul2 __attribute__((ext_vector_type(2)));
  *reinterpret_cast<ul2*>(dst) = ul2{lo[0], lo[1]};
  *reinterpret_cast<ul2*>(dst + kPart) = ul2{lo[2], hi[0]};
  *reinterpret_cast<ul2*>(dst + 2 * kPart) = ul2{hi[1], hi[2]};
}

// The two rows of unit u = 0 .. 511 of a (row tile, K step): the first of them, how far on the other is, and fragment
__device__ __forceinline__ int repack6_row(int u, int gb) {
  const int blk = __builtin_amdgcn_readfirstlane(u >> 6);  // (the same for a wave)
  return (blk >> 2) * 128 + (int)row_of_rest6((uint32_t)(blk & 3) * 16, gb) + (int)row_of_rest6((uint32_t)u & 7, gb) + (((u >> 3) & 1) << gb);
}
__device__ __forceinline__ int repack6_dist(int gb) { return (int)row_of_rest6(8, gb); }
__device__ __forceinline__ int repack6_frag(int u) { return (u >> 4) & 3; }
// packed 4-bit rows -> operand: block `blk` = (row tile, K step), unit u of it
__device__ __forceinline__ void repack6_rows(const uint8_t* __restrict__ q_lo, uint8_t* __restrict__ a6, size_t blk, int u, int gb) {
  const uint8_t* src = q_lo + blk * (256 * 64) + repack6_row(u, gb) * 64 + repack6_frag(u) * 16;
  repack6_store(a6 + blk * kStageA6 + (u >> 6) * kBlock6 + (u & 63) * 16, *reinterpret_cast<const u4*>(src),
                *reinterpret_cast<const u4*>(src + repack6_dist(gb) * 64));
}

}  // namespace stamp_gemm

#endif  // STAMP_HI6_H_
