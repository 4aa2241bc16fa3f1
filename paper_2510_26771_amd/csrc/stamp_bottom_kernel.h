// Device code of the bottom kernels of the activation path (see stamp_actquant.hip) and their launchers for one block length.
#ifndef STAMP_BOTTOM_KERNEL_H_
#define STAMP_BOTTOM_KERNEL_H_

#include <utility>

#include "stamp_fp6.h"
#include "stamp_internal.h"

namespace {

using stamp_gemm::cell2d;
using stamp_gemm::kBlock6;
using stamp_gemm::kPart;
using stamp_gemm::kStageA6;
using stamp_gemm::nib8_to_48;
using stamp_gemm::chan_off6;
using stamp_gemm::hi_half6;
using stamp_gemm::row_half6;
using stamp_gemm::row_lane6;
using stamp_gemm::row_off6;
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef uint32_t u2v __attribute__((ext_vector_type(2)));

constexpr float kInvSqrt2 = 0.70710678118654752440f;  // 0x3F3504F3
constexpr float kMagicLo = 12582920.0f;               // 1.5 * 2^23 + 8: fp32 add rounds to integer (RNE), low 4 bits = code + 8
constexpr uint32_t kMagicLoBits = 0x4B400000u;        // bit pattern of 1.5 * 2^23
constexpr uint32_t kPackBias = kMagicLoBits * 0x11111111u;  // sum over 8 nibble positions of the pattern's high bits (mod 2^32)

__device__ __forceinline__ float haar_norm(int level) {
  // 2^(-level/2): a power of two for even levels, fl(1/sqrt 2) times a power of two for odd ones
  return ldexpf((level & 1) ? kInvSqrt2 : 1.0f, -(level >> 1));
}

__device__ __forceinline__ float bf16lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// unsigned max over the 64 lanes (bit patterns of non-negative floats, or order keys of any floats);
// result is wave-uniform
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
  uint32_t y;
  y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, false);  // quad_perm [1,0,3,2]
  x = max(x, y);
  y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, false);  // quad_perm [2,3,0,1]
  x = max(x, y);
  y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xF, 0xF, false);  // row_half_mirror
  x = max(x, y);
  y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x140, 0xF, 0xF, false);  // row_mirror
  x = max(x, y);
  const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)x, 0);
  const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)x, 16);
  const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)x, 32);
  const uint32_t d = (uint32_t)__builtin_amdgcn_readlane((int)x, 48);
  return max(max(a, b), max(c, d));
}

// Order key of a float of either sign: a < b as floats  <=>  key(a) < key(b) as unsigned integers
// (negative: all bits flipped, otherwise the sign bit set).  0 is below the key of every number, so it is
// the neutral element of an unsigned max.  The asymmetric quantizer reduces max T and max -T in this form.
__device__ __forceinline__ uint32_t fkey(float f) {
  const uint32_t b = __float_as_uint(f);
  return b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u);
}
__device__ __forceinline__ float fkey_inv(uint32_t k) {
  return __uint_as_float(k ^ ((uint32_t)((int32_t)~k >> 31) | 0x80000000u));
}

__device__ __forceinline__ uint32_t absbits(float f) { return __float_as_uint(f) & 0x7FFFFFFFu; }

__device__ __forceinline__ uint32_t row_absmax_bits(const float (&v)[8]) {
  float m = fmaxf(fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3]))),
                  fmaxf(fmaxf(fabsf(v[4]), fabsf(v[5])), fmaxf(fabsf(v[6]), fabsf(v[7]))));
  return __float_as_uint(m);
}

// 8 codes -> one dword of two's complement nibbles (channel c in nibble c).
// p[c] = T * inv, |p| <= 7 (+1 ulp).  fl(p + magic) has rne(p) + 8 in its low 4 bits.
__device__ __forceinline__ uint32_t pack8_int4(const float (&p)[8]) {
  uint32_t acc = __float_as_uint(__fadd_rn(p[7], kMagicLo));
#pragma unroll
  for (int c = 6; c >= 0; --c) acc = (acc << 4) + __float_as_uint(__fadd_rn(p[c], kMagicLo));
  return (acc - kPackBias) ^ 0x88888888u;
}

// Asymmetric form: p already clamped to [-z, 15 - z]; the nibble to store is that of q - 8 with
// q = rne(p) + z.  The addend must be EVEN, or a tie p = n + 1/2 would be broken by the parity of the sum
// instead of that of n: magic = 1.5 * 2^23 + 16 + (z - z % 2) puts rne(p) + z - z % 2 + 16 (15..31) into
// the low bits; the 16s and the constant pattern bits leave with the bias, z % 2 is added to all eight
// nibbles at once (no nibble exceeds 31 - 16 = 15), and the final XOR turns q into q - 8.
__device__ __forceinline__ uint32_t pack8_uint4(const float (&p)[8], float z) {
  const float zodd = z - 2.0f * floorf(0.5f * z);
  const float magic = __fadd_rn(12582928.0f, z - zodd);  // 1.5 * 2^23 + 16 + even part of z
  uint32_t acc = __float_as_uint(__fadd_rn(p[7], magic));
#pragma unroll
  for (int c = 6; c >= 0; --c) acc = (acc << 4) + __float_as_uint(__fadd_rn(p[c], magic));
  return ((acc - (kPackBias + 0x11111110u)) + (zodd != 0.0f ? 0x11111111u : 0u)) ^ 0x88888888u;
}

// ---- codes straight to the FP6 GEMMs' operand layout (stamp_gemm6.hip; a thread owns 8 channels = 48 bits, the four
// threads of a quad one 24-byte fragment of 32 channels) ----

// byte offset, from its row's place on, of the 8 bytes that this thread stores for a row of half 0: thread t of a quad
// stores bytes 8 t .. 8 t + 7 of the fragment (t = 3 stores nothing); c = the thread's first channel
__device__ __forceinline__ uint32_t off48(int c, uint32_t kt_bytes) {
  const int t = (c >> 3) & 3;
  return chan_off6((uint32_t)c, kt_bytes) + (uint32_t)((t >> 1) * kPart + (t & 1) * 8);
}

// the quad's 4 x 48 bits -> 24 bytes (half: row_half6 of the row, hi_half6 of an 8-bit one); every lane of the quad has to call this
__device__ __forceinline__ void store48(uint8_t* dst, bool half, uint32_t w0, uint32_t w1, int c, bool active) {
  const uint32_t n0 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w0, 0xF9, 0xF, 0xF, false);  // quad_perm [1,2,3,3]
  const uint32_t n1 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w1, 0xF9, 0xF, 0xF, false);
  const uint32_t d1 = w1 | (n0 << 16), d2 = (n0 >> 16) | (n1 << 16);  // w0, d1, d2: 96 bits from this thread's first one on
  const int t = (c >> 3) & 3;
  const uint32_t a = t == 2 ? d1 : __builtin_amdgcn_alignbit(d1, w0, 16 * t);
  const uint32_t b = t == 2 ? d2 : __builtin_amdgcn_alignbit(d2, d1, 16 * t);
  // half 1 starts at byte 24 of the lane's 48
  if (active && t != 3) *reinterpret_cast<u2v*>(dst + (half ? (t == 1 ? 2 * kPart - 8 : kPart + 8) : 0)) = u2v{a, b};
}

constexpr int gb_of(int rows_log) { return rows_log < 2 ? 2 : rows_log > 6 ? 6 : rows_log; }
// row m of the 4-bit operand: byte offset of its place in K step 0
__device__ __forceinline__ size_t a6_row(size_t m, int KT, int gb) {
  return (m >> 8) * (size_t)KT * kStageA6 + row_off6((uint32_t)m & 255, gb);
}

// an 8-bit row: codes 16 h + l to the operand of the kernel for few rows (stamp_hi6.h), row m of it
typedef StampHiOut Hi6Out;
// K step stride of that operand, and every place of row m: store(its h fragments' lane in K step 0, their half, where the l ones
// follow, their half)
__device__ __forceinline__ uint32_t hi_step_bytes(const Hi6Out& o) { return o.ht.on ? (uint32_t)kBlock6 : (uint32_t)(2 * o.np * kBlock6); }
template <typename Store>
__device__ __forceinline__ void hi_rows(const Hi6Out& o, int m, int KT, Store store) {
  if (o.ht.on) {
    const int b = m / o.seq;
    int tile, ntiles, place;
    stamp_hi_places(o.ht, b, m - b * o.seq, &tile, &ntiles, &place);
    for (int i = 0; i < ntiles; ++i) store(o.p + (size_t)(tile + i) * KT * kBlock6 + place * 16, false, 0, true);
  } else {
    const int gr = 32 * o.np, grp = m / gr, r = m - grp * gr;
    store(o.p + (size_t)grp * KT * (2 * o.np * kBlock6) + (r >> 5) * (2 * kBlock6) + row_lane6(r & 31), hi_half6(r), kBlock6, hi_half6(r));
  }
}
__device__ __forceinline__ void store_hi48(const Hi6Out& o, int m, int KT, const int (&q)[8], int c, bool active) {
  uint64_t h = 0, l = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int hv = (q[i] + 8) >> 4, lv = q[i] - 16 * hv;
    h |= (uint64_t)((uint32_t)abs(hv) | ((uint32_t)(hv >> 31) & 32u)) << (6 * i);
    l |= (uint64_t)((uint32_t)abs(lv) | ((uint32_t)(lv >> 31) & 32u)) << (6 * i);
  }
  const uint32_t off = off48(c, hi_step_bytes(o));
  hi_rows(o, m, KT, [&](uint8_t* dst, bool hh, int lo, bool lh) {
    store48(dst + off, hh, (uint32_t)h, (uint32_t)(h >> 32), c, active);
    store48(dst + off + lo, lh, (uint32_t)l, (uint32_t)(l >> 32), c, active);
  });
}

// max over the 8 values of v and of -v, as order keys
__device__ __forceinline__ void row_posneg_bits(const float (&v)[8], uint32_t& pos, uint32_t& neg) {
  float mx = fmaxf(fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])), fmaxf(fmaxf(v[4], v[5]), fmaxf(v[6], v[7])));
  float mn = fminf(fminf(fminf(v[0], v[1]), fminf(v[2], v[3])), fminf(fminf(v[4], v[5]), fminf(v[6], v[7])));
  pos = fkey(mx);
  neg = fkey(-mn);
}

// range, scale, reciprocal and offset of one token from hi = max T and nlo = max -T, qmax = 2^b - 1
__device__ __forceinline__ void asym_params(float hi, float nlo, float qmax, float& scale, float& inv, float& z) {
  float range = __fadd_rn(hi, nlo);
  if (range == 0.0f) range = fabsf(hi);  // max = min: the token is reproduced through range = |value|
  scale = 0.0f;
  inv = 0.0f;
  if (range > 0.0f) {
    scale = __fdiv_rn(range, qmax);
    inv = __fdiv_rn(qmax, range);
  }
  z = rintf(__fmul_rn(nlo, inv));
}

__device__ __forceinline__ void load8(const void* X, size_t elem_off, bool bf16, bool active, float (&v)[8]) {
  if (!active) {
#pragma unroll
    for (int c = 0; c < 8; ++c) v[c] = 0.0f;
    return;
  }
  if (bf16) {
    const uint4 w = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(X) + elem_off);
    v[0] = bf16lo(w.x); v[1] = bf16hi(w.x); v[2] = bf16lo(w.y); v[3] = bf16hi(w.y);
    v[4] = bf16lo(w.z); v[5] = bf16hi(w.z); v[6] = bf16lo(w.w); v[7] = bf16hi(w.w);
  } else {
    const float4* p = reinterpret_cast<const float4*>(reinterpret_cast<const float*>(X) + elem_off);
    const float4 a = p[0], b = p[1];
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  }
}

constexpr int trailing_ones(int x) { int n = 0; while (x & 1) { ++n; x >>= 1; } return n; }
constexpr int cmin(int a, int b) { return a < b ? a : b; }

// Shared tail of one streaming step: NR finished rows (unnormalised values rowv[r][0..7], level
// and in-block position given per row) are reduced over the workgroup, scaled, rounded, packed and
// stored.  `step` numbers the steps of this workgroup (rotating LDS buffers).
struct RowMeta { int level; int e; int pos; };  // e: where the row goes (block position, or slot), pos: block position
constexpr int kMaxRows = 18;  // most rows finished by one streaming step (2-D: 12 + 3 + 3)
constexpr int kPartWords = 2 * kMaxRows * 16;  // per-wave partial maxima of one step: [2 signs][row][wave]

// Channel split.  A workgroup covers at most 1024 (1-D) / 512 (2-D) threads x 8 channels; wider layers
// are split over blockIdx.z and run in two passes, because a row's range spans all channels:
//   PASS 1  transform, reduce each row over the workgroup's channels, write the partial maxima
//           gpart[sign][split][B*s] (no codes);
//   PASS 2  transform again, take each row's maximum over the splits from LDS (s_amax[sign][e], filled
//           from gpart before the first step), quantize and store.
//   PASS 0  is the single-pass kernel (one workgroup sees all channels).
struct SplitArgs {
  uint32_t* gpart;     // partial row maxima (bit patterns), PASS 1 writes / PASS 2 reads
  size_t part_rows;    // B * s
  int nsplit;
  int c_split;         // channels per split (a multiple of 8)
  int8_t* q_hi;        // non-null: the plan has no top levels (L = 0), so the block sum is itself a finished
  int khi;             // coefficient and the bottom kernel quantizes it (8 bits for blocks < khi, else 4)
  Hi6Out hi6;          // OUT6: the 8-bit ones go there instead, row b * khi + slot
};
constexpr int kMaxBlockRows = 128;

// Blocks of a 1-D Haar transform of any length (StampRag): butterflies (x0 +- x1) / sqrt 2, a node without partner carried
// up unchanged, rows in STaMP order (RowMeta::e is the slot, < 0: no such coefficient).
struct RagArgs {
  StampRag q;
  int j, m;      // block, its tokens
  int Kpad;
  int tile_row;  // OUT6: the block's first row in its 256-row tile
};

// ASYM: the asymmetric form of the quantizer; zeros_off = distance (in floats) from a row's scale to its offset z.
// RAG: q_lo_blk is the whole buffer, row0 the sequence's first row, scales_blk its first scale, m_kpad the row pitch.
// OUT6: 4-bit codes as FP6 operand: q_lo_blk = K step 0 of the block's 256-row tile, row0 = the block's first row in the tile.
template <int NR, bool IS2D, bool ASYM, int PASS, bool RAG = false, bool OUT6 = false, typename MetaFn>
__device__ __forceinline__ void flush_rows(float (&rowv)[NR][8], MetaFn meta, int step, uint32_t (*s_max)[kPartWords],
                                           uint8_t* q_lo_blk /* row e=0 of the block, channel 0 (workgroup-uniform) */,
                                           uint32_t q_off /* this thread's byte offset inside a row */,
                                           float* scales_blk, size_t zeros_off, bool active, int tid,
                                           uint32_t* gpart_blk /* PASS 1: this split's partial maxima of the block's row e=0 */,
                                           size_t gpart_neg /* PASS 1: distance to the negative parts */,
                                           const uint32_t* s_amax /* PASS 2: [2][kMaxBlockRows] */, bool write_scales,
                                           size_t row0 = 0, int Kpad = 0, int nwaves = 0 /* waves that share a row, 0: the workgroup's */,
                                           int gb = 2 /* OUT6: row_off6 */) {
  // Values derived from the thread index are recomputed in every step from an opaque copy: cheap, and it
  // keeps them from being carried (and spilled: a scratch reload waits for ALL outstanding memory
  // operations, the asynchronous loads of the next batches included) across the whole unrolled kernel.
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wave = tid >> 6;
  // [row][wave] partial maxima, double buffered; asymmetric: a second array for the negative parts
  uint32_t* part = &s_max[0][0] + (step & 1) * kPartWords;
  uint32_t* part_neg = part + kMaxRows * 16;
  if constexpr (PASS != 2) {
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    if constexpr (ASYM) {
      uint32_t pos, neg;
      row_posneg_bits(rowv[r], pos, neg);
      if (!active) pos = neg = 0u;  // lanes beyond the last channel hold zeros, which are not part of the token
      pos = wave_max_u32(pos);
      neg = wave_max_u32(neg);
      if (lane == 0) { part[r * 16 + wave] = pos; part_neg[r * 16 + wave] = neg; }
    } else {
      const uint32_t m = wave_max_u32(row_absmax_bits(rowv[r]));
      if (lane == 0) part[r * 16 + wave] = m;
    }
  }
  // Workgroup barrier that waits for this wave's LDS traffic only: __syncthreads() would also wait for
  // the global -> LDS loads of the next batch, which are meant to stay in flight across it.
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  }
  // lane r prepares row r: a = fl(absmaxU * norm); scale = a / 7; inv = 7 / a
  // (asymmetric: hi = fl(max t * norm), nlo = fl(max -t * norm), then asym_params with qmax = 15)
  float mul_lane = 0.0f;
  [[maybe_unused]] float z_lane = 0.0f;
  {
    const int r = lane < NR ? lane : 0;
    const RowMeta rm = meta(r);
    const int nw = nwaves != 0 ? nwaves : (int)(blockDim.x >> 6);
    // The partial maxima are read by hand-written LDS reads: the compiler cannot tell this array from the
    // staging buffer that the asynchronous global -> LDS loads of the NEXT batches are writing, and would
    // make every ordinary LDS read here wait for all of them (vmcnt(0)), i.e. serialise memory and compute.
    auto reduce_waves = [&](const uint32_t* arr) {
      if constexpr (PASS == 2) {
        // the row's maximum over all channels, reduced before the first step
        const uint32_t adr1 = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint32_t*)(
            s_amax + (arr == part ? 0 : kMaxBlockRows) + rm.e);
        uint32_t bits;
        asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(bits) : "v"(adr1) : "memory");
        return bits;
      }
      const uint32_t adr = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint32_t*)(arr + r * 16);
      u4 v0, v1, v2, v3;
      asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:16\n\tds_read_b128 %2, %4 offset:32\n\t"
                   "ds_read_b128 %3, %4 offset:48\n\ts_waitcnt lgkmcnt(0)"
                   : "=&v"(v0), "=&v"(v1), "=&v"(v2), "=&v"(v3)
                   : "v"(adr)
                   : "memory");
      const u4 vv[4] = {v0, v1, v2, v3};
      uint32_t mbits = 0u;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (4 * q + 0 < nw) mbits = max(mbits, vv[q].x);
        if (4 * q + 1 < nw) mbits = max(mbits, vv[q].y);
        if (4 * q + 2 < nw) mbits = max(mbits, vv[q].z);
        if (4 * q + 3 < nw) mbits = max(mbits, vv[q].w);
      }
      return mbits;
    };
    if constexpr (PASS == 1) {
      const uint32_t mpos = reduce_waves(part);
      if (tid < NR) gpart_blk[rm.e] = mpos;
      if constexpr (ASYM) {
        const uint32_t mneg = reduce_waves(part_neg);
        if (tid < NR) gpart_blk[gpart_neg + rm.e] = mneg;
      }
      return;
    }
    const float nrm = IS2D ? ldexpf(1.0f, -rm.level) : haar_norm(rm.level);
    float scale = 0.0f, inv = 0.0f;
    if constexpr (ASYM) {
      const float hi = __fmul_rn(fkey_inv(reduce_waves(part)), nrm), nlo = __fmul_rn(fkey_inv(reduce_waves(part_neg)), nrm);
      asym_params(hi, nlo, 15.0f, scale, inv, z_lane);
      if (tid < NR && write_scales && (!RAG || rm.e >= 0)) scales_blk[zeros_off + rm.e] = z_lane;
    } else {
      const float a = __fmul_rn(__uint_as_float(reduce_waves(part)), nrm);
      if (a > 0.0f) {
        scale = __fdiv_rn(a, 7.0f);
        inv = __fdiv_rn(7.0f, a);
      }
    }
    // even 1-D levels and all 2-D levels have a power-of-two norm: fold it into the multiplier
    const bool fold = IS2D || ((rm.level & 1) == 0);
    mul_lane = fold ? __fmul_rn(inv, nrm) : inv;
    if (tid < NR && write_scales && (!RAG || rm.e >= 0)) scales_blk[rm.e] = scale;
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const RowMeta rm = meta(r);  // r is a compile-time constant here
    const float mul = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, mul_lane), r));
    float p[8];
    const bool fold = IS2D || ((rm.level & 1) == 0);
    if (fold) {
#pragma unroll
      for (int c = 0; c < 8; ++c) p[c] = __fmul_rn(rowv[r][c], mul);
    } else {
      const float nrm = haar_norm(rm.level);
#pragma unroll
      for (int c = 0; c < 8; ++c) p[c] = __fmul_rn(__fmul_rn(rowv[r][c], nrm), mul);
    }
    uint32_t w;
    if constexpr (ASYM) {
      const float z = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, z_lane), r));
      const float lo = -z, hi = 15.0f - z;  // clamp before rounding = clamp after it (integer bounds)
#pragma unroll
      for (int c = 0; c < 8; ++c) p[c] = __builtin_amdgcn_fmed3f(p[c], lo, hi);
      w = pack8_uint4(p, z);
    } else {
      w = pack8_int4(p);
    }
    if constexpr (OUT6) {
      uint32_t w0, w1;
      nib8_to_48(w, w0, w1);
      const uint32_t m = (uint32_t)row0 + (uint32_t)rm.pos;
      store48(q_lo_blk + row_off6(m, gb) + q_off, row_half6(m, gb), w0, w1, tid * 8, active && (!RAG || rm.e >= 0));
    } else if constexpr (RAG) {
      if (active && rm.e >= 0) *reinterpret_cast<uint32_t*>(q_lo_blk + stamp_qlo_offset(row0 + rm.e, 0, Kpad) + q_off) = w;
    } else {
      if (active) *reinterpret_cast<uint32_t*>(q_lo_blk + rm.e * 64 + q_off) = w;  // tiled layout: 64 bytes per row and K step
    }
  }
}

// Plans without top levels: the block sum, times the norm of the blocks' level, is STaMP slot j.  The whole
// workgroup reduces its range over the channels and quantizes it like any other top row: 8 bits for the first
// khi slots, 4-bit codes held as int8 beyond.  Called after the last streaming step (no loads in flight).
// The 4-bit ones also go, packed like every other 4-bit row, to the block's row 0 of q_lo (q_lo_row: this thread's
// word of it), which no other coefficient uses: the 4-bit rows' GEMM can then take the block sum from its own rows.
// RAG: 4-bit rows have no place in q_hi.
// OUT6: q_lo_row is this thread's place in the FP6 operand, the 8-bit rows go to hi6 (row hi_row).
// Channel split: row 0 of a block's maxima is free (no bottom coefficient has position 0) and holds the block sum's:
// PASS 1 leaves its part in part_max[0] and [part_neg], PASS 2 reads the whole from s_amax[0] and [kMaxBlockRows].
template <bool IS2D, bool ASYM, bool RAG = false, bool OUT6 = false, int PASS = 0>
__device__ __forceinline__ void finish_top_row(const float (&top)[8], int level, uint32_t* part /* >= 32 words, free */,
                                               int8_t* q_hi_row, uint8_t* q_lo_row, float* scale_out, size_t zeros_off,
                                               bool row8, bool active, int tid, Hi6Out hi6 = Hi6Out{}, int hi_row = 0, int KT = 0, int c0 = 0,
                                               uint32_t* part_max = nullptr, size_t part_neg = 0, const uint32_t* s_amax = nullptr,
                                               bool half6 = false /* OUT6: row_half6 of the row */) {
  const int lane = tid & 63, wave = tid >> 6, nw = (int)(blockDim.x >> 6);
  const float nrm = IS2D ? ldexpf(1.0f, -level) : haar_norm(level);
  float t[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) t[c] = __fmul_rn(top[c], nrm);
  uint32_t mp = 0u, mn = 0u;
  if constexpr (PASS == 2) {
    mp = s_amax[0];
    mn = s_amax[kMaxBlockRows];
  } else {
    uint32_t pos = 0u, neg = 0u;
    if constexpr (PASS == 1) {  // maxima of the patterns, as the top part's kernel takes them: a NaN is the largest
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        pos = max(pos, ASYM ? fkey(t[c]) : absbits(t[c]));
        if constexpr (ASYM) neg = max(neg, fkey(-t[c]));
      }
      if (ASYM && !active) pos = neg = 0u;
    } else if constexpr (ASYM) {
      row_posneg_bits(t, pos, neg);
      if (!active) pos = neg = 0u;
    } else {
      pos = row_absmax_bits(t);
    }
    pos = wave_max_u32(pos);
    neg = wave_max_u32(neg);
    if (lane == 0) { part[wave] = pos; part[16 + wave] = neg; }
    __syncthreads();
    for (int i = 0; i < nw; ++i) { mp = max(mp, part[i]); mn = max(mn, part[16 + i]); }
    if constexpr (PASS == 1) {
      if (tid == 0) {
        part_max[0] = mp;
        if constexpr (ASYM) part_max[part_neg] = mn;
      }
      return;
    }
  }
  const float qmax = ASYM ? (row8 ? 255.0f : 15.0f) : (row8 ? 127.0f : 7.0f);
  float scale = 0.0f, inv = 0.0f, z = 0.0f;
  if constexpr (ASYM) {
    asym_params(fkey_inv(mp), fkey_inv(mn), qmax, scale, inv, z);
  } else {
    const float a = __uint_as_float(mp);
    if (a > 0.0f) {
      scale = __fdiv_rn(a, qmax);
      inv = __fdiv_rn(qmax, a);
    }
  }
  if (tid == 0 && (PASS == 0 || blockIdx.z == 0)) {
    scale_out[0] = scale;
    if constexpr (ASYM) scale_out[zeros_off] = z;
  }
  const float qlo = ASYM ? 0.0f : -qmax, qhi = qmax, shift = ASYM ? (row8 ? 128.0f : 8.0f) : 0.0f;
  uint32_t w[2] = {0u, 0u}, w4 = 0u;
  int qi[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    float q = __fadd_rn(rintf(__fmul_rn(t[i], inv)), z);
    q = fminf(fmaxf(q, qlo), qhi) - shift;
    qi[i] = (int)q;
    w[i >> 2] |= ((uint32_t)((int)q) & 0xFFu) << (8 * (i & 3));
    w4 |= ((uint32_t)((int)q) & 0xFu) << (4 * i);
  }
  if constexpr (OUT6) {
    if (row8) {
      store_hi48(hi6, hi_row, KT, qi, c0, active);
    } else {
      uint32_t w0, w1;
      nib8_to_48(w4, w0, w1);
      store48(q_lo_row, half6, w0, w1, c0, active);
    }
    return;
  }
  if (active) {
    if (!RAG || row8) *reinterpret_cast<uint2*>(q_hi_row) = make_uint2(w[0], w[1]);
    if (!row8) *reinterpret_cast<uint32_t*>(q_lo_row) = w4;
  }
}

// ------------------------------------------------------------------------------------------
// 1-D bottom kernel
// ------------------------------------------------------------------------------------------
// level and in-block position of row r finished by streaming step IT (4 tokens) of a 1-D block of
// 2^RLOG tokens: rows 0,1 = level-1 differences, row 2 = level 2, row r >= 3 = level r (carry chain)
template <int RLOG, int IT>
__device__ __forceinline__ RowMeta meta1d(int r) {
  constexpr int R = 1 << RLOG;
  RowMeta m;
  if (r < 2) { m.level = 1; m.e = (R >> 1) + 2 * IT + r; }
  else if (r == 2) { m.level = 2; m.e = (R >> 2) + IT; }
  else { m.level = r; m.e = (R >> r) + (IT >> (r - 2)); }
  m.pos = m.e;
  return m;
}

// The block's token rows are streamed through an LDS staging buffer by asynchronous global -> LDS
// loads (no registers are held while they are in flight): the buffer holds two batches of 4 token
// rows; batch IT+2 is requested as soon as batch IT has been read out of its half into registers,
// so two batches are always in flight or ready.  Every lane reads back exactly the 16-byte chunks it
// requested, so no barrier guards the buffer, only this wave's own vmcnt.
// Layout of one half: chunk (t, h) of thread tid at ((t * CPR + h) * nthreads + tid) * 16, CPR =
// 16-byte chunks per thread and row (1 for bf16, 2 for fp32).
template <bool BF16>
__device__ __forceinline__ void request_batch(const uint8_t* X_row /* row 0 of the batch, channel 0 (workgroup-uniform) */,
                                              uint32_t x_off /* byte offset of this thread's 8 channels in a row */,
                                              size_t row_bytes, uint8_t* half, int nthreads, int wave, int last = 3 /* rows beyond: row `last` again */) {
  constexpr int CPR = BF16 ? 1 : 2;
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int h = 0; h < CPR; ++h)
      __builtin_amdgcn_global_load_lds(
          (const void __attribute__((address_space(1)))*)(X_row + (ptrdiff_t)min(t, last) * (ptrdiff_t)row_bytes + 16 * h + x_off),
          (void __attribute__((address_space(3)))*)(half + ((t * CPR + h) * nthreads + wave * 64) * 16), 16, 0, 0);
}

template <int RLOG, int L, int IDX, int SLOT, bool RAG, int NP, int MAXR>
__device__ __forceinline__ void chain1d(float (&cur)[8], float (&pend)[NP][8], float (&rowv)[MAXR][8], float (&top)[8], int m) {
  if constexpr (L == RLOG) {
#pragma unroll
    for (int c = 0; c < 8; ++c) top[c] = cur[c];
  } else if constexpr ((IDX & 1) != 0) {
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      float a = __fadd_rn(pend[L - 2][c], cur[c]);
      rowv[SLOT][c] = __fsub_rn(pend[L - 2][c], cur[c]);
      if constexpr (RAG) {
        a = (IDX << L) < m ? __fmul_rn(a, kInvSqrt2) : pend[L - 2][c];
        rowv[SLOT][c] = __fmul_rn(rowv[SLOT][c], kInvSqrt2);
      }
      cur[c] = a;
    }
    chain1d<RLOG, L + 1, (IDX >> 1), SLOT + 1, RAG, NP, MAXR>(cur, pend, rowv, top, m);
  } else {
#pragma unroll
    for (int c = 0; c < 8; ++c) pend[L - 2][c] = cur[c];
  }
}

template <int RLOG, bool BF16, bool ASYM, int PASS, bool RAG, bool OUT6, int IT, int NP>
__device__ __forceinline__ void step1d(const uint8_t* X_blk, uint32_t x_off, size_t row_bytes, uint8_t* stage, int nthreads,
                                       bool active, int tid, float (&pend)[NP][8], float (&top)[8],
                                       uint32_t (*s_max)[kPartWords], uint8_t* q_lo_blk, uint32_t q_off, float* scales_blk,
                                       size_t zeros_off, uint32_t* gpart_blk, size_t gpart_neg, const uint32_t* s_amax,
                                       bool write_scales, const RagArgs& rg, size_t row0) {
  constexpr int R = 1 << RLOG;
  constexpr int NIT = R / 4;
  constexpr int CH = cmin(trailing_ones(IT), RLOG - 2);
  constexpr int NR = 3 + CH;
  constexpr int CPR = BF16 ? 1 : 2;
  uint8_t* half = stage + (IT & 1) * (4 * CPR * nthreads * 16);
  // Wait until this wave's loads of batch IT have landed: everything requested after it (batch IT+1:
  // 4 * CPR loads) may stay in flight.  Stores issued since also count, so this can only over-wait.
  asm volatile("" ::: "memory");
  if constexpr (IT + 1 < NIT) __builtin_amdgcn_s_waitcnt(0x0F70 | (4 * CPR));  // vmcnt(4 * CPR)
  else __builtin_amdgcn_s_waitcnt(0x0F70);                                      // vmcnt(0)
  asm volatile("" ::: "memory");
  u4 raw[4][CPR];
  {
    int tid_l = tid;
    asm volatile("" : "+v"(tid_l));  // see flush_rows: recomputed, not carried
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int h = 0; h < CPR; ++h)
        raw[t][h] = *reinterpret_cast<const u4*>(half + ((t * CPR + h) * nthreads + tid_l) * 16);
  }
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the half has been read before it is requested again
  asm volatile("" ::: "memory");
  if constexpr (IT + 2 < NIT)
    request_batch<BF16>(X_blk + (size_t)(4 * (IT + 2)) * row_bytes, x_off, row_bytes, half, nthreads, tid >> 6,
                        RAG ? rg.m - 1 - 4 * (IT + 2) : 3);

  float rowv[NR][8];
  float a1[2][8];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    float x0[8], x1[8];
    const int t = 2 * u;
    if constexpr (BF16) {
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        x0[2 * w] = bf16lo(raw[t][0][w]);
        x0[2 * w + 1] = bf16hi(raw[t][0][w]);
        x1[2 * w] = bf16lo(raw[t + 1][0][w]);
        x1[2 * w + 1] = bf16hi(raw[t + 1][0][w]);
      }
    } else {
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        x0[w] = __uint_as_float(raw[t][0][w]);
        x0[4 + w] = __uint_as_float(raw[t][CPR - 1][w]);
        x1[w] = __uint_as_float(raw[t + 1][0][w]);
        x1[4 + w] = __uint_as_float(raw[t + 1][CPR - 1][w]);
      }
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      a1[u][c] = __fadd_rn(x0[c], x1[c]);
      rowv[u][c] = __fsub_rn(x0[c], x1[c]);
      if constexpr (RAG) {
        a1[u][c] = 4 * IT + t + 1 < rg.m ? __fmul_rn(a1[u][c], kInvSqrt2) : x0[c];
        rowv[u][c] = __fmul_rn(rowv[u][c], kInvSqrt2);
      }
    }
  }
  float cur[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    cur[c] = __fadd_rn(a1[0][c], a1[1][c]);
    rowv[2][c] = __fsub_rn(a1[0][c], a1[1][c]);
    if constexpr (RAG) {
      cur[c] = 4 * IT + 2 < rg.m ? __fmul_rn(cur[c], kInvSqrt2) : a1[0][c];
      rowv[2][c] = __fmul_rn(rowv[2][c], kInvSqrt2);
    }
  }
  chain1d<RLOG, 2, IT, 3, RAG, NP, NR>(cur, pend, rowv, top, rg.m);
  if constexpr (RAG) {
    auto meta = [&rg](int r) -> RowMeta { 
      const int e = meta1d<RLOG, IT>(r).e;
      return RowMeta{0, stamp_rag_slot(rg.q, rg.j, e), e};
    };
    flush_rows<NR, false, ASYM, PASS, true, OUT6>(rowv, meta, IT, s_max, q_lo_blk, q_off, scales_blk, zeros_off, active, tid, gpart_blk,
                                            gpart_neg, s_amax, write_scales, OUT6 ? (size_t)rg.tile_row : row0, rg.Kpad, 0, gb_of(RLOG));
  } else {
    auto meta = [](int r) -> RowMeta { return meta1d<RLOG, IT>(r); };
    flush_rows<NR, false, ASYM, PASS, false, OUT6>(rowv, meta, IT, s_max, q_lo_blk, q_off, scales_blk, zeros_off, active, tid, gpart_blk,
                                                   gpart_neg, s_amax, write_scales, row0, 0, 0, gb_of(RLOG));
  }
}

template <int RLOG, bool BF16, bool ASYM, int PASS, bool RAG = false, bool OUT6 = false, int NP, int... ITS>
__device__ __forceinline__ void run1d(std::integer_sequence<int, ITS...>, const uint8_t* X_blk, uint32_t x_off,
                                      size_t row_bytes, uint8_t* stage, int nthreads, bool active, int tid,
                                      float (&pend)[NP][8], float (&top)[8], uint32_t (*s_max)[kPartWords],
                                      uint8_t* q_lo_blk, uint32_t q_off, float* scales_blk, size_t zeros_off,
                                      uint32_t* gpart_blk, size_t gpart_neg, const uint32_t* s_amax, bool write_scales,
                                      const RagArgs& rg = RagArgs{}, size_t seq_row0 = 0) {
  (step1d<RLOG, BF16, ASYM, PASS, RAG, OUT6, ITS, NP>(X_blk, x_off, row_bytes, stage, nthreads, active, tid, pend, top, s_max, q_lo_blk,
                                                q_off, scales_blk, zeros_off, gpart_blk, gpart_neg, s_amax, write_scales, rg,
                                                seq_row0), ...);
}

// PASS 2: every row's maximum over the splits -> s_amax[sign][e] (before the first step; ordinary loads)
template <bool ASYM>
__device__ __forceinline__ void gather_row_maxima(const SplitArgs& sp, size_t row0, int R, int tid, uint32_t* s_amax) {
  if (tid < R) {
    uint32_t mpos = 0u, mneg = 0u;
    for (int q = 0; q < sp.nsplit; ++q) {
      mpos = max(mpos, sp.gpart[(size_t)q * sp.part_rows + row0 + tid]);
      if constexpr (ASYM) mneg = max(mneg, sp.gpart[((size_t)sp.nsplit + q) * sp.part_rows + row0 + tid]);
    }
    s_amax[tid] = mpos;
    s_amax[kMaxBlockRows + tid] = mneg;
  }
  __syncthreads();
}

template <int RLOG, bool BF16, bool ASYM, int PASS, bool OUT6>
__global__ __launch_bounds__(1024) void k_bottom1d(const void* __restrict__ X, uint8_t* __restrict__ q_lo,
                                                   float* __restrict__ scales, float* __restrict__ abot, int s, int d,
                                                   int k, int Kpad, size_t zeros_off, SplitArgs sp) {
  constexpr int R = 1 << RLOG;
  constexpr int NP = RLOG > 2 ? RLOG - 2 : 1;
  constexpr int CPR = BF16 ? 1 : 2;
  extern __shared__ __attribute__((aligned(16))) uint8_t stage[];  // 2 halves x 4 rows x nthreads x (16 | 32) bytes
  __shared__ __attribute__((aligned(16))) uint32_t s_max[2][kPartWords];
  __shared__ uint32_t s_amax[PASS == 2 ? 2 * kMaxBlockRows : 1];
  const int j = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
  const int nthreads = blockDim.x;
  // channels of this workgroup: [c_lo, c_hi)
  const int c_lo = (PASS == 0) ? 0 : (int)blockIdx.z * sp.c_split;
  const int c_hi = (PASS == 0) ? d : min(d, c_lo + sp.c_split);
  const int c0 = c_lo + tid * 8;
  const bool active = c0 < c_hi;
  const size_t esz = BF16 ? 2 : 4;
  const size_t row0 = (size_t)b * s + (size_t)j * R;
  if constexpr (PASS == 2) gather_row_maxima<ASYM>(sp, row0, R, tid, s_amax);
  // threads beyond d_in / 8 (the workgroup is a whole number of waves) redo the last channel group:
  // duplicates cannot change a row maximum, and they store nothing
  // addresses = workgroup-uniform base + a 32-bit per-thread offset (keeps the per-thread state small)
  const uint8_t* X_blk = reinterpret_cast<const uint8_t*>(X) + row0 * d * esz;
  const uint32_t x_off = (uint32_t)(min(c0, c_hi - 8) * (int)esz);
  const uint32_t q_off = OUT6 ? off48(min(c0, c_hi - 8), kStageA6) : (uint32_t)(stamp_qlo_offset(0, min(c0, c_hi - 8), Kpad));
  // first row of the block in the output: its place in q_lo, or the FP6 tile (a block does not leave its tile)
  uint8_t* const q_blk = OUT6 ? q_lo + (row0 >> 8) * (size_t)(Kpad >> 7) * kStageA6 : q_lo + stamp_qlo_offset(row0, 0, Kpad);
  const size_t row_bytes = (size_t)d * esz;
  request_batch<BF16>(X_blk, x_off, row_bytes, stage, nthreads, tid >> 6);
  if (R > 4) request_batch<BF16>(X_blk + 4 * row_bytes, x_off, row_bytes, stage + 4 * CPR * nthreads * 16, nthreads, tid >> 6);
  float pend[NP][8];
  float top[8];
  uint32_t* gpart_blk = (PASS == 1) ? sp.gpart + (size_t)blockIdx.z * sp.part_rows + row0 : nullptr;
  run1d<RLOG, BF16, ASYM, PASS, false, OUT6>(std::make_integer_sequence<int, R / 4>{}, X_blk, x_off, row_bytes, stage, nthreads, active,
                                             tid, pend, top, s_max, q_blk, q_off, scales + row0, zeros_off, gpart_blk,
                                             (size_t)sp.nsplit * sp.part_rows, s_amax, PASS == 0 || blockIdx.z == 0, RagArgs{}, row0 & 255);
  if (sp.q_hi != nullptr) {
    // s_max[R/4 & 1] was last used two steps ago: every thread has passed a barrier since
    finish_top_row<false, ASYM, false, OUT6, PASS>(top, RLOG, &s_max[(R / 4) & 1][0], sp.q_hi + ((size_t)b * k + j) * d + c0,
                                                   (OUT6 ? q_lo + a6_row(row0, Kpad >> 7, gb_of(RLOG)) : q_blk) + q_off, scales + row0, zeros_off,
                                                   j < sp.khi, active, tid, sp.hi6, b * sp.khi + j, Kpad >> 7, c0, gpart_blk,
                                                   (size_t)sp.nsplit * sp.part_rows, s_amax, row_half6((uint32_t)row0, gb_of(RLOG)));
    return;
  }
  if (active && PASS != 1) {
    float4* o = reinterpret_cast<float4*>(abot + ((size_t)b * k + j) * d + c0);
    o[0] = make_float4(top[0], top[1], top[2], top[3]);
    o[1] = make_float4(top[4], top[5], top[6], top[7]);
  }
}

// The same for a 1-D Haar transform of any length, optionally with the first token left out: one workgroup per block
// (blockIdx.x < nb) of 2^RLOG tokens, one more for the token that was left out.  Codes and scales leave in STaMP order;
// X is read once and T never leaves the chip (levels as passes over fp32 buffers and a row quantizer, 2048 tokens x 4096
// channels, 3 levels: 19.5 + 8.6 us; this kernel 10.1).
template <int RLOG, bool BF16, bool ASYM, bool OUT6>
__global__ __launch_bounds__(1024) void k_bottom1d_rag(const void* __restrict__ X, int8_t* __restrict__ q_hi, uint8_t* __restrict__ q_lo,
                                                       float* __restrict__ scales, int s, int d, int khi, int Kpad, size_t zeros_off,
                                                       StampRag q, Hi6Out hi6) {
  constexpr int R = 1 << RLOG;
  constexpr int NP = RLOG > 2 ? RLOG - 2 : 1;
  constexpr int CPR = BF16 ? 1 : 2;
  extern __shared__ __attribute__((aligned(16))) uint8_t stage[];
  __shared__ __attribute__((aligned(16))) uint32_t s_max[2][kPartWords];
  const int j = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
  const int nthreads = blockDim.x;
  const int c0 = tid * 8;
  const bool active = c0 < d;
  const size_t esz = BF16 ? 2 : 4, row_bytes = (size_t)d * esz, seq0 = (size_t)b * s;
  const uint32_t x_off = (uint32_t)(min(c0, d - 8) * (int)esz);
  const uint32_t q_off = OUT6 ? off48(min(c0, d - 8), kStageA6) : (uint32_t)(stamp_qlo_offset(0, min(c0, d - 8), Kpad));
  const size_t brow = ((size_t)b * q.nb + j) * R;  // OUT6: rows in block order (the token left out has none: it is an 8-bit row)
  float top[8];
  int slot = 0;
  if (j == q.nb) {
    load8(X, seq0 * d + min(c0, d - 8), BF16, true, top);
  } else {
    const RagArgs rg = {q, j, j == q.nb - 1 ? q.mlast : R, Kpad, (int)(brow & 255)};
    const uint8_t* X_blk = reinterpret_cast<const uint8_t*>(X) + (seq0 + q.o + (size_t)j * R) * row_bytes;
    request_batch<BF16>(X_blk, x_off, row_bytes, stage, nthreads, tid >> 6, rg.m - 1);
    request_batch<BF16>(X_blk + 4 * row_bytes, x_off, row_bytes, stage + 4 * CPR * nthreads * 16, nthreads, tid >> 6, rg.m - 5);
    float pend[NP][8];
    uint8_t* const q_out = OUT6 ? q_lo + (brow >> 8) * (size_t)(Kpad >> 7) * kStageA6 : q_lo;
    run1d<RLOG, BF16, ASYM, 0, true, OUT6>(std::make_integer_sequence<int, R / 4>{}, X_blk, x_off, row_bytes, stage, nthreads, active, tid,
                                     pend, top, s_max, q_out, q_off, scales + seq0, zeros_off, nullptr, 0, nullptr, true, rg, seq0);
    slot = q.o + j;
  }
  finish_top_row<false, ASYM, true, OUT6>(top, 0, &s_max[(R / 4) & 1][0], q_hi + ((size_t)b * khi + slot) * d + c0,
                                          q_lo + (OUT6 ? a6_row(brow, Kpad >> 7, gb_of(RLOG)) : stamp_qlo_offset(seq0 + slot, 0, Kpad)) + q_off,
                                          scales + seq0 + slot, zeros_off, slot < khi, active, tid, hi6, b * khi + slot, Kpad >> 7, c0, nullptr, 0, nullptr,
                                          row_half6((uint32_t)brow, gb_of(RLOG)));
}

// ------------------------------------------------------------------------------------------
// 2-D bottom kernel: block of g x g tokens (g = 2^RLOG, RLOG in {2,3}), streamed in 4x4 sub-blocks
// ------------------------------------------------------------------------------------------
// 16 tokens from eoff0 on (4 x 4) -> 12 coefficients of level 1 and 3 of level 2 (rowv), their sum
template <bool BF16, int NR>
__device__ __forceinline__ void quad2d(const void* X, size_t eoff0, int gridW, int d, bool active, float (&rowv)[NR][8], float (&ll2)[8]) {
  float ll1[4][8];
  // all 16 tokens of the sub-block are requested before the first cell is computed (one memory latency per
  // sub-block instead of one per cell); the raw words give way to finished rows as the cells are consumed
  constexpr int WPT = BF16 ? 1 : 2;  // 16-byte words per token and thread
  uint4 raw[16][WPT];
#pragma unroll
  for (int tkn = 0; tkn < 16; ++tkn) {
    const int ci = tkn >> 2, q = tkn & 3;
    const int y = 2 * (ci >> 1) + (q >> 1), x = 2 * (ci & 1) + (q & 1);
    const size_t eoff = eoff0 + ((size_t)y * gridW + x) * d;
#pragma unroll
    for (int h = 0; h < WPT; ++h) {
      if (active) {
        raw[tkn][h] = BF16 ? *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(X) + eoff)
                           : *reinterpret_cast<const uint4*>(reinterpret_cast<const float*>(X) + eoff + 4 * h);
      } else {
        raw[tkn][h] = make_uint4(0u, 0u, 0u, 0u);
      }
    }
  }
#pragma unroll
  for (int ci = 0; ci < 4; ++ci) {
    float t[4][8];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint4 w0 = raw[4 * ci + q][0];
      if constexpr (BF16) {
        t[q][0] = bf16lo(w0.x); t[q][1] = bf16hi(w0.x); t[q][2] = bf16lo(w0.y); t[q][3] = bf16hi(w0.y);
        t[q][4] = bf16lo(w0.z); t[q][5] = bf16hi(w0.z); t[q][6] = bf16lo(w0.w); t[q][7] = bf16hi(w0.w);
      } else {
        const uint4 w1 = raw[4 * ci + q][WPT - 1];
        t[q][0] = __uint_as_float(w0.x); t[q][1] = __uint_as_float(w0.y); t[q][2] = __uint_as_float(w0.z);
        t[q][3] = __uint_as_float(w0.w); t[q][4] = __uint_as_float(w1.x); t[q][5] = __uint_as_float(w1.y);
        t[q][6] = __uint_as_float(w1.z); t[q][7] = __uint_as_float(w1.w);
      }
    }
    cell2d(t[0], t[1], t[2], t[3], ll1[ci], rowv[3 * ci + 0], rowv[3 * ci + 1], rowv[3 * ci + 2]);
  }
  cell2d(ll1[0], ll1[1], ll1[2], ll1[3], ll2, rowv[12], rowv[13], rowv[14]);
}

// level and in-block position of row r of sub-block (sby, sbx)
template <int RLOG>
__device__ __forceinline__ RowMeta meta2d(int r, int sby, int sbx) {
  constexpr int g = 1 << RLOG;
  RowMeta m;
  if (r < 12) {
    const int ci = r / 3, bd = r - 3 * ci;
    constexpr int g1 = g >> 1;
    m.level = 1;
    m.e = g1 * g1 * (1 + bd) + (2 * sby + (ci >> 1)) * g1 + (2 * sbx + (ci & 1));
  } else if (r < 15) {
    constexpr int g2 = g >> 2;
    m.level = 2;
    m.e = g2 * g2 * (1 + (r - 12)) + sby * g2 + sbx;
  } else {
    m.level = 3;
    m.e = 1 + (r - 15);
  }
  m.pos = m.e;
  return m;
}

template <int RLOG, bool BF16, bool ASYM, int PASS, int SB>
__device__ __forceinline__ void step2d(const void* X, size_t blk_elem_off, int gridW, int d, int c0, bool active, int tid,
                                       float (&pend)[4][8], float (&top)[8], uint32_t (*s_max)[kPartWords],
                                       uint8_t* q_lo_blk, uint32_t q_off, float* scales_blk, size_t zeros_off,
                                       uint32_t* gpart_blk, size_t gpart_neg, const uint32_t* s_amax, bool write_scales) {
  constexpr int g = 1 << RLOG;
  constexpr int sby = (g == 4) ? 0 : (SB >> 1), sbx = (g == 4) ? 0 : (SB & 1);
  constexpr bool LAST = (g == 8) && (SB == 3);
  constexpr int NR = LAST ? 18 : 15;
  float rowv[NR][8];
  float ll2[8];
  quad2d<BF16, NR>(X, blk_elem_off + ((size_t)(4 * sby) * gridW + 4 * sbx) * d, gridW, d, active, rowv, ll2);
  if constexpr (g == 4) {
#pragma unroll
    for (int c = 0; c < 8; ++c) top[c] = ll2[c];
  } else if constexpr (LAST) {
    cell2d(pend[0], pend[1], pend[2], ll2, top, rowv[15], rowv[16], rowv[17]);
  } else {
#pragma unroll
    for (int c = 0; c < 8; ++c) pend[SB][c] = ll2[c];
  }
  auto meta = [](int r) -> RowMeta { return meta2d<RLOG>(r, sby, sbx); };
  flush_rows<NR, true, ASYM, PASS>(rowv, meta, SB, s_max, q_lo_blk, q_off, scales_blk, zeros_off, active, tid, gpart_blk,
                                   gpart_neg, s_amax, write_scales);
}

template <int RLOG, bool BF16, bool ASYM, int PASS, int... SBS>
__device__ __forceinline__ void run2d(std::integer_sequence<int, SBS...>, const void* X, size_t blk_elem_off, int gridW,
                                      int d, int c0, bool active, int tid, float (&pend)[4][8], float (&top)[8],
                                      uint32_t (*s_max)[kPartWords], uint8_t* q_lo_blk, uint32_t q_off, float* scales_blk,
                                      size_t zeros_off, uint32_t* gpart_blk, size_t gpart_neg, const uint32_t* s_amax,
                                      bool write_scales) {
  (step2d<RLOG, BF16, ASYM, PASS, SBS>(X, blk_elem_off, gridW, d, c0, active, tid, pend, top, s_max, q_lo_blk, q_off,
                                       scales_blk, zeros_off, gpart_blk, gpart_neg, s_amax, write_scales), ...);
}

template <int RLOG, bool BF16, bool ASYM, int PASS>
__global__ __launch_bounds__(512) void k_bottom2d(const void* __restrict__ X, uint8_t* __restrict__ q_lo,
                                                  float* __restrict__ scales, float* __restrict__ abot, int s, int d, int G,
                                                  int gridW, int Kpad, size_t zeros_off, SplitArgs sp) {
  constexpr int g = 1 << RLOG;
  constexpr int R = g * g;
  __shared__ __attribute__((aligned(16))) uint32_t s_max[2][kPartWords];
  __shared__ uint32_t s_amax[PASS == 2 ? 2 * kMaxBlockRows : 1];
  const int j = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
  const int bi = j / G, bj = j - bi * G;
  const int c_lo = (PASS == 0) ? 0 : (int)blockIdx.z * sp.c_split;
  const int c_hi = (PASS == 0) ? d : min(d, c_lo + sp.c_split);
  const int c0 = c_lo + tid * 8;
  const bool active = c0 < c_hi;
  const int k = G * G;
  const size_t tok0 = (size_t)b * s + (size_t)(bi * g) * gridW + (size_t)bj * g;  // first token of the block
  const size_t prow0 = (size_t)b * s + (size_t)j * R;                              // first physical row of the block
  if constexpr (PASS == 2) gather_row_maxima<ASYM>(sp, prow0, R, tid, s_amax);
  float pend[4][8];
  float top[8];
  uint32_t* gpart_blk = (PASS == 1) ? sp.gpart + (size_t)blockIdx.z * sp.part_rows + prow0 : nullptr;
  uint8_t* const q_blk = q_lo + stamp_qlo_offset(prow0, 0, Kpad);
  const uint32_t q_off = (uint32_t)stamp_qlo_offset(0, c0, Kpad);
  run2d<RLOG, BF16, ASYM, PASS>(std::make_integer_sequence<int, (g == 4 ? 1 : 4)>{}, X, tok0 * d + c0, gridW, d, c0, active,
                                      tid, pend, top, s_max, q_blk, q_off, scales + prow0, zeros_off, gpart_blk,
                                      (size_t)sp.nsplit * sp.part_rows, s_amax, PASS == 0 || blockIdx.z == 0);
  if (sp.q_hi != nullptr) {
    constexpr int nsteps = (g == 4) ? 1 : 4;
    finish_top_row<true, ASYM, false, false, PASS>(top, RLOG, &s_max[nsteps & 1][0], sp.q_hi + ((size_t)b * k + j) * d + c0, q_blk + q_off,
                                                   scales + prow0, zeros_off, j < sp.khi, active, tid, Hi6Out{}, 0, 0, c0, gpart_blk,
                                                   (size_t)sp.nsplit * sp.part_rows, s_amax);
    return;
  }
  if (active && PASS != 1) {
    float4* o = reinterpret_cast<float4*>(abot + ((size_t)b * k + j) * d + c0);
    o[0] = make_float4(top[0], top[1], top[2], top[3]);
    o[1] = make_float4(top[4], top[5], top[6], top[7]);
  }
}

// 8 x 8 blocks of up to 1536 channels: the four 4 x 4 sub-blocks side by side, a group of waves each (nthr threads), their
// sums through LDS, the last level's four rows a group each.  A block's rows need all its channels, so there are no more
// workgroups than blocks: k_bottom2d, whose workgroup takes the sub-blocks one after another, left the CUs three waves each.
// Packed codes (FP6 operands: stamp_lanes2d.hip).  Bound by the instructions of the rounding and the packing on the CUs that have
// a block.  Layers, k_bottom2d against this
// one, microseconds: 2 x 4096 tokens 1152 -> 4608 72.4, 64.5; 512 -> 1152 39.5, 26.9; 4096 tokens 1536 -> 1536, 6 levels 58.9,
// 47.5; 6 x 4096 tokens (384 blocks) 1152 -> 1152 70.4, 68.7; 16 x 4096 tokens (1024 blocks) 149.7, 151.2.
template <bool BF16, bool ASYM>
__global__ __launch_bounds__(768) void k_bottom2d_quads(const void* __restrict__ X, uint8_t* __restrict__ q_lo, float* __restrict__ scales,
                                                         float* __restrict__ abot, int s, int d, int G, int gridW, int Kpad,
                                                         size_t zeros_off, SplitArgs sp) {
  __shared__ __attribute__((aligned(16))) uint32_t s_max[4][2][kPartWords];
  __shared__ uint32_t s_amax[2 * kMaxBlockRows];
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];  // [4][nthr][8] sums
  float* const s_sum = reinterpret_cast<float*>(smem);
  const int nthr = (int)blockDim.x >> 2, nw = nthr >> 6;
  const int j = blockIdx.x, b = blockIdx.y, qd = __builtin_amdgcn_readfirstlane((int)threadIdx.x / nthr), tid = (int)threadIdx.x - qd * nthr;
  const int by = j / G, bx = j - by * G, k = G * G, c0 = tid * 8, sby = qd >> 1, sbx = qd & 1;
  const bool active = c0 < d;
  const size_t tok0 = (size_t)b * s + (size_t)(by * 8 + 4 * sby) * gridW + bx * 8 + 4 * sbx, prow0 = (size_t)b * s + (size_t)j * 64;
  uint8_t* const q_blk = q_lo + stamp_qlo_offset(prow0, 0, Kpad);
  const uint32_t q_off = (uint32_t)stamp_qlo_offset(0, c0, Kpad);
  // two rows of cells after one another: 15 finished rows at once would not fit the registers of 12 waves
  {
    constexpr int WPT = BF16 ? 1 : 2;
    uint4 raw[2][8][WPT];
    const size_t eoff0 = tok0 * d + min(c0, d - 8);  // threads beyond d_in / 8 redo the last channels, see k_bottom1d
    auto request = [&](int h) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const size_t eoff = eoff0 + ((size_t)(2 * h + ((i >> 1) & 1)) * gridW + 2 * (i >> 2) + (i & 1)) * d;
#pragma unroll
        for (int w = 0; w < WPT; ++w)
          raw[h][i][w] = BF16 ? *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(X) + eoff)
                              : *reinterpret_cast<const uint4*>(reinterpret_cast<const float*>(X) + eoff + 4 * w);
      }
    };
    float ll1[4][8];
    auto cell = [&](int h, int x, float (&W)[8], float (&H)[8], float (&D)[8]) {
      float t[4][8];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint4 w0 = raw[h][4 * x + q][0], w1 = raw[h][4 * x + q][WPT - 1];
        if constexpr (BF16) {
          t[q][0] = bf16lo(w0.x); t[q][1] = bf16hi(w0.x); t[q][2] = bf16lo(w0.y); t[q][3] = bf16hi(w0.y);
          t[q][4] = bf16lo(w0.z); t[q][5] = bf16hi(w0.z); t[q][6] = bf16lo(w0.w); t[q][7] = bf16hi(w0.w);
        } else {
          t[q][0] = __uint_as_float(w0.x); t[q][1] = __uint_as_float(w0.y); t[q][2] = __uint_as_float(w0.z);
          t[q][3] = __uint_as_float(w0.w); t[q][4] = __uint_as_float(w1.x); t[q][5] = __uint_as_float(w1.y);
          t[q][6] = __uint_as_float(w1.z); t[q][7] = __uint_as_float(w1.w);
        }
      }
      cell2d(t[0], t[1], t[2], t[3], ll1[2 * h + x], W, H, D);
    };
    request(0);
    if constexpr (BF16) request(1);
    {
      float rowv[6][8];
      cell(0, 0, rowv[0], rowv[1], rowv[2]);
      cell(0, 1, rowv[3], rowv[4], rowv[5]);
      if constexpr (!BF16) request(1);
      auto meta = [=](int r) -> RowMeta { return meta2d<3>(r, sby, sbx); };
      flush_rows<6, true, ASYM, 0>(rowv, meta, 0, s_max[qd], q_blk, q_off, scales + prow0, zeros_off, active, tid, nullptr, 0, nullptr,
                                true, 0, 0, nw);
    }
    float rowv[9][8], sum[8];
    cell(1, 0, rowv[0], rowv[1], rowv[2]);
    cell(1, 1, rowv[3], rowv[4], rowv[5]);
    cell2d(ll1[0], ll1[1], ll1[2], ll1[3], sum, rowv[6], rowv[7], rowv[8]);
    float4* const mine = reinterpret_cast<float4*>(s_sum + (size_t)threadIdx.x * 8);
    mine[0] = make_float4(sum[0], sum[1], sum[2], sum[3]);
    mine[1] = make_float4(sum[4], sum[5], sum[6], sum[7]);
    auto meta = [=](int r) -> RowMeta { return meta2d<3>(r + 6, sby, sbx); };
    flush_rows<9, true, ASYM, 0>(rowv, meta, 1, s_max[qd], q_blk, q_off, scales + prow0, zeros_off, active, tid, nullptr, 0, nullptr,
                                true, 0, 0, nw);
  }
  __syncthreads();
  float row[1][8], ll[4][8];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float4* o = reinterpret_cast<const float4*>(s_sum + (size_t)(q * nthr + tid) * 8);
    const float4 v0 = o[0], v1 = o[1];
    ll[q][0] = v0.x; ll[q][1] = v0.y; ll[q][2] = v0.z; ll[q][3] = v0.w;
    ll[q][4] = v1.x; ll[q][5] = v1.y; ll[q][6] = v1.z; ll[q][7] = v1.w;
  }
  float LL[8], W[8], H[8], D[8];
  cell2d(ll[0], ll[1], ll[2], ll[3], LL, W, H, D);
#pragma unroll
  for (int c = 0; c < 8; ++c) row[0][c] = qd == 0 ? LL[c] : qd == 1 ? W[c] : qd == 2 ? H[c] : D[c];
  // the row's range, one group each: parts per wave, then s_amax[row] (the block sum's: of its normalised values)
  uint32_t pos, neg = 0u;
  {
    float v[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) v[c] = qd == 0 ? __fmul_rn(row[0][c], 0.125f) : row[0][c];
    if constexpr (ASYM) {
      row_posneg_bits(v, pos, neg);
      if (!active) pos = neg = 0u;
    } else {
      pos = row_absmax_bits(v);
    }
  }
  pos = wave_max_u32(pos);
  neg = wave_max_u32(neg);
  uint32_t* const part = &s_max[qd][0][0];  // flush_rows used [1] last
  if ((tid & 63) == 0) { part[tid >> 6] = pos; part[16 + (tid >> 6)] = neg; }
  __syncthreads();
  if (tid == 0) {
    for (int i = 0; i < nw; ++i) { pos = max(pos, part[i]); neg = max(neg, part[16 + i]); }
    s_amax[qd] = pos;
    s_amax[kMaxBlockRows + qd] = neg;
  }
  __syncthreads();
  if (qd != 0) {
    auto meta = [=](int) -> RowMeta { return RowMeta{3, qd, qd}; };
    flush_rows<1, true, ASYM, 2>(row, meta, 0, s_max[qd], q_blk, q_off, scales + prow0, zeros_off, active, tid, nullptr, 0,
                                              s_amax, true, 0, 0, nw);
  } else if (sp.q_hi != nullptr) {
    finish_top_row<true, ASYM, false, false, 2>(row[0], 3, nullptr, sp.q_hi + ((size_t)b * k + j) * d + c0,
                                               q_blk + q_off, scales + prow0, zeros_off, j < sp.khi,
                                               active, tid, sp.hi6, b * sp.khi + j, Kpad >> 7, c0, nullptr, 0, s_amax);
  } else if (active) {
    float4* o = reinterpret_cast<float4*>(abot + ((size_t)b * k + j) * d + c0);
    o[0] = make_float4(row[0][0], row[0][1], row[0][2], row[0][3]);
    o[1] = make_float4(row[0][4], row[0][5], row[0][6], row[0][7]);
  }
}

template <int RLOG, bool BF16, bool ASYM, int PASS, bool OUT6>
hipError_t launch_bottom1d_pass(const stamp_plan* p, const void* X, uint8_t* q_lo, float* scales, float* abot, int nthreads,
                                const SplitArgs& sp, hipStream_t st) {
  const StampGeom& g = p->geom;
  const size_t lds = (size_t)8 * nthreads * (BF16 ? 16 : 32);  // staging buffer: 2 batches of 4 token rows
  if (lds > 160 * 1024 - 2048) return hipErrorInvalidValue;
  static size_t lds_done[kStampMaxDevices] = {};
  hipError_t e = stamp_allow_lds(reinterpret_cast<const void*>(&k_bottom1d<RLOG, BF16, ASYM, PASS, OUT6>), lds, lds_done);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_bottom1d<RLOG, BF16, ASYM, PASS, OUT6>), dim3(g.k, g.B, PASS == 0 ? 1 : sp.nsplit), dim3(nthreads), lds, st,
                     X, q_lo, scales, abot, g.s, g.d, g.k, p->Kpad, (size_t)g.B * g.s, sp);
  return hipGetLastError();
}

// one pass when a workgroup can hold all channels, else maxima pass + quantization pass over channel splits
template <int RLOG, bool BF16, bool ASYM>
hipError_t launch_bottom1d(const stamp_plan* p, const void* X, uint8_t* q_lo, float* scales, float* abot, int nthreads,
                           const SplitArgs& sp, hipStream_t st) {
  constexpr bool kOut6 = RLOG <= 4;  // direct_route: larger blocks leave their codes packed
  const bool out6 = sp.hi6.p != nullptr;
  if (out6 && !kOut6) return hipErrorInvalidValue;
  if (sp.nsplit == 1)
    return out6 ? launch_bottom1d_pass<RLOG, BF16, ASYM, 0, kOut6>(p, X, q_lo, scales, abot, nthreads, sp, st)
                : launch_bottom1d_pass<RLOG, BF16, ASYM, 0, false>(p, X, q_lo, scales, abot, nthreads, sp, st);
  const hipError_t e = launch_bottom1d_pass<RLOG, BF16, ASYM, 1, false>(p, X, q_lo, scales, abot, nthreads, sp, st);
  if (e != hipSuccess) return e;
  return out6 ? launch_bottom1d_pass<RLOG, BF16, ASYM, 2, kOut6>(p, X, q_lo, scales, abot, nthreads, sp, st)
              : launch_bottom1d_pass<RLOG, BF16, ASYM, 2, false>(p, X, q_lo, scales, abot, nthreads, sp, st);
}

template <int RLOG, bool BF16, bool ASYM, bool OUT6>
hipError_t launch_rag_o(const stamp_plan* p, const void* X, int8_t* q_hi, uint8_t* q_lo, float* scales, const Hi6Out& hi6, hipStream_t st) {
  const StampGeom& g = p->geom;
  const int nthreads = (g.d / 8 + 63) / 64 * 64;
  const size_t lds = (size_t)8 * nthreads * (BF16 ? 16 : 32);
  static size_t lds_done[kStampMaxDevices] = {};
  const hipError_t e = stamp_allow_lds(reinterpret_cast<const void*>(&k_bottom1d_rag<RLOG, BF16, ASYM, OUT6>), lds, lds_done);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_bottom1d_rag<RLOG, BF16, ASYM, OUT6>), dim3(p->rag.nb + p->rag.o, g.B), dim3(nthreads), lds, st, X, q_hi, q_lo, scales,
                     g.s, g.d, g.khi, p->Kpad, (size_t)g.B * g.s, p->rag, hi6);
  return hipGetLastError();
}
template <int RLOG, bool BF16, bool ASYM>
hipError_t launch_rag(const stamp_plan* p, const void* X, int8_t* q_hi, uint8_t* q_lo, float* scales, const Hi6Out& hi6, hipStream_t st) {
  if (hi6.p != nullptr && RLOG > 4) return hipErrorInvalidValue;
  return hi6.p != nullptr ? launch_rag_o<RLOG, BF16, ASYM, (RLOG <= 4)>(p, X, q_hi, q_lo, scales, hi6, st)
                          : launch_rag_o<RLOG, BF16, ASYM, false>(p, X, q_hi, q_lo, scales, hi6, st);
}
template <int RLOG>
hipError_t launch_rag_t(const stamp_plan* p, const void* X, int8_t* q_hi, uint8_t* q_lo, float* scales, const Hi6Out& hi6, hipStream_t st) {
  const StampGeom& g = p->geom;
  if (g.x_bf16) return g.asym ? launch_rag<RLOG, true, true>(p, X, q_hi, q_lo, scales, hi6, st) : launch_rag<RLOG, true, false>(p, X, q_hi, q_lo, scales, hi6, st);
  return g.asym ? launch_rag<RLOG, false, true>(p, X, q_hi, q_lo, scales, hi6, st) : launch_rag<RLOG, false, false>(p, X, q_hi, q_lo, scales, hi6, st);
}

}  // namespace

#endif  // STAMP_BOTTOM_KERNEL_H_
