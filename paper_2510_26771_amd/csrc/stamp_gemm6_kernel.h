// The FP6 GEMM kernel over the 4-bit rows and its launchers for one tile size (STAMP_GEMM6_WAVES waves per workgroup: 8 or 4; with
// STAMP_GEMM6_PAIR two workgroups of 4 per CU).
// Operand layout: stamp_gemm6.hip.
#ifndef STAMP_GEMM6_KERNEL_H_
#define STAMP_GEMM6_KERNEL_H_

#include <type_traits>

#include "stamp_epilogue_reg.h"
#include "stamp_fp6.h"

namespace {

using namespace stamp_gemm;

// Workgroup: 8 waves (2 x 4), tile 256 x 256, one workgroup per CU with two waves on every SIMD, all
// eight sharing one operand stage: 48 KB per K step for 256 x 256 x 128 products, a third less L2 -> LDS
// traffic per product than two independent 256 x 128 workgroups would need (the FP6 pipeline consumes a K
// step in half the time of the int8 one, which makes that traffic the bound).  S stages (kNumStage6: three, PAIR
// two): while step kt is multiplied, the stages of the S - 1 steps after it have landed or are in flight; the request
// for step kt + S goes out late in step kt, into the stage that step kt has just given up.
//
// The kernel is persistent: the workgroups (one per CU, PAIR: two) walk their shares of the tiles (the XCD-aware order of
// tile_of_sid, every workgroup of an XCD taking every wx-th tile of that XCD's range), and the operand
// pipeline runs on across tile boundaries: the first S K steps of the next tile are requested during the last
// S steps of the current one, so they, and the stores of the epilogue, are in flight while the epilogue
// computes.  The epilogue works in registers (stamp_epilogue_reg.h) and leaves the operand stages alone.
//
// Inside a step nothing waits for what it has just asked for: the LDS reads of an activation block fly under the
// MFMAs of the block before it, the one workgroup barrier sits before the last block (whose MFMAs cover the reads
// of the next step's first fragments), and the loads of a stage request are issued one at a time among MFMAs, three in that last
// block, the others in the next step.
//
// WAVES = 4: tile 128 x 256, one wave on every SIMD, 36 KB per K step; the same loop, nine loads per wave and step.  A tile
// takes 0.64 of the time of a 256 x 256 one (8.5 us + 0.455 us per K step against 12.8 + 0.72, all CUs busy; measured while the products were 32 x 32 x 64
// MFMAs): for shapes that leave CUs idle (the rule stands at stamp_gemm6_half_tiles).
//
// PAIR (WAVES = 4): two workgroups per CU, two stages each (72 KB): one multiplies while the other is in its epilogue, and the last
// tiles are half as large; but a CU moves half as much again per product.  For shallow layers of more than one round (the rule
// stands at stamp_gemm6_pairs).
//
// HI (WAVES = 4): the tile's 8-bit rows ride along as a fifth block of 32 operand rows (h of 16 places, then l; stamp_hi_places),
// 3 KB more per K step and eight MFMAs more per wave and step; their sums, the levels above and the block sums stay in
// registers.  A launch and the stream of the weights a second time are saved (figures at stamp_hi_tiles).  Not for WAVES = 8: the
// matrix pipe has no time to spare there (2048 x 4096 -> 11008 58 us and 17 for the rows' own kernel, 72 in one; 8 x 4096 x 4096 -> 4096
// 261 and 38, 324).
constexpr int BN6 = 256;
constexpr int vm_wait6(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }  // s_waitcnt vmcnt(n)

template <int WAVES, bool HI = false>
struct Tile6 {
  static constexpr int BMW = 32 * WAVES;                    // rows
  static constexpr int kStageA = BMW / 32 * kBlock6;        // bytes of the activation part of a stage
  static constexpr int kStageAB = kStageA + 2 * kStageB6;
  static constexpr int kStage = kStageAB + (HI ? kBlock6 : 0);  // 48, 36 or 39 KB
};
constexpr int kHiInfoBytes = 2 * kHiPlaces * 4;  // row factors and offsets of the places

// whether one of the tile's blocks has an 8-bit row (or lends its place to the token left out)
__device__ __forceinline__ bool hi_tile_has(const StampHiTiles& t, int tile) {
  if (t.L > 0) return true;
  const int j = (tile << t.lognb) % t.k;
  return j < t.khi || j + (1 << t.lognb) > t.k;
}
// row factor and offset of one of a tile's places (0 where it has no row); the sums are of whole codes
template <bool RAG>
__device__ __forceinline__ void hi_place_info(const GemmArgs& a, int tile, int p, float& fac, float& rz) {
  const StampGeom& g = a.g;
  const StampHiTiles& t = a.ht;
  fac = rz = 0.0f;
  int b, up;
  const int slot = stamp_hi_slot_of_place(t, g.B, tile, p, &b, &up);
  if (slot < 0) return;
  const size_t row = RAG ? (size_t)b * g.s + slot : (size_t)b * g.s + (size_t)slot * g.R;
  const size_t zeros_off = (size_t)g.B * g.s;
  fac = a.scales[row] * (RAG ? 1.0f : haar_norm_dev(g.r + up, g.is2d));
  if (g.asym) rz = a.scales[zeros_off + row] - (slot < g.khi ? 128.0f : 8.0f);
}
// The 8-bit rows' block -> sums of the lane's blocks (eo.P); the token left out -> Y.  acch: the row
// tile of h (th = 0) and that of l, of 16 places each.  Same operations in the same order as k_hi6.
template <int RL, bool YBF16, bool SYM, bool RAG, typename Eo>
__device__ __forceinline__ void hi_block_sums(const GemmArgs& a, const AccTiles (&acch)[2], const float* info, Eo& eo, int tile, int nw, int lane) {
  constexpr int lognb = 7 - RL, nb = 1 << lognb;
  const StampHiTiles& t = a.ht;
  const int l32 = lane & 31, kg = lane >> 5, n = nw + 2 * l32;
  float val[kHiPlaces][2];
#pragma unroll
  for (int ni = 0; ni < 2; ++ni) {
    float x[8], y[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = __builtin_fmaf(16.0f, acch[ni][8 * (i >> 2) + (i & 3)], acch[ni][8 * (i >> 2) + 4 + (i & 3)]) * 64.0f;
    swap16x4(x[0], x[4], x[1], x[5], x[2], x[6], x[3], x[7]);  // x[i]: place 8 kg + i of column l32
#pragma unroll
    for (int i = 0; i < 8; ++i) y[i] = x[i];
#pragma unroll
    for (int i = 0; i < 8; i += 4) swap32x4(x[i], y[i], x[i + 1], y[i + 1], x[i + 2], y[i + 2], x[i + 3], y[i + 3]);
#pragma unroll
    for (int i = 0; i < 8; ++i) {  // x: lane group 0's place, y: lane group 1's, in both
      val[i][ni] = x[i];
      val[8 + i][ni] = y[i];
    }
  }
#pragma unroll
  for (int p = 0; p < kHiPlaces; ++p) {
    const float fac = info[p], rz = SYM ? 0.0f : info[kHiPlaces + p];
#pragma unroll
    for (int ni = 0; ni < 2; ++ni) {
      const float af = SYM ? val[p][ni] : __builtin_fmaf(-rz, eo.cs[ni], val[p][ni]);
      val[p][ni] = (af * fac) * eo.sw[ni];
    }
  }
  if constexpr (RAG) {
    if (t.o) {  // the token left out has the place of block khi - 1
      const int g0 = tile << lognb;
      int b = g0 / t.k, j = g0 - b * t.k;
#pragma unroll
      for (int p = 0; p < nb; ++p) {
        if (j == t.khi - 1 && b < a.g.B && kg == 0 && n < a.N)
          put_pair<YBF16, false>(a.out, (size_t)b * a.g.s * a.N + n, val[p][0] + eo.bias[0], val[p][1] + eo.bias[1], a.N - n);
        if (++j == t.k) {
          j = 0;
          ++b;
        }
      }
    }
    const float nrm = haar_norm_dev(a.g.r, 0);
#pragma unroll
    for (int p = 0; p < nb; ++p)
#pragma unroll
      for (int ni = 0; ni < 2; ++ni) val[p][ni] *= nrm;
  } else if (t.L > 0) {
    const int j0 = (tile << lognb) % t.k;
#pragma unroll
    for (int p = kHiPlaces - 1; p >= nb; --p) {  // the levels above the tile's sub-tree, coarsest first
      const int up = lognb + 1 + p - nb;
      if (up <= t.L) {
        const float s = (j0 >> (up - 1)) & 1 ? -1.0f : 1.0f;
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) val[0][ni] = __builtin_fmaf(val[p][ni], s, val[0][ni]);
      }
    }
#pragma unroll
    for (int lev = lognb; lev >= 1; --lev)
      if (lev <= t.L) {
#pragma unroll
        for (int i = 0; i < nb; i += 1 << lev)
#pragma unroll
          for (int ni = 0; ni < 2; ++ni) {
            const float x = val[i][ni], d = val[i + (1 << (lev - 1))][ni];
            val[i][ni] = x + d;
            val[i + (1 << (lev - 1))][ni] = x - d;
          }
      }
  }
#pragma unroll
  for (int q = 0; q < nb / 2; ++q)
#pragma unroll
    for (int ni = 0; ni < 2; ++ni) eo.P[q][ni] = kg ? val[RegMap<RL>::block(q, 1)][ni] : val[RegMap<RL>::block(q, 0)][ni];
}

// tile of position sid in the walk: 8 M-tiles, then the next N-tile, group of 8 M-tiles after group
__device__ __forceinline__ void tile_of_sid(int sid, int mt, int nt, int& tm, int& tn) {
  const int per_group = kGroupM * nt;
  const int grp = sid / per_group, in_grp = sid - grp * per_group;
  const int gm = min(kGroupM, mt - grp * kGroupM);
  tm = grp * kGroupM + in_grp % gm;
  tn = in_grp / gm;
}

// SYM: a fused-mode kernel for plans with symmetric activation codes (no offset term in the epilogue)
// RAG: fused mode over the blocks of a 1-D Haar transform of any length (StampRag); ODD: for odd d_out
template <int EPI, int RB, bool IS2D, bool YBF16, bool SYM = false, bool RAG = false, bool ODD = false, int WAVES = 8, bool HI = false, bool PAIR = false>
__global__ __launch_bounds__(64 * WAVES, (WAVES == 8 || HI ? 1 : 2)) void k_gemm6(const GemmArgs a) {
  using Acc = AccF6Lo;
  request_args<GemmArgs>();
  constexpr int BMW = Tile6<WAVES, HI>::BMW, kStageA = Tile6<WAVES, HI>::kStageA, kStage6 = Tile6<WAVES, HI>::kStage;
  constexpr int kStageAB = Tile6<WAVES, HI>::kStageAB;
  constexpr int NIW = NI;  // 32-column MFMA blocks per wave along N
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  constexpr int NT = 64 * WAVES;  // threads
  constexpr int kNumStage6 = PAIR ? 2 : 3;
  constexpr int kMainBytes = kNumStage6 * kStage6;
  uint8_t* const row_info = smem + kMainBytes;  // two buffers, alternating from tile to tile
  constexpr int kHiInfo = kRowInfoBytes + (RAG ? 256 : 0);  // RAG: + the token factors of a short block
  constexpr int kRowInfo = kHiInfo + (HI ? kHiInfoBytes : 0);
  constexpr int nA = kStageA / (NT * 16), nB = 2 * kStageB6 / (NT * 16);  // 16-byte chunks per thread and step
  constexpr int kLoadsPerStep = nA + nB + (HI ? 1 : 0);

  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform, kept in a scalar register
  // wave tile: rows [128 wm, +128), columns [32 NIW wn, +32 NIW)
  const int wm = wave >> 2, wn = wave & 3;
  const int KT = a.Kpad / BK;
  const int mt = (a.M + BMW - 1) / BMW, nt = a.Npad / BN6, total = mt * nt;

  // tiles of this workgroup: the XCD's contiguous range of the walk, every wx-th position from `local` on
  const int nwg = (int)gridDim.x, xcd = (int)blockIdx.x % kNumXcd, local = (int)blockIdx.x / kNumXcd;
  const int wx = (nwg - xcd + kNumXcd - 1) / kNumXcd;  // workgroups that run on this XCD
  const int tall = total / kNumXcd, rem = total % kNumXcd;
  const int first = xcd * tall + min(xcd, rem), count = tall + (xcd < rem ? 1 : 0);
  if (local >= count) return;

  // global image = LDS image: chunk q = i * NT + tid of an operand's stage goes to byte 16 q.  The
  // weight stage is two column tiles of 128 (KT * 12 KB apart in memory): chunks 0..767 and 768..1535;
  // the boundary falls between waves, so the source tile of a pass is wave-uniform.  Addresses are a
  // wave-uniform base (tile, K step, pass, wave) plus the lane's 32-bit offset.
  // (the lane number is read anew for every tile and every epilogue, so that nothing per lane is live across an epilogue, which has no
  // register to spare: a value kept in scratch memory would be reloaded behind all stores)
  auto lane_now = []() __attribute__((always_inline)) {
    uint32_t l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
  };
  uint32_t lane16 = lane_now() * 16u;
  const uint32_t wave1k = (uint32_t)wave * 1024u;
  // cursor of the requests: request rq_kt of the tile at position rq_pos of this workgroup's walk (all scalar).  The
  // loads address memory through two buffer descriptors (the tile's activation panel; its two weight panels, KT * 12 KB
  // apart) + a scalar byte offset + the lane's 32-bit offset: no vector address arithmetic per load.
  // K step of a tile's first request.  The workgroups of an XCD that share an operand panel (same row or column of
  // the XCD's 8 x 4 window of tiles) ask for a line at the same moment when they walk K in step: one misses L2, the
  // others wait on the same miss.  Started a few K steps apart (every tile walks all KT steps once, from its own
  // start, wrapping: an fp32 sum of these integers is exact in any order), most of them find the line in L2.
  int rq_k0;
  {
    int tm0_, tn0_;
    tile_of_sid(first + local, mt, nt, tm0_, tn0_);
    rq_k0 = (((tm0_ & 7) + 2 * (tn0_ & 3)) & 7) % KT;
  }
  int rq_pos = local, rq_kt = 0, rq_stg = 0, rq_kk = rq_k0;  // rq_kt counts the tile's requests, rq_kk is their K step
  __amdgpu_buffer_rsrc_t rdA, rdB;
  [[maybe_unused]] __amdgpu_buffer_rsrc_t rdH;  // HI: no records where the tile has no 8-bit row
  auto rq_tile = [&]() {
    int tm_, tn_;
    tile_of_sid(first + rq_pos, mt, nt, tm_, tn_);
    // (a 128-row tile is one half of a 256-row tile of the layout: its blocks are contiguous in every K step)
    const uint8_t* pa_ = WAVES == 8 ? a.A + (size_t)tm_ * KT * kStageA6 : a.A + (size_t)(tm_ >> 1) * KT * kStageA6 + (tm_ & 1) * kStageA;
    rdA = __builtin_amdgcn_make_buffer_rsrc((void*)pa_, 0, 0x7fffffff, 0x00020000);
    rdB = __builtin_amdgcn_make_buffer_rsrc((void*)(a.Bq + (size_t)(2 * tn_) * KT * kStageB6), 0, 0x7fffffff, 0x00020000);
    if constexpr (HI)
      rdH = __builtin_amdgcn_make_buffer_rsrc((void*)(a.H + (size_t)tm_ * KT * kBlock6), 0, hi_tile_has(a.ht, tm_) ? 0x7fffffff : 0, 0x00020000);
  };
  rq_tile();
  // A request = the kLoadsPerStep loads of the next K step of the walk into the next stage of the ring.  rq_begin
  // fixes its addresses and advances the cursor, rq_issue<i> issues its i-th load: the
  // main loop spreads them among its MFMAs (eight waves issuing all their loads at once keep the address unit busy
  // for several hundred cycles, during which none of them can issue anything else).
  // Three of its loads go out among the MFMAs of the step's last block (three more beside the 8-bit rows'), the others in the next step (rq_tail: still to be
  // issued), with two MFMAs or more between any two: one load keeps the address unit busy for 16 cycles, an MFMA the matrix pipe for 17.
  // (Spread evenly over the whole step the last ones land too late: 2048 x 11008 -> 4096 60.3 us against 57.7.)
  bool rq_tail = false;
  uint8_t* rq_so = nullptr;
  [[maybe_unused]] uint32_t rq_oh = 0;
  uint32_t rq_oa = 0, rq_ob = 0;  // byte offsets of the request's K step in the activation / weight panels
  auto rq_begin = [&]() {
    if (__builtin_expect(rq_kt == KT, 0)) {  // the tile of the request before this one is complete: its descriptors are no longer needed
      rq_kt = 0;
      rq_pos += wx;
      if (rq_pos < count) {
        rq_tile();
      } else {
        // the walk is over: the remaining requests read nothing (a descriptor without records; the loads still count,
        // so every wait of the main loop is for the same number of them)
        rdA = __builtin_amdgcn_make_buffer_rsrc((void*)a.A, 0, 0, 0x00020000);
        rdB = rdA;
        if constexpr (HI) rdH = rdA;
      }
    }
    rq_so = smem + rq_stg * kStage6 + wave * 1024;
    rq_oa = (uint32_t)rq_kk * (uint32_t)kStageA6 + wave1k;
    rq_ob = (uint32_t)rq_kk * (uint32_t)kStageB6 + wave1k;
    if constexpr (HI) rq_oh = (uint32_t)rq_kk * (uint32_t)kBlock6;
    rq_kk = (rq_kk == KT - 1) ? 0 : rq_kk + 1;
    rq_stg = (rq_stg == kNumStage6 - 1) ? 0 : rq_stg + 1;
    ++rq_kt;
  };
  auto rq_issue = [&](auto i_tag) __attribute__((always_inline)) {
    constexpr int li = decltype(i_tag)::value;
    if constexpr (li < nA) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rdA, (void __attribute__((address_space(3)))*)(rq_so + li * (NT * 16)), 16, lane16,
                                               rq_oa + (uint32_t)(li * (NT * 16)), 0, 0);
    } else if constexpr (li >= nA + nB) {
      // three waves' worth: the fourth asks for the first kilobyte again, so that every wave counts the same number of loads
      const int part = (wave % 3) * kPart;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rdH, (void __attribute__((address_space(3)))*)(rq_so - wave * 1024 + kStageAB + part), 16,
                                               lane16, rq_oh + (uint32_t)part, 0, 0);
    } else {
      constexpr int i = li - nA;
      // chunk i * NT + tid of the 1536: column tile 1 (KT stages further on) from chunk 768 on (a whole number of waves)
      const bool half = (i * NT + wave * 64) >= 768;
      const uint32_t ob = rq_ob + (half ? (uint32_t)KT * (uint32_t)kStageB6 + (uint32_t)(i * NT * 16 - 768 * 16) : (uint32_t)(i * NT * 16));
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rdB, (void __attribute__((address_space(3)))*)(rq_so + kStageA + i * (NT * 16)), 16,
                                               lane16, ob, 0, 0);
    }
  };
  static_assert(kLoadsPerStep <= 10, "the main loop has places for ten loads per wave and step");
  // loads FROM .. of the request
  auto rq_rest = [&](auto from_tag) __attribute__((always_inline)) {
    constexpr int from = decltype(from_tag)::value;
    auto one = [&](auto i) __attribute__((always_inline)) {
      if constexpr (i.value >= from && i.value < kLoadsPerStep) rq_issue(i);
    };
    one(std::integral_constant<int, 0>{});
    one(std::integral_constant<int, 1>{});
    one(std::integral_constant<int, 2>{});
    one(std::integral_constant<int, 3>{});
    one(std::integral_constant<int, 4>{});
    one(std::integral_constant<int, 5>{});
    one(std::integral_constant<int, 6>{});
    one(std::integral_constant<int, 7>{});
    one(std::integral_constant<int, 8>{});
    one(std::integral_constant<int, 9>{});
  };
  auto request_next = [&]() {
    rq_begin();
    rq_rest(std::integral_constant<int, 0>{});
  };

  // LDS byte addresses of part 0 of a wave's 48 bytes in stage 0: 32-row block (then lane * 16)
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)smem;
  const uint32_t adrA0 = (uint32_t)((wm * 4) * kBlock6);
  const uint32_t adrH0 = (uint32_t)kStageAB;
  const uint32_t adrB0 = (uint32_t)(kStageA + (wn >> 1) * kStageB6 + ((wn & 1) * 2) * kBlock6);

  // ---- prologue: all stages but one requested, landed and published by a barrier; the last one requested ----
#pragma unroll
  for (int i = 0; i < kNumStage6 - 1; ++i) request_next();
  {
    int tm0, tn0;
    tile_of_sid(first + local, mt, nt, tm0, tn0);
    if (tid < BMW) store_row_info<Acc, EPI, RAG>(a, tm0 * BMW, tid, row_info);
    if constexpr (HI) {
      if (tid >= BMW && tid < BMW + kHiPlaces) {
        float fac, rz;
        hi_place_info<RAG>(a, tm0, tid - BMW, fac, rz);
        reinterpret_cast<float*>(row_info + kHiInfo)[tid - BMW] = fac;
        reinterpret_cast<float*>(row_info + kHiInfo)[kHiPlaces + tid - BMW] = rz;
      }
    }
    if constexpr (RAG) {
      if (tid < 64) {
        const float f = tid < a.rag.mlast ? rag_leaf(a.rag, tid) : 0.0f;
        reinterpret_cast<float*>(row_info + kRowInfoBytes)[tid] = f;
        reinterpret_cast<float*>(row_info + kRowInfo + kRowInfoBytes)[tid] = f;
      }
    }
  }
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  request_next();
  int landed = kNumStage6 - 2;  // steps from here on whose loads are known to have landed (their barrier needs no wait)
  int stg = 0;     // stage of the step about to be multiplied
  int rbuf = 0;    // row-info buffer of the current tile

  // Fragment registers.  A lane's 48 bytes of one 32-row block and K step are the 24-byte MFMA operands of the block's
  // two tiles of 16 rows, read as three 16-byte parts.  The parts of a fragment must land in 12 CONSECUTIVE registers (the
  // first operand is registers 0..5, the second 6..11), which the register allocator does not arrange for separate
  // asm outputs (it copies parts into fresh tuples and runs out of registers); the fragments therefore live in fixed
  // registers v184..v255: two activation sets (block mi + 1 is read while block mi is multiplied) and the weights'
  // NIW = 2 blocks double-buffered from step to step.
  static_assert(NIW == 2, "fixed fragment registers are laid out for two weight blocks per wave");
  struct Frag {
    u6 h0, h1;
  };
#define STAMP_RD3(f, H0, H1, P0, P1, P2, base, off)                                                                   \
  asm volatile("ds_read_b128 " P0 ", %2 offset:%3\n\tds_read_b128 " P1 ", %2 offset:%4\n\tds_read_b128 " P2 ", %2 offset:%5" \
               : "=&{" H0 "}"(f.h0), "=&{" H1 "}"(f.h1)                                                               \
               : "v"(base), "n"(off), "n"((off) + kPart), "n"((off) + 2 * kPart))
#define STAMP_RD_AS0(base, off) STAMP_RD3(As0, "v[184:189]", "v[190:195]", "v[184:187]", "v[188:191]", "v[192:195]", base, off)
#define STAMP_RD_HS(base, off) STAMP_RD3(Hs, "v[172:177]", "v[178:183]", "v[172:175]", "v[176:179]", "v[180:183]", base, off)
#define STAMP_WAIT_HS(cnt) STAMP_WAIT1(cnt, Hs, "v[172:177]", "v[178:183]")
#define STAMP_RD_AS1(base, off) STAMP_RD3(As1, "v[196:201]", "v[202:207]", "v[196:199]", "v[200:203]", "v[204:207]", base, off)
#define STAMP_RD_B00(base) STAMP_RD3(B00, "v[208:213]", "v[214:219]", "v[208:211]", "v[212:215]", "v[216:219]", base, 0)
#define STAMP_RD_B01(base) STAMP_RD3(B01, "v[220:225]", "v[226:231]", "v[220:223]", "v[224:227]", "v[228:231]", base, kBlock6)
#define STAMP_RD_B10(base) STAMP_RD3(B10, "v[232:237]", "v[238:243]", "v[232:235]", "v[236:239]", "v[240:243]", base, 0)
#define STAMP_RD_B11(base) STAMP_RD3(B11, "v[244:249]", "v[250:255]", "v[244:247]", "v[248:251]", "v[252:255]", base, kBlock6)
  // a wait names the fragments it covers (same registers in and out), which keeps their MFMAs behind it
#define STAMP_WAIT2(cnt, x, XR, y, YR) asm volatile("s_waitcnt lgkmcnt(" #cnt ")" : "={" XR "}"(x), "={" YR "}"(y) : "0"(x), "1"(y))
#define STAMP_WAIT_AS0B(cnt, b, H0, H1)                                                                                     \
  asm volatile("s_waitcnt lgkmcnt(" #cnt ")"                                                                                \
               : "={v[184:189]}"(As0.h0), "={v[190:195]}"(As0.h1), "={" H0 "}"(b.h0), "={" H1 "}"(b.h1)                      \
               : "0"(As0.h0), "1"(As0.h1), "2"(b.h0), "3"(b.h1))
#define STAMP_WAIT1(cnt, f, H0, H1) asm volatile("s_waitcnt lgkmcnt(" #cnt ")" : "={" H0 "}"(f.h0), "={" H1 "}"(f.h1) : "0"(f.h0), "1"(f.h1))
#define STAMP_WAIT_AS0(cnt) STAMP_WAIT1(cnt, As0, "v[184:189]", "v[190:195]")
#define STAMP_WAIT_AS1(cnt) STAMP_WAIT1(cnt, As1, "v[196:201]", "v[202:207]")

  for (int pos = local; pos < count; pos += wx) {
    int tm, tn;
    tile_of_sid(first + pos, mt, nt, tm, tn);
    const int m0 = tm * BMW, n0 = tn * BN6;
    const int nw = n0 + wn * (32 * NIW);

    AccTiles acc[4][NIW];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < NIW; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[i][j].q[q] = (f4){0.0f, 0.0f, 0.0f, 0.0f};

    [[maybe_unused]] AccTiles acch[NIW];  // HI: the 8-bit rows' block
    [[maybe_unused]] const bool has_hi = HI && hi_tile_has(a.ht, tm);
    if constexpr (HI) {
#pragma unroll
      for (int j = 0; j < NIW; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) acch[j].q[q] = (f4){0.0f, 0.0f, 0.0f, 0.0f};
    }
    [[maybe_unused]] Frag Hs;
    Frag As0, As1, B00, B01, B10, B11;  // per tile: no fragment is carried across the epilogue
    // row tile th of an activation block against column tile tc of a weight block
    auto mfma = [&](f4& c, const u6& A, const u6& W) __attribute__((always_inline)) {
      c = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(widen((v6i)A), widen((v6i)W), c, 2, 2, 0, 0, 0, 0);
    };
    // The eight MFMAs of an activation block; each shares an operand with the one before.  after(i): what goes between the i-th and the next
    auto mfma8 = [&](AccTiles (&c)[NIW], const Frag& A, const Frag& W0, const Frag& W1, auto after) __attribute__((always_inline)) {
      auto then = [&](auto i) __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        after(i);
        __builtin_amdgcn_sched_barrier(0);
      };
      mfma(c[0].q[0], A.h0, W0.h0);
      mfma(c[0].q[1], A.h1, W0.h0);
      then(std::integral_constant<int, 2>{});
      mfma(c[0].q[3], A.h1, W0.h1);
      mfma(c[0].q[2], A.h0, W0.h1);
      then(std::integral_constant<int, 4>{});
      mfma(c[1].q[2], A.h0, W1.h1);
      mfma(c[1].q[3], A.h1, W1.h1);
      then(std::integral_constant<int, 6>{});
      mfma(c[1].q[1], A.h1, W1.h0);
      mfma(c[1].q[0], A.h0, W1.h0);
    };
    // load i of the request of the step before, if it has that many
    auto tail = [&](auto i) __attribute__((always_inline)) {
      constexpr int li = decltype(i)::value;
      if constexpr (li < kLoadsPerStep) {
        if (rq_tail) rq_issue(i);
      }
    };
    constexpr int kFirst = HI ? 6 : 3;  // loads of a request in the step itself

    // Step kt (pb = 0: weights in B00, B01, the next step's go to B10, B11; pb = 1: the other way round).  On entry
    // the reads of the step's weights and of activation block 0 have been issued (by the head of the tile or by the
    // step before).  Block 1 is requested, block 0 multiplied, block 2 requested, block 1 multiplied, ...: the LDS
    // reads of a block fly under the MFMAs of the block before.  After block 2 every read of this stage has
    // returned: the wave waits for its own loads of the NEXT step's stage (with three stages the step after that may
    // still be in flight), meets the others at the workgroup barrier (next stage visible, this stage free), requests the
    // step kNumStage6 ahead into this stage, issues the reads of the next step's block 0 and weights, and multiplies block 3
    // under them.  One barrier per step, none between a read and its use.
    auto step = [&](auto pb_tag) __attribute__((always_inline)) {
      constexpr int pb = decltype(pb_tag)::value;
      const uint32_t sa = lds0 + (uint32_t)(stg * kStage6);
      __builtin_amdgcn_sched_barrier(0);
      STAMP_RD_AS1(sa + adrA0 + lane16, 1 * kBlock6);
      // block 0: of the 12 reads in flight the first 6 feed the first four MFMAs, 9 the others
      if constexpr (pb == 0) {
        STAMP_WAIT_AS0B(6, B00, "v[208:213]", "v[214:219]");
        mfma(acc[0][0].q[0], As0.h0, B00.h0);
        mfma(acc[0][0].q[1], As0.h1, B00.h0);
        __builtin_amdgcn_sched_barrier(0);
        tail(std::integral_constant<int, kFirst>{});
        __builtin_amdgcn_sched_barrier(0);
        mfma(acc[0][0].q[3], As0.h1, B00.h1);
        mfma(acc[0][0].q[2], As0.h0, B00.h1);
        __builtin_amdgcn_sched_barrier(0);
        STAMP_WAIT2(3, B01.h0, "v[220:225]", B01.h1, "v[226:231]");
        mfma(acc[0][1].q[2], As0.h0, B01.h1);
        mfma(acc[0][1].q[3], As0.h1, B01.h1);
        __builtin_amdgcn_sched_barrier(0);
        tail(std::integral_constant<int, kFirst + 1>{});
        __builtin_amdgcn_sched_barrier(0);
        mfma(acc[0][1].q[1], As0.h1, B01.h0);
        mfma(acc[0][1].q[0], As0.h0, B01.h0);
      } else {
        STAMP_WAIT_AS0B(6, B10, "v[232:237]", "v[238:243]");
        mfma(acc[0][0].q[0], As0.h0, B10.h0);
        mfma(acc[0][0].q[1], As0.h1, B10.h0);
        __builtin_amdgcn_sched_barrier(0);
        tail(std::integral_constant<int, kFirst>{});
        __builtin_amdgcn_sched_barrier(0);
        mfma(acc[0][0].q[3], As0.h1, B10.h1);
        mfma(acc[0][0].q[2], As0.h0, B10.h1);
        __builtin_amdgcn_sched_barrier(0);
        STAMP_WAIT2(3, B11.h0, "v[244:249]", B11.h1, "v[250:255]");
        mfma(acc[0][1].q[2], As0.h0, B11.h1);
        mfma(acc[0][1].q[3], As0.h1, B11.h1);
        __builtin_amdgcn_sched_barrier(0);
        tail(std::integral_constant<int, kFirst + 1>{});
        __builtin_amdgcn_sched_barrier(0);
        mfma(acc[0][1].q[1], As0.h1, B11.h0);
        mfma(acc[0][1].q[0], As0.h0, B11.h0);
      }
      __builtin_amdgcn_sched_barrier(0);
      STAMP_RD_AS0(sa + adrA0 + lane16, 2 * kBlock6);
      STAMP_WAIT_AS1(3);
      mfma8(acc[1], As1, pb == 0 ? B00 : B10, pb == 0 ? B01 : B11, [&](auto i) __attribute__((always_inline)) {
        if constexpr (i.value == 2) tail(std::integral_constant<int, kFirst + 2>{});
        if constexpr (i.value == 4) tail(std::integral_constant<int, kFirst + 3>{});
        if constexpr (i.value == 6) tail(std::integral_constant<int, kFirst + 4>{});
      });
      __builtin_amdgcn_sched_barrier(0);
      STAMP_RD_AS1(sa + adrA0 + lane16, 3 * kBlock6);
      if constexpr (HI) {
        STAMP_RD_HS(sa + adrH0 + lane16, 0);
        STAMP_WAIT_AS0(6);
      } else {
        STAMP_WAIT_AS0(3);
      }
      const int stg1 = (stg == kNumStage6 - 1) ? 0 : stg + 1;
      const uint32_t sn = lds0 + (uint32_t)(stg1 * kStage6);
      mfma8(acc[2], As0, pb == 0 ? B00 : B10, pb == 0 ? B01 : B11, [&](auto i) __attribute__((always_inline)) {
        if constexpr (i.value == 2) {
          tail(std::integral_constant<int, kFirst + 5>{});
          rq_begin();  // (addresses alone: the stage is asked for behind the barrier)
        }
      });
      __builtin_amdgcn_sched_barrier(0);
      STAMP_WAIT_AS1(0);
      if constexpr (HI) STAMP_WAIT_HS(0);
      // ---- the next step's stage ----
      asm volatile("" ::: "memory");
      if (landed > 0) {
        --landed;
      } else {
        __builtin_amdgcn_s_waitcnt(vm_wait6(kLoadsPerStep * (kNumStage6 - 2)));  // three stages: the request of the step before may be in flight
      }
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      stg = stg1;
      // block 3; among its MFMAs the reads of the next step's block 0 and weights, and the first loads of the request.  (After the
      // tile's last step these reads fetch the next tile's first fragments, which the epilogue's registers cannot keep: they
      // are dropped and read again by the next head.)
      const Frag& W0 = pb == 0 ? B00 : B10;
      const Frag& W1 = pb == 0 ? B01 : B11;
      STAMP_RD_AS0(sn + adrA0 + lane16, 0);
      mfma8(acc[3], As1, W0, W1, [&](auto i) __attribute__((always_inline)) {
        if constexpr (i.value == 2) {
          if constexpr (pb == 0) STAMP_RD_B10(sn + adrB0 + lane16);
          else STAMP_RD_B00(sn + adrB0 + lane16);
        }
        if constexpr (i.value == 4) {
          if constexpr (pb == 0) STAMP_RD_B11(sn + adrB0 + lane16);
          else STAMP_RD_B01(sn + adrB0 + lane16);
        }
        rq_issue(std::integral_constant<int, i.value / 2 - 1>{});
      });
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (HI) {
        auto more = [&](auto i) __attribute__((always_inline)) { rq_issue(std::integral_constant<int, 2 + i.value / 2>{}); };
        if (has_hi) {
          mfma8(acch, Hs, W0, W1, more);
        } else {
          more(std::integral_constant<int, 2>{});
          more(std::integral_constant<int, 4>{});
          more(std::integral_constant<int, 6>{});
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      rq_tail = true;  // the other loads follow among the MFMAs of the next step (or after the tile's last step)
    };
    // head of the tile: the barrier that published its first stage lies behind (prologue, or the last step of the
    // tile before)
    {
      lane16 = lane_now() * 16u;
      const uint32_t sh = lds0 + (uint32_t)(stg * kStage6);
      STAMP_RD_AS0(sh + adrA0 + lane16, 0);
      STAMP_RD_B00(sh + adrB0 + lane16);
      STAMP_RD_B01(sh + adrB0 + lane16);
    }
    for (int kt = 0; kt + 1 < KT; kt += 2) {
      step(std::integral_constant<int, 0>{});
      step(std::integral_constant<int, 1>{});
    }
    if (KT & 1) step(std::integral_constant<int, 0>{});
    if (rq_tail) rq_rest(std::integral_constant<int, kFirst>{});
    rq_tail = false;
    // the last step's look-ahead reads must have returned before their registers are used for anything else
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");

    // Everything requested so far (the next tile's first steps included) must have landed before the epilogue issues
    // its stores: the counter retires in order, so a later wait for a load would also wait for every store before
    // it.  The epilogue waits for that itself, after its lane swaps (the plain modes: before they start); after it
    // the next kNumStage6 - 1 steps therefore need no wait.
    landed = kNumStage6 - 1;
    // Per-lane values of the epilogue are derived from an opaque copy of the lane number, so that they are
    // computed here, once per tile, instead of being carried in registers across the main loop (which has none
    // to spare: a spilled value would be reloaded with a wait for all outstanding loads inside that loop).
    int lane_e = (int)lane_now(), tid_e = wave * 64 + lane_e;
    asm volatile("" : "+v"(lane_e), "+v"(tid_e));
    // the epilogue's operands from global memory: their latency passes under the lane swaps
    RegEpiOperands<EPI, (IS2D ? 2 * RB : RB), RAG> eo;
    if constexpr (EPI >= 1) eo.template request<!HI>(a, m0, nw, wm, lane_e);
    // row factors of the next tile: loaded now, written to the other buffer after the epilogue (a barrier of
    // the next tile's first step publishes them long before its epilogue reads them)
    float nfac = 0.0f, nrz = 0.0f;
    int ndst = -1;
    const bool has_next = pos + wx < count;
    if (has_next && tid_e < BMW) {
      int tm1, tn1;
      tile_of_sid(first + pos + wx, mt, nt, tm1, tn1);
      compute_row_info<Acc, EPI, RAG>(a, tm1 * BMW, tid_e, nfac, ndst, nrz);
    }
    if constexpr (HI) {
      if (has_next && tid_e >= BMW && tid_e < BMW + kHiPlaces) {
        int tm1, tn1;
        tile_of_sid(first + pos + wx, mt, nt, tm1, tn1);
        hi_place_info<RAG>(a, tm1, tid_e - BMW, nfac, nrz);
      }
    }
    const uint8_t* ri = row_info + rbuf * kRowInfo;
    if constexpr (EPI != 2) {
      // The loads just requested complete here, on every path and in a form the compiler's wait-count bookkeeping
      // sees: a load it believed pending at the end of the tile would make it wait for ALL loads inside the next
      // main loop.  (The fused epilogue places this wait after its lane swaps.)
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    }
    if constexpr (HI) {
      // (their loads have landed: eo.sw, eo.cs)
      if (has_hi) hi_block_sums<(IS2D ? 2 * RB : RB), YBF16, SYM, RAG>(a, acch, reinterpret_cast<const float*>(ri + kHiInfo), eo, tm, nw, lane_e);
    }
    if constexpr (EPI >= 1) {
      epilogue_reg<EPI, RB, IS2D, YBF16, NI, 0, SYM, RAG, ODD>(a, acc, ri, eo, m0, nw, wm, lane_e);
    } else {
      EpiOperands<EPI, RB, IS2D> none;
      v16f accv[4][NIW];
#pragma unroll
      for (int mi = 0; mi < 4; ++mi)
#pragma unroll
        for (int ni = 0; ni < NIW; ++ni) {
          float r[16];
#pragma unroll
          for (int v = 0; v < 16; ++v) r[v] = acc[mi][ni][v];
          columns16(r);
#pragma unroll
          for (int v = 0; v < 16; ++v) accv[mi][ni][v] = r[v];
        }
      epilogue<Acc, EPI, RB, IS2D, YBF16, true>(a, accv, smem, ri, none, m0, n0, lane_e, wave, wm, wn);
    }
    rbuf ^= 1;
    if (has_next && tid_e < BMW) write_row_info(row_info + rbuf * kRowInfo, tid_e, nfac, ndst, nrz);
    if constexpr (HI) {
      if (has_next && tid_e >= BMW && tid_e < BMW + kHiPlaces) {
        float* t = reinterpret_cast<float*>(row_info + rbuf * kRowInfo + kHiInfo) + tid_e - BMW;
        t[0] = nfac;
        t[kHiPlaces] = nrz;
      }
    }
  }
}

#ifdef STAMP_GEMM6_PAIR
constexpr bool kPair = true;
#else
constexpr bool kPair = false;
#endif
// whether this file's kernels take the 8-bit rows along
#ifdef STAMP_GEMM6_HI
constexpr bool kHiTiles = true;
#else
constexpr bool kHiTiles = false;
#endif

int gemm6_workgroups(int tiles) {
  const int most = (kPair ? 2 : 1) * stamp_device_cus();
  return tiles < most ? tiles : most;
}

template <int EPI, int RB, bool IS2D, bool YBF16, bool SYM, bool RAG = false, bool ODD = false, bool HI = kHiTiles>
hipError_t launch_k(const GemmArgs& a, hipStream_t st) {
  constexpr int WAVES = STAMP_GEMM6_WAVES;
  constexpr size_t lds = (size_t)(kPair ? 2 : 3) * Tile6<WAVES, HI>::kStage + 2 * (kRowInfoBytes + (RAG ? 256 : 0) + (HI ? kHiInfoBytes : 0));
  static size_t lds_done[kStampMaxDevices] = {};
  hipError_t e = stamp_allow_lds(reinterpret_cast<const void*>(&k_gemm6<EPI, RB, IS2D, YBF16, SYM, RAG, ODD, WAVES, HI, kPair>), lds, lds_done);
  if (e != hipSuccess) return e;
  const int mt = (a.M + Tile6<WAVES>::BMW - 1) / Tile6<WAVES>::BMW, nt = a.Npad / BN6;
  hipLaunchKernelGGL((k_gemm6<EPI, RB, IS2D, YBF16, SYM, RAG, ODD, WAVES, HI, kPair>), dim3(gemm6_workgroups(mt * nt)), dim3(64 * WAVES), lds, st, a);
  return hipGetLastError();
}

template <int EPI, int RB, bool IS2D, bool YBF16>
hipError_t launch_y(const GemmArgs& a, hipStream_t st) {
  if constexpr (EPI == 2) {
    if (!a.g.asym) return launch_k<EPI, RB, IS2D, YBF16, true>(a, st);
  }
  return launch_k<EPI, RB, IS2D, YBF16, false>(a, st);
}

template <int EPI, int RB, bool IS2D>
hipError_t launch(const GemmArgs& a, hipStream_t st) {
  if constexpr (EPI >= 2) {
    if (a.g.y_bf16) return launch_y<EPI, RB, IS2D, true>(a, st);
  }
  return launch_y<EPI, RB, IS2D, false>(a, st);
}


template <int RB, bool ODD>
hipError_t launch_rag_n(const GemmArgs& a, hipStream_t st) {
  if (a.g.y_bf16) return a.g.asym ? launch_k<2, RB, false, true, false, true, ODD>(a, st) : launch_k<2, RB, false, true, true, true, ODD>(a, st);
  return a.g.asym ? launch_k<2, RB, false, false, false, true, ODD>(a, st) : launch_k<2, RB, false, false, true, true, ODD>(a, st);
}
template <int RB>
hipError_t launch_rag(const GemmArgs& a, hipStream_t st) {
  return (a.N & 1) ? launch_rag_n<RB, true>(a, st) : launch_rag_n<RB, false>(a, st);
}

// the GEMM of one mode on this tile size
hipError_t gemm6_run(const GemmArgs& a, int mode, hipStream_t st) {
#ifndef STAMP_GEMM6_HI
  if (mode == 1) return launch<1, 0, false>(a, st);
  if (mode == 3) return launch<3, 0, false>(a, st);
#endif
#if STAMP_GEMM6_WAVES == 8
  if (mode == 0) return launch<0, 0, false>(a, st);
#endif
  if (mode != 2) return hipErrorInvalidValue;
  if (a.rag.on) {
    switch (a.g.r) {
      case 3: return launch_rag<3>(a, st);
      case 4: return launch_rag<4>(a, st);
      case 5: return launch_rag<5>(a, st);
      case 6: return launch_rag<6>(a, st);
      default: return hipErrorInvalidValue;
    }
  }
  if (!a.g.is2d) {
    switch (a.g.r) {
      case 3: return launch<2, 3, false>(a, st);
      case 4: return launch<2, 4, false>(a, st);
      case 5: return launch<2, 5, false>(a, st);
      case 6: return launch<2, 6, false>(a, st);
      default: return hipErrorInvalidValue;
    }
  }
  switch (a.g.r) {
    case 2: return launch<2, 2, true>(a, st);
    case 3: return launch<2, 3, true>(a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

#endif  // STAMP_GEMM6_KERNEL_H_
