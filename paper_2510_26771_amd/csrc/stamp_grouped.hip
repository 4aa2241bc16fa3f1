// Per-block scales (one per 64 channels, for activations and weights: the image-model setting) on the blocked 2-D Haar
// transform: quantizer, operand conversion, and the GEMM on the FP6 pipeline with the inverse transform in its epilogue.
//
//   Y'[m, n] = sum_g acc_g[m, n] * sa[m, g] * sw[g, n],   acc_g = sum over the 64 channels of group g of code * code
//
// One v_mfma_f32_32x32x64_f8f6f4 is exactly one group, and leaves acc_g / 64 exactly in fp32.  What bounds such a GEMM is the
// rescaling of every output once per group, on the vector ALU.  Here it is one vector instruction, acc += t * S with S = sa sw:
// the products S of two 32 x 32 blocks are one v_mfma_f32_32x32x1_2b_f32 (the outer product of the row and column scales,
// each product rounded once, as a vector multiplication would).  fp32 MFMAs run on the vector ALU (measured: next to
// v_fma_f32 in another wave both take the sum of their times, an FP6 MFMA next to it the longer one), but two blocks of
// products cost it 64 cycles there against 128 as vector multiplications.  Per two blocks and group: 64 + 128 cycles of the
// vector ALU, 64 of the matrix pipe; measured about 275 per SIMD.  8192 x 1152 x 4608 with the inverse in the epilogue:
// 66 us; the int8 kernel of the general path, three vector instructions per output and group and fp32 output, takes 124 us,
// its inverse passes 45 us.
#include "stamp_epilogue_reg.h"
#include "stamp_hi6.h"

namespace {

using namespace stamp_gemm;

typedef float v32f __attribute__((ext_vector_type(32)));

__device__ __forceinline__ float bf16lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// max over the 8 lanes that hold a group's 64 channels (non-negative floats order like their bit patterns)
__device__ __forceinline__ float max8(float a) {
  int x = (int)__float_as_uint(a), y;
  y = __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, false); x = max(x, y);   // quad_perm [1,0,3,2]
  y = __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, false); x = max(x, y);   // quad_perm [2,3,0,1]
  y = __builtin_amdgcn_update_dpp(0, x, 0x141, 0xF, 0xF, false); x = max(x, y);  // row_half_mirror
  return __uint_as_float((uint32_t)x);
}

// 8 channels of one coefficient row: range of the group, codes, scale (the arithmetic of the row quantizer, per group)
__device__ __forceinline__ void quant_row8(const float (&t)[8], float qmax, int8_t* code, float* scale_out, bool active, bool first) {
  float a = 0.0f;
#pragma unroll
  for (int c = 0; c < 8; ++c) a = fmaxf(a, fabsf(t[c]));
  a = max8(a);
  float scale = 0.0f, inv = 0.0f;
  if (a > 0.0f) {
    scale = __fdiv_rn(a, qmax);
    inv = __fdiv_rn(qmax, a);
  }
  uint32_t w[2] = {0u, 0u};
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const float q = fminf(fmaxf(rintf(__fmul_rn(t[c], inv)), -qmax), qmax);
    w[c >> 2] |= ((uint32_t)((int)q) & 0xFFu) << (8 * (c & 3));
  }
  if (active) *reinterpret_cast<uint2*>(code) = make_uint2(w[0], w[1]);
  if (active && first) *scale_out = scale;
}

// X -> codes and scales in STaMP order.  A wave takes 64 tokens (one 8 x 8 block, or four 4 x 4 blocks: RLOG 3 or 2) of
// 128 channels: a lane one 4 x 4 sub-block of 8 channels, held in registers; the third level of an 8 x 8 block exchanges
// the four sub-blocks' sums between lanes 16 and 32 apart.  Ranges are per 64 channels, i.e. over 8 lanes: no LDS, no
// barrier.  L > 0: the block sums go to abot for k_grp_top, else they are quantized here.  Bound by how many waves there
// are: B * s / 64 * d / 128 of them (2 x 4096 x 1152: 1152; 13 us, against 26 + 5 + 9 for level passes and quantizer).
template <int RLOG, bool BF16>
__global__ __launch_bounds__(256) void k_grp_quant(const void* __restrict__ X, int8_t* __restrict__ codes, float* __restrict__ scales,
                                                   float* __restrict__ abot, const StampGeom g, int KT, int nwaves) {
  const int wid = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (wid >= nwaves) return;
  const int lane = threadIdx.x & 63, oct = lane & 15, sb = lane >> 4;
  const int unit = wid / KT, kt = wid - unit * KT;  // 64 physical rows, 128 channels
  const int row0 = unit * 64, b = row0 / g.s, pr0 = row0 - b * g.s;
  const int j = RLOG == 3 ? pr0 / 64 : pr0 / 16 + sb;
  const int bi = j / g.G, bj = j - bi * g.G;
  const int sby = RLOG == 3 ? sb >> 1 : 0, sbx = RLOG == 3 ? sb & 1 : 0;
  const int d = g.d, c0 = kt * 128 + oct * 8;
  const bool active = c0 < d, first = (oct & 7) == 0;
  const int cl = min(c0, d - 8), ng = d >> 6;
  const size_t seq0 = (size_t)b * g.s;
  const size_t tok0 = seq0 + (size_t)((bi << RLOG) + 4 * sby) * g.gridW + (size_t)((bj << RLOG) + 4 * sbx);
  constexpr int WPT = BF16 ? 1 : 2;
  uint4 raw[16][WPT];
#pragma unroll
  for (int t = 0; t < 16; ++t) {
    const int ci = t >> 2, q = t & 3;
    const size_t e = (tok0 + (size_t)(2 * (ci >> 1) + (q >> 1)) * g.gridW + (2 * (ci & 1) + (q & 1))) * d + cl;
#pragma unroll
    for (int h = 0; h < WPT; ++h)
      raw[t][h] = BF16 ? *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(X) + e)
                       : *reinterpret_cast<const uint4*>(reinterpret_cast<const float*>(X) + e + 4 * h);
  }
  // level l, in-block position e -> slot, norm 2^-l (exact)
  auto emit = [&](float (&v)[8], int level, int e, float qmax) __attribute__((always_inline)) {
    const int slot = e == 0 ? j : stamp_slot_of_block_e_2d(bi, bj, e, g.G);
    const float nrm = ldexpf(1.0f, -level);
#pragma unroll
    for (int c = 0; c < 8; ++c) v[c] = __fmul_rn(v[c], nrm);
    quant_row8(v, qmax, codes + (seq0 + slot) * d + c0, scales + (seq0 + slot) * ng + (c0 >> 6), active, first);
  };
  constexpr int g1 = 1 << (RLOG - 1), g2 = 1 << (RLOG - 2);
  float ll1[4][8], band[3][8];
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
        t[q][0] = __uint_as_float(w0.x); t[q][1] = __uint_as_float(w0.y); t[q][2] = __uint_as_float(w0.z); t[q][3] = __uint_as_float(w0.w);
        t[q][4] = __uint_as_float(w1.x); t[q][5] = __uint_as_float(w1.y); t[q][6] = __uint_as_float(w1.z); t[q][7] = __uint_as_float(w1.w);
      }
    }
    cell2d(t[0], t[1], t[2], t[3], ll1[ci], band[0], band[1], band[2]);
#pragma unroll
    for (int bd = 0; bd < 3; ++bd)
      emit(band[bd], 1, g1 * g1 * (1 + bd) + (2 * sby + (ci >> 1)) * g1 + 2 * sbx + (ci & 1), 7.0f);
  }
  float ll2[8];
  cell2d(ll1[0], ll1[1], ll1[2], ll1[3], ll2, band[0], band[1], band[2]);
#pragma unroll
  for (int bd = 0; bd < 3; ++bd) emit(band[bd], 2, g2 * g2 * (1 + bd) + sby * g2 + sbx, 7.0f);
  int e_top = 0;
  if constexpr (RLOG == 3) {
    // lanes (sby, sbx) hold p, q, u, v of the last cell: t0 = p + q, t1 = p - q, t2 = u + v, t3 = u - v across sbx, then
    // t0 + t2, t1 + t3 (lower lanes), t0 - t2, t1 - t3 (upper lanes) across sby: lane (dy, dx) ends with one coefficient
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const float o = __shfl_xor(ll2[c], 16, 64);
      const float t = sbx ? __fsub_rn(o, ll2[c]) : __fadd_rn(ll2[c], o);
      const float u = __shfl_xor(t, 32, 64);
      ll2[c] = sby ? __fsub_rn(u, t) : __fadd_rn(t, u);
    }
    e_top = sby ? (sbx ? 3 : 2) : sbx;  // W, H, D at 1, 2, 3
  }
  if (g.L > 0 && e_top == 0) {
    if (active) {
      float4* o = reinterpret_cast<float4*>(abot + ((size_t)b * g.k + j) * d + c0);
      o[0] = make_float4(ll2[0], ll2[1], ll2[2], ll2[3]);
      o[1] = make_float4(ll2[4], ll2[5], ll2[6], ll2[7]);
    }
  } else {
    emit(ll2, RLOG, e_top, (e_top == 0 && j < g.khi) ? 127.0f : 7.0f);
  }
}

// The top L levels over the G x G block sums of a sequence, G waves per 64 channels (a group), lane = channel: every wave
// holds and transforms all of them in registers, and quantizes one line of G; the group's range is the wave's.  All of them
// are 8-bit rows.  Bound by the chain of a row's quantization: with one wave for all 64 rows 23.2 us (8 x 8, 2 x 640
// channels), now 5.9.
template <int G>
__global__ __launch_bounds__(64 * G) void k_grp_top(const float* __restrict__ abot, int8_t* __restrict__ codes, float* __restrict__ scales,
                                                const StampGeom g) {
  const int lane = threadIdx.x & 63, line = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int gr = blockIdx.x, b = blockIdx.y, d = g.d, c = gr * 64 + lane;
  float v[G][G];
  const float* src = abot + (size_t)b * (G * G) * d + c;
#pragma unroll
  for (int y = 0; y < G; ++y)
#pragma unroll
    for (int x = 0; x < G; ++x) v[y][x] = src[(size_t)(y * G + x) * d];
#pragma unroll
  for (int st = 2; st <= G; st <<= 1) {
    if (st <= (1 << g.L)) {
      const int h = st >> 1;
#pragma unroll
      for (int y = 0; y < G; y += st)
#pragma unroll
        for (int x = 0; x < G; x += st) {
          const float p = v[y][x], q = v[y][x + h], u = v[y + h][x], w = v[y + h][x + h];
          const float t0 = __fadd_rn(p, q), t1 = __fsub_rn(p, q), t2 = __fadd_rn(u, w), t3 = __fsub_rn(u, w);
          v[y][x] = __fadd_rn(t0, t2);
          v[y][x + h] = __fadd_rn(t1, t3);
          v[y + h][x] = __fsub_rn(t0, t2);
          v[y + h][x + h] = __fsub_rn(t1, t3);
        }
    }
  }
  const size_t row0 = (size_t)b * g.s;
#pragma unroll
  for (int y = 0; y < G; ++y) {
    if (y != line) continue;
#pragma unroll
    for (int x = 0; x < G; ++x) {
      int lvl;
      const int slot = stamp_top_slot_2d(y, x, G, g.L, &lvl);
      const float t = __fmul_rn(v[y][x], ldexpf(1.0f, -(g.r + lvl)));
      float a = fabsf(t);
#pragma unroll
      for (int sh = 1; sh < 64; sh <<= 1) a = fmaxf(a, __shfl_xor(a, sh, 64));
      float scale = 0.0f, inv = 0.0f;
      if (a > 0.0f) {
        scale = __fdiv_rn(a, 127.0f);
        inv = __fdiv_rn(127.0f, a);
      }
      const float q = fminf(fmaxf(rintf(__fmul_rn(t, inv)), -127.0f), 127.0f);
      codes[(row0 + slot) * d + c] = (int8_t)(int)q;
      if (lane == 0) scales[(row0 + slot) * (d >> 6) + gr] = scale;
    }
  }
}

// Codes and scales in STaMP order -> FP6 operands in block order.  4-bit rows: codes as in stamp_gemm6.hip, scales
// (times the norm of the row's level and the 64 of the operand format, both powers of two) [M tile][K step][256 rows][2
// groups]; rows that are not in this GEMM (8-bit block sums) get scale 0.  8-bit rows: stamp_hi6.h, scales alike.
// One thread per 32 channels of a row.
struct GrpPack {
  const int8_t* codes;
  const float* scales;
  uint8_t *a6, *h6;
  float *sa, *sh;
  StampGeom g;
  int KT, M, own, hi_used, np, nhi;  // nhi: threads of the 8-bit rows
};
__device__ __forceinline__ void load_codes32(const int8_t* q, u4 (&w)[2]) {
  w[0] = reinterpret_cast<const u4*>(q)[0];
  w[1] = reinterpret_cast<const u4*>(q)[1];
}
__device__ __forceinline__ f2 row_scales(const GrpPack& q, size_t row, int kt, float f) {
  const int ng = q.g.d >> 6;
  const float* s = q.scales + row * ng + 2 * kt;
  return f2{s[0] * f, 2 * kt + 1 < ng ? s[1] * f : 0.0f};
}
__global__ __launch_bounds__(256) void k_grp_pack(const GrpPack q) {
  const StampGeom& g = q.g;
  int i = blockIdx.x * 256 + threadIdx.x;
  const int nhi = (q.nhi + 255) / 256 * 256;
  u4 w[2] = {};
  f16v ev, od;
  if (i < nhi) {
    if (i >= q.nhi) return;
    const int nf = q.KT * 4, m = i / nf, frag = i - m * nf, kt = frag >> 2, f = frag & 3;
    const int gr = 32 * q.np, grp = m / gr, r = m - grp * gr, Mh = g.B * q.hi_used;
    const int b = m / q.hi_used, slot = m - b * q.hi_used;
    const bool there = m < Mh;
    const size_t row = (size_t)b * g.s + slot;
    if (there && frag * 32 < g.d) load_codes32(q.codes + row * g.d + frag * 32, w);
    codes32(w, ev, od);
    u6v h, l;
    split_hi(ev, od, h, l);
    uint8_t* dst = q.h6 + ((size_t)grp * q.KT + kt) * (2 * q.np * kBlock6) + (r >> 5) * (2 * kBlock6) + (f & 1) * 512 + (r & 31) * 16;
    store24(dst, h, f >> 1);
    store24(dst + kBlock6, l, f >> 1);
    if (f == 0) {
      f2 s = {0.0f, 0.0f};
      if (there) s = row_scales(q, row, kt, ldexpf(64.0f, -stamp_level_of_top_slot(slot, g.k, g.G, 1, g.r, g.L)));
      *reinterpret_cast<f2*>(q.sh + (((size_t)grp * q.KT + kt) * gr + r) * 2) = s;
    }
    return;
  }
  // consecutive threads: the four fragments of a row, then the rows of a tile
  i -= nhi;
  const int f = i & 3, row = (i >> 2) & 255, tk = i >> 10, mt = tk / q.KT, kt = tk - mt * q.KT;
  const int m = mt * 256 + row;
  f2 s = {0.0f, 0.0f};
  if (m < q.M) {
    const int b = m / g.s, pr = m - b * g.s, j = pr / g.R, e = pr - j * g.R;
    if (e != 0 || (q.own && j >= g.khi)) {
      const int slot = e == 0 ? j : stamp_slot_of_block_e_2d(j / g.G, j % g.G, e, g.G);
      const size_t r = (size_t)b * g.s + slot;
      if (kt * 128 + f * 32 < g.d) load_codes32(q.codes + r * g.d + kt * 128 + f * 32, w);
      if (f == 0) s = row_scales(q, r, kt, ldexpf(64.0f, -(e == 0 ? g.r : stamp_level_of_e_2d(e, g.r))));
    }
  }
  codes32(w, ev, od);
  store24(q.a6 + (size_t)tk * kStageA6 + (row >> 5) * kBlock6 + (f & 1) * 512 + (row & 31) * 16, to_e2m3(ev, od), f >> 1);
  if (f == 0) *reinterpret_cast<f2*>(q.sa + ((size_t)tk * 256 + row) * 2) = s;
}

// plan time: codes [Npad][d] int8 and scales [d / 64][Npad] -> FP6 operand (columns in pairs, as in k_w_quant6) and
// [Npad256 / 128][K step][4 blocks][32 columns][2 groups]; thread = (column, 32-channel fragment)
__global__ __launch_bounds__(256) void k_grp_wpack(const int8_t* __restrict__ qw, const float* __restrict__ sw, uint8_t* __restrict__ b6,
                                                   float* __restrict__ swp, int d, int Npad, int Npad256, int KT) {
  const int n = blockIdx.x * 256 + threadIdx.x, frag = blockIdx.y, kt = frag >> 2, f = frag & 3;
  if (n >= Npad256) return;
  u4 w[2] = {};
  f16v ev, od;
  if (n < Npad && frag * 32 < d) load_codes32(qw + (size_t)n * d + frag * 32, w);
  codes32(w, ev, od);
  const int blk = ((n & 127) >> 6) * 2 + (n & 1), r = (n & 63) >> 1;
  const size_t tk = (size_t)(n >> 7) * KT + kt;
  store24(b6 + tk * kStageB6 + (size_t)blk * kBlock6 + (f & 1) * 512 + r * 16, to_e2m3(ev, od), f >> 1);
  if (f == 0) {
    const int ng = d >> 6, g0 = 2 * kt;
    f2 s = {0.0f, 0.0f};
    if (n < Npad) s = f2{sw[(size_t)g0 * Npad + n], g0 + 1 < ng ? sw[(size_t)(g0 + 1) * Npad + n] : 0.0f};
    *reinterpret_cast<f2*>(swp + (tk * 128 + blk * 32 + r) * 2) = s;
  }
}

// The GEMM over the 4-bit rows.  256 x 128 outputs per workgroup, 4 waves of 128 x 64 = 4 x 2 blocks, two workgroups per CU.
// A K step (codes of both operands and their scales: 39 KB, images as in memory) is staged by asynchronous copies while the
// one before is multiplied.  The registers are full: accumulators (128), group results (32), scale products (32), fragments (48).  (Reading them straight
// from memory instead, without LDS: 86 us against 66 at 8192 x 1152 x 4608: every block waited for its loads.)
struct GrpGemm {
  GemmArgs a;
  const float *sa, *sw;
};
constexpr int kGrpSA = kStageA6, kGrpB = kGrpSA + 256 * 2 * 4, kGrpSW = kGrpB + kStageB6, kGrpStage = kGrpSW + 128 * 2 * 4;

// Fragments live in fixed registers (the three 16-byte parts of a fragment must land in 12 consecutive ones, see
// stamp_gemm6.hip): two activation sets, block i + 1 is read while block i is multiplied, and the two weight blocks.  Reads
// and waits are written by hand (the compiler would make an ordinary LDS read wait for the copies in flight); a wait names
// what it covers, which keeps the uses behind it.
struct GFrag {
  u6 h0, h1;
};
#define GRP_RD(f, sc, H0, H1, SC, P0, P1, P2, adr, sadr, off, soff)                                                                      \
  asm volatile("ds_read_b128 " P0 ", %3 offset:%5\n\tds_read_b128 " P1 ", %3 offset:%6\n\tds_read_b128 " P2                             \
               ", %3 offset:%7\n\tds_read_b64 " SC ", %4 offset:%8"                                                                      \
               : "=&{" H0 "}"(f.h0), "=&{" H1 "}"(f.h1), "=&{" SC "}"(sc)                                                                \
               : "v"(adr), "v"(sadr), "n"(off), "n"((off) + kPart), "n"((off) + 2 * kPart), "n"(soff))
#define GRP_WAIT(f, sc, H0, H1, SC) \
  asm volatile("s_waitcnt lgkmcnt(0)" : "={" H0 "}"(f.h0), "={" H1 "}"(f.h1), "={" SC "}"(sc) : "0"(f.h0), "1"(f.h1), "2"(sc))
#define GRP_A0 "v[208:213]", "v[214:219]", "v[200:201]"
#define GRP_A1 "v[220:225]", "v[226:231]", "v[202:203]"
#define GRP_B0 "v[232:237]", "v[238:243]", "v[204:205]"
#define GRP_B1 "v[244:249]", "v[250:255]", "v[206:207]"
#define GRP_RD_X(...) GRP_RD(__VA_ARGS__)
#define GRP_WAIT_X(...) GRP_WAIT(__VA_ARGS__)
#define GRP_RD_A0(i) GRP_RD_X(fa0, sa0, GRP_A0, "v[208:211]", "v[212:215]", "v[216:219]", aA, aS, (i) * kBlock6, (i) * 256)
#define GRP_RD_A1(i) GRP_RD_X(fa1, sa1, GRP_A1, "v[220:223]", "v[224:227]", "v[228:231]", aA, aS, (i) * kBlock6, (i) * 256)
#define GRP_RD_B0() GRP_RD_X(fb0, sw, GRP_B0, "v[232:235]", "v[236:239]", "v[240:243]", aB, aW, 0, 0)
#define GRP_RD_B1() GRP_RD_X(fb1, sw1, GRP_B1, "v[244:247]", "v[248:251]", "v[252:255]", aB, aW, kBlock6, 0)

template <int RB, bool YBF16>
__global__ __launch_bounds__(256, 2) void k_gemm6_grp(const GrpGemm ga) {
  const GemmArgs& a = ga.a;
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1, l32 = lane & 31, kg = lane >> 5;
  const int KT = a.Kpad / BK;
  int tm, tn;
  tile_of_block(a.M, (a.N + 127) / 128 * 128, 128, tm, tn);
  const int m0 = tm * BM, nw = tn * 128 + wn * 64;
  const uint8_t *gA = a.A + (size_t)tm * KT * kStageA6, *gB = a.Bq + (size_t)tn * KT * kStageB6;
  const uint8_t *gSA = reinterpret_cast<const uint8_t*>(ga.sa) + (size_t)tm * KT * 2048,
                *gSW = reinterpret_cast<const uint8_t*>(ga.sw) + (size_t)tn * KT * 1024;
  auto copy = [&](const uint8_t* src, uint8_t* dst) __attribute__((always_inline)) {  // 1 KB per wave
    __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)(src + lane * 16),
                                     (void __attribute__((address_space(3)))*)dst, 16, 0, 0);
  };
  auto request = [&](int kt, int stg) __attribute__((always_inline)) {
    uint8_t* so = smem + stg * kGrpStage;
    const uint8_t *sA = gA + (size_t)kt * kStageA6 + wave * 1024, *sB = gB + (size_t)kt * kStageB6 + wave * 1024;
#pragma unroll
    for (int i = 0; i < kStageA6 / 4096; ++i) copy(sA + i * 4096, so + i * 4096 + wave * 1024);
#pragma unroll
    for (int i = 0; i < kStageB6 / 4096; ++i) copy(sB + i * 4096, so + kGrpB + i * 4096 + wave * 1024);
    if (wave < 2) copy(gSA + (size_t)kt * 2048 + wave * 1024, so + kGrpSA + wave * 1024);
    else if (wave == 2) copy(gSW + (size_t)kt * 1024, so + kGrpSW);
  };
  request(0, 0);
  v16f acc[4][NI];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
  const v16f zero16 = {};
  const v32f zero32 = {};
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)smem;
  const uint32_t adrA = lds0 + (uint32_t)(wm * 4 * kBlock6 + lane * 16), adrS = lds0 + (uint32_t)(kGrpSA + (wm * 128 + l32) * 8);
  const uint32_t adrB = lds0 + (uint32_t)(kGrpB + wn * 2 * kBlock6 + lane * 16), adrW = lds0 + (uint32_t)(kGrpSW + ((wn * 2 + kg) * 32 + l32) * 8);
  for (int kt = 0; kt < KT; ++kt) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's copies of step kt have landed
    __builtin_amdgcn_s_barrier();        // everybody's have, and step kt - 1 has been read out
    asm volatile("" ::: "memory");
    if (kt + 1 < KT) request(kt + 1, (kt + 1) & 1);
    const uint32_t so = (uint32_t)((kt & 1) * kGrpStage);
    const uint32_t aA = adrA + so, aS = adrS + so, aB = adrB + so, aW = adrW + so;
    GFrag fa0, fa1, fb0, fb1;
    f2 sa0, sa1, sw, sw1;
    GRP_RD_A0(0);
    GRP_RD_B0();
    GRP_RD_B1();
    GRP_WAIT_X(fb0, sw, GRP_B0);
    GRP_WAIT_X(fb1, sw1, GRP_B1);
    // one block of rows: both halves of the step (groups) against both blocks of columns
    auto block = [&](const GFrag& fa, f2 sa, auto i_tag) __attribute__((always_inline)) {
      constexpr int i = decltype(i_tag)::value;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const v16f t0 = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(widen((v6i)(h ? fa.h1 : fa.h0)), widen((v6i)(h ? fb0.h1 : fb0.h0)), zero16,
                                                                        2, 2, 0, 0, 0, 0);
        const v16f t1 = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(widen((v6i)(h ? fa.h1 : fa.h0)), widen((v6i)(h ? fb1.h1 : fb1.h0)), zero16,
                                                                        2, 2, 0, 0, 0, 0);
        // block 0 from lanes 0..31, block 1 from lanes 32..63
        __builtin_amdgcn_sched_barrier(0);
        const v32f S = __builtin_amdgcn_mfma_f32_32x32x1f32(sa[h], sw[h], zero32, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][0][v] = __builtin_fmaf(t0[v], S[v], acc[i][0][v]);
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][1][v] = __builtin_fmaf(t1[v], S[16 + v], acc[i][1][v]);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    GRP_WAIT_X(fa0, sa0, GRP_A0);
    GRP_RD_A1(1);
    block(fa0, sa0, std::integral_constant<int, 0>{});
    GRP_WAIT_X(fa1, sa1, GRP_A1);
    GRP_RD_A0(2);
    block(fa1, sa1, std::integral_constant<int, 1>{});
    GRP_WAIT_X(fa0, sa0, GRP_A0);
    GRP_RD_A1(3);
    block(fa0, sa0, std::integral_constant<int, 2>{});
    GRP_WAIT_X(fa1, sa1, GRP_A1);
    block(fa1, sa1, std::integral_constant<int, 3>{});
  }
  RegEpiOperands<2, 2 * RB, false, true> eo;
  eo.request(a, m0, nw, wm, lane);
  eo.sw = f2{1.0f, 1.0f};
  epilogue_reg_impl<2, RB, true, YBF16, true, NI, 0, true, false, true>(a, acc, nullptr, eo, m0, nw, wm, lane);
}

template <int RB, bool YBF16>
hipError_t launch_grp(const GrpGemm& ga, hipStream_t st) {
  const int tiles = ((ga.a.M + BM - 1) / BM) * ((ga.a.N + 127) / 128);  // Npad may end in a tile without columns
  static size_t lds_done[kStampMaxDevices] = {};
  const hipError_t e = stamp_allow_lds(reinterpret_cast<const void*>(&k_gemm6_grp<RB, YBF16>), 2 * kGrpStage, lds_done);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_gemm6_grp<RB, YBF16>), dim3(tiles), dim3(256), 2 * kGrpStage, st, ga);
  return hipGetLastError();
}

template <int RLOG>
hipError_t launch_quant(const stamp_plan* p, const void* X, int8_t* codes, float* scales, float* abot, hipStream_t st) {
  const StampGeom& g = p->bgeom;
  const int KT = p->Kpad / 128, n = g.B * (g.s / 64) * KT;
  if (g.x_bf16) hipLaunchKernelGGL((k_grp_quant<RLOG, true>), dim3((n + 3) / 4), dim3(256), 0, st, X, codes, scales, abot, g, KT, n);
  else hipLaunchKernelGGL((k_grp_quant<RLOG, false>), dim3((n + 3) / 4), dim3(256), 0, st, X, codes, scales, abot, g, KT, n);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || g.L == 0) return e;
  const dim3 grid(g.d / 64, g.B);
  switch (g.G) {
    case 2: hipLaunchKernelGGL(k_grp_top<2>, grid, dim3(64 * 2), 0, st, abot, codes, scales, g); break;
    case 4: hipLaunchKernelGGL(k_grp_top<4>, grid, dim3(64 * 4), 0, st, abot, codes, scales, g); break;
    case 8: hipLaunchKernelGGL(k_grp_top<8>, grid, dim3(64 * 8), 0, st, abot, codes, scales, g); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

int grp_own(const stamp_plan* p) { return p->bgeom.L == 0 && p->bgeom.khi < p->bgeom.k; }
int grp_hi_rows(const stamp_plan* p) { return p->bgeom.B * (grp_own(p) ? p->bgeom.khi : p->bgeom.k); }
int grp_np(const stamp_plan* p) { return grp_hi_rows(p) <= 32 ? 1 : 2; }
size_t up256(size_t x) { return (x + 255) & ~size_t(255); }

}  // namespace

// scratch: [0] FP6 operand of the 4-bit rows, [1] their scales, [2] operand of the 8-bit rows, [3] their scales
void stamp_grp_bytes(const stamp_plan* p, size_t (&n)[4]) {
  const size_t KT = p->Kpad / 128, mt = p->Mpad / 256, gr = 32 * grp_np(p), hg = (grp_hi_rows(p) + gr - 1) / gr;
  n[0] = up256(mt * KT * kStageA6);
  n[1] = up256(mt * KT * 256 * 2 * sizeof(float));
  n[2] = up256(hg * KT * 2 * grp_np(p) * kBlock6);
  n[3] = up256(hg * KT * gr * 2 * sizeof(float));
}

hipError_t stamp_grp_plan_weights(stamp_plan* p, hipStream_t st) {
  const int N = p->geom.N, Npad = (N + 127) / 128 * 128, KT = p->Kpad / 128;
  hipError_t e = hipMalloc(reinterpret_cast<void**>(&p->qWg6_dev), (size_t)(p->Npad / 128) * KT * kStageB6);
  if (e != hipSuccess) return e;
  e = hipMalloc(reinterpret_cast<void**>(&p->swg6_dev), (size_t)(p->Npad / 128) * KT * 128 * 2 * sizeof(float));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_grp_wpack, dim3(p->Npad / 256, KT * 4), dim3(256), 0, st, p->qWg_dev, p->swg_dev, p->qWg6_dev, p->swg6_dev, p->geom.d,
                     Npad, p->Npad, KT);
  return hipGetLastError();
}

hipError_t stamp_launch_grp_quant(const stamp_plan* p, const void* X, int8_t* codes, float* scales, float* abot, hipStream_t st) {
  return p->bgeom.r == 3 ? launch_quant<3>(p, X, codes, scales, abot, st) : launch_quant<2>(p, X, codes, scales, abot, st);
}

hipError_t stamp_launch_grp_forward(const stamp_plan* p, const int8_t* codes, const float* scales, uint8_t* const (&buf)[4], float* P, void* Y,
                                    hipStream_t st) {
  const StampGeom& g = p->bgeom;
  GrpPack q = {};
  q.codes = codes;
  q.scales = scales;
  q.a6 = buf[0];
  q.sa = reinterpret_cast<float*>(buf[1]);
  q.h6 = buf[2];
  q.sh = reinterpret_cast<float*>(buf[3]);
  q.g = g;
  q.KT = p->Kpad / 128;
  q.M = g.B * g.s;
  q.own = grp_own(p);
  q.hi_used = q.own ? g.khi : g.k;
  q.np = grp_np(p);
  const int gr = 32 * q.np;
  q.nhi = (grp_hi_rows(p) + gr - 1) / gr * gr * q.KT * 4;
  const long total = (long)((q.nhi + 255) / 256) + (long)(p->Mpad / 256) * q.KT * 4;
  hipLaunchKernelGGL(k_grp_pack, dim3((unsigned)total), dim3(256), 0, st, q);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (grp_hi_rows(p) > 0) {
    e = stamp_launch_hi6_grp(p, buf[2], q.sh, P, q.own, st);
    if (e != hipSuccess) return e;
  }
  GrpGemm ga = {};
  ga.a = stamp_gemm_args(p, nullptr, Y);
  ga.a.A = buf[0];
  ga.a.Bq = p->qWg6_dev;
  ga.a.M = q.M;
  ga.a.P = P;
  ga.a.own_top = q.own;
  ga.a.g = g;
  ga.sa = q.sa;
  ga.sw = p->swg6_dev;
  if (g.r == 3) return g.y_bf16 ? launch_grp<3, true>(ga, st) : launch_grp<3, false>(ga, st);
  return g.y_bf16 ? launch_grp<2, true>(ga, st) : launch_grp<2, false>(ga, st);
}
