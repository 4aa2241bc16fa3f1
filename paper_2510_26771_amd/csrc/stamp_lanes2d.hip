// Bottom kernel of a token grid by lanes: 4 x 4 and 8 x 8 blocks -> FP6 operands (stamp_lanes1d.hip has the form on a line).
//
// A lane holds 32 channels of a cell of 2 x 2 tokens: three finished rows and the cell's sum; each level above adds and subtracts
// from lane to lane, along x and then along y, and leaves its four outcomes in the four lanes of a cell.  So a lane ends with four
// rows, a block's rows meet in one exchange of maxima, one barrier.  Same operations on the same values as k_bottom2d, same codes.
// What bounds it: the vector ALU of the CUs that have a block (8 x 8 blocks of 1152 channels: nine waves, 1800 instructions each).
// 2 x 4096 tokens x 1152 in 8 x 8 blocks 15.7 us (18.3 with the sub-blocks side by side and 8 channels a thread).  Layers, us,
// that form or packed codes against this: 32 x 4096 x 512 -> 512 92.3, 79.9, 64 x 4096 x 256 135, 105; 4 x 4 blocks 64 x 256 x 64 26.4,
// 18.5, 2 x 4096 x 4096 70.1, 53.4.
#include "stamp_lanes.h"

namespace {

// bit of a lane's index -> its partner's value
template <int bit>
__device__ __forceinline__ float across(float x) {
  if constexpr (bit < 3) return partner<bit + 2>(x);
  else return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xF, 0xF, true));  // row_ror 8
}

// 768 threads: three waves per SIMD have 168 registers each, which four rows of 32 channels need
template <int RLOG, bool BF16, bool ASYM>
__global__ __launch_bounds__(768) void k_lanes2d(const LaneArgs a) {
  constexpr int GB = 1 << RLOG, RK = GB * GB, NL = RK / 4, CPR = BF16 ? 4 : 8;  // block edge, tokens, lanes per group of channels
  constexpr int G1 = GB / 2, G2 = GB / 4;
  __shared__ __attribute__((aligned(16))) uint32_t s_max[2][RK][16];  // [sign][row][wave]
  extern __shared__ __attribute__((aligned(16))) uint8_t s_row[];     // the x differences, [8][threads] 16 bytes
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = (int)(blockDim.x >> 6);
  const int tl = lane & (NL - 1), b = blockIdx.y, j = unit_of_block<RLOG == 3 ? 64 : 16>(blockIdx.x, gridDim.x), by = j / a.G, bx = j - by * a.G;
  // cell (qx, qy) of the block: bits 0, 2 and 1, 3 of the lane
  const int qx = (tl & 1) | ((tl >> 1) & 2), qy = ((tl >> 1) & 1) | ((tl >> 2) & 2);
  const size_t seq0 = (size_t)b * a.s;
  const int c = (wave * (64 / NL) + lane / NL) * 32;
  const bool active = c < a.d;
  const uint8_t* src = reinterpret_cast<const uint8_t*>(a.X) +
                       ((seq0 + (size_t)(by * GB + 2 * qy) * a.gridW + bx * GB + 2 * qx) * a.d + min(c, a.d - 32)) * (BF16 ? 2 : 4);
  u4 raw[4][CPR];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const uint8_t* p = src + ((size_t)(t >> 1) * a.gridW + (t & 1)) * a.d * (BF16 ? 2 : 4);
#pragma unroll
    for (int h = 0; h < CPR; ++h) raw[t][h] = *reinterpret_cast<const u4*>(p + 16 * h);
  }
  float sg[4];  // sign of a lane's own value at a bit: + in the lower lane
#pragma unroll
  for (int i = 0; i < 4; ++i) sg[i] = (tl >> i) & 1 ? -1.0f : 1.0f;
  const bool cell_sum = (tl & 3) == 0;  // takes part in the third level
  // x difference (in LDS: four rows do not fit the registers beside their codes), y difference, both, the lane's row of a level above
  float row[4][32];
  RowMax<ASYM> mx[4];
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    if ((i & 7) == 0) __builtin_amdgcn_sched_barrier(0);  // the loaded words give way to the rows
    float x[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if constexpr (BF16) x[t] = (i & 1) ? bf16hi(raw[t][i >> 3][(i >> 1) & 3]) : bf16lo(raw[t][i >> 3][(i >> 1) & 3]);
      else x[t] = __uint_as_float(raw[t][BF16 ? 0 : i >> 2][i & 3]);
    }
    const float t0 = __fadd_rn(x[0], x[1]), t1 = __fsub_rn(x[0], x[1]), t2 = __fadd_rn(x[2], x[3]), t3 = __fsub_rn(x[2], x[3]);
    float s = __fadd_rn(t0, t2);
    row[0][i] = __fadd_rn(t1, t3);
    row[1][i] = __fsub_rn(t0, t2);
    row[2][i] = __fsub_rn(t1, t3);
    // lower lane: own + partner's, upper lane: partner's - own (the product is exact)
    s = __builtin_fmaf(s, sg[0], across<0>(s));
    s = __builtin_fmaf(s, sg[1], across<1>(s));
    if constexpr (RLOG == 3) {
      float r = __builtin_fmaf(s, sg[2], across<2>(s));
      r = __builtin_fmaf(r, sg[3], across<3>(r));
      s = cell_sum ? r : s;
    }
    row[3][i] = s;
    // made here, not where they are used: two values would wait for each of them
    asm volatile("" : "+v"(row[1][i]), "+v"(row[2][i]), "+v"(row[3][i]));
#pragma unroll
    for (int q = 0; q < 4; ++q) mx[q].template add<false>(i, row[q][i]);
    if ((i & 3) == 3)
      *reinterpret_cast<float4*>(s_row + ((i >> 2) * (int)blockDim.x + tid) * 16) = make_float4(row[0][i - 3], row[0][i - 2], row[0][i - 1], row[0][i]);
  }
  // lanes beyond d_in hold duplicates of the last channels, which change no magnitude; the asymmetric form's keys must not see them
  const bool live = !ASYM || active;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t pos = across_groups<NL>(live ? mx[q].pos() : 0u);
    uint32_t neg = 0u;
    if constexpr (ASYM) neg = across_groups<NL>(live ? mx[q].neg() : 0u);
    if (lane < NL) {
      s_max[0][q * NL + tl][wave] = pos;
      if constexpr (ASYM) s_max[1][q * NL + tl][wave] = neg;
    }
  }
  __syncthreads();
  const bool sum_out = a.abot != nullptr, row8 = !sum_out && j < a.khi;  // (uniform)
  const float nrm3 = cell_sum ? 1.0f / GB : 0.25f;
  const int e3 = cell_sum ? tl >> 2 : G2 * G2 * (tl & 3) + (RLOG == 3 ? (qy >> 1) * G2 + (qx >> 1) : 0);
  const size_t brow = seq0 + (size_t)j * RK;
  uint8_t* const out = a.a6 + (brow >> 8) * (size_t)a.KT * kStageA6 + chan_off6((uint32_t)c, kStageA6);
#pragma unroll
  for (int o = 0; o < 4; ++o) {
    const int q = o == 2 ? 0 : (o == 3 ? 3 : o + 1);  // (8-bit rows need registers of their own: last)
    if (q == 0) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float4 v = *reinterpret_cast<const float4*>(s_row + (i * (int)blockDim.x + tid) * 16);
        row[0][4 * i] = v.x;
        row[0][4 * i + 1] = v.y;
        row[0][4 * i + 2] = v.z;
        row[0][4 * i + 3] = v.w;
      }
    }
    const int e = q < 3 ? G1 * G1 * (1 + q) + qy * G1 + qx : e3;
    const float nrm = q < 3 ? 0.5f : nrm3;
    const bool top = q == 3 && tl == 0;
    const float qmax = ASYM ? (top && row8 ? 255.0f : 15.0f) : (top && row8 ? 127.0f : 7.0f);
    float scale, inv, z;
    if constexpr (ASYM)
      row_params<true>(__fmul_rn(fkey_inv(max_of_waves(s_max[0][q * NL + tl], nw)), nrm),
                       __fmul_rn(fkey_inv(max_of_waves(s_max[1][q * NL + tl], nw)), nrm), qmax, scale, inv, z);
    else
      row_params<false>(__fmul_rn(__uint_as_float(max_of_waves(s_max[0][q * NL + tl], nw)), nrm), 0.0f, qmax, scale, inv, z);
    if (tid < NL && !(top && sum_out)) {
      a.scales[brow + e] = scale;
      if constexpr (ASYM) a.scales[a.zeros_off + brow + e] = z;
    }
    if (q == 3 && active && tl == 0) {
      if (sum_out) {
        float4* o = reinterpret_cast<float4*>(a.abot + ((size_t)b * a.k + j) * a.d + c);
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] = make_float4(row[q][4 * i], row[q][4 * i + 1], row[q][4 * i + 2], row[q][4 * i + 3]);
      } else if (row8) {
        const float qlo = ASYM ? 0.0f : -127.0f, qhi = ASYM ? 255.0f : 127.0f, shift = ASYM ? 128.0f : 0.0f;
        f16v qe, qo;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          qe[i] = fminf(fmaxf(__fadd_rn(rintf(__fmul_rn(__fmul_rn(row[q][2 * i], nrm), inv)), z), qlo), qhi) - shift;
          qo[i] = fminf(fmaxf(__fadd_rn(rintf(__fmul_rn(__fmul_rn(row[q][2 * i + 1], nrm), inv)), z), qlo), qhi) - shift;
        }
        store_hi24(a.hi6, b * a.khi + j, a.KT, qe, qo, c);
      }
    }
    const float mul = __fmul_rn(inv, nrm);  // a power of two
    f16v ev, od;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float p = __fmul_rn(row[q][2 * i], mul), r = __fmul_rn(row[q][2 * i + 1], mul);
      ev[i] = ASYM ? __builtin_amdgcn_fmed3f(__fadd_rn(rintf(p), z - 8.0f), -8.0f, 7.0f) : p;
      od[i] = ASYM ? __builtin_amdgcn_fmed3f(__fadd_rn(rintf(r), z - 8.0f), -8.0f, 7.0f) : r;
    }
    const u6v w = to_e2m3(ev, od);
    const uint32_t m = (uint32_t)(brow & 255) + (uint32_t)e;
    if (active && !(top && (sum_out || row8))) store24(out + row_off6(m, 2 * RLOG), w, row_half6(m, 2 * RLOG));
    __builtin_amdgcn_sched_barrier(0);
  }
}

template <int RLOG, bool BF16, bool ASYM>
hipError_t launch2d_(const LaneArgs& a, int waves, int B, hipStream_t st) {
  static size_t lds_done[kStampMaxDevices] = {};
  const size_t lds = (size_t)waves * 64 * 128;
  const hipError_t e = stamp_allow_lds(reinterpret_cast<const void*>(&k_lanes2d<RLOG, BF16, ASYM>), lds, lds_done);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_lanes2d<RLOG, BF16, ASYM>), dim3(a.k, B), dim3(waves * 64), lds, st, a);
  return hipGetLastError();
}
template <int RLOG>
hipError_t launch2d(const LaneArgs& a, int x_bf16, int asym, int B, hipStream_t st) {
  constexpr int CW = 64 / (1 << (2 * RLOG - 2)) * 32;  // channels of a wave
  const int waves = (a.d + CW - 1) / CW;
  if (waves > 12) return hipErrorInvalidValue;
  if (x_bf16) return asym ? launch2d_<RLOG, true, true>(a, waves, B, st) : launch2d_<RLOG, true, false>(a, waves, B, st);
  return asym ? launch2d_<RLOG, false, true>(a, waves, B, st) : launch2d_<RLOG, false, false>(a, waves, B, st);
}

}  // namespace

// The channels that 12 waves hold.  4 x 4 blocks below top levels, layers to 256 outputs, us, packed codes that are converted beside
// these levels against this: 2 x 64 tokens x 160 26.1, 24.8, 64 x 256 x 512 37.4, 36.9, 128 x 256 x 1152 73.9, 67.0, 32 x 1024 x 1152 73.2,
// 66.9, 128 x 256 x 2048 100.3, 92.9; not narrow layers of more than 4096 blocks (128 x 1024 x 64 81.8, 87.9, x 160 90.5, 93.8; x 512 118.6,
// 115.9), whose conversion is small, nor wide ones of few blocks (256 x 4096 44.0, 44.8, 4 x 1024 x 2048 44.2, 44.4).
bool stamp_lanes2d_fits(const stamp_plan* p) {
  const StampGeom& g = p->geom;
  if (!g.is2d || g.ident || g.d > (g.r == 3 ? 1536 : 4096)) return false;
  if (g.r == 3 || g.L == 0) return true;
  const int64_t blocks = (int64_t)g.B * g.k;
  return g.d <= 1536 ? blocks <= 4096 || g.d >= 512 : blocks >= 256;
}

hipError_t stamp_launch_lanes2d(const stamp_plan* p, const void* X, uint8_t* a6, float* scales, float* abot, const StampHiOut& hi, hipStream_t st) {
  const StampGeom& g = p->geom;
  LaneArgs a = {};
  a.X = X;
  a.a6 = a6;
  a.scales = scales;
  a.abot = abot;
  a.s = g.s;
  a.d = g.d;
  a.k = g.k;
  a.khi = g.khi;
  a.KT = p->Kpad >> 7;
  a.zeros_off = (size_t)g.B * g.s;
  a.hi6 = hi;
  a.G = g.G;
  a.gridW = g.gridW;
  return g.r == 3 ? launch2d<3>(a, g.x_bf16, g.asym, g.B, st) : launch2d<2>(a, g.x_bf16, g.asym, g.B, st);
}
