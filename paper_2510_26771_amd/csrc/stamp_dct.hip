// DCT-II of 512 to 4096 tokens (powers of two) and its inverse: an fp64 FFT in registers, LDS only to hand points from one
// thread to another.
//
// The steps are those of k_gen_dct_fft (stamp_general.hip): N = 2 M real tokens of a channel as M complex points, T = FFT of
// M points, then pairs (k, M - k) of T give four coefficients.  Here M = 16 x 16 x R, a thread holds 16 points: radix 16,
// exchange, radix 16, exchange, radix R (R = 1, 2, 4, 8).  A thread takes the last pass's butterflies j and 256 - j, so both
// points of every pair are its own; the inverse runs the same passes backwards.  Real and imaginary parts are exchanged one
// after the other, so that a workgroup needs 8 bytes of LDS per point and two workgroups of 2048 tokens share a CU: one loads
// while the other computes.
// What bounds it: the fp64 vector ALU (about 900 operations per 16 points and direction, 7 us for 2048 tokens x 4096 channels),
// beside rows that arrive and leave in runs of CH channels; the forward form of 4096 tokens also moves 16 values a thread through
// scratch memory.  2048 x 4096, forward and inverse: 20.4 and 23.7 us, 36.7 and 38.6
// with every radix-4 pass through LDS.
#include "stamp_gen_io.h"

namespace {

constexpr double kSqrtHalf = 0.70710678118654752440;

template <bool INV>
__device__ __forceinline__ void radix4(cd& a, cd& b, cd& c, cd& d) {
  const cd s0 = c_add(a, c), s1 = c_sub(a, c), s2 = c_add(b, d), s3 = c_sub(b, d);
  const cd i3 = INV ? cd{-s3.im, s3.re} : cd{s3.im, -s3.re};
  a = c_add(s0, s2);
  b = c_add(s1, i3);
  c = c_sub(s0, s2);
  d = c_sub(s1, i3);
}
// times e^{-2 pi i m / 16} (conjugated: INV)
template <bool INV, int m>
__device__ __forceinline__ cd mul_w16(cd x) {
  constexpr double C1 = 0.92387953251128675613, S1 = 0.38268343236508977173;  // cos, sin of pi / 8
  if constexpr (m == 0) return x;
  else if constexpr (m == 2) return INV ? cd{kSqrtHalf * (x.re - x.im), kSqrtHalf * (x.re + x.im)} : cd{kSqrtHalf * (x.re + x.im), kSqrtHalf * (x.im - x.re)};
  else if constexpr (m == 4) return INV ? cd{-x.im, x.re} : cd{x.im, -x.re};
  else if constexpr (m == 6) return INV ? cd{-kSqrtHalf * (x.re + x.im), kSqrtHalf * (x.re - x.im)} : cd{kSqrtHalf * (x.im - x.re), -kSqrtHalf * (x.re + x.im)};
  else {
    constexpr double c = m == 1 ? C1 : m == 3 ? S1 : -C1, s = m == 1 ? S1 : m == 3 ? C1 : -S1;  // m = 9: minus m = 1
    static_assert(m == 1 || m == 3 || m == 9, "");
    return c_mul(x, cd{c, INV ? s : -s});
  }
}
// in place; result k stands at index 4 (k % 4) + k / 4
__device__ __host__ constexpr int pos16(int k) { return 4 * (k & 3) + (k >> 2); }
template <bool INV>
__device__ __forceinline__ void radix16(cd (&v)[16]) {
#pragma unroll
  for (int b = 0; b < 4; ++b) radix4<INV>(v[b], v[4 + b], v[8 + b], v[12 + b]);
  v[5] = mul_w16<INV, 1>(v[5]);
  v[6] = mul_w16<INV, 2>(v[6]);
  v[7] = mul_w16<INV, 3>(v[7]);
  v[9] = mul_w16<INV, 2>(v[9]);
  v[10] = mul_w16<INV, 4>(v[10]);
  v[11] = mul_w16<INV, 6>(v[11]);
  v[13] = mul_w16<INV, 3>(v[13]);
  v[14] = mul_w16<INV, 6>(v[14]);
  v[15] = mul_w16<INV, 9>(v[15]);
#pragma unroll
  for (int c = 0; c < 4; ++c) radix4<INV>(v[4 * c], v[4 * c + 1], v[4 * c + 2], v[4 * c + 3]);
}
// in place on v[0 .. R); result k stands at index posr<R>(k)
template <int R>
__device__ __host__ constexpr int posr(int k) { return R == 8 ? 4 * (k & 1) + (k >> 1) : k; }
template <bool INV, int R>
__device__ __forceinline__ void radix_last(cd* v) {
  if constexpr (R == 2) {
    const cd x = v[0], y = v[1];
    v[0] = c_add(x, y);
    v[1] = c_sub(x, y);
  } else if constexpr (R == 4) {
    radix4<INV>(v[0], v[1], v[2], v[3]);
  } else if constexpr (R == 8) {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const cd x = v[b], y = v[4 + b];
      v[b] = c_add(x, y);
      v[4 + b] = c_sub(x, y);
    }
    v[5] = mul_w16<INV, 2>(v[5]);
    v[6] = mul_w16<INV, 4>(v[6]);
    v[7] = mul_w16<INV, 6>(v[7]);
    radix4<INV>(v[0], v[1], v[2], v[3]);
    radix4<INV>(v[4], v[5], v[6], v[7]);
  }
}
// v[at(q)] *= w^q, w = e^{-2 pi i base / M} (conjugated: INV); four factors from the table, the others as products of two or
// three of them
struct Tw {
  cd w1, w2, w4, w8;
};
__device__ __forceinline__ Tw load_tw(const cd* __restrict__ tab, int base) { return {tab[base], tab[2 * base], tab[4 * base], tab[8 * base]}; }
template <bool INV, typename At>
__device__ __forceinline__ void twiddle16(cd (&v)[16], const Tw& tw, At at) {
  cd w1 = tw.w1, w2 = tw.w2, w4 = tw.w4, w8 = tw.w8;
  if constexpr (INV) {
    w1.im = -w1.im;
    w2.im = -w2.im;
    w4.im = -w4.im;
    w8.im = -w8.im;
  }
  const cd w3 = c_mul(w1, w2);
  v[at(1)] = c_mul(v[at(1)], w1);
  v[at(2)] = c_mul(v[at(2)], w2);
  v[at(3)] = c_mul(v[at(3)], w3);
  v[at(4)] = c_mul(v[at(4)], w4);
  v[at(5)] = c_mul(v[at(5)], c_mul(w4, w1));
  v[at(6)] = c_mul(v[at(6)], c_mul(w4, w2));
  v[at(7)] = c_mul(v[at(7)], c_mul(w4, w3));
  v[at(8)] = c_mul(v[at(8)], w8);
  v[at(9)] = c_mul(v[at(9)], c_mul(w8, w1));
  v[at(10)] = c_mul(v[at(10)], c_mul(w8, w2));
  v[at(11)] = c_mul(v[at(11)], c_mul(w8, w3));
  const cd w12 = c_mul(w8, w4);
  v[at(12)] = c_mul(v[at(12)], w12);
  v[at(13)] = c_mul(v[at(13)], c_mul(w12, w1));
  v[at(14)] = c_mul(v[at(14)], c_mul(w12, w2));
  v[at(15)] = c_mul(v[at(15)], c_mul(w12, w3));
}

// LDS places of the two exchanges (points; the paddings keep the 64-byte rows of a half wave apart)
template <int R>
struct Places {
  static constexpr int T = 16 * R;                                  // threads per channel
  static constexpr int S1 = T + (R < 4 ? R : 0);                    // between k1
  static constexpr int S2 = 256 + (R >= 4 ? 1 : R == 2 ? 2 : 0);    // between m2
  static constexpr int kPoints = 16 * S1 > R * S2 ? 16 * S1 : R * S2;
};

// real, then imaginary parts through LDS: point wr(i) of this thread's channel <- v[i], v[i] <- point rd(i)
template <int CH, typename Wr, typename Rd>
__device__ __forceinline__ void exchange(cd (&v)[16], double* s, Wr wr, Rd rd) {
#pragma unroll
  for (int i = 0; i < 16; ++i) s[wr(i) * CH] = v[i].re;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i].re = s[rd(i) * CH];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 16; ++i) s[wr(i) * CH] = v[i].im;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i].im = s[rd(i) * CH];
  __syncthreads();
}

// tab: the factors of k_gen_dct_factors for N.  Rows of `ld` channels; byte offsets within a sequence fit 31 bits.
template <int R, int CH, bool INV>
__global__ __launch_bounds__(16 * R * CH, 4) void k_dct_reg(const cd* __restrict__ tab, const void* __restrict__ src, int in_kind,
                                                            float* __restrict__ Tout, void* __restrict__ Y,
                                                            const float* __restrict__ bias, int y_bf16, int ld) {
  using Pl = Places<R>;
  constexpr int M = 256 * R, N = 2 * M, T = Pl::T, NB = 16 / R;  // NB butterflies of the last pass
  constexpr double kNrm = (R == 1 ? 1.0 : R == 2 ? kSqrtHalf : R == 4 ? 0.5 : 0.5 * kSqrtHalf) / 16.0;  // sqrt(2 / N)
  // sqrt(1 / N): a power of two for 1024 and 4096, so that a sum of bf16 tokens that lies between two fp32 numbers is rounded as such
  constexpr double kNrm0 = (R == 1 ? kSqrtHalf : R == 2 ? 0.5 : R == 4 ? 0.5 * kSqrtHalf : 0.25) / 16.0;
  extern __shared__ __attribute__((aligned(16))) uint8_t dct_reg_smem[];  // [Places::kPoints][CH]
  const int tid = threadIdx.x, ch = tid % CH, t = tid / CH;
  // neighbouring channel groups share cache lines: keep them on one XCD
  const int ngrp = gridDim.x, xcd = blockIdx.x & 7, tall = ngrp >> 3, rem = ngrp & 7;
  const int grp = xcd * tall + min(xcd, rem) + (int)(blockIdx.x >> 3);
  const bool live = grp * CH + ch < ld;
  const int c = min(grp * CH + ch, ld - 1);
  const size_t seq0 = (size_t)blockIdx.y * N * ld;
  const cd *te = tab + M, *tn = te + M + 1;
  double* const s = reinterpret_cast<double*>(dct_reg_smem) + ch;
  cd v[16];
  const int k1 = t / R, m2 = t % R;
  // places: first exchange [k1][n2], second [m2][j]
  auto w1 = [&](int q) { return q * Pl::S1 + t; };
  auto r1 = [&](int q) { return k1 * Pl::S1 + q * R + m2; };
  auto w2 = [&](int q) { return m2 * Pl::S2 + k1 + 16 * q; };
  const bool first = t == 0;  // its first two butterflies are 0 and 128: pairs of their own
  auto butterfly = [&](int b) { return (b & 1) ? (b == 1 && first ? 128 : 256 - (t + T * (b >> 1))) : t + T * (b >> 1); };
  auto r2 = [&](int i) { return (i % R) * Pl::S2 + butterfly(i / R); };

  if constexpr (!INV) {
    const Tw tw1 = load_tw(tab, t);  // asked for before the rows
    {
      // point j = n1 T + t: tokens 4 j, 4 j + 2 for the first half, 2 N - 1 - 4 j, 2 N - 3 - 4 j for the second
      float x[32];
      double xd[32];
      const uint32_t es = in_kind == 2 ? 2 : 4, row = (uint32_t)ld * es, up = (uint32_t)(4 * t) * row + (uint32_t)c * es;
      const uint32_t down = (uint32_t)(2 * N - 3 - 8 * (N / 8) - 4 * t) * row + (uint32_t)c * es;  // token 2 N - 3 - 4 j of n1 = 8
      const uint8_t* const p = static_cast<const uint8_t*>(src) + seq0 * es;
      if (in_kind == 2) {
        uint32_t w[32];
#pragma unroll
        for (int n1 = 0; n1 < 8; ++n1) {
          const uint8_t *pu = p + (size_t)((uint32_t)(n1 * (N / 8)) * row), *pd = p - (size_t)((uint32_t)(n1 * (N / 8)) * row);
          w[2 * n1] = *reinterpret_cast<const uint16_t*>(pu + up);
          w[2 * n1 + 1] = *reinterpret_cast<const uint16_t*>(pu + 2 * row + up);
          w[16 + 2 * n1] = *reinterpret_cast<const uint16_t*>(pd + 2 * row + down);
          w[16 + 2 * n1 + 1] = *reinterpret_cast<const uint16_t*>(pd + down);
        }
#pragma unroll
        for (int i = 0; i < 32; ++i) x[i] = __uint_as_float(w[i] << 16);
      } else {
#pragma unroll
        for (int n1 = 0; n1 < 8; ++n1) {
          const uint8_t *pu = p + (size_t)((uint32_t)(n1 * (N / 8)) * row), *pd = p - (size_t)((uint32_t)(n1 * (N / 8)) * row);
          x[2 * n1] = *reinterpret_cast<const float*>(pu + up);
          x[2 * n1 + 1] = *reinterpret_cast<const float*>(pu + 2 * row + up);
          x[16 + 2 * n1] = *reinterpret_cast<const float*>(pd + 2 * row + down);
          x[16 + 2 * n1 + 1] = *reinterpret_cast<const float*>(pd + down);
        }
      }
      dct_in(x, xd);
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] = {xd[2 * i], xd[2 * i + 1]};
    }
    radix16<false>(v);
    twiddle16<false>(v, tw1, [](int q) { return pos16(q); });
    exchange<CH>(v, s, [&](int i) { return w1(pos16(i)); }, r1);  // index i holds result pos16(i): pos16 is its own inverse
    radix16<false>(v);
    if constexpr (R > 1) twiddle16<false>(v, load_tw(tab, 16 * m2), [](int q) { return pos16(q); });
    exchange<CH>(v, s, [&](int i) { return w2(pos16(i)); }, r2);
#pragma unroll
    for (int b = 0; b < NB; ++b) radix_last<false, R>(&v[b * R]);
    // z(b, l) = T[butterfly(b) + 256 l]
    const uint32_t row = (uint32_t)ld * 4u;
    uint8_t* const o = reinterpret_cast<uint8_t*>(Tout + seq0 + c);
    auto put = [&](uint32_t off, double x) { if (live) *reinterpret_cast<float*>(o + off) = (float)x; };
#pragma unroll
    for (int i = 0; i < NB / 2; ++i)
#pragma unroll
      for (int l = 0; l < R; ++l) {
        cd a = v[2 * i * R + posr<R>(l)], b = v[(2 * i + 1) * R + posr<R>(R - 1 - l)];
        int k = t + T * i + 256 * l;
        if (i == 0) {
          // butterflies 0 and 128: (0, M / 2), then (256 l, M - 256 l), then (128 + 256 l, M - 128 - 256 l)
          const int h = R / 2;
          const cd a0 = l < h || R == 1 ? v[posr<R>(l)] : v[R + posr<R>(l - h)];
          const cd b0 = R == 1 ? v[1] : l == 0 ? v[posr<R>(h)] : l < h ? v[posr<R>(R - l)] : v[R + posr<R>(R - 1 - (l - h))];
          a = {first ? a0.re : a.re, first ? a0.im : a.im};
          b = {first ? b0.re : b.re, first ? b0.im : b.im};
          if (l >= h && R > 1) k = first ? 128 + 256 * (l - h) : k;
          if (l == 0 && first) {
            const cd hh = c_mul(te[M / 2], c_conj(b));
            put(0, (a.re + a.im) * kNrm0);
            put((uint32_t)M * row, (a.re - a.im) * kNrm0);
            put((uint32_t)(M / 2) * row, kNrm * hh.re);
            put((uint32_t)(M + M / 2) * row, -kNrm * hh.im);
            continue;
          }
        }
        const cd e = te[k], f = tn[k];
        const cd fe = {a.re + b.re, a.im - b.im}, fo = {a.im + b.im, b.re - a.re};
        const cd g = c_mul(f, fo);
        const cd p = c_mul(e, c_add(fe, g));  // 2 e^{-i pi k / 2N} V[k]
        const cd q = c_mul(e, c_sub(fe, g));  // e^{-i pi (M-k) / 2N} V[M-k] = e^{-i pi / 4} conj of half of it
        const uint32_t u = (uint32_t)k * row;
        put(u, 0.5 * kNrm * p.re);
        put((uint32_t)N * row - u, -0.5 * kNrm * p.im);
        put((uint32_t)M * row - u, 0.5 * kNrm * kSqrtHalf * (q.re - q.im));
        put((uint32_t)M * row + u, 0.5 * kNrm * kSqrtHalf * (q.re + q.im));
      }
  } else {
    constexpr double sc = 1.0 / (M * kNrm);  // sqrt(N / 2) / M
    {
      const uint32_t row = (uint32_t)ld * 4u;
      const uint8_t* const p = reinterpret_cast<const uint8_t*>(static_cast<const float*>(src) + seq0 + c);
      auto get = [&](uint32_t off) { return *reinterpret_cast<const float*>(p + off); };
      float x[32];
      double xd[32];
#pragma unroll
      for (int i = 0; i < NB / 2; ++i)
#pragma unroll
        for (int l = 0; l < R; ++l) {
          const int h = R / 2, e = 4 * (i * R + l);
          int k = t + T * i + 256 * l;
          if (i == 0 && l >= h && R > 1) k = first ? 128 + 256 * (l - h) : k;
          const bool zero = i == 0 && l == 0 && first;  // k = 0 comes with M / 2
          const uint32_t u = (uint32_t)k * row, ml = (uint32_t)M * row;
          x[e] = get(u);
          x[e + 1] = get(zero ? ml : 2 * ml - u);
          x[e + 2] = get(zero ? ml / 2 : ml - u);
          x[e + 3] = get(zero ? ml + ml / 2 : ml + u);
        }
      dct_in(x, xd);
#pragma unroll
      for (int i = 0; i < NB / 2; ++i) {
        cd za[R], zb[R];
#pragma unroll
        for (int l = 0; l < R; ++l) {
          const int h = R / 2, e = 4 * (i * R + l);
          int k = t + T * i + 256 * l;
          if (i == 0 && l >= h && R > 1) k = first ? 128 + 256 * (l - h) : k;
          const double x0 = xd[e], x1 = xd[e + 1], x2 = xd[e + 2], x3 = xd[e + 3];
          if (i == 0 && l == 0 && first) {
            const double v0 = x0 * (sc * 2.0 * kSqrtHalf), vm = x1 * (sc * 2.0 * kSqrtHalf);
            za[l] = {0.5 * (v0 + vm), 0.5 * (v0 - vm)};
            zb[l] = c_mul(te[M / 2], cd{sc * x2, sc * x3});
          } else {
            // V[k] = conj(te) (x0 - i x1), conj V[M-k] = conj(te) e^{-i pi / 4} (x2 + i x3)
            const double pr = kSqrtHalf * (x2 + x3), pi = kSqrtHalf * (x3 - x2);
            const cd cte = c_conj(te[k]), hs = {0.5 * sc * (x0 + pr), 0.5 * sc * (pi - x1)}, hd = {0.5 * sc * (x0 - pr), -0.5 * sc * (x1 + pi)};
            const cd fe = c_mul(cte, hs), fo = c_mul(c_conj(tn[k]), c_mul(cte, hd));
            za[l] = {fe.re - fo.im, fe.im + fo.re};  // Fe + i Fo
            zb[l] = {fe.re + fo.im, fo.re - fe.im};  // conj Fe + i conj Fo
          }
        }
#pragma unroll
        for (int l = 0; l < R; ++l) {
          v[2 * i * R + l] = za[l];
          v[(2 * i + 1) * R + l] = zb[R - 1 - l];
        }
        if (i == 0 && R > 1) {
          constexpr int h = R > 1 ? R / 2 : 1;
#pragma unroll
          for (int l = 0; l < R; ++l) {
            const cd a0 = l < h ? za[l] : l == h ? zb[0] : zb[R - l];
            const cd b0 = l < h ? za[h + l] : zb[h + (R - 1 - l)];
            if (first) {
              v[l] = a0;
              v[R + l] = b0;
            }
          }
        }
      }
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) radix_last<true, R>(&v[b * R]);
    // index b R + posr(m2) holds place [m2][butterfly(b)]
    exchange<CH>(v, s, [&](int i) { const int r = i % R, m = R == 8 ? (r >> 2) + 2 * (r & 3) : r; return m * Pl::S2 + butterfly(i / R); }, w2);
    if constexpr (R > 1) twiddle16<true>(v, load_tw(tab, 16 * m2), [](int q) { return q; });
    radix16<true>(v);
    exchange<CH>(v, s, [&](int i) { return r1(pos16(i)); }, w1);
    twiddle16<true>(v, load_tw(tab, t), [](int q) { return q; });
    radix16<true>(v);
    const float bv = bias != nullptr ? bias[c] : 0.0f;
    const uint32_t es = y_bf16 ? 2 : 4, row = (uint32_t)ld * es, up = (uint32_t)(4 * t) * row + (uint32_t)c * es;
    const uint32_t down = (uint32_t)(2 * N - 3 - 8 * (N / 8) - 4 * t) * row + (uint32_t)c * es;
    uint8_t* const p = static_cast<uint8_t*>(Y) + seq0 * es;
    if (!live) return;
    auto out = [&](auto store) {
#pragma unroll
      for (int n1 = 0; n1 < 8; ++n1) {
        uint8_t *pu = p + (size_t)((uint32_t)(n1 * (N / 8)) * row), *pd = p - (size_t)((uint32_t)(n1 * (N / 8)) * row);
        const cd z = v[pos16(n1)], y = v[pos16(n1 + 8)];
        store(pu + up, (float)z.re + bv);
        store(pu + 2 * row + up, (float)z.im + bv);
        store(pd + 2 * row + down, (float)y.re + bv);
        store(pd + down, (float)y.im + bv);
      }
    };
    if (y_bf16) out([](uint8_t* q, float f) { *reinterpret_cast<uint16_t*>(q) = f32_to_bf16_rne(f); });
    else out([](uint8_t* q, float f) { *reinterpret_cast<float*>(q) = f; });
  }
}

template <int R, int CH>
hipError_t launch_ch(const stamp_plan* p, int inv, const void* src, int in_kind, float* T, void* Y, const float* bias, int ld, hipStream_t st) {
  const dim3 grid((ld + CH - 1) / CH, p->geom.B), blk(16 * R * CH);
  constexpr size_t lds = sizeof(double) * Places<R>::kPoints * CH;
  static size_t done[2][kStampMaxDevices] = {};
  const void* fn = inv ? reinterpret_cast<const void*>(&k_dct_reg<R, CH, true>) : reinterpret_cast<const void*>(&k_dct_reg<R, CH, false>);
  const hipError_t e = stamp_allow_lds(fn, lds, done[inv]);
  if (e != hipSuccess) return e;
  const cd* tab = reinterpret_cast<const cd*>(p->dct_dev);
  if (inv) hipLaunchKernelGGL((k_dct_reg<R, CH, true>), grid, blk, lds, st, tab, src, in_kind, T, Y, bias, p->geom.y_bf16, ld);
  else hipLaunchKernelGGL((k_dct_reg<R, CH, false>), grid, blk, lds, st, tab, src, in_kind, T, Y, bias, 0, ld);
  return hipGetLastError();
}

template <int R>
hipError_t launch(const stamp_plan* p, int inv, const void* src, int in_kind, float* T, void* Y, const float* bias, int ld, hipStream_t st) {
  // eight channels per workgroup while that leaves no CU without one, else four: 2048 x 2048 62.1 us with eight (66.6), 2048 x 512
  // 48.4 (44.0), 4096 x 1024 78.6 (71.5), 1024 x 1024 43.8 (43.1) a layer
  if ((int64_t)((ld + 7) / 8) * p->geom.B < stamp_device_cus()) return launch_ch<R, 4>(p, inv, src, in_kind, T, Y, bias, ld, st);
  return launch_ch<R, 8>(p, inv, src, in_kind, T, Y, bias, ld, st);
}

}  // namespace

// 512 tokens: only where there are channels for the CUs, a thread's serial share is too long otherwise (2 x 512 tokens, 64 -> 33
// channels 33.1 us through LDS, 34.0 here; 2048 -> 4096 47.9, 46.4; 16 x 512 tokens, 2048 -> 2048 172, 120)
bool stamp_dct_in_registers(int s, int B, int ld) {
  if (s < 512 || s > 4096 || (s & (s - 1)) != 0 || (int64_t)s * ld * 4 >= ((int64_t)1 << 31)) return false;
  return s > 512 || (int64_t)((ld + 7) / 8) * B >= stamp_device_cus();
}

hipError_t stamp_launch_dct_reg(const stamp_plan* p, int inv, const void* src, int in_kind, float* T, void* Y, const float* bias, int ld,
                                hipStream_t st) {
  switch (p->geom.s) {
    case 512: return launch<1>(p, inv, src, in_kind, T, Y, bias, ld, st);
    case 1024: return launch<2>(p, inv, src, in_kind, T, Y, bias, ld, st);
    case 2048: return launch<4>(p, inv, src, in_kind, T, Y, bias, ld, st);
    case 4096: return launch<8>(p, inv, src, in_kind, T, Y, bias, ld, st);
    default: return hipErrorInvalidValue;
  }
}
