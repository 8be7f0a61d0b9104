// K-point complex FFTs held in registers: K = 256 R (R = 4, 8, 16) by
// NTf = K/16 threads of 16 values each, index m = t + NTf r.  A radix-16
// stage over r in registers, an LDS exchange, a radix-16 stage, an LDS
// exchange, a radix-R stage; F = 256/NTf independent FFTs share a
// 256-thread workgroup.  Also the small in-register DFTs (2 to 16 points)
// these stages are built from.
#pragma once

#include "dev_common.h"

namespace rfd {

// cos / sin (2 pi k / 16), k < 16
__device__ __forceinline__ float2 w16(int k, int sign) {
  constexpr float c[16] = {1.0f, 0.92387953251128674f, 0.70710678118654752f, 0.38268343236508977f,
                           0.0f, -0.38268343236508977f, -0.70710678118654752f, -0.92387953251128674f,
                           -1.0f, -0.92387953251128674f, -0.70710678118654752f, -0.38268343236508977f,
                           0.0f, 0.38268343236508977f, 0.70710678118654752f, 0.92387953251128674f};
  return make_float2(c[k & 15], sign * c[(k + 12) & 15]);   // sin x = cos(x - pi/2)
}

// dft4 of the products a = xa ga, b = xb gb, c = xc gc, d = xd gd: the first
// sums take a's and b's products as fused multiply-adds onto c's and d's, and
// the differences follow as a - c = (a + c) - 2c: 28 operations instead of the
// 32 of four complex products and a dft4.
__device__ __forceinline__ void dft4_prod(float2& a, float2& b, float2& c, float2& d, float2 xa, float2 ga,
                                          float2 xb, float2 gb, float2 xc, float2 gc, float2 xd, float2 gd,
                                          int sign) {
  const float2 pc = cmul(xc, gc), pd = cmul(xd, gd);
  const float2 s0 = make_float2(fmaf(xa.x, ga.x, fmaf(-xa.y, ga.y, pc.x)), fmaf(xa.x, ga.y, fmaf(xa.y, ga.x, pc.y)));
  const float2 s2 = make_float2(fmaf(xb.x, gb.x, fmaf(-xb.y, gb.y, pd.x)), fmaf(xb.x, gb.y, fmaf(xb.y, gb.x, pd.y)));
  const float2 s1 = make_float2(fmaf(-2.f, pc.x, s0.x), fmaf(-2.f, pc.y, s0.y));
  const float2 s3 = cmul_si(make_float2(fmaf(-2.f, pd.x, s2.x), fmaf(-2.f, pd.y, s2.y)), sign);
  a = cadd(s0, s2);
  c = csub(s0, s2);
  b = cadd(s1, s3);
  d = csub(s1, s3);
}

// The scalar of a complex type and the fused multiply-add of either precision.
template <typename V> struct ScalarOf;
template <> struct ScalarOf<float2> { typedef float type; };
template <> struct ScalarOf<double2> { typedef double type; };
template <typename V> using scalar_t = typename ScalarOf<V>::type;
__device__ __forceinline__ float fma_s(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fma_s(double a, double b, double c) { return fma(a, b, c); }
template <typename V>
__device__ __forceinline__ V make_c(scalar_t<V> x, scalar_t<V> y) { V v; v.x = x; v.y = y; return v; }

// A twiddle w = c (1 + i tau) in the form the butterflies below take: (c, tau).
// Where Re w = 0 the tables hold a c of 2^-30 (FP64: 2^-60): the product with
// w is then off by as much, below the type's rounding.
//
// a +- w b as t = b (1 + i tau), a +- c t: six fused multiply-adds instead of the
// eight operations of a complex product and two sums, with one rounding of
// the product instead of two.
template <typename V>
__device__ __forceinline__ void bf_tw(V& a, V& b, V w) {
  const V t = make_c<V>(fma_s(-w.y, b.y, b.x), fma_s(w.y, b.x, b.y));
  b = make_c<V>(fma_s(-w.x, t.x, a.x), fma_s(-w.x, t.y, a.y));
  a = make_c<V>(fma_s(w.x, t.x, a.x), fma_s(w.x, t.y, a.y));
}
// the same with the twiddle s i w (s = +-1)
template <typename V>
__device__ __forceinline__ void bf_tw_si(V& a, V& b, V w, int s) {
  const V t = make_c<V>(fma_s(-w.y, b.y, b.x), fma_s(w.y, b.x, b.y));
  const scalar_t<V> c = s > 0 ? w.x : -w.x;
  b = make_c<V>(fma_s(c, t.y, a.x), fma_s(-c, t.x, a.y));
  a = make_c<V>(fma_s(-c, t.y, a.x), fma_s(c, t.x, a.y));
}
// 4-point DFT of (a, w b, w^2 c, w^3 d) from the twiddles w2 = w^2 and w
template <typename V>
__device__ __forceinline__ void dft4_tw(V& a, V& b, V& c, V& d, V w2, V w, int sign) {
  bf_tw(a, c, w2);
  bf_tw(b, d, w2);
  bf_tw(a, b, w);              // outputs 0 and 2
  bf_tw_si(c, d, w, sign);     // outputs 1 and 3
  const V x2 = b;
  b = c;
  c = x2;
}
// ... with the twiddles s i w2 and w
template <typename V>
__device__ __forceinline__ void dft4_tw_i(V& a, V& b, V& c, V& d, V w2, V w, int sign) {
  bf_tw_si(a, c, w2, sign);
  bf_tw_si(b, d, w2, sign);
  bf_tw(a, b, w);
  bf_tw_si(c, d, w, sign);
  const V x2 = b;
  b = c;
  c = x2;
}

// Second half of the 16-point DFT (after the first radix-4 layer over n2):
// for each k the 4-point DFT of v[4 k + n1] w_16^(n1 k).
template <int SIGN, typename V>
__device__ __forceinline__ void dft16_rest(V (&v)[16]) {
  using S = scalar_t<V>;
  constexpr S c1 = (S)0.92387953251128674, t1 = (S)0.41421356237309503;   // cos, tan of pi / 8
  constexpr S c3 = (S)0.38268343236508977, t3 = (S)2.41421356237309515;   // of 3 pi / 8
  constexpr S r = (S)0.70710678118654752, sg = (S)SIGN;
  dft4(v[0], v[1], v[2], v[3], SIGN);
  dft4_tw(v[4], v[5], v[6], v[7], make_c<V>(r, sg), make_c<V>(c1, sg * t1), SIGN);
  {                                                     // k = 2: w^2 is a quarter turn
    V s0 = v[8], s1 = v[9];
    const V c = cmul_si(v[10], SIGN), d = cmul_si(v[11], SIGN);
    V m0 = csub(s0, c), m1 = csub(s1, d);
    s0 = cadd(s0, c);
    s1 = cadd(s1, d);
    bf_tw(s0, s1, make_c<V>(r, sg));
    bf_tw_si(m0, m1, make_c<V>(r, sg), SIGN);
    v[8] = s0;
    v[9] = m0;
    v[10] = s1;
    v[11] = m1;
  }
  dft4_tw_i(v[12], v[13], v[14], v[15], make_c<V>(r, sg), make_c<V>(c3, sg * t3), SIGN);
}

// Twiddles of a 16-point DFT of x[q] w^q (w any unit complex number), as (c, tau):
// w^8, w^4, w^2, w^2 w_8, w, w w_16, w w_16^2, w w_16^3: the other factors that its
// radix-2 layers need are quarter turns of these.  Of an 8-point one: w^4,
// w^2, w, w w_8; of a 4-point one: w^2, w.
// Taking the inter-stage twiddles inside the butterflies like this costs
// 192 operations per 16 points, against 60 for 15 products and 160 for a plain
// DFT after them.
constexpr int kTw16 = 8;
// entry i of those of an R-point DFT at w = e^{2 pi i m / 4096}: its exponent over 4096
template <int R>
__device__ __forceinline__ constexpr int tw_exponent(int i, int m) {
  if (R == 16) return (i == 0 ? 8 * m : i == 1 ? 4 * m : i < 4 ? 2 * m + 512 * (i - 2) : m + 256 * (i - 4)) & 4095;
  if (R == 8) return (i == 0 ? 4 * m : i == 1 ? 2 * m : m + 512 * (i - 2)) & 4095;
  if (R == 4) return (i == 0 ? 2 * m : m) & 4095;
  return m & 4095;
}
// DFTs (R = 2, 4, 8, 16) of v[g R + u] w_g^u on consecutive groups of R slots; slot
// order of the results as dft_r.  w(i): entry i of the 16 / R groups' twiddles, group by group.
template <int R, int SIGN, typename V, typename W>
__device__ __forceinline__ void dft_tw(V (&v)[16], const W& w) {
  if constexpr (R == 16) {
    const V w8 = w(0), w4 = w(1), w2 = w(2), w2b = w(3);
#pragma unroll
    for (int n1 = 0; n1 < 4; ++n1) dft4_tw(v[n1], v[n1 + 4], v[n1 + 8], v[n1 + 12], w8, w4, SIGN);
    dft4_tw(v[0], v[1], v[2], v[3], w2, w(4), SIGN);
    dft4_tw(v[4], v[5], v[6], v[7], w2b, w(5), SIGN);
    dft4_tw_i(v[8], v[9], v[10], v[11], w2, w(6), SIGN);
    dft4_tw_i(v[12], v[13], v[14], v[15], w2b, w(7), SIGN);
  } else if constexpr (R == 8) {
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      V* u = v + 8 * g;
      dft4_tw(u[0], u[2], u[4], u[6], w(4 * g), w(4 * g + 1), SIGN);
      dft4_tw(u[1], u[3], u[5], u[7], w(4 * g), w(4 * g + 1), SIGN);
      bf_tw(u[0], u[1], w(4 * g + 2));
      bf_tw(u[2], u[3], w(4 * g + 3));
      bf_tw_si(u[4], u[5], w(4 * g + 2), SIGN);
      bf_tw_si(u[6], u[7], w(4 * g + 3), SIGN);
    }
  } else if constexpr (R == 2) {
#pragma unroll
    for (int g = 0; g < 8; ++g) bf_tw(v[2 * g], v[2 * g + 1], w(g));
  } else {
#pragma unroll
    for (int g = 0; g < 4; ++g)
      dft4_tw(v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3], w(2 * g), w(2 * g + 1), SIGN);
  }
}

// 16-point DFT in registers, V[k] = sum_n v[n] e^{sign 2 pi i n k / 16}.
// On return slot s holds V[(s >> 2) + 4 (s & 3)].
template <int SIGN, typename V>
__device__ __forceinline__ void dft16(V (&v)[16]) {
#pragma unroll
  for (int n1 = 0; n1 < 4; ++n1) dft4(v[n1], v[n1 + 4], v[n1 + 8], v[n1 + 12], SIGN);
  dft16_rest<SIGN>(v);
}
// The same DFT where v[8..16) is zero (and not read).
template <int SIGN, typename V>
__device__ __forceinline__ void dft16_half(V (&v)[16]) {
#pragma unroll
  for (int n1 = 0; n1 < 4; ++n1) {
    const V a = v[n1], b = v[n1 + 4], ib = cmul_si(b, SIGN);
    v[n1] = cadd(a, b);
    v[n1 + 4] = cadd(a, ib);
    v[n1 + 8] = csub(a, b);
    v[n1 + 12] = csub(a, ib);
  }
  dft16_rest<SIGN>(v);
}
// The same DFT of the products x[n] g[n].
template <int SIGN>
__device__ __forceinline__ void dft16_prod(float2 (&v)[16], const float2 (&x)[16], const float2 (&g)[16]) {
#pragma unroll
  for (int n1 = 0; n1 < 4; ++n1)
    dft4_prod(v[n1], v[n1 + 4], v[n1 + 8], v[n1 + 12], x[n1], g[n1], x[n1 + 4], g[n1 + 4], x[n1 + 8], g[n1 + 8],
              x[n1 + 12], g[n1 + 12], SIGN);
  dft16_rest<SIGN>(v);
}
__device__ __forceinline__ constexpr int dft16_freq(int s) { return (s >> 2) + 4 * (s & 3); }

// R-point DFTs (R = 2, 4, 8, 16) on consecutive groups of R slots of v; slot
// g R + s holds V_g[dftR_freq(s)].
template <int R, int SIGN>
__device__ __forceinline__ void dft_r(float2 (&v)[16]) {
  if constexpr (R == 16) {
    dft16<SIGN>(v);
  } else if constexpr (R == 2) {
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      const float2 a = v[2 * g], b = v[2 * g + 1];
      v[2 * g] = cadd(a, b);
      v[2 * g + 1] = csub(a, b);
    }
  } else if constexpr (R == 4) {
#pragma unroll
    for (int g = 0; g < 4; ++g) dft4(v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3], SIGN);
  } else {   // R == 8: n = n1 + 2 n2, DFT4 over n2, twiddle, DFT2 over n1
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      float2* u = v + 8 * g;
      dft4(u[0], u[2], u[4], u[6], SIGN);
      dft4(u[1], u[3], u[5], u[7], SIGN);
#pragma unroll
      for (int k = 1; k < 4; ++k) u[2 * k + 1] = cmul(u[2 * k + 1], w16(2 * k, SIGN));
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float2 a = u[2 * k], b = u[2 * k + 1];
        u[2 * k] = cadd(a, b);
        u[2 * k + 1] = csub(a, b);
      }
    }
  }
}
template <int R>
__device__ __forceinline__ constexpr int dftr_freq(int s) {
  return R == 16 ? dft16_freq(s) : (R <= 4 ? s : (s >> 1) + 4 * (s & 1));
}

template <int K>
struct BlockFft {
  static constexpr int NTf = K / 16;       // threads per FFT
  static constexpr int R = K / 256;        // last radix
  static constexpr int G = 16 / R;         // last-stage groups per thread
  static constexpr int F = 256 / NTf;      // FFTs per workgroup
  // LDS layouts of the two exchanges, chosen so that no access of either
  // exchange meets an LDS bank twice within a pass (a 64-bit access is
  // serviced half a wave at a time):
  //  exchange 1: element (k1, t) at k1 S1 + t, S1 = NTf + R.  A stage-B reader
  //    takes elements u + R q of row k1 = t / R; the rows of one half-wave
  //    start 2R banks apart, so their R-wide column groups tile the banks.
  //  exchange 2: element (k2, k1, u) at (16 k2 + k1) R + k2 / G + u: rows of R
  //    values, each group of G rows (one stage-C reader's rows) skewed by one
  //    more element, so the readers, which take R consecutive values from
  //    rows 16 (G g + e) + k1, start in distinct banks; every offset is a
  //    compile-time constant past one per-thread base.
  // (The earlier strides S1 = NTf + 4 and S2 = R + 4 left the stage-C reads
  // 8-16-way conflicted: LDS bank-conflict cycles at 1.9x the busy cycles of
  // the 4096-point overlap-save kernel.)
  static constexpr int S1 = NTf + R;
  static constexpr int X1 = 16 * S1;                 // float2 of exchange 1
  static constexpr int X2 = 256 * R + R;             // float2 of exchange 2
  static constexpr int LDS = X1 > X2 ? X1 : X2;      // float2 per FFT
};

// Twiddles of the transform.  With m = t + NTf r, t = u + R q and the output index
// k1 + 16 k2 + 256 k3, stage A's DFT over r needs none, stage B's over q takes
// w = e^{2 pi i k1 / 256} and stage C's over u takes w = e^{2 pi i (k1 + 16 k2) / K}; each
// stage takes its w inside its butterflies (dft_tw).  A thread keeps the eight of stage C
// in registers (16 / R groups of k2); stage B's depend on k1 only, so a workgroup
// table of 16 rows in LDS serves every thread.
constexpr int kTwbStride = 9;    // row stride of the table: the rows' reads meet distinct banks
constexpr int kTwbSize = 16 * kTwbStride;
template <int K>
struct BlockFftTw {
  float2 c[kTw16];
  const float2* b;    // LDS row of this thread's k1
};
// Fills the table (every thread of the workgroup calls it; a barrier must
// follow before the first block_fft) and this thread's stage-C twiddles.
// ct: the (c, tau) of e^{2 pi i m / 4096}, m < 4096.
template <int K, int SIGN>
__device__ __forceinline__ void block_fft_twiddles(BlockFftTw<K>& w, const float2* __restrict__ ct, int t,
                                                   float2* table) {
  using S = BlockFft<K>;
  if (threadIdx.x < 16 * kTw16) {
    const int k1 = threadIdx.x / kTw16, i = threadIdx.x % kTw16;
    float2 x = ct[tw_exponent<16>(i, 16 * k1)];
    if (SIGN < 0) x.y = -x.y;
    table[k1 * kTwbStride + i] = x;
  }
  const int k1 = t / S::R, g = t % S::R;
  constexpr int per = kTw16 * S::R / 16;      // entries per group
#pragma unroll
  for (int i = 0; i < kTw16; ++i) {
    const int m = (k1 + 16 * (g * S::G + i / per)) * (4096 / K);
    float2 x = ct[tw_exponent<S::R>(i % per, m)];
    if (SIGN < 0) x.y = -x.y;
    w.c[i] = x;
  }
  w.b = table + k1 * kTwbStride;
}

// Exchange barrier: one wave per FFT (K = 1024) needs only wave-level
// ordering of its LDS traffic, so the workgroup's four FFTs run
// independently; larger FFTs span waves and synchronise the workgroup.
template <int NTf>
__device__ __forceinline__ void block_fft_sync() {
  if constexpr (NTf <= 64) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// K-point DFT of v (thread t of its FFT holds x[t + NTf r] in v[r]) with
// sign SIGN.  On return v[e * R + s] holds X[out_index(t, e, s)].  All
// threads of the workgroup call it together (it synchronises).
template <int K, int SIGN>
__device__ __forceinline__ void block_fft_after_a(float2 (&v)[16], float2* buf, int t, const BlockFftTw<K>& w);

template <int K, int SIGN>
__device__ __forceinline__ void block_fft(float2 (&v)[16], float2* buf, int t, const BlockFftTw<K>& w) {
  dft16<SIGN>(v);      // stage A: radix 16 over r
  block_fft_after_a<K, SIGN>(v, buf, t, w);
}
// The rest of block_fft once stage A's radix-16 DFT is in v (a caller can
// form that DFT itself, e.g. with dft16_prod).
template <int K, int SIGN>
__device__ __forceinline__ void block_fft_after_a(float2 (&v)[16], float2* buf, int t, const BlockFftTw<K>& w) {
  using S = BlockFft<K>;
  constexpr int NTf = S::NTf, R = S::R;
#pragma unroll
  for (int s = 0; s < 16; ++s) buf[dft16_freq(s) * S::S1 + t] = v[s];
  block_fft_sync<NTf>();
  // stage B: thread (k1, u) = (t / R, t % R), radix 16 over q of t' = u + R q
  {
    const int k1 = t / R, u = t % R;
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = buf[k1 * S::S1 + u + R * q];
  }
  block_fft_sync<NTf>();
  dft_tw<16, SIGN>(v, [&](int i) { return w.b[i]; });
  {
    const int k1 = t / R, u = t % R;
    float2* row = buf + k1 * R + u;
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      const int k2 = dft16_freq(s);
      row[k2 * 16 * R + k2 / S::G] = v[s];
    }
  }
  block_fft_sync<NTf>();
  // stage C: thread (k1, g) = (t / R, t % R) takes k2 = g G + e, radix R over u
  {
    const int k1 = t / R, g = t % R;
    const float2* row = buf + (g * S::G * 16 + k1) * R + g;
#pragma unroll
    for (int e = 0; e < S::G; ++e) {
#pragma unroll
      for (int u = 0; u < R; ++u) v[e * R + u] = row[e * 16 * R + u];
    }
  }
  block_fft_sync<NTf>();
  dft_tw<R, SIGN>(v, [&](int i) { return w.c[i]; });
}

// Output index of slot e * R + s of thread t after block_fft.
template <int K>
__device__ __forceinline__ int block_fft_out(int t, int e, int s) {
  using S = BlockFft<K>;
  const int k1 = t / S::R, g = t % S::R;
  const int k2 = g * (16 / S::R) + e;
  return k1 + 16 * k2 + 256 * dftr_freq<S::R>(s);
}
// ... as an offset from that of slot 0 (the same for every thread)
template <int K>
__device__ __forceinline__ constexpr int block_fft_step(int e, int s) {
  return 16 * e + 256 * dftr_freq<BlockFft<K>::R>(s);
}

// Place of element m of a K-point row in the order that the threads of a transform load:
// thread t takes m = t + NTf r, r < 16, two of them side by side per 16-byte load.
template <int K>
__device__ __forceinline__ constexpr int block_fft_place(int m) {
  constexpr int NTf = BlockFft<K>::NTf;
  const int t = m % NTf, r = m / NTf;
  return (r >> 1) * 2 * NTf + 2 * t + (r & 1);
}
template <int K>
__device__ __forceinline__ void block_fft_load(float2 (&v)[16], const float2* __restrict__ row, uint32_t t) {
#pragma unroll
  for (int p = 0; p < 8; ++p) {
    const float4 x = (reinterpret_cast<const float4*>(row) + p * BlockFft<K>::NTf)[t];
    v[2 * p] = make_float2(x.x, x.y);
    v[2 * p + 1] = make_float2(x.z, x.w);
  }
}

}  // namespace rfd
