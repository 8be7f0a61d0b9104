// L-point transforms (L = 256 R3: 256, 512, 1024, 2048) of C columns by one workgroup, FP32
// or FP64: 16 values per thread in registers, a radix-16 stage, an LDS exchange, a
// radix-16 stage, an LDS exchange and a radix-R3 stage (none at L = 256).  The stages'
// inputs and outputs are the caller's registers, so a first stage can come straight from
// global memory and a last one go straight back, and each value passes LDS twice (a
// radix-4 transform in LDS passes it five times at L = 1024).
#pragma once

#include "block_fft.h"

namespace rfd {

template <typename V_, int L_, int C_>
struct ColFft {
  typedef V_ V;
  static constexpr int L = L_, C = C_;
  static constexpr int J = L / 16;              // threads per column
  static constexpr int NT = C * J;              // threads of the workgroup
  static constexpr int R3 = L / 256;            // last radix
  // column stride in LDS: lanes go over columns first, then over neighbouring elements; the group
  // of lanes that one LDS pass serves (8 of 16 bytes, 16 of 8: 128 bytes) then meets each bank once when the
  // stride is G / C modulo G.  (Groups of 256 bytes had half of the FP32 passes' LDS cycles in conflicts: 32
  // stretches of 3072 lags 124 -> 116 us without.)
  static constexpr int G = sizeof(V) == 16 ? 8 : 16;
  static constexpr int LP = L + L / 16 + (((C < G ? G / C : 1) - L - L / 16) % G + G) % G;
  static constexpr int LDS = C * LP;            // values
  static constexpr int TWB = 16 * kTwbStride;   // values of the second stage's twiddle table
  // the third stage's twiddles are the 256 butterflies' own, in LDS: the 8 of a thread would take 16
  // registers, or 32 in FP64, beside the 32 or 64 of the values
  static constexpr int PER = R3 > 1 ? kTw16 * R3 / 16 : 0;    // per butterfly
  static constexpr int TW3 = 256 * PER;
  static constexpr size_t lds_bytes = (size_t)(LDS + TWB + TW3) * sizeof(V);
  static_assert(G % C == 0 || C % G == 0, "columns of a workgroup");
};

// Twiddles of a thread.  All threads load them; a barrier must follow.  ct: (c, tau) of
// e^{2 pi i m / 4096}; table: LDS behind the values.
template <class F, int SIGN>
struct ColTw {
  typedef typename F::V V;
  const V* b;      // second stage: the row of j % 16
  const V* t3;     // third stage: entries i of butterfly j + J g at t3[256 i + J g]
  static __device__ __forceinline__ V at(const V* __restrict__ ct, int m) {
    V x = ct[m];
    if (SIGN < 0) x.y = -x.y;
    return x;
  }
  __device__ __forceinline__ void load(const V* __restrict__ ct, V* table, int j) {
    for (int e = threadIdx.x; e < 16 * kTw16; e += F::NT)
      table[(e / kTw16) * kTwbStride + e % kTw16] = at(ct, tw_exponent<16>(e % kTw16, 16 * (e / kTw16)));
    b = table + (j % 16) * kTwbStride;
    t3 = table + F::TWB + j;
    for (int e = threadIdx.x; e < F::TW3; e += F::NT)
      table[F::TWB + e] = at(ct, tw_exponent<F::R3>(e / 256, (e % 256) * (4096 / F::L)));
  }
  __device__ __forceinline__ V third(int i) const { return t3[256 * (i % F::PER) + F::J * (i / F::PER)]; }
};

// The stages after the first.  On entry v holds the first stage's DFT of the thread (c0, j0):
// slot s its frequency dft16_freq(s) over x[j0 + J r], r < 16.  On return slot q of thread (c, j)
// holds output col_fft_out(j, q) of column c.  (c0, j0) and (c, j) are two numberings of the threads.
// The caller puts a barrier between its last use of LDS and the call, none after it is needed
// before the next call's writes but the one this function ends with.
template <class F, int SIGN>
__device__ __forceinline__ void col_fft_rest(typename F::V (&v)[16], typename F::V* buf, const ColTw<F, SIGN>& tw,
                                             int c0, int j0, int c, int j) {
  typedef typename F::V V;
  V* in = buf + c0 * F::LP + 17 * j0;
#pragma unroll
  for (int s = 0; s < 16; ++s) in[dft16_freq(s)] = v[s];
  __syncthreads();
  V* col = buf + c * F::LP + lpad(j);
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = col[r * (F::J + F::J / 16)];
  __syncthreads();
  dft_tw<16, SIGN>(v, [&](int i) { return tw.b[i]; });
  if constexpr (F::R3 > 1) {
    V* mid = buf + c * F::LP + (j / 16) * 272 + (j % 16);
#pragma unroll
    for (int s = 0; s < 16; ++s) mid[17 * dft16_freq(s)] = v[s];
    __syncthreads();
#pragma unroll
    for (int g = 0; g < 16 / F::R3; ++g)
#pragma unroll
      for (int u = 0; u < F::R3; ++u) v[g * F::R3 + u] = col[g * (F::J + F::J / 16) + 272 * u];
    __syncthreads();
    dft_tw<F::R3, SIGN>(v, [&](int i) { return tw.third(i); });
  }
}
// Output index of slot q: j + a constant.
template <class F>
__device__ __forceinline__ constexpr int col_fft_step(int q) {
  if (F::R3 == 1) return 16 * dft16_freq(q);
  return F::J * (q / F::R3) + 256 * dftr_freq<F::R3>(q % F::R3);
}

}  // namespace rfd
