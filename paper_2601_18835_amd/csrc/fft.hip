// Two-pass Stockham FFTs with fused loads and stores.
//
// N = N1 * N2.  For z[n] = sum_i Q[i] exp(s 2 pi i i n / N) with
// i = i1 + N1 i2 and n = n2 + N2 n1:
//   pass A (per column i1): X[i1][n2] = sum_i2 Q[i1 + N1 i2] exp(s 2 pi i i2 n2 / N2),
//           times exp(s 2 pi i i1 n2 / N), stored at Y[n2 N1 + i1];
//   pass B (per row n2):    z[n2 + N2 n1] = sum_i1 Y[n2 N1 + i1] exp(s 2 pi i i1 n1 / N1).
// Each workgroup transforms C adjacent columns (pass A) or rows (pass B) in
// LDS, so every global access is a run of C contiguous elements.  The first
// pass fuses the pointwise product of Eq. 1 (data x conj(template) x weight);
// the second fuses the consumer: spectrum store, reference-series store with
// its 16-bit hi/lo planes.  Tap construction evaluates only the T
// correlation lags it keeps: each pass-A workgroup reduces its columns at
// once to its share of every kept lag (k_corr_part, k_corr_reduce), or, where
// those shares would not fit the work buffer, pass A stores the rows the lags
// read and k_lags_direct sums them.  FINDCHIRP's own transforms live with its
// kernels.
#include <algorithm>
#include <type_traits>

#include "col_fft.h"
#include "dev_common.h"
#include "rfd_internal.h"

namespace rfd {

constexpr int kNT = 256;

template <typename V> struct Cols;
template <> struct Cols<float2> { static constexpr int value(int L) { return L >= 2048 ? 4 : 8; } };   // 8 columns of 2048 spill registers
template <> struct Cols<double2> { static constexpr int value(int L) { return L >= 2048 ? 2 : 4; } };

template <typename V, int L, int C>
constexpr size_t lds_bytes() { return (size_t)C * lds_col<L>() * sizeof(V) + (size_t)(L + L / 16) * sizeof(V); }

// ---------------------------------------------------------------- loaders
__device__ __forceinline__ uint32_t clamp_bin(int i, int64_t lo, int64_t hi) {
  return (uint32_t)std::min<int>(std::max<int>(i, (int)lo), (int)hi);
}
// For the transforms of col_fft.h a loader gives each element as an operand that every batch entry
// shares (fixed: read once per thread) and one of the entry (var: the load alone), joined by join.
// kHalf: elements past bin N / 2 - 1 vanish.  Bins outside the band carry a zero in `fixed` and
// read the first bin of the band, so that what a caller keeps there is never met.
struct LoadData64 {        // real FP64 series, scaled, FP64 complex
  static constexpr bool kHalf = false;
  typedef double Fixed; typedef double Var;
  __device__ double fixed(int) const { return scale; }
  __device__ double var(int, int i) const { return x[i]; }
  __device__ double2 join(int, int, double s, double v) const { return make_double2(v * s, 0.0); }
  const double* x; double scale;
  __device__ double2 operator()(int, int64_t i) const { return make_double2(x[i] * scale, 0.0); }
};
// References of one batched dechirp, carried by value in the kernel arguments
// (so eager launches and captured graphs need no pointer table in memory).
struct DechirpRefs {
  const double2* h[kDechirpBatch];   // reference templates, complex128 [nb]
  int32_t slot[kDechirpBatch];       // reference-series slots they fill
};
// Loaders with a Raw type split an element into fetch (the loads only, no
// branch: an out-of-band lane reads bin i_low and gets a zero weight) and make
// (the arithmetic), so that a thread can have the loads of several elements
// in flight before it combines any (see gather_columns).
struct LoadDechirpRefs {   // s_i w_i conj(h_b,i) / (sigma_b alpha) over the band, FP64
  const double2* s; const double* w; DechirpRefs r; const double* scale; int64_t i_low, i_high;
  static constexpr bool kHalf = true;
  typedef double2 Fixed; typedef double2 Var;
  __device__ double2 fixed(int i) const {
    if (i < i_low || i > i_high) return make_double2(0.0, 0.0);
    const double2 x = s[i];
    return make_double2(w[i] * x.x, w[i] * x.y);
  }
  __device__ double2 var(int b, int i) const { return r.h[b][clamp_bin(i, i_low, i_high)]; }
  __device__ double2 join(int b, int, double2 f, double2 h) const {
    const double2 v = cmul(f, cconj(h));
    return make_double2(v.x * scale[b], v.y * scale[b]);
  }
  struct Raw { double2 h, s; double w; };
  __device__ Raw fetch(int b, int64_t i) const {
    const bool in = i >= i_low && i <= i_high;
    const int64_t k = in ? i : i_low;
    Raw x;
    x.h = r.h[b][k];
    x.s = s[k];
    x.w = w[k];
    if (!in) x.w = 0.0;
    return x;
  }
  __device__ double2 make(int b, int64_t, const Raw& x) const {
    const double f = x.w * scale[b];
    return cmul(x.s, make_double2(f * x.h.x, -f * x.h.y));
  }
  __device__ double2 operator()(int b, int64_t i) const { return make(b, i, fetch(b, i)); }
};
struct LoadDechirpRefs32 { // the same integrand, formed in FP64 and rounded once to FP32
  LoadDechirpRefs d;
  static constexpr bool kHalf = true;
  typedef double2 Fixed; typedef double2 Var;
  __device__ double2 fixed(int i) const { return d.fixed(i); }
  __device__ double2 var(int b, int i) const { return d.var(b, i); }
  __device__ float2 join(int b, int i, double2 f, double2 h) const {
    const double2 v = d.join(b, i, f, h);
    return make_float2((float)v.x, (float)v.y);
  }
  using Raw = LoadDechirpRefs::Raw;
  __device__ Raw fetch(int b, int64_t i) const { return d.fetch(b, i); }
  __device__ float2 make(int b, int64_t i, const Raw& x) const {
    const double2 v = d.make(b, i, x);
    return make_float2((float)v.x, (float)v.y);
  }
  __device__ float2 operator()(int b, int64_t i) const { return make(b, i, fetch(b, i)); }
};
struct LoadBands {         // the integrand of one reference on bins [e[b], e[b + 1]), FP64
  const double2* s; const double* w; const double2* h; const double* scale;
  const int32_t* e;          // the batch's edges, on the device
  int nb;                    // its bands
  static constexpr bool kHalf = true;
  typedef double2 Fixed; typedef int2 Var;     // (nothing differs between bands but the range)
  __device__ double2 fixed(int i) const {
    if (i < e[0] || i >= e[nb]) return make_double2(0.0, 0.0);
    const double f = w[i] * scale[0];
    const double2 x = h[i];
    return cmul(s[i], make_double2(f * x.x, -f * x.y));
  }
  __device__ int2 var(int b, int) const { return make_int2(e[b], e[b + 1]); }
  __device__ double2 join(int, int i, double2 f, int2 range) const {
    return i >= range.x && i < range.y ? f : make_double2(0.0, 0.0);
  }
  struct Raw { double2 h, s; double w; };
  __device__ Raw fetch(int b, int64_t i) const {
    const bool in = i >= e[b] && i < e[b + 1];
    const int64_t k = in ? i : e[b];
    Raw x;
    x.h = h[k];
    x.s = s[k];
    x.w = w[k];
    if (!in) x.w = 0.0;
    return x;
  }
  __device__ double2 make(int b, int64_t, const Raw& x) const {
    const double f = x.w * scale[0];
    return cmul(x.s, make_double2(f * x.h.x, -f * x.h.y));
  }
  __device__ double2 operator()(int b, int64_t i) const { return make(b, i, fetch(b, i)); }
};
struct LoadFindchirp {     // s_i * F_j,i with F_j stored over band bins
  const float2* s; const float2* f; int64_t i_low, i_high, n_band;
  __device__ float2 operator()(int b, int64_t i) const {
    if (i < i_low || i > i_high) return make_float2(0.f, 0.f);
    return cmul(s[i], f[(int64_t)b * n_band + (i - i_low)]);
  }
};
struct LoadCorr64 {        // FP64 correlation integrands (tap construction, streaming series)
  const double* w; const double2* hr; const double2* ht; int64_t nb, i_low, i_high; int mode;
  const double* bscale;    // mode 0: per-member factor folded into the integrand (nullptr: none)
  static constexpr bool kHalf = true;
  typedef double2 Fixed; typedef double2 Var;
  __device__ double2 fixed(int i) const {
    if (i < i_low || i > i_high) return make_double2(0.0, 0.0);
    const double2 r = hr[i];
    const double rr = r.x * r.x + r.y * r.y;
    if (mode == 1) return make_double2(w[i] * rr, 0.0);
    if (mode == 0) return make_double2(w[i] * r.x, -w[i] * r.y);
    return w[i] * rr > 0.0 ? make_double2(r.x / rr, -r.y / rr) : make_double2(0.0, 0.0);
  }
  __device__ double2 var(int b, int i) const { return (ht + (int64_t)b * nb)[clamp_bin(i, i_low, i_high)]; }
  __device__ double2 join(int b, int, double2 f, double2 t) const {
    if (mode == 1) return f;
    const double2 v = cmul(f, t);
    return bscale ? make_double2(v.x * bscale[b], v.y * bscale[b]) : v;
  }
  struct Raw { double2 r, t; double w; };
  __device__ Raw fetch(int b, int64_t i) const {
    const bool in = i >= i_low && i <= i_high;
    const int64_t k = in ? i : i_low;
    Raw x;
    x.r = hr[k];
    x.t = ht[(int64_t)b * nb + k];     // (mode 1: ht is hr, unused)
    x.w = w[k];
    if (!in) x.w = 0.0;
    return x;
  }
  __device__ double2 make(int b, int64_t, const Raw& x) const {
    const double2 r = x.r, t = x.t;
    double wi = x.w;
    if (mode == 1) return make_double2(wi * (r.x * r.x + r.y * r.y), 0.0);
    if (bscale) wi *= bscale[b];
    if (mode == 0) return make_double2(wi * (t.x * r.x + t.y * r.y), wi * (t.y * r.x - t.x * r.y));
    // mode 2: ratio R = t / r where the chi^2 weight w |r|^2 is non-zero
    const double rr = r.x * r.x + r.y * r.y;
    if (!(wi * rr > 0.0)) return make_double2(0.0, 0.0);
    return make_double2((t.x * r.x + t.y * r.y) / rr, (t.y * r.x - t.x * r.y) / rr);
  }
  __device__ double2 operator()(int b, int64_t i) const { return make(b, i, fetch(b, i)); }
};

// The same integrands rounded once to FP32.  w_i alone is of order 1 / S_n
// (about 1e46 for a strain PSD), so an unnormalised integrand overflows FP32:
// FP32 callers fold the normalisation of the result in through bscale (the
// streaming series use 1 / (sigma_ref alpha), as the FP32 dechirp passes do).
struct LoadCorr32 {
  LoadCorr64 d;
  static constexpr bool kHalf = true;
  typedef double2 Fixed; typedef double2 Var;
  __device__ double2 fixed(int i) const { return d.fixed(i); }
  __device__ double2 var(int b, int i) const { return d.var(b, i); }
  __device__ float2 join(int b, int i, double2 f, double2 t) const {
    const double2 v = d.join(b, i, f, t);
    return make_float2((float)v.x, (float)v.y);
  }
  using Raw = LoadCorr64::Raw;
  __device__ Raw fetch(int b, int64_t i) const { return d.fetch(b, i); }
  __device__ float2 make(int b, int64_t i, const Raw& x) const {
    const double2 v = d.make(b, i, x);
    return make_float2((float)v.x, (float)v.y);
  }
  __device__ float2 operator()(int b, int64_t i) const { return make(b, i, fetch(b, i)); }
};

// ---------------------------------------------------------------- storers
struct StoreSpectrum64 {   // FP64 spectrum and its FP32 copy (FINDCHIRP operand)
  double2* s64; float2* s32; int64_t half;
  __device__ void operator()(int, int64_t n, double2 v) const {
    if (n <= half) {
      s64[n] = v;
      s32[n] = make_float2((float)v.x, (float)v.y);
    }
  }
};
// Reference series are stored as FP32 only; the 16-bit hi/lo planes the MFMA
// forms read are split from them by the FIR launch, over the window it reads.
struct StoreRefSlots {     // FP64 series -> FP32, into the slot of batch entry b
  float2* z; int64_t n; DechirpRefs r;
  __device__ void operator()(int b, int64_t m, double2 v) const {
    z[(int64_t)r.slot[b] * n + m] = make_float2((float)v.x, (float)v.y);
  }
};
struct StoreRefSlots32 {   // FP32 series into the slot of batch entry b
  float2* z; int64_t n; DechirpRefs r;
  __device__ void operator()(int b, int64_t m, float2 v) const { z[(int64_t)r.slot[b] * n + m] = v; }
};
struct StoreBand {         // FP64 series -> FP32 band series [b][n]
  float2* z; int64_t n;
  __device__ void operator()(int b, int64_t m, double2 v) const {
    z[(int64_t)b * n + m] = make_float2((float)v.x, (float)v.y);
  }
};

// ------------------------------------------------------------------ passes
template <typename V, int L>
__device__ void load_twl(V* twl, const V* __restrict__ tab, int stride = 1) {
  for (int k = threadIdx.x; k < L; k += kNT) twl[lpad(k)] = tab[k * stride];
}

// The C columns c0 + c (stride n1 through the input) into LDS, [C][LP]
// padded.  Each thread issues U elements' loads before storing any, so U
// memory round trips overlap (one at a time, the loop waited for every load).
template <class LD, class = void> struct HasRaw : std::false_type {};
template <class LD> struct HasRaw<LD, std::void_t<typename LD::Raw>> : std::true_type {};

// elements per thread in flight: at most U, and no more than a thread has
// (C L and kNT are powers of two, so U * kNT divides C L when C L >= kNT)
template <int E, int U>
__host__ __device__ constexpr int gather_batch() { return E / kNT >= U ? U : (E / kNT >= 1 ? E / kNT : 1); }

template <typename V, int L, int C, int U0, class LD>
__device__ __forceinline__ void gather_columns(V* buf, const LD& ld, int b, int c0, int n1) {
  constexpr int LP = lds_col<L>();
  constexpr int E = C * L;
  constexpr int U = gather_batch<E, U0>();
  for (int e0 = 0; e0 < E; e0 += U * kNT) {
    if constexpr (HasRaw<LD>::value) {
      typename LD::Raw x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = e0 + u * kNT + (int)threadIdx.x;
        if (E % (U * kNT) == 0 || e < E) x[u] = ld.fetch(b, (int64_t)(c0 + e % C) + (int64_t)n1 * (e / C));
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = e0 + u * kNT + (int)threadIdx.x;
        if (E % (U * kNT) == 0 || e < E)
          buf[(e % C) * LP + lpad(e / C)] = ld.make(b, (int64_t)(c0 + e % C) + (int64_t)n1 * (e / C), x[u]);
      }
    } else {
      V v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = e0 + u * kNT + (int)threadIdx.x;
        if (E % (U * kNT) == 0 || e < E) v[u] = ld(b, (int64_t)(c0 + e % C) + (int64_t)n1 * (e / C));
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = e0 + u * kNT + (int)threadIdx.x;
        if (E % (U * kNT) == 0 || e < E) buf[(e % C) * LP + lpad(e / C)] = v[u];
      }
    }
  }
}
constexpr int kGatherU = 8;

// pass A: L = N2-point transforms of C columns; writes Y with the inter-pass
// twiddle.  tabL[k * tab_stride] = exp(+2 pi i k / L).  Only the rows n2 in
// [row_lo, row_lo + row_cnt) mod L are written (all rows: 0, L): a consumer
// that evaluates a few outputs of the second pass reads no others.
template <typename V, int L, class LD>
__global__ __launch_bounds__(kNT) void k_pass_a(LD ld, V* __restrict__ Y, const V* __restrict__ coarse,
                                              const V* __restrict__ fine, const V* __restrict__ tabL,
                                              int n1, int sign, int tab_stride, int row_lo, int row_cnt) {
  constexpr int C = Cols<V>::value(L);
  constexpr int LP = lds_col<L>();
  extern __shared__ __align__(16) unsigned char smem[];
  V* buf = reinterpret_cast<V*>(smem);
  V* twl = buf + C * LP;
  const int b = blockIdx.y;
  const int c0 = blockIdx.x * C;
  const int64_t n = (int64_t)n1 * L;
  load_twl<V, L>(twl, tabL, tab_stride);
  gather_columns<V, L, C, kGatherU>(buf, ld, b, c0, n1);
  __syncthreads();
  lds_fft<V, L, C, kNT>(buf, twl, sign);
  V* Yb = Y + (int64_t)b * n;
  for (int e = threadIdx.x; e < C * L; e += kNT) {
    int c = e % C, n2 = e / C;
    if (((n2 - row_lo) & (L - 1)) >= row_cnt) continue;
    int i1 = c0 + c;
    V v = buf[c * LP + lpad(n2)];
    uint32_t p = (uint32_t)i1 * (uint32_t)n2;   // < N
    if (p) v = cmul(v, twiddle_n(coarse, fine, p, sign));
    Yb[(int64_t)n2 * n1 + i1] = v;
  }
}

template <typename V, int L>
__device__ void pass_b_load(const V* __restrict__ Yb, V* buf, V* twl, const V* __restrict__ tabL, int r0) {
  constexpr int C = Cols<V>::value(L);
  constexpr int LP = lds_col<L>();
  load_twl<V, L>(twl, tabL);
  constexpr int E = C * L;
  constexpr int U = gather_batch<E, kGatherU>();
  for (int e0 = 0; e0 < E; e0 += U * kNT) {      // U loads in flight per thread
    V v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * kNT + (int)threadIdx.x;
      if (E % (U * kNT) == 0 || e < E) v[u] = Yb[(int64_t)(r0 + e / L) * L + e % L];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * kNT + (int)threadIdx.x;
      if (E % (U * kNT) == 0 || e < E) buf[(e / L) * LP + lpad(e % L)] = v[u];
    }
  }
  __syncthreads();
}

// storers that also reduce over a workgroup's outputs
template <class ST, class = void> struct HasDone : std::false_type {};
template <class ST> struct HasDone<ST, std::void_t<decltype(&ST::done)>> : std::true_type {};

// pass B: L = N1-point transforms of C rows, generic storer
template <typename V, int L, class ST>
__global__ __launch_bounds__(kNT) void k_pass_b(const V* __restrict__ Y, ST st, const V* __restrict__ tabL,
                                              int n2, int sign) {
  constexpr int C = Cols<V>::value(L);
  constexpr int LP = lds_col<L>();
  extern __shared__ __align__(16) unsigned char smem[];
  V* buf = reinterpret_cast<V*>(smem);
  V* twl = buf + C * LP;
  const int b = blockIdx.y;
  const int r0 = blockIdx.x * C;
  const V* Yb = Y + (int64_t)b * L * n2;
  pass_b_load<V, L>(Yb, buf, twl, tabL, r0);
  lds_fft<V, L, C, kNT>(buf, twl, sign);
  for (int e = threadIdx.x; e < C * L; e += kNT) {
    int c = e % C, n1 = e / C;
    st(b, (int64_t)(r0 + c) + (int64_t)n2 * n1, buf[c * LP + lpad(n1)]);
  }
  if constexpr (HasDone<ST>::value) st.done(b, blockIdx.x, gridDim.x);
}


// ------------------------------------------- passes with register transforms
// Columns per workgroup: 512 to 1024 threads per CU with two to four workgroups' LDS, and runs of
// 64 to 256 contiguous bytes in every global access.
template <typename V, int L> struct ColsOf;
template <int L> struct ColsOf<float2, L> { static constexpr int value = L == 256 ? 16 : (L == 2048 ? 4 : 8); };
template <int L> struct ColsOf<double2, L> { static constexpr int value = L == 256 ? 16 : (L == 512 ? 8 : 4); };
template <typename V, int L> using Fft = ColFft<V, L, ColsOf<V, L>::value>;

__device__ __forceinline__ double2 to_v(double2 v, double2) { return v; }
__device__ __forceinline__ float2 to_v(double2 v, float2) { return make_float2((float)v.x, (float)v.y); }

// A thread's first-stage inputs x[j + J r] of column i1 for batch entry b.
template <class F, class LD>
struct ColInput {
  static constexpr int NR = LD::kHalf ? 8 : 16;
  typename LD::Fixed f[NR];
  typename LD::Var x[NR];
  int i0, step;
  __device__ __forceinline__ void init(const LD& ld, int i1, int j, int n1) {
    i0 = i1 + n1 * j;
    step = n1 * F::J;
#pragma unroll
    for (int r = 0; r < NR; ++r) f[r] = ld.fixed(i0 + step * r);
  }
  __device__ __forceinline__ void fetch(const LD& ld, int b) {
#pragma unroll
    for (int r = 0; r < NR; ++r) x[r] = ld.var(b, i0 + step * r);
  }
  template <int SIGN>
  __device__ __forceinline__ void first_stage(const LD& ld, int b, typename F::V (&v)[16]) {
#pragma unroll
    for (int r = 0; r < NR; ++r) v[r] = ld.join(b, i0 + step * r, f[r], x[r]);
    if constexpr (LD::kHalf) dft16_half<SIGN>(v);
    else dft16<SIGN>(v);
  }
};

// Pass A (as k_pass_a): columns [g C, (g + 1) C) of batch entries [y JT, (y + 1) JT), the next entry's
// operands fetched during the current transform.  The inter-pass factor w_N^(i1 n2) of a
// thread's outputs turns by constant angles from one to the next: FP64 rotations from three table
// values, rounded to V.  In FP64, where chains of up to 16 doubled the error of the correlations, every fourth factor
// is a table product of its own.  Neighbouring column groups, whose runs share cache lines, go to one XCD.
// Bound by memory where the batch is large: 16 FP64 correlations at N = 2^20 read 134 MB and write
// 268 MB in 96 us (325 us with the radix-4 transform in LDS, k_pass_a, which the lengths
// below 256 keep); 8 FP32 reference integrands 66 -> 36 us; the data transform 24 -> 13 us.
template <class F, int SIGN, class LD>
__global__ __launch_bounds__(F::NT) __attribute__((amdgpu_waves_per_eu(2))) void k_cols(LD ld, typename F::V* __restrict__ Y,
                                               const double2* __restrict__ coarse, const double2* __restrict__ fine,
                                               const typename F::V* __restrict__ ct, int n1, int count, int JT,
                                               int row_lo, int row_cnt) {
  typedef typename F::V V;
  extern __shared__ __align__(16) unsigned char smem[];
  V* buf = reinterpret_cast<V*>(smem);
  const int c = threadIdx.x % F::C, j = threadIdx.x / F::C;
  const int i1 = (int)xcd_contiguous(blockIdx.x, gridDim.x) * F::C + c;
  ColTw<F, SIGN> tw;
  tw.load(ct, buf + F::LDS, j);
  const int b0 = blockIdx.y * JT, b1 = min(b0 + JT, count);
  ColInput<F, LD> in;
  in.init(ld, i1, j, n1);
  in.fetch(ld, b0);
  const uint32_t nmask = (uint32_t)n1 * F::L - 1;
  const double2 base = twiddle_n(coarse, fine, (uint32_t)i1 * (uint32_t)j & nmask, SIGN);
  const double2 turn_g = twiddle_n(coarse, fine, (uint32_t)i1 * (uint32_t)F::J & nmask, SIGN);
  const double2 turn_f = twiddle_n(coarse, fine, (uint32_t)i1 * (F::R3 == 1 ? 16u : 256u) & nmask, SIGN);
  __syncthreads();       // the twiddle table is complete
  for (int b = b0; b < b1; ++b) {
    V v[16];
    in.template first_stage<SIGN>(ld, b, v);
    in.fetch(ld, min(b + 1, b1 - 1));
    col_fft_rest<F, SIGN>(v, buf, tw, c, j, c, j);
    V* Yb = Y + (int64_t)b * n1 * F::L;
    int jo = j;                                      // formed anew: 16 row addresses carried through
    asm volatile("" : "+v"(jo));                     // the loop would take 32 registers
    constexpr bool kAnew = sizeof(V) == 16;
    constexpr int RF = F::R3 == 1 ? 16 : F::R3;      // outputs per group, turn_f apart
    double2 wg = base;                               // (likewise: 16 factors would take 64)
    if constexpr (!kAnew) asm volatile("" : "+v"(wg.x), "+v"(wg.y));
#pragma unroll
    for (int g = 0; g < 16 / RF; ++g) {
      double2 w = wg;
#pragma unroll
      for (int f = 0; f < RF; ++f) {
        int q = g * RF;                              // slot of the group's frequency f
#pragma unroll
        for (int s = 0; s < RF; ++s)
          if ((F::R3 == 1 ? dft16_freq(s) : dftr_freq<F::R3>(s)) == f) q = g * RF + s;
        const int n2 = jo + col_fft_step<F>(q);
        if (kAnew && (g * RF + f) % 4 == 0) {
          w = twiddle_n(coarse, fine, (uint32_t)i1 * (uint32_t)n2 & nmask, SIGN);
          if (f == 0) wg = w;
        }
        if (((n2 - row_lo) & (F::L - 1)) < row_cnt) Yb[(uint32_t)(n2 * n1 + i1)] = cmul(v[q], to_v(w, V{}));
        if (f + 1 < RF && !(kAnew && (f + 1) % 4 == 0)) w = cmul(w, turn_f);
      }
      if (g + 1 < 16 / RF && !(kAnew && (g + 1) * RF % 4 == 0)) wg = cmul(wg, turn_g);
    }
  }
}

// Pass B (as k_pass_b): rows [x C, (x + 1) C) of batch entries [y JT, (y + 1) JT).  The first stage's
// threads run along a row, the last one's across the rows.  (8 FP32 series at N = 2^20: 41 -> 30 us; 16 FP64
// ones to |b|^2 193 -> 119; 16 chi^2 bands at 2^19 94 -> 41.)
template <class F, int SIGN, class ST>
__global__ __launch_bounds__(F::NT) __attribute__((amdgpu_waves_per_eu(2))) void k_rows(const typename F::V* __restrict__ Y, ST st,
                                               const typename F::V* __restrict__ ct, int n2, int count, int JT) {
  typedef typename F::V V;
  extern __shared__ __align__(16) unsigned char smem[];
  V* buf = reinterpret_cast<V*>(smem);
  const int j0 = threadIdx.x % F::J, c0 = threadIdx.x / F::J;
  const int c = threadIdx.x % F::C, j = threadIdx.x / F::C;
  const int r0 = (int)xcd_contiguous(blockIdx.x, gridDim.x) * F::C;
  ColTw<F, SIGN> tw;
  tw.load(ct, buf + F::LDS, j);
  const int b0 = blockIdx.y * JT, b1 = min(b0 + JT, count);
  const int64_t n = (int64_t)n2 * F::L;
  const V* row = Y + (int64_t)(r0 + c0) * F::L + j0;
  V nx[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) nx[r] = row[b0 * n + r * F::J];
  __syncthreads();       // the twiddle table is complete
  for (int b = b0; b < b1; ++b) {
    V v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = nx[r];
    const int bn = min(b + 1, b1 - 1);
#pragma unroll
    for (int r = 0; r < 16; ++r) nx[r] = row[bn * n + r * F::J];
    dft16<SIGN>(v);
    col_fft_rest<F, SIGN>(v, buf, tw, c0, j0, c, j);
    int jo = j;                                      // (as in k_cols)
    asm volatile("" : "+v"(jo));
#pragma unroll
    for (int q = 0; q < 16; ++q) st(b, r0 + c + n2 * (jo + col_fft_step<F>(q)), v[q]);
    if constexpr (HasDone<ST>::value) st.done(b, blockIdx.x, gridDim.x);
  }
}

// Batch entries per workgroup: enough workgroups for `per_cu` on every CU first, then as many entries
// as share a thread's tables and operands, up to 8.
static int entries_per_wg(int64_t groups, int count, int n_cu, int per_cu) {
  int jt = 1;
  while (jt < 8 && groups * ((count + 2 * jt - 1) / (2 * jt)) >= (int64_t)per_cu * n_cu) jt *= 2;
  return jt;
}
static const float2* tangents(const Plan& p, float2) { return p.ols_ct32; }
static const double2* tangents(const Plan& p, double2) { return p.ct64; }

// -------------------------------------------------------------- dispatch
template <int SIGN, typename V, class LD>
static int run_pass_a(Plan& p, LD ld, V* Y, const V* coarse, const V* fine, const V* tab2, int batch,
                      int row_lo = 0, int row_cnt = 1 << 30) {
  dim3 blk(kNT);
  switch (p.n2) {
#define CASE_A(LL)                                                                         \
  case LL: {                                                                               \
    constexpr int C = Cols<V>::value(LL);                                                  \
    size_t sh = lds_bytes<V, LL, C>();                                                     \
    hipLaunchKernelGGL((k_pass_a<V, LL, LD>), dim3(p.n1 / C, batch), blk, sh, p.stream, ld, Y, coarse, \
                       fine, tab2, p.n1, SIGN, 1, row_lo & (LL - 1), std::min(row_cnt, LL));  \
    break;                                                                                 \
  }
#define CASE_R(LL)                                                                                        \
  case LL: {                                                                                              \
    using F = Fft<V, LL>;                                                                                 \
    const int groups = p.n1 / F::C, jt = entries_per_wg(groups, batch, p.n_cu, 2);                         \
    const dim3 grid((unsigned)groups, (unsigned)((batch + jt - 1) / jt));                                  \
    const int lo = row_lo & (LL - 1), cnt = std::min(row_cnt, LL);                                         \
    hipLaunchKernelGGL((k_cols<F, SIGN, LD>), grid, dim3(F::NT), F::lds_bytes, p.stream, ld, Y,             \
                         (const double2*)p.tw64c, (const double2*)p.tw64f, tangents(p, V{}), p.n1, batch, jt, lo, cnt); \
    break;                                                                                                \
  }
    CASE_A(32) CASE_A(64) CASE_A(128)
    CASE_R(256) CASE_R(512) CASE_R(1024) CASE_R(2048)
#undef CASE_A
#undef CASE_R
    default: return fail(RFD_E_UNSUPPORTED, "fft: unsupported N2");
  }
  RFD_CHECK_LAUNCH();
  return RFD_OK;
}

template <int SIGN, typename V, class ST>
static int run_pass_b(Plan& p, const V* Y, ST st, const V* tab1, int batch) {
  dim3 blk(kNT);
  switch (p.n1) {
#define CASE_B(LL)                                                                          \
  case LL: {                                                                                \
    constexpr int C = Cols<V>::value(LL);                                                   \
    size_t sh = lds_bytes<V, LL, C>();                                                      \
    hipLaunchKernelGGL((k_pass_b<V, LL, ST>), dim3(p.n2 / C, batch), blk, sh, p.stream, Y, st, tab1, \
                       p.n2, SIGN);                                                         \
    break;                                                                                  \
  }
#define CASE_R(LL)                                                                                       \
  case LL: {                                                                                             \
    using F = Fft<V, LL>;                                                                                \
    const int groups = p.n2 / F::C, jt = entries_per_wg(groups, batch, p.n_cu, 2);                        \
    const dim3 grid((unsigned)groups, (unsigned)((batch + jt - 1) / jt));                                 \
    hipLaunchKernelGGL((k_rows<F, SIGN, ST>), grid, dim3(F::NT), F::lds_bytes, p.stream, Y, st, tangents(p, V{}), \
                         p.n2, batch, jt);                                                               \
    break;                                                                                               \
  }
    CASE_B(32) CASE_B(64) CASE_B(128)
    CASE_R(256) CASE_R(512) CASE_R(1024) CASE_R(2048)
#undef CASE_B
#undef CASE_R
    default: return fail(RFD_E_UNSUPPORTED, "fft: unsupported N1");
  }
  RFD_CHECK_LAUNCH();
  return RFD_OK;
}

// Only the T lags m = (k0 + l) mod N, l < T, of pass B's output, each as a
// direct sum over its row, z[m] = sum_i1 Y[n2 N1 + i1] exp(+2 pi i i1 n1 / N1)
// with n2 = m mod N2 and n1 = m div N2: tap construction keeps T of N
// outputs, and T N1 terms cost far less than the whole pass.  One wave per
// lag, FP64.
__global__ __launch_bounds__(256) void k_lags_direct(const double2* __restrict__ Y, int64_t n, int n1, int n2,
                                                   const double2* __restrict__ tab1, int k0,
                                                   const int32_t* __restrict__ k0s, int T, double scale,
                                                   double2* __restrict__ out, int64_t stride) {
  const int l = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (l >= T) return;                      // uniform per wave
  if (k0s) k0 = k0s[blockIdx.y];           // per-template lag window
  const int64_t m = ((int64_t)k0 + l) & (n - 1);
  const int64_t r = m % n2, c = m / n2;
  const double2* row = Y + (int64_t)blockIdx.y * n + r * n1;
  double re = 0.0, im = 0.0;
  for (int i1 = lane; i1 < n1; i1 += 64) {
    const double2 y = row[i1];
    const double2 w = tab1[(int)((i1 * c) & (n1 - 1))];
    re += y.x * w.x - y.y * w.y;
    im += y.x * w.y + y.y * w.x;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    re += __shfl_xor(re, o);
    im += __shfl_xor(im, o);
  }
  if (lane == 0) out[(int64_t)blockIdx.y * stride + l] = make_double2(re * scale, im * scale);
}

// Correlation lags without the pass-A intermediate: the workgroup's C
// column transforms (as k_pass_a, inter-pass twiddle included) are reduced at
// once to their share of every kept lag m = k0 + l,
//   part[b][g][l] = sum_{i1 in group g} Y[m mod N2][i1] exp(+2 pi i i1 (m div N2) / N1),
// and k_corr_reduce adds the N1 / C shares of each lag in a fixed order.
// V = double2: FP64 column transforms and shares (tap construction); V =
// float2: FP32 column transforms of the integrand rounded once from FP64, each
// share summed in FP64 and stored in FP32 (half the share traffic), the shares
// then added in FP64 (the streaming reference series, like the FP32 dechirp
// passes).
template <typename V, int L, class LD>
__global__ __launch_bounds__(kNT) void k_corr_part(LD ld, V* __restrict__ part, const double2* __restrict__ coarse,
                                                 const double2* __restrict__ fine, const V* __restrict__ tabL,
                                                 int n1, int k0, const int32_t* __restrict__ k0s, int T) {
  constexpr int C = Cols<V>::value(L);
  constexpr int LP = lds_col<L>();
  extern __shared__ __align__(16) unsigned char smem[];
  V* buf = reinterpret_cast<V*>(smem);
  V* twl = buf + C * LP;
  const int b = blockIdx.y;
  if (k0s) k0 = k0s[b];                    // per-template lag window
  // column group of this workgroup: consecutive workgroups go to different
  // XCDs (round robin over 8), so groups g and g + 1, which read the two
  // halves of the same cache lines, are given to workgroups of one XCD
  const int G = gridDim.x;
  const int g = (G % 8 == 0) ? (int)(blockIdx.x % 8) * (G / 8) + (int)(blockIdx.x / 8) : (int)blockIdx.x;
  const int c0 = g * C;
  const int64_t n = (int64_t)n1 * L;
  load_twl<V, L>(twl, tabL, 1);
  gather_columns<V, L, C, kGatherU>(buf, ld, b, c0, n1);
  __syncthreads();
  lds_fft<V, L, C, kNT>(buf, twl, +1);
  __syncthreads();
  // share of lag m = k0 + l: sum_c Y_c[m mod L] e^{+2 pi i (c0 + c) m / N}
  // (the inter-pass twiddle and the N1-point DFT at m div L in one factor).
  // The factor is e^{+2 pi i c0 m / N} (e^{+2 pi i m / N})^c, in FP64: the
  // first part turns by e^{+2 pi i c0 kNT / N} from one of the thread's lags
  // to its next, the second is read at m (consecutive over a wave's lanes), so
  // no table read depends on the column.
  V* pb = part + ((int64_t)b * G + g) * T;
  const uint64_t nmask = (uint64_t)n - 1;
  const uint64_t m_first = (uint64_t)((int64_t)k0 + (int64_t)threadIdx.x) & nmask;
  const double2 adv = twiddle_n(coarse, fine, (uint32_t)(((uint64_t)c0 * kNT) & nmask), +1);
  double2 base = twiddle_n(coarse, fine, (uint32_t)(((uint64_t)c0 * m_first) & nmask), +1);
  for (int l = threadIdx.x; l < T; l += kNT) {
    const uint32_t m = (uint32_t)((uint64_t)((int64_t)k0 + l) & nmask);
    const int r = (int)(m % L);
    const double2 step = twiddle_n(coarse, fine, m, +1);
    double2 f = base;
    double re = 0.0, im = 0.0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const V v = buf[c * LP + lpad(r)];
      re += (double)v.x * f.x - (double)v.y * f.y;
      im += (double)v.x * f.y + (double)v.y * f.x;
      if (c + 1 < C) f = cmul(f, step);
    }
    if constexpr (std::is_same<V, float2>::value)
      pb[l] = make_float2((float)re, (float)im);
    else
      pb[l] = make_double2(re, im);
    base = cmul(base, adv);
  }
}

// The same shares with the transforms of col_fft.h: the workgroup's columns pass through their
// stages in registers (as k_cols, batch entries [y JT, (y + 1) JT) in turn) and return to LDS in
// natural order, where each lag finds its row.  (16 FP64 correlations at N = 2^20, T = 1024: 208 -> 73 us
// against k_corr_part; 32 FP32 stretches of 3072 lags: 252 -> 116 us.)
// FP32 columns of 512 and 1024 points do without the fetch ahead: two workgroups then fit a CU
// (128 registers) and the one's loads pass under the other's lag sums (148 -> 122 us for those
// stretches).  The other lengths would spill.
template <class F> constexpr bool kLagAhead = sizeof(typename F::V) == 16 || F::L == 256 || F::L == 2048;
template <class F, class LD>
__global__ __launch_bounds__(F::NT) __attribute__((amdgpu_waves_per_eu(kLagAhead<F> ? 2 : 4))) void k_col_lags(
    LD ld, typename F::V* __restrict__ part, const double2* __restrict__ coarse, const double2* __restrict__ fine,
    const typename F::V* __restrict__ ct, int n1, int k0, const int32_t* __restrict__ k0s, int T, int count, int JT) {
  typedef typename F::V V;
  extern __shared__ __align__(16) unsigned char smem[];
  V* buf = reinterpret_cast<V*>(smem);
  const int c = threadIdx.x % F::C, j = threadIdx.x / F::C;
  const int g = (int)xcd_contiguous(blockIdx.x, gridDim.x);
  const int c0 = g * F::C;
  ColTw<F, 1> tw;
  tw.load(ct, buf + F::LDS, j);
  const int b0 = blockIdx.y * JT, b1 = min(b0 + JT, count);
  ColInput<F, LD> in;
  in.init(ld, c0 + c, j, n1);
  if constexpr (kLagAhead<F>) in.fetch(ld, b0);
  const uint32_t nmask = (uint32_t)n1 * F::L - 1;
  const double2 adv = twiddle_n(coarse, fine, (uint32_t)c0 * (uint32_t)F::NT & nmask, +1);
  __syncthreads();       // the twiddle table is complete
  for (int b = b0; b < b1; ++b) {
    V v[16];
    if constexpr (!kLagAhead<F>) in.fetch(ld, b);
    in.template first_stage<1>(ld, b, v);
    if constexpr (kLagAhead<F>) in.fetch(ld, min(b + 1, b1 - 1));
    col_fft_rest<F, 1>(v, buf, tw, c, j, c, j);
#pragma unroll
    for (int q = 0; q < 16; ++q) buf[c * F::LP + lpad(j + col_fft_step<F>(q))] = v[q];
    __syncthreads();
    if (k0s) k0 = k0s[b];                  // per-template lag window
    V* pb = part + ((int64_t)b * gridDim.x + g) * T;
    // share of lag m = k0 + l: e^{+2 pi i c0 m / N} sum_c Y_c[m mod L] (e^{+2 pi i m / N})^c, the sum by Horner's
    // rule and the factor before it turning from one of the thread's lags to its next, in FP64.  FP64 columns are
    // added four at a time: the error of e^{2 pi i m / N} grows with its power, at 16 to twice that of table products
    double2 base = twiddle_n(coarse, fine, (uint32_t)c0 * (uint32_t)(k0 + (int)threadIdx.x) & nmask, +1);
    for (int l = threadIdx.x; l < T; l += F::NT) {
      const uint32_t m = (uint32_t)(k0 + l) & nmask;
      const V* row = buf + lpad(m % F::L);
      const double2 step = twiddle_n(coarse, fine, m, +1);
      constexpr int Q = sizeof(V) == 16 && F::C > 4 ? 4 : F::C;
      auto horner = [&](double2 a, double2 w, V y) {
        return make_double2(fma(a.x, w.x, fma(-a.y, w.y, (double)y.x)), fma(a.x, w.y, fma(a.y, w.x, (double)y.y)));
      };
      auto columns = [&](int k) {            // k .. k + Q - 1
        double2 a = make_double2(row[(k + Q - 1) * F::LP].x, row[(k + Q - 1) * F::LP].y);
#pragma unroll
        for (int i = Q - 2; i >= 0; --i) a = horner(a, step, row[(k + i) * F::LP]);
        return a;
      };
      double2 acc = columns(F::C - Q);
      if constexpr (Q < F::C) {
        const double2 turn = twiddle_n(coarse, fine, Q * m & nmask, +1);
#pragma unroll
        for (int k = F::C - 2 * Q; k >= 0; k -= Q) acc = horner(acc, turn, columns(k));
      }
      pb[l] = to_v(cmul(acc, base), V{});
      if (sizeof(V) == 16 && l / F::NT % 4 == 3 && l + F::NT < T)       // (and chains of four here)
        base = twiddle_n(coarse, fine, (uint32_t)c0 * (uint32_t)(k0 + l + F::NT) & nmask, +1);
      else
        base = cmul(base, adv);
    }
    __syncthreads();                       // the next entry's first stage overwrites the rows
  }
}

// 32 lags per workgroup; 8 slices of the groups per lag (slice s adds groups
// s, s + 8, ...), then the slices in order: a fixed summation order.
template <typename V>
__global__ __launch_bounds__(256) void k_corr_reduce(const V* __restrict__ part, int groups, int T,
                                                   double scale, double2* __restrict__ out, int64_t stride) {
  __shared__ double2 red[8][32];
  const int ll = threadIdx.x & 31, sl = threadIdx.x >> 5;
  const int l = blockIdx.x * 32 + ll;
  double re = 0.0, im = 0.0;
  if (l < T) {
    const V* pb = part + (int64_t)blockIdx.y * groups * T + l;
    for (int g = sl; g < groups; g += 8) {
      const V v = pb[(int64_t)g * T];
      re += v.x;
      im += v.y;
    }
  }
  red[sl][ll] = make_double2(re, im);
  __syncthreads();
  if (sl == 0 && l < T) {
#pragma unroll
    for (int k = 1; k < 8; ++k) {
      re += red[k][ll].x;
      im += red[k][ll].y;
    }
    out[(int64_t)blockIdx.y * stride + l] = make_double2(re * scale, im * scale);
  }
}

// ------------------------------------------------------- small kernels
// sigma^2 = sum_i w_i |h_i|^2 in FP64 by one workgroup (fixed order).
__global__ __launch_bounds__(1024) void k_sigma_sq(const double* __restrict__ w, const double2* __restrict__ h,
                                                  int64_t nb, int64_t stride, double* __restrict__ out) {
  __shared__ double red[1024];
  const double2* hb = h + (int64_t)blockIdx.x * stride;
  double acc = 0.0;
  for (int64_t i = threadIdx.x; i < nb; i += 1024) {
    double2 v = hb[i];
    acc += w[i] * (v.x * v.x + v.y * v.y);
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 512; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = red[0];
}

// sigma^2 of each reference of a batch in two steps of fixed order:
// kSigParts workgroups per reference reduce contiguous bin ranges to
// partial sums, then one wave per reference adds its partials and
// stores sigma^2 by slot and the filter scale 1 / (sigma alpha): the workgroup that finishes last
// (LAST), or k_sigma_final.  A launch of its own costs 3 us and the gap before it (16
// FP32 templates on one reference: 76 us against 70 for the whole call), but each workgroup's release
// of its partial writes its L2 back, which 1024 of them pay for (16 references: 44 us, 90 with LAST).
// done: workgroups finished so far, a multiple of kSigParts between launches.
__device__ __forceinline__ void sigma_store(DechirpRefs& r, int b, double s2, double* sig2_by_slot, double* scale,
                                            double inv_alpha) {
#pragma unroll
  for (int o = kSigParts / 2; o > 0; o >>= 1) s2 += __shfl_xor(s2, o);
  if (threadIdx.x == 0) {
    sig2_by_slot[r.slot[b]] = s2;
    scale[b] = inv_alpha / sqrt(s2);
  }
}
template <bool LAST>
__global__ __launch_bounds__(256) void k_sigma_part(const double* __restrict__ w, DechirpRefs r, int64_t nb,
                                                   double* part, unsigned int* done,
                                                   double* __restrict__ sig2_by_slot, double* __restrict__ scale,
                                                   double inv_alpha) {
  __shared__ double red[4];
  __shared__ bool last;
  const double2* hb = r.h[blockIdx.y];
  const int64_t chunk = (nb + kSigParts - 1) / kSigParts;
  const int64_t i0 = (int64_t)blockIdx.x * chunk, i1 = std::min<int64_t>(i0 + chunk, nb);
  double acc = 0.0;
  int64_t i = i0 + threadIdx.x;
  for (; i + 256 * 7 < i1; i += 256 * 8) {       // eight bins' loads in flight (one at a time: 24 us for
    double2 v[8];                                // 8 references at N = 2^20)
    double u[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      v[k] = hb[i + 256 * k];
      u[k] = w[i + 256 * k];
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) acc += u[k] * (v[k].x * v[k].x + v[k].y * v[k].y);
  }
  for (; i < i1; i += 256) acc += w[i] * (hb[i].x * hb[i].x + hb[i].y * hb[i].y);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  double* mine = part + blockIdx.y * kSigParts;
  static_assert(kSigParts == 64, "one wave adds them (and the count wraps at a multiple)");
  if (threadIdx.x == 0) {
    mine[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
    if constexpr (LAST)
      last = __hip_atomic_fetch_add(done + blockIdx.y, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) % kSigParts ==
             kSigParts - 1;
  }
  if constexpr (LAST) {
    __syncthreads();
    if (!last || threadIdx.x >= kSigParts) return;
    const double s2 = __hip_atomic_load(mine + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    sigma_store(r, blockIdx.y, s2, sig2_by_slot, scale, inv_alpha);
  }
}
__global__ __launch_bounds__(kSigParts) void k_sigma_final(DechirpRefs r, const double* __restrict__ part,
                                                         double* __restrict__ sig2_by_slot,
                                                         double* __restrict__ scale, double inv_alpha) {
  sigma_store(r, blockIdx.x, part[blockIdx.x * kSigParts + threadIdx.x], sig2_by_slot, scale, inv_alpha);
}

// F[i] = w_i conj(h_i) / (sigma * alpha), FP64 then rounded to FP32.
__global__ void k_build_filter(const double* __restrict__ w, const double2* __restrict__ h, int64_t nb,
                               int64_t hstride, const double* __restrict__ sigma_sq, double inv_alpha,
                               int64_t i_low, int64_t n_band, float2* __restrict__ out, int64_t ostride,
                               int band_only) {
  const int b = blockIdx.y;
  const double s = inv_alpha / sqrt(sigma_sq[b]);
  int64_t cnt = band_only ? n_band : nb;
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < cnt; k += (int64_t)gridDim.x * blockDim.x) {
    int64_t i = band_only ? k + i_low : k;
    double2 v = h[(int64_t)b * hstride + i];
    double f = w[i] * s;
    out[(int64_t)b * ostride + k] = make_float2((float)(f * v.x), (float)(-f * v.y));
  }
}

__global__ void k_sqrt_to(const double* __restrict__ in, double* __restrict__ out, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = sqrt(in[i]);
}

// ------------------------------------------------------------ launchers
// The segment transform and the reference filters run in FP64: they are
// cheap (once per segment / per reference) and the ratio FIR amplifies any
// white rounding noise in the reference series by its out-of-band gain.
int launch_data_fft(Plan& p, const double* data) {
  LoadData64 ld{data, p.data_scale / p.fs};
  int rc = run_pass_a<-1, double2>(p, ld, p.work64, p.tw64c, p.tw64f, p.tw64_n2, 1);
  if (rc) return rc;
  StoreSpectrum64 st{p.stilde64, p.stilde, p.n / 2};
  return run_pass_b<-1, double2>(p, p.work64, st, p.tw64_n1, 1);
}

int dechirp_batch_size(const Plan& p) {
  // intermediates of a batch (FP32 or FP64 complex): at most 128 MiB and
  // kDechirpBatch references.  A batch's pass-A output then stays within
  // the 256 MB last-level cache when pass B reads it back, and its four launches
  // are few (32 references at N = 2^20, with the copies out: 651 us at 64 MiB, 619 at 128,
  // 596 at 256)
  const int64_t elem = p.dechirp_fp64 ? (int64_t)sizeof(double2) : (int64_t)sizeof(float2);
  int64_t b = ((int64_t)128 << 20) / (p.n * elem);
  return (int)std::max<int64_t>(1, std::min<int64_t>(b, kDechirpBatch));
}

size_t dechirp_work_double2(const Plan& p) {
  const int64_t elem = p.dechirp_fp64 ? (int64_t)sizeof(double2) : (int64_t)sizeof(float2);
  return (size_t)((dechirp_batch_size(p) * p.n * elem + (int64_t)sizeof(double2) - 1) / (int64_t)sizeof(double2));
}

// Every reference through the same launches, in batches: sigma^2 (by slot,
// into p.dref_sig2, from kSigParts partial sums each), then pass A with the filter formed on the fly, then
// pass B into each reference's slot of the series store.
int launch_dechirp_refs(Plan& p, int n_refs, const int32_t* ref_ids, const double* const* h_refs) {
  const int bs = dechirp_batch_size(p);
  double2* work = bs > 1 ? p.work64b : p.work64;
  if (bs > 1 && p.work64b_cap < dechirp_work_double2(p)) return fail(RFD_E_STATE, "dechirp: batch buffer too small");
  for (int r0 = 0; r0 < n_refs; r0 += bs) {
    const int nr = std::min(bs, n_refs - r0);
    DechirpRefs refs{};
    for (int b = 0; b < nr; ++b) {
      refs.h[b] = reinterpret_cast<const double2*>(h_refs[r0 + b]);
      refs.slot[b] = ref_ids[r0 + b];
    }
    const double inv_alpha = 1.0 / p.data_scale;
    const dim3 grid(kSigParts, (unsigned)nr);
    if (nr <= 2) {
      hipLaunchKernelGGL(k_sigma_part<true>, grid, dim3(256), 0, p.stream, p.w, refs, p.nb, p.dref_part, p.dref_done,
                         p.dref_sig2, p.dref_scale, inv_alpha);
    } else {
      hipLaunchKernelGGL(k_sigma_part<false>, grid, dim3(256), 0, p.stream, p.w, refs, p.nb, p.dref_part, p.dref_done,
                         p.dref_sig2, p.dref_scale, inv_alpha);
      RFD_CHECK_LAUNCH();
      hipLaunchKernelGGL(k_sigma_final, dim3((unsigned)nr), dim3(kSigParts), 0, p.stream, refs,
                         (const double*)p.dref_part, p.dref_sig2, p.dref_scale, inv_alpha);
    }
    RFD_CHECK_LAUNCH();
    LoadDechirpRefs ld{p.stilde64, p.w, refs, p.dref_scale, p.i_low, p.i_high};
    int rc;
    if (p.dechirp_fp64) {
      rc = run_pass_a<1, double2>(p, ld, work, p.tw64c, p.tw64f, p.tw64_n2, nr);
      if (rc) return rc;
      StoreRefSlots st{p.zref, p.n, refs};
      rc = run_pass_b<1, double2>(p, work, st, p.tw64_n1, nr);
    } else {
      // the integrand (and the reference norm) in FP64, both transform passes in
      // FP32 with twiddles rounded once from FP64
      float2* w32 = reinterpret_cast<float2*>(work);
      rc = run_pass_a<1, float2>(p, LoadDechirpRefs32{ld}, w32, p.tw32c, p.tw32f, p.tw32_n2, nr);
      if (rc) return rc;
      StoreRefSlots32 st{p.zref, p.n, refs};
      rc = run_pass_b<1, float2>(p, w32, st, p.tw32_n1, nr);
    }
    if (rc) return rc;
  }
  return RFD_OK;
}

// Band series of one reference: the dechirp integrand restricted to bins
// [edges[b], edges[b+1]) (on the device, as the reference's p.dref_scale is) and transformed, for bands
// [b0, b0 + nb) (FP32 out, [band][N]) through `work` (nb N values): one band's passes
// are 128 to 256 workgroups, half a wave of the chip, and 12 us each (16 bands of a 2^19
// segment: 390 us one by one, 75 us together).
int launch_band_cols(Plan& p, const double* h_ref, const int32_t* edges, int b0, int nb, double2* work) {
  const LoadBands ld{p.stilde64, p.w, reinterpret_cast<const double2*>(h_ref), p.dref_scale, edges + b0, nb};
  return run_pass_a<1, double2>(p, ld, work, p.tw64c, p.tw64f, p.tw64_n2, nb);
}

int launch_band_rows(Plan& p, int b0, int nb, float2* out, const double2* work) {
  return run_pass_b<1, double2>(p, work, StoreBand{out + (int64_t)b0 * p.n, p.n}, p.tw64_n1, nb);
}

int launch_findchirp_prepare(Plan& p, const double* h, int64_t count, float2* filt, double* sigma) {
  // sigma^2 into the output buffer (or scratch), then the filters
  double* s2 = sigma;
  for (int64_t b0 = 0; b0 < count; b0 += 65535) {
    int64_t nbat = count - b0 < 65535 ? count - b0 : 65535;
    hipLaunchKernelGGL(k_sigma_sq, dim3((unsigned)nbat), dim3(1024), 0, p.stream, p.w,
                       (const double2*)h + b0 * p.nb, p.nb, p.nb, s2 + b0);
    RFD_CHECK_LAUNCH();
    hipLaunchKernelGGL(k_build_filter, dim3(64, (unsigned)nbat), dim3(256), 0, p.stream, p.w,
                       (const double2*)h + b0 * p.nb, p.nb, p.nb, (const double*)(s2 + b0), 1.0 / p.data_scale,
                       p.i_low, p.n_band, filt + b0 * p.n_band, p.n_band, 1);
    RFD_CHECK_LAUNCH();
  }
  hipLaunchKernelGGL(k_sqrt_to, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, p.stream, s2, s2, count);
  RFD_CHECK_LAUNCH();
  return RFD_OK;
}

// FINDCHIRP pass A for N2 = N / 4096 > 256 (segments of 2^21 and 2^22
// samples): the LDS Stockham column transform into the [N2][4096] layout of
// the register-FFT row pass, twiddles from the 4096-entry table.
int launch_fc_cols_lds(Plan& p, const float2* filt, int nb, float2* Y, int n1, int n2) {
  LoadFindchirp ld{p.stilde, filt, p.i_low, p.i_high, p.n_band};
  dim3 blk(kNT);
  switch (n2) {
#define CASE_L(LL)                                                                             \
  case LL: {                                                                                   \
    constexpr int C = Cols<float2>::value(LL);                                                 \
    size_t sh = lds_bytes<float2, LL, C>();                                                    \
    hipLaunchKernelGGL((k_pass_a<float2, LL, LoadFindchirp>), dim3(n1 / C, nb), blk, sh, p.stream, \
                       ld, Y, p.tw32c, p.tw32f, p.ols_tw32, n1, +1, 4096 / LL, 0, LL);         \
    break;                                                                                     \
  }
    CASE_L(512) CASE_L(1024)
#undef CASE_L
    default: return fail(RFD_E_UNSUPPORTED, "findchirp: unsupported column length");
  }
  RFD_CHECK_LAUNCH();
  return RFD_OK;
}

// columns per workgroup of the lag shares at column length n2
template <typename V>
static int corr_columns(int n2) {
  switch (n2) {
    case 256: return Fft<V, 256>::C;
    case 512: return Fft<V, 512>::C;
    case 1024: return Fft<V, 1024>::C;
    case 2048: return Fft<V, 2048>::C;
    default: return Cols<V>::value(n2);
  }
}

// work-buffer values of one batch entry: the shares of its T lags, or its whole column transform
static int corr_groups(const Plan& p, bool fp32) {
  return p.n1 / (fp32 ? corr_columns<float2>(p.n2) : corr_columns<double2>(p.n2));
}
int64_t corr64_work(const Plan& p, int T) { return std::min<int64_t>((int64_t)corr_groups(p, false) * T, p.n); }

int launch_corr64(Plan& p, Taps& tp, int mode, const double* h_r, const double* h_t, int64_t batch, int T,
                  int k0, double2* out, int64_t out_stride, int64_t lo, int64_t hi, const int32_t* k0s, bool fp32,
                  const double* bscale) {
  const int groups = corr_groups(p, fp32);
  const bool shares = (int64_t)groups * T <= p.n;
  if (tp.work64_cap < (size_t)(batch * (shares ? (int64_t)groups * T : p.n)))
    return fail(RFD_E_INVALID, "corr64: work buffer too small");
  if (fp32 && mode == 0 && !bscale) return fail(RFD_E_INVALID, "corr64: FP32 integrands need their normalisation");
  // (a single-spectrum mode reads its spectrum as the second one too: the
  // loads need no branch on the mode)
  LoadCorr64 ld{p.w, (const double2*)h_r, (const double2*)(h_t ? h_t : h_r), h_t ? p.nb : 0,
                lo >= 0 ? lo : p.i_low, hi >= 0 ? hi : p.i_high, mode, mode == 0 ? bscale : nullptr};
  const double scale = mode == 2 ? 1.0 / (double)p.n : 1.0;
  // fused form: per-workgroup lag shares in the work buffer, then their sums
  if (shares) {
    dim3 blk(kNT);
    const int jt = entries_per_wg(groups, (int)batch, p.n_cu, 2);
    const dim3 grid_r((unsigned)groups, (unsigned)((batch + jt - 1) / jt));
    switch (p.n2) {
#define CASE_C(LL)                                                                                       \
  case LL: {                                                                                             \
    if (fp32) {                                                                                          \
      const size_t sh = lds_bytes<float2, LL, Cols<float2>::value(LL)>();                                \
      hipLaunchKernelGGL((k_corr_part<float2, LL, LoadCorr32>), dim3(groups, (unsigned)batch), blk, sh,  \
                         p.stream, LoadCorr32{ld}, (float2*)tp.work64, (const double2*)p.tw64c,             \
                         (const double2*)p.tw64f, p.tw32_n2, p.n1, k0, k0s, T);                            \
    } else {                                                                                             \
      const size_t sh = lds_bytes<double2, LL, Cols<double2>::value(LL)>();                              \
      hipLaunchKernelGGL((k_corr_part<double2, LL, LoadCorr64>), dim3(groups, (unsigned)batch), blk, sh, \
                         p.stream, ld, tp.work64, (const double2*)p.tw64c, (const double2*)p.tw64f,          \
                         p.tw64_n2, p.n1, k0, k0s, T);                                                     \
    }                                                                                                    \
    break;                                                                                               \
  }
#define CASE_R(LL)                                                                                       \
  case LL: {                                                                                             \
    if (fp32) {                                                                                          \
      using F = Fft<float2, LL>;                                                                         \
      hipLaunchKernelGGL((k_col_lags<F, LoadCorr32>), grid_r, dim3(F::NT), F::lds_bytes, p.stream,        \
                         LoadCorr32{ld}, (float2*)tp.work64, (const double2*)p.tw64c,                       \
                         (const double2*)p.tw64f, (const float2*)p.ols_ct32, p.n1, k0, k0s, T, (int)batch, jt); \
    } else {                                                                                             \
      using F = Fft<double2, LL>;                                                                        \
      hipLaunchKernelGGL((k_col_lags<F, LoadCorr64>), grid_r, dim3(F::NT), F::lds_bytes, p.stream, ld,    \
                         tp.work64, (const double2*)p.tw64c, (const double2*)p.tw64f,                       \
                         (const double2*)p.ct64, p.n1, k0, k0s, T, (int)batch, jt);                         \
    }                                                                                                    \
    break;                                                                                               \
  }
      CASE_C(32) CASE_C(64) CASE_C(128)
      CASE_R(256) CASE_R(512) CASE_R(1024) CASE_R(2048)
#undef CASE_C
#undef CASE_R
      default: return fail(RFD_E_UNSUPPORTED, "fft: unsupported N2");
    }
    RFD_CHECK_LAUNCH();
    if (fp32)
      hipLaunchKernelGGL(k_corr_reduce<float2>, dim3((unsigned)((T + 31) / 32), (unsigned)batch), dim3(256), 0,
                         p.stream, (const float2*)tp.work64, groups, T, scale, out, out_stride);
    else
      hipLaunchKernelGGL(k_corr_reduce<double2>, dim3((unsigned)((T + 31) / 32), (unsigned)batch), dim3(256), 0,
                         p.stream, (const double2*)tp.work64, groups, T, scale, out, out_stride);
    RFD_CHECK_LAUNCH();
    return RFD_OK;
  }
  // k_lags_direct reads the pass-A rows (k0 + l) mod N2, l < T (every row
  // when the lag window differs per template)
  const int row_lo = k0s ? 0 : (int)(((int64_t)k0 % p.n2 + p.n2) % p.n2);
  int rc = run_pass_a<1, double2>(p, ld, tp.work64, p.tw64c, p.tw64f, p.tw64_n2, (int)batch, row_lo,
                               k0s ? p.n2 : T);
  if (rc) return rc;
  hipLaunchKernelGGL(k_lags_direct, dim3((unsigned)((T + 3) / 4), (unsigned)batch), dim3(256), 0, p.stream,
                     (const double2*)tp.work64, p.n, p.n1, p.n2, (const double2*)p.tw64_n1, k0, k0s, T, scale, out,
                     out_stride);
  RFD_CHECK_LAUNCH();
  return RFD_OK;
}


// ------------------------------------------------- lag of the correlation peak
// Pass B's output b (natural order) and the largest |b|^2 of each workgroup's outputs with its
// index, the lowest on exact ties.
// (the correlations pass by the caches: little of them is read again, and they would evict the intermediates that
// this pass and the next batch's read from the last-level cache: 8 templates at N = 2^20 57 + 53 us -> 50 + 49)
struct StorePeak {
  double2* z;
  int64_t n;
  double* pv;        // [batch][groups]
  int32_t* pi;
  double best = -1.0;
  int at = 0;
  __device__ __forceinline__ void take(double v, int i) {
    if (v > best || (v == best && i < at)) {
      best = v;
      at = i;
    }
  }
  __device__ __forceinline__ void operator()(int b, int64_t i, double2 v) {
    typedef __attribute__((ext_vector_type(2))) double V;
    __builtin_nontemporal_store(__builtin_bit_cast(V, v), reinterpret_cast<V*>(z + (int64_t)b * n + i));
    take(v.x * v.x + v.y * v.y, (int)i);
  }
  __device__ __forceinline__ void done(int b, int group, int groups) {
    __shared__ double sv[16];
    __shared__ int si[16];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) take(__shfl_xor(best, o), __shfl_xor(at, o));
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
      sv[wave] = best;
      si[wave] = at;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int k = 1; k < (int)(blockDim.x >> 6); ++k) take(sv[k], si[k]);
      pv[(int64_t)b * groups + group] = best;
      pi[(int64_t)b * groups + group] = at;
    }
    __syncthreads();
    best = -1.0;
    at = 0;
  }
};

// Per template: the lag of the largest |b[l]|^2 over all N lags (lowest
// index 0..N-1 on exact ties) from its workgroups' maxima, mapped into
// (-N/2, N/2]; the lag window k0_j = peak - floor(T/2); and (out not NULL) the
// T lags k0_j + l of its full correlation. 256 lags per workgroup, whose
// waves each find the peak for themselves: one latency more in place of a launch before (4.7 + 4.6 us per
// batch of 8 templates, now 5).
__global__ __launch_bounds__(256) void k_peak(const double* __restrict__ pv, const int32_t* __restrict__ pi, int groups,
                                            const double2* __restrict__ z, int64_t n, int T,
                                            int32_t* __restrict__ k0_out, double2* __restrict__ out) {
  const int64_t t = blockIdx.y;
  StorePeak m{nullptr, 0, nullptr, nullptr};
  for (int c = threadIdx.x & 63; c < groups; c += 64) m.take(pv[t * groups + c], pi[t * groups + c]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m.take(__shfl_xor(m.best, o), __shfl_xor(m.at, o));
  const int k0 = (int)(m.at <= n / 2 ? m.at : m.at - n) - T / 2;
  if (blockIdx.x == 0 && threadIdx.x == 0) k0_out[t] = k0;
  const int l = blockIdx.x * 256 + threadIdx.x;
  if (out && l < T) out[t * T + l] = z[t * n + (((int64_t)k0 + l) & (n - 1))];
}

// workgroups per template of the FP64 row pass
static int row_groups(const Plan& p) {
  switch (p.n1) {
    case 256: return p.n2 / Fft<double2, 256>::C;
    case 512: return p.n2 / Fft<double2, 512>::C;
    case 1024: return p.n2 / Fft<double2, 1024>::C;
    case 2048: return p.n2 / Fft<double2, 2048>::C;
    default: return p.n2 / Cols<double2>::value(p.n1);
  }
}

// The correlations stay in z [batch][N]: with the lag windows chosen, least squares reads its right-hand sides from
// them (out, may be NULL) instead of transforming the templates again.  16 templates at
// N = 2^20, T = 1024: 365 us while the row pass kept |b|^2 alone, a second pass searched it and the kept lags were
// summed from a second column transform.
int launch_corr_peak(Plan& p, Taps& tp, const double* h_r, const double* h_t, int64_t batch, int T, double2* z,
                     int32_t* k0_out, double2* out) {
  if (tp.work64_cap < (size_t)batch * p.n) return fail(RFD_E_INVALID, "corr peak: work buffer too small");
  const int groups = row_groups(p);
  if (tp.peak_cap < (size_t)batch * p.n || tp.peak_parts_cap < (size_t)batch * kPeakParts || groups > kPeakParts)
    return fail(RFD_E_INVALID, "corr peak: scratch too small");
  LoadCorr64 ld{p.w, (const double2*)h_r, (const double2*)h_t, p.nb, p.i_low, p.i_high, 0, nullptr};
  int rc = run_pass_a<1, double2>(p, ld, tp.work64, p.tw64c, p.tw64f, p.tw64_n2, (int)batch);
  if (rc) return rc;
  rc = run_pass_b<1, double2>(p, (const double2*)tp.work64, StorePeak{z, p.n, tp.peak_part, tp.peak_idx}, p.tw64_n1,
                              (int)batch);
  if (rc) return rc;
  hipLaunchKernelGGL(k_peak, dim3(out ? (unsigned)((T + 255) / 256) : 1u, (unsigned)batch), dim3(256), 0, p.stream,
                     (const double*)tp.peak_part, (const int32_t*)tp.peak_idx, groups, (const double2*)z, p.n, T,
                     k0_out, out);
  RFD_CHECK_LAUNCH();
  return RFD_OK;
}

// Offsets of the lag windows from the sub-bank's k0.  Not part of the peak search: a call that is refused after its
// search leaves the offsets of the taps that stand.
__global__ void k_lag_shifts(const int32_t* __restrict__ k0s, int k0_sb, int64_t n, int32_t* __restrict__ d) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) d[i] = k0s[i] - k0_sb;
}
int launch_lag_shifts(Plan& p, const int32_t* k0s, int k0_sb, int64_t count, int32_t* d_out) {
  hipLaunchKernelGGL(k_lag_shifts, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, p.stream, k0s, k0_sb, count, d_out);
  RFD_CHECK_LAUNCH();
  return RFD_OK;
}

}  // namespace rfd
