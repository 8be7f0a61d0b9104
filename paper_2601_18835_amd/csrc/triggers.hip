// Trigger accumulation (Table II's last stage): slot clearing, deterministic
// compaction of the per-(template, window) peak keys by prefix sum, and the
// FP32 re-evaluation of the complex SNR at each trigger.
#include <algorithm>

#include "dev_common.h"
#include "rfd_internal.h"

namespace rfd {

constexpr int kSegThreads = 256;
constexpr int kSegPer = 16;
constexpr int kSeg = kSegThreads * kSegPer;   // slots per compaction block
// Each wave of a compaction block takes kSegPer rounds of 64 consecutive
// slots (1024 in all, coalesced 512-byte reads); the waves of a block and the
// blocks follow each other in slot order, so the triggers come out in
// ascending slot order.

// template and window of visit v (a 64-bit division costs tens of instructions: 32 bits serve
// nearly every call)
__device__ __forceinline__ void map_visit(const WinMap& m, int64_t v, int64_t& t, int64_t& qi) {
  t = v <= 0xFFFFFFFFll ? (int64_t)((uint32_t)v / (uint32_t)m.nq) : v / m.nq;
  qi = v - t * m.nq;
}
__device__ __forceinline__ int64_t map_window(const WinMap& m, int64_t qi) {
  return qi < m.cnt0 ? m.lo0 + qi : m.lo1 + (qi - m.cnt0);
}
__device__ __forceinline__ int64_t map_slot(const WinMap& m, int64_t v) {
  int64_t t, qi;
  map_visit(m, v, t, qi);
  return t * m.nwin + map_window(m, qi);
}
// every window of every template, in order: slot index = visit index
__device__ __forceinline__ bool map_identity(const WinMap& m) {
  return m.nq == m.nwin && m.cnt0 == m.nq && m.lo0 == 0;
}

__global__ void k_fill_u64(unsigned long long* __restrict__ p, int64_t n, WinMap m, unsigned long long* also) {
  const bool ident = map_identity(m);
  if (also && blockIdx.x == 0 && threadIdx.x == 0) *also = 0ull;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[ident ? i : map_slot(m, i)] = 0ull;
}

__device__ __forceinline__ bool slot_fires(unsigned long long k, float thr2) {
  return k != 0ull && __uint_as_float((uint32_t)(k >> 32)) > thr2;
}

// lanes below this one whose bit is set in a wave-wide mask
__device__ __forceinline__ int lanes_below(unsigned long long mask) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// The wave's keys and firing masks over its kSegPer rounds.  The visits of a lane are 64 apart, so
// its template and window follow from the round before by an addition: one division per
// lane, not one per slot (unrolled, those were most of 19 KB of code in k_count and, with those
// of the triggers, 58 KB in k_write, which a launch reads into cold instruction caches: one
// block 12 -> 4 us, a stream's 4096 slots 22 -> 10, 256 blocks 10 -> 5).
struct WaveSlots {
  unsigned long long key[kSegPer];
  unsigned long long fire[kSegPer];
  int count;
};
__device__ __forceinline__ void wave_slots(WaveSlots& w, const unsigned long long* __restrict__ slots, int64_t n,
                                           float thr2, const WinMap& m, int64_t base) {
  const int64_t v0 = base + (threadIdx.x & 63);
  const int left = (int)min(n - v0, (int64_t)64 * kSegPer);
  if (map_identity(m)) {
    slots += v0;
#pragma unroll
    for (int r = 0; r < kSegPer; ++r) w.key[r] = 64 * r < left ? slots[64 * r] : 0ull;
  } else {
    const int nq = (int)m.nq, dt = 64 / nq, dq = 64 % nq;          // (windows are at most N)
    int64_t t0, q0;
    map_visit(m, v0, t0, q0);
    slots += t0 * m.nwin;
    int qi = (int)q0;
#pragma unroll
    for (int r = 0; r < kSegPer; ++r) {
      w.key[r] = 64 * r < left ? slots[map_window(m, qi)] : 0ull;
      qi += dq;
      slots += dt * m.nwin;
      if (qi >= nq) {
        qi -= nq;
        slots += m.nwin;
      }
    }
  }
  w.count = 0;
#pragma unroll
  for (int r = 0; r < kSegPer; ++r) {
    w.fire[r] = __ballot(slot_fires(w.key[r], thr2));
    w.count += __popcll(w.fire[r]);
  }
}

__global__ __launch_bounds__(kSegThreads) void k_count(const unsigned long long* __restrict__ slots, int64_t n,
                                                     float thr2, long long* __restrict__ counts, WinMap m) {
  __shared__ int wc[kSegThreads / 64];
  const int wave = threadIdx.x >> 6;
  WaveSlots w;
  wave_slots(w, slots, n, thr2, m, (int64_t)blockIdx.x * kSeg + (int64_t)wave * 64 * kSegPer);
  if ((threadIdx.x & 63) == 0) wc[wave] = w.count;
  __syncthreads();
  if (threadIdx.x == 0) {
    long long c = 0;
    for (int i = 0; i < kSegThreads / 64; ++i) c += wc[i];
    counts[blockIdx.x] = c;
  }
}

// single-workgroup exclusive scan of the block counts; total at counts[nblk]
__global__ __launch_bounds__(1024) void k_scan(long long* __restrict__ counts, int64_t nblk,
                                             long long* __restrict__ total, long long* __restrict__ total_host) {
  __shared__ long long sh[1024];
  __shared__ long long carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int64_t b0 = 0; b0 < nblk; b0 += 1024) {
    int64_t i = b0 + threadIdx.x;
    long long v = i < nblk ? counts[i] : 0;
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
      long long x = threadIdx.x >= (unsigned)o ? sh[threadIdx.x - o] : 0;
      __syncthreads();
      sh[threadIdx.x] += x;
      __syncthreads();
    }
    if (i < nblk) counts[i] = carry + sh[threadIdx.x] - v;
    long long add = sh[1023];
    __syncthreads();
    if (threadIdx.x == 0) carry += add;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *total = carry;
    *total_host = carry;
  }
}

__device__ __forceinline__ int find_subbank(const int64_t* first, int nsb, int64_t t) {
  int lo = 0, hi = nsb - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (first[mid] <= t) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// counts: the blocks' trigger counts, or with SCANNED their exclusive sums.  Without, each
// block adds the counts before its own (few enough, see launch_compact_impl) and the last
// one stores the total, on the device and in the plan's host word.
template <bool SCANNED>
__global__ __launch_bounds__(kSegThreads) void k_write(const unsigned long long* __restrict__ slots, int64_t n,
                                                     float thr2, const long long* __restrict__ counts, int64_t W,
                                                     rfd_trigger* __restrict__ out, int64_t capacity,
                                                     const int64_t* __restrict__ sb_first, int nsb, WinMap m,
                                                     const int32_t* __restrict__ shift, int64_t nseg,
                                                     long long* __restrict__ total, long long* __restrict__ total_host) {
  __shared__ int wc[kSegThreads / 64];
  __shared__ long long part[kSegThreads / 64];
  __shared__ unsigned long long keys[kSeg];      // the block's firing slots, in order
  __shared__ uint16_t at[kSeg];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t base = (int64_t)blockIdx.x * kSeg;
  long long before = 0;
  if constexpr (!SCANNED) {
    for (int64_t i = threadIdx.x; i < (int64_t)blockIdx.x; i += kSegThreads) before += counts[i];
  }
  WaveSlots w;
  wave_slots(w, slots, n, thr2, m, base + wave * 64 * kSegPer);
  if constexpr (!SCANNED) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o);
  }
  if (lane == 0) {
    wc[wave] = w.count;
    part[wave] = before;
  }
  __syncthreads();
  int64_t pos = 0;
  int fired = 0;
  for (int i = 0; i < kSegThreads / 64; ++i) fired += wc[i];
  if constexpr (SCANNED) {
    pos = counts[blockIdx.x];
  } else {
    for (int i = 0; i < kSegThreads / 64; ++i) pos += part[i];
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
      *total = pos + fired;
      *total_host = pos + fired;
    }
  }
  int e = 0;
  for (int i = 0; i < wave; ++i) e += wc[i];
#pragma unroll
  for (int r = 0; r < kSegPer; ++r) {
    if ((w.fire[r] >> lane) & 1ull) {
      const int k = e + lanes_below(w.fire[r]);
      keys[k] = w.key[r];
      at[k] = (uint16_t)(wave * 64 * kSegPer + 64 * r + lane);
    }
    e += __popcll(w.fire[r]);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < fired && pos + i < capacity; i += kSegThreads) {
    const unsigned long long k = keys[i];
    int64_t tmpl, qi;
    map_visit(m, base + at[i], tmpl, qi);
    rfd_trigger t;
    // filter index m of the peak; sample n = m - d (mod N) under lag centring
    t.sample = map_window(m, qi) * W + (int64_t)(0xFFFFFFFFu - (uint32_t)(k & 0xFFFFFFFFull));
    if (shift) t.sample = (t.sample - shift[tmpl]) & (nseg - 1);
    t.tmpl = (int32_t)tmpl;
    t.subbank = sb_first ? find_subbank(sb_first, nsb, tmpl) : 0;
    t.rho = sqrtf(__uint_as_float((uint32_t)(k >> 32)));
    t.z_re = 0.f;
    t.z_im = 0.f;
    t.flags = 1u;       // complex SNR not yet evaluated
    out[pos + i] = t;
  }
}

// z_j[n] = sum_k c_j[k] zhat[(n + k0 + d_j + k) mod N]: one wave per
// trigger, grid-stride over the triggers (the count is known only on the
// device).
__global__ __launch_bounds__(256) void k_fir_z(rfd_trigger* __restrict__ out, const long long* __restrict__ total,
                                             int64_t capacity, const float2* __restrict__ c32,
                                             const float2* __restrict__ zref, int64_t n,
                                             const int64_t* __restrict__ sb_first, const int32_t* __restrict__ meta,
                                             const int64_t* __restrict__ abase, const int32_t* __restrict__ shift) {
  const int64_t lim = *total < capacity ? *total : capacity;
  const int lane = threadIdx.x & 63;
  for (int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); i < lim; i += (int64_t)gridDim.x * 4) {
    const rfd_trigger t = out[i];
    const int b = t.subbank;
    const int ref = meta[4 * b + 0], T = meta[4 * b + 1], Tp = meta[4 * b + 2];
    const int k0 = meta[4 * b + 3] + shift[t.tmpl];
    const float2* c = c32 + abase[b] + (int64_t)(t.tmpl - sb_first[b]) * Tp;
    const float2* z = zref + (int64_t)ref * n;
    float re = 0.f, im = 0.f;
    for (int k = lane; k < T; k += 64) {
      const float2 v = cmul(c[k], z[(t.sample + k0 + k) & (n - 1)]);
      re += v.x;
      im += v.y;
    }
    for (int o = 32; o > 0; o >>= 1) {
      re += __shfl_xor(re, o);
      im += __shfl_xor(im, o);
    }
    if (lane == 0) {
      out[i].z_re = re;
      out[i].z_im = im;
      out[i].flags = 0u;
    }
  }
}

// FINDCHIRP: z_j[n] = sum_band s_i F_j,i exp(+2 pi i i n / N) at each trigger.
// One block per trigger (segments of at most 4096 samples: a few bins per
// thread) ...
__global__ __launch_bounds__(256) void k_fc_z(rfd_trigger* __restrict__ out, const long long* __restrict__ total,
                                            int64_t capacity, const float2* __restrict__ s,
                                            const float2* __restrict__ filt, int64_t i_low, int64_t n_band,
                                            int64_t n, const float2* __restrict__ coarse,
                                            const float2* __restrict__ fine) {
  __shared__ float red[2][256];
  int64_t lim = *total < capacity ? *total : capacity;
  int64_t i = blockIdx.x;
  if (i >= lim) return;
  rfd_trigger t = out[i];
  const float2* f = filt + (int64_t)t.tmpl * n_band;
  float re = 0.f, im = 0.f;
  for (int64_t k = threadIdx.x; k < n_band; k += 256) {
    int64_t bin = k + i_low;
    uint32_t p = (uint32_t)((bin * t.sample) & (n - 1));
    float2 v = cmul(cmul(s[bin], f[k]), twiddle_n(coarse, fine, p, +1));
    re += v.x;
    im += v.y;
  }
  red[0][threadIdx.x] = re;
  red[1][threadIdx.x] = im;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) {
      red[0][threadIdx.x] += red[0][threadIdx.x + o];
      red[1][threadIdx.x] += red[1][threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[i].z_re = red[0][0];
    out[i].z_im = red[1][0];
    out[i].flags = 0u;
  }
}

// ... or, for long segments, from the rows of the intermediate [template][N2][N1] that pass B has just
// transformed: z[m] = sum_i1 Y[m mod N2][i1] e^{2 pi i i1 (m div N2) / N1}, N1 terms (32 KB) per trigger in place of
// the N / 2 of its filter (4 MB at N = 2^20; 250 triggers then read 1 GB again, 238 us).  Each batch
// of templates lists its firing slots with their z, summed in FP64, in any order; k_fc_z_final gives them to the
// triggers after compaction.  More than kFcZList firing slots (beyond what gets a z at all) are
// left to the sums over the filters, all of them, so that no result depends on the order.
constexpr int kFcZSlots = 32;            // slots per workgroup
struct FcZ {
  long long slot;
  float2 z;
};
__global__ __launch_bounds__(256) void k_fc_z_rows(const unsigned long long* __restrict__ slots, int64_t tmpl0, int count,
                                                 float thr2, int64_t nwin, int64_t W, const float2* __restrict__ Y,
                                                 int64_t N2, const double2* __restrict__ tab,
                                                 FcZ* __restrict__ list, unsigned long long* __restrict__ listed) {
  __shared__ double red[2][4];
  __shared__ bool full;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  // a signal fires the same windows of every template: neighbouring workgroups, which run on
  // different compute units, take the same windows of different templates
  const int64_t b = blockIdx.x % (uint32_t)count, q0 = (int64_t)(blockIdx.x / (uint32_t)count) * kFcZSlots;
  slots += (tmpl0 + b) * nwin + q0;
  const unsigned long long k = lane < kFcZSlots && q0 + lane < nwin ? slots[lane] : 0ull;   // (in every wave)
  unsigned long long mask = __ballot(slot_fires(k, thr2));
  if (mask == 0) return;
  if (threadIdx.x == 0)                    // (no use for more z than the list takes)
    full = __hip_atomic_load(listed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > (unsigned long long)kFcZList;
  __syncthreads();
  for (; mask != 0 && !full; mask &= mask - 1) {
    const int at = __ffsll(mask) - 1;
    const uint32_t off = 0xFFFFFFFFu - (uint32_t)__shfl((int)(uint32_t)(k & 0xFFFFFFFFull), at);
    const int64_t q = q0 + at, m = q * W + (int64_t)off;
    const float2* __restrict__ row = Y + (b * N2 + (m & (N2 - 1))) * kFcN1 + threadIdx.x;
    const uint32_t turn = (uint32_t)(m / N2);                     // of N1: at most 4096
    // a thread's values are 256 apart: their factors turn by a sixteenth root of unity
    float2 y[kFcN1 / 256];
#pragma unroll
    for (int r = 0; r < kFcN1 / 256; ++r) y[r] = row[256 * r];
    double2 w = tab[threadIdx.x * turn & (kFcN1 - 1)];
    const double2 step = tab[256 * turn & (kFcN1 - 1)];
    double re = 0.0, im = 0.0;
#pragma unroll
    for (int r = 0; r < kFcN1 / 256; ++r) {
      re += (double)y[r].x * w.x - (double)y[r].y * w.y;
      im += (double)y[r].x * w.y + (double)y[r].y * w.x;
      w = cmul(w, step);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      re += __shfl_xor(re, o);
      im += __shfl_xor(im, o);
    }
    if (lane == 0) {
      red[0][wv] = re;
      red[1][wv] = im;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      const unsigned long long e = atomicAdd(listed, 1ull);
      full = e >= (unsigned long long)kFcZList;
      if (e < (unsigned long long)kFcZList)
        list[e] = FcZ{(long long)((tmpl0 + b) * nwin + q), make_float2((float)((red[0][0] + red[0][1]) + (red[0][2] + red[0][3])),
                                                                   (float)((red[1][0] + red[1][1]) + (red[1][2] + red[1][3])))};
    }
    __syncthreads();
  }
}
// the z of list entry x to its trigger, unless that lies beyond the first lim
__device__ __forceinline__ void fc_z_match(rfd_trigger* __restrict__ out, int64_t lim, int64_t nwin, int64_t W,
                                           const FcZ& x) {
  const int64_t tmpl = x.slot / nwin, first = (x.slot - tmpl * nwin) * W;
  int64_t lo = 0, hi = lim;                // triggers are in slot order
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    const int64_t t = out[mid].tmpl;
    if (t < tmpl || (t == tmpl && out[mid].sample < first)) lo = mid + 1; else hi = mid;
  }
  if (lo >= lim || out[lo].tmpl != tmpl || out[lo].sample < first || out[lo].sample >= first + W) return;
  out[lo].z_re = x.z.x;
  out[lo].z_im = x.z.y;
  out[lo].flags = 0u;
}

// ... or, where those lists do not serve, kZParts blocks per trigger over contiguous bin
// ranges (grid-stride over the triggers), their partial sums then added in
// a fixed order by one thread per trigger.  A thread's bins are 256 apart, so
// its factor e^{2 pi i bin n / N} turns by the same angle from each bin to the next: an
// FP64 rotation, rounded to FP32 per bin (at most N / 2 / kZParts / 256 turns, far below
// FP32 rounding).  Bound by reading the filters, with kZU bins' loads in flight
// per thread: 250 triggers at N = 2^20 408 -> 237 us (one bin at a time, its factor from two
// scattered FP32 table reads).
constexpr int kZU = 8;
__global__ __launch_bounds__(256) void k_fc_z_part(const rfd_trigger* __restrict__ out,
                                                 const long long* __restrict__ total, int64_t capacity,
                                                 const float2* __restrict__ s, const float2* __restrict__ filt,
                                                 int64_t i_low, int64_t n_band, int64_t n,
                                                 const double2* __restrict__ coarse, const double2* __restrict__ fine,
                                                 float2* __restrict__ part,
                                                 const unsigned long long* __restrict__ listed) {
  __shared__ float red[2][4];
  if (listed && *listed <= (unsigned long long)kFcZList) return;
  const int64_t lim = *total < capacity ? *total : capacity;
  const int64_t chunk = (n_band + kZParts - 1) / kZParts;
  const int64_t k0 = (int64_t)blockIdx.x * chunk, k1 = std::min<int64_t>(k0 + chunk, n_band);
  const float2* sb = s + i_low;
  for (int64_t i = blockIdx.y; i < lim; i += gridDim.y) {
    const int64_t sample = out[i].sample;
    const float2* f = filt + (int64_t)out[i].tmpl * n_band;
    double2 w = twiddle_n(coarse, fine, (uint32_t)(((k0 + threadIdx.x + i_low) * sample) & (n - 1)), +1);
    const double2 step = twiddle_n(coarse, fine, (uint32_t)((256 * sample) & (n - 1)), +1);
    float re = 0.f, im = 0.f;
    auto add = [&](float2 x, float2 y) {
      const float2 v = cmul(cmul(x, y), make_float2((float)w.x, (float)w.y));
      re += v.x;
      im += v.y;
      w = cmul(w, step);
    };
    int64_t k = k0 + threadIdx.x;
    for (; k + 256 * (kZU - 1) < k1; k += 256 * kZU) {
      float2 x[kZU], y[kZU];
#pragma unroll
      for (int u = 0; u < kZU; ++u) {
        x[u] = sb[k + 256 * u];
        y[u] = f[k + 256 * u];
      }
#pragma unroll
      for (int u = 0; u < kZU; ++u) add(x[u], y[u]);
    }
    for (; k < k1; k += 256) add(sb[k], f[k]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      re += __shfl_xor(re, o);
      im += __shfl_xor(im, o);
    }
    if ((threadIdx.x & 63) == 0) {
      red[0][threadIdx.x >> 6] = re;
      red[1][threadIdx.x >> 6] = im;
    }
    __syncthreads();
    if (threadIdx.x == 0)
      part[i * kZParts + blockIdx.x] = make_float2((red[0][0] + red[0][1]) + (red[0][2] + red[0][3]),
                                                   (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]));
    __syncthreads();
  }
}
__global__ __launch_bounds__(256) void k_fc_z_final(rfd_trigger* __restrict__ out, const long long* __restrict__ total,
                                                  int64_t capacity, const float2* __restrict__ part,
                                                  const FcZ* __restrict__ list,
                                                  const unsigned long long* __restrict__ listed, int64_t nwin,
                                                  int64_t W) {
  const int64_t lim = *total < capacity ? *total : capacity;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (listed && *listed <= (unsigned long long)kFcZList) {
    if ((unsigned long long)i < *listed) fc_z_match(out, lim, nwin, W, list[i]);
    return;
  }
  if (i >= lim) return;
  float re = 0.f, im = 0.f;
  for (int k = 0; k < kZParts; ++k) {
    const float2 v = part[i * kZParts + k];
    re += v.x;
    im += v.y;
  }
  out[i].z_re = re;
  out[i].z_im = im;
  out[i].flags = 0u;
}

// ------------------------------------------------------------ launchers
WinMap win_map_all(int64_t nwin) { return WinMap{nwin, nwin, nwin, 0, 0}; }

bool win_map_range(int64_t nwin, int64_t W, int pieces, const int64_t* lo, const int64_t* hi, WinMap* m) {
  int64_t a[2], b[2];       // inclusive window runs
  for (int k = 0; k < pieces; ++k) {
    a[k] = lo[k] / W;
    b[k] = (hi[k] - 1) / W;
  }
  if (pieces == 2) {
    if (a[1] < a[0]) {      // increasing q
      std::swap(a[0], a[1]);
      std::swap(b[0], b[1]);
    }
    if (a[1] <= b[0] + 1) { // overlapping or adjacent runs merge
      b[0] = std::max(b[0], b[1]);
      pieces = 1;
    }
  }
  if (pieces == 1) {
    *m = WinMap{nwin, b[0] - a[0] + 1, b[0] - a[0] + 1, a[0], 0};
    return true;
  }
  if (pieces != 2) return false;
  *m = WinMap{nwin, (b[0] - a[0] + 1) + (b[1] - a[1] + 1), b[0] - a[0] + 1, a[0], a[1]};
  return true;
}

// also: a counter to clear with them, or NULL
static int slots_clear(Plan& p, int64_t n_visit, const WinMap& m, unsigned long long* also) {
  int64_t blocks = (n_visit + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_fill_u64, dim3((unsigned)blocks), dim3(256), 0, p.stream, p.slots, n_visit, m, also);
  RFD_CHECK_LAUNCH();
  return RFD_OK;
}

int launch_slots_clear(Plan& p, int64_t n_slots) {
  // every slot: templates x windows, identity order
  return slots_clear(p, n_slots, win_map_all(std::max<int64_t>(n_slots, 1)), p.fcz_count);
}

int launch_slots_clear_map(Plan& p, int64_t n_visit, const WinMap& m) { return slots_clear(p, n_visit, m, nullptr); }

int launch_compact_impl(Plan& p, int64_t n_slots, int64_t W, float threshold, rfd_trigger* out, int64_t capacity,
                        const int64_t* sb_first, int nsb, const WinMap& m,
                        const int32_t* shift = nullptr) {
  int64_t nblk = (n_slots + kSeg - 1) / kSeg;
  if ((size_t)nblk > p.counts_cap) return fail(RFD_E_INVALID, "compaction scratch too small");
  float thr2 = threshold * threshold;
  // One block needs no counts.  Up to 4096 blocks (16.8 million slots) each add the counts before
  // them in place of the single-workgroup scan between the two passes (at 2 to 2048
  // blocks 5 us of the chain's 20 to 30).  Beyond that the sums would be more
  // work than the scan.
  if (nblk > 1) {
    hipLaunchKernelGGL(k_count, dim3((unsigned)nblk), dim3(kSegThreads), 0, p.stream, p.slots, n_slots, thr2,
                       p.counts, m);
    RFD_CHECK_LAUNCH();
  }
  if (nblk <= 4096) {
    hipLaunchKernelGGL(k_write<false>, dim3((unsigned)nblk), dim3(kSegThreads), 0, p.stream,
                       p.slots, n_slots, thr2, (const long long*)p.counts, W, out, capacity, sb_first, nsb, m,
                       shift, p.n, p.total, p.total_host);
    RFD_CHECK_LAUNCH();
    return RFD_OK;
  }
  hipLaunchKernelGGL(k_scan, dim3(1), dim3(1024), 0, p.stream, p.counts, nblk, p.total, p.total_host);
  RFD_CHECK_LAUNCH();
  hipLaunchKernelGGL(k_write<true>, dim3((unsigned)nblk), dim3(kSegThreads), 0, p.stream, p.slots, n_slots, thr2,
                     (const long long*)p.counts, W, out, capacity, sb_first, nsb, m, shift, p.n, p.total,
                     p.total_host);
  RFD_CHECK_LAUNCH();
  return RFD_OK;
}

int launch_compact(Plan& p, int64_t n_slots, int64_t nwin, int64_t W, float threshold, rfd_trigger* out,
                   int64_t capacity) {
  return launch_compact_impl(p, n_slots, W, threshold, out, capacity, nullptr, 1, win_map_all(nwin));
}

int compaction_blocks(int64_t n_slots) { return (int)((n_slots + kSeg - 1) / kSeg); }

int launch_compact_bank(Plan& p, const Taps& tp, int64_t n_slots, int64_t nwin, int64_t W, float threshold,
                        rfd_trigger* out, int64_t capacity, const WinMap* m) {
  // the lag offsets are always read (zero where a template is not centred), so
  // a captured graph stays right when taps are later re-made with or without
  // centring
  return launch_compact_impl(p, n_slots, W, threshold, out, capacity, tp.d_first, (int)tp.sb.size(),
                             m ? *m : win_map_all(nwin), tp.d_shift);
}

int launch_fir_z(Plan& p, const Taps& tp, rfd_trigger* out, int64_t capacity) {
  if (capacity <= 0) return RFD_OK;
  const int64_t blocks = std::min<int64_t>((capacity + 3) / 4, 1024);
  hipLaunchKernelGGL(k_fir_z, dim3((unsigned)blocks), dim3(256), 0, p.stream, out, (const long long*)p.total,
                     capacity, tp.c32, p.zref, p.n, tp.d_first, tp.d_meta, tp.d_abase, (const int32_t*)tp.d_shift);
  RFD_CHECK_LAUNCH();
  return RFD_OK;
}

// The lists pay where a call's filters are much to read again and its slots few against its
// intermediates.  250 templates of 2^20 samples, one trigger each and windows of 2048: 1260 -> 1103 us, 1072 with
// the sums' loads all in flight (no trigger at all: 1020 -> 1034); before that windows of 64: 1267 -> 1142 (1033 -> 1092), of 16: 1376 -> 1332 (1091 -> 1293).
// 64 templates of 2^20: 384 -> 339; 250 of 2^18: 415 -> 379; 64 of 2^18: 147 -> 143 (119 -> 123); 8 of 2^20: 107 -> 110.
static bool fc_z_lists(const Plan& p, int64_t n_templates, int64_t W) {
  return W >= 256 && n_templates * p.n >= (int64_t)1 << 25 && p.n > 4096;
}

int launch_findchirp_z_batch(Plan& p, int64_t n_templates, int64_t tmpl0, int count, int64_t N1, int64_t N2, int64_t W,
                             int64_t nwin, float thr2) {
  if (!fc_z_lists(p, n_templates, W)) return RFD_OK;
  hipLaunchKernelGGL(k_fc_z_rows, dim3((unsigned)((nwin + kFcZSlots - 1) / kFcZSlots * count)), dim3(256), 0, p.stream,
                     (const unsigned long long*)p.slots, tmpl0, count, thr2, nwin, W, (const float2*)p.fc_work, N2,
                     (const double2*)p.ols_tw64, (FcZ*)p.fcz_list, p.fcz_count);
  RFD_CHECK_LAUNCH();
  return RFD_OK;
}

int launch_findchirp_z(Plan& p, const float2* filt, int64_t n_templates, rfd_trigger* out, int64_t capacity, int64_t W,
                       int64_t nwin) {
  if (capacity <= 0) return RFD_OK;
  const unsigned long long* listed = fc_z_lists(p, n_templates, W) ? p.fcz_count : nullptr;
  if (p.fc_work && p.fc_work_cap >= (size_t)capacity * kZParts) {
    // partial sums in FINDCHIRP's (now idle) intermediate buffer
    const unsigned gy = (unsigned)std::min<int64_t>(capacity, 256);
    hipLaunchKernelGGL(k_fc_z_part, dim3(kZParts, gy), dim3(256), 0, p.stream, (const rfd_trigger*)out,
                       (const long long*)p.total, capacity, p.stilde, filt, p.i_low, p.n_band, p.n, (const double2*)p.tw64c,
                       (const double2*)p.tw64f, p.fc_work, listed);
    RFD_CHECK_LAUNCH();
    const int64_t items = listed ? std::max<int64_t>(capacity, kFcZList) : capacity;
    hipLaunchKernelGGL(k_fc_z_final, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, p.stream, out,
                       (const long long*)p.total, capacity, (const float2*)p.fc_work, (const FcZ*)p.fcz_list, listed,
                       nwin, W);
    RFD_CHECK_LAUNCH();
    return RFD_OK;
  }
  hipLaunchKernelGGL(k_fc_z, dim3((unsigned)capacity), dim3(256), 0, p.stream, out, (const long long*)p.total,
                     capacity, p.stilde, filt, p.i_low, p.n_band, p.n, p.tw32c, p.tw32f);
  RFD_CHECK_LAUNCH();
  return RFD_OK;
}

}  // namespace rfd
