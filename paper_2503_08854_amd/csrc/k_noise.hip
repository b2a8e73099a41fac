// k_noise.hip -- per-image noise sigma by an iterated median absolute
// deviation (Sec. 3): S = finite pixels; m = median(S),
// sigma = 1.4826 median{|x - m| : x in S}; S' = {finite x : |x - m| <=
// kappa sigma}; repeat until S' == S or max_iter steps.  The median of an
// even count is the mean of the two middle values.
//
// Every set S is an interval of the sorted finite pixels (the FP64 predicate
// |x - m| <= thr is monotone on each side of m), so a step needs order
// statistics at five places only: the middle of S, m -+ the deviation median
// and the two cuts.  The image is therefore read twice, not once per digit
// and step:
//   sample   a sorted sample of each image runs the iteration and says where
//            those places are; it sets a monotone map of values to
//            NZ_BINS bins, fine around the median and around m -+ the
//            deviation median (~5e-5 sigma), coarse (~1e-3 sigma) elsewhere;
//   bins     one read of the images: the histogram of that map;
//   plan     the iteration on the interpolated histogram; the bins around
//            every place it visits are marked;
//   collect  a second read: the values of the marked bins are listed (a few
//            thousand per image); of bins that are too full because one value
//            repeats (integer or zero-filled images) only the other values;
//   solve    the exact iteration on ranks: number of pixels below a bin (the
//            histogram) + position in the sorted list.  Each rank it uses is
//            checked to fall in a marked bin (or a gap without pixels); if
//            one does not, the image is solved by radix selection over its
//            pixels (pixels, a kernel that ends at once if there is none).
// The counts of the histogram route are 32-bit: an image of 2^32 pixels or
// more goes straight to the radix selection, whose counts are 64-bit.
// All comparisons that decide the result are the FP64 ones of the definition,
// so the result is exact on either route.
//
// Two image reads bound it.  200 FP32 2048^2 images (3.36 GB), one kernel
// trace: bins 0.71 ms (4.7 TB/s, the copy rate), collect 0.66 ms, sample +
// plan + solve 0.055 + 0.047 + 0.131 ms (one workgroup per image, latency),
// 1.60 ms together; 1.53 ms a call without the trace, 32.2 ms before, when
// every 11-bit digit of every median and deviation of every step read the
// images again (26 reads).  48 FP32 2048 x 1536 images: 0.43 ms, 6.9 before.
// (In sample and solve the middle deviation is found by wavefronts over the
// values sorted by their deviation on either side; with every value trying
// itself and one atomic minimum they took 0.39 ms instead of 0.19.)
#include <algorithm>
#include <cstddef>
#include <type_traits>

#include "dt_common.hpp"

namespace dtk {

constexpr int NZ_BINS = 16384;        // histogram bins per image (64 KB of LDS in the counting pass)
constexpr int NZ_COARSE = 5120;       // of which over the whole range
constexpr int NZ_CENTER = 3072;       // in the window around the median (the rest: 2 x 4094 around m -+ d)
constexpr int NZ_TX = 1024;           // threads of every workgroup here
constexpr int NZ_WAVES = NZ_TX / 64;
constexpr int NZ_SAMPLE = 4096;       // sample size
constexpr int NZ_SAMPLE_STEPS = 6;    // clip steps followed on the sample
constexpr int64_t NZ_WHOLE = 16384;   // images up to this size are listed whole
constexpr int64_t NZ_MOST = 0xffffffffll;  // images beyond it are solved from their pixels
constexpr int NZ_LIST = 32768;        // listed values per image
constexpr int NZ_TAB = 512;           // marked bins per image
constexpr int NZ_STAGE = 2048;        // values a collecting workgroup stages in LDS
constexpr int NZ_PIECES = 256;        // most pieces of an image solved from its pixels
constexpr int NZ_DHAT = 16;           // steps whose planned deviation median is kept

// Monotone map of a value to a bin: the sum of clamped, scaled differences
// from the sample median (each term is non-decreasing in x, also rounded).
struct NoiseMap {
  float mc;          // sample median
  float T;           // half range
  float wc;          // half width of the window around the median
  float q0, q1;      // deviation window
  float a0, a1, a2;  // bins per unit
  float off;
};

struct NoiseImage {
  NoiseMap map;
  uint32_t n;       // finite pixels
  uint32_t n_list;  // values listed
  int32_t n_tab;    // marked bins; -1: too many, solve from the pixels
  int32_t whole;    // one bin, every value listed
  int32_t n_sample; // finite values of the sample
  int32_t todo;     // the plan missed: solve from the pixels
  uint32_t n_todo;  // first image: images with todo
  uint32_t role, done;       // workgroups that came to it, pieces done
  uint32_t call;             // number of the pass; 0: none yet, ~0: done
  uint32_t taken[NZ_PIECES]; // pass in which a piece was taken last
  uint64_t task[7];          // the pass
  float dhat[NZ_DHAT];  // the plan's deviation medians, by step (0: none)
  uint32_t bin[NZ_TAB], below[NZ_TAB], cnt[NZ_TAB];  // marked bins: index, pixels below, pixels in
  uint32_t heavy[NZ_TAB];                            // key of the value that is not listed (0: none)
  uint16_t mode[NZ_BINS];                            // 0 not listed, 0xffff listed, else 1 + table entry (heavy value)
  alignas(8) uint32_t hist[NZ_BINS];  // in the radix selection: 64-bit sums of a pass
  uint32_t sample[NZ_SAMPLE];  // sorted keys
  alignas(8) uint32_t list[NZ_LIST];  // keys; in the radix selection: 64-bit ones
};

typedef float nz_f4 __attribute__((ext_vector_type(4)));
typedef _Float16 nz_h8 __attribute__((ext_vector_type(8)));

// Order-preserving key of a float, one for both zeros (never 0 or 0xffffffff
// for a finite value).
__device__ __forceinline__ uint32_t fkey(float x) {
  const uint32_t u = __float_as_uint(x == 0.f ? 0.f : x);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float fkey_value(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

__device__ __forceinline__ float clampf(float y, float lo, float hi) { return fminf(fmaxf(y, lo), hi); }
__device__ __forceinline__ float map_pos(const NoiseMap& M, float y) {
  float g = fmaf(M.a0, clampf(y, -M.T, M.T), M.off);
  g = fmaf(M.a1, clampf(y, -M.wc, M.wc), g);
  return fmaf(M.a2, clampf(y, M.q0, M.q1) + clampf(y, -M.q1, -M.q0), g);
}
__device__ __forceinline__ int pos_bin(float g) { return (int)fminf(fmaxf(g, 0.f), (float)(NZ_BINS - 1)); }
__device__ __forceinline__ int map_bin(const NoiseMap& M, float x) { return pos_bin(map_pos(M, x - M.mc)); }

// f(x) for every pixel of an image, the pixels shared by `blocks` workgroups
// of which this is `block`: 16-byte loads, U in flight per thread; the
// unaligned head and the tail one by one.
template <typename T, int U = 4, typename F>
__device__ __forceinline__ void for_pixels(const void* img, int64_t n, int block, int blocks, F&& f) {
  constexpr int V = 16 / sizeof(T);
  using Vec = std::conditional_t<sizeof(T) == 4, nz_f4, nz_h8>;
  const T* p = static_cast<const T*>(img);
  const int64_t head = std::min<int64_t>(n, (int64_t)((16 - ((uintptr_t)p & 15)) & 15) / (int64_t)sizeof(T));
  const int64_t nv = (n - head) / V;
  const int64_t gid = (int64_t)block * NZ_TX + threadIdx.x, stride = (int64_t)blocks * NZ_TX;
  const auto* pv = (const __attribute__((address_space(1))) Vec*)(p + head);
  const auto* ps = global_ptr(p);
  for (int64_t v = gid; v < nv; v += stride * U) {
    Vec x[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (v + u * stride < nv) x[u] = pv[v + u * stride];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (v + u * stride < nv) {
#pragma unroll
        for (int j = 0; j < V; ++j) f((float)x[u][j]);
      }
  }
  const int64_t tail0 = head + nv * V;
  if (gid < head) f((float)ps[gid]);
  if (tail0 + gid < n) f((float)ps[tail0 + gid]);  // fewer than V <= 8 pixels
}

// Exclusive prefix sum over the workgroup; *total is the sum.  tmp: NZ_WAVES
// values in LDS.
template <typename C>
__device__ __forceinline__ C block_scan(C v, C* tmp, C* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  C inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const C u = __shfl_up(inc, o, 64);
    if (lane >= o) inc += u;
  }
  __syncthreads();  // earlier readers of tmp
  if (lane == 63) tmp[w] = inc;
  __syncthreads();
  C base = 0, sum = 0;
  for (int i = 0; i < NZ_WAVES; ++i) {
    if (i < w) base += tmp[i];
    sum += tmp[i];
  }
  *total = sum;
  return base + inc - v;
}

// Smallest j of [0, n) with f(j), n if there is none, for an f that stays true
// from there on: 64 places per round, by a whole wavefront.
template <typename F>
__device__ __forceinline__ int wave_first(int n, F&& f) {
  const int lane = threadIdx.x & 63;
  int lo = 0, hi = n;
  while (lo < hi) {
    const int w = (hi - lo + 63) >> 6;
    const uint64_t m = __ballot(f(min(lo + (lane + 1) * w, hi) - 1));
    if (!m) return hi;
    const int k = __builtin_ctzll(m);
    hi = min(lo + (k + 1) * w, hi) - 1;
    lo += k * w;
  }
  return hi;
}

// Ascending bitonic sort of the NZ_TX * PER keys in s (LDS).  Thread t holds
// keys PER t .. PER t + PER - 1: a compare-exchange at distance j is in
// registers for j < PER, between lanes for j < 64 PER, and through LDS, with
// barriers, only beyond (10 of the 78 stages of 4096 keys).
template <int PER>
__device__ __forceinline__ void sort_per(uint32_t* s) {
  constexpr int S = NZ_TX * PER;
  const int t = threadIdx.x;
  uint32_t r[PER];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < PER; ++q) r[q] = s[PER * t + q];
  __syncthreads();
#pragma unroll 1
  for (int k = 2; k <= S; k <<= 1) {
#pragma unroll 1
    for (int j = k >> 1; j >= PER; j >>= 1) {
      const bool low = ((PER * t) & j) == 0, up = ((PER * t) & k) == 0;
      uint32_t o[PER];
      if (j >= 64 * PER) {
        // key PER t + q at q NZ_TX + t: the lanes touch consecutive words
#pragma unroll
        for (int q = 0; q < PER; ++q) s[q * NZ_TX + t] = r[q];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PER; ++q) o[q] = s[q * NZ_TX + (t ^ (j / PER))];
        __syncthreads();
      } else {
#pragma unroll
        for (int q = 0; q < PER; ++q) o[q] = (uint32_t)__shfl_xor((int)r[q], j / PER, 64);
      }
#pragma unroll
      for (int q = 0; q < PER; ++q) r[q] = low == up ? std::min(r[q], o[q]) : std::max(r[q], o[q]);
    }
#pragma unroll
    for (int j = PER / 2; j > 0; j >>= 1) {
      if (j > (k >> 1)) continue;
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        if (q & j) continue;
        const uint32_t a = std::min(r[q], r[q | j]), b = std::max(r[q], r[q | j]);
        const bool up = ((PER * t + q) & k) == 0;
        r[q] = up ? a : b;
        r[q | j] = up ? b : a;
      }
    }
  }
#pragma unroll
  for (int q = 0; q < PER; ++q) s[PER * t + q] = r[q];
  __syncthreads();
}

// Where the iteration goes on a sample, and the map from it; clears the
// image's histogram.
template <typename T>
__global__ __launch_bounds__(NZ_TX) void k_noise_sample(const void* const* imgs, const int64_t* npix, NoiseImage* st,
                                                        double kappa, int max_iter) {
  const int img = blockIdx.x;
  const int tid = threadIdx.x;
  const int64_t n = npix[img];
  NoiseImage& S = st[img];
  __shared__ uint32_t s[NZ_SAMPLE];
  __shared__ uint32_t tmp[NZ_WAVES];
  __shared__ float sh_d;
  for (int b = tid; b < NZ_BINS; b += NZ_TX) S.hist[b] = 0u;
  if (tid < NZ_DHAT) S.dhat[tid] = 0.f;
  if (tid < NZ_PIECES) S.taken[tid] = 0u;
  if (tid == 0) {
    S.n = 0;
    S.n_list = 0;
    S.n_tab = 0;
    S.whole = n <= NZ_WHOLE;
    S.n_sample = 0;
    S.role = 0;
    S.n_todo = 0;
    S.call = 0;
  }
  if (n <= NZ_WHOLE) {  // every value is listed: one bin
    if (tid == 0) S.map = NoiseMap{0.f, 1.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    return;
  }
  if (n > NZ_MOST) {
    if (tid == 0) S.n_tab = -1;
    return;
  }
  const auto* p = global_ptr(static_cast<const T*>(imgs[img]));
  uint32_t mine = 0;
  for (int i = tid; i < NZ_SAMPLE; i += NZ_TX) {
    // one pixel of each of NZ_SAMPLE runs, at a place that varies from run to run
    const double fr = 0.6180339887498949 * i;
    const int64_t at = (int64_t)(((double)i + (fr - floor(fr))) * ((double)n / NZ_SAMPLE));
    const float x = (float)p[std::min<int64_t>(at, n - 1)];
    const bool ok = __builtin_isfinite(x);
    s[i] = ok ? fkey(x) : 0xffffffffu;
    mine += ok ? 1u : 0u;
  }
  uint32_t ns_u;
  (void)block_scan(mine, tmp, &ns_u);
  sort_per<NZ_SAMPLE / NZ_TX>(s);
  const int ns = (int)ns_u;
  // all values below are the same in every thread
  float m = 0.f, m_lo = 0.f, m_hi = 0.f, m0 = 0.f, d_lo = 0.f, d_hi = 0.f, sig = 0.f, sig_max = 0.f;
  int lo = 0, hi = ns;
  for (int it = 0; it < min(max_iter, NZ_SAMPLE_STEPS) && hi > lo; ++it) {
    const int c = hi - lo;
    m = 0.5f * fkey_value(s[lo + (c - 1) / 2]) + 0.5f * fkey_value(s[lo + c / 2]);
    // first position in [lo, hi) whose value is >= v (strict: > v)
    auto pos = [&](float v, bool strict) {
      int a = lo, b = hi;
      while (a < b) {
        const int k = (a + b) >> 1;
        const float x = fkey_value(s[k]);
        if (strict ? x <= v : x < v) a = k + 1;
        else b = k;
      }
      return a;
    };
    // the deviation that covers half of the members: the k-th smallest of the
    // sorted deviations right and left of the median, i of them from the right
    if (tid < 64) {
      const int p = lo + wave_first(c, [&](int j) { return fkey_value(s[lo + j]) >= m; });
      const int k = (c + 1) / 2, nr = hi - p, nl = p - lo;
      auto right = [&](int j) { return j < nr ? fkey_value(s[p + j]) - m : __builtin_inff(); };
      auto left = [&](int j) { return j < nl ? m - fkey_value(s[p - 1 - j]) : __builtin_inff(); };
      const int i = wave_first(k + 1, [&](int j) { return j == k || right(j) >= left(k - 1 - j); });
      if (tid == 0) sh_d = fmaxf(i > 0 ? right(i - 1) : 0.f, i < k ? left(k - 1 - i) : 0.f);
    }
    __syncthreads();
    const float d = sh_d;
    sig = 1.4826f * d;
    if (it == 0) {
      m0 = m_lo = m_hi = m;
      d_lo = d_hi = d;
      sig_max = sig;
    } else {
      m_lo = fminf(m_lo, m);
      m_hi = fmaxf(m_hi, m);
      d_lo = fminf(d_lo, d);
      d_hi = fmaxf(d_hi, d);
      sig_max = fmaxf(sig_max, sig);
    }
    const float thr = (float)fmin(kappa * (double)sig, 3e38);
    const int nl = pos(m - thr, false), nh = pos(m + thr, true);
    if (nl == lo && nh == hi) break;
    lo = nl;
    hi = nh;
    __syncthreads();  // sh_d is read
  }
  for (int i = tid; i < NZ_SAMPLE; i += NZ_TX) S.sample[i] = s[i];
  if (tid == 0) {
    S.n_sample = ns;
    NoiseMap M;
    M.mc = m0;
    if (!(sig > 0.f)) {  // over half of the sample is one value: some other scale
      if (ns > 0) sig = (fkey_value(s[(int)(0.95f * (ns - 1))]) - fkey_value(s[(int)(0.05f * (ns - 1))])) / 3.f;
      if (!(sig > 0.f) && ns > 0) sig = (fkey_value(s[ns - 1]) - fkey_value(s[0])) / 8.f;
      if (!(sig > 0.f)) sig = fmaxf(fabsf(m0) * 1e-3f, 1e-30f);
    }
    // (a scale outside this range makes a useless map, never a wrong result)
    sig = clampf(sig, 1e-30f, 1e30f);
    sig_max = clampf(fmaxf(sig_max, sig), 1e-30f, 1e30f);
    // a median of NZ_SAMPLE values is within 0.02 sigma (one standard error)
    const float w = 0.1f * sig;
    M.wc = clampf(fmaxf(m_hi - m0, m0 - m_lo), 0.f, 1e30f) + w;
    M.q0 = fmaxf(d_lo - M.wc, 0.f);
    M.q1 = fminf(d_hi, 1e30f) + M.wc;
    M.q0 = fminf(M.q0, M.q1 - w);
    M.T = fmaxf((float)fmin(1.1 * kappa, 8.0) * sig_max + M.wc, M.q1);
    M.a0 = 0.5f * NZ_COARSE / M.T;
    M.a1 = 0.5f * NZ_CENTER / M.wc;
    M.a2 = 0.5f * (float)(NZ_BINS - 4 - NZ_COARSE - NZ_CENTER) / (M.q1 - M.q0);
    M.off = 0.5f * (float)(NZ_BINS - 4) + 1.f;
    S.map = M;
  }
}

template <typename T>
__global__ __launch_bounds__(NZ_TX) void k_noise_bins(const void* const* imgs, const int64_t* npix, NoiseImage* st) {
  const int img = blockIdx.y;
  NoiseImage& S = st[img];
  if (S.n_tab < 0) return;
  __shared__ uint32_t h[NZ_BINS];
  for (int b = threadIdx.x; b < NZ_BINS; b += NZ_TX) h[b] = 0u;
  const NoiseMap M = S.map;
  __syncthreads();
  for_pixels<T>(imgs[img], npix[img], blockIdx.x, gridDim.x, [&](float x) {
    if (__builtin_isfinite(x)) atomicAdd(&h[map_bin(M, x)], 1u);
  });
  __syncthreads();
  for (int b = threadIdx.x; b < NZ_BINS; b += NZ_TX)
    if (h[b]) atomicAdd(&S.hist[b], h[b]);
}

// The iteration on the interpolated histogram (the first wavefront; 64
// candidates per search round), marking the bins around each place visited;
// then the table of marked bins.
__global__ __launch_bounds__(NZ_TX) void k_noise_plan(NoiseImage* st, double kappa, int max_iter) {
  const int tid = threadIdx.x, lane = tid & 63;
  NoiseImage& S = st[blockIdx.x];
  if (S.n_tab < 0) return;
  __shared__ uint32_t C[NZ_BINS + 1];
  __shared__ uint32_t mark[NZ_BINS / 32];
  __shared__ uint32_t tmp[NZ_WAVES];
  constexpr int PER = NZ_BINS / NZ_TX;
  uint32_t h[PER], sum = 0, N;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    h[j] = S.hist[tid * PER + j];
    sum += h[j];
  }
  uint32_t base = block_scan(sum, tmp, &N);
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    C[tid * PER + j] = base;
    base += h[j];
  }
  if (tid == 0) C[NZ_BINS] = N;
  for (int i = tid; i < NZ_BINS / 32; i += NZ_TX) mark[i] = 0u;
  __syncthreads();
  const NoiseMap M = S.map;
  if (S.whole) {
    if (tid == 0) mark[0] = 1u;
  } else if (tid < 64 && N > 0) {
    auto cum = [&](float g) {
      const int b = pos_bin(g);
      const double f = fmin(fmax((double)g - b, 0.0), 1.0);
      return (double)C[b] + f * (double)(C[b + 1] - C[b]);
    };
    auto at = [&](float y) {  // pixels below mc + y
      if (y >= M.T) return (double)N;
      if (y <= -M.T) return 0.0;
      return cum(map_pos(M, y));
    };
    // smallest y in [lo, hi] with test(y), to ~1e-9 of the range
    auto find = [&](float lo, float hi, auto&& test) {
      for (int r = 0; r < 5; ++r) {
        const float step = (hi - lo) * (1.f / 64.f);
        const uint64_t m = __ballot(test(lo + step * (float)(lane + 1)));
        const int f = m ? __builtin_ctzll(m) : 63;
        hi = lo + step * (float)(f + 1);
        lo = lo + step * (float)f;
      }
      return hi;
    };
    auto set = [&](int b) {
      if (b >= 0 && b < NZ_BINS) atomicOr(&mark[b >> 5], 1u << (b & 31));
    };
    auto mark_bins = [&](int b0, int b1) {  // lanes share the bins
      for (int b = b0 + lane; b <= b1; b += 64) set(b);
    };
    auto mark_ranks = [&](double r, int e) {  // the bins of the pixels of ranks r - e .. r + e
      if (lane <= 2 * e) {
        const double q = fmin(fmax(floor(r) + (double)(lane - e), 0.0), (double)N - 1.0);
        const uint32_t k = (uint32_t)q;
        int a = 0, b = NZ_BINS;  // last bin whose count below is <= k
        while (b - a > 1) {
          const int c = (a + b) >> 1;
          if (C[c] <= k) a = c;
          else b = c;
        }
        set(a);
      }
    };
    double L = 0.0, U = (double)N;
    for (int it = 0; it < max_iter && U - L >= 0.5; ++it) {
      const double n = U - L;
      const double mid = L + 0.5 * n;
      const float ym = find(-M.T, M.T, [&](float y) { return at(y) >= mid; });
      mark_ranks(mid, 4);
      const int bm = pos_bin(map_pos(M, ym));
      mark_bins(bm - 1, bm + 1);
      const float d = find(0.f, 2.f * M.T, [&](float v) {
        return fmin(at(ym + v), U) - fmax(at(ym - v), L) >= 0.5 * n;
      });
      const float thr = (float)fmin(1.4826 * kappa * (double)d, 3e38);
      if (lane == 0 && it < NZ_DHAT) S.dhat[it] = d;
      // m and d are good to a bin or two here; the cuts move kappa * 1.4826 times as far as d
      const float cut = (float)fmin(1.4826 * kappa, 1e3) * 1.5f / (M.a2 + M.a0) + 1.5f / (M.a1 + M.a0);
#pragma unroll
      for (int sgn = -1; sgn <= 1; sgn += 2) {
        const float yd = ym + sgn * d, yc = ym + sgn * thr;
        const int bd = pos_bin(map_pos(M, yd));
        mark_bins(bd - 2, bd + 2);
        mark_ranks(at(yd), 4);
        mark_bins(pos_bin(map_pos(M, yc - cut)) - 1, pos_bin(map_pos(M, yc + cut)) + 1);
      }
      const double nl = at(ym - thr), nu = at(ym + thr);
      const bool same = fabs(nl - L) < 0.25 && fabs(nu - U) < 0.25;
      L = nl;
      U = nu;
      if (same) break;
    }
  }
  __syncthreads();
  // table of the marked bins; all are listed while that fits
  const uint32_t bits = (mark[tid * PER >> 5] >> ((tid * PER) & 31)) & ((1u << PER) - 1u);
  uint32_t n_tab, total;
  const uint32_t first = block_scan((uint32_t)__builtin_popcount(bits), tmp, &n_tab);
  uint32_t c = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j)
    if (bits >> j & 1u) c += std::min<uint32_t>(h[j], NZ_LIST + 1u);
  (void)block_scan(c, tmp, &total);
  const bool all = total <= (uint32_t)NZ_LIST;
  const int ns = S.n_sample;
  uint32_t k = first;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    uint16_t mode = 0;
    if (bits >> j & 1u) {
      if (k < (uint32_t)NZ_TAB) {
        const int b = tid * PER + j;
        uint32_t heavy = 0;
        mode = 0xffffu;
        if (!all && h[j] > (uint32_t)NZ_LIST / 64) {
          // too full to list: the sample value that fills nine tenths of it (of
          // its sorted sample values, then, the middle one) is left out; a bin
          // without such a value stays unlisted
          auto first = [&](auto&& from) {  // first sample key from which on from(key)
            int lo = 0, hi = ns;
            while (lo < hi) {
              const int q = (lo + hi) >> 1;
              if (from(S.sample[q])) hi = q;
              else lo = q + 1;
            }
            return lo;
          };
          const int lo = first([&](uint32_t key) { return map_bin(M, fkey_value(key)) >= b; });
          const int n_in = first([&](uint32_t key) { return map_bin(M, fkey_value(key)) > b; }) - lo;
          if (n_in > 0) heavy = S.sample[lo + n_in / 2];
          const int most = first([&](uint32_t key) { return key > heavy; }) - first([&](uint32_t key) { return key >= heavy; });
          const bool use = 10 * most >= 9 * n_in && n_in > 0;
          mode = use ? (uint16_t)(k + 1) : (uint16_t)0;
          if (!use) heavy = 0;
        }
        S.bin[k] = (uint32_t)b;
        S.below[k] = C[b];
        S.cnt[k] = h[j];
        S.heavy[k] = heavy;
      }
      ++k;
    }
    S.mode[tid * PER + j] = mode;
  }
  if (tid == 0) {
    S.n = N;
    S.n_tab = n_tab <= (uint32_t)NZ_TAB ? (int32_t)n_tab : -1;
  }
}

// The values of the marked bins.
template <typename T>
__global__ __launch_bounds__(NZ_TX) void k_noise_collect(const void* const* imgs, const int64_t* npix,
                                                         NoiseImage* st) {
  const int img = blockIdx.y;
  NoiseImage& S = st[img];
  if (S.n_tab < 0) return;
  __shared__ uint16_t mode[NZ_BINS];
  __shared__ uint32_t buf[NZ_STAGE];
  __shared__ unsigned int cnt, base;
  for (int b = threadIdx.x; b < NZ_BINS / 2; b += NZ_TX)
    reinterpret_cast<uint32_t*>(mode)[b] = reinterpret_cast<const uint32_t*>(S.mode)[b];
  if (threadIdx.x == 0) cnt = 0u;
  const NoiseMap M = S.map;
  __syncthreads();
  for_pixels<T>(imgs[img], npix[img], blockIdx.x, gridDim.x, [&](float x) {
    if (!__builtin_isfinite(x)) return;
    const uint16_t md = mode[map_bin(M, x)];
    if (md == 0) return;
    const uint32_t key = fkey(x);
    if (md != 0xffffu && key == S.heavy[md - 1]) return;
    const unsigned int i = atomicAdd(&cnt, 1u);
    if (i < (unsigned)NZ_STAGE) {
      buf[i] = key;
    } else {  // staging full: append directly
      const unsigned int g = atomicAdd(&S.n_list, 1u);
      if (g < (unsigned)NZ_LIST) S.list[g] = key;
    }
  });
  __syncthreads();
  const unsigned int c = std::min<unsigned>(cnt, NZ_STAGE);
  if (threadIdx.x == 0) base = c ? atomicAdd(&S.n_list, c) : 0u;
  __syncthreads();
  for (unsigned int i = threadIdx.x; i < c; i += NZ_TX)
    if (base + i < (unsigned)NZ_LIST) S.list[base + i] = buf[i];
}

// Result of one image.
struct NoiseResult {
  double sigma;
  int64_t used;
  int iter;
};

__device__ __forceinline__ void noise_result(const NoiseResult& R, int img, int n_img, double* sigma, int64_t* n_used,
                                             int32_t* iters, ExpMeta* meta) {
  if (threadIdx.x == 0) {
    if (sigma) sigma[img] = R.sigma;
    if (n_used) n_used[img] = R.used;
    if (iters) iters[img] = R.iter;
  }
  if (meta) {
    // meta is in epoch order; meta[i].src names the image
    for (int i = threadIdx.x; i < n_img; i += NZ_TX)
      if (meta[i].src == img) meta[i].vs = (float)(R.sigma * R.sigma);
  }
}

__global__ __launch_bounds__(NZ_TX) void k_noise_solve(NoiseImage* st, double kappa, int max_iter, int n_img,
                                                       double* sigma, int64_t* n_used, int32_t* iters,
                                                       ExpMeta* meta) {
  const int img = blockIdx.x, tid = threadIdx.x;
  NoiseImage& S = st[img];
  __shared__ uint32_t A[NZ_LIST];  // the listed keys, sorted
  __shared__ float elo[NZ_TAB], ehi[NZ_TAB], heavy[NZ_TAB];  // first value of a bin and after it; value not listed
  __shared__ uint32_t below[NZ_TAB], cnt[NZ_TAB], off[NZ_TAB];
  __shared__ uint32_t n_heavy[NZ_TAB];  // pixels of the value that is not listed
  __shared__ uint8_t known[NZ_TAB];
  __shared__ uint32_t tmp[NZ_WAVES];
  __shared__ unsigned long long dmin[2];
  __shared__ uint32_t q_rank[16];
  __shared__ int q_bad;
  const uint32_t N = S.n;
  const int nt = S.n_tab;
  bool good = nt >= 0 && S.n_list <= (uint32_t)NZ_LIST;
  NoiseResult R{__builtin_nan(""), 0, 0};
  if (good && N > 0) {
    const NoiseMap M = S.map;
    const int n_list = (int)S.n_list;
    int per = 1;
    while (per * NZ_TX < n_list) per <<= 1;
    for (int i = tid; i < per * NZ_TX; i += NZ_TX) A[i] = i < n_list ? S.list[i] : 0xffffffffu;
    switch (per) {
      case 1: sort_per<1>(A); break;
      case 2: sort_per<2>(A); break;
      case 4: sort_per<4>(A); break;
      case 8: sort_per<8>(A); break;
      case 16: sort_per<16>(A); break;
      default: sort_per<32>(A); break;
    }
    if (tid == 0) q_bad = 0;
    {
      // a bin's lower edge by one half of the workgroup, its upper edge by the other
      static_assert(2 * NZ_TAB == NZ_TX, "two threads per marked bin");
      const int e = tid & (NZ_TAB - 1);
      const bool upper = tid >= NZ_TAB;
      if (e < nt) {
        const int b = (int)S.bin[e] + upper;
        // key of the first value with bin >= b (+inf's when there is none)
        uint32_t lo = fkey(-3.4028234664e38f), hi = fkey(3.4028234664e38f) + 1u;
        if (S.whole) lo = hi = upper ? hi : lo;
        while (lo < hi) {
          const uint32_t k = lo + (hi - lo) / 2;
          if (map_bin(M, fkey_value(k)) >= b) hi = k;
          else lo = k + 1;
        }
        int l = 0, r = n_list;  // listed keys below it
        while (l < r) {
          const int k = (l + r) >> 1;
          if (A[k] < lo) l = k + 1;
          else r = k;
        }
        (upper ? ehi : elo)[e] = fkey_value(lo);
        (upper ? n_heavy : off)[e] = (uint32_t)l;
      }
    }
    __syncthreads();
    if (tid < nt) {
      below[tid] = S.below[tid];
      cnt[tid] = S.cnt[tid];
      const uint32_t rest = S.cnt[tid] - (n_heavy[tid] - off[tid]);
      n_heavy[tid] = rest;
      heavy[tid] = fkey_value(S.heavy[tid]);
      known[tid] = rest == 0 || S.heavy[tid] != 0u;
    }
    __syncthreads();
    // The pixels for which `pred` holds, pred true for a prefix of the sorted
    // pixels: their number, and exact = false when it ends among pixels that
    // are not known.
    auto rank_of = [&](auto&& pred, bool& exact) -> uint32_t {
      int a = 0, b = nt;  // first entry whose first value fails
      while (a < b) {
        const int k = (a + b) >> 1;
        if (pred(elo[k])) a = k + 1;
        else b = k;
      }
      const int j = a - 1;
      if (j < 0) {
        exact &= (nt > 0 ? below[0] : N) == 0u;
        return 0u;
      }
      const uint32_t end = below[j] + cnt[j];
      if (pred(ehi[j])) {  // past this bin, before the next marked one
        exact &= (j + 1 < nt ? below[j + 1] : N) == end;
        return end;
      }
      exact &= known[j] != 0;
      int l = 0, r = (int)(cnt[j] - n_heavy[j]);
      const uint32_t* q = A + off[j];
      while (l < r) {
        const int k = (l + r) >> 1;
        if (pred(fkey_value(q[k]))) l = k + 1;
        else r = k;
      }
      return below[j] + (uint32_t)l + (n_heavy[j] && pred(heavy[j]) ? n_heavy[j] : 0u);
    };
    // The value of the pixel of rank r.
    auto value_at = [&](uint32_t r, bool& exact) -> double {
      int a = 0, b = nt;  // last entry with below <= r (entries of empty bins come before the one that holds r)
      while (a < b) {
        const int k = (a + b) >> 1;
        if (below[k] <= r) a = k + 1;
        else b = k;
      }
      const int j = a - 1;
      if (j < 0 || r >= below[j] + cnt[j] || !known[j]) {
        exact = false;
        return 0.0;
      }
      r -= below[j];
      const uint32_t* q = A + off[j];
      if (n_heavy[j]) {
        int l = 0, e = (int)(cnt[j] - n_heavy[j]);  // listed values below the heavy one
        while (l < e) {
          const int k = (l + e) >> 1;
          if (fkey_value(q[k]) < heavy[j]) l = k + 1;
          else e = k;
        }
        if (r >= (uint32_t)l) {
          if (r < (uint32_t)l + n_heavy[j]) return (double)heavy[j];
          r -= n_heavy[j];
        }
      }
      return (double)fkey_value(q[r]);
    };
    // pixels up to m + D (right) or below m - D
    auto rank_at = [&](double m, double D, bool right, bool& exact) {
      return rank_of([&](float x) {
        const double y = (double)x;
        return right ? y < m || y - m <= D : y < m && m - y > D;
      }, exact);
    };
    uint32_t L = 0, U = N;
    while (U > L) {
      const uint32_t n = U - L;
      const uint32_t k[2] = {(n - 1) / 2, n / 2};
      bool exact = true;
      const double m = 0.5 * (value_at(L + k[0], exact) + value_at(L + k[1], exact));
      // the middle deviations are deviations of listed (or heavy) values: the
      // smallest one that covers more than k pixels of the set
      if (tid < 2) dmin[tid] = ~0ull;
      __syncthreads();
      const float dh = R.iter < NZ_DHAT ? S.dhat[R.iter] : 0.f;
      const double slack = 0.03 * (double)dh + 2.0 / (double)M.a0;  // the plan's value is good to a bin or two
      const double near0 = dh > 0.f ? dh - slack : 0.0, near1 = dh > 0.f ? dh + slack : __builtin_inf();
      // pixels of the set within D of m (never less for a larger D)
      auto within = [&](double D) -> uint32_t {
        bool e = true;
        const uint32_t hi = std::min(rank_at(m, D, true, e), U), lo = std::max(rank_at(m, D, false, e), L);
        return hi > lo ? hi - lo : 0u;
      };
      if (tid < 256) {
        // listed values, sorted by their deviation on either side of m: a wavefront for each side and middle
        const int t = tid >> 7;
        const bool right = (tid >> 6) & 1;
        const int p = wave_first(n_list, [&](int i) { return (double)fkey_value(A[i]) >= m; });
        auto dev_at = [&](int j) { return fabs((double)fkey_value(A[right ? p + j : p - 1 - j]) - m); };
        const int n_side = right ? n_list - p : p;
        const int j0 = wave_first(n_side, [&](int j) { return dev_at(j) >= near0; });
        const int n_near = wave_first(n_side - j0, [&](int j) { return dev_at(j0 + j) > near1; });
        const int j = wave_first(n_near, [&](int i) { return within(dev_at(j0 + i)) > k[t]; });
        if (j < n_near && (tid & 63) == 0)
          atomicMin(&dmin[t], (unsigned long long)__double_as_longlong(dev_at(j0 + j)));
      } else {
        for (int i = tid - 256; i < nt; i += NZ_TX - 256) {
          if (!n_heavy[i]) continue;
          const double D = fabs((double)heavy[i] - m);
          if (!(D >= near0 && D <= near1)) continue;
          const uint32_t c = within(D);
          for (int t = 0; t < 2; ++t)
            if (c > k[t]) atomicMin(&dmin[t], (unsigned long long)__double_as_longlong(D));
        }
      }
      __syncthreads();
      const double dev[2] = {__longlong_as_double((long long)dmin[0]), __longlong_as_double((long long)dmin[1])};
      exact &= dmin[0] != ~0ull && dmin[1] != ~0ull;
      if (!exact) {
        good = false;
        break;
      }
      const double sigma_new = 1.4826 * (0.5 * (dev[0] + dev[1]));
      const double thr = kappa * sigma_new;
      // proof: the pixels within each deviation, and within the next smaller
      // number, counted exactly; and the cuts (ten ranks, one per lane)
      if (tid < 10) {
        bool e = true;
        const int t = tid >> 2;
        const uint64_t bits = t < 2 ? dmin[t] : (uint64_t)__double_as_longlong(thr);
        const bool prev = t < 2 && (tid & 2);
        // (below zero: no deviation, nothing to count)
        const double D = __longlong_as_double((long long)(prev && bits > 0 ? bits - 1 : bits));
        q_rank[tid] = rank_at(m, D, (tid & 1) != 0, e);
        if (!e) q_bad = 1;
      }
      __syncthreads();
      good = q_bad == 0;
      auto inside = [&](int q) -> uint32_t {
        const uint32_t hi = std::min(q_rank[q + 1], U), lo = std::max(q_rank[q], L);
        return hi > lo ? hi - lo : 0u;
      };
      for (int t = 0; t < 2; ++t) {
        good &= inside(4 * t) > k[t];
        if (dmin[t] > 0) good &= inside(4 * t + 2) <= k[t];
      }
      const uint32_t l2 = q_rank[8], u2 = q_rank[9];
      if (!good) break;
      R.sigma = sigma_new;
      R.used = n;
      R.iter++;
      if ((l2 == L && u2 == U) || R.iter >= max_iter) break;
      L = l2;
      U = u2;
      __syncthreads();  // dmin and q_rank are read
    }
  }
  // (every thread computed the same `good` and R)
  if (tid == 0) {
    S.todo = !good;
    if (!good) atomicAdd(&st[0].n_todo, 1u);
  }
  if (good) noise_result(R, img, n_img, sigma, n_used, iters, meta);
}

// The iteration by radix selection over the pixels (11-bit digits of the float
// key, then of the bits of |x - m|), for the images whose places the plan
// missed.  The first workgroup to arrive at such an image leads it: it
// publishes one pass over the pixels at a time (`call`: its number), takes
// pieces like every other workgroup here (`taken`: the last pass a piece was
// taken in), and reads the sums when all pieces are done.  A workgroup
// waits only for pieces that a running workgroup took and, as a helper, for
// the leader, which is running: none that has yet to start is waited for, so
// any number of them may be resident.  All that workgroups share goes through
// relaxed device-scope atomics, ordered by waiting for them (settle): a
// release or acquire of the whole device would write back or drop the L2 each
// time (100 images at once 844 ms instead of 69, before the rest below).
// A step takes at most six passes while the values do not repeat: two digits
// of the median, two of the deviation, the deviations that share these two
// digits as a list (the leader finds the rest there; as soon as few enough are
// left, for the median too), and the clip, which counts the change of the set
// and is the first digit of the next median.
//
// Latency bounds a pass of one image (20 to 35 us: the call, one piece of
// 16384 pixels a workgroup, the sums' atomics), the LDS atomics of equal digits
// many.  Against a launch per pass over every image (26 reads and up to 110
// launches, an image the plan holds among them): 2048^2 FP32 pixels, half of
// them 10^6 times narrower than the others (five steps): one image 1.09 ms ->
// 0.77, 16 images 3.2 -> 2.65, 100 images 19.8 -> 12.0; two far groups (one
// step) 1.36, 3.1 and 15.4 -> 0.37, 1.43 and 8.6; log-normal values (ten steps)
// 1.85, 5.8 and 36.6 -> 1.72, 4.7 and 28.0.  (With a pass of its own for the
// size of a set and no list, eleven passes a step: 1.54, 5.2 and 24.3 in the
// first; with every workgroup calling at every image in turn 64 images of 512^2
// in two groups took 1.57 ms instead of 0.55.)  Where every image is solved
// before, the kernel costs its launch (200 images: within the noise of 1.5 ms).
enum NoisePass { NZ_DIGIT, NZ_DEV_DIGIT, NZ_KEYS, NZ_DEV_KEYS, NZ_CLIP };
struct NoiseTask {
  double m, thr, mn, tn;  // the set |x - m| <= thr; center of the deviations; the next set
  uint64_t pre[2];        // digits found above bit `hi`
  int pass, hi, lo;
};

// Waits for the memory operations this wavefront has issued.
__device__ __forceinline__ void settle() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory"); }
__device__ __forceinline__ uint64_t shared_get(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void shared_set(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint32_t shared_get(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A piece of the current pass for workgroup r of an image: its own one (r)
// first, then every R-th from there (R: workgroups here), then any that nobody
// took (256 workgroups that draw from one counter get in each other's way:
// 1.7 ms a pass; so do 32 that go for the same next piece).  < 0 when there is none left (for
// the leader, which alone starts a pass) or the image is done (for a helper,
// which waits for the next pass).  last: the pass whose own piece was tried.
// sh: 3 words of LDS.
__device__ __forceinline__ int noise_take(NoiseImage& S, int pieces, int r, uint32_t& last, NoiseTask* t,
                                          uint32_t* sh) {
  const int tid = threadIdx.x;
  for (;;) {
    __syncthreads();  // t and sh are read
    if (tid == 0) {
      sh[0] = shared_get(&S.call);
      sh[1] = ~0u;
      sh[2] = min(shared_get(&S.role), (uint32_t)pieces);  // workgroups here
      settle();
    }
    __syncthreads();
    const uint32_t seq = sh[0];
    if (seq == ~0u) return -1;
    int want = r;
    if (seq == last) {
      const int R = (int)sh[2];
      if (tid < pieces && shared_get(&S.taken[tid]) < seq)
        atomicMin(&sh[1], (uint32_t)((tid % R + R - r % R) % R * NZ_PIECES + tid));
      __syncthreads();
      want = sh[1] == ~0u ? -1 : (int)(sh[1] % NZ_PIECES);
    }
    last = seq;
    if (want < 0 || seq == 0) {
      if (r == 0) return -1;
      if (tid == 0)
        while (shared_get(&S.call) == seq) __builtin_amdgcn_s_sleep(32);
      continue;
    }
    if (tid == 0) {
      t->m = __longlong_as_double((long long)shared_get(&S.task[0]));
      t->thr = __longlong_as_double((long long)shared_get(&S.task[1]));
      t->mn = __longlong_as_double((long long)shared_get(&S.task[2]));
      t->tn = __longlong_as_double((long long)shared_get(&S.task[3]));
      t->pre[0] = shared_get(&S.task[4]);
      t->pre[1] = shared_get(&S.task[5]);
      const uint32_t w = (uint32_t)shared_get(&S.task[6]);
      t->pass = w & 255;
      t->hi = w >> 8 & 255;
      t->lo = w >> 16;
      settle();
      // taken: the pass has not ended before this piece is done, so what was read above is its own
      sh[2] = __hip_atomic_fetch_max(&S.taken[want], seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < seq;
    }
    __syncthreads();
    if (sh[2]) return want;
  }
}

constexpr int NZ_DIGITS = 2048;
constexpr int NZ_CHANGED = NZ_DIGITS;  // clip: the pixels in one of the two sets only, after the digits
constexpr int NZ_MOST_KEYS = NZ_LIST / 2;
static_assert(2 * NZ_DIGITS * 2 <= NZ_BINS, "64-bit sums in the histogram's place");
typedef unsigned long long NoiseSum;
__device__ __forceinline__ NoiseSum* noise_sums(NoiseImage& S) { return reinterpret_cast<NoiseSum*>(S.hist); }

__device__ __forceinline__ int noise_bins(const NoiseTask& t) {  // of them, in use by a pass
  return t.pass == NZ_CLIP ? NZ_CHANGED + 1
         : t.pass == NZ_KEYS || t.pass == NZ_DEV_KEYS ? 0 : t.pre[0] != t.pre[1] ? 2 * NZ_DIGITS : NZ_DIGITS;
}

// One piece (fewer than 2^32 pixels): its histogram added to the image's, or
// its keys to the list.
template <typename T>
__device__ __forceinline__ void noise_piece(const void* img, int64_t n, int piece, int pieces, NoiseImage& S,
                                            const NoiseTask& t, uint32_t* h, uint32_t* tmp, uint32_t* cnt) {
  const double m = t.m, thr = t.thr, mn = t.mn, tn = t.tn;
  const bool two = t.pre[0] != t.pre[1], dev = t.pass == NZ_DEV_DIGIT || t.pass == NZ_DEV_KEYS;
  const int hi = t.hi, lo = t.lo;
  const uint64_t p0 = t.pre[0] >> hi, p1 = t.pre[1] >> hi;
  auto key_of = [&](float x) {
    return dev ? (uint64_t)__double_as_longlong(fabs((double)x - mn)) : (uint64_t)fkey(x);
  };
  if (t.pass == NZ_KEYS || t.pass == NZ_DEV_KEYS) {
    uint64_t* stage = reinterpret_cast<uint64_t*>(h);
    uint64_t* list = reinterpret_cast<uint64_t*>(S.list);
    if (threadIdx.x == 0) *cnt = 0u;
    __syncthreads();
    for_pixels<T, 2>(img, n, piece, pieces, [&](float x) {
      if (!(__builtin_isfinite(x) && fabs((double)x - m) <= thr)) return;
      const uint64_t key = key_of(x);
      if (key >> hi != p0 && !(two && key >> hi == p1)) return;
      const uint32_t i = atomicAdd(cnt, 1u);
      if (i < (uint32_t)NZ_DIGITS) {
        stage[i] = key;
      } else {  // staging full: append directly
        const uint32_t g = atomicAdd(&S.n_list, 1u);
        if (g < (uint32_t)NZ_MOST_KEYS) shared_set(list + g, key);
      }
    });
    __syncthreads();
    const uint32_t c = min(*cnt, (uint32_t)NZ_DIGITS);
    if (threadIdx.x == 0) tmp[0] = c ? atomicAdd(&S.n_list, c) : 0u;
    __syncthreads();
    const uint32_t base = tmp[0];
    for (uint32_t i = threadIdx.x; i < c; i += NZ_TX)
      if (base + i < (uint32_t)NZ_MOST_KEYS) shared_set(list + base + i, stage[i]);
  } else {
    const int bins = two ? 2 * NZ_DIGITS : NZ_DIGITS;
    for (int b = threadIdx.x; b < bins; b += NZ_TX) h[b] = 0u;
    __syncthreads();
    if (t.pass == NZ_CLIP) {
      uint32_t c = 0, total;
      for_pixels<T, 2>(img, n, piece, pieces, [&](float x) {
        if (!__builtin_isfinite(x)) return;
        const bool in = fabs((double)x - mn) <= tn;
        c += in != (fabs((double)x - m) <= thr) ? 1u : 0u;
        if (in) atomicAdd(&h[fkey(x) >> 21], 1u);
      });
      (void)block_scan(c, tmp, &total);
      if (threadIdx.x == 0 && total) atomicAdd(&noise_sums(S)[NZ_CHANGED], (NoiseSum)total);
    } else {
      const uint32_t mask = (1u << (hi - lo)) - 1u;
      for_pixels<T, 2>(img, n, piece, pieces, [&](float x) {
        if (!(__builtin_isfinite(x) && fabs((double)x - m) <= thr)) return;
        const uint64_t key = key_of(x);
        const uint32_t d = (uint32_t)(key >> lo) & mask;
        if (key >> hi == p0) atomicAdd(&h[d], 1u);
        if (two && key >> hi == p1) atomicAdd(&h[NZ_DIGITS + d], 1u);
      });
    }
    __syncthreads();
    for (int b = threadIdx.x; b < bins; b += NZ_TX)
      if (h[b]) atomicAdd(&noise_sums(S)[b], (NoiseSum)h[b]);
  }
  settle();
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_fetch_add(&S.done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Where the leader of an image stands (in LDS, so that nothing of it is live
// through the pixels of a pass): the pass that was published, and the
// selection it belongs to.
struct NoiseLead {
  NoiseTask task;
  int64_t n, rank[2], left;  // size of the set; ranks among the keys with the digits found; those keys
  double sigma;
  uint32_t seq;  // passes so far
  int iter, dev;  // steps so far; the selection is of deviations
};

// The pass in L.task, open for all workgroups: its sums and keys cleared.
__device__ __forceinline__ void noise_publish(NoiseImage& S, NoiseLead& L) {
  const int tid = threadIdx.x;
  for (int b = tid; b < noise_bins(L.task); b += NZ_TX)
    __hip_atomic_store(&noise_sums(S)[b], (NoiseSum)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  settle();
  __syncthreads();
  if (tid == 0) {
    const NoiseTask& t = L.task;
    shared_set(&S.task[0], (uint64_t)__double_as_longlong(t.m));
    shared_set(&S.task[1], (uint64_t)__double_as_longlong(t.thr));
    shared_set(&S.task[2], (uint64_t)__double_as_longlong(t.mn));
    shared_set(&S.task[3], (uint64_t)__double_as_longlong(t.tn));
    shared_set(&S.task[4], t.pre[0]);
    shared_set(&S.task[5], t.pre[1]);
    shared_set(&S.task[6], (uint64_t)(t.pass | t.hi << 8 | t.lo << 16));
    __hip_atomic_store(&S.n_list, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&S.done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    settle();
    __hip_atomic_store(&S.call, ++L.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Reads the sums of the pass that has ended and sets the next one; false when
// the result is final.
__device__ __forceinline__ bool noise_advance(NoiseImage& S, NoiseLead& L, NoiseSum* sums, NoiseSum* tmp, uint64_t* sh,
                                              double kappa, int max_iter) {
  const int tid = threadIdx.x;
  NoiseTask t = L.task;
  int64_t n = L.n, rank0 = L.rank[0], rank1 = L.rank[1], left = L.left;
  double sigma = L.sigma;
  int iter = L.iter, dev = L.dev;
  bool more = true;
  for (int b = tid; b < noise_bins(t); b += NZ_TX)
    sums[b] = __hip_atomic_load(&noise_sums(S)[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();  // (L is read, too)
  // the digit (at bit lo) that holds the rank among the keys H counts; the keys that have it
  auto digit = [&](const NoiseSum* H, int lo, uint64_t& pre, int64_t& rank) {
    const NoiseSum c0 = H[2 * tid], c1 = H[2 * tid + 1];
    NoiseSum total;
    const NoiseSum e = block_scan(c0 + c1, tmp, &total);
    const NoiseSum r = (NoiseSum)rank;
    if (r >= e && r < e + c0 + c1) {
      const bool second = r >= e + c0;
      sh[0] = (uint64_t)(2 * tid + (second ? 1 : 0));
      sh[1] = e + (second ? c0 : 0);
      sh[2] = second ? c1 : c0;
    }
    __syncthreads();
    pre |= sh[0] << lo;
    rank -= (int64_t)sh[1];
    const int64_t c = (int64_t)sh[2];
    __syncthreads();
    return c;
  };
  auto digits = [&](int lo) {
    const bool two = t.pre[0] != t.pre[1];
    const int64_t c0 = digit(sums, lo, t.pre[0], rank0);
    const int64_t c1 = digit(two ? sums + NZ_DIGITS : sums, lo, t.pre[1], rank1);
    left = t.pre[0] != t.pre[1] ? c0 + c1 : c0;
    t.hi = lo;
  };
  auto begin = [&](int bits) {
    t.pre[0] = t.pre[1] = 0;
    rank0 = (n - 1) / 2;
    rank1 = n / 2;
    left = n;
    t.hi = bits;
  };
  if (t.pass == NZ_CLIP) {
    const bool changed = sums[NZ_CHANGED] != 0;
    NoiseSum total;
    (void)block_scan(sums[2 * tid] + sums[2 * tid + 1], tmp, &total);
    n = (int64_t)total;
    t.m = t.mn;
    t.thr = t.tn;
    more = n > 0 && (iter == 0 || (changed && iter < max_iter));
    begin(32);
    dev = 0;
    if (more) digits(21);  // the clip's digits are the first ones of the values
  } else if (t.pass == NZ_DIGIT || t.pass == NZ_DEV_DIGIT) {
    digits(t.lo);
  } else {
    // the rest of the digits among the listed keys
    const uint64_t* list = reinterpret_cast<const uint64_t*>(S.list);
    const int n_keys = (int)left;
    while (t.hi > 0) {
      const int lo = max(t.hi - 11, 0);
      const bool two = t.pre[0] != t.pre[1];
      for (int b = tid; b < 2 * NZ_DIGITS; b += NZ_TX) sums[b] = 0;
      __syncthreads();
      for (int i = tid; i < n_keys; i += NZ_TX) {
        const uint64_t key = shared_get(list + i);
        const uint32_t d = (uint32_t)(key >> lo) & ((1u << (t.hi - lo)) - 1u);
        if (key >> t.hi == t.pre[0] >> t.hi) atomicAdd(&sums[d], (NoiseSum)1);
        if (two && key >> t.hi == t.pre[1] >> t.hi) atomicAdd(&sums[NZ_DIGITS + d], (NoiseSum)1);
      }
      __syncthreads();
      digits(lo);
    }
  }
  if (more && t.hi == 0) {  // both middle values
    if (!dev) {
      t.mn = 0.5 * ((double)fkey_value((uint32_t)t.pre[0]) + (double)fkey_value((uint32_t)t.pre[1]));
      begin(63);
      dev = 1;
    } else {
      sigma = 1.4826 *
              (0.5 * (__longlong_as_double((long long)t.pre[0]) + __longlong_as_double((long long)t.pre[1])));
      t.tn = kappa * sigma;
      iter++;
      t.pre[0] = t.pre[1] = 0;
    }
  }
  if (t.hi == 0) {
    t.pass = NZ_CLIP;
  } else {
    t.pass = left <= NZ_MOST_KEYS ? (dev ? NZ_DEV_KEYS : NZ_KEYS) : (dev ? NZ_DEV_DIGIT : NZ_DIGIT);
    t.lo = max(t.hi - 11, 0);
  }
  if (tid == 0) {
    L.task = t;
    if (more) L.n = n;  // (what a last clip finds is not a set that was used)
    L.rank[0] = rank0;
    L.rank[1] = rank1;
    L.left = left;
    L.sigma = sigma;
    L.iter = iter;
    L.dev = dev;
  }
  __syncthreads();
  return more;
}

// Pieces of a pass over an image of n pixels: one for each workgroup that an
// image gets (a piece costs its histogram of up to 4096 words), of 16 pixels a
// thread or more and of fewer than 2^32 pixels (memory ends before the most
// pieces of that size).
__device__ __forceinline__ int noise_pieces(int64_t n, uint32_t n_todo) {
  const int64_t most = std::min<uint32_t>(NZ_PIECES, std::max<uint32_t>(8u, gridDim.x / n_todo));
  return (int)std::min<int64_t>(std::max<int64_t>(most, std::min<int64_t>(NZ_PIECES, (n >> 31) + 1)),
                                (n + NZ_TX * 16 - 1) / (NZ_TX * 16));
}

template <typename T>
__global__ __launch_bounds__(NZ_TX) void k_noise_pixels(const void* const* imgs, const int64_t* npix, NoiseImage* st,
                                                        double kappa, int max_iter, int n_img, double* sigma,
                                                        int64_t* n_used, int32_t* iters, ExpMeta* meta) {
  __shared__ alignas(8) uint32_t h[2 * NZ_DIGITS];
  __shared__ NoiseSum sums[2 * NZ_DIGITS];
  __shared__ uint32_t tmp[NZ_WAVES];
  __shared__ NoiseSum tmp_sum[NZ_WAVES];
  __shared__ uint64_t sh[3];
  __shared__ NoiseTask task;
  __shared__ NoiseLead L;
  __shared__ uint32_t sh_i[3], sh_n;
  const int tid = threadIdx.x;
  const uint32_t n_todo = st[0].n_todo;
  if (n_todo == 0u) return;
  for (;;) {
    // the next image, from this workgroup's own one on, that is not done and has fewer workgroups than pieces (all
    // images are looked at together: one after another took 2 us each)
    if (tid == 0) sh_n = ~0u;
    __syncthreads();
    for (int v = tid; v < n_img; v += NZ_TX) {
      const int i = (int)(((int64_t)blockIdx.x + v) % n_img);
      NoiseImage& S = st[i];
      if (S.todo && shared_get(&S.role) < (uint32_t)noise_pieces(npix[i], n_todo) && shared_get(&S.call) != ~0u)
        atomicMin(&sh_n, (uint32_t)v);
    }
    __syncthreads();
    if (sh_n == ~0u) return;
    const int img = (int)(((int64_t)blockIdx.x + sh_n) % n_img);
    NoiseImage& S = st[img];
    const int64_t n_pix = npix[img];
    const int pieces = noise_pieces(n_pix, n_todo);
    if (tid == 0) sh_i[0] = __hip_atomic_fetch_add(&S.role, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int role = (int)sh_i[0];
    if (role >= pieces) continue;  // others came first
    if (role == 0) {
      if (tid == 0) {
        L.task = NoiseTask{0.0, __builtin_inf(), 0.0, __builtin_inf(), {0, 0}, NZ_CLIP, 0, 0};
        L.n = 0;
        L.sigma = __builtin_nan("");
        L.seq = 0;
        L.iter = L.dev = 0;
      }
      __syncthreads();
      noise_publish(S, L);
    }
    uint32_t last = 0;
    for (;;) {
      const int i = noise_take(S, pieces, role, last, &task, sh_i);
      if (i >= 0) {
        noise_piece<T>(imgs[img], n_pix, i, pieces, S, task, h, tmp, &sh_n);
        continue;
      }
      if (role > 0) break;
      if (tid == 0)
        while (__hip_atomic_load(&S.done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < (uint32_t)pieces)
          __builtin_amdgcn_s_sleep(2);
      settle();
      __syncthreads();
      if (noise_advance(S, L, sums, tmp_sum, sh, kappa, max_iter)) {
        noise_publish(S, L);
        continue;
      }
      if (tid == 0) __hip_atomic_store(&S.call, ~0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      noise_result(NoiseResult{L.sigma, L.n, L.iter}, img, n_img, sigma, n_used, iters, meta);
      break;
    }
    __syncthreads();  // L and sh_n are read
  }
}

size_t noise_pixels_offset() { return offsetof(NoiseImage, n_todo); }

size_t noise_scratch_bytes(int n_img) { return sizeof(NoiseImage) * (size_t)n_img; }

template <typename T>
static hipError_t noise_t(const void* const* d_imgs, const int64_t* d_npix, int64_t max_pix, int n_img, double kappa,
                          int max_iter, void* scratch, double* d_sigma, int64_t* d_used, int32_t* d_iters,
                          ExpMeta* d_meta, hipStream_t s) {
  NoiseImage* st = static_cast<NoiseImage*>(scratch);
  // about four workgroups per resident one (two fit a CU) for balance, while
  // each has 64 pixels per thread or more: its histogram costs 16384 adds
  const int64_t per = std::max<int64_t>(1, 2048 / n_img);
  const unsigned bx = (unsigned)std::min<int64_t>(per, std::max<int64_t>(1, (max_pix + NZ_TX * 64 - 1) / (NZ_TX * 64)));
  const dim3 grid(bx, (unsigned)n_img), blk(NZ_TX);
  hipLaunchKernelGGL(k_noise_sample<T>, dim3(n_img), blk, 0, s, d_imgs, d_npix, st, kappa, max_iter);
  hipLaunchKernelGGL(k_noise_bins<T>, grid, blk, 0, s, d_imgs, d_npix, st);
  hipLaunchKernelGGL(k_noise_plan, dim3(n_img), blk, 0, s, st, kappa, max_iter);
  hipLaunchKernelGGL(k_noise_collect<T>, grid, blk, 0, s, d_imgs, d_npix, st);
  hipLaunchKernelGGL(k_noise_solve, dim3(n_img), blk, 0, s, st, kappa, max_iter, n_img, d_sigma, d_used, d_iters,
                     d_meta);
  if (max_pix > NZ_WHOLE)  // (images listed whole are always solved above)
    hipLaunchKernelGGL(k_noise_pixels<T>, dim3(512), blk, 0, s, d_imgs, d_npix, st, kappa, max_iter, n_img, d_sigma,
                       d_used, d_iters, d_meta);
  return hipGetLastError();
}

hipError_t launch_noise(const void* const* d_imgs, const int64_t* d_npix, int64_t max_pix, int n_img, dt_dtype dtype,
                        double kappa, int max_iter, void* scratch, double* d_sigma, int64_t* d_used, int32_t* d_iters,
                        ExpMeta* d_meta, hipStream_t s) {
  if (n_img <= 0) return hipSuccess;
  return dtype == DT_F16 ? noise_t<_Float16>(d_imgs, d_npix, max_pix, n_img, kappa, max_iter, scratch, d_sigma, d_used,
                                             d_iters, d_meta, s)
                         : noise_t<float>(d_imgs, d_npix, max_pix, n_img, kappa, max_iter, scratch, d_sigma, d_used,
                                          d_iters, d_meta, s);
}

}  // namespace dtk
