// k_clip.hip -- per-intersection outlier trimming of candidate orbits
// (Sec. 5.2.3): an artifact in one image can carry a chance alignment above
// threshold; under the constant-flux model each valid intersection e is an
// independent flux estimate f_e = psi_e / phi_e of variance 1 / phi_e, so the
// residuals chi_e = (psi_e - F phi_e) / sqrt(phi_e) about the expectation F
// are standard normal.  Iteration 1 takes F = median(f_e), so that one dominant
// artifact cannot set it; every later round takes the weighted mean
// F = sum psi / sum phi of the samples the previous round kept.  A round
// keeps the samples with |chi_e| <= kappa; it stops when a round keeps
// exactly the set it started from, or after max_iter rounds.
//
// One wavefront per candidate, or per four (launch_clip).  Its exposures are
// cut into 64 runs (16), one lane walking each from a cold start with the
// stack's device code (a candidate's walk is a serial chain: one lane over all
// exposures, two wavefronts for a hundred candidates, took 117 us for 200
// exposures, and 28 us more in a second kernel for the rest; this takes 16 us
// together); the samples' (psi, phi) meet in LDS, where the lanes, each owning
// up to 8 exposures, find the median by ranking the valid ones and iterate the
// clipping with FP64 wave reductions.  The per-sample arithmetic of the fit is
// FP64 without contraction, as in the definition.
#include "dt_stack.hpp"

namespace dtk {

constexpr int CLIP_PER_LANE = 8;  // exposures per lane: n_exp <= 512

// (psi, phi) of candidate o's exposures ({0, 0} where no valid sample) into
// smp, by `lanes` lanes of which this is `lane`.
__device__ __forceinline__ void clip_samples(const StackArgs& A, int64_t o, float2* smp, int lane, int lanes) {
  double a = 0, e = 0, inc = 0, node = 0, peri = 0, m0 = 0;
  bool ok = o >= 0 && o < A.n;
  if (ok) {
    a = A.a[o]; e = A.e[o]; inc = A.inc[o]; node = A.node[o]; peri = A.peri[o]; m0 = A.m0[o];
    ok = orbit_ok(a, e, inc, node, peri, m0);
  }
  const int ch = (A.n_exp + lanes - 1) / lanes;
  const int ex0 = lane * ch, cnt = min(ch, A.n_exp - ex0);
  if (!ok) {
    for (int i = 0; i < cnt; ++i) smp[ex0 + i] = make_float2(0.f, 0.f);
    return;
  }
  if (cnt <= 0) return;
  Orbit ob;
  orbit_prep(a, e, inc, node, peri, m0, ob);
  walk_orbit<false>(ob, A.meta + ex0, cnt, A.epoch, [&](int i, const SampleOut& so) {
    const ExpMeta& x = A.meta[ex0 + i];
    float2 v = make_float2(0.f, 0.f);
    if (so.inside) {
      v = A.planes[x.plane_off + (int64_t)so.iy * x.W + so.ix];
      if (!(v.y > 0.f)) v = make_float2(0.f, 0.f);
    }
    smp[ex0 + i] = v;
  });
}

__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// The trimming of candidate r from its samples, by a wavefront; fl: LDS for
// the fluxes psi / phi of the valid samples, in epoch order.
__device__ __forceinline__ void clip_fit(const float2* smp, int n_exp, int64_t r, double kappa, int max_iter, double* fl,
                                         float* __restrict__ snr, float* __restrict__ flux,
                                         int32_t* __restrict__ nkept) {
#pragma clang fp contract(off)
  const int lane = threadIdx.x;
  double ps[CLIP_PER_LANE], ph[CLIP_PER_LANE];
  int at[CLIP_PER_LANE];  // place among the valid samples
  bool valid[CLIP_PER_LANE], kept[CLIP_PER_LANE];
  int nvalid = 0;
#pragma unroll
  for (int q = 0; q < CLIP_PER_LANE; ++q) {
    const int ex = lane + 64 * q;
    const float2 v = ex < n_exp ? smp[ex] : make_float2(0.f, 0.f);
    ps[q] = v.x;
    ph[q] = v.y;
    valid[q] = v.y > 0.f;
    kept[q] = valid[q];
    const uint64_t m = __ballot(valid[q]);
    at[q] = nvalid + __popcll(m & ((1ull << lane) - 1ull));
    nvalid += __popcll(m);
    if (valid[q]) fl[at[q]] = ps[q] / ph[q];
  }
  __syncthreads();
  // iteration 1 expectation: the median of the per-sample fluxes (ranks with
  // ties broken by exposure order; mean of the two middle values)
  const int lo = (nvalid - 1) / 2, hi = nvalid / 2;
  double vlo = 0.0, vhi = 0.0;
#pragma unroll
  for (int q = 0; q < CLIP_PER_LANE; ++q) {
    if (!valid[q]) continue;
    const double f = fl[at[q]];
    int rank = 0;
    for (int j = 0; j < nvalid; ++j) rank += (fl[j] < f || (fl[j] == f && j < at[q])) ? 1 : 0;
    if (rank == lo) vlo = f;
    if (rank == hi) vhi = f;
  }
  // exactly one lane holds each middle value; the others add zeros
  double F = 0.5 * (wave_sum_d(vlo) + wave_sum_d(vhi));
  for (int it = 0; it < max_iter && nvalid > 0; ++it) {
    if (it > 0) {
      double P = 0.0, Q = 0.0;
#pragma unroll
      for (int q = 0; q < CLIP_PER_LANE; ++q)
        if (kept[q]) {
          P += ps[q];
          Q += ph[q];
        }
      F = wave_sum_d(P) / wave_sum_d(Q);
    }
    bool changed = false;
#pragma unroll
    for (int q = 0; q < CLIP_PER_LANE; ++q) {
      if (!valid[q]) continue;
      const bool k = fabs(ps[q] - F * ph[q]) / sqrt(ph[q]) <= kappa;
      changed |= k != kept[q];
      kept[q] = k;
    }
    if (it > 0 && __ballot(changed) == 0ull) break;
  }
  double P = 0.0, Q = 0.0;
  int cnt = 0;
#pragma unroll
  for (int q = 0; q < CLIP_PER_LANE; ++q)
    if (kept[q]) {
      P += ps[q];
      Q += ph[q];
      cnt++;
    }
  P = wave_sum_d(P);
  Q = wave_sum_d(Q);
  cnt = (int)wave_sum_d((double)cnt);
  if (lane == 0) {
    if (snr) snr[r] = Q > 0.0 ? (float)(P / sqrt(Q)) : 0.f;
    if (flux) flux[r] = Q > 0.0 ? (float)(P / Q) : 0.f;
    if (nkept) nkept[r] = cnt;
  }
}

// A wavefront takes C candidates, 64 / C lanes each for the walk.
template <int C>
__global__ __launch_bounds__(64) void k_clip(StackArgs A, const int64_t* __restrict__ ids, int64_t m, double kappa,
                                             int max_iter, float* __restrict__ snr, float* __restrict__ flux,
                                             int32_t* __restrict__ nkept) {
  __shared__ float2 smp[64 * CLIP_PER_LANE];
  __shared__ double fl[64 * CLIP_PER_LANE];
  constexpr int LANES = 64 / C;
  const int64_t r0 = (int64_t)blockIdx.x * C;
  const int c = threadIdx.x / LANES;
  if (r0 + c < m) clip_samples(A, ids[r0 + c], smp + c * A.n_exp, threadIdx.x % LANES, LANES);
#pragma unroll 1
  for (int q = 0; q < C && r0 + q < m; ++q) {
    __syncthreads();  // the samples are there; fl is read
    clip_fit(smp + q * A.n_exp, A.n_exp, r0 + q, kappa, max_iter, fl, snr, flux, nkept);
  }
}

hipError_t launch_clip(const StackArgs& a, const int64_t* d_ids, int64_t m, double kappa, int max_iter, float* snr,
                       float* flux, int32_t* nkept, hipStream_t s) {
  if (m <= 0) return hipSuccess;
  if (a.n_exp > 64 * CLIP_PER_LANE) return hipErrorInvalidValue;
  auto launch = [&](auto k) {
    constexpr int C = decltype(k)::value;
    hipLaunchKernelGGL(k_clip<C>, dim3((unsigned)((m + C - 1) / C)), dim3(64), 0, s, a, d_ids, m, kappa, max_iter, snr,
                       flux, nkept);
  };
  // A cold start costs several warm ones, so with more candidates than fill the
  // chip, and few exposures, sixteen lanes walk one: 10^5 candidates x 5, 20 and
  // 100 exposures 312, 318 and 385 us -> 185, 217 and 277; 10^4 56, 59 and 66 ->
  // 50, 56 and 65; 4000 40 -> 43 (20 exposures), 100 28 -> 39.  (Eight lanes:
  // 171 and 195, but 10^4 64.)  One lane per candidate and a second kernel for
  // the fit: 219, 255 and 709 us for 10^5.
  if (m >= 8192 && a.n_exp <= 16 * CLIP_PER_LANE) launch(std::integral_constant<int, 4>{});
  else launch(std::integral_constant<int, 1>{});
  return hipGetLastError();
}

}  // namespace dtk
