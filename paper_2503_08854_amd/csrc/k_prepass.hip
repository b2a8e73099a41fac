// k_prepass.hip -- exposure metadata and the matched-filter pre-pass.
//
// Sec. 3 (FindLocalSignal): detection significance comes from a matched
// filter with a Gaussian PSF whose width is in the image header, weighted by
// the pixel noise variance.  For a stamp P centred on the nearest pixel of an
// intersection, the filter output is psi = sum P D / V and its variance is
// phi = sum P^2 / V.  Both are linear in the pixels, so evaluating them once
// per pixel of every exposure ("planes") and gathering at the intersection
// gives exactly the per-intersection filter.  The Gaussian stamp is
// separable, so each plane is a row pass followed by a column pass of a 1-D
// kernel over LDS-staged tiles.
#include <algorithm>

#include "dt_common.hpp"

namespace dtk {

// ----------------------------------------------------------------------------
// Exposure metadata (one thread per exposure).  TAN (gnomonic) projection
// with the native pole at LONPOLE = 180 deg: intermediate coordinates are
// xi = u.east / u.centre and eta = u.north / u.centre (radians) for a
// direction u; pixels are CRPIX - 1 + CD^-1 (xi, eta) in degrees.  The basis
// is rotated from equatorial to ecliptic J2000 so that samples need no frame
// rotation.
// ----------------------------------------------------------------------------
__global__ void k_exposure_prep(const dt_exposure* __restrict__ in, const int64_t* __restrict__ plane_off,
                                const int32_t* __restrict__ src, const int32_t* __restrict__ rad, int n,
                                ExpMeta* __restrict__ out) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const dt_exposure x = in[i];
  const double d2r = PI / 180.0;
  double sa, ca, sd, cd;
  sincos(x.crval_deg[0] * d2r, &sa, &ca);
  sincos(x.crval_deg[1] * d2r, &sd, &cd);
  double eps = OBLIQUITY_ARCSEC / 3600.0 * d2r;
  double se, ce;
  sincos(eps, &se, &ce);
  // equatorial basis
  double c[3] = {cd * ca, cd * sa, sd};
  double ea[3] = {-sa, ca, 0.0};
  double no[3] = {-sd * ca, -sd * sa, cd};
  // equatorial -> ecliptic: (x, ce*y + se*z, -se*y + ce*z)
  auto to_ecl = [&](const double v[3], double w[3]) {
    w[0] = v[0];
    w[1] = ce * v[1] + se * v[2];
    w[2] = -se * v[1] + ce * v[2];
  };
  double cE[3], eE[3], nE[3];
  to_ecl(c, cE);
  to_ecl(ea, eE);
  to_ecl(no, nE);
  double det = x.cd_deg[0] * x.cd_deg[3] - x.cd_deg[1] * x.cd_deg[2];
  double i00 = x.cd_deg[3] / det, i01 = -x.cd_deg[1] / det;
  double i10 = -x.cd_deg[2] / det, i11 = x.cd_deg[0] / det;
  double r2d = 180.0 / PI;
  ExpMeta m;
  m.t = x.t;
  m.ox = x.obs_xyz_au[0];
  m.oy = x.obs_xyz_au[1];
  m.oz = x.obs_xyz_au[2];
  m.cx = cE[0];
  m.cy = cE[1];
  m.cz = cE[2];
  m.a0x = r2d * (i00 * eE[0] + i01 * nE[0]);
  m.a0y = r2d * (i00 * eE[1] + i01 * nE[1]);
  m.a0z = r2d * (i00 * eE[2] + i01 * nE[2]);
  m.a1x = r2d * (i10 * eE[0] + i11 * nE[0]);
  m.a1y = r2d * (i10 * eE[1] + i11 * nE[1]);
  m.a1z = r2d * (i10 * eE[2] + i11 * nE[2]);
  m.px0 = x.crpix[0] - 1.0;
  m.py0 = x.crpix[1] - 1.0;
  m.gap = i > 0 ? x.t - in[i - 1].t : 0.0;  // input is in epoch order
  m.inv_gap = m.gap > 0.0 ? 1.0 / m.gap : 0.0;
  m.plane_off = plane_off[i];
  m.W = x.width;
  m.H = x.height;
  m.src = src[i];
  m.fwhm = x.psf_fwhm_px;
  m.R = rad[i];
  m.vs = 0.f;
  // first later exposure whose epoch exceeds this one by more than CK_SPAN
  // (the input is in epoch order and t_j - t is non-decreasing in j); n + 1
  // when there is none
  int lo = i + 1, hi = n;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (in[mid].t - x.t > CK_SPAN) hi = mid;
    else lo = mid + 1;
  }
  m.ck_next = lo < n ? lo : n + 1;
  m.strip = prep_strip(m.R, m.W);
  // Sky cone of the image.  The pixel (x, y) is the direction
  // c + xi e + eta n with (xi, eta) = CD (x - px0, y - py0) in radians; the
  // axis is the centre pixel's direction and the half-angle is the largest
  // angle to a corner of the rectangle widened by one pixel.  The cone's
  // trace on the tangent plane is an ellipse (convex) when the axis is within
  // ~78 deg of c and the half-angle below ~6 deg, so holding the four corners
  // it holds the whole rectangle.  Otherwise no cone is used.
  auto dir = [&](double px, double py, double d[3]) {
    const double dx = px - m.px0, dy = py - m.py0;
    const double xi = d2r * (x.cd_deg[0] * dx + x.cd_deg[1] * dy);
    const double eta = d2r * (x.cd_deg[2] * dx + x.cd_deg[3] * dy);
    for (int k = 0; k < 3; ++k) d[k] = cE[k] + xi * eE[k] + eta * nE[k];
  };
  double u[3];
  dir(0.5 * (x.width - 1), 0.5 * (x.height - 1), u);
  const double un = 1.0 / sqrt(u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);
  for (int k = 0; k < 3; ++k) u[k] *= un;
  bool cone = (u[0] * cE[0] + u[1] * cE[1] + u[2] * cE[2]) > 0.2;
  double tmax = 0.0;
  for (int q = 0; q < 4; ++q) {
    double d[3];
    dir((q & 1) ? x.width + 0.5 : -1.5, (q & 2) ? x.height + 0.5 : -1.5, d);
    const double cs = u[0] * d[0] + u[1] * d[1] + u[2] * d[2];
    const double c0 = u[1] * d[2] - u[2] * d[1], c1 = u[2] * d[0] - u[0] * d[2], c2 = u[0] * d[1] - u[1] * d[0];
    const double sn = sqrt(c0 * c0 + c1 * c1 + c2 * c2);
    if (!(cs > 0.0)) cone = false;
    else tmax = fmax(tmax, sn / cs);
  }
  cone = cone && tmax <= 0.1;
  m.ux = cone ? u[0] : 0.0;
  m.uy = cone ? u[1] : 0.0;
  m.uz = cone ? u[2] : 0.0;
  m.cone_tan = cone ? tmax * 1.0001 + 1e-12 : 0.0;
  m.cone_lim = cone ? 0.0 : __builtin_inf();
  // the scaled rectangle test (see ExpMeta)
  {
    const double hx = 0.5 * x.width + 0.01, hy = 0.5 * x.height + 0.01;
    const double dx = m.px0 - 0.5 * (x.width - 1), dy = m.py0 - 0.5 * (x.height - 1);
    const double X[3] = {m.a0x + dx * cE[0], m.a0y + dx * cE[1], m.a0z + dx * cE[2]};
    const double Y[3] = {m.a1x + dy * cE[0], m.a1y + dy * cE[1], m.a1z + dy * cE[2]};
    const double cn = sqrt(cE[0] * cE[0] + cE[1] * cE[1] + cE[2] * cE[2]);
    const double sx = 1.0 / (sqrt(X[0] * X[0] + X[1] * X[1] + X[2] * X[2]) + hx * cn);
    const double sy = 1.0 / (sqrt(Y[0] * Y[0] + Y[1] * Y[1] + Y[2] * Y[2]) + hy * cn);
    // (numbers beyond FP32's range: zeros, which no position fails)
    const double o1 = fabs(x.obs_xyz_au[0]) + fabs(x.obs_xyz_au[1]) + fabs(x.obs_xyz_au[2]);
    const bool fits = o1 < 1e15 && sx > 0.0 && sy > 0.0 && sx < 1e300 && sy < 1e300;
    for (int k = 0; k < 3; ++k) {
      m.fX[k] = fits ? (float)(sx * X[k]) : 0.f;
      m.fY[k] = fits ? (float)(sy * Y[k]) : 0.f;
      m.fZ[k] = fits ? (float)cE[k] : 0.f;
      m.fo[k] = fits ? (float)x.obs_xyz_au[k] : 0.f;
    }
    m.kx = fits ? (float)(sx * hx) : 0.f;
    m.ky = fits ? (float)(sy * hy) : 0.f;
  }
  out[i] = m;
  if (i == n - 1) out[n] = m;  // the repeated last record
}

hipError_t launch_exposure_prep(const dt_exposure* d_in, const int64_t* d_plane_off, const int32_t* d_src,
                                const int32_t* d_R, int n, ExpMeta* d_out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_exposure_prep, dim3((n + 63) / 64), dim3(64), 0, s, d_in, d_plane_off, d_src, d_R, n,
                     d_out);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------
// Matched-filter planes.  One wavefront per strip of up to prep_width(R) output
// columns and up to a few hundred output rows; wavefronts share nothing, so
// there is no barrier.  It streams the input rows y0 - R .. y0 + ny + R - 1:
// each lane holds two adjacent columns (two groups of them up to R = 6, so
// 256 input columns per row), loads them with one access per image and
// group, PREP_DEPTH rows ahead, turns them into {D w, w} with w = 1/V (0
// where the pixel is masked or off the image) in an LDS row, filters along x
// for its output columns (16-byte LDS reads, two pixels each) and pushes the
// result into a chain of 2R+1 partial sums per column: partial sum j of an
// output row becomes partial sum j + 1 with the next input row's term, so the
// filter along y is one fused multiply-add per tap and no register is moved.
// Sums run in the order of the taps, as the definition's.
//
// HBM bounds it: 57 vector instructions per pixel at R = 4 (120 with one
// column per thread, of them 18 moves of the row window and 12 of rows in
// flight, each of which waited for the newest row).  Images are read with
// ordinary loads: neighbouring strips share halo rows and the cache lines at
// their edges, which the non-temporal hint drops (100 FP32 2048^2 images at
// R = 4 1.49 ms with it, 1.42 without; 40 FP16 4096^2 1.84 and 1.69; 60 FP16
// 1000^2 at R = 1 0.170 and 0.116).  One column per thread: 1.45, 3.09 and
// 0.255 ms; 57 FP16 of 1031 x 773 0.29 -> 0.136.  A device copy reaches 4.8
// TB/s (6.7 GB of the first in 1.40 ms, 8.1 GB of the second in 1.68); where
// the buffers lie moves a time by up to 8 %.  Four rows in flight measured as
// six and three do.
// ----------------------------------------------------------------------------
// The image pointers come from a device array, so they are generic to the
// compiler; reading through global pointers keeps these loads off the LDS
// counter (a generic load is counted with the LDS operations, so the waits
// for a row's LDS reads would also wait for rows still in flight).
//
// Two adjacent pixels of a row, loaded together at the element's alignment
// (image rows of odd width start anywhere).  use(): the pair as it is
// filtered: `second` (all ones or zero per lane) puts the second pixel first,
// `kill[j]` of all ones makes pixel j a NaN.
template <typename T>
struct Pair;
template <>
struct Pair<float> {
  typedef uint32_t vec __attribute__((ext_vector_type(2), aligned(4)));
  vec v;
  __device__ __forceinline__ void load(const float* p, int c) {
    v = *(const __attribute__((address_space(1))) vec*)(global_ptr(p) + c);
  }
  // {pixel 0, pixel 1}
  __device__ __forceinline__ float2 use(bool second, uint32_t kill0, uint32_t kill1) const {
    return make_float2(__uint_as_float((second ? v[1] : v[0]) | kill0), __uint_as_float(v[1] | kill1));
  }
};
template <>
struct Pair<_Float16> {
  typedef uint32_t word __attribute__((aligned(2)));
  uint32_t v;
  __device__ __forceinline__ void load(const _Float16* p, int c) {
    v = *(const __attribute__((address_space(1))) word*)(global_ptr(p) + c);
  }
  __device__ __forceinline__ float2 use(bool second, uint32_t kill0, uint32_t kill1) const {
    const uint32_t u = (second ? v >> 16 : v) | (kill0 & 0xffffu) | (kill1 << 16);
    return make_float2((float)__builtin_bit_cast(_Float16, (uint16_t)(u & 0xffffu)),
                       (float)__builtin_bit_cast(_Float16, (uint16_t)(u >> 16)));
  }
};

// {D w, w}, w = 1/V; zeros unless D is finite and V finite and positive
// (selected, not branched: masked pixels are rare and scattered).
__device__ __forceinline__ float2 weight_pair(float d, float v) {
  constexpr int FINITE = 0x1f8, POSITIVE = 0x180;  // v_cmp_class: any finite value; positive normal or denormal
  const bool ok = __builtin_amdgcn_classf(d, FINITE) & __builtin_amdgcn_classf(v, POSITIVE);
  const float w = 1.0f / v;
  return make_float2(ok ? d * w : 0.f, ok ? w : 0.f);
}

// g a + s into a register of its own: the partial sums move one place per
// row, and the two-address form the compiler prefers copies each of them.
__device__ __forceinline__ float chain(float g, float a, float s) {
  float d;
  asm("v_fma_f32 %0, %1, %2, %3" : "=v"(d) : "s"(g), "v"(a), "v"(s));
  return d;
}

__device__ __forceinline__ unsigned xcd_tile(unsigned b, unsigned nb) {
  constexpr unsigned NX = 8;
  const unsigned q = nb / NX, r = nb % NX;
  const unsigned x = b % NX, l = b / NX;
  return x < r ? x * (q + 1) + l : r * (q + 1) + (x - r) * q + l;
}

__device__ __forceinline__ double lane_value(double v, int lane) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

typedef float plane4_t __attribute__((ext_vector_type(4)));
typedef uint32_t store4_t __attribute__((ext_vector_type(4)));
constexpr int STORE_NT = 2;  // buffer cache policy: non-temporal

template <typename T, int R, bool VAR>
__global__ __launch_bounds__(64) void k_prepass(const ExpMeta* __restrict__ meta, const PrepTile* __restrict__ tiles,
                                                const void* const* __restrict__ flux,
                                                const void* const* __restrict__ var, float2* __restrict__ planes) {
  constexpr int K = 2 * R + 1;
  constexpr int G = prep_groups(R);     // column pairs per lane
  constexpr int RA = prep_lead(R);      // input columns left of the first output column (even)
  constexpr int OFF = RA - R;           // first tap of output column c is input column c + OFF
  constexpr int NP = (OFF + K + 2) / 2; // pairs read for two output columns
  constexpr int DEPTH = PREP_DEPTH;     // input rows in flight per lane
  __shared__ float4 row[64 * G + NP];   // {D w, w} of two columns each
  // XCD-aware order: workgroups are dispatched round-robin over the 8 XCDs,
  // so give each XCD a contiguous run of tiles; neighbouring tiles (which
  // share halo rows and halo cache lines) then meet in the same L2
  const PrepTile tl = tiles[xcd_tile(blockIdx.x, gridDim.x)];
  const ExpMeta& m = meta[tl.e];
  const int W = m.W, H = m.H;  // W >= 2
  const int lane = threadIdx.x;
  // 1-D weights g and g^2 (lane j computes tap j; wave-uniform values); the
  // 2-D stamp is g(dx) g(dy) / Z with Z = (sum g)^2
  const double sig = (double)m.fwhm / (2.0 * sqrt(2.0 * log(2.0)));
  const double gd = (double)(min(lane, K - 1) - R);
  const double gl = exp(-gd * gd / (2.0 * sig * sig));
  float g1[K], g2[K];
  double zs = 0.0;
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const double g = lane_value(gl, j);
    zs += g;
    g1[j] = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint((float)g)));
    g2[j] = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint((float)(g * g))));
  }
  const double z = zs * zs;
  const float n1 = (float)(1.0 / z), n2 = (float)(1.0 / (z * z));
  const T* Dp = static_cast<const T*>(flux[m.src]);
  const T* Vp = VAR ? static_cast<const T*>(var[m.src]) : nullptr;
  const float vs = m.vs;
  // This lane's columns: group g holds c and c + 1.  The loop over rows has
  // no branch (one around a load or a store makes the waits cover all loads
  // in flight): every lane loads a pair inside the row on every row; rows and
  // columns off the image read the nearest ones and are masked.  x0 and RA
  // are even, so only the right edge cuts a pair; its one column is the
  // second one loaded.
  int cs[G];
  bool cut[G];
  uint32_t kill0[G], kill1[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const int c = tl.x0 - RA + 128 * g + 2 * lane;
    cs[g] = min(max(c, 0), W - 2);
    cut[g] = c == W - 1;
    kill0[g] = c >= 0 && c < W ? 0u : ~0u;
    kill1[g] = c >= 0 && c + 1 < W ? 0u : ~0u;
  }
  const int rows = tl.ny + 2 * R;
  Pair<T> D[DEPTH][G], V[DEPTH][G];
  auto fetch = [&](int r, Pair<T>* d, Pair<T>* v) {
    const int64_t base = (int64_t)min(max(tl.y0 - R + r, 0), H - 1) * W;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      d[g].load(Dp + base, cs[g]);
      if (VAR) v[g].load(Vp + base, cs[g]);
    }
  };
#pragma unroll
  for (int q = 0; q < DEPTH; ++q) {
    fetch(q, D[q], V[q]);
    __builtin_amdgcn_sched_barrier(0);  // in the order of their use, as in the loop
  }
  // partial sums of the output rows the last K input rows belong to
  float sa[2 * G][K], sb[2 * G][K];
#pragma unroll
  for (int c = 0; c < 2 * G; ++c)
#pragma unroll
    for (int j = 0; j < K; ++j) sa[c][j] = sb[c][j] = 0.f;
  // Output rows are stored through a buffer whose range is the row's part in
  // this strip (nothing for the rows before the first one and past the last
  // one): the hardware drops the lanes past it.  The pair that an odd width
  // cuts is stored on its own.
  const int n_out = min(W - tl.x0, R <= PREP_EVEN_R ? m.strip : prep_width(R));
  const bool odd = (n_out & 1) != 0;
  float2* out = planes + m.plane_off + (int64_t)(tl.y0 - 2 * R) * W + tl.x0;
#pragma unroll 1
  for (int r0 = 0; r0 < rows; r0 += DEPTH) {
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) {  // row r sits in slot u: nothing moves
      const int r = r0 + u;
      const int gy = tl.y0 - R + r;
      const uint32_t off = gy >= 0 && gy < H ? 0u : ~0u;
      float a[2 * G], b[2 * G];
#pragma unroll
      for (int c = 0; c < 2 * G; ++c) a[c] = b[c] = 0.f;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float2 d = D[u][g].use(cut[g], kill0[g] | off, kill1[g] | off);
        const float2 v = VAR ? V[u][g].use(cut[g], 0u, 0u) : make_float2(vs, vs);
        const float2 p0 = weight_pair(d.x, v.x), p1 = weight_pair(d.y, v.y);
        row[64 * g + lane] = make_float4(p0.x, p0.y, p1.x, p1.y);
      }
      // The loads into slot u are issued after its last use, into the same
      // registers: moved above it they would need others, and a copy of
      // values in flight, which waits for them, at the end of the loop.
      __builtin_amdgcn_sched_barrier(0);
      fetch(r + DEPTH, D[u], V[u]);
      __builtin_amdgcn_sched_barrier(0);
      // LDS operations of one wavefront complete in order: only the compiler
      // has to keep the reads between this row's writes and the next one's
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
      for (int g = 0; g < G; ++g) {
#pragma unroll
        for (int q = 0; q < NP; ++q) {
          const float4 v = row[64 * g + lane + q];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int i = 2 * q + h - OFF;  // tap of the first of the two output columns
            const float x = h ? v.z : v.x, w = h ? v.w : v.y;
            if (i >= 0 && i < K) {
              a[2 * g] = fmaf(g1[i], x, a[2 * g]);
              b[2 * g] = fmaf(g2[i], w, b[2 * g]);
            }
            if (i >= 1 && i - 1 < K) {
              a[2 * g + 1] = fmaf(g1[i - 1], x, a[2 * g + 1]);
              b[2 * g + 1] = fmaf(g2[i - 1], w, b[2 * g + 1]);
            }
          }
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
      for (int c = 0; c < 2 * G; ++c) {
#pragma unroll
        for (int j = K - 1; j > 0; --j) {
          sa[c][j] = chain(g1[j], a[c], sa[c][j - 1]);
          sb[c][j] = chain(g2[j], b[c], sb[c][j - 1]);
        }
        sa[c][0] = chain(g1[0], a[c], 0.f);
        sb[c][0] = chain(g2[0], b[c], 0.f);
      }
      const bool keep = r >= 2 * R && r < rows;
      float2* q = keep ? out + (int64_t)r * W : planes;
      const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(q, (short)0, keep ? 8 * (n_out & ~1) : 0, 0x00020000);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const plane4_t v = {sa[2 * g][K - 1] * n1, sb[2 * g][K - 1] * n2, sa[2 * g + 1][K - 1] * n1,
                            sb[2 * g + 1][K - 1] * n2};
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(store4_t, v), rsrc, 8 * (128 * g + 2 * lane), 0,
                                               STORE_NT);
        if (odd && keep && 128 * g + 2 * lane == n_out - 1) q[n_out - 1] = make_float2(v[0], v[1]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// Images one column wide: one thread per output row.
template <typename T>
__global__ __launch_bounds__(256) void k_prepass_column(const ExpMeta* __restrict__ meta,
                                                        const PrepTile* __restrict__ tiles,
                                                        const void* const* __restrict__ flux,
                                                        const void* const* __restrict__ var,
                                                        float2* __restrict__ planes) {
  const PrepTile tl = tiles[blockIdx.x];
  const ExpMeta& m = meta[tl.e];
  const T* Dp = static_cast<const T*>(flux[m.src]);
  const T* Vp = static_cast<const T*>(var[m.src]);
  const double sig = (double)m.fwhm / (2.0 * sqrt(2.0 * log(2.0)));
  auto tap = [&](int j) { return exp(-(double)(j * j) / (2.0 * sig * sig)); };
  double zs = 0.0;
  for (int j = -m.R; j <= m.R; ++j) zs += tap(j);
  const double z = zs * zs;
  for (int64_t y = (int64_t)tl.y0 + threadIdx.x; y < (int64_t)tl.y0 + tl.ny; y += 256) {  // (past 2^31 in the tallest)
    float a = 0.f, b = 0.f;
    for (int j = -m.R; j <= m.R; ++j) {
      if (y + j < 0 || y + j >= m.H) continue;
      const float2 p = weight_pair((float)Dp[y + j], Vp ? (float)Vp[y + j] : m.vs);
      const double g = tap(j);  // (the tap across the column, 0, is 1)
      a = fmaf((float)g, p.x, a);
      b = fmaf((float)(g * g), p.y, b);
    }
    planes[m.plane_off + y] = make_float2(a * (float)(1.0 / z), b * (float)(1.0 / (z * z)));
  }
}

template <typename T, bool VAR>
static hipError_t launch_prepass_t(int R, const ExpMeta* d_meta, const PrepTile* d_tiles, unsigned g,
                                   const void* const* d_flux, const void* const* d_var, float2* d_planes,
                                   hipStream_t s) {
  switch (R) {
    case 0:
      hipLaunchKernelGGL((k_prepass_column<T>), dim3(g), dim3(256), 0, s, d_meta, d_tiles, d_flux, d_var, d_planes);
      break;
#define DT_CASE(RR)                                                                                        \
  case RR:                                                                                                 \
    hipLaunchKernelGGL((k_prepass<T, RR, VAR>), dim3(g), dim3(64), 0, s, d_meta, d_tiles, d_flux, d_var,   \
                       d_planes);                                                                          \
    break;
    DT_CASE(1) DT_CASE(2) DT_CASE(3) DT_CASE(4) DT_CASE(5) DT_CASE(6)
    DT_CASE(7) DT_CASE(8) DT_CASE(9) DT_CASE(10) DT_CASE(11)
#undef DT_CASE
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_prepass(const ExpMeta* d_meta, const PrepTile* d_tiles, const int64_t* group_off,
                          const int32_t* group_R, int n_groups, const void* const* d_flux,
                          const void* const* d_var, bool has_var, dt_dtype dtype, float2* d_planes, hipStream_t s) {
  for (int gi = 0; gi < n_groups; ++gi) {
    const int64_t beg = group_off[gi], end = group_off[gi + 1];
    for (int64_t off = beg; off < end; off += 0x7fffffff) {
      const unsigned g = (unsigned)std::min<int64_t>(end - off, 0x7fffffff);
      const auto launch = dtype == DT_F32 ? (has_var ? launch_prepass_t<float, true> : launch_prepass_t<float, false>)
                                          : (has_var ? launch_prepass_t<_Float16, true>
                                                     : launch_prepass_t<_Float16, false>);
      const hipError_t e = launch(group_R[gi], d_meta, d_tiles + off, g, d_flux, d_var, d_planes, s);
      if (e != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

}  // namespace dtk
