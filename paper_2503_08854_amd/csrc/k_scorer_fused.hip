// k_scorer_fused.hip -- inference forward of the cell scorer in one kernel.
//
// The same network, rounding points and K order as the training path (every
// activation rounded to BF16 after bias and ReLU, FP32 accumulation in steps
// of 32, conv1's nine taps in one of 16), the 1152-deep layer in two halves
// that are then added, with every intermediate kept in LDS.
//
// A workgroup of twelve waves (three per SIMD; the LDS holds one workgroup per
// CU) takes 16 cells at a time and makes them the columns of every product,
// the weights being the rows: pixel arithmetic is uniform across the wave, an
// operand is a contiguous read of 16 or 32 channels of a pixel of every cell,
// and a lane's four results are four channels of one cell, one 8-byte write.
// The weights of the convolutions stay in registers: both channel tiles of
// conv2, so that one LDS read feeds two products, and one of conv3's.  The
// convolutions run as a pipeline with one barrier per conv2 row: in step t the
// waves compute row t of conv2, rows 2t + 2 and 2t + 3 of conv1 for the next
// step and, every other step, a row of conv3 from finished conv2 rows, over
// ring buffers of five and four rows.  Per cell only the 441 + 16 BF16 inputs
// are read and one FP32 logit is written.
//
// 10 000 cells in 52.8 us (a group in 16 us, three rounds of 256; 4 us of
// start: weights and stamps from memory).  It is bound by the issue of the
// vector instructions around the products (40 % of the cycles) and by LDS
// (41 %), with the matrix cores busy for 24 %.  Before, 165 us: products of
// K = 16 with cells as the rows (four 2-byte writes per tile), weights read
// from LDS for each product, sixteen 2-byte reads for conv1's taps of four
// pixels, three barriers per row.  On the way: 64-byte steps between cells in
// an operand and unaligned stamp reads cost 12.5 M of 32.5 M CU cycles in bank
// conflicts (65 us); the three parts of a step in another order in each wave
// of a SIMD, 77 us; weights of the 1152-deep layer read ahead during the
// convolutions, more registers than there are (spills, 97 us).
#include "dt_common.hpp"

namespace dtk {

namespace {
typedef short s4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef float f2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf2_t __attribute__((ext_vector_type(2)));

// two values to BF16 in one hardware conversion (round to nearest even)
__device__ __forceinline__ uint32_t cvt2(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2_t{a, b}, bf2_t));
}
__device__ __forceinline__ bf8_t ld8(const uint16_t* p) { return *reinterpret_cast<const bf8_t*>(p); }
__device__ __forceinline__ f4_t ld4f(const float* p) { return *reinterpret_cast<const f4_t*>(p); }
__device__ __forceinline__ f4_t mfma(bf8_t a, bf8_t b, f4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// bias, ReLU and rounding of four channels, stored at o
__device__ __forceinline__ uint2 act4(f4_t d, f4_t b) {
  return make_uint2(cvt2(fmaxf(d[0] + b[0], 0.f), fmaxf(d[1] + b[1], 0.f)),
                    cvt2(fmaxf(d[2] + b[2], 0.f), fmaxf(d[3] + b[3], 0.f)));
}
__device__ __forceinline__ void put4(uint16_t* o, f4_t d, f4_t b) { *reinterpret_cast<uint2*>(o) = act4(d, b); }
__device__ __forceinline__ bf8_t keep8(bf8_t v, bool keep) {
  uint4 u = __builtin_bit_cast(uint4, v);
  u.x = keep ? u.x : 0u;
  u.y = keep ? u.y : 0u;
  u.z = keep ? u.z : 0u;
  u.w = keep ? u.w : 0u;
  return __builtin_bit_cast(bf8_t, u);
}

constexpr int G = 16;            // cells at a time
constexpr int NW = 12;           // waves
constexpr int NTH = 64 * NW;
constexpr int SROW = 24, SCELL = 23 * SROW + 2;  // a cell's stamp with a one-pixel zero border; odd in words
constexpr int PX1 = G * 16, PX2 = G * 32;    // a pixel's channels of all cells
constexpr int R1 = 5, R2 = 4;    // rows of the rings
constexpr int C1 = 22, C2 = 12;  // their columns, the first one zero (the last row is followed by one more)
constexpr int BB2 = 16, BB3 = 48, BB4 = 80, BB5 = 144, BB6 = 208, BB7 = 272, BIAS = 276;
constexpr f4_t ZERO4 = {0.f, 0.f, 0.f, 0.f};
constexpr bf8_t ZERO8 = {};

struct __align__(16) GroupLds {
  uint16_t stg[G * SCELL + 8];           // stamps [cell][bordered row][24]
  // activations [pixel][channel / 8][cell][8]: the lanes of an operand read one contiguous piece
  uint16_t h1r[(R1 * C1 + 1) * PX1];     // conv1 rows [row][x + 1]
  uint16_t h2r[(R2 * C2 + 1) * PX2];     // conv2 rows [row][x + 1]
  uint16_t h3s[36 * PX2];                // conv3 output
  uint16_t ftg[G * 16];
  float bias[BIAS];                      // layer after layer
  int64_t srow[2][G];                    // this and the next group's rows of the inputs and logits
};
static_assert(sizeof(GroupLds) <= 160 * 1024, "LDS of a CU");
}  // namespace

template <bool ROWS>
__global__ __launch_bounds__(NTH) void k_scorer_fused(ScorerFusedArgs A) {
  __shared__ GroupLds L;
  uint16_t* const stg = L.stg;
  uint16_t* const h1r = L.h1r;
  uint16_t* const h2r = L.h2r;
  uint16_t* const h3s = L.h3s;
  uint16_t* const ftg = L.ftg;
  float* const bias = L.bias;
  int64_t(*const srow)[G] = L.srow;
  // the fully connected layers work where conv1's first two ring rows are (the zero columns are left alone)
  uint16_t* const cat = h1r + PX1;
  uint16_t* const h6 = cat + G * 128;
  f4_t* const red = reinterpret_cast<f4_t*>(h1r + (C1 + 1) * PX1);  // partial sums handed on: [2][output tile][lane]
  static_assert(G * (128 + 64) <= 21 * PX1 && 2 * 4 * 64 * 8 <= 21 * PX1, "room in a ring row");
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = (int)__builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kq = lane >> 4;
  const uint16_t* wf = A.wf + 8 * lane;
  const int put = ((kq >> 1) * 16 + r16) * 8 + 4 * (kq & 1);  // a lane's four results: channels 4 kq .. of cell r16
  const int n_groups = (A.B + G - 1) / G;
  // a group's stamps: thread px reads its pixel of every cell, before the last layers of the group before
  const int px = min(tid, 440);
  uint32_t next[G / 2];
  auto load_stamps = [&](int grp, const int64_t* rows) {
    if (tid >= 448) return;
#pragma unroll
    for (int c = 0; c < G; ++c) {
      const uint32_t v = A.stamps[(ROWS ? rows[c] : (int64_t)min(grp * G + c, A.B - 1)) * 441 + px];
      next[c / 2] = c & 1 ? next[c / 2] | (v << 16) : v;
    }
  };
  auto load_rows = [&](int grp, int64_t* rows) {
    if (tid < G) rows[tid] = A.rows[min(grp * G + tid, A.B - 1)];
  };
  if (ROWS) {
    load_rows(blockIdx.x, srow[0]);
    __syncthreads();
  }
  load_stamps(blockIdx.x, srow[0]);
  // convolution weights: one copy to LDS (the conv3 output's place), from there to every wave's registers
  for (int i = tid; i < SCORER_F4 / 8; i += NTH)
    reinterpret_cast<uint4*>(h3s)[i] = reinterpret_cast<const uint4*>(A.wf)[i];
  static_assert(SCORER_F4 <= 36 * PX2, "room for the convolutions' weights");
  for (int i = tid; i <= BB7; i += NTH) {
    const int l = (i >= BB2) + (i >= BB3) + (i >= BB4) + (i >= BB5) + (i >= BB6) + (i >= BB7);
    const int first = l == 0 ? 0 : l == 1 ? BB2 : l == 2 ? BB3 : l == 3 ? BB4 : l == 4 ? BB5 : l == 5 ? BB6 : BB7;
    bias[i] = A.w[A.b_off[l] + i - first];
  }
  // the zero borders, never written below: the stamps' and the columns left and right of the ring rows
  for (int i = tid; i < (G * SCELL + 8) / 8; i += NTH) reinterpret_cast<uint4*>(stg)[i] = make_uint4(0, 0, 0, 0);
  for (int i = tid; i < (R1 + 1) * PX1 / 8; i += NTH)
    reinterpret_cast<uint4*>(h1r + (i / (PX1 / 8)) * C1 * PX1)[i % (PX1 / 8)] = make_uint4(0, 0, 0, 0);
  for (int i = tid; i < (R2 + 1) * PX2 / 8; i += NTH)
    reinterpret_cast<uint4*>(h2r + (i / (PX2 / 8)) * C2 * PX2)[i % (PX2 / 8)] = make_uint4(0, 0, 0, 0);
  __syncthreads();
  const int n3 = w & 1;
  bf8_t a2[2][5], a3[9];
#pragma unroll
  for (int n = 0; n < 2; ++n)
#pragma unroll
    for (int s = 0; s < 5; ++s) a2[n][s] = ld8(h3s + 8 * lane + SCORER_F2 + (5 * n + s) * 512);
#pragma unroll
  for (int s = 0; s < 9; ++s) a3[s] = ld8(h3s + 8 * lane + SCORER_F3 + (9 * n3 + s) * 512);
  // conv1 takes K = 16: lanes kq = 0 hold taps 0 1 2 5, kq = 1 taps 6 7 3 4, kq = 2 tap 8 (the products of eight K
  // are summed together, so the order within them is free).  A lane reads runs of neighbouring pixels z, x, y in
  // aligned words and forms the pairs of taps of output pixel j by a byte selector that also writes the zeros:
  //   kq = 0: z = row 0 (taps 0, 1)   x, y = rows 0 and 1, two pixels on (taps 2, 5)
  //   kq = 1: z = row 2 (taps 6, 7)   x, y = row 1 and the same two pixels on (taps 3, 4)
  //   kq = 2: z = row 2, two pixels on (tap 8)
  s4_t a1;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int k = kq == 0 ? (i < 3 ? i : 5) : kq == 1 ? (i < 2 ? 6 + i : 1 + i) : 8 + i + 4 * (kq - 2);
    a1[i] = (short)h3s[SCORER_F1 + ((k >> 3) * 16 + r16) * 8 + (k & 7)];
  }
  const int oz = r16 * SCELL + (kq == 0 ? 0 : 2 * SROW) + (kq >= 2 ? 2 : 0);
  const int ox = r16 * SCELL + (kq == 1 ? SROW : 2), oy = r16 * SCELL + SROW + 2;
  const uint32_t ze = kq < 2 ? 0x03020100u : kq == 2 ? 0x0c0c0100u : 0x0c0c0c0cu,
                 zo = kq < 2 ? 0x05040302u : kq == 2 ? 0x0c0c0302u : 0x0c0c0c0cu,
                 qe = kq == 0 ? 0x05040100u : kq == 1 ? 0x03020100u : 0x0c0c0c0cu,
                 qo = kq == 0 ? 0x07060302u : kq == 1 ? 0x05040302u : 0x0c0c0c0cu;
  const int x1 = 4 * (w % 6);  // of row y or y + 1; the sixth share of a row is its last pixel
  auto conv1 = [&](int y) {
    y += w >= 6;
    uint16_t* o = h1r + ((unsigned)y % R1 * C1 + 1 + x1) * PX1 + put;
    uint2 v[4];
    if (y > 20) {  // the row below the image
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = make_uint2(0, 0);
    } else {
      const uint16_t* p = stg + y * SROW + x1;  // output pixel (y, x) reads bordered pixels (y + dy, x + dx)
      const uint32_t* z = reinterpret_cast<const uint32_t*>(p + oz);
      const uint32_t* x = reinterpret_cast<const uint32_t*>(p + ox);
      const uint32_t* q = reinterpret_cast<const uint32_t*>(p + oy);
      const f4_t bs = ld4f(bias + 4 * kq);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = j / 2;
        const uint2 b = j & 1 ? make_uint2(__builtin_amdgcn_perm(z[i + 1], z[i], zo), __builtin_amdgcn_perm(q[i], x[i], qo))
                              : make_uint2(__builtin_amdgcn_perm(z[i], z[i], ze), __builtin_amdgcn_perm(q[i], x[i], qe));
        v[j] = act4(__builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a1, __builtin_bit_cast(s4_t, b), ZERO4, 0, 0, 0), bs);
      }
    }
    *reinterpret_cast<uint2*>(o) = v[0];
    if (x1 < 20) {
#pragma unroll
      for (int j = 1; j < 4; ++j) *reinterpret_cast<uint2*>(o + j * PX1) = v[j];
    }
  };
  // conv2 row t, pixel w: two taps per K step, the second one's by the lanes kq >= 2
  const int c2 = 8 * (lane & 31), c2n = 8 * lane;  // the next pixel for the second tap
  const bool second = kq >= 2;
  auto conv2 = [&](int t) {
    const int o0 = ((unsigned)(2 * t - 1 + R1) % R1 * C1 + 2 * w) * PX1;
    const int o1 = ((unsigned)(2 * t) % R1 * C1 + 2 * w) * PX1, o2 = ((unsigned)(2 * t + 1) % R1 * C1 + 2 * w) * PX1;
    bf8_t b[5];
    b[0] = ld8(h1r + o0 + c2n);                                     // (0, 0) (0, 1)
    b[1] = ld8(h1r + (second ? o1 + c2 : o0 + 2 * PX1 + c2));       // (0, 2) (1, 0)
    b[2] = ld8(h1r + o1 + PX1 + c2n);                               // (1, 1) (1, 2)
    b[3] = ld8(h1r + o2 + c2n);                                     // (2, 0) (2, 1)
    b[4] = ld8(h1r + (second ? c2 : o2 + 2 * PX1 + c2));            // (2, 2), zero
    f4_t acc[2] = {ZERO4, ZERO4};
#pragma unroll
    for (int s = 0; s < 5; ++s)
#pragma unroll
      for (int n = 0; n < 2; ++n) acc[n] = mfma(a2[n][s], b[s], acc[n]);
    uint16_t* o = h2r + ((t % R2) * C2 + 1 + w) * PX2 + put;
#pragma unroll
    for (int n = 0; n < 2; ++n) put4(o + 256 * n, acc[n], ld4f(bias + BB2 + 16 * n + 4 * kq));
  };
  // conv3 row q, pixel w / 2: one tap per K step; below: its row 2q + 1 is in the image
  auto conv3 = [&](int q, bool below) {
    f4_t acc = ZERO4;
#pragma unroll
    for (int y = 0; y < 3; ++y) {
      const uint16_t* p = h2r + ((unsigned)(2 * q + y - 1 + R2) % R2 * C2 + 2 * (w >> 1)) * PX2 + 8 * lane;
#pragma unroll
      for (int x = 0; x < 3; ++x) acc = mfma(a3[3 * y + x], y == 2 && !below ? ZERO8 : ld8(p + x * PX2), acc);
    }
    put4(h3s + (q * 6 + (w >> 1)) * PX2 + 256 * n3 + put, acc, ld4f(bias + BB3 + 16 * n3 + 4 * kq));
  };

  // FC4 (1152 -> 64; K step = conv3 pixel): output tile w & 3 in two sums over steps 0 .. 17 and 18 .. 35.  Wave n
  // takes steps 0 .. 11 of its tile, wave n + 4 the rest of the first sum and 18 .. 23, wave n + 8 the last twelve
  const int n4 = w & 3, part = w >> 2;
  int buf = 0;
  for (int grp = blockIdx.x; grp < n_groups; grp += gridDim.x, buf ^= 1) {
    // read again for every group: hoisted out of this loop, the weights of the fully connected layers would
    // not fit the registers
    int again = 0;
    asm volatile("" : "+s"(again));
    const uint16_t* wg = wf + again;
    __syncthreads();  // the previous group's readers of stg / h3s / cat / h6 / srow are done
    const int cell0 = grp * G;
    if (tid < 441) {
      uint16_t* o = stg + (px / 21 + 1) * SROW + px % 21 + 1;
#pragma unroll
      for (int c = 0; c < G; ++c) o[c * SCELL] = (uint16_t)(c & 1 ? next[c / 2] >> 16 : next[c / 2]);
    } else if (tid >= 512) {
      const int r = (tid - 512) / 16, c = tid % 16;
      ftg[((c >> 3) * G + r) * 8 + (c & 7)] = A.feats[(ROWS ? srow[buf][r] : (int64_t)min(cell0 + r, A.B - 1)) * 16 + c];
    }
    // the rows above the images: the last slots of the rings
    if (tid < 21 * PX1 / 8)
      reinterpret_cast<uint4*>(h1r + ((R1 - 1) * C1 + 1) * PX1)[tid] = make_uint4(0, 0, 0, 0);
    if (tid < 11 * PX2 / 8)
      reinterpret_cast<uint4*>(h2r + ((R2 - 1) * C2 + 1) * PX2)[tid] = make_uint4(0, 0, 0, 0);
    if (ROWS && grp + (int)gridDim.x < n_groups) load_rows(grp + gridDim.x, srow[buf ^ 1]);
    __syncthreads();
    conv1(0);
    __syncthreads();
#pragma unroll 1
    for (int t = 0; t < 11; ++t) {
      if (t < 10) conv1(2 * t + 2);
      if (w < 11) conv2(t);
      if (t >= 2 && !(t & 1)) conv3(t / 2 - 1, true);
      __syncthreads();
    }
    conv3(5, false);
    if (grp + (int)gridDim.x < n_groups) load_stamps(grp + gridDim.x, srow[buf ^ 1]);
    __syncthreads();
    f4_t acc4 = ZERO4;
    const uint16_t* h = h3s + 8 * lane;
    const uint16_t* p4 = wg + SCORER_F4 + n4 * 36 * 512;
    auto steps4 = [&](int s) {  // six K steps from s on
      bf8_t a4[6];
#pragma unroll
      for (int i = 0; i < 6; ++i) a4[i] = ld8(p4 + (s + i) * 512);
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        acc4 = mfma(a4[i], ld8(h + (s + i) * PX2), acc4);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    if (part < 2) {
      steps4(18 * part);
      if (part == 0) steps4(6);
      red[(part * 4 + n4) * 64 + lane] = acc4;
    } else {  // FC5 (16 -> 64)
      const f4_t d = mfma(ld8(wg + SCORER_F5 + n4 * 512), keep8(ld8(ftg + 8 * (lane & 31)), kq < 2), ZERO4);
      put4(cat + 256 * (4 + n4) + put, d, ld4f(bias + BB5 + 16 * n4 + 4 * kq));
    }
    __syncthreads();
    if (part == 1) {
      acc4 = red[n4 * 64 + lane];
      steps4(12);
      red[n4 * 64 + lane] = acc4;
    } else if (part == 2) {
      acc4 = red[(4 + n4) * 64 + lane];
      steps4(24);
      steps4(30);
    }
    bf8_t a6[4], a7[2];
#pragma unroll
    for (int s = 0; s < 4; ++s) a6[s] = ld8(wg + SCORER_F6 + (n4 * 4 + s) * 512);
#pragma unroll
    for (int s = 0; s < 2; ++s) a7[s] = ld8(wg + SCORER_F7 + s * 512);
    __syncthreads();
    if (part == 2)
      put4(cat + 256 * n4 + put, red[n4 * 64 + lane] + acc4, ld4f(bias + BB4 + 16 * n4 + 4 * kq));
    __syncthreads();
    if (w < 4) {  // FC6 (128 -> 64)
      f4_t acc = ZERO4;
#pragma unroll
      for (int s = 0; s < 4; ++s) acc = mfma(a6[s], ld8(cat + 512 * s + 8 * lane), acc);
      put4(h6 + 256 * w + put, acc, ld4f(bias + BB6 + 16 * w + 4 * kq));
    }
    __syncthreads();
    if (w == 0) {  // FC7 (64 -> 1), no ReLU: row 0 of a 16-high tile
      f4_t acc = ZERO4;
#pragma unroll
      for (int s = 0; s < 2; ++s) acc = mfma(a7[s], ld8(h6 + 512 * s + 8 * lane), acc);
      const int cell = cell0 + lane;
      if (lane < G && cell < A.B) A.z[ROWS ? srow[buf][lane] : (int64_t)cell] = acc[0] + bias[BB7];
    }
  }
}

hipError_t launch_scorer_fused(const ScorerFusedArgs& a, hipStream_t s) {
  if (a.B <= 0) return hipSuccess;
  int dev = 0, n_cu = 256;
  if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
  const int groups = (a.B + G - 1) / G;
  const int grid = groups < n_cu ? groups : n_cu;
  if (a.rows)
    hipLaunchKernelGGL(k_scorer_fused<true>, dim3((unsigned)grid), dim3(NTH), 0, s, a);
  else
    hipLaunchKernelGGL(k_scorer_fused<false>, dim3((unsigned)grid), dim3(NTH), 0, s, a);
  return hipGetLastError();
}

}  // namespace dtk
