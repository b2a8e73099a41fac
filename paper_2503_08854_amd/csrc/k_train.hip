// k_train.hip -- the cell scorer's forward pass, loss and gradients.
//
// k_train_cells: a workgroup of sixteen wavefronts takes two cells at a time
// through the whole network and back, with every activation and every delta
// of both in LDS: three convolutions, four fully connected layers, the loss,
// the deltas down to the first convolution, and the convolutions' weight
// gradients, which stay in registers over the cells of the workgroup.  What
// leaves it is one record of gradient sums per workgroup and, per cell, the
// inputs and deltas of the fully connected layers (3 KB), whose weight
// gradients contract over the batch; k_train_sum forms those, adds the
// records, and writes the gradient or applies Adam.
//
// Every product is v_mfma_f32_16x16x32_bf16 with the weights as the A operand
// (rows = channels) and pixels, or the cells, as the columns, so a lane's
// four results are four channels of one pixel: one 8-byte write.  A column
// holds one pixel's K values in (tap, channel) order, eight per lane, read as
// one 16-byte word from bordered [pixel][channel] images; the weight
// gradients, whose K is the pixels, read the same images transposed
// (ds_read_b64_tr_b16).  The weights are kept in the order in which the lanes
// of a product hold them, so a wavefront reads 1 KB in one piece.  The K
// order, the rounding of every activation and delta to BF16 and the order of
// the taps in a delta are those of the layer definitions (K in steps of 32,
// the 1152-deep layer in `splits` partial sums).
//
// Loss and gradient of a batch, where one kernel per operation (im2col, GEMM,
// mask, column sum, split-K sum, ...) took 45 launches and column and delta
// buffers in memory: 512 cells 1297 -> 33.6 us, one cell 246 -> 25 us, 32 768
// cells 66.5 -> 1.46 ms; logits of 512 cells 258 -> 9.7 us.
#include "dt_common.hpp"

namespace dtk {

namespace {
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf2_t __attribute__((ext_vector_type(2)));
typedef float f2_t __attribute__((ext_vector_type(2)));
typedef uint16_t u8_t __attribute__((ext_vector_type(8)));
typedef short s4_t __attribute__((ext_vector_type(4)));

constexpr int NW = 16;           // wavefronts
constexpr int NT = 64 * NW;
constexpr int NS = 2;            // cells at a time
constexpr int S1 = 24, S2 = 40;  // strides (BF16) of a pixel in the images: 16-byte reads, few bank conflicts
constexpr int FC4_STEPS = 36;
// parameter vector (the scorer's layer table)
constexpr int W1 = 0, B1 = 144, W2 = 160, B2 = 4768, W3 = 4800, B3 = 14016, W4 = 14048, B4 = 87776, W5 = 87840,
              B5 = 88864, W6 = 88928, B6 = 97120, W7 = 97184, B7 = 97248, NP = 97249;
// fragments of the BF16 weights
constexpr int FRAG = SCORER_FRAG;
constexpr int F1 = SCORER_F1, F2 = SCORER_F2, F3 = SCORER_F3, F4 = SCORER_F4, F5 = SCORER_F5, F6 = SCORER_F6,
              F7 = SCORER_F7, G2 = SCORER_G2, G3 = SCORER_G3, G4 = SCORER_G4, G6 = SCORER_G6;
// a workgroup's record: the convolutions' parameters as in the vector, the biases B4 B5 B6, layer 7 and the loss
constexpr int R4 = W4, R5 = R4 + 64, R6 = R5 + 64, R7 = R6 + 64, RL = R7 + 65, RN = RL + 1;
static_assert(RN <= TRAIN_RECORD, "record size");

__device__ __forceinline__ float bf2f(uint32_t h) { return __uint_as_float(h << 16); }
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ uint2 pack4(f4_t v) {
  uint2 r;
  r.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2_t{v[0], v[1]}, bf2_t));
  r.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2_t{v[2], v[3]}, bf2_t));
  return r;
}
__device__ __forceinline__ bf8_t ld8(const uint16_t* p) { return *reinterpret_cast<const bf8_t*>(p); }
__device__ __forceinline__ uint2 ld4(const uint16_t* p) { return *reinterpret_cast<const uint2*>(p); }
__device__ __forceinline__ void st4(uint16_t* p, uint2 v) { *reinterpret_cast<uint2*>(p) = v; }
__device__ __forceinline__ f4_t mfma(bf8_t a, bf8_t b, f4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
constexpr f4_t ZERO4 = {0.f, 0.f, 0.f, 0.f};

// bias and ReLU of four channels
__device__ __forceinline__ f4_t act(f4_t v, f4_t b) {
  f4_t r;
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = fmaxf(v[i] + b[i], 0.f);
  return r;
}
__device__ __forceinline__ f4_t ld4f(const float* p) { return f4_t{p[0], p[1], p[2], p[3]}; }
// v where the four BF16 activations are positive, else 0
__device__ __forceinline__ f4_t mask4(f4_t v, uint2 h) {
  return f4_t{bf2f(h.x & 0xffffu) > 0.f ? v[0] : 0.f, bf2f(h.x >> 16) > 0.f ? v[1] : 0.f,
              bf2f(h.y & 0xffffu) > 0.f ? v[2] : 0.f, bf2f(h.y >> 16) > 0.f ? v[3] : 0.f};
}
// v where keep, else 0: reads stay unconditional (a read under a condition is a branch and a wait of its own)
__device__ __forceinline__ bf8_t keep8(bf8_t v, bool keep) {
  uint4 u = __builtin_bit_cast(uint4, v);
  u.x = keep ? u.x : 0u;
  u.y = keep ? u.y : 0u;
  u.z = keep ? u.z : 0u;
  u.w = keep ? u.w : 0u;
  return __builtin_bit_cast(bf8_t, u);
}
// the first n of eight values, zero from there on
__device__ __forceinline__ bf8_t first8(bf8_t v, int n) {
  uint4 u = __builtin_bit_cast(uint4, v);
  auto two = [&](uint32_t x, int i) { return n > i + 1 ? x : n > i ? x & 0xffffu : 0u; };
  u.x = two(u.x, 0);
  u.y = two(u.y, 2);
  u.z = two(u.z, 4);
  u.w = two(u.w, 6);
  return __builtin_bit_cast(bf8_t, u);
}
// eight values p[off[i]]
__device__ __forceinline__ bf8_t gather8(const uint16_t* p, u8_t off) {
  u8_t v;
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = p[off[i]];
  return __builtin_bit_cast(bf8_t, v);
}
// Operand whose K runs over pixels, from [pixel][channel] images: each
// sixteen lanes read four pixels x 16 channels twice, and each lane gets its
// channel of the eight pixels.  p0, p1: this lane's share, channels
// 4 (lane & 3) .. of pixel 8 kq + (r16 >> 2), and of the pixel four further on.
__device__ __forceinline__ bf8_t ld_tr(const uint16_t* p0, const uint16_t* p1) {
  typedef __attribute__((address_space(3))) s4_t lds4;
  union {
    s4_t h[2];
    bf8_t v;
  } u;
  u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4*)p0);
  u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4*)p1);
  return u.v;
}

// The input pixels of a stride-2, pad-1, 3x3 layer of odd side SIDE, by the
// parity of (y, x): an even coordinate is read by the middle tap only, an odd
// one by the outer two, all of them inside the output.  Units are tiles of 16
// pixels of one class, the classes of most taps first.
template <int SIDE>
struct DeltaTiles {
  static constexpr int E = (SIDE + 1) / 2, O = SIDE / 2;
  static constexpr int OO = (O * O + 15) / 16, EO = (E * O + 15) / 16, N = OO + 2 * EO + (E * E + 15) / 16;
};
// Delta at pixel (y, x) of a lane: its taps (ky, kx) in order, one product of
// K = the output channels each; d holds the output deltas [pixel][S2].
template <int SIDE, int PY, int PX>
__device__ __forceinline__ f4_t delta_taps(const bf8_t (&a)[9], const uint16_t* d, int q, int& y, int& x, bool& ok) {
  using D = DeltaTiles<SIDE>;
  constexpr int NX = PX ? D::O : D::E, N = NX * (PY ? D::O : D::E);
  ok = q < N;
  const int c = ok ? q : 0;
  y = 2 * (c / NX) + PY;
  x = 2 * (c % NX) + PX;
  f4_t v = ZERO4;
#pragma unroll
  for (int ky = 1 - PY; ky < 3; ky += 2)
#pragma unroll
    for (int kx = 1 - PX; kx < 3; kx += 2) {
      const int oy = (y + 1 - ky) >> 1, ox = (x + 1 - kx) >> 1;
      v += mfma(a[ky * 3 + kx], ld8(d + (oy * D::E + ox) * S2), ZERO4);
    }
  return v;
}
template <int SIDE>
__device__ __forceinline__ f4_t delta_unit(const bf8_t (&a)[9], const uint16_t* d, int u, int r16, int& y, int& x,
                                           bool& ok) {
  using D = DeltaTiles<SIDE>;
  if (u < D::OO) return delta_taps<SIDE, 1, 1>(a, d, 16 * u + r16, y, x, ok);
  u -= D::OO;
  if (u < D::EO) return delta_taps<SIDE, 0, 1>(a, d, 16 * u + r16, y, x, ok);
  u -= D::EO;
  if (u < D::EO) return delta_taps<SIDE, 1, 0>(a, d, 16 * u + r16, y, x, ok);
  u -= D::EO;
  return delta_taps<SIDE, 0, 0>(a, d, 16 * u + r16, y, x, ok);
}

// LDS of one cell.  The forward pass alone uses the part before d3.
struct __align__(16) CellLds {
  uint16_t st[23 * 23 + 7];   // the stamp, one-pixel zero border
  uint16_t h1[23 * 23 * S1];  // conv1 output, bordered
  uint16_t h2[13 * 13 * S2];  // conv2 output, bordered
  uint16_t h3[36 * 32];       // conv3 output [pixel][channel]
  uint16_t ft[16], cat[128], h6[64], d6[64], d4[64];
  float part[4][64];          // FC4 partial sums
  float dz, pad[3];
  float gb6[64], gw7[64], gbc[128], gb7, loss, pad2[2];  // gradient and loss sums over the workgroup's cells
};
struct __align__(16) CellBack {
  uint16_t d3[64 * S2];   // output deltas [pixel][channel]; pixels past the last are zero
  uint16_t d2[128 * S2];
  uint16_t d1[448 * 16];
};
static_assert(sizeof(CellLds) % 16 == 0 && sizeof(CellBack) % 16 == 0, "cleared in 16-byte words");
static_assert(NS * (sizeof(CellLds) + sizeof(CellBack)) + 1280 <= 160 * 1024, "LDS of a CU");
}  // namespace

// What bounds it: a pair of cells reads 400 KB of weights, most of them the
// 1152-deep layer's, forward and back (two spans of 10 000 cycles of the
// pair's 70 000, at about 14 bytes per cycle and CU from L2), and the rest is
// the latency of sixteen phases between barriers.  Two cells share each
// weight read: with one cell per workgroup of eight wavefronts, two
// workgroups per CU, 512 cells took 55 us instead of 30.5, with rows of
// [N][K] weights (64 bytes of a line per row) instead of fragments and the
// weight gradients' operands gathered by 2-byte reads.  Up to 256 cells the
// second slot stays empty: each cell has a CU of its own.
// BACK false: the logits only.
template <bool BACK>
__global__ __launch_bounds__(NT) void k_train_cells(TrainArgs A) {
  __shared__ CellLds C[NS];
  __shared__ CellBack Q[BACK ? NS : 1];
  // offsets of the pixels of each layer's output in its bordered input
  __shared__ __align__(16) uint16_t at1[BACK ? 448 : 8], at2[BACK ? 128 : 8], at3[BACK ? 64 : 8];
  const int tid = threadIdx.x;
  const int wave = (int)__builtin_amdgcn_readfirstlane(tid >> 6);
  // one stamp pixel per thread, the next cells' while these are worked on: threads 0.. and 512..
  const int sl = tid >> 9, px = tid & 511;
  auto pixel = [&](int cell) { return px < 441 && cell < A.B ? A.stamps[(int64_t)cell * 441 + px] : (uint16_t)0; };
  uint16_t next = pixel(blockIdx.x + sl * gridDim.x);
  for (int i = tid; i < NS * (int)sizeof(CellLds) / 16; i += NT)
    reinterpret_cast<uint4*>(C)[i] = make_uint4(0, 0, 0, 0);
  if (BACK) {
    for (int i = tid; i < NS * (int)sizeof(CellBack) / 16; i += NT)
      reinterpret_cast<uint4*>(Q)[i] = make_uint4(0, 0, 0, 0);
    if (tid < 448) at1[tid] = (uint16_t)(tid < 441 ? (tid / 21) * 23 + tid % 21 : 0);
    else if (tid < 576) {
      const int i = tid - 448;
      at2[i] = (uint16_t)(i < 121 ? ((i / 11) * 46 + (i % 11) * 2) * S1 : 0);
    } else if (tid < 640) {
      const int i = tid - 576;
      at3[i] = (uint16_t)(i < 36 ? ((i / 6) * 26 + (i % 6) * 2) * S2 : 0);
    }
  }
  // weight gradients: rows = (tap, input channel), columns = output channel.  Row tiles j = w + 16 i of
  // conv3 (j < 18), then of conv2 (one per tap)
  f4_t g[2][2], g1 = ZERO4, gb1 = ZERO4, gb2 = ZERO4, gb3 = ZERO4;
#pragma unroll
  for (int i = 0; i < 2; ++i) g[i][0] = g[i][1] = ZERO4;

  for (int cell0 = blockIdx.x; cell0 < A.B; cell0 += NS * gridDim.x) {
    // Values that the compiler cannot see through: the weights are read and their addresses computed again
    // for every pair of cells (hoisted out of this loop they would not fit the registers).  Each phase's
    // weights are read before the barrier that it waits for.
    int again = 0, w = wave, tid = threadIdx.x;
    asm volatile("" : "+s"(again), "+s"(w), "+v"(tid));
    const int lane = tid & 63, r16 = lane & 15, kq = lane >> 4, ct = w & 1;  // ct: channel tile of conv2, conv3
    const uint16_t* wf = A.wf + again + 8 * lane;  // fragments
    const float* par = A.w + again;
    const int ns = cell0 + (int)gridDim.x < A.B ? 2 : 1;  // cells of this pass: cell0 and cell0 + gridDim.x
    const int col = r16 & 1;                              // the cell in this lane's column (fully connected layers)
    const int64_t col_cell = cell0 + (int64_t)col * gridDim.x;
    __syncthreads();  // the previous cells' readers are done; the borders are zero
    if (px < 441) C[sl].st[(px / 21 + 1) * 23 + px % 21 + 1] = next;
    if (tid < 32) {
      const int c = tid >> 4, k = tid & 15;
      if (c < ns) {
        const int64_t cell = cell0 + (int64_t)c * gridDim.x;
        const uint16_t f = A.feats[cell * 16 + k];
        C[c].ft[k] = f;
        if (BACK) A.ft[cell * 16 + k] = f;
      }
    }
    u8_t tap1;  // this lane's conv1 taps as offsets (k >= 9 is padding)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int k = min(8 * kq + i, 8);
      tap1[i] = (uint16_t)((k / 3) * 23 + k % 3);
    }
    const bf8_t a1 = ld8(wf + F1);
    const f4_t bias1 = ld4f(par + B1 + 4 * kq);
    __syncthreads();
    bf8_t a2[5];
#pragma unroll
    for (int s = 0; s < 5; ++s) a2[s] = ld8(wf + F2 + (5 * ct + s) * FRAG);
    const f4_t bias2 = ld4f(par + B2 + 16 * ct + 4 * kq);
    next = pixel(cell0 + (2 + sl) * (int)gridDim.x);
    // conv1: 16 channels x 16 pixels per product
    for (int u = w; u < 28 * ns; u += NW) {
      const int c = u >= 28, p = 16 * (u - 28 * c) + r16, q = min(p, 440), y = q / 21, x = q % 21;
      const bf8_t b = first8(gather8(C[c].st + y * 23 + x, tap1), 9 - 8 * kq);
      const f4_t d = act(mfma(a1, b, ZERO4), bias1);
      if (p < 441) st4(&C[c].h1[((y + 1) * 23 + x + 1) * S1 + 4 * kq], pack4(d));
    }
    __syncthreads();
    bf8_t a3[9];
#pragma unroll
    for (int s = 0; s < 9; ++s) a3[s] = ld8(wf + F3 + (9 * ct + s) * FRAG);
    // conv2: wavefront w takes pixel tile w / 2 of channel tile ct
    for (int c = 0; c < ns; ++c) {
      const int p = 16 * (w >> 1) + r16, q = min(p, 120), oy = q / 11, ox = q % 11;
      const uint16_t* b = C[c].h1 + (46 * oy + 2 * ox) * S1;
      f4_t acc = ZERO4;
#pragma unroll
      for (int s = 0; s < 5; ++s) {
        const int k = 32 * s + 8 * kq, tap = min(k >> 4, 8);
        bf8_t v = ld8(b + ((tap / 3) * 23 + tap % 3) * S1 + (k & 15));
        if (s == 4) v = keep8(v, kq < 2);
        acc = mfma(a2[s], v, acc);
      }
      if (p < 121) st4(&C[c].h2[((oy + 1) * 13 + ox + 1) * S2 + 16 * ct + 4 * kq], pack4(act(acc, bias2)));
    }
    const int steps = FC4_STEPS / A.splits;
    const int u4 = min(w, 4 * A.splits - 1);
    const uint16_t* w4 = wf + F4 + ((u4 & 3) * FC4_STEPS + (u4 >> 2) * steps) * FRAG;
    const f4_t bias3 = ld4f(par + B3 + 16 * ct + 4 * kq);
    __syncthreads();
    bf8_t a4[9];
    // conv3: three pixel tiles x two channel tiles of each cell
    if (w < 6 * NS) {
      const int c = w >= 6, p = 16 * ((w >> 1) - 3 * c) + r16, q = min(p, 35), oy = q / 6, ox = q % 6;
      const uint16_t* b = C[c].h2 + (26 * oy + 2 * ox) * S2 + 8 * kq;
      f4_t acc = ZERO4;
#pragma unroll
      for (int s = 0; s < 9; ++s) acc = mfma(a3[s], ld8(b + ((s / 3) * 13 + s % 3) * S2), acc);
#pragma unroll
      for (int i = 0; i < 9; ++i) a4[i] = ld8(w4 + i * FRAG);
      if (c < ns && p < 36) {
        const uint2 b = pack4(act(acc, bias3));
        st4(&C[c].h3[p * 32 + 16 * ct + 4 * kq], b);
        if (BACK) st4(A.h3 + (cell0 + (int64_t)c * gridDim.x) * 1152 + p * 32 + 16 * ct + 4 * kq, b);
      }
    }
    else {  // FC5
#pragma unroll
      for (int i = 0; i < 9; ++i) a4[i] = ld8(w4 + i * FRAG);
      const int t = w - 6 * NS;
      const f4_t d = act(mfma(ld8(wf + F5 + t * FRAG), keep8(ld8(C[col].ft + 8 * (kq & 1)), kq < 2), ZERO4),
                         ld4f(par + B5 + 16 * t + 4 * kq));
      if (r16 < 2) st4(&C[col].cat[64 + 16 * t + 4 * kq], pack4(d));
    }
    __syncthreads();
    // FC4 (the cells in the columns in turn): channel tile u & 3, partial sum u >> 2
    bf8_t a6[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) a6[s] = ld8(wf + F6 + ((w & 3) * 4 + s) * FRAG);
    if (w < 4 * A.splits) {
      f4_t acc = ZERO4;
      const uint16_t* b = C[col].h3 + 32 * (w >> 2) * steps + 8 * kq;
      for (int s = 0; s < steps; s += 9) {
        if (s != 0) {
#pragma unroll
          for (int i = 0; i < 9; ++i) a4[i] = ld8(w4 + (s + i) * FRAG);
        }
#pragma unroll
        for (int i = 0; i < 9; ++i) acc = mfma(a4[i], ld8(b + 32 * (s + i)), acc);
      }
      if (r16 < 2) *reinterpret_cast<f4_t*>(&C[col].part[w >> 2][16 * (w & 3) + 4 * kq]) = acc;
    }
    const float bias4 = par[B4 + lane];
    const f4_t bias6 = ld4f(par + B6 + 16 * (w & 3) + 4 * kq);
    __syncthreads();
    if (w < 2) {
      float v = C[w].part[0][lane];
      for (int s = 1; s < A.splits; ++s) v += C[w].part[s][lane];
      C[w].cat[lane] = f2bf(fmaxf(v + bias4, 0.f));
    }
    bf8_t a7[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) a7[s] = ld8(wf + F7 + s * FRAG);
    const float bias7 = par[B7], label = BACK && r16 < ns ? A.labels[col_cell] : 0.f, w7 = bf2f(f2bf(par[W7 + lane]));
    __syncthreads();
    if (w < 4) {  // FC6
      f4_t acc = ZERO4;
#pragma unroll
      for (int s = 0; s < 4; ++s) acc = mfma(a6[s], ld8(C[col].cat + 32 * s + 8 * kq), acc);
      if (r16 < 2) st4(&C[col].h6[16 * w + 4 * kq], pack4(act(acc, bias6)));
    }
    bf8_t b6[2];
    if (BACK) {
#pragma unroll
      for (int s = 0; s < 2; ++s) b6[s] = ld8(wf + G6 + ((w & 7) * 2 + s) * FRAG);
    }
    __syncthreads();
    if (w == 0) {  // FC7: row 0 of the tile
      f4_t acc = ZERO4;
#pragma unroll
      for (int s = 0; s < 2; ++s) acc = mfma(a7[s], ld8(C[col].h6 + 32 * s + 8 * kq), acc);
      if (lane < ns) {
        const float z = acc[0] + bias7;
        A.z[col_cell] = z;
        if (BACK) {
          C[col].loss += fmaxf(z, 0.f) - z * label + log1pf(expf(-fabsf(z)));
          const float d = (1.f / (1.f + expf(-z)) - label) / (float)A.B;
          C[col].dz = d;
          C[col].gb7 += d;
        }
      }
    }
    if (!BACK) continue;
    __syncthreads();
    bf8_t b4[5][2];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) b4[i][h] = ld8(wf + G4 + (min(w + NW * i, 71) * 2 + h) * FRAG);
    // delta of FC6's output
    if (w < 2) {
      uint16_t b = 0;
      if (w < ns) {
        const uint16_t dz = f2bf(C[w].dz);
        float v = bf2f(dz) * w7;
        const float h = bf2f(C[w].h6[lane]);
        C[w].gw7[lane] += h * bf2f(dz);
        if (!(h > 0.f)) v = 0.f;
        C[w].gb6[lane] += v;
        b = f2bf(v);
        A.d6[(cell0 + (int64_t)w * gridDim.x) * 64 + lane] = b;
      }
      C[w].d6[lane] = b;
    } else if (w < 2 + 2 * ns) {
      const int c = (w - 2) >> 1, k = 64 * (w & 1) + lane;
      A.cat[(cell0 + (int64_t)c * gridDim.x) * 128 + k] = C[c].cat[k];
    }
    __syncthreads();
    // deltas of FC4's and FC5's outputs: 16 of the 128 per wavefront
    if (w < 8) {
      f4_t acc = ZERO4;
#pragma unroll
      for (int s = 0; s < 2; ++s) acc = mfma(b6[s], ld8(C[col].d6 + 32 * s + 8 * kq), acc);
      const f4_t d = mask4(acc, ld4(C[col].cat + 16 * w + 4 * kq));
      if (r16 < 2) {
        *reinterpret_cast<f4_t*>(&C[col].gbc[16 * w + 4 * kq]) += d;
        const uint2 b = pack4(d);
        if (w < 4) st4(&C[col].d4[16 * w + 4 * kq], b);
        if (r16 < ns) st4((w < 4 ? A.d4 : A.d5) + col_cell * 64 + 16 * (w & 3) + 4 * kq, b);
      }
    }
    __syncthreads();
    // delta of conv3's output: 72 tiles of 16
    {
      const bf8_t b0 = ld8(C[col].d4 + 8 * kq), b1 = ld8(C[col].d4 + 32 + 8 * kq);
#pragma unroll
      for (int i = 0; i < 5; ++i) {
        const int t = w + NW * i;
        if (i < 2) {
#pragma unroll
          for (int h = 0; h < 2; ++h) b4[i + 3][h] = ld8(wf + G4 + (min(t + 3 * NW, 71) * 2 + h) * FRAG);
        }
        if (t >= 72) break;
        const f4_t acc = mfma(b4[i][1], b1, mfma(b4[i][0], b0, ZERO4));
        const int k = 16 * t + 4 * kq;
        const f4_t d = mask4(acc, ld4(C[col].h3 + k));
        gb3 += d;
        if (r16 < 2) st4(&Q[col].d3[(k >> 5) * S2 + (k & 31)], pack4(d));
      }
    }
    bf8_t bt[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) bt[k] = ld8(wf + G3 + (k * 2 + ct) * FRAG);
    __syncthreads();
    // delta of conv2's output
    for (int u = w >> 1; u < DeltaTiles<11>::N * ns; u += NW / 2) {
      const int c = u >= DeltaTiles<11>::N;
      int y, x;
      bool ok;
      const f4_t v = delta_unit<11>(bt, Q[c].d3 + 8 * kq, u - c * DeltaTiles<11>::N, r16, y, x, ok);
      if (ok) {
        const f4_t d = mask4(v, ld4(C[c].h2 + ((y + 1) * 13 + x + 1) * S2 + 16 * ct + 4 * kq));
        gb2 += d;
        st4(&Q[c].d2[(y * 11 + x) * S2 + 16 * ct + 4 * kq], pack4(d));
      }
    }
#pragma unroll
    for (int k = 0; k < 9; ++k) bt[k] = ld8(wf + G2 + k * FRAG);
    __syncthreads();
    // delta of conv1's output
    for (int u = w; u < DeltaTiles<21>::N * ns; u += NW) {
      const int c = u >= DeltaTiles<21>::N;
      int y, x;
      bool ok;
      const f4_t v = delta_unit<21>(bt, Q[c].d2 + 8 * kq, u - c * DeltaTiles<21>::N, r16, y, x, ok);
      if (ok) {
        const f4_t d = mask4(v, ld4(C[c].h1 + ((y + 1) * 23 + x + 1) * S1 + 4 * kq));
        gb1 += d;
        st4(&Q[c].d1[(y * 21 + x) * 16 + 4 * kq], pack4(d));
      }
    }
    __syncthreads();
    // weight gradients, K = pixels: this lane's share of a transposed read is pixel kr (and kr + 4), channels c4
    const int kr = 8 * kq + (r16 >> 2), c4 = 4 * (r16 & 3);
    for (int c = 0; c < ns; ++c) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int j = w + NW * i;
        if (j < 18) {
          const uint16_t* h = C[c].h2 + (((j >> 1) / 3) * 13 + (j >> 1) % 3) * S2 + 16 * (j & 1) + c4;
          const uint16_t* d = Q[c].d3 + kr * S2 + c4;
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            bf8_t a = ld_tr(h + at3[32 * s + kr], h + at3[32 * s + kr + 4]);
            if (s == 1) a = first8(a, 36 - 32 - 8 * kq);
#pragma unroll
            for (int n = 0; n < 2; ++n)
              g[i][n] = mfma(a, ld_tr(d + 32 * s * S2 + 16 * n, d + (32 * s + 4) * S2 + 16 * n), g[i][n]);
          }
        } else if (j < 27) {
          const uint16_t* h = C[c].h1 + (((j - 18) / 3) * 23 + (j - 18) % 3) * S1 + c4;
          const uint16_t* d = Q[c].d2 + kr * S2 + c4;
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            bf8_t a = ld_tr(h + at2[32 * s + kr], h + at2[32 * s + kr + 4]);
            if (s == 3) a = first8(a, 121 - 96 - 8 * kq);
#pragma unroll
            for (int n = 0; n < 2; ++n)
              g[i][n] = mfma(a, ld_tr(d + 32 * s * S2 + 16 * n, d + (32 * s + 4) * S2 + 16 * n), g[i][n]);
          }
        }
      }
    }
    // conv1's by the wavefronts with the fewest of the products above
    if (w >= 11) {
      const int tap = min(r16, 8);
      for (int u = w - 11; u < 14 * ns; u += NW - 11) {
        const int c = u >= 14, s = u - 14 * c;
        const u8_t o = *reinterpret_cast<const u8_t*>(&at1[32 * s + 8 * kq]);
        const bf8_t a = first8(gather8(C[c].st + (tap / 3) * 23 + tap % 3, o), r16 < 9 ? 441 - 32 * s - 8 * kq : 0);
        const uint16_t* d = Q[c].d1 + (32 * s + kr) * 16 + c4;
        g1 = mfma(a, ld_tr(d, d + 64), g1);
      }
    }
  }
  if (!BACK) return;
  // the record: what one wavefront holds goes out as it is; sums over
  // wavefronts (first layer, biases) and over the pixel columns meet in LDS
  const int w = wave, lane = tid & 63, r16 = lane & 15, kq = lane >> 4;
  float* rec = A.records + (int64_t)blockIdx.x * TRAIN_RECORD;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int j = w + NW * i, row = j < 18 ? W3 + 16 * j * 32 : W2 + 16 * (j - 18) * 32;
    if (j >= 27) break;
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) rec[row + (4 * kq + r) * 32 + 16 * n + r16] = g[i][n][r];
  }
#pragma unroll
  for (int o = 8; o > 0; o >>= 1)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      gb1[r] += __shfl_xor(gb1[r], o, 64);
      gb2[r] += __shfl_xor(gb2[r], o, 64);
    }
#pragma unroll
  for (int r = 0; r < 4; ++r) {  // the two cells' columns
    gb3[r] += __shfl_xor(gb3[r], 1, 64);
  }
  __syncthreads();
  // [wavefronts 11 ..][9 x 16]; three biases of 16 per wavefront
  float* red = reinterpret_cast<float*>(C[0].h1);
  constexpr int RB = (NW - 11) * 144;
  static_assert((RB + NW * 48) * 4 <= (int)sizeof(C[0].h1), "room for the sums over wavefronts");
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (w >= 11 && 4 * kq + r < 9) red[(w - 11) * 144 + (4 * kq + r) * 16 + r16] = g1[r];
    if (r16 == 0) {
      red[RB + (w * 3 + 0) * 16 + 4 * kq + r] = gb1[r];
      red[RB + (w * 3 + 1) * 16 + 4 * kq + r] = gb2[r];
      red[RB + (w * 3 + 2) * 16 + 4 * kq + r] = gb3[r];
    }
  }
  if (tid == 0) {
    rec[R7 + 64] = C[0].gb7 + C[1].gb7;
    rec[RL] = C[0].loss + C[1].loss;
  }
  __syncthreads();
  if (tid < 144) {
    float v = 0.f;
    for (int q = 0; q < NW - 11; ++q) v += red[q * 144 + tid];
    rec[W1 + tid] = v;
  } else if (tid < 160) {
    float v = 0.f;
    for (int q = 0; q < NW; ++q) v += red[RB + q * 48 + tid - 144];
    rec[B1 + tid - 144] = v;
  } else if (tid >= 192 && tid < 256) {
    // channels 16 c .. of conv2 (k = 1) and conv3 (k = 2): wavefronts c, c + 2, ...
    const int k = 1 + ((tid - 192) >> 5), ch = tid & 31;
    float v = 0.f;
    for (int q = ch >> 4; q < NW; q += 2) v += red[RB + (q * 3 + k) * 16 + (ch & 15)];
    rec[(k == 1 ? B2 : B3) + ch] = v;
  } else if (tid >= 256 && tid < 384) {
    rec[R4 + tid - 256] = C[0].gbc[tid - 256] + C[1].gbc[tid - 256];
  } else if (tid >= 384 && tid < 448) {
    rec[R6 + tid - 384] = C[0].gb6[tid - 384] + C[1].gb6[tid - 384];
  } else if (tid >= 448 && tid < 512) {
    rec[R7 + tid - 448] = C[0].gw7[tid - 448] + C[1].gw7[tid - 448];
  }
}

// Position of weight (k, n) of a layer within its fragments: `steps` K steps of 32 per row tile of 16.
__device__ __forceinline__ int frag_at(int row, int k, int steps) {
  return ((row >> 4) * steps + (k >> 5)) * FRAG + (((k & 31) >> 3) * 16 + (row & 15)) * 8 + (k & 7);
}
// The BF16 copies of parameter i in the forward and back fragments.
__device__ __forceinline__ void put_weight(uint16_t* wf, int i, uint16_t b) {
  int k, n;
  if (i < B1) {
    k = i / 16, n = i % 16;
    wf[F1 + frag_at(n, k, 1)] = b;
  } else if (i >= W2 && i < B2) {
    k = (i - W2) / 32, n = (i - W2) % 32;
    wf[F2 + frag_at(n, k, 5)] = b;
    wf[G2 + (k / 16) * FRAG + frag_at(k % 16, n, 1)] = b;
  } else if (i >= W3 && i < B3) {
    k = (i - W3) / 32, n = (i - W3) % 32;
    wf[F3 + frag_at(n, k, 9)] = b;
    wf[G3 + (k / 32) * 2 * FRAG + frag_at(k % 32, n, 1)] = b;
  } else if (i >= W4 && i < B4) {
    k = (i - W4) / 64, n = (i - W4) % 64;
    wf[F4 + frag_at(n, k, FC4_STEPS)] = b;
    wf[G4 + frag_at(k, n, 2)] = b;
  } else if (i >= W5 && i < B5) {
    k = (i - W5) / 64, n = (i - W5) % 64;
    wf[F5 + frag_at(n, k, 1)] = b;
  } else if (i >= W6 && i < B6) {
    k = (i - W6) / 64, n = (i - W6) % 64;
    wf[F6 + frag_at(n, k, 4)] = b;
    wf[G6 + frag_at(k, n, 2)] = b;
  } else if (i >= W7 && i < B7) {
    wf[F7 + frag_at(0, i - W7, 2)] = b;
  }
}

// Adam (Kingma & Ba) on the FP32 master weights, refreshing their BF16 copies.
__device__ __forceinline__ void adam(const AdamArgs& P, int i, float g) {
  const float m = P.b1 * P.m[i] + (1.f - P.b1) * g;
  const float v = P.b2 * P.v[i] + (1.f - P.b2) * g * g;
  P.m[i] = m;
  P.v[i] = v;
  const float x = P.w[i] - P.lr * (m / P.c1) / (sqrtf(v / P.c2) + P.eps);
  P.w[i] = x;
  put_weight(P.wf, i, f2bf(x));
}

// The gradient from the records and from the inputs and deltas of the fully
// connected layers, to grad or with STEP straight into Adam; every sum is in
// a fixed order.  Blocks below FC_BLOCKS: dW = X^T d of 32 rows (input
// channels) and all 64 columns, eight wavefronts sharing the cells, 32 per
// product: a lane reads two neighbouring rows and four neighbouring columns
// of eight cells, the two and four tiles of its products.  The other blocks
// add 64 entries of the records, eight wavefronts sharing the records.  5.9 us
// for 512 cells (15 MB of records): 64 KB of LDS so that two workgroups share
// a CU and all are resident; sixteen wavefronts and 128 KB took 14.2 us.
constexpr int SUM_T = 512, SUM_W = SUM_T / 64;
constexpr int FC_BLOCKS = 36 + 1 + 4;
constexpr int SUM_BLOCKS = (RN + 63) / 64;
template <bool STEP>
__global__ __launch_bounds__(SUM_T) void k_train_sum(TrainArgs A, int n_rec, float* __restrict__ loss,
                                                     float* __restrict__ grad, AdamArgs P) {
  __shared__ __align__(16) float red[SUM_W][32 * 64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r16 = lane & 15, kq = lane >> 4;
  if (blockIdx.x >= FC_BLOCKS) {
    const int e = (blockIdx.x - FC_BLOCKS) * 64 + lane;
    float v = 0.f;
    if (e < RN)
#pragma unroll 8
      for (int r = w; r < n_rec; r += SUM_W) v += A.records[(int64_t)r * TRAIN_RECORD + e];
    red[w][lane] = v;
    __syncthreads();
    if (w != 0 || e >= RN) return;
    for (int q = 1; q < SUM_W; ++q) v += red[q][lane];
    if (e == RL) {
      if (loss) *loss = v / (float)A.B;
      return;
    }
    const int i = e < W4 ? e : e < R5 ? B4 + e - R4 : e < R6 ? B5 + e - R5 : e < R7 ? B6 + e - R6 : W7 + e - R7;
    if (STEP) adam(P, i, v);
    else grad[i] = v;
    return;
  }
  const int mb = blockIdx.x;
  const uint16_t *X, *D;
  int ldx, rows = 32, out;
  if (mb < 36) { X = A.h3 + 32 * mb; ldx = 1152; D = A.d4; out = W4 + 32 * mb * 64; }
  else if (mb == 36) { X = A.ft; ldx = 16; rows = 16; D = A.d5; out = W5; }
  else { X = A.cat + 32 * (mb - 37); ldx = 128; D = A.d6; out = W6 + 32 * (mb - 37) * 64; }
  const bool in_row = 2 * r16 < rows;
  f4_t acc[2][4];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int n = 0; n < 4; ++n) acc[m][n] = ZERO4;
  for (int c0 = 32 * w; c0 < A.B; c0 += 32 * SUM_W) {
    uint32_t x[8];
    uint2 d[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int c = c0 + 8 * kq + i;
      x[i] = c < A.B && in_row ? *reinterpret_cast<const uint32_t*>(X + (int64_t)c * ldx + 2 * r16) : 0u;
      d[i] = c < A.B ? *reinterpret_cast<const uint2*>(D + (int64_t)c * 64 + 4 * r16) : make_uint2(0u, 0u);
    }
    u8_t a[2], b[4];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      a[0][i] = (uint16_t)x[i];
      a[1][i] = (uint16_t)(x[i] >> 16);
      b[0][i] = (uint16_t)d[i].x;
      b[1][i] = (uint16_t)(d[i].x >> 16);
      b[2][i] = (uint16_t)d[i].y;
      b[3][i] = (uint16_t)(d[i].y >> 16);
    }
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int n = 0; n < 4; ++n)
        acc[m][n] = mfma(__builtin_bit_cast(bf8_t, a[m]), __builtin_bit_cast(bf8_t, b[n]), acc[m][n]);
  }
  // row 2 (4 kq + r) + m, column 4 r16 + n
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      *reinterpret_cast<f4_t*>(&red[w][(2 * (4 * kq + r) + m) * 64 + 4 * r16]) =
          f4_t{acc[m][0][r], acc[m][1][r], acc[m][2][r], acc[m][3][r]};
  __syncthreads();
#pragma unroll
  for (int h = 0; h < 32 * 64 / SUM_T; ++h) {
    const int e = tid + SUM_T * h;
    if (e >= rows * 64) break;
    float v = red[0][e];
    for (int q = 1; q < SUM_W; ++q) v += red[q][e];
    if (STEP) adam(P, out + e, v);
    else grad[out + e] = v;
  }
}

// The BF16 copies of all parameters.
__global__ void k_scorer_weights(const float* __restrict__ w, uint16_t* __restrict__ wf) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < NP) put_weight(wf, i, f2bf(w[i]));
}

hipError_t launch_scorer_weights(const float* w, uint16_t* wf, hipStream_t s) {
  hipLaunchKernelGGL(k_scorer_weights, dim3((NP + 255) / 256), dim3(256), 0, s, w, wf);
  return hipGetLastError();
}

// Partial sums of the 1152-deep layer, a property of the result (the sums
// round differently): four up to 16 320 cells, two up to 32 704, then one.
int train_splits(int B) {
  const int tiles = (B + 63) / 64;
  return tiles < 256 ? 4 : tiles < 512 ? 2 : 1;
}
int train_groups(int B) { return B < 256 ? B : 256; }

hipError_t launch_train_forward(const TrainArgs& a, hipStream_t s) {
  if (a.B <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_train_cells<false>, dim3((unsigned)train_groups(a.B)), dim3(NT), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_train_grad(const TrainArgs& a, float* loss, float* grad, const AdamArgs* step, hipStream_t s) {
  if (a.B <= 0) return hipSuccess;
  const int groups = train_groups(a.B);
  hipLaunchKernelGGL(k_train_cells<true>, dim3((unsigned)groups), dim3(NT), 0, s, a);
  const dim3 g(FC_BLOCKS + SUM_BLOCKS);
  if (step)
    hipLaunchKernelGGL(k_train_sum<true>, g, dim3(SUM_T), 0, s, a, groups, loss, nullptr, *step);
  else
    hipLaunchKernelGGL(k_train_sum<false>, g, dim3(SUM_T), 0, s, a, groups, loss, grad, AdamArgs{});
  return hipGetLastError();
}

}  // namespace dtk
