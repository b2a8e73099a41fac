// k_nn.hip -- a BF16 MFMA GEMM, and the parameter initialisation of the
// learned cell scorer.
//
// GEMM: C[M x N] = op(A)[M x K] op(B)[K x N], A and B bfloat16, FP32
// accumulation on gfx950's v_mfma_f32_16x16x32_bf16.  A workgroup of four
// waves owns a 64 x 64 tile of C (each wave 32 x 32 = 2 x 2 MFMA tiles); K
// advances in steps of 32 (one MFMA per tile) through LDS tiles stored
// K-contiguous so that every lane's MFMA operand (eight consecutive K values)
// is one 16-byte LDS read.  A lane's A and B operands cover the same eight K
// indices, so the products the instruction pairs are those of one K.  Split-K writes
// FP32 partial tiles that a second kernel sums in a fixed order, so results
// are deterministic.
#include "dt_common.hpp"

namespace dtk {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));

constexpr int GT_M = 64, GT_N = 64, GT_K = 32;

// Partial GEMM over k in [k0, k1).  Output: if part != null, raw FP32 tile to
// part (ldc = N); otherwise the epilogue (bias, ReLU).
__global__ __launch_bounds__(256) void k_gemm_bf16(const uint16_t* __restrict__ A, int lda, int transA,
                                                   const uint16_t* __restrict__ B, int ldb, int transB, int M,
                                                   int N, int K, int k_per_split, float* __restrict__ part,
                                                   const float* __restrict__ bias, int relu, float* __restrict__ Cf,
                                                   int ldcf) {
  // [m][k] and [n][k]; rows of 80 bytes keep every 8-element operand 16-byte aligned
  __shared__ __attribute__((aligned(16))) uint16_t sA[GT_M][GT_K + 8];
  __shared__ __attribute__((aligned(16))) uint16_t sB[GT_N][GT_K + 8];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m0 = blockIdx.x * GT_M, n0 = blockIdx.y * GT_N;
  const int kb = blockIdx.z * k_per_split;
  const int ke = min(K, kb + k_per_split);
  const int wm = (wave & 1) * 32, wn = (wave >> 1) * 32;
  float4_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = float4_t{0.f, 0.f, 0.f, 0.f};
  for (int k0 = kb; k0 < ke; k0 += GT_K) {
    // stage A (64 x 32) and B (32 x 64): 2048 elements each, 8 per thread
    // consecutive threads walk the dimension that is contiguous in memory
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int idx = tid + q * 256;
      int r, c;  // r: m (or n), c: k
      if (!transA) { r = idx >> 5; c = idx & 31; } else { c = idx >> 6; r = idx & 63; }
      const int gm = m0 + r, gk = k0 + c;
      uint16_t va = 0;
      if (gm < M && gk < ke) va = transA ? A[(int64_t)gk * lda + gm] : A[(int64_t)gm * lda + gk];
      sA[r][c] = va;
      if (transB) { r = idx >> 5; c = idx & 31; } else { c = idx >> 6; r = idx & 63; }
      const int gn = n0 + r, gk2 = k0 + c;
      uint16_t vb = 0;
      if (gn < N && gk2 < ke) vb = transB ? B[(int64_t)gn * ldb + gk2] : B[(int64_t)gk2 * ldb + gn];
      sB[r][c] = vb;
    }
    __syncthreads();
    {
      const int kk = 8 * (lane >> 4);
      bf16x8_t a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[i] = *(const bf16x8_t*)&sA[wm + 16 * i + (lane & 15)][kk];
        b[i] = *(const bf16x8_t*)&sB[wn + 16 * i + (lane & 15)][kk];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }
  // D layout: lane holds column (lane & 15), rows 4 * (lane >> 4) + r
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int gm = m0 + wm + 16 * i + 4 * (lane >> 4) + r;
        const int gn = n0 + wn + 16 * j + (lane & 15);
        if (gm >= M || gn >= N) continue;
        float v = acc[i][j][r];
        if (part) {
          part[((int64_t)blockIdx.z * M + gm) * N + gn] = v;
          continue;
        }
        if (bias) v += bias[gn];
        if (relu) v = fmaxf(v, 0.f);
        Cf[(int64_t)gm * ldcf + gn] = v;
      }
}

__global__ void k_splitk_reduce(const float* __restrict__ part, int splits, int M, int N,
                                const float* __restrict__ bias, int relu, float* __restrict__ Cf, int ldcf) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)M * N) return;
  const int gm = (int)(i / N), gn = (int)(i % N);
  float v = 0.f;
  for (int s = 0; s < splits; ++s) v += part[(int64_t)s * M * N + i];
  if (bias) v += bias[gn];
  if (relu) v = fmaxf(v, 0.f);
  Cf[(int64_t)gm * ldcf + gn] = v;
}

hipError_t launch_gemm_bf16(const GemmArgs& g, float* d_part, size_t part_elems, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  const int gm = (g.M + GT_M - 1) / GT_M, gn = (g.N + GT_N - 1) / GT_N;
  int splits = 1;
  // split long K so that small outputs still fill the machine
  while (splits < 256 && (int64_t)gm * gn * splits < 512 && g.K / (splits * 2) >= 256) splits *= 2;
  if (splits > 1 && (size_t)splits * g.M * g.N > part_elems) splits = 1;
  int kps = ((g.K + splits - 1) / splits + GT_K - 1) / GT_K * GT_K;
  splits = kps > 0 ? (g.K + kps - 1) / kps : 1;
  if (splits < 1) splits = 1;
  if (splits == 1) {
    hipLaunchKernelGGL(k_gemm_bf16, dim3(gm, gn, 1), dim3(256), 0, s, g.A, g.lda, g.transA, g.B, g.ldb, g.transB,
                       g.M, g.N, g.K, g.K > 0 ? ((g.K + GT_K - 1) / GT_K) * GT_K : GT_K, nullptr, g.bias, g.relu,
                       g.Cf, g.ldcf);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_gemm_bf16, dim3(gm, gn, splits), dim3(256), 0, s, g.A, g.lda, g.transA, g.B, g.ldb,
                     g.transB, g.M, g.N, g.K, kps, d_part, nullptr, 0, nullptr, 0);
  const int64_t mn = (int64_t)g.M * g.N;
  hipLaunchKernelGGL(k_splitk_reduce, dim3((unsigned)((mn + 255) / 256)), dim3(256), 0, s, d_part, splits, g.M, g.N,
                     g.bias, g.relu, g.Cf, g.ldcf);
  return hipGetLastError();
}

// He-normal weights (std sqrt(2 / fan_in)) and zero biases from a counter-based
// generator: splitmix64 of (seed, index) -> two uniforms -> Box-Muller.
__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}
__global__ void k_init_params(float* __restrict__ w, int64_t off, int64_t n, int fan_in, uint64_t seed,
                              int is_bias) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  if (is_bias) {
    w[off + i] = 0.f;
    return;
  }
  const uint64_t r = splitmix64(seed ^ splitmix64((uint64_t)(off + i)));
  const double u1 = ((double)(r >> 11) + 1.0) * (1.0 / 9007199254740993.0);
  const double u2 = (double)(splitmix64(r) >> 11) * (1.0 / 9007199254740992.0);
  const double z = sqrt(-2.0 * log(u1)) * cos(2.0 * PI * u2);
  w[off + i] = (float)(z * sqrt(2.0 / fan_in));
}

static unsigned g1d(int64_t n) { return (unsigned)((n + 255) / 256); }

hipError_t launch_init_params(float* w, int64_t off, int64_t n, int fan_in, uint64_t seed, int is_bias,
                              hipStream_t s) {
  hipLaunchKernelGGL(k_init_params, dim3(g1d(n)), dim3(256), 0, s, w, off, n, fan_in, seed, is_bias);
  return hipGetLastError();
}

}  // namespace dtk
