// dt_common.hpp -- structures and helpers shared by the host API and the HIP
// kernels of libdtrack (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "dtrack.h"

namespace dtk {

// Gaussian gravitational constant k (AU^1.5/day); GM_sun = k^2 (Sec. 3:
// two-body motion about the Sun, the asteroid's mass neglected).
constexpr double K_GAUSS = 0.01720209895;
constexpr double MU_SUN = K_GAUSS * K_GAUSS;
// Speed of light in AU/day from the SI metre, second and the IAU astronomical unit.
constexpr double C_AU_DAY = 299792458.0 * 86400.0 / 149597870700.0;
// Mean obliquity of the ecliptic at J2000 (IAU 2006), arcseconds.
constexpr double OBLIQUITY_ARCSEC = 84381.448;
constexpr double PI = 3.14159265358979323846;

// Days of epochs between checkpoints of the checkpoint walk (at least this often).
constexpr double CK_SPAN = 12.0;

// Per-exposure constants, prepared on the device from a dt_exposure.
// Everything is expressed in the heliocentric ecliptic frame so no rotation
// is needed per sample: the TAN basis is rotated once per exposure instead.
struct alignas(16) ExpMeta {
  // The fields every step of the checkpoint walk reads come first (64 bytes:
  // four scalar loads issued together, one wait).  A position q (AU from the observer) projects into the
  // pixel rectangle only if c.q > 0, |A0'.q| <= (W / 2) c.q and likewise for y,
  // with A0' = a0 + (px0 - (W - 1) / 2) c; kx X = A0' and so on are those scaled
  // so that a displacement of q by d changes |X.q| - kx c.q by at most d.
  double t;                 // epoch (days)
  float fX[3], fY[3], fZ[3];  // scaled A0', A1'; c
  float kx, ky;             // scaled half sizes (widened by 0.01 px)
  float fo[3];              // observer (AU, ecliptic)
  double ox, oy, oz;        // observer (AU, ecliptic)
  // Sky cone holding every direction that projects into the pixel rectangle
  // widened by one pixel: unit axis u, tangent of the half-angle, and the
  // limit of the cone test (0; +inf with u = 0 when no cone is used).
  double ux, uy, uz, cone_tan, cone_lim;
  double cx, cy, cz;        // tangent-point direction (ecliptic)
  double a0x, a0y, a0z;     // row 0 of (180/pi) CD^-1 [east; north] (px per unit, ecliptic)
  double a1x, a1y, a1z;     // row 1
  double px0, py0;          // CRPIX - 1
  double gap, inv_gap;      // epoch step from the previous exposure (epoch order) and its reciprocal
  int64_t plane_off;        // offset of this exposure's plane (in float2 units)
  int32_t W, H;             // image size
  int32_t src;              // caller's index of this exposure
  float fwhm;               // PSF FWHM (px)
  int32_t R;                // stamp half-width ceil(3 sigma)
  float vs;                 // scalar pixel variance when the patch has no variance planes
  int32_t ck_next;          // first exposure (epoch order) more than CK_SPAN days after this one (n + 1 when none)
  int32_t strip;            // columns of a pre-pass tile (prep_strip)
};
// A patch holds n + 1 records: the last exposure's record is repeated once
// (the checkpoint walk's final queue-serving step reads it, uses nothing of it).
static_assert(sizeof(ExpMeta) == 272, "ExpMeta layout");

// Exposure records, planes and elements seen through a named address space.
// A pointer read from device memory (a batched launch's per-patch
// descriptor) is generic to the compiler, and generic (flat) loads count as
// possibly per-lane: a wave-uniform record read through one would make the
// whole exposure walk per-lane (vector registers, masked branches).  The
// records are read through the constant address space (device memory no
// kernel writes while it runs), so a uniform record is read with scalar
// loads even where the kernel also stores to global memory; planes and
// elements through the global one.  Functions that take a generic
// reference get an explicit cast, which the compiler sees through.
typedef const __attribute__((address_space(4))) ExpMeta GExpMeta;
__device__ __forceinline__ GExpMeta* global_meta(const ExpMeta* p) { return (GExpMeta*)p; }
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(1))) T* global_ptr(const T* p) {
  return (const __attribute__((address_space(1))) T*)p;
}
template <typename T>
__device__ __forceinline__ T global_load(const T* p, int64_t i) {
  return *(const T*)&global_ptr(p)[i];
}

// One tile of the matched-filter pre-pass.
struct PrepTile {
  int32_t e;       // exposure (sorted index)
  int32_t x0, y0;  // tile origin (x0 even)
  int32_t ny;      // output rows
};

constexpr int PREP_TY = 128;      // output rows a wavefront streams, about; down to
constexpr int PREP_TY_MIN = 16;   // this in patches of fewer than
constexpr int PREP_TILES = 1536;  // tiles (the card holds 3072 wavefronts of this kernel)
constexpr int PREP_DEPTH = 4; // input rows each lane keeps in flight
// A lane holds `groups` pairs of columns (one where the partial sums of two
// would leave a single wavefront per SIMD); a wavefront's 128 x groups input
// columns start prep_lead(R) columns before its prep_width(R) output columns.
constexpr int prep_groups(int R) { return R <= 6 ? 2 : 1; }
constexpr int prep_lead(int R) { return (R + 1) & ~1; }
constexpr int prep_width(int R) { return (128 * prep_groups(R) - prep_lead(R) - R) & ~1; }
// Columns of the tiles of an image W wide.  Strips are as wide as can be.  The
// narrowest stamps leave nothing but memory to wait for: where the image's rows
// are whole 128-byte lines of the plane, their strips are as many of equal width
// in whole lines if that still fits, so that no line is written by two (100 FP32
// 2048^2 images at R = 1: 1.48 ms in strips of 252 columns, 1.37 of 240; 1.41 and
// 1.39 at R = 4).  More strips for the sake of whole lines gain nothing (40 of
// 4096^2: 2.38 and 2.39).
constexpr int PREP_EVEN_R = 2;
__host__ __device__ inline int prep_strip(int R, int W) {
  const int most = prep_width(R), n = (int)(((int64_t)W + most - 1) / most);
  const int w = (int)(((int64_t)W + n - 1) / n + 15) / 16 * 16;
  return R <= PREP_EVEN_R && W % 16 == 0 && w <= most ? w : most;
}
constexpr int PREP_RMAX = 11; // largest stamp half-width supported (FWHM <= 8 px gives R = 11)

// Launchers (defined in the .hip files; all enqueue on `s`).
hipError_t launch_exposure_prep(const dt_exposure* d_in, const int64_t* d_plane_off, const int32_t* d_src,
                                const int32_t* d_R, int n, ExpMeta* d_out, hipStream_t s);
// Tiles are grouped by stamp half-width: group gi covers tiles
// [group_off[gi], group_off[gi+1]) whose exposures all have R = group_R[gi];
// group_R 0: the images one column wide, of any half-width.
hipError_t launch_prepass(const ExpMeta* d_meta, const PrepTile* d_tiles, const int64_t* group_off,
                          const int32_t* group_R, int n_groups, const void* const* d_flux,
                          const void* const* d_var, bool has_var, dt_dtype dtype, float2* d_planes, hipStream_t s);

// Stamp half-width for a PSF FWHM: R = ceil(3 sigma), sigma = FWHM / (2 sqrt(2 ln 2)).
inline int stamp_radius(double fwhm) {
  double sig = fwhm / (2.0 * __builtin_sqrt(2.0 * __builtin_log(2.0)));
  return (int)__builtin_ceil(3.0 * sig);
}

struct StackArgs {
  const ExpMeta* meta;
  int32_t n_exp;
  const float2* planes;
  int64_t n;
  double epoch;
  const double *a, *e, *inc, *node, *peri, *m0;
  float* snr;
  float* flux;
  int32_t* nvalid;
  // Bound on the observer's speed (AU/day) between any two exposures of the
  // patch: the largest |obs_i - obs_j| / (t_i - t_j) over epoch neighbours
  // (infinite when two exposures share an epoch but not an observer).
  double vobs = __builtin_inf();
  // Work counters of the checkpoint walk (measurement only; NULL = off):
  // WORK_SLOTS slots of WORK_N counters, slot = workgroup index mod WORK_SLOTS.
  unsigned long long* work = nullptr;
  // Deferral (NULL = not allowed): a wavefront of the checkpoint walk whose
  // samples land often appends its first orbit index to defer_list (slot from
  // *defer_count, zeroed before the launch) and writes no outputs; the
  // deferred-walk kernel then stacks those orbits per sample.
  int64_t* defer_list = nullptr;
  unsigned int* defer_count = nullptr;
  int64_t plane_bytes = 0;  // of all planes (the launch's choice of where wavefronts defer)
};

// 1 / stack_switch(a): the share of its samples queued above which a wavefront
// of a launch that allows it defers.  The queue saves the arithmetic of samples
// that miss, but its gathers are waited for, which the per-sample walk's are
// not, so the larger the planes (the further beyond the 256 MiB Infinity Cache),
// the sooner a wavefront gives up.  Measured at 1/4, 1/5, 1/6, 1/7 and, last,
// with the FP64 cone at 1/5, whose queue is up to half as large again (ms;
// 2 x 10^6 to 10^7 orbits):
//   0.13 GB 0.05 AU away 0.75 0.86 0.84 0.87   0.78
//   0.25 GB main belt    0.35 0.45 0.80 0.80   0.79
//   0.25 GB near Earth   0.37 0.39 0.70 0.80   0.64
//   0.84 GB 0.05 AU away 1.47 1.50 1.68 1.75   1.49
//   0.84 GB 0.015 AU     1.90 1.61 1.52 1.49   1.63
//   1.0 GB distant       2.67 2.49 2.37 2.36   2.41
//   2.0 GB main belt     0.60 0.65 0.65 0.88   0.81
//   2.0 GB near Earth    0.62 0.66 0.68 0.94   0.75
//   4.0 GB distant       3.18 4.06 4.06 3.69   3.70
//   16 GB main belt      2.39 2.18 2.06 1.98   2.05
//   53 GB distant        44.0 36.4 33.3 32.2   32.2
constexpr int64_t SWITCH_TINY = 256ll << 20, SWITCH_SMALL = 1000000000, SWITCH_LARGE = 3000000000;  // bytes of planes
inline int stack_switch(const StackArgs& a) {
  return a.plane_bytes < SWITCH_TINY ? 4 : a.plane_bytes < SWITCH_SMALL ? 5 : a.plane_bytes < SWITCH_LARGE ? 6 : 7;
}
// f(std::integral_constant<int, stack_switch(a)>): picks a kernel instance.
template <typename F>
inline void with_switch(const StackArgs& a, F&& f) {
  switch (stack_switch(a)) {
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    default: f(std::integral_constant<int, 7>{}); break;
  }
}

// Work counters (one slot; see dt_ctx_count_work): samples tested by
// prediction, queued exact solves, checkpoint solves, samples walked by the
// per-sample tail, tail samples that took the full path, wavefronts that
// switched to the tail.
enum { WORK_PRED = 0, WORK_QUEUED, WORK_CKPT, WORK_TAIL, WORK_TAIL_FULL, WORK_SWITCHED, WORK_N = 8 };
constexpr int WORK_SLOTS = 64;

struct DebugArgs {
  const int64_t* ids;
  int64_t m;
  double *px, *py, *tau;
  int32_t *ix, *iy, *flags;
  float *psi, *phi;
};

// Work item of the batched persistent launch: orbits [begin, begin + count)
// of patch `patch`.
struct WorkItem {
  int32_t patch;
  int32_t count;
  int64_t begin;
};

// Wavefronts that share 64 orbits of a small launch (their exposures cut
// into that many ranges, split_walk), 0: one wavefront walks all exposures.
// A launch of up to 48 x 1024 orbits leaves most of the chip's wavefront slots
// empty and takes as long as one walk; cut, it does up to twice the work
// (samples solved one by one, a cold start per range) in parallel.  The line
// is where that work fills the chip: three workgroups of four wavefronts per
// CU, or one of eight, with their samples in LDS.  Measured (checkpoint walk
// -> split): 10^4 orbits x 20 exposures 25 -> 13.5 us, x 200 88-114 -> 33-35
// (distant objects, which land often: 389 -> 50); 3 x 10^4 x 60 42-49 -> 27-32;
// 6 x 10^4 x 60 43-51 -> 42-50 (equal); 1.3 x 10^5 x 60 50-59 -> 68-86.
// Launches that count their work run the checkpoint walk, which is what the
// counters are about (the sums are the same).
inline size_t stack_split_lds(int n_exp) { return sizeof(float2) * 64 * (size_t)n_exp; }
// Allows kernel f the dynamic LDS of a split launch.
inline hipError_t stack_split_attr(const void* f, size_t lds) {
  return lds > 65536 ? hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) : hipSuccess;
}
inline int stack_split(const StackArgs& a) {
  constexpr int64_t CUS = 256, LDS = 156 * 1024;
  const int64_t per_cu = (a.n + 64 * CUS - 1) / (64 * CUS);
  if (a.work || a.n_exp < 2 || per_cu > 3 || per_cu * (int64_t)(stack_split_lds(a.n_exp) + 4096) > LDS) return 0;
  return per_cu == 1 ? 8 : 4;
}

// The stack: the checkpoint walk (then, when a.defer_list is set, the
// per-sample walk of the wavefronts it deferred), or the per-sample walk for
// an unbounded observer speed.
hipError_t launch_stack(const StackArgs& a, hipStream_t s);
hipError_t launch_zero_u32(unsigned int* p, hipStream_t s);
hipError_t launch_batched(const StackArgs* d_descs, const WorkItem* d_items, int n_items, unsigned int* d_counter,
                          int n_wg, hipStream_t s);
hipError_t launch_debug(const StackArgs& a, const DebugArgs& d, hipStream_t s);
// The same table from the walk launch_stack runs on this patch (solved samples only).
hipError_t launch_debug_stack(const StackArgs& a, const DebugArgs& d, hipStream_t s);
hipError_t launch_validate(const StackArgs& a, unsigned long long* d_bad, hipStream_t s);

// BF16 GEMM C = op(A) op(B) (+ bias, ReLU) with FP32 accumulation; op(A) is
// M x K (A stored [K x M] when transA), op(B) is K x N (B stored [N x K] when
// transB).  d_part is split-K scratch of part_elems floats.
struct GemmArgs {
  const uint16_t* A;
  int lda, transA;
  const uint16_t* B;
  int ldb, transB;
  int M, N, K;
  const float* bias;
  int relu;
  float* Cf;
  int ldcf;
};
hipError_t launch_gemm_bf16(const GemmArgs& g, float* d_part, size_t part_elems, hipStream_t s);
hipError_t launch_init_params(float* w, int64_t off, int64_t n, int fan_in, uint64_t seed, int is_bias,
                              hipStream_t s);

// Training path of the cell scorer (any output of the backward pass may be
// null in a forward pass).
// BF16 weights in fragments: 512 weights, eight consecutive K of row lane & 15
// for each lane in turn (K 8 (lane >> 4) ..).  Forward (rows = output
// channels): layer l from F<l>, row tile by row tile, K steps of 32 (padded
// with zeros).  Back (rows = inputs, K = outputs): layer l from G<l>;
// convolutions tap by tap, row tile by row tile.
constexpr int SCORER_FRAG = 512;
constexpr int SCORER_F1 = 0, SCORER_F2 = SCORER_F1 + SCORER_FRAG, SCORER_F3 = SCORER_F2 + 10 * SCORER_FRAG,
              SCORER_F4 = SCORER_F3 + 18 * SCORER_FRAG, SCORER_F5 = SCORER_F4 + 144 * SCORER_FRAG,
              SCORER_F6 = SCORER_F5 + 4 * SCORER_FRAG, SCORER_F7 = SCORER_F6 + 16 * SCORER_FRAG,
              SCORER_G2 = SCORER_F7 + 2 * SCORER_FRAG, SCORER_G3 = SCORER_G2 + 9 * SCORER_FRAG,
              SCORER_G4 = SCORER_G3 + 18 * SCORER_FRAG, SCORER_G6 = SCORER_G4 + 144 * SCORER_FRAG,
              SCORER_FRAGS = SCORER_G6 + 16 * SCORER_FRAG;
constexpr int TRAIN_RECORD = 14336;  // floats of one workgroup's gradient record (14 306 used, whole 128-byte lines)
struct TrainArgs {
  const uint16_t* stamps;  // B x 441 BF16
  const uint16_t* feats;   // B x 16 BF16
  const float* labels;     // B
  int B;
  int splits;              // partial sums of the 1152-deep layer (1, 2 or 4)
  const float* w;          // FP32 parameters (the biases are read here)
  const uint16_t* wf;      // BF16 weights, SCORER_FRAGS
  float* z;                // B logits
  uint16_t *h3, *ft, *cat;  // inputs of the fully connected layers, B x 1152, 16, 128
  uint16_t *d4, *d5, *d6;   // their output deltas, B x 64 each
  float* records;          // train_groups(B) x TRAIN_RECORD
};
struct AdamArgs {
  float *w, *m, *v;
  uint16_t* wf;
  float lr, b1, b2, eps, c1, c2;
};
int train_groups(int B);
int train_splits(int B);
hipError_t launch_train_forward(const TrainArgs& a, hipStream_t s);
// step: apply Adam instead of writing grad.
hipError_t launch_train_grad(const TrainArgs& a, float* loss, float* grad, const AdamArgs* step, hipStream_t s);
// BF16 copies of the parameters w, SCORER_FRAGS (the padding stays as it is: zero).
hipError_t launch_scorer_weights(const float* w, uint16_t* wf, hipStream_t s);

// Coarse stamps (21 x 21) and 16 features per representative orbit; d_track
// is n x n_exp int2 scratch.  Any output may be null.
constexpr int STAMP_MAX_EXP = 1024;  // the stamps keep three walks of every exposure in LDS
hipError_t launch_cell_stamps(const StackArgs& reps, double da, double dm, uint16_t* st_bf, float* st_f,
                              uint16_t* ft_bf, float* ft_f, hipStream_t s);
hipError_t launch_segment_max(const float* x, int64_t n_seg, int seg, float* out, hipStream_t s);
hipError_t launch_cell_members_near(const StackArgs& a, const int64_t* d_cells, int64_t n_sel, int cell_size,
                                    const float* d_uv, int uv_stride, double da, double dm, double radius,
                                    int64_t* d_ids, int64_t* d_count, hipStream_t s);
// Id lists whose count (read on the device) is at most STACK_IDS_SHORT are
// walked per sample with the exposures split over eight wavefronts per 64
// orbits (latency-bound sizes); longer ones by the checkpoint walk with
// deferral.  Both kernels are launched when m_max exceeds STACK_IDS_SHORT;
// the one not meant for the count returns at once.
constexpr int64_t STACK_IDS_SHORT = (int64_t)1 << 17;
hipError_t launch_stack_ids(const StackArgs& a, const int64_t* d_ids, const int64_t* d_count, int64_t m_max,
                            hipStream_t s);
hipError_t launch_stack_cells(const StackArgs& a, const int64_t* d_cells, int64_t n_sel, int cell_size,
                              hipStream_t s);

// Outlier trimming of m candidate orbits (n_exp <= 512).
hipError_t launch_clip(const StackArgs& a, const int64_t* d_ids, int64_t m, double kappa, int max_iter, float* snr,
                       float* flux, int32_t* nkept, hipStream_t s);

// Fused inference forward of the cell scorer.
struct ScorerFusedArgs {
  const uint16_t* stamps;  // B x 441 BF16
  const uint16_t* feats;   // B x 16 BF16
  int B;
  const uint16_t* wf;      // BF16 weights, SCORER_FRAGS
  const float* w;          // FP32 master parameters (the biases are read here)
  int64_t b_off[7];
  float* z;                // B logits
  const int64_t* rows;     // NULL, or cell i of the batch is row rows[i] of stamps / feats and of z
};
// Top-k of many S/N arrays at once (device tables, one entry per array or
// per TOPK tile; see launch_topk_segmented).
struct SegTopkArgs {
  const float* const* snr;    // [arrays]
  const int64_t* n;           // [arrays]
  const int64_t* tile_first;  // [arrays + 1] first tile of each array
  const int32_t* tile_patch;  // [tiles] array of each tile
  uint64_t* keys;             // [tiles * k] scratch
  float thr;
  int32_t k;
  int64_t* idx;               // [arrays * k]
  float* val;                 // [arrays * k]
  int32_t* cnt;               // [arrays]
};
int64_t topk_seg_tile();      // keys per tile
int64_t topk_seg_max_keys();  // largest k * tiles of one array
hipError_t launch_topk_segmented(const SegTopkArgs& a, int n_tiles, int n_arrays, hipStream_t s);

hipError_t launch_scorer_fused(const ScorerFusedArgs& a, hipStream_t s);

// Replay of a recorded gather stream (measurement yardstick).
hipError_t launch_record_gathers(const StackArgs& a, int64_t* cnt, const int64_t* gstart, int64_t* list,
                                 hipStream_t s);
hipError_t launch_gather_replay(const float2* planes, const int64_t* gstart, const int64_t* list, int64_t n,
                                float* snr, hipStream_t s);

// Per-image iterated-MAD noise.
constexpr double NOISE_KAPPA = 3.0;   // clip half-width in sigma (patches without variance planes)
constexpr int NOISE_MAX_ITER = 10;
size_t noise_scratch_bytes(int n_img);
// Where the scratch holds the number (uint32) of images solved from their pixels.
size_t noise_pixels_offset();
hipError_t launch_noise(const void* const* d_imgs, const int64_t* d_npix, int64_t max_pix, int n_img, dt_dtype dtype,
                        double kappa, int max_iter, void* scratch, double* d_sigma, int64_t* d_used, int32_t* d_iters,
                        ExpMeta* d_meta, hipStream_t s);

// Device-side orbit sampling (GenerateOrbits) and generate-and-stack.
hipError_t launch_generate(const dt_orbit_sampler& S, int64_t first, int64_t n, double* a, double* e, double* inc,
                           double* node, double* peri, double* m0, hipStream_t s);
hipError_t launch_stack_generated(const StackArgs& a, const dt_orbit_sampler& S, int64_t first, hipStream_t s);
// Per-sample walk of every generated orbit (no checkpoint kernel, no list).
hipError_t launch_stack_generated_walk(const StackArgs& a, const dt_orbit_sampler& S, int64_t first, hipStream_t s);


// Resolves, with `device` current, the device address of the allocation-free
// top-k's fixed scratch array (once per device).
hipError_t topk_noalloc_setup(int device);
// Top-k scratch requirement (bytes) for n inputs and k outputs.
size_t topk_scratch_bytes(int64_t n, int32_t k);
// ordered false: inputs of at most 16384 keys skip the final sort (the
// selection is the same; larger inputs come out sorted either way).
hipError_t launch_topk(const float* d_snr, int64_t n, int32_t k, float thr, int64_t* d_idx, float* d_val,
                       int32_t* d_count, void* d_scratch, hipStream_t s, bool ordered = true);

}  // namespace dtk
