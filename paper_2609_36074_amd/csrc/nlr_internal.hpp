// Internal declarations shared by the host controller and the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "nlr.h"

namespace nlr {

constexpr int kThreads = 256;     // threads of a workgroup (4 wave64), where a kernel has no number of its own
constexpr int kHistCap = 4096;    // per-iteration record ring
constexpr int kTPA = 64;          // rows per pass-A tile
constexpr int kTPB = 128;         // rows per pass-B super-tile (4 waves x 32 rows)
constexpr int kMaxR = 448;        // largest supported rank (fp32 two-pass form above 256)
constexpr int kMaxPanelR = 256;   // largest rank of the split-fp16 panel form
constexpr int kPowerIters = 16;   // refinement power iterations after the squaring phase
constexpr int kSquarings = 20;    // C -> C^(2^20) before the refinement

// DevCtl::breakdown values besides 0: the normalisation breakdown of Algorithm 1,
// and a split-fp16 operand of W out of fp16's range (both stop the iteration, U then
// holds W).
constexpr int32_t kBreakdown = 1;
constexpr int32_t kRangeError = 2;

// Device control block, read uniformly by every kernel at entry.  A launch writes it from one
// workgroup at most: workgroup 0 of the controls (of several workgroups themselves, so what one of
// them tests at entry and workgroup 0 sets is read once a workgroup), of the initialisation's and
// the panel form's small kernels.
struct alignas(16) DevCtl {
  int32_t stop;        // stopping rule fired during the current host call: 1, two-pass forms 2 from the next control on
  int32_t breakdown;   // sticky: kBreakdown (normalisation breakdown) or kRangeError
  int32_t gate;        // dual gate of the latest primal step
  int32_t degenerate;  // init: a = ||X_c||_2 is zero or not finite
  int64_t t_done;      // completed primal steps
  int64_t rows_run;    // one-pass iterations whose row work ran in its own pass first
  float c_f;           // lazy scale of the factor buffer (1 when materialised)
  float x_scale;       // power of two keeping |Xhat| x_scale < 2^15 (split-fp16 products)
  float th_scale;      // power of two keeping |Theta| th_scale < 2^15 (panel pass B operand)
  int32_t rows_first;  // one-pass iteration: the row pass runs before the pass -- 1 the stop may
                       // fire (s from the Gram terms), 2 no Gram terms yet (s from the rows)
  double a, b, h;      // fused statistics of the latest primal step
  double Delta;        // squared movement estimate
  double delta;        // movement estimate
  double rho;          // ||q||/sqrt(n) of the current factor
  double objective;    // fhat at the start of the latest iteration
  double theta_fro2;
  double spectral_a;   // ||X_c||_2
  double c_gram;       // scale c of the factor whose Gram terms are stored (one-pass iteration)
};

// Scalars of one iteration, passed by value.
struct StepArgs {
  float alpha_f;       // alpha
  float two_alpha_f;   // 2 alpha
  float gamma_f;       // beta / n (the implementation's penalty on the stored dual)
  float pad;
  double beta;
  double eps_d;
  double eps_c;
  double K;
  double inv_n;
  int64_t T_min;
  int32_t end_work;    // apply the pending end-of-iteration vector work (dual step, rho, stop test)
  int32_t pad32;
};

// Launch geometry; a pure function of (n, d, r) so that reduction orders,
// and therefore results, do not depend on the device.
struct Geometry {
  int64_t n;
  int32_t d, r, K;
  int32_t d32, r32;     // d, r rounded up to multiples of 32
  int32_t MB, NB;       // 32-wide blocks of d and r
  // pass A
  int32_t MBG, NBG;     // m-blocks (1, 2 or 4) / n-blocks (1, 2, 4, 5 or 7) per workgroup group
  int32_t mgroups, ngroups;
  int32_t GA;           // row-chunk workgroups per group
  int64_t tilesA;       // ceil(n / kTPA)
  int32_t a_rows;       // 1: register-resident pass A (k_pass_a_rows)
  int32_t a_un;         // 1: with rows of X or U that are not whole 16-byte pieces
  int32_t a_fv, a_ngf, a_cv;  // its features per lane, feature groups, columns per lane
  int32_t RT;           // workgroups of the Theta sum (64 entries each)
  // pass B
  int32_t GB;
  int64_t tilesB;       // ceil(n / kTPB)
  int32_t nch;          // 32-feature chunks of d
  int32_t theta_lds;    // 1: Theta staged whole in LDS
  int32_t b_res;        // 1: resident-tile pass B (k_pass_b_res)
  int32_t split_a, split_b;  // 1: split-fp16 products in pass A / pass B
  int32_t fused;        // 1: single-Xhat-pass iteration (row pass + fused pass B)
  int32_t uflat;        // 1: the fused pass B moves U as whole 32-row slabs (r % 4 != 0)
  int32_t fused8;       // 1: the fused pass B in its eight-wave form (k_pass_bf8), one-pass iteration
  int32_t theta_cols;   // floats per row of the Theta partials: d32 r32 (+ r32 r32 of W^T W, one-pass)
  int32_t ldsB_bytes;
  // init
  int32_t GI;           // row-chunk workgroups of the init reductions
  int32_t GG;           // row-chunk workgroups of the Gram partials
  int32_t vec_x, vec_u; // 16-byte vector loads allowed on X / U rows
  int32_t GAF;          // workgroups of the finish pass (generic pass A form)
  // split-fp16 panel form (large d x r, two passes)
  int32_t panel;        // 1: k_pass_a_panel / k_pass_b_panel iteration
  int32_t pnbw;         // 32-column blocks per column wave (1, 2 or 4): 64 pnbw columns
  int32_t pfb;          // 256-feature blocks of pass A
  int32_t PS;           // row splits of pass A
  int32_t GPA;          // pass A workgroups (PS pfb: groups of 8 splits on one XCD each, then the rest)
  int64_t tilesP;       // 128-row tiles of pass B
  float su;             // power-of-two scale of U in the split (|u| <= sqrt(K))
};

// Pointers into caller memory and the workspace.
struct Bufs {
  float* X;            // n x d (Xhat after init)
  float* U;            // n x r
  float* y;            // n (stored dual)
  DevCtl* ctl;
  nlr_iter_stats* hist;   // kHistCap records
  float* theta;        // d32*r32, pass-B operand layout
  float* p;            // r32
  float* s;            // r32
  float* theta_part;   // rows of theta_cols floats (GA, GB or PS rows)
  size_t union_bytes;  // bytes of the region it starts, which the init and the label recovery use too
  double* a_part;      // GA x (4 + r32): ||q||^2, ytilde^T q, -, -, s partials
  double* th2_part;    // RT
  double* b_part;      // GB x (4 + r32): a, b, h, -, column sums
  DevCtl* mirror;      // host memory that the control after a finish pass copies ctl to (or null)
  nlr_iter_stats* mirror_rec;  // and the latest iteration's record
  float* dump;         // 256 bytes that masked-off lanes store to (never read)
  float* thmax_part;   // RT: per-workgroup max |Theta| of the reduction
  float* ybar;         // n: ybar of the current iteration (panel form: pass A -> pass B)
  void* theta_split;   // panel form: split Theta^T chunks, 64 bytes per (16 features, column)
  // one-pass iteration (eight-wave fused pass B)
  double* gram_vec;    // 3 r32: column sums P of W, W^T ytilde, (W^T W) P (fixed-order sums)
  // init temporaries (alias the pass-A partial region)
  double* i_colsum;    // GI x d
  double* i_xbar;      // d
  double* i_gram;      // GG x d x d
  double* i_C;         // d x d
  double* i_B0;        // d x d
  double* i_B1;        // d x d
  double* i_scal;      // c of the projection
  double* i_trace;     // 2 x 64: traces of the squarings' diagonal blocks
  double* i_proj;      // GI x (4 + r32)
  // data-informed start (FP64, not aliased)
  double* s_C;         // d x d: Xhat^T Xhat
  double* s_M;         // d x r: Xhat^T Z
  double* s_CM;        // d x r
  double* s_G;         // r x r: M^T C M, then its Cholesky factor L (lower)
  double* s_T;         // d x r: M L^{-T}
};

// Scratch of the spectral label recovery (carved from the Theta-partial region,
// which is free between host calls).
constexpr int kLabMaxK = 128;
constexpr int kLabMaxSweeps = 60;   // Jacobi sweeps at most
constexpr int kLabJacParts = 32;    // partial sums of the off-diagonal mass (7 pivot + 21 other blocks at most)
struct LabScratch {
  int32_t GU;          // row chunks of the U^T U partials
  int32_t W;           // row chunks of the cluster sums
  int32_t r64;         // r rounded up to a multiple of 64: row stride of A and V
  double* gpart;       // GU x r x r (before the passes)
  long long* spart;    // W x K x r: integer cluster sums (same memory as gpart)
  int32_t* cpart;      // W x K: rows per cluster
  double* A;           // r64 x r64: U^T U, diagonalised in place
  double* V;           // r64 x r64: eigenvectors
  double* Q;           // 64 x 64 rotations of each pair of column blocks
  double* jpart;       // 2 kLabJacParts: squared off-diagonal, diagonal entries
  double* P;           // r x K: V_K Lambda_K^(-1/2)
  double* Pt;          // K x r: its transpose
  void* Mimg;          // P cent^T split in fp16 halves, in the assignment's operand order (r32 x K32)
  double* Mt;          // K x r: its transpose
  double* minv;        // K: inverse scale of a cluster's split column
  double* centT;       // K x K centroids, component-major
  double* cn;          // K: |cent_k|^2
  double* cscale;      // r: power-of-two scale of the integer sums
  double* cinv;        // r: its inverse
  double* ubound;      // r: bounds on |u| by column
  double* scal;        // 1 / sqrt(K-th eigenvalue), a bound on the norm of P; power-of-two scale of U
  unsigned long long* changed;  // labels changed by the pass
  int64_t* seeds;      // K seed rows
  int32_t* grp;        // K: first cluster with the same seed row
  int32_t* lead;       // K: first cluster whose centroid is equal by that (k itself: none before it)
  int32_t* flag;       // [0] degenerate spectrum, [1] iteration done, [2] passes, [3] Jacobi converged
};
size_t lab_scratch_bytes(int64_t n, int32_t r, int32_t K);
// region: bytes at base (lab_scratch_bytes or more)
LabScratch carve_lab_scratch(int64_t n, int32_t r, int32_t K, char* base, size_t region);

// aligned16: X and U start on 16-byte boundaries (enables the vector-load kernels)
// split: split-fp16 products requested (NLR_INIT_SPLIT_F16)
Geometry make_geometry(int64_t n, int32_t d, int32_t r, int32_t K, bool aligned16, bool split = false,
                       bool fused = false);
// dynamic LDS of the fused pass B for (NB, nch, split, U moved as whole slabs)
int fused_lds_need(int NB, int nch, bool split, bool uflat);
bool fused8_shape(int NB, int nch, int r);
// above 128 columns the row-work launch of pass A (GAF workgroups streaming rows of U) stores ybar
// for pass B
__host__ __device__ inline bool pass_a_split(const Geometry& g) { return !g.a_rows && g.r32 > 128; }
constexpr int kMaxFusedLds = 160 << 10;
size_t carve_workspace(const Geometry& g, char* base, Bufs* out);  // base may be null (size only)

// ---- kernel launchers (each returns the launch error) ----
hipError_t launch_ctl_init(const Bufs& b, float gamma_f, hipStream_t st);
hipError_t launch_clear_stop(const Bufs& b, hipStream_t st);
hipError_t launch_colsum(const Geometry& g, const Bufs& b, hipStream_t st);
hipError_t launch_gram(const Geometry& g, const Bufs& b, hipStream_t st);
// partials (one d x d array a row chunk) of (M - 1 mean^T)^T (M - 1 mean^T), blocks on and above
// the diagonal of 64 x 64 blocks; mean null: M^T M
hipError_t launch_gram_partials(const float* M, int64_t n, int d, const double* mean, double* part, int chunks,
                                hipStream_t st);
hipError_t launch_spectral(const Geometry& g, const Bufs& b, hipStream_t st);
hipError_t launch_normalise(const Geometry& g, const Bufs& b, hipStream_t st);
hipError_t launch_project(const Geometry& g, const Bufs& b, double K, int in_omega, hipStream_t st);
hipError_t launch_zero_y(const Geometry& g, const Bufs& b, hipStream_t st);

hipError_t launch_pass_a(const Geometry& g, const Bufs& b, const StepArgs& a, bool finish,
                         hipStream_t st);
hipError_t launch_pass_u(const Geometry& g, const Bufs& b, const StepArgs& a, hipStream_t st);
hipError_t launch_pass_bf(const Geometry& g, const Bufs& b, const StepArgs& a, hipStream_t st);
hipError_t launch_pass_b(const Geometry& g, const Bufs& b, const StepArgs& a, hipStream_t st);
// Theta from `rows` partial rows (scaled: Xhat^T W of the fused pass B, times c_f; gamma_f >= 0: the
// one-pass iteration's next s too), and with the control after pass A in the two-pass form
hipError_t launch_theta_sum(const Geometry& g, const Bufs& b, const StepArgs& a, int64_t rows, bool scaled,
                            float gamma_f, bool with_ctl_a, hipStream_t st);
// rows: a_part rows of the latest producer (pass A grid, finish grid or panel splits)
hipError_t launch_ctl_a(const Geometry& g, const Bufs& b, const StepArgs& a, int64_t rows, bool finish,
                        hipStream_t st);
// defer: ||Theta||_F^2 (formed with the control after pass A, in one launch) joins the objective here
hipError_t launch_ctl_b(const Geometry& g, const Bufs& b, const StepArgs& a, bool defer, hipStream_t st);
hipError_t launch_xscale(const Geometry& g, const Bufs& b, hipStream_t st);
hipError_t launch_split_x(const Geometry& g, const Bufs& b, hipStream_t st);
hipError_t launch_pass_b_split(const Geometry& g, const Bufs& b, const StepArgs& a, hipStream_t st);
hipError_t launch_data_start(const Geometry& g, const Bufs& b, const StepArgs& a0, bool x_normalised,
                             hipStream_t st);
// U^T U, `count` Jacobi sweeps from sweep `first` on (all of them up to 64 columns), the basis
// and the seed centroids, one assignment pass with its centroids
hipError_t launch_lab_gram(const Geometry& g, const Bufs& b, const LabScratch& L, hipStream_t st);
hipError_t launch_lab_sweeps(const LabScratch& L, int r, int first, int count, hipStream_t st);
hipError_t launch_lab_embed(const Geometry& g, const Bufs& b, const LabScratch& L, int K, hipStream_t st);
hipError_t launch_lab_pass(const Geometry& g, const Bufs& b, const LabScratch& L, int K, int32_t* labels,
                           hipStream_t st);
hipError_t launch_labels(const Geometry& g, const Bufs& b, int32_t* labels, hipStream_t st);
hipError_t launch_pass_a_panel(const Geometry& g, const Bufs& b, const StepArgs& a, hipStream_t st);
hipError_t launch_theta_split_panel(const Geometry& g, const Bufs& b, hipStream_t st);
hipError_t launch_pass_b_panel(const Geometry& g, const Bufs& b, const StepArgs& a, hipStream_t st);
hipError_t launch_split_x8(const Geometry& g, const Bufs& b, hipStream_t st);
hipError_t launch_ctl_one(const Geometry& g, const Bufs& b, const StepArgs& a, hipStream_t st);
// start of a host call of the one-pass iteration: s from the stored Gram terms (when
// valid) and whether the first iteration's row pass runs before its pass
hipError_t launch_onepass_begin(const Geometry& g, const Bufs& b, const StepArgs& a, bool gram_valid,
                                hipStream_t st);

// ---- device helpers ----
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// D += A * B on the 32x32x2 fp32 matrix core.  Lane l supplies A[l%32][l/32]
// and B[l/32][l%32]; lane l, register v of D holds D[8(v/4)+4(l/32)+v%4][l%32].
__device__ __forceinline__ f32x16 mfma32x32x2(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ double shfl_xor_d(double v, int mask) {
  return __shfl_xor(v, mask, 64);
}
__device__ __forceinline__ float shfl_xor_f(float v, int mask) {
  return __shfl_xor(v, mask, 64);
}

// Fixed-order sum of one double per thread over a 256-thread workgroup.
// Result valid in thread 0.  `red` must hold 4 doubles of shared memory.
__device__ __forceinline__ double block_sum_d(double v, double* red) {
  for (int m = 32; m >= 1; m >>= 1) v += shfl_xor_d(v, m);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0) r = ((red[0] + red[1]) + red[2]) + red[3];
  __syncthreads();
  return r;
}

}  // namespace nlr
