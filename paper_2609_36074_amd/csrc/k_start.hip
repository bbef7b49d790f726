// Data-informed starting factor (Appendix D, "Initialization") for gfx950.
//
// The randomized range finder on the Gram matrix of the normalised data,
//     V = Xhat Xhat^T Z,   V = Q R,   U_0 = Pi_Omega(Q),
// with the QR taken as the appendix's Cholesky QR in feature space:
//     M = Xhat^T Z (d x r),  C = Xhat^T Xhat (d x d, reused from the spectral
//     normalisation),  V^T V = M^T C M = R^T R,  Q = Xhat (M R^{-1}).
// M comes from one Theta product of pass A over (Xhat, Z); the d x r and r x r algebra runs in
// FP64 on the fp64 matrix cores in 64 x 64 blocks spread over workgroups (one workgroup with
// scalar FMAs: 113 ms at 768 x 256; in blocks: under 1 ms); Q = Xhat T is one more pass over
// Xhat, written over Z, after which the usual projection onto Omega follows.  A pivot that is
// not above 1e-14 of its diagonal entry (V numerically rank deficient) marks the control block
// degenerate.
#include "k_common.hpp"

namespace nlr {

constexpr int kStartLd = 65;  // LDS row stride (doubles) of the 64 x 64 blocks

__global__ void k_start_prep(Bufs B, int r32) {
  for (int c = threadIdx.x; c < r32; c += blockDim.x) B.p[c] = 0.f;  // pass A reads p for its row work
}

// C / a^2 = Xhat^T Xhat from the centred Gram matrix of the normalisation.
__global__ __launch_bounds__(kThreads) void k_start_copy_c(Geometry g, Bufs B) {
  const double a = B.ctl->spectral_a;
  const double s = 1.0 / (a * a);
  const int64_t dd = (int64_t)g.d * g.d;
  for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < dd; e += (int64_t)gridDim.x * kThreads)
    B.s_C[e] = B.i_C[e] * s;
}

__global__ void k_start_zero_xbar(Geometry g, Bufs B) {
  for (int f = threadIdx.x; f < g.d; f += blockDim.x) B.i_xbar[f] = 0.0;
}

// M[f][c] = sum of the Theta partials (fixed order), FP64.
__global__ __launch_bounds__(kRedThreads) void k_start_m(Geometry g, Bufs B) {
  __shared__ double red[kRedThreads];
  const int64_t e = (int64_t)blockIdx.x * 64 + (threadIdx.x & 63);  // d32 r32 is a multiple of 1024
  const double sum = part_sum64(B.theta_part, g.GA, g.theta_cols, e, red);
  const int f = (int)(e / g.r32), c = (int)(e % g.r32);
  if (threadIdx.x < 64 && f < g.d && c < g.r) B.s_M[(int64_t)f * g.r + c] = sum;
}

// out = A^T Bm (A k x m, Bm k x n, row-major): 64 x 64 blocks, workgroup (column, row block).  Operands
// are read from L2 in whole 128-byte pieces, eight steps in flight.
__global__ __launch_bounds__(kThreads) void k_start_gemm(const double* __restrict__ A, const double* __restrict__ Bm,
                                                         double* __restrict__ out, int m, int n, int kk) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, kq = lane >> 4, cl = lane & 15;
  const int i0 = 64 * blockIdx.y + 16 * w + cl, j0 = 64 * blockIdx.x + cl;
  const bool oki = i0 < m;
  f64x4 acc[4];
  mm64_zero(acc);
  mm64<8>((kk + 3) / 4,
          [&](int k0) {
            const int k = k0 + kq;
            const double v = A[(int64_t)(k < kk ? k : kk - 1) * m + (oki ? i0 : 0)];
            return (k < kk && oki) ? v : 0.0;
          },
          [&](int k0, int J) {
            const int k = k0 + kq, j = j0 + 16 * J;
            const double v = Bm[(int64_t)(k < kk ? k : kk - 1) * n + (j < n ? j : 0)];
            return (k < kk && j < n) ? v : 0.0;
          },
          acc);
#pragma unroll
  for (int J = 0; J < 4; ++J)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = 64 * blockIdx.y + 16 * w + 4 * v + kq, j = j0 + 16 * J;
      if (i < m && j < n) out[(int64_t)i * n + j] = acc[J][v];
    }
}

// S -= R R_J^T over the columns before block J: R the rows (of stride r) of this 64-row block, R_J
// those of block row J of L; rows at or beyond `rows` count as zero.
__device__ __forceinline__ void start_update(const double* __restrict__ R, int rows, const double* __restrict__ Lj,
                                             int jrows, int r, int J, double* S) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, kq = lane >> 4, cl = lane & 15;
  const int i = 16 * w + cl;
  f64x4 acc[4];
  mm64_zero(acc);
  mm64<8>(16 * J, [&](int k0) { return i < rows ? R[(int64_t)i * r + k0 + kq] : 0.0; },
          [&](int k0, int Jc) { return 16 * Jc + cl < jrows ? Lj[(int64_t)(16 * Jc + cl) * r + k0 + kq] : 0.0; }, acc);
#pragma unroll
  for (int Jc = 0; Jc < 4; ++Jc)
#pragma unroll
    for (int v = 0; v < 4; ++v) S[(16 * w + 4 * v + kq) * kStartLd + 16 * Jc + cl] -= acc[Jc][v];
}

// Diagonal block J of the Cholesky factorisation G = L L^T, in place (one workgroup, 64 x 64 in
// LDS): G_JJ less the products of the blocks before it, then one column a step -- the trailing
// block takes S_ij S_kj / s_jj, and L_ij = S_ij / sqrt(s_jj) at the end, so that a step needs one
// barrier.
__global__ __launch_bounds__(kThreads) void k_start_diag(Geometry g, Bufs B, int J) {
  __shared__ double S[64 * kStartLd];
  __shared__ double g0[64], piv[64];
  const int tid = threadIdx.x, r = g.r, nr = r - 64 * J < 64 ? r - 64 * J : 64;
  double* G = B.s_G + (int64_t)64 * J * r;
  for (int e = tid; e < 64 * 64; e += kThreads) {
    const int i = e >> 6, j = e & 63;
    const double v = (i < nr && j < nr) ? G[(int64_t)i * r + 64 * J + j] : (i == j ? 1.0 : 0.0);
    S[i * kStartLd + j] = v;
    if (i == j) g0[i] = v;
  }
  __syncthreads();
  start_update(G, nr, G, nr, r, J, S);
  __syncthreads();
  bool bad = false;
  for (int j = 0; j < nr; ++j) {
    const double s = S[j * kStartLd + j];
    // a pivot at rounding level of the diagonal means V has (numerically) dependent columns
    if (!(s > 1e-14 * g0[j]) || !isfinite(s)) bad = true;
    const double inv = s > 0.0 ? 1.0 / s : 1.0;
    if (tid == 0) piv[j] = s > 0.0 ? sqrt(s) : 1.0;
    const int k = tid & 63;
    if (k > j) {
      const double skj = S[k * kStartLd + j] * inv;
      for (int i = tid >> 6; i < nr; i += kThreads / 64)
        if (i >= k) S[i * kStartLd + k] -= S[i * kStartLd + j] * skj;
    }
    __syncthreads();
  }
  for (int e = tid; e < 64 * 64; e += kThreads) {
    const int i = e >> 6, j = e & 63;
    if (i < nr && j <= i) G[(int64_t)i * r + 64 * J + j] = i == j ? piv[j] : S[i * kStartLd + j] / piv[j];
  }
  if (tid == 0 && bad) B.ctl->degenerate = 1;
}

// The blocks below diagonal block J and block column J of T = M L^{-T}, which is the same
// recurrence: R_J = (A_J - sum_{K<J} R_K L_JK^T) L_JJ^{-T}.  Workgroups take 64 rows each: first the
// rows of G below block J (A in place), then all rows of M (R to s_T).
constexpr size_t kPanelStartLds = (64 * kStartLd + 64 * 64) * sizeof(double);
__global__ __launch_bounds__(kThreads) void k_start_panel(Geometry g, Bufs B, int J) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* S = reinterpret_cast<double*>(smem_raw);
  double* Lj = S + 64 * kStartLd;
  const int tid = threadIdx.x, r = g.r, nr = r - 64 * J < 64 ? r - 64 * J : 64;
  const int below = (r + 63) / 64 - J - 1;
  const bool isG = (int)blockIdx.x < below;
  const int row0 = 64 * (isG ? J + 1 + (int)blockIdx.x : (int)blockIdx.x - below);
  const int total = isG ? r : g.d;
  const int rows = total - row0 < 64 ? total - row0 : 64;
  const double* src = (isG ? B.s_G : B.s_M) + (int64_t)row0 * r;
  double* dst = (isG ? B.s_G : B.s_T) + (int64_t)row0 * r;
  const double* GJ = B.s_G + (int64_t)64 * J * r;
  for (int e = tid; e < 64 * 64; e += kThreads) {
    const int i = e >> 6, j = e & 63;
    S[i * kStartLd + j] = (i < rows && j < nr) ? src[(int64_t)i * r + 64 * J + j] : 0.0;
    Lj[e] = (i < nr && j <= i) ? GJ[(int64_t)i * r + 64 * J + j] : 0.0;
  }
  __syncthreads();
  start_update(dst, rows, GJ, nr, r, J, S);
  __syncthreads();
  // forward substitution, right-looking: thread (row i, quarter q) keeps the row's x_j in LDS
  const int i = tid & 63, q = tid >> 6;
  for (int j = 0; j < nr; ++j) {
    const double x = S[i * kStartLd + j] / Lj[j * 64 + j];
    for (int k = j + 1 + q; k < nr; k += kThreads / 64) S[i * kStartLd + k] -= x * Lj[k * 64 + j];
    __syncthreads();
  }
  for (int e = tid; e < 64 * 64; e += kThreads) {
    const int ii = e >> 6, j = e & 63;
    if (ii < rows && j < nr) dst[(int64_t)ii * r + 64 * J + j] = S[ii * kStartLd + j] / Lj[j * 64 + j];
  }
}

// U = Xhat T (FP64 products and sums, rounded once), on the fp64 matrix cores.  A wave takes 64 rows
// (four groups of 16) x CT tiles of 16 columns; a step's 4 features are 16 q + 4 (l / 16) + s for
// s = 0..3, so a lane reads 16 consecutive bytes of its row of Xhat, two chunks of 16 features
// ahead; the chunk's rows of T pass through LDS (one of two buffers, shared by the four waves, a
// chunk ahead), read in the four rotations of the 4x4x4 form.  Loads complete in order, so T's are
// issued before Xhat's: with T read by each wave between the products, every chunk waited for
// Xhat's HBM latency (matrix cores 42% busy, 24 ms at 2e6 x 768 x 256).  Column groups of 64 of the
// same rows are workgroups 8 apart (one XCD), so that Xhat comes from HBM about once.  Bound by the
// matrix cores: 2 n d r flops.
template <int CT, bool VEC>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_start_apply(Geometry g, Bufs B,
                                                                                                     int cgroups) {
  if (B.ctl->degenerate) return;
  __shared__ double ts[2][16][16 * CT + 4];  // rows 4 apart (lanes 16 apart) on the other half of the banks
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, lg = lane >> 4, lr = lane & 15;
  const int d = g.d, r = g.r;
  const int64_t n = g.n;
  const int64_t per = (int64_t)8 * cgroups, id = blockIdx.x;
  const int64_t tile = id / per * 8 + id % per % 8;
  const int cg = (int)(id % per / 8);
  const int64_t row0 = tile * 256 + 64 * w;
  if (tile * 256 >= n) return;
  const float* xp[4];
#pragma unroll
  for (int gq = 0; gq < 4; ++gq) {
    const int64_t row = row0 + 16 * gq + lr;
    xp[gq] = B.X + (row < n ? row : n - 1) * d;
  }
  double acc[4][CT][4];
#pragma unroll
  for (int gq = 0; gq < 4; ++gq)
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
      for (int R = 0; R < 4; ++R) acc[gq][t][R] = 0.0;
  auto load_x = [&](int q, float (&x)[4][4]) {
    const int c0 = 16 * q + 4 * lg;
#pragma unroll
    for (int gq = 0; gq < 4; ++gq) {
      if constexpr (VEC) {
        const f32x4 t = *reinterpret_cast<const f32x4*>(xp[gq] + (c0 < d ? c0 : 0));
#pragma unroll
        for (int s = 0; s < 4; ++s) x[gq][s] = t[s];
      } else {
#pragma unroll
        for (int s = 0; s < 4; ++s) x[gq][s] = xp[gq][c0 + s < d ? c0 + s : 0];
      }
    }
  };
  // CT elements of the chunk's 16 x 16 CT of T a thread; features beyond d are zero (what Xhat's
  // clamped loads hold there does not matter), columns beyond r are not stored
  double tn[CT];
  auto load_t = [&](int q) {
#pragma unroll
    for (int u = 0; u < CT; ++u) {
      const int e = tid + u * kThreads, f = 16 * q + e / (16 * CT), c = 64 * cg + e % (16 * CT);
      const double v = B.s_T[(int64_t)(f < d ? f : 0) * r + (c < r ? c : 0)];
      tn[u] = f < d ? v : 0.0;
    }
  };
  auto put_t = [&](int b) {
#pragma unroll
    for (int u = 0; u < CT; ++u) {
      const int e = tid + u * kThreads;
      ts[b][e / (16 * CT)][e % (16 * CT)] = tn[u];
    }
  };
  const int nq = (d + 15) >> 4;
  float x0[4][4], x1[4][4];
  load_t(0);
  load_x(0, x0);
  load_x(nq > 1 ? 1 : 0, x1);
  put_t(0);
  __syncthreads();
  // chunk q from xc; afterwards xc holds chunk q + 2
  auto chunk = [&](int q, float (&xc)[4][4]) {
    double a[4][4];
#pragma unroll
    for (int gq = 0; gq < 4; ++gq)
#pragma unroll
      for (int s = 0; s < 4; ++s) a[gq][s] = (double)xc[gq][s];
    if (q + 1 < nq) load_t(q + 1);
    if (q + 2 < nq) load_x(q + 2, xc);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int t = 0; t < CT; ++t)
#pragma unroll
        for (int R = 0; R < 4; ++R) {
          const double b = ts[q & 1][4 * lg + s][16 * t + ((lr + 4 * R) & 15)];
#pragma unroll
          for (int gq = 0; gq < 4; ++gq) acc[gq][t][R] = mfma4x4x4d(a[gq][s], b, acc[gq][t][R]);
        }
    if (q + 1 < nq) put_t((q + 1) & 1);
    __syncthreads();
  };
  for (int q = 0; q < nq; q += 2) {
    chunk(q, x0);
    if (q + 1 < nq) chunk(q + 1, x1);
  }
  const int bl = (lane >> 2) & 3;
#pragma unroll
  for (int gq = 0; gq < 4; ++gq) {
    const int64_t row = row0 + 16 * gq + 4 * bl + lg;
    if (row < n)
#pragma unroll
      for (int t = 0; t < CT; ++t)
#pragma unroll
        for (int R = 0; R < 4; ++R) {
          const int c = 64 * cg + 16 * t + 4 * ((bl + R) & 3) + (lane & 3);
          if (c < r) B.U[row * r + c] = (float)acc[gq][t][R];
        }
  }
}

template <int CT>
static hipError_t start_apply(const Geometry& g, const Bufs& b, hipStream_t st) {
  const int cgroups = (g.r + 63) / 64;
  const int64_t tiles = ((g.n + 255) / 256 + 7) / 8 * 8;
  const int64_t blocks = tiles * cgroups;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  if (g.vec_x)
    hipLaunchKernelGGL((k_start_apply<CT, true>), dim3((unsigned)blocks), dim3(kThreads), 0, st, g, b, cgroups);
  else
    hipLaunchKernelGGL((k_start_apply<CT, false>), dim3((unsigned)blocks), dim3(kThreads), 0, st, g, b, cgroups);
  return hipGetLastError();
}

hipError_t launch_data_start(const Geometry& g, const Bufs& b, const StepArgs& a0, bool x_normalised,
                             hipStream_t st) {
  hipError_t e;
  if (x_normalised) {
    // C = Xhat^T Xhat from the given Xhat (no re-centring)
    hipLaunchKernelGGL(k_start_zero_xbar, dim3(1), dim3(kThreads), 0, st, g, b);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = launch_gram(g, b, st)) != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_start_copy_c, dim3(64), dim3(kThreads), 0, st, g, b);
  hipLaunchKernelGGL(k_start_prep, dim3(1), dim3(kThreads), 0, st, b, g.r32);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // M = Xhat^T Z: the pass-A product with U = Z (c_f = 1)
  if ((e = launch_pass_a(g, b, a0, false, st)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_start_m, dim3(g.RT), dim3(kRedThreads), 0, st, g, b);
  // C M (C is symmetric) and M^T (C M)
  const int rb = (g.r + 63) / 64, db = (g.d + 63) / 64;
  hipLaunchKernelGGL(k_start_gemm, dim3(rb, db), dim3(kThreads), 0, st, (const double*)b.s_C, (const double*)b.s_M,
                     b.s_CM, g.d, g.r, g.d);
  hipLaunchKernelGGL(k_start_gemm, dim3(rb, rb), dim3(kThreads), 0, st, (const double*)b.s_M, (const double*)b.s_CM,
                     b.s_G, g.r, g.r, g.d);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_start_panel), hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)kPanelStartLds);
  if (e != hipSuccess) return e;
  for (int J = 0; J < rb; ++J) {
    hipLaunchKernelGGL(k_start_diag, dim3(1), dim3(kThreads), 0, st, g, b, J);
    hipLaunchKernelGGL(k_start_panel, dim3(rb - J - 1 + db), dim3(kThreads), kPanelStartLds, st, g, b, J);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  switch (g.r > 48 ? 4 : (g.r + 15) / 16) {
    case 1: return start_apply<1>(g, b, st);
    case 2: return start_apply<2>(g, b, st);
    case 3: return start_apply<3>(g, b, st);
    default: return start_apply<4>(g, b, st);
  }
}

}  // namespace nlr
