// Initialisation kernels for gfx950: centring and spectral normalisation
// (Section 3: X_c = X - 1 xbar^T, a = ||X_c||_2, Xhat = X_c / a), projection of
// the starting factor onto Omega (eq. projected-primal-step) and p = U^T 1.
//
// a is found as sqrt(lambda_max(C)) with C = X_c^T X_c (FP64), by the power
// method: C is first squared kSquarings times with trace normalisation
// (B_{k+1} = (B_k / tr B_k)^2, i.e. the power C^(2^k) up to scale), the column
// of the last B with the largest diagonal entry starts kPowerIters ordinary
// power iterations on C, and the Rayleigh quotient of the final unit vector is
// lambda_max.  Appendix D notes C is reused from this normalisation by the
// data-informed initialisation.
#include "k_common.hpp"

namespace nlr {

__global__ void k_ctl_init(Bufs B, float gamma_f) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    DevCtl* c = B.ctl;
    c->stop = 0;
    c->breakdown = 0;
    c->gate = 0;
    c->degenerate = 0;
    c->t_done = 0;
    c->c_f = 1.0f;
    c->x_scale = 1.0f;
    c->th_scale = 1.0f;
    c->rows_first = 0;
    c->rows_run = 0;
    c->a = c->b = c->h = 0.0;
    c->Delta = c->delta = 0.0;
    c->rho = c->objective = c->theta_fro2 = 0.0;
    c->spectral_a = 1.0;
    c->c_gram = 1.0;
  }
}

__global__ void k_clear_stop(Bufs B) {
  if (threadIdx.x == 0 && blockIdx.x == 0) B.ctl->stop = 0;
}

// Sum of p[k * stride] over k = first, first + step, ... below count, UN loads in flight, added in
// order.
template <int UN>
__device__ __forceinline__ double strided_sum(const double* __restrict__ p, int64_t stride, int first, int step,
                                              int count) {
  double t = 0.0;
  int k = first;
  for (; k + (UN - 1) * step < count; k += UN * step) {
    double v[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) v[u] = p[(int64_t)(k + u * step) * stride];
#pragma unroll
    for (int u = 0; u < UN; ++u) t += v[u];
  }
  for (; k < count; k += step) t += p[(int64_t)k * stride];
  return t;
}

// Column sums of X over row chunks (FP64).  Threads map to (column, row offset).
__global__ __launch_bounds__(kThreads) void k_colsum(Geometry g, Bufs B) {
  __shared__ double red[kThreads];
  const int tid = threadIdx.x;
  const int64_t n = g.n;
  const int d = g.d;
  const int64_t r0 = (int64_t)blockIdx.x * n / g.GI;
  const int64_t r1 = (int64_t)(blockIdx.x + 1) * n / g.GI;
  double* out = B.i_colsum + (int64_t)blockIdx.x * d;
  if (d <= kThreads) {
    const int rstep = kThreads / d;
    const int col = tid % d;
    const int rsub = tid / d;
    double acc = 0.0;
    if (rsub < rstep) {
      // sixteen rows' loads in flight, added in row order
      int64_t i = r0 + rsub;
      for (; i + 15 * rstep < r1; i += 16 * rstep) {
        float v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = B.X[(i + u * rstep) * d + col];
#pragma unroll
        for (int u = 0; u < 16; ++u) acc += (double)v[u];
      }
      for (; i < r1; i += rstep) acc += (double)B.X[i * d + col];
    }
    red[tid] = acc;
    __syncthreads();
    if (tid < d) {
      double t = 0.0;
      for (int k = 0; k < rstep; ++k) t += red[tid + k * d];
      out[tid] = t;
    }
  } else {
    for (int col = tid; col < d; col += kThreads) {
      double acc = 0.0;
      int64_t i = r0;
      for (; i + 7 < r1; i += 8) {  // eight rows' loads in flight, added in row order
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = B.X[(i + u) * d + col];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += (double)v[u];
      }
      for (; i < r1; ++i) acc += (double)B.X[i * d + col];
      out[col] = acc;
    }
  }
}

// Means from the chunk sums: 16 columns a workgroup, 16 groups of threads over the chunks (eight
// loads in flight), added in a fixed order.  One thread a column over all 512 chunks took 95 to
// 206 us, a dependent load at a time.
__global__ __launch_bounds__(kThreads) void k_colmean(Geometry g, Bufs B) {
  __shared__ double red[kThreads];
  const int tid = threadIdx.x, cl = tid & 15, gq = tid >> 4;
  const int j = blockIdx.x * 16 + cl;
  red[tid] = j < g.d ? strided_sum<8>(B.i_colsum + j, g.d, gq, 16, g.GI) : 0.0;
  __syncthreads();
  if (tid < 16 && j < g.d) {
    double t = 0.0;
    for (int k = 0; k < 16; ++k) t += red[16 * k + cl];
    B.i_xbar[j] = t / (double)g.n;
  }
}

// Partial centred Gram blocks on the fp64 matrix cores (v_mfma_f64_16x16x4f64):
// workgroup (chunk gx, block pair bp) adds the 64 x 64 block (bi, bj), bi <= bj, of
// the sum over the chunk's rows of (x - xbar)(x - xbar)^T.  Wave w owns the block
// rows 16 w .. 16 w + 15 and all 64 columns (four 16 x 16 tiles).  A product step
// takes 4 data rows: lane l reads row l / 16 of the step and feature l % 16 of its
// tile from LDS (the A operand from the block's rows, the B operands from its columns), and
// holds result element (4 v + l / 16, l % 16) of a tile in entry v.  The blocks
// below the diagonal are not formed (the sum is symmetric; k_gram_reduce reads
// their mirror).
static_assert(kThreads == 256, "k_gram stages a 32 x 64 operand as 8 elements per thread of 4 waves");
__global__ __launch_bounds__(kThreads) void k_gram(const float* __restrict__ M, int64_t n, int d,
                                                   const double* __restrict__ mean, double* __restrict__ part) {
  const int tid = threadIdx.x;
  const int nb = (d + 63) / 64;
  int bp = blockIdx.y, bi = 0;
  while (bp >= nb - bi) {
    bp -= nb - bi;
    ++bi;
  }
  const int bj = bi + bp;
  const int64_t r0 = (int64_t)blockIdx.x * n / gridDim.x;
  const int64_t r1 = (int64_t)(blockIdx.x + 1) * n / gridDim.x;
  const int lane = tid & 63, w = tid >> 6;
  const int kq = lane >> 4, cl = lane & 15;
  f64x4 acc[4];
#pragma unroll
  for (int J = 0; J < 4; ++J) acc[J] = (f64x4){0.0, 0.0, 0.0, 0.0};
  // Rounds of 32 rows.  The round's centred values of the block's 64 row features
  // and 64 column features are formed once in FP64 by the workgroup and staged in
  // LDS (rows padded to 80 doubles, so that the 32 lanes of a read pass meet all 64
  // banks); the next round's raw values are loaded while the matrix cores take this
  // round's.
  __shared__ double xs[2][32][80];
  const bool same = bi == bj;
  // element k = tid + 256 q (q = 0..7) of a 32 x 64 operand: row k / 64, feature k % 64
  const int sf = tid & 63, sr = tid >> 6;  // feature, first row (rows sr + 4 q)
  const int fsa = 64 * bi + sf, fsb = 64 * bj + sf;
  const bool oksa = fsa < d, oksb = fsb < d;
  const double msa = (oksa && mean) ? mean[fsa] : 0.0, msb = (oksb && mean) ? mean[fsb] : 0.0;
  float ra[8], rb[8];
  auto load_round = [&](int64_t t0) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int64_t row = t0 + sr + 4 * q;
      const int64_t rb0 = (row < r1 ? row : r0) * (int64_t)d;
      ra[q] = M[rb0 + (oksa ? fsa : 0)];
      rb[q] = same ? 0.f : M[rb0 + (oksb ? fsb : 0)];
    }
  };
  if (r0 < r1) load_round(r0);
  for (int64_t t0 = r0; t0 < r1; t0 += 32) {
    __syncthreads();  // the previous round's operands are consumed
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const bool okr = t0 + sr + 4 * q < r1;
      xs[0][sr + 4 * q][sf] = (okr && oksa) ? (double)ra[q] - msa : 0.0;
      if (!same) xs[1][sr + 4 * q][sf] = (okr && oksb) ? (double)rb[q] - msb : 0.0;
    }
    __syncthreads();
    if (t0 + 32 < r1) load_round(t0 + 32);
    const int ob = same ? 0 : 1;
#pragma unroll
    for (int st = 0; st < 8; ++st) {
      const int row = 4 * st + kq;
      const double a = xs[0][row][16 * w + cl];
#pragma unroll
      for (int J = 0; J < 4; ++J) {
        const double b = xs[ob][row][16 * J + cl];
        acc[J] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[J], 0, 0, 0);
      }
    }
  }
  double* out = part + (int64_t)blockIdx.x * d * d;
#pragma unroll
  for (int J = 0; J < 4; ++J)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int ia = 64 * bi + 16 * w + 4 * v + kq;
      const int jb = 64 * bj + 16 * J + cl;
      if (ia < d && jb < d) out[(int64_t)ia * d + jb] = acc[J][v];
    }
}

// C = the sum of the chunks' partials; entries below the block diagonal from the mirrored entry.
// Small matrices share an entry's chunks among 16 groups of threads (EPG = 16 entries a workgroup),
// added in a fixed order: one thread an entry left d = 32 on four workgroups with 256 dependent
// loads each (63 us).
template <int EPG>
__global__ __launch_bounds__(kThreads) void k_gram_reduce(Geometry g, Bufs B) {
  __shared__ double red[kThreads];
  constexpr int NG = kThreads / EPG;
  const int64_t dd = (int64_t)g.d * g.d;
  const int cl = threadIdx.x % EPG, gq = threadIdx.x / EPG;
  const int64_t e = (int64_t)blockIdx.x * EPG + cl;
  double t = 0.0;
  if (e < dd) {
    const int i = (int)(e / g.d), j = (int)(e - (int64_t)i * g.d);
    const int64_t src = (i / 64 > j / 64) ? (int64_t)j * g.d + i : e;
    t = strided_sum<8>(B.i_gram + src, dd, gq, NG, g.GG);
  }
  if constexpr (NG > 1) {
    red[threadIdx.x] = t;
    __syncthreads();
    if (gq == 0) {
      t = 0.0;
      for (int k = 0; k < NG; ++k) t += red[EPG * k + cl];
    }
  }
  if (gq == 0 && e < dd) B.i_C[e] = t;
}

// Up to 64 features: the whole power method in one workgroup of 16 waves, the matrix (zero padded to
// D = 16, 32 or 64) in LDS.  A squaring is one 16 x 16 tile a wave on the fp64 matrix cores (the
// matrix is symmetric, so both operands are read by rows), its trace summed on the way; then the
// power iterations on C, 16 threads a row.  As 20 squarings, 21 traces and the iteration in launches
// of their own: 210 us at d = 32, nearly all of it latency.
template <int D>
__global__ __launch_bounds__(1024) void k_power_small(Geometry g, Bufs B) {
  constexpr int LD = D + 2, NT = D / 16;
  __shared__ double C[D * LD], M[D * LD];
  __shared__ double v[D], y[D];
  __shared__ double sc;
  __shared__ int j0;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, d = g.d;
  for (int e = tid; e < D * D; e += 1024) {
    const int i = e / D, j = e % D;
    const double t = (i < d && j < d) ? B.i_C[i * d + j] : 0.0;
    C[i * LD + j] = t;
    M[i * LD + j] = t;
  }
  __syncthreads();
  for (int k = 0; k < kSquarings; ++k) {
    if (tid < 64) {
      double t = tid < D ? M[tid * LD + tid] : 0.0;
      for (int m = 32; m >= 1; m >>= 1) t += shfl_xor_d(t, m);
      if (tid == 0) sc = (t > 0.0 && isfinite(t)) ? 1.0 / t : 0.0;
    }
    __syncthreads();
    const double s = sc;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    const int ti = w / NT, tj = w % NT, kq = lane >> 4, cl = lane & 15;
    if (w < NT * NT)
#pragma unroll
      for (int st = 0; st < D / 4; ++st) {
        const int row = (4 * st + kq) * LD;
        const double a = M[row + 16 * ti + cl] * s;
#pragma unroll
        for (int R = 0; R < 4; ++R) acc[R] = mfma4x4x4d(a, M[row + 16 * tj + ((cl + 4 * R) & 15)] * s, acc[R]);
      }
    __syncthreads();
    if (w < NT * NT) {
      const int bl = (lane >> 2) & 3;
#pragma unroll
      for (int R = 0; R < 4; ++R)
        M[(16 * ti + 4 * bl + kq) * LD + 16 * tj + 4 * ((bl + R) & 3) + (lane & 3)] = acc[R];
    }
    __syncthreads();
  }
  // start column: largest diagonal entry, lowest index on ties
  if (tid == 0) {
    double best = -1.0;
    int arg = 0;
    for (int j = 0; j < d; ++j)
      if (M[j * LD + j] > best) {
        best = M[j * LD + j];
        arg = j;
      }
    j0 = arg;
  }
  __syncthreads();
  if (tid < D) y[tid] = M[tid * LD + j0];
  __syncthreads();
  double lam = 0.0;
  for (int it = 0; it <= kPowerIters; ++it) {
    // v = y / |y|, each wave for itself
    const double yl = lane < D ? y[lane] : 0.0;
    double nn = yl * yl;
    for (int m = 32; m >= 1; m >>= 1) nn += shfl_xor_d(nn, m);
    const double vl = nn > 0.0 ? yl / sqrt(nn) : 0.0;
    if (w == 0 && lane < D) v[lane] = vl;
    __syncthreads();
    const int row = tid >> 4, c0 = tid & 15;  // 16 threads a row
    if (row < D) {
      double t = 0.0;
#pragma unroll
      for (int j = 0; j < D / 16; ++j) t += C[row * LD + c0 + 16 * j] * v[c0 + 16 * j];
      t = row16_sum_d(t);
      if (c0 == 0) y[row] = t;
    }
    __syncthreads();
    if (it == kPowerIters) {  // Rayleigh quotient of the last unit vector
      double q = lane < D ? vl * y[lane] : 0.0;
      for (int m = 32; m >= 1; m >>= 1) q += shfl_xor_d(q, m);
      lam = q;
    }
  }
  if (tid == 0) {
    const double a = (lam > 0.0) ? sqrt(lam) : 0.0;
    B.ctl->spectral_a = a;
    if (!(a > 0.0) || !isfinite(a)) B.ctl->degenerate = 1;
  }
}

// out = (in s)^2 for a symmetric d x d matrix, s = 1 / tr in (0 when the trace is not positive),
// above 64 features: 64 x 64 blocks on the fp64 matrix cores, those on and above the diagonal
// (blockIdx.x), each written with its mirror; a wave takes a quarter (32 x 32).  Both operands are
// rows of the input, staged 32 rows at a time.  A diagonal block also writes its part of the trace,
// from which the next launch forms its s.  (A thread a row and scalar FMAs, with a launch for each
// trace: 127 us a squaring at d = 768.)
constexpr int kSqMax = 64;  // diagonal blocks at most (d <= 4096)
__global__ __launch_bounds__(kThreads) void k_square(Geometry g, const double* __restrict__ in, double* __restrict__ out,
                                                     const double* __restrict__ tr_in, double* __restrict__ tr_out) {
  __shared__ double xs[2][32][80];
  __shared__ double red[8];
  const int d = g.d, tid = threadIdx.x, lane = tid & 63, w = tid >> 6, kq = lane >> 4, cl = lane & 15;
  const int nb = (d + 63) / 64;
  int bp = blockIdx.x, bi = 0;
  while (bp >= nb - bi) {
    bp -= nb - bi;
    ++bi;
  }
  const int bj = bi + bp;
  const bool same = bi == bj;
  double tr = 0.0;
  if (tr_in) {
    for (int k = 0; k < nb; ++k) tr += tr_in[k];
  } else {
    for (int k = tid; k < d; k += kThreads) tr += in[(int64_t)k * d + k];
    tr = block_sum_d(tr, red);
    if (tid == 0) red[4] = tr;
    __syncthreads();
    tr = red[4];
    __syncthreads();
  }
  const double s = (tr > 0.0 && isfinite(tr)) ? 1.0 / tr : 0.0;
  const int wi = 32 * (w >> 1), wj = 32 * (w & 1);
  double acc[2][2][4];
#pragma unroll
  for (int I = 0; I < 2; ++I)
#pragma unroll
    for (int J = 0; J < 2; ++J)
#pragma unroll
      for (int R = 0; R < 4; ++R) acc[I][J][R] = 0.0;
  const int sf = tid & 63, sr = tid >> 6;
  const int fa = 64 * bi + sf, fb = 64 * bj + sf;
  double ra[8], rb[8];
  auto load_round = [&](int k0) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int k = k0 + sr + 4 * q;
      const int64_t row = (int64_t)(k < d ? k : 0) * d;
      ra[q] = (k < d && fa < d) ? in[row + (fa < d ? fa : 0)] : 0.0;
      rb[q] = (k < d && fb < d) ? in[row + (fb < d ? fb : 0)] : 0.0;
    }
  };
  load_round(0);
  for (int k0 = 0; k0 < d; k0 += 32) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      xs[0][sr + 4 * q][sf] = ra[q] * s;
      xs[1][sr + 4 * q][sf] = rb[q] * s;
    }
    __syncthreads();
    if (k0 + 32 < d) load_round(k0 + 32);
#pragma unroll
    for (int st = 0; st < 8; ++st) {
      const int row = 4 * st + kq;
      double a[2];
#pragma unroll
      for (int I = 0; I < 2; ++I) a[I] = xs[0][row][wi + 16 * I + cl];
#pragma unroll
      for (int J = 0; J < 2; ++J)
#pragma unroll
        for (int R = 0; R < 4; ++R) {
          const double b = xs[1][row][wj + 16 * J + ((cl + 4 * R) & 15)];
#pragma unroll
          for (int I = 0; I < 2; ++I) acc[I][J][R] = mfma4x4x4d(a[I], b, acc[I][J][R]);
        }
    }
  }
  const int bl = (lane >> 2) & 3;
  double t = 0.0;
#pragma unroll
  for (int I = 0; I < 2; ++I)
#pragma unroll
    for (int J = 0; J < 2; ++J)
#pragma unroll
      for (int R = 0; R < 4; ++R) {
        const int ia = 64 * bi + wi + 16 * I + 4 * bl + kq;
        const int jb = 64 * bj + wj + 16 * J + 4 * ((bl + R) & 3) + (lane & 3);
        if (ia < d && jb < d) {
          out[(int64_t)ia * d + jb] = acc[I][J][R];
          if (!same) out[(int64_t)jb * d + ia] = acc[I][J][R];
          if (ia == jb) t += acc[I][J][R];
        }
      }
  if (same) {
    t = block_sum_d(t, red);
    if (tid == 0) tr_out[bi] = t;
  }
}

// The power iterations above 64 features, the products spread over workgroups.  x_0 is the column of
// Bf with the largest diagonal entry (lowest index on ties); launch `it` forms v = x / |x| (every
// workgroup for itself, in the same order) and writes y = C v, the next launch's x; a wave takes a
// row of C at a time.
__global__ __launch_bounds__(kThreads) void k_power_mv(Geometry g, const double* __restrict__ C,
                                                       const double* __restrict__ Bf, const double* __restrict__ x,
                                                       double* __restrict__ y) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* v = reinterpret_cast<double*>(smem_raw);  // d
  __shared__ double red[8];
  __shared__ double sh;
  __shared__ double bv[kThreads];
  __shared__ int bk[kThreads];
  const int d = g.d, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  int j0 = 0;
  if (!x) {
    double best = -1.0;
    int arg = d;
    for (int j = tid; j < d; j += kThreads) {
      const double t = Bf[(int64_t)j * d + j];
      if (t > best) {
        best = t;
        arg = j;
      }
    }
    bv[tid] = best;
    bk[tid] = arg;
    __syncthreads();
    for (int h = kThreads / 2; h >= 1; h >>= 1) {
      if (tid < h && (bv[tid + h] > bv[tid] || (bv[tid + h] == bv[tid] && bk[tid + h] < bk[tid]))) {
        bv[tid] = bv[tid + h];
        bk[tid] = bk[tid + h];
      }
      __syncthreads();
    }
    j0 = bk[0] < d ? bk[0] : 0;
  }
  double nn = 0.0;
  for (int i = tid; i < d; i += kThreads) {
    const double t = x ? x[i] : Bf[(int64_t)i * d + j0];
    v[i] = t;
    nn += t * t;
  }
  nn = block_sum_d(nn, red);
  if (tid == 0) sh = nn > 0.0 ? 1.0 / sqrt(nn) : 0.0;
  __syncthreads();
  const double inv = sh;
  const int rows = gridDim.x * (kThreads / 64);
  for (int i = blockIdx.x * (kThreads / 64) + w; i < d; i += rows) {
    double t = 0.0;
#pragma unroll 4
    for (int j = lane; j < d; j += 64) t += C[(int64_t)i * d + j] * (v[j] * inv);
    for (int m = 32; m >= 1; m >>= 1) t += shfl_xor_d(t, m);
    if (lane == 0) y[i] = t;
  }
}

// a = sqrt of the Rayleigh quotient v . C v, v = x / |x|, y = C v.
__global__ __launch_bounds__(kThreads) void k_power_end(Geometry g, Bufs B, const double* __restrict__ x,
                                                        const double* __restrict__ y) {
  __shared__ double red[8];
  double nn = 0.0, xy = 0.0;
  for (int i = threadIdx.x; i < g.d; i += kThreads) {
    nn += x[i] * x[i];
    xy += x[i] * y[i];
  }
  nn = block_sum_d(nn, red);
  xy = block_sum_d(xy, red);
  if (threadIdx.x == 0) {
    const double lam = nn > 0.0 ? xy / sqrt(nn) : 0.0;
    const double a = (lam > 0.0) ? sqrt(lam) : 0.0;
    B.ctl->spectral_a = a;
    if (!(a > 0.0) || !isfinite(a)) B.ctl->degenerate = 1;
  }
}

// X <- (X - 1 xbar^T) / a in place; 256 rows per workgroup.
// Threads map to (column, row offset) as in k_colsum, eight rows' loads in flight.
__global__ __launch_bounds__(kThreads) void k_normalise(Geometry g, Bufs B) {
  if (B.ctl->degenerate) return;
  const double a = B.ctl->spectral_a;
  const int d = g.d;
  const int tid = threadIdx.x;
  const int64_t row0 = (int64_t)blockIdx.x * 256;
  const int64_t row1 = (g.n - row0) < 256 ? g.n : row0 + 256;
  auto one = [&](int64_t i, int col, double xb) {
    float* p = B.X + i * d + col;
    *p = (float)(((double)*p - xb) / a);
  };
  if (d <= kThreads) {
    const int rstep = kThreads / d;
    const int col = tid % d;
    const int rsub = tid / d;
    if (rsub >= rstep) return;
    const double xb = B.i_xbar[col];
    int64_t i = row0 + rsub;
    for (; i + 7 * rstep < row1; i += 8 * rstep) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = B.X[(i + u * rstep) * d + col];
#pragma unroll
      for (int u = 0; u < 8; ++u) B.X[(i + u * rstep) * d + col] = (float)(((double)v[u] - xb) / a);
    }
    for (; i < row1; i += rstep) one(i, col, xb);
  } else {
    for (int col = tid; col < d; col += kThreads) {
      const double xb = B.i_xbar[col];
      int64_t i = row0;
      for (; i + 7 < row1; i += 8) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = B.X[(i + u) * d + col];
#pragma unroll
        for (int u = 0; u < 8; ++u) B.X[(i + u) * d + col] = (float)(((double)v[u] - xb) / a);
      }
      for (; i < row1; ++i) one(i, col, xb);
    }
  }
}

// Projection statistics over row chunks: sum of (u_+)^2 and column sums of u_+.
__global__ __launch_bounds__(kThreads) void k_proj_partial(Geometry g, Bufs B) {
  __shared__ double red[kThreads];
  __shared__ double red8[8];
  const int tid = threadIdx.x;
  const int64_t n = g.n;
  const int r = g.r;
  const int64_t r0 = (int64_t)blockIdx.x * n / g.GI;
  const int64_t r1 = (int64_t)(blockIdx.x + 1) * n / g.GI;
  double* out = B.i_proj + (int64_t)blockIdx.x * (4 + g.r32);
  // r <= 256: column tid % r, every (256 / r)-th row; else columns tid, tid + 256, every row
  const int rstep = r <= kThreads ? kThreads / r : 1;
  const int col = tid % r;
  const int rsub = r <= kThreads ? tid / r : 0;
  double cs = 0.0, sq = 0.0;
  if (r > kThreads) {
    for (int c = tid; c < r; c += kThreads) {
      double csc = 0.0;
      int64_t i = r0;
      for (; i + 15 < r1; i += 16) {  // sixteen rows' loads in flight, added in row order
        float v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = B.U[(i + u) * r + c];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
          const float uu = fmaxf(v[u], 0.f);
          csc += (double)uu;
          sq += (double)uu * (double)uu;
        }
      }
      for (; i < r1; ++i) {
        const float u = fmaxf(B.U[i * r + c], 0.f);
        csc += (double)u;
        sq += (double)u * (double)u;
      }
      out[4 + c] = csc;
    }
  } else if (rsub < rstep) {
    // sixteen rows' loads in flight, added in row order
    int64_t i = r0 + rsub;
    for (; i + 15 * rstep < r1; i += 16 * rstep) {
      float v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = B.U[(i + u * rstep) * r + col];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const float uu = fmaxf(v[u], 0.f);
        cs += (double)uu;
        sq += (double)uu * (double)uu;
      }
    }
    for (; i < r1; i += rstep) {
      const float u = fmaxf(B.U[i * r + col], 0.f);
      cs += (double)u;
      sq += (double)u * (double)u;
    }
  }
  red[tid] = cs;
  __syncthreads();
  if (tid < r && r <= kThreads) {
    double t = 0.0;
    for (int k = 0; k < rstep; ++k) t += red[tid + k * r];
    out[4 + tid] = t;
  }
  const double tsq = block_sum_d(sq, red8);
  if (tid == 0) {
    out[0] = tsq;
    out[1] = out[2] = out[3] = 0.0;
  }
}

// c_f = FP32(sqrt(K) / ||U_+||_F) (1 when U is already in Omega); p = FP32(c colsum).  Workgroup b
// takes columns 16 b .. 16 b + 15, 16 groups of threads over the chunks; each forms the sum of
// squares for itself, in the same order (a thread a column over all 512 chunks: 100 to 160 us).
__global__ __launch_bounds__(kThreads) void k_proj_ctl(Geometry g, Bufs B, double K, int in_omega) {
  __shared__ double red[kThreads];
  __shared__ double red8[8];
  __shared__ double cbuf[1];
  const int tid = threadIdx.x;
  const int stride = 4 + g.r32;
  double S = 0.0;
  for (int gx = tid; gx < g.GI; gx += kThreads) S += B.i_proj[(int64_t)gx * stride];
  S = block_sum_d(S, red8);
  if (tid == 0) {
    double c = 1.0;
    if (!in_omega) {
      const double nu = sqrt(S);
      if (!(nu > 1e-20) || !isfinite(S)) {
        if (blockIdx.x == 0) B.ctl->breakdown = 1;
        c = 0.0;
      } else {
        c = (double)(float)(sqrt(K) / nu);
      }
    }
    cbuf[0] = c;
    if (blockIdx.x == 0) B.i_scal[0] = c;
  }
  const int cl = tid & 15, gq = tid >> 4, col = blockIdx.x * 16 + cl;
  red[tid] = col < g.r ? strided_sum<8>(B.i_proj + 4 + col, stride, gq, 16, g.GI) : 0.0;
  __syncthreads();
  if (tid < 16 && col < g.r32) {
    double t = 0.0;
    for (int k = 0; k < 16; ++k) t += red[16 * k + cl];
    B.p[col] = (col < g.r) ? (float)(cbuf[0] * t) : 0.f;
  }
}

__global__ __launch_bounds__(kThreads) void k_proj_apply(Geometry g, Bufs B) {
  if (B.ctl->breakdown) return;
  const float cf = (float)B.i_scal[0];
  const int64_t tot = g.n * (int64_t)g.r;
  for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < tot; e += (int64_t)gridDim.x * kThreads)
    B.U[e] = cf * fmaxf(B.U[e], 0.f);
}

__global__ __launch_bounds__(kThreads) void k_zero_y(Geometry g, Bufs B) {
  for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < g.n; e += (int64_t)gridDim.x * kThreads)
    B.y[e] = 0.f;
}

// ---------------------------------------------------------------------------
hipError_t launch_ctl_init(const Bufs& b, float gamma_f, hipStream_t st) {
  hipLaunchKernelGGL(k_ctl_init, dim3(1), dim3(64), 0, st, b, gamma_f);
  return hipGetLastError();
}

hipError_t launch_clear_stop(const Bufs& b, hipStream_t st) {
  hipLaunchKernelGGL(k_clear_stop, dim3(1), dim3(64), 0, st, b);
  return hipGetLastError();
}

hipError_t launch_colsum(const Geometry& g, const Bufs& b, hipStream_t st) {
  hipLaunchKernelGGL(k_colsum, dim3(g.GI), dim3(kThreads), 0, st, g, b);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_colmean, dim3((g.d + 15) / 16), dim3(kThreads), 0, st, g, b);
  return hipGetLastError();
}

hipError_t launch_gram_partials(const float* M, int64_t n, int d, const double* mean, double* part, int chunks,
                                hipStream_t st) {
  const int nb = (d + 63) / 64;
  hipLaunchKernelGGL(k_gram, dim3(chunks, nb * (nb + 1) / 2), dim3(kThreads), 0, st, M, n, d, mean, part);
  return hipGetLastError();
}

hipError_t launch_gram(const Geometry& g, const Bufs& b, hipStream_t st) {
  hipError_t e = launch_gram_partials(b.X, g.n, g.d, b.i_xbar, b.i_gram, g.GG, st);
  if (e != hipSuccess) return e;
  const int64_t dd = (int64_t)g.d * g.d;
  // enough entries to fill the chip with a thread each, or not
  if (dd >= (int64_t)256 * kThreads)
    hipLaunchKernelGGL(k_gram_reduce<kThreads>, dim3((unsigned)((dd + kThreads - 1) / kThreads)), dim3(kThreads), 0, st,
                       g, b);
  else
    hipLaunchKernelGGL(k_gram_reduce<16>, dim3((unsigned)((dd + 15) / 16)), dim3(kThreads), 0, st, g, b);
  return hipGetLastError();
}

hipError_t launch_spectral(const Geometry& g, const Bufs& b, hipStream_t st) {
  // up to 64 features the matrix fits one workgroup's LDS
  if (g.d <= 64) {
    if (g.d <= 16)
      hipLaunchKernelGGL(k_power_small<16>, dim3(1), dim3(1024), 0, st, g, b);
    else if (g.d <= 32)
      hipLaunchKernelGGL(k_power_small<32>, dim3(1), dim3(1024), 0, st, g, b);
    else
      hipLaunchKernelGGL(k_power_small<64>, dim3(1), dim3(1024), 0, st, g, b);
    return hipGetLastError();
  }
  // B_0 = C; B_{k+1} = (B_k / tr B_k)^2, ping-ponging B0/B1; the traces' block sums likewise
  const int nb = (g.d + 63) / 64;
  const double* in = b.i_C;
  double* bufs[2] = {b.i_B0, b.i_B1};
  for (int k = 0; k < kSquarings; ++k) {
    double* out = bufs[k & 1];
    hipLaunchKernelGGL(k_square, dim3(nb * (nb + 1) / 2), dim3(kThreads), 0, st, g, in, out,
                       k ? (const double*)(b.i_trace + ((k - 1) & 1) * kSqMax) : nullptr,
                       b.i_trace + (k & 1) * kSqMax);
    in = out;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // x and y in the buffer the last squaring did not write (d >= 65: 2 d entries fit)
  double* xy = (in == b.i_B0) ? b.i_B1 : b.i_B0;
  const double* x = nullptr;
  double* y = xy;
  const int grid = (g.d + 3) / 4 < 256 ? (g.d + 3) / 4 : 256;
  for (int it = 0; it <= kPowerIters; ++it) {
    y = xy + (it & 1) * g.d;
    hipLaunchKernelGGL(k_power_mv, dim3(grid), dim3(kThreads), (size_t)g.d * sizeof(double), st, g,
                       (const double*)b.i_C, in, x, y);
    if (it < kPowerIters) x = y;
  }
  hipLaunchKernelGGL(k_power_end, dim3(1), dim3(kThreads), 0, st, g, b, x, (const double*)y);
  return hipGetLastError();
}

hipError_t launch_normalise(const Geometry& g, const Bufs& b, hipStream_t st) {
  const int64_t blocks = (g.n + 255) / 256;
  hipLaunchKernelGGL(k_normalise, dim3((unsigned)blocks), dim3(kThreads), 0, st, g, b);
  return hipGetLastError();
}

hipError_t launch_project(const Geometry& g, const Bufs& b, double K, int in_omega, hipStream_t st) {
  hipLaunchKernelGGL(k_proj_partial, dim3(g.GI), dim3(kThreads), 0, st, g, b);
  hipLaunchKernelGGL(k_proj_ctl, dim3(g.r32 / 16), dim3(kThreads), 0, st, g, b, K, in_omega);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || in_omega) return e;
  hipLaunchKernelGGL(k_proj_apply, dim3(2048), dim3(kThreads), 0, st, g, b);
  return hipGetLastError();
}

hipError_t launch_zero_y(const Geometry& g, const Bufs& b, hipStream_t st) {
  hipLaunchKernelGGL(k_zero_y, dim3(1024), dim3(kThreads), 0, st, g, b);
  return hipGetLastError();
}

}  // namespace nlr
