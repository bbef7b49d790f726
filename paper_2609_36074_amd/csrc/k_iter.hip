// Per-iteration kernels of the NLR iteration (Algorithm 1, Section 4) for gfx950.
//
// One iteration is
//   pass A        Theta partials = Xhat^T U over row chunks (fp32 matrix cores),
//                 fused with the row work that ends the previous iteration and
//                 prepares this one: u = fl(c_f w) (lazy normalisation), q = u.p - 1,
//                 gated dual step ytilde += (beta/n) q, ybar = ytilde + (beta/n) q,
//                 s partials = U^T ybar, ||q||^2 and ytilde^T q partials
//                 (eq. gpu-vectors; Appendix C call sites 2, 3, 7-11);
//   theta_sum     fixed-order FP64 sum of the Theta partials, ||Theta||_F^2;
//   ctl_a         s, rho, objective fhat (eq. normalized), stopping rule (Section 4.3);
//   pass B        G = Xhat Theta on fp32 matrix cores with the epilogue of
//                 eq. (entrywise-fusion): w = max(u + 2 alpha G - alpha ybar p - alpha s, 0),
//                 FP64 statistics a = ||W||^2, b = ||U||^2, h = <W, U> (eq. fused-statistics)
//                 and column sums of W, W stored over U in place;
//   ctl_b         a, b, h, column sums -> c_f = FP32(sqrt(K)/sqrt(a)), breakdown test,
//                 Delta = max(c^2 a + b - 2 c h, 0), delta, dual gate Delta < eps_d^2 K,
//                 p = FP32(c * colsum) (eq. movement-estimate, Appendix B Alg. 2 (d)-(f)).
// The rescale U <- c W is never a separate pass: every consumer reads fl(c_f w).
// "finish" is pass A without the matrix product: it materialises U = fl(c_f w)
// and applies the pending end-of-iteration work, so a host call always returns
// a materialised factor.
#include "k_common.hpp"

namespace nlr {

// ---------------------------------------------------------------------------
// Pass A where Theta does not fit one wave's registers runs as two launches: the row work
// (k_rows_wide, below) and this product, Theta = Xhat^T U.  Grid (GA, mgroups * ngroups).
// Workgroup (gx, gy) owns a contiguous range of kTPA-row tiles and the Theta blocks of group gy
// (MBG x NBG blocks of 32 x 32).  Wave w owns m-block w % MBG and all NBG n-blocks, over the
// k-slice w / MBG of each tile (KS = 4 / MBG slices).  The next tile's rows are loaded into
// registers while the matrix cores work on the current one: per tile a thread holds XV + UV
// pieces of four; loads past the last row or column read a valid address and are zeroed, so none
// waits behind a branch.  The waves whose m-block lies past the last feature skip the product
// (their partial rows are not written).  UN: rows of X or U not 16-byte aligned.  Bound by the
// fp32 matrix cores (74% busy at 2e6 x 768 x 256); rows that are not 16-byte aligned used to be
// staged a float a thread with nothing in flight meanwhile (13 to 20 TFLOP/s).
// ---------------------------------------------------------------------------
template <int MBG, int NBG, bool UN>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(NBG >= 7 ? 1 : 2, 8))) void k_theta_wide(
    Geometry g, Bufs B) {
  if (halted(B.ctl)) return;
  constexpr int KS = 4 / MBG;
  constexpr int XS = MBG * 32 + 4;                // LDS row strides (floats)
  constexpr int US = NBG * 32 + 4;
  constexpr int XR4 = MBG * 8, UR4 = NBG * 8;     // 16-byte pieces per tile row
  constexpr int XV = kTPA * XR4 / kThreads;       // pieces per thread and tile
  constexpr int UV = kTPA * UR4 / kThreads;
  static_assert(XV * kThreads == kTPA * XR4 && UV * kThreads == kTPA * UR4, "whole pieces per thread");
  extern __shared__ __align__(16) unsigned char smem_raw[];
  float* Xs = reinterpret_cast<float*>(smem_raw);  // kTPA x XS
  float* Us = Xs + kTPA * XS;                      // kTPA x US

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int gx = blockIdx.x;
  const int gy = blockIdx.y;
  const int mg = gy / g.ngroups;
  const int ng = gy - mg * g.ngroups;
  const int64_t n = g.n;
  const int d = g.d, r = g.r, r32 = g.r32;
  const int f0 = mg * MBG * 32;
  const int c0 = ng * NBG * 32;
  const float cf = B.ctl->c_f;
  const int64_t tb = (int64_t)gx * g.tilesA / gridDim.x;
  const int64_t te = (int64_t)(gx + 1) * g.tilesA / gridDim.x;
  const int mb = wave % MBG;
  const int ks = wave / MBG;
  const bool active = f0 + mb * 32 < g.d32;

  // this thread's pieces: tile row and column offset (fixed), validity of the column
  int xo[XV], uo[UV];
  bool xk[XV], uk[UV];
#pragma unroll
  for (int i = 0; i < XV; ++i) {
    const int v = tid + i * kThreads, row = v / XR4, c = 4 * (v - row * XR4);
    xk[i] = f0 + c < d;
    xo[i] = row * d + (xk[i] ? f0 + c : 0);
  }
#pragma unroll
  for (int i = 0; i < UV; ++i) {
    const int v = tid + i * kThreads, row = v / UR4, c = 4 * (v - row * UR4);
    uk[i] = c0 + c < r;
    uo[i] = row * r + (uk[i] ? c0 + c : 0);
  }
  f32x4 xr[XV], ur[UV];
  // rows of tile t: a row past the last is read as row 0 of the tile and zeroed
  auto load = [&](int64_t tile) {
    const int64_t row0 = tile * kTPA;
    const int valid = (int)((n - row0) < kTPA ? (n - row0) : kTPA);
    const float* xb = B.X + row0 * d;
    const float* ub = B.U + row0 * r;
    if (UN && (row0 + kTPA >= n || d < 3 || r < 3)) {
#pragma unroll
      for (int i = 0; i < XV; ++i) {
        const int v = tid + i * kThreads, row = v / XR4, c = 4 * (v - row * XR4);
        xr[i] = load4_edge(xb + (row < valid ? row : 0) * d, xk[i] ? f0 + c : 0, d);
      }
#pragma unroll
      for (int i = 0; i < UV; ++i) {
        const int v = tid + i * kThreads, row = v / UR4, c = 4 * (v - row * UR4);
        ur[i] = load4_edge(ub + (row < valid ? row : 0) * r, uk[i] ? c0 + c : 0, r);
      }
      return;
    }
#pragma unroll
    for (int i = 0; i < XV; ++i) {
      const int row = (tid + i * kThreads) / XR4;
      xr[i] = load4<UN>(xb + (row < valid ? xo[i] : xo[i] - row * d));
    }
#pragma unroll
    for (int i = 0; i < UV; ++i) {
      const int row = (tid + i * kThreads) / UR4;
      ur[i] = load4<UN>(ub + (row < valid ? uo[i] : uo[i] - row * r));
    }
  };

  f32x16 acc[NBG];
#pragma unroll
  for (int j = 0; j < NBG; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;

  if (tb < te) load(tb);
  for (int64_t tile = tb; tile < te; ++tile) {
    const int64_t row0 = tile * kTPA;
    const int valid = (int)((n - row0) < kTPA ? (n - row0) : kTPA);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < XV; ++i) {
      const int v = tid + i * kThreads, row = v / XR4, c = 4 * (v - row * XR4);
      const bool ok = xk[i] && row < valid;
      f32x4 t = xr[i];
#pragma unroll
      for (int e = 0; e < 4; ++e) t[e] = (UN ? ok && f0 + c + e < d : ok) ? t[e] : 0.f;
      *reinterpret_cast<f32x4*>(Xs + row * XS + c) = t;
    }
#pragma unroll
    for (int i = 0; i < UV; ++i) {
      const int v = tid + i * kThreads, row = v / UR4, c = 4 * (v - row * UR4);
      const bool ok = uk[i] && row < valid;
      f32x4 t = ur[i];
#pragma unroll
      for (int e = 0; e < 4; ++e) t[e] = (UN ? ok && c0 + c + e < r : ok) ? t[e] * cf : 0.f;
      *reinterpret_cast<f32x4*>(Us + row * US + c) = t;
    }
    __syncthreads();
    if (tile + 1 < te) load(tile + 1);
    if (active) {
      const int kbeg = ks * (kTPA / KS);
      const int kend = kbeg + kTPA / KS;
      const int lr = lane >> 5;
      const int lc = lane & 31;
#pragma unroll 4
      for (int k = kbeg; k < kend; k += 2) {
        const float a = Xs[(k + lr) * XS + mb * 32 + lc];
#pragma unroll
        for (int j = 0; j < NBG; ++j) {
          const float bv = Us[(k + lr) * US + j * 32 + lc];
          acc[j] = mfma32x32x2(a, bv, acc[j]);
        }
      }
    }
  }

  // combine k-slices (waves with the same m-block) in a fixed order, then write
  __syncthreads();
  float* comb = Xs;  // MBG * NBG * 16 * 64 floats
  for (int slice = 1; slice < KS; ++slice) {
    if (ks == slice) {
#pragma unroll
      for (int j = 0; j < NBG; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) comb[((mb * NBG + j) * 16 + v) * 64 + lane] = acc[j][v];
    }
    __syncthreads();
    if (ks == 0) {
#pragma unroll
      for (int j = 0; j < NBG; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[j][v] += comb[((mb * NBG + j) * 16 + v) * 64 + lane];
    }
    __syncthreads();
  }
  if (ks == 0 && active) {
    float* part = B.theta_part + (int64_t)gx * g.theta_cols;
    const int lr = lane >> 5, lc = lane & 31;
#pragma unroll
    for (int j = 0; j < NBG; ++j) {
      const int col = c0 + j * 32 + lc;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int f = f0 + mb * 32 + 8 * (v >> 2) + 4 * lr + (v & 3);
        if (f < g.d32 && col < r32) part[(int64_t)f * r32 + col] = acc[j][v];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Row work of pass A where Theta does not fit one wave (its first launch), and the finish pass of
// those shapes and of the panel form: no LDS staging; LPR lanes stream whole rows of U, lane l
// holding the columns l + LPR j (CPL of them), RPI rows at a time each.  Per row:
// u = fl(c_f w), q = u.p - 1 (FP64, summed over the row's lanes by an xor butterfly, so every lane has
// the same bits), the gated dual step (eq. of the stored dual), ybar (stored for pass B above 128
// columns); then s += ybar u, ||q||^2 and ytilde^T q in FP64.  FINISH: materialises u instead of
// forming s and ybar.  Grid GAF; workgroup gx takes a contiguous range of rows, its waves every
// fourth piece of it, and writes partial row gx (qq, yq, 0, 0, s).  Bound by the row stream (the
// finish pass as LDS-staged tiles took 1.94 ms at 1e6 x 300, 2.4 GB).  Up to 16 and 32 columns a row
// has 16 or 32 lanes: with a whole wave a row the butterflies of mostly idle lanes bound it (row pass
// over 1e6 x 5 and 1e6 x 30: 142 us, now 28 and 50; finish pass at 2,911,497 x 12: 0.43 ms).
// ---------------------------------------------------------------------------
// Sum over the LPR lanes of a row, bitwise the same in all of them: v[l] + v[l ^ m], m from LPR / 2 down
// to 1.  (Below 16, after the step for 2 m the values repeat every 2 m lanes, so a rotation of the DPP
// row by m brings the same value as l ^ m.)
template <int LPR>
__device__ __forceinline__ double lanes_sum_d(double v) {
  if constexpr (LPR >= 64) v += shfl_xor_d(v, 32);
  if constexpr (LPR >= 32) v += shfl_xor_d(v, 16);
  v += dpp_d<0x128>(v);  // row_ror 8, 4, 2, 1
  v += dpp_d<0x124>(v);
  v += dpp_d<0x122>(v);
  v += dpp_d<0x121>(v);
  return v;
}
template <int LPR, int CPL, bool FINISH>
__global__ __launch_bounds__(kThreads) void k_rows_wide(Geometry g, Bufs B, StepArgs S) {
  // the finish pass runs after a stop (it still materialises U) but not after a breakdown
  if (FINISH ? (B.ctl->breakdown != 0) : halted(B.ctl)) return;
  const bool stopped = FINISH && (B.ctl->stop != 0);
  static_assert(LPR == 64 || CPL == 1, "narrow rows: one column a lane");
  constexpr int RPI = 8;           // rows per lane and step
  constexpr int NR = 64 / LPR;     // rows of a wave at a time
  __shared__ double sred[4 * LPR * CPL];
  __shared__ double dred[kThreads + 8];
  const int tid = threadIdx.x;
  const int lane = tid & (LPR - 1);       // within the row
  const int grp = (tid & 63) / LPR;       // row of the wave's NR
  const int wave = tid >> 6;
  const int64_t n = g.n;
  const int r = g.r;
  const float cf = B.ctl->c_f;
  // after a stop the end-of-iteration work was already done by pass A
  const bool gate = (S.end_work != 0) && (B.ctl->gate != 0) && !stopped;
  const float gam = S.gamma_f;

  float pl[CPL];
  bool okc[CPL];
  int colo[CPL];  // column read (0 for the lanes past the last column)
#pragma unroll
  for (int j = 0; j < CPL; ++j) {
    const int col = lane + LPR * j;
    okc[j] = col < r;
    colo[j] = okc[j] ? col : 0;
    pl[j] = okc[j] ? B.p[col] : 0.f;
  }
  double sacc[CPL];
#pragma unroll
  for (int j = 0; j < CPL; ++j) sacc[j] = 0.0;
  double acc_qq = 0.0, acc_yq = 0.0;

  const int64_t rb = (int64_t)blockIdx.x * n / gridDim.x;
  const int64_t re = (int64_t)(blockIdx.x + 1) * n / gridDim.x;
  for (int64_t base = rb + (int64_t)wave * RPI * NR + grp; base - grp < re; base += 4 * RPI * NR) {
    float u[RPI][CPL];
    float yt[RPI];
    // every load reads a valid address (row rb, column 0 in place of those out of range)
    // and the value is dropped afterwards, so that no load sits behind a branch; all
    // loads of the step are issued before any of their values is used
#pragma unroll
    for (int i = 0; i < RPI; ++i) {
      const int64_t row = base + i * NR;
      const float* src = B.U + (row < re ? row : rb) * r;
#pragma unroll
      for (int j = 0; j < CPL; ++j) u[i][j] = src[colo[j]];
      yt[i] = B.y[row < re ? row : rb];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < RPI; ++i) {
      const bool okr = base + i * NR < re;
#pragma unroll
      for (int j = 0; j < CPL; ++j) u[i][j] = (okr && okc[j]) ? u[i][j] * cf : 0.f;
      yt[i] = okr ? yt[i] : 0.f;
    }
    double dot[RPI];
#pragma unroll
    for (int i = 0; i < RPI; ++i) {
      dot[i] = 0.0;
#pragma unroll
      for (int j = 0; j < CPL; ++j) dot[i] += (double)u[i][j] * (double)pl[j];
    }
#pragma unroll
    for (int i = 0; i < RPI; ++i) dot[i] = lanes_sum_d<LPR>(dot[i]);
#pragma unroll
    for (int i = 0; i < RPI; ++i) {
      const int64_t row = base + i * NR;
      if (row < re) {
        const float q = (float)(dot[i] - 1.0);
        float y = yt[i];
        if (gate) {
          y = fmaf(gam, q, y);
          if (lane == 0) B.y[row] = y;
        }
        const float ybar = fmaf(gam, q, y);
        if (lane == 0) {
          if (!FINISH && CPL > 2) B.ybar[row] = ybar;
          acc_qq += (double)q * (double)q;
          acc_yq += (double)y * (double)q;
        }
#pragma unroll
        for (int j = 0; j < CPL; ++j) {
          if constexpr (FINISH) {
            if (okc[j]) B.U[row * r + colo[j]] = u[i][j];
          } else {
            sacc[j] += (double)ybar * (double)u[i][j];
          }
        }
      }
    }
  }

  double* ap = B.a_part + (int64_t)blockIdx.x * (4 + g.r32);
  const double qq = block_sum_d(acc_qq, dred);
  const double yq = block_sum_d(acc_yq, dred);
  if (tid == 0) {
    ap[0] = qq;
    ap[1] = yq;
    ap[2] = ap[3] = 0.0;
  }
  if (FINISH) {
    for (int c = tid; c < g.r32; c += kThreads) ap[4 + c] = 0.0;
    return;
  }
  // s: the rows of a wave, then the four waves' sums of a column, added in wave order
#pragma unroll
  for (int m = LPR; m < 64; m <<= 1) sacc[0] += shfl_xor_d(sacc[0], m);
  if (grp == 0)
#pragma unroll
    for (int j = 0; j < CPL; ++j) sred[(wave * CPL + j) * LPR + lane] = sacc[j];
  __syncthreads();
  for (int c = tid; c < g.r32; c += kThreads) {
    double t = 0.0;
    if (c < LPR * CPL) {
      const int j = c / LPR, l = c & (LPR - 1);
      t = ((sred[(0 * CPL + j) * LPR + l] + sred[(1 * CPL + j) * LPR + l]) + sred[(2 * CPL + j) * LPR + l]) +
          sred[(3 * CPL + j) * LPR + l];
    }
    ap[4 + c] = t;
  }
}

// ---------------------------------------------------------------------------
// Pass A, register-resident form on the 16x16x4 fp32 matrix core (all of Theta
// fits one wave: FV*NGF*CV <= 32 blocks of 16x16).  Grid GA; each wave owns a
// contiguous range of 4-row steps.  Per k-step lane l works on row 4k + l/16:
// it loads FV consecutive features for each of NGF groups (feature
// 16*FV*g + FV*(l%16) + e) and CV consecutive columns of U (column CV*(l%16) + c);
// MFMA (g, e, c) accumulates Theta[16*FV*g + FV*i + e][CV*j + c] at D[i][j].
// A row's columns live in one 16-lane DPP row, so the row work (q = u.p - 1,
// dual step, ybar, s, ||q||^2, ytilde^T q) uses a 4-step DPP butterfly whose
// result is bitwise identical in all 16 lanes.
// MODE kPassFinish: no matrix product; writes u = fl(c_f w) back (materialises U).
// MODE kPassRows: no matrix product and no write of U: the row work of the fused
// iteration, whose Theta comes from the previous pass B.
// ---------------------------------------------------------------------------
// UN: rows of X or U that are not a whole number of aligned pieces (any d <= 128, r <= 64).
template <int FV, int NGF, int CV, int MODE, bool UN>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_pass_a_rows(
    Geometry g, Bufs B, StepArgs S) {
  constexpr bool FINISH = MODE == kPassFinish;
  constexpr bool THETA = MODE == kPassIter;
  // on breakdown the unnormalised update W already holds the factor's place
  const float* Usrc = B.U;
  if (FINISH && B.ctl->breakdown != 0) return;
  if (!FINISH && halted(B.ctl)) return;
  // the one-pass iteration launches the row pass every iteration; it runs only when
  // the previous iteration's stopping rule may fire (the pass then does no row work)
  if (MODE == kPassRows && g.fused8 && !B.ctl->rows_first) return;
  const bool stopped = FINISH && (B.ctl->stop != 0);
  constexpr int NBLK = FV * NGF * CV;  // 16x16 blocks of Theta
  // k-steps in flight: fewer when Theta takes 128 registers, more when only U and y stream
  constexpr int PF = THETA ? (NBLK >= 32 ? 2 : 4) : 8;
  __shared__ double dred[kThreads + 8];
  __shared__ float comb[THETA ? 2 * NBLK * 4 * 64 : 4];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int grp = lane >> 4;   // row within the k-step
  const int li = lane & 15;    // lane within the DPP row
  const int64_t n = g.n;
  const int d = g.d, r = g.r;
  const float cf = B.ctl->c_f;
  const bool gate = (S.end_work != 0) && (B.ctl->gate != 0) && !stopped;
  const float gam = S.gamma_f;

  float pl[CV];
#pragma unroll
  for (int c = 0; c < CV; ++c) {
    const int col = CV * li + c;
    pl[c] = (col < r) ? B.p[col] : 0.f;
  }

  // 4-row steps of this wave
  const int64_t steps = (n + 3) >> 2;
  const int64_t wid = (int64_t)blockIdx.x * 4 + wave;
  const int64_t nw = (int64_t)g.GA * 4;
  const int64_t k0 = wid * steps / nw;
  const int64_t k1 = (wid + 1) * steps / nw;

  f32x4v acc[NBLK];
  if (THETA) {
#pragma unroll
    for (int b = 0; b < NBLK; ++b) acc[b] = (f32x4v){0.f, 0.f, 0.f, 0.f};
  }
  double s_acc[CV];
#pragma unroll
  for (int c = 0; c < CV; ++c) s_acc[c] = 0.0;
  double qq = 0.0, yq = 0.0;

  float xr[PF][NGF][FV];
  float ur[PF][CV];
  float yr[PF];
  // The ring holds raw loads; masks and the lazy scale are applied where the
  // values are used, so that no instruction waits on a load right after issuing it.
  bool fx[NGF];
#pragma unroll
  for (int gg = 0; gg < NGF; ++gg) fx[gg] = (16 * FV * gg + FV * li) < d;
  const int cu = CV * li;
  const bool cx = cu < r;
  auto issue = [&](int slot, int64_t k) {
    const int64_t row = 4 * k + grp;
    const bool ok = (k < k1) && (row < n);
    const int64_t rr = ok ? row : 0;
    if constexpr (UN) {
      // the step that holds the last row, and any where a row is shorter than a piece: by elements
      const bool edge = 4 * k + 4 >= n || n <= 4 || d < 3 || r < 3;
      if (THETA) {
#pragma unroll
        for (int gg = 0; gg < NGF; ++gg) {
          const int f = 16 * FV * gg + FV * li;
          load_piece<FV>(xr[slot][gg], B.X + rr * d, f < d ? f : 0, d, edge);
        }
      }
      load_piece<CV>(ur[slot], Usrc + rr * r, cx ? cu : 0, r, edge);
    } else {
      if (THETA) {
#pragma unroll
        for (int gg = 0; gg < NGF; ++gg) {
          const int f = 16 * FV * gg + FV * li;
          load_vec<FV>(xr[slot][gg], B.X + rr * d + (f < d ? f : 0), true);
        }
      }
      load_vec<CV>(ur[slot], Usrc + rr * r + (cx ? cu : 0), true);
    }
    yr[slot] = B.y[rr];
  };
#pragma unroll
  for (int i = 0; i < PF; ++i) {
    __builtin_amdgcn_sched_barrier(0);
    issue(i, k0 + i);
  }
  __builtin_amdgcn_sched_barrier(0);

  for (int64_t kb = k0; kb < k1; kb += PF) {
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      // keep consumption of slot i and the refill of slot i in program order, so
      // that the loads of the other slots stay in flight
      __builtin_amdgcn_sched_barrier(0);
      const int64_t k = kb + i;
      const int64_t row = 4 * k + grp;
      const bool valid = (k < k1) && (row < n);
      float u[CV];
#pragma unroll
      for (int c = 0; c < CV; ++c) u[c] = (valid && (UN ? cu + c < r : cx)) ? ur[i][c] * cf : 0.f;
      if (THETA) {
#pragma unroll
        for (int gg = 0; gg < NGF; ++gg)
#pragma unroll
          for (int e = 0; e < FV; ++e) {
            const float x = (UN ? 16 * FV * gg + FV * li + e < d : fx[gg]) ? xr[i][gg][e] : 0.f;
#pragma unroll
            for (int c = 0; c < CV; ++c)
              acc[(gg * FV + e) * CV + c] = mfma16x16x4(x, u[c], acc[(gg * FV + e) * CV + c]);
          }
      }
      // q = u.p - 1 over the 16 lanes of this row (FP64)
      double dot = 0.0;
#pragma unroll
      for (int c = 0; c < CV; ++c) dot += (double)u[c] * (double)pl[c];
      dot = row16_sum_d(dot);
      const float q = (float)(dot - 1.0);
      float yt = valid ? yr[i] : 0.f;
      if (gate) yt = fmaf(gam, q, yt);
      const float ybar = fmaf(gam, q, yt);
      // branch-free: invalid rows have u = 0; stores of invalid lanes go to the dump slot
      if (gate) *(valid ? (B.y + row) : B.dump) = yt;  // the 16 lanes of a row store the same value
#pragma unroll
      for (int c = 0; c < CV; ++c) s_acc[c] += (double)ybar * (double)u[c];
      const bool lead = valid && li == 0;
      qq += lead ? (double)q * (double)q : 0.0;
      yq += lead ? (double)yt * (double)q : 0.0;
      if (FINISH) {
        float* dst = (valid && cx) ? (B.U + row * r + cu) : B.dump;
        if constexpr (UN) {
#pragma unroll
          for (int c = 0; c < CV; ++c)
            if (valid && cu + c < r) B.U[row * r + cu + c] = u[c];
        } else if constexpr (CV == 4) {
          f32x4 o = {u[0], u[1], u[2], u[3]};
          *reinterpret_cast<f32x4*>(dst) = o;
        } else if constexpr (CV == 2) {
          typedef float f32x2 __attribute__((ext_vector_type(2)));
          f32x2 o = {u[0], u[1]};
          *reinterpret_cast<f32x2*>(dst) = o;
        } else {
          dst[0] = u[0];
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      issue(i, k + PF);
    }
  }
  __builtin_amdgcn_sched_barrier(0);

  // ---- partials ----
  if (THETA) {
    // Theta: ((wave0 + wave2) + (wave1 + wave3)) through two LDS regions
    constexpr int REG = NBLK * 4 * 64;
    if (wave < 2) {
      float* dst = comb + wave * REG;
#pragma unroll
      for (int b = 0; b < NBLK; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) dst[(b * 4 + v) * 64 + lane] = acc[b][v];
    }
    __syncthreads();
    if (wave >= 2) {
      float* dst = comb + (wave - 2) * REG;
#pragma unroll
      for (int b = 0; b < NBLK; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int idx = (b * 4 + v) * 64 + lane;
          dst[idx] = dst[idx] + acc[b][v];
        }
    }
    __syncthreads();
    float* part = B.theta_part + (int64_t)blockIdx.x * g.theta_cols;
    const int tot = g.d32 * g.r32;
    for (int e = tid; e < tot; e += kThreads) {
      const int f = e / g.r32, col = e - (e / g.r32) * g.r32;
      const int gg = f / (16 * FV), rem = f - gg * 16 * FV;
      const int i = rem / FV, ef = rem - i * FV;
      const int c = col % CV, j = col / CV;
      float val = 0.f;
      if (gg < NGF && j < 16) {
        const int idx = (((gg * FV + ef) * CV + c) * 4 + (i & 3)) * 64 + 16 * (i >> 2) + j;
        val = comb[idx] + comb[REG + idx];
      }
      part[e] = val;
    }
  }
  // s: rows 0..3 of a k-step hold the same columns; waves hold disjoint rows
  __syncthreads();
#pragma unroll
  for (int c = 0; c < CV; ++c) {
    double v = s_acc[c] + shfl_xor_d(s_acc[c], 16);
    v = v + shfl_xor_d(v, 32);
    if (grp == 0) dred[wave * 16 * CV + CV * li + c] = v;  // 4 * 16 * CV <= 256
  }
  __syncthreads();
  double* ap = B.a_part + (int64_t)blockIdx.x * (4 + g.r32);
  for (int c = tid; c < g.r32; c += kThreads) {
    double t = 0.0;
    if (c < 16 * CV)
      t = ((dred[c] + dred[16 * CV + c]) + dred[32 * CV + c]) + dred[48 * CV + c];
    ap[4 + c] = FINISH ? 0.0 : t;
  }
  const double tq = block_sum_d(qq, dred + kThreads);
  const double ty = block_sum_d(yq, dred + kThreads);
  if (tid == 0) {
    ap[0] = tq;
    ap[1] = ty;
    ap[2] = ap[3] = 0.0;
  }
}

// ---------------------------------------------------------------------------
// Row pass and finish pass of the single-Xhat-pass form for narrow factors (r <= 16,
// r even): eight lanes per row (two columns each, 8-byte loads) and eight rows per
// wave and step, so that the per-row work (the FP64 dot and its butterfly, q, the
// dual step, ybar and the FP64 statistics) is not repeated over 16 lanes for a few
// columns.  The row dot sums over the 8 lanes of a DPP half row (row8_sum_d); both
// modes use it, so q, ytilde and ybar agree bitwise whichever of them does the row
// work (nlr_run(T) equals T nlr_step).  Outputs as k_pass_a_rows.
// ---------------------------------------------------------------------------
template <int MODE>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_rows_narrow(
    Geometry g, Bufs B, StepArgs S) {
  constexpr bool FINISH = MODE == kPassFinish;
  static_assert(MODE == kPassFinish || MODE == kPassRows, "row work only");
  const float* Usrc = B.U;
  if (FINISH && B.ctl->breakdown != 0) return;
  if (!FINISH && halted(B.ctl)) return;
  // the one-pass iteration launches the row pass every iteration; it runs only when
  // the previous iteration's stopping rule may fire (the pass then does no row work)
  if (MODE == kPassRows && g.fused8 && !B.ctl->rows_first) return;
  const bool stopped = FINISH && (B.ctl->stop != 0);
  constexpr int PF = 8;  // steps in flight (16 halves the waves per SIMD: no more bytes in flight)
  __shared__ double dred[kThreads + 8];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int grp = lane >> 3;  // row within the step
  const int li = lane & 7;    // lane within the row
  const int64_t n = g.n;
  const int r = g.r;
  const float cf = B.ctl->c_f;
  const bool gate = (S.end_work != 0) && (B.ctl->gate != 0) && !stopped;
  const float gam = S.gamma_f;
  const int cu = 2 * li;
  const bool cx = cu < r;  // r even: both columns of the lane are valid, or neither
  const float pl[2] = {cx ? B.p[cu] : 0.f, cx ? B.p[cu + 1] : 0.f};

  const int64_t steps = (n + 7) >> 3;
  const int64_t wid = (int64_t)blockIdx.x * 4 + wave;
  const int64_t nw = (int64_t)g.GA * 4;
  const int64_t k0 = wid * steps / nw;
  const int64_t k1 = (wid + 1) * steps / nw;

  double s_acc[2] = {0.0, 0.0};
  double qq = 0.0, yq = 0.0;
  float ur[PF][2];
  float yr[PF];
  auto issue = [&](int slot, int64_t k) {
    const int64_t row = 8 * k + grp;
    const bool ok = (k < k1) && (row < n);
    const int64_t rr = ok ? row : 0;
    load_vec<2>(ur[slot], Usrc + rr * r + (cx ? cu : 0), true);
    yr[slot] = B.y[rr];
  };
#pragma unroll
  for (int i = 0; i < PF; ++i) {
    __builtin_amdgcn_sched_barrier(0);
    issue(i, k0 + i);
  }
  __builtin_amdgcn_sched_barrier(0);

  for (int64_t kb = k0; kb < k1; kb += PF) {
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      __builtin_amdgcn_sched_barrier(0);
      const int64_t k = kb + i;
      const int64_t row = 8 * k + grp;
      const bool valid = (k < k1) && (row < n);
      float u[2];
#pragma unroll
      for (int c = 0; c < 2; ++c) u[c] = (valid && cx) ? ur[i][c] * cf : 0.f;
      double dot = 0.0;
#pragma unroll
      for (int c = 0; c < 2; ++c) dot += (double)u[c] * (double)pl[c];
      dot = row8_sum_d(dot);
      const float q = (float)(dot - 1.0);
      float yt = valid ? yr[i] : 0.f;
      if (gate) yt = fmaf(gam, q, yt);
      const float ybar = fmaf(gam, q, yt);
      if (gate) *(valid ? (B.y + row) : B.dump) = yt;  // the 8 lanes of a row store the same value
#pragma unroll
      for (int c = 0; c < 2; ++c) s_acc[c] += (double)ybar * (double)u[c];
      const bool lead = valid && li == 0;
      qq += lead ? (double)q * (double)q : 0.0;
      yq += lead ? (double)yt * (double)q : 0.0;
      if (FINISH) {
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        float* dst = (valid && cx) ? (B.U + row * r + cu) : B.dump;
        *reinterpret_cast<f32x2*>(dst) = (f32x2){u[0], u[1]};
      }
      __builtin_amdgcn_sched_barrier(0);
      issue(i, k + PF);
    }
  }
  __builtin_amdgcn_sched_barrier(0);

  // s: the eight rows of a step hold the same columns; waves hold disjoint rows
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    double v = s_acc[c] + shfl_xor_d(s_acc[c], 8);
    v = v + shfl_xor_d(v, 16);
    v = v + shfl_xor_d(v, 32);
    if (grp == 0) dred[wave * 16 + cu + c] = v;
  }
  __syncthreads();
  double* ap = B.a_part + (int64_t)blockIdx.x * (4 + g.r32);
  for (int c = tid; c < g.r32; c += kThreads) {
    double t = 0.0;
    if (c < 16) t = ((dred[c] + dred[16 + c]) + dred[32 + c]) + dred[48 + c];
    ap[4 + c] = FINISH ? 0.0 : t;
  }
  const double tq = block_sum_d(qq, dred + kThreads);
  const double ty = block_sum_d(yq, dred + kThreads);
  if (tid == 0) {
    ap[0] = tq;
    ap[1] = ty;
    ap[2] = ap[3] = 0.0;
  }
}

// ---------------------------------------------------------------------------
// The control kernels sum the partial rows (row statistics, column sums) themselves: a workgroup
// takes 8 columns, its threads spread over the rows, so that the rows, which other XCDs wrote,
// come in over several compute units (one workgroup for all columns: 7 to 13 us for 147 to
// 440 KB; a launch of segment sums in front of a one-workgroup control: 9.5 to 14 us for the two).
// Column c of the row layout is a statistic below 4 and column c - 4 of the factor above.
// ---------------------------------------------------------------------------
constexpr int kCtlCols = 8;
static int ctl_blocks(const Geometry& g) { return (4 + g.r32 + kCtlCols - 1) / kCtlCols; }

// Fixed-order sums over the R <= 1024 rows of the partial rows of a_part (HA) and b_part (HB), every
// load issued before the first is used (one after the other they cost a load latency of about 2 us
// each): in every thread its column of the workgroup's eight (NT / 8 threads over the rows) and the
// array's leading statistics (a thread a row), which have the same bits in every workgroup; with th2,
// the sum of its RT entries.  `red`: kRedDoubles of LDS.  NT = 256 threads where the launch is the
// control's own: with 1024, the shuffles of sixteen waves on one compute unit's LDS took 3 us.
constexpr int kRedDoubles = 2 * 128 + 7 * 16 + 23;
struct CtlSums {
  double col_a, col_b;  // this thread's column
  double qq, yq;        // HA: ||q||^2, ytilde^T q
  double a, b, h, over; // HB
  double th2;
};
// sum over the wave, in every lane of its last 16 and in lanes 0..15 alike (four DPP steps, two shuffles)
__device__ __forceinline__ double wave_sum_d(double v) {
  v = row16_sum_d(v);
  v += shfl_xor_d(v, 16);
  return v + shfl_xor_d(v, 32);
}
template <bool HA, bool HB, int NT, int UN>
__device__ __forceinline__ CtlSums ctl_sums_un(const double* __restrict__ pa, const double* __restrict__ pb, int rows,
                                               int C, int blk, const double* __restrict__ th2, int RT, double* red) {
  constexpr int PH = NT / 8, NW = NT / 64, SR = (PH * UN + NT - 1) / NT;
  const int tid = threadIdx.x, ph = tid >> 3, w = tid >> 6;
  int c = kCtlCols * blk + (tid & 7);
  c = c < C ? c : C - 1;
  double va[UN], vb[UN], s[7][SR], t2 = 0.0;
#pragma unroll
  for (int i = 0; i < UN; ++i) {
    const int row = ph + PH * i;
    const uint32_t o = (uint32_t)((row < rows ? row : 0) * C + c);
    if (HA) va[i] = pa[o];
    if (HB) vb[i] = pb[o];
  }
#pragma unroll
  for (int k = 0; k < SR; ++k) {
    const int row = tid + NT * k;
    const uint32_t o = (uint32_t)((row < rows ? row : 0) * C);
#pragma unroll
    for (int i = 0; i < 2; ++i) s[i][k] = HA ? pa[o + i] : 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) s[2 + i][k] = HB ? pb[o + i] : 0.0;
  }
  if (th2 && RT <= NT) {
    if (tid < RT) t2 = th2[tid];
  } else if (th2) {
    for (int k0 = tid; k0 < RT; k0 += 8 * NT) {  // eight loads in flight, added in order
      double v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = th2[k0 + NT * i < RT ? k0 + NT * i : k0];
#pragma unroll
      for (int i = 0; i < 8; ++i) t2 += k0 + NT * i < RT ? v[i] : 0.0;
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  auto col = [&](const double (&v)[UN], double* r) {
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < UN; ++i) t += ph + PH * i < rows ? v[i] : 0.0;
    t += dpp_d<0x128>(t);  // row_ror 8: the row's other half
    t += shfl_xor_d(t, 16);
    t += shfl_xor_d(t, 32);
    if ((tid & 63) < 8) r[8 * w + (tid & 7)] = t;
  };
  if (HA) col(va, red);
  if (HB) col(vb, red + 128);
#pragma unroll
  for (int i = 0; i < 7; ++i) {
    if (!(i < 2 ? HA : (i < 6 ? HB : th2 != nullptr))) continue;
    double t = i == 6 ? t2 : 0.0;
    if (i < 6)
#pragma unroll
      for (int k = 0; k < SR; ++k) t += tid + NT * k < rows ? s[i][k] : 0.0;
    t = wave_sum_d(t);
    if ((tid & 63) == 0) red[256 + 16 * i + w] = t;
  }
  __syncthreads();
  // the waves' sums, added by a thread each
  if (tid < 16 + 7) {
    const double* r = tid < 16 ? red + 128 * (tid >> 3) + (tid & 7) : red + 256 + 16 * (tid - 16);
    const int st = tid < 16 ? 8 : 1;
    const bool used = tid < 8 ? HA : (tid < 16 ? HB : (tid < 18 ? HA : (tid < 22 ? HB : th2 != nullptr)));
    double t = 0.0;
    if (used)
#pragma unroll 4
      for (int k = 0; k < NW; ++k) t += r[st * k];
    red[256 + 7 * 16 + tid] = t;
  }
  __syncthreads();
  const double* f = red + 256 + 7 * 16;
  const int cl = tid & 7;
  return {f[cl], f[8 + cl], f[16], f[17], f[18], f[19], f[20], f[21], f[22]};
}
template <bool HA, bool HB, int NT>
__device__ __forceinline__ CtlSums ctl_sums(const double* __restrict__ pa, const double* __restrict__ pb, int64_t R,
                                            int C, int blk, const double* __restrict__ th2, int RT, double* red) {
  if constexpr (NT == 1024)
    return ctl_sums_un<HA, HB, NT, 8>(pa, pb, (int)R, C, blk, th2, RT, red);
  else
    return R <= 256 ? ctl_sums_un<HA, HB, NT, 8>(pa, pb, (int)R, C, blk, th2, RT, red)
                    : (R <= 512 ? ctl_sums_un<HA, HB, NT, 16>(pa, pb, (int)R, C, blk, th2, RT, red)
                                : ctl_sums_un<HA, HB, NT, 32>(pa, pb, (int)R, C, blk, th2, RT, red));
}

// The scale c of U = c W from a = ||W||_F^2 (FP32 of an FP64 ratio), 0 on a breakdown; `over`: W left
// its split operand's range.
__device__ __forceinline__ float norm_scale(double a, double over, double K) {
  const double nu = sqrt(a);
  if (over > 0.0 || !(nu > 1e-20) || !isfinite(a)) return 0.f;
  return (float)(sqrt(K) / nu);
}

// ---------------------------------------------------------------------------
// Control after pass A or a row pass: s (workgroup b its columns), and in workgroup 0 rho, the
// objective and the stopping rule of the previous iteration.  finish = the call after the finish
// pass (workgroup 0 alone), which also writes the control block and the record of the latest iteration
// to the host's mirror.  rows: the partial rows.  A stop, set here, does not keep the other
// workgroups from their columns: after a stop the partial rows stay as they are, and so does s.
// defer (two-pass form): ||Theta||_F^2 is formed by the same launch, so the control after pass B
// adds it to the objective.
// ---------------------------------------------------------------------------
template <int NT>
__device__ __forceinline__ void ctl_a_work(const Geometry& g, const Bufs& B, const StepArgs& S, int blk, int finish,
                                           int64_t rows, int defer, double* red) {
  DevCtl* ctl = B.ctl;
  if (ctl->breakdown) return;
  if (blk == 0 && ctl->stop) {
    // stopped earlier in this call: the finish pass only materialised U
    if (finish && threadIdx.x == 0) ctl->c_f = 1.0f;
    return;
  }
  // one-pass iteration: after its row pass only (which runs when the stop may fire)
  if (g.fused8 && !finish && !ctl->rows_first) return;
  const int tid = threadIdx.x;
  const int C = 4 + g.r32;
  const int64_t t = ctl->t_done;
  const double Delta = ctl->Delta, delta = ctl->delta;
  const CtlSums sm =
      ctl_sums<true, false, NT>(B.a_part, nullptr, rows, C, blk, (blk > 0 || finish || defer) ? nullptr : B.th2_part, g.RT, red);
  // (one-pass iteration with valid Gram terms, rows_first == 1: s is the Gram-derived
  // one already in place, as when the pass does the row work itself)
  if (!finish && !(g.fused8 && ctl->rows_first == 1)) {
    const int c = kCtlCols * blk + tid - 4;
    if (tid < kCtlCols && c >= 0 && c < g.r32) B.s[c] = (c < g.r) ? (float)sm.col_a : 0.f;
  }
  if (blk > 0) return;
  if (tid == 0) {
    const double qq = sm.qq, yq = sm.yq, th2 = sm.th2;
    const double rho = sqrt(qq * S.inv_n);
    ctl->rho = rho;
    int stop = 0;
    if (S.end_work && t > 0) {
      nlr_iter_stats* prev = &B.hist[(t - 1) % kHistCap];
      stop = (Delta < S.eps_d * S.eps_d * S.K) && (delta < S.eps_c) && (rho < S.eps_c) && (t >= S.T_min);
      prev->rho = rho;
      prev->stop = stop;
      if (stop) ctl->stop = 1;
    }
    if (!finish && !stop) {
      const double obj = -th2 + yq + 0.5 * S.beta * S.inv_n * qq;
      ctl->objective = obj;
      ctl->theta_fro2 = th2;
      nlr_iter_stats* cur = &B.hist[t % kHistCap];
      cur->t = t;
      cur->objective = obj;
      cur->theta_fro2 = th2;
      cur->a = cur->b = cur->h = cur->delta = 0.0;
      cur->rho = 0.0;
      cur->c = 0.f;
      cur->dual_step = 0;
      cur->stop = 0;
      cur->breakdown = 0;
    }
    if (finish) ctl->c_f = 1.0f;
    if (g.fused8 && !finish) ctl->rows_run += 1;
  }
}

__global__ __launch_bounds__(kThreads) void k_ctl_a(Geometry g, Bufs B, StepArgs S, int finish, int64_t rows) {
  __shared__ double red[kRedDoubles];
  ctl_a_work<kThreads>(g, B, S, blockIdx.x, finish, rows, 0, red);
  if (finish && B.mirror) {  // (one workgroup)
    __syncthreads();
    const uint32_t* src = reinterpret_cast<const uint32_t*>(B.ctl);
    uint32_t* dst = reinterpret_cast<uint32_t*>(B.mirror);
    for (int i = threadIdx.x; i < (int)(sizeof(DevCtl) / 4); i += blockDim.x) dst[i] = src[i];
    const int64_t t = B.ctl->t_done - (B.ctl->breakdown ? 0 : 1);
    if (t >= 0) {
      const uint32_t* rec = reinterpret_cast<const uint32_t*>(B.hist + t % kHistCap);
      uint32_t* out = reinterpret_cast<uint32_t*>(B.mirror_rec);
      for (int i = threadIdx.x; i < (int)(sizeof(nlr_iter_stats) / 4); i += blockDim.x) out[i] = rec[i];
    }
  }
}

// ---------------------------------------------------------------------------
// s = U^T ybar of the one-pass iteration from the Gram terms of the pass that
// produced U = c W.  Per row q = u.p - 1 = c^2 w.P - 1 and ybar = ytilde_prev +
// (1 + gate) gamma q (the pending gated dual step, then the penalty term; gamma =
// beta / n), so
//   s = c W^T ytilde_prev + (1 + gate) gamma c (c^2 (W^T W) P - P)
// with W^T W (the columns after Theta in the Theta partial rows, reduced with them
// and multiplied by P in k_theta_sum), P and W^T ytilde_prev summed in a fixed
// order (FP64).  The last term is U^T q: small near feasibility and weighted by
// gamma, so the fp32-accumulated Gram partials carry it well below the iteration's
// rounding.  k_theta_sum forms s right after the pass with the step arguments of
// the call; k_onepass_begin forms it again at the start of a host call,
// whose step arguments (beta) may differ.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float s_from_gram(const Bufs& B, int r32, int k, double gp, float gamma_f) {
  const double c = B.ctl->c_gram;
  const double gmul = (1.0 + (B.ctl->gate ? 1.0 : 0.0)) * (double)gamma_f;
  const double P = B.gram_vec[k], wy = B.gram_vec[r32 + k];
  return (float)(c * wy + gmul * c * (c * c * gp - P));
}

// ---------------------------------------------------------------------------
// Theta = sum of the partial rows (fixed order, FP64), written in the pass-B
// operand layout, plus per-workgroup ||Theta||_F^2 and max |Theta| partials; 64 entries a workgroup.
// Layout: chunk ch of 32 features, quarter j (4 features), m-block mb, lane l,
// element e  <->  Theta[32 ch + 16 (l/32) + 4 j + e][32 mb + l%32].
// scaled: partials of Xhat^T W (fused pass B), which carry the scale c of U = c W.
// One-pass iteration: the workgroups after the RT of Theta take the W^T W columns of the partial
// rows, times P (the column sums of W): (W^T W P)_k, and with gamma_f >= 0 form s for the next pass.
// Two-pass form (ctl_rows > 0): the last ctl_blocks workgroups do the control after pass A meanwhile
// (both only need pass A's partials); Theta is then formed whatever the control decides, since a
// stop leaves its partials as they were.
// ---------------------------------------------------------------------------
// WIDE: 256 entries a workgroup, one a thread (in the same order), from kThetaWide blocks of 64 on:
// two waves a SIMD without a second thread an entry.  In sixteens the workgroups come in many rounds
// there, with more masked loads than rows: 768 x 256 (42 partial rows) 20.5 us, wide 11.8; 4096 x 448
// (16 rows) 140 and 31; below, 224 x 320 (128 rows) takes 13 us in sixteens.
// After a stop of an earlier iteration (2, see k_ctl_b) there is nothing to do: formed all the same, 38
// iterations enqueued past a stop at 60,000 x 768 x 256 took 0.55 ms more.
constexpr int kThetaWide = 2048;
template <bool WIDE>
__global__ __launch_bounds__(WIDE ? kThreads : kRedThreads) void k_theta_sum(Geometry g, Bufs B, StepArgs S,
                                                                             int64_t rows, int scaled, float gamma_f,
                                                                             int64_t ctl_rows) {
  constexpr int NT = WIDE ? kThreads : kRedThreads;
  __shared__ double red[WIDE ? kRedDoubles : kRedThreads];  // (also the control's: kRedDoubles)
  const int tb = WIDE ? g.RT >> 2 : g.RT;  // workgroups of Theta
  if (ctl_rows > 0) {
    if (B.ctl->breakdown != 0 || B.ctl->stop == 2) return;
    if ((int)blockIdx.x >= tb) {
      ctl_a_work<NT>(g, B, S, (int)blockIdx.x - tb, 0, ctl_rows, 1, red);
      return;
    }
  } else if (halted(B.ctl)) {
    return;
  }
  const int tid = threadIdx.x, r32 = g.r32;
  const bool gram = !WIDE && (int)blockIdx.x >= g.RT;
  int64_t e;
  double sum;
  if constexpr (WIDE) {
    e = (int64_t)blockIdx.x * kThreads + tid;
    sum = part_sum16(B.theta_part, rows, g.theta_cols, e);
  } else {
    e = ((int64_t)blockIdx.x - (gram ? g.RT : 0)) * 64 + (tid & 63);
    sum = part_sum64(B.theta_part, rows, g.theta_cols, e + (gram ? (int64_t)g.d32 * r32 : 0), red);
    if (tid >= 64) return;
  }
  if (gram) {
    const int k = (int)e / r32, l = (int)e - k * r32;  // r32 = 32 or 64 entries of a row: lanes of this wave
    double gp = sum * B.gram_vec[l];
    for (int m = r32 >> 1; m >= 1; m >>= 1) gp += shfl_xor_d(gp, m);
    if (l == 0) {
      B.gram_vec[2 * r32 + k] = gp;
      if (gamma_f >= 0.f) {
        const float sk = s_from_gram(B, r32, k, gp, gamma_f);
        B.s[k] = (k < g.r) ? sk : 0.f;
      }
    }
    return;
  }
  const int f = (int)(e / r32), c = (int)(e - (int64_t)f * r32);
  if (scaled) sum *= (double)B.ctl->c_f;
  if (f >= g.d) sum = 0.0;  // padded features: zero rows of Theta
  const int ch = f >> 5, fin = f & 31;
  const int hh = fin >> 4, j = (fin & 15) >> 2, ee = fin & 3;
  const int mbk = c >> 5, l = hh * 32 + (c & 31);
  const int64_t idx = ((((int64_t)ch * 4 + j) * g.NB + mbk) * 64 + l) * 4 + ee;
  B.theta[idx] = (float)sum;
  double t2 = sum * sum;
  float m = fabsf((float)sum);
  for (int k = 32; k >= 1; k >>= 1) {
    t2 += shfl_xor_d(t2, k);
    m = fmaxf(m, shfl_xor_f(m, k));
  }
  if ((tid & 63) == 0) {
    const int64_t w = WIDE ? 4 * (int64_t)blockIdx.x + (tid >> 6) : blockIdx.x;
    B.th2_part[w] = t2;
    B.thmax_part[w] = m;  // (the panel form scales its split Theta operand by it)
  }
}

// W of four columns c .. c + 3 of a row (ok: the row exists and c < r), as one store where all four
// exist.
template <bool UN>
__device__ __forceinline__ void store4(float* urow, int c, int r, bool ok, const float* w) {
  if (!ok) return;
  if constexpr (UN) {
    if (c + 4 <= r) {
      *reinterpret_cast<f32x4u*>(urow + c) = (f32x4u){w[0], w[1], w[2], w[3]};
    } else {
#pragma unroll
      for (int e = 0; e < 3; ++e)
        if (c + e < r) urow[c + e] = w[e];
    }
  } else {
    *reinterpret_cast<f32x4*>(urow + c) = (f32x4){w[0], w[1], w[2], w[3]};
  }
}

// ---------------------------------------------------------------------------
// Pass B with Theta streamed through LDS, for every shape the resident form below does not hold.
// Grid GB, persistent over 128-row super-tiles; wave w computes rows [32w, 32w+32) of each:
//   acc (D layout) = Theta^T (A operand) x Xhat^T (B operand, lane l loads row l%32, features
//   32ch + 16 (l/32) + [0, 16)),
// then the epilogue per element, w = max(u + 2 alpha acc - alpha ybar p - alpha s, 0).  The columns
// go in groups of CG blocks (the last group may be short): per super-tile, for each group
// and each 32-feature chunk, the workgroup stages the chunk's Theta operands (4 KiB
// per block) in one of two LDS buffers and every wave multiplies its rows by them.
// The next chunk's Theta operands and Xhat features are loaded into registers while
// the matrix cores work on the current one (one barrier per chunk); during a group's
// last chunk the rows of U its epilogue needs are loaded instead, and the next
// group's first chunk during the epilogue.  Loads past the last row, feature, block
// or column read a valid address and are zeroed or unused, so that no load waits
// behind a branch.  Above 128 columns ybar comes from the row launch of pass A
// (which stores it), else from q = u.p - 1 formed here.  Column sums: lanes l and
// l ^ 1 combined, then added to the wave's row of an LDS table per super-tile.
// UN: rows of X or U not 16-byte aligned.
// ---------------------------------------------------------------------------
template <int CG, bool UN>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_pass_b_stream(
    Geometry g, Bufs B, StepArgs S) {
  if (halted(B.ctl)) return;
  constexpr int TCF = 4 * CG * 256;  // floats of a chunk's Theta operands
  extern __shared__ __align__(16) unsigned char smem_raw[];
  float* tbuf = reinterpret_cast<float*>(smem_raw);           // 2 x TCF
  double* colred = reinterpret_cast<double*>(tbuf + 2 * TCF);  // 4 x r32
  float* ps = reinterpret_cast<float*>(colred + 4 * g.r32);    // r32
  float* ss = ps + g.r32;                                      // r32
  double* dred = reinterpret_cast<double*>(ss + g.r32);       // 4

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int h = lane >> 5;
  const int li = lane & 31;
  const int64_t n = g.n;
  const int d = g.d, r = g.r, r32 = g.r32, NB = g.NB;
  const int nch = g.nch;
  const int ngr = (NB + CG - 1) / CG;  // column groups
  const bool ystored = pass_a_split(g);  // the row launch of pass A stored ybar
  const float cf = B.ctl->c_f;
  const float gam = S.gamma_f;
  const float two_alpha = S.two_alpha_f;
  const float neg_alpha = -S.alpha_f;

  for (int c = tid; c < r32; c += kThreads) {
    ps[c] = B.p[c];
    ss[c] = B.s[c];
  }
  for (int c = tid; c < 4 * r32; c += kThreads) colred[c] = 0.0;
  __syncthreads();  // p and s are read before the first chunk's barrier (q below 129 columns)

  double sa = 0.0, sb = 0.0, sh = 0.0;
  int base = 0;  // local index (8 qd + e ordering) of the column sum this lane keeps
  if (li & 16) base += 8;
  if (li & 8) base += 4;
  if (li & 4) base += 2;
  if (li & 2) base += 1;

  const int64_t sb0 = (int64_t)blockIdx.x * g.tilesB / g.GB;
  const int64_t sb1 = (int64_t)(blockIdx.x + 1) * g.tilesB / g.GB;

  // Theta operands of chunk (group cgi, chunk ch): piece v = tid + 256 i of the chunk is
  // j = v / (64 CG), block m = v / 64 % CG (clamped to the last block), lane v % 64
  int tj[CG], tm[CG];
#pragma unroll
  for (int i = 0; i < CG; ++i) {
    const int v = tid + kThreads * i;
    tj[i] = v / (64 * CG);
    tm[i] = (v / 64) % CG;
  }
  f32x4 tr[CG];
  f32x4 xr[4];
  // super-tiles from this one on read rows by elements (it holds the last row)
  const int64_t edge_st = g.tilesB - 1;
  auto load_chunk = [&](int64_t st, int cgi, int ch) {
    // (an opaque zero keeps the address arithmetic here, not hoisted out of the loops
    // into registers that would stay live across them)
    int z = 0;
    asm volatile("" : "+v"(z));
#pragma unroll
    for (int i = 0; i < CG; ++i) {
      const int mb = cgi * CG + tm[i] < NB ? cgi * CG + tm[i] : NB - 1;
      const int64_t piece = (((int64_t)ch * 4 + tj[i]) * NB + mb) * 64 + ((tid + z) & 63);
      tr[i] = *reinterpret_cast<const f32x4*>(B.theta + piece * 4);
    }
    const int64_t pt = st * kTPB + wave * 32 + li + z;
    const float* xrow = B.X + (pt < n ? pt : 0) * (int64_t)d;
    const int fb = ch * 32 + h * 16;
    if (UN && (st >= edge_st || d < 3)) {
#pragma unroll
      for (int q = 0; q < 4; ++q) xr[q] = load4_edge(xrow, fb + 4 * q < d ? fb + 4 * q : 0, d);
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) xr[q] = load4<UN>(xrow + (fb + 4 * q < d ? fb + 4 * q : 0));
    }
  };

  if (sb0 < sb1) load_chunk(sb0, 0, 0);
  int kbuf = 0;
  for (int64_t st = sb0; st < sb1; ++st) {
    const int64_t pt = st * kTPB + wave * 32 + li;
    const bool vpt = pt < n;
    float* urow = B.U + (vpt ? pt : 0) * (int64_t)r;
    const bool uedge = UN && (st >= edge_st || r < 3);
    // (the opaque copy keeps the p/s reads inside the tile loop instead of hoisting
    // loop-invariant registers out of it)
    int lds_off = 0;
    asm volatile("" : "+v"(lds_off));
    const float* psl = ps + lds_off;
    const float* ssl = ss + lds_off;
    float ybar;
    if (ystored) {
      // ybar of the row pass of this iteration (q from an FP64 dot)
      const float yb = B.ybar[vpt ? pt : 0];
      ybar = vpt ? yb : 0.f;
    } else {
      // q = u.p - 1 over the whole row (fp32 dot over the lane's half, then the other half)
      float dotf = 0.f;
      for (int m = 0; m < NB; ++m)
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) {
          const int c = 32 * m + 8 * qd + 4 * h;
          const f32x4 t = (UN && uedge) ? load4_edge(urow, c < r ? c : 0, r) : load4<UN>(urow + (c < r ? c : 0));
          const bool ok = vpt && c < r;
          const f32x4 pv = *reinterpret_cast<const f32x4*>(psl + c);
          dotf = fmaf(ok ? t.x * cf : 0.f, pv.x, dotf);
          dotf = fmaf((UN ? ok && c + 1 < r : ok) ? t.y * cf : 0.f, pv.y, dotf);
          dotf = fmaf((UN ? ok && c + 2 < r : ok) ? t.z * cf : 0.f, pv.z, dotf);
          dotf = fmaf((UN ? ok && c + 3 < r : ok) ? t.w * cf : 0.f, pv.w, dotf);
        }
      dotf += shfl_xor_f(dotf, 32);
      const float yv = B.y[vpt ? pt : 0];
      ybar = vpt ? fmaf(gam, dotf - 1.0f, yv) : 0.f;
    }

    for (int cgi = 0; cgi < ngr; ++cgi) {
      const int nbg = NB - cgi * CG < CG ? NB - cgi * CG : CG;  // blocks of this group
      f32x16 acc[CG];
#pragma unroll
      for (int m = 0; m < CG; ++m)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[m][v] = 0.f;
      // one chunk: stage its Theta operands (the barrier also ends every wave's reads of
      // the buffer two chunks back), then `next` issues the loads that overlap the
      // products, then the products
      auto chunk = [&](int ch, auto&& next) {
        float* tb = tbuf + kbuf * TCF;
#pragma unroll
        for (int i = 0; i < CG; ++i) *reinterpret_cast<f32x4*>(tb + (tid + kThreads * i) * 4) = tr[i];
        float xv[16];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const bool ok = vpt && (ch * 32 + h * 16 + 4 * q < d);
          xv[4 * q + 0] = ok ? xr[q].x : 0.f;
          xv[4 * q + 1] = ok ? xr[q].y : 0.f;
          xv[4 * q + 2] = ok ? xr[q].z : 0.f;
          xv[4 * q + 3] = ok ? xr[q].w : 0.f;
        }
        __syncthreads();
        next();
        // the loads are issued before the products (not sunk below them to reuse the
        // registers of this chunk's X operands)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          f32x4 a[CG];
#pragma unroll
          for (int m = 0; m < CG; ++m) a[m] = *reinterpret_cast<const f32x4*>(tb + ((j * CG + m) * 64 + lane) * 4);
          // every block of the group, also past the last of a short group (its operands
          // are the last block's, its products unused): a conditional product would make
          // the compiler copy the accumulators
#pragma unroll
          for (int m = 0; m < CG; ++m) {
            acc[m] = mfma32x32x2(a[m].x, xv[4 * j + 0], acc[m]);
            acc[m] = mfma32x32x2(a[m].y, xv[4 * j + 1], acc[m]);
            acc[m] = mfma32x32x2(a[m].z, xv[4 * j + 2], acc[m]);
            acc[m] = mfma32x32x2(a[m].w, xv[4 * j + 3], acc[m]);
          }
        }
        kbuf ^= 1;
      };
      for (int ch = 0; ch + 1 < nch; ++ch) chunk(ch, [&]() { load_chunk(st, cgi, ch + 1); });
      // the last chunk: the rows of U the epilogue needs are loaded meanwhile
      f32x4 ua[CG][4];
      chunk(nch - 1, [&]() {
#pragma unroll
        for (int m = 0; m < CG; ++m)
#pragma unroll
          for (int qd = 0; qd < 4; ++qd) {
            const int c = 32 * (cgi * CG + m) + 8 * qd + 4 * h;
            ua[m][qd] = (UN && uedge) ? load4_edge(urow, c < r ? c : 0, r) : load4<UN>(urow + (c < r ? c : 0));
          }
      });
      // ---- epilogue of the group: lane holds row pt, columns 32 (CG cgi + m) + 8 qd + 4 h + e ----
#pragma unroll
      for (int m = 0; m < CG; ++m) {
        if (m == CG / 2) {
          // the next group's (or super-tile's) first chunk, behind the rest of the epilogue
          // (in the registers of the blocks done)
          const bool ng = cgi + 1 < ngr;
          const int64_t st2 = ng ? st : st + 1;
          if (st2 < sb1) load_chunk(st2, ng ? cgi + 1 : 0, 0);
        }
        if (m < nbg) {
          const int mb = cgi * CG + m;
          float wv[16];
#pragma unroll
          for (int qd = 0; qd < 4; ++qd) {
            const int c = 32 * mb + 8 * qd + 4 * h;
            const bool ok = vpt && c < r;
            float u4[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) u4[e] = (UN ? ok && c + e < r : ok) ? ua[m][qd][e] * cf : 0.f;
            const f32x4 pv = *reinterpret_cast<const f32x4*>(psl + c);
            const f32x4 sv = *reinterpret_cast<const f32x4*>(ssl + c);
            const float pe[4] = {pv.x, pv.y, pv.z, pv.w};
            const float se[4] = {sv.x, sv.y, sv.z, sv.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float uu = u4[e];
              float t = fmaf(two_alpha, acc[m][4 * qd + e], uu);
              t = fmaf(neg_alpha, ybar * pe[e], t);
              t = fmaf(neg_alpha, se[e], t);
              float w = fmaxf(t, 0.f);
              if (!vpt || c + e >= r) w = 0.f;
              wv[4 * qd + e] = w;
              const double wd = (double)w, ud = (double)uu;
              sa = fma(wd, wd, sa);
              sb = fma(ud, ud, sb);
              sh = fma(wd, ud, sh);
            }
            store4<UN>(urow, c, r, ok, &wv[4 * qd]);
          }
          reduce_scatter<16, 16>(wv, li);
          const double v = (double)wv[0] + shfl_xor_d((double)wv[0], 1);
          if ((li & 1) == 0) colred[wave * r32 + 32 * mb + 8 * (base >> 2) + 4 * h + (base & 3)] += v;
        }
        // one block at a time (its LDS reads are not hoisted above the previous block)
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  // ---- workgroup partials ----
  __syncthreads();
  double* out = B.b_part + (int64_t)blockIdx.x * (4 + r32);
  for (int c = tid; c < r32; c += kThreads)
    out[4 + c] = ((colred[c] + colred[r32 + c]) + colred[2 * r32 + c]) + colred[3 * r32 + c];
  const double ta = block_sum_d(sa, dred);
  const double tb2 = block_sum_d(sb, dred);
  const double th = block_sum_d(sh, dred);
  if (tid == 0) {
    out[0] = ta;
    out[1] = tb2;
    out[2] = th;
    out[3] = 0.0;
  }
}

// ---------------------------------------------------------------------------
// Pass B, resident-tile form (d <= 128, r <= 128, Theta in LDS).  Same
// arithmetic and partial layout as the streamed form; each wave holds its tile's whole
// Xhat slab (NCH chunks) and U slab in registers: the U loads of a tile are
// issued before its matrix product and the next tile's Xhat before its epilogue.
// UN: rows of X or U not 16-byte aligned: the same in 16-byte pieces at 4-byte addresses, by elements
// in the tile with the last row (52 us at 700,001 x 51 x 13, 4.2 TB/s of its bytes).
// ---------------------------------------------------------------------------
template <int NB, int NCH, bool UN>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_pass_b_res(
    Geometry g, Bufs B, StepArgs S) {
  if (halted(B.ctl)) return;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  float* th_s = reinterpret_cast<float*>(smem_raw);  // d32*r32
  float* ps = th_s + g.d32 * g.r32;                   // r32
  float* ss = ps + g.r32;                             // r32
  double* colred = reinterpret_cast<double*>(ss + g.r32);
  double* dred = colred + 4 * g.r32;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int h = lane >> 5;
  const int li = lane & 31;
  const int64_t n = g.n;
  const int d = g.d, r = g.r, r32 = g.r32;
  const float cf = B.ctl->c_f;
  const float gam = S.gamma_f;
  const float two_alpha = S.two_alpha_f;
  const float neg_alpha = -S.alpha_f;

  {
    const int tot4 = (g.d32 * r32) >> 2;
    const f32x4* src = reinterpret_cast<const f32x4*>(B.theta);
    f32x4* dst = reinterpret_cast<f32x4*>(th_s);
    for (int v = tid; v < tot4; v += kThreads) dst[v] = src[v];
  }
  for (int c = tid; c < r32; c += kThreads) {
    ps[c] = B.p[c];
    ss[c] = B.s[c];
  }
  __syncthreads();

  double sa = 0.0, sb = 0.0, sh = 0.0;
  double colacc[NB];
#pragma unroll
  for (int m = 0; m < NB; ++m) colacc[m] = 0.0;
  int base = 0;
  if (li & 16) base += 8;
  if (li & 8) base += 4;
  if (li & 4) base += 2;
  if (li & 2) base += 1;

  const int64_t sb0 = (int64_t)blockIdx.x * g.tilesB / g.GB;
  const int64_t sb1 = (int64_t)(blockIdx.x + 1) * g.tilesB / g.GB;

  // tiles from this one on read rows by elements (it holds the last row)
  const int64_t edge_st = g.tilesB - 1;
  float xv[NCH][16];
  auto load_x = [&](int64_t st, int ch) {
    const int64_t pt = st * kTPB + wave * 32 + li;
    const bool ok = (st < sb1) && (pt < n);
    const float* xrow = B.X + (ok ? pt : 0) * (int64_t)d;
    // raw values: features >= d meet zero rows of Theta, rows >= n are masked in the epilogue
    if (UN && (st >= edge_st || d < 3)) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int f = ch * 32 + h * 16 + 4 * q;
        const f32x4 t = load4_edge(xrow, f < d ? f : 0, d);
#pragma unroll
        for (int e = 0; e < 4; ++e) xv[ch][4 * q + e] = t[e];
      }
      return;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int f = ch * 32 + h * 16 + 4 * q;
      const f32x4 t = load4<UN>(xrow + (f < d ? f : 0));
      xv[ch][4 * q + 0] = t.x;
      xv[ch][4 * q + 1] = t.y;
      xv[ch][4 * q + 2] = t.z;
      xv[ch][4 * q + 3] = t.w;
    }
  };
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
    __builtin_amdgcn_sched_barrier(0);
    load_x(sb0, ch);
  }
  __builtin_amdgcn_sched_barrier(0);

  for (int64_t st = sb0; st < sb1; ++st) {
    __builtin_amdgcn_sched_barrier(0);
    const int64_t pt = st * kTPB + wave * 32 + li;
    const bool vpt = pt < n;
    float* urow = B.U + (vpt ? pt : 0) * (int64_t)r;
    // epilogue operands, issued before the matrix product (raw; scaled and masked at use)
    f32x4 uraw[NB][4];
    if (UN && (st >= edge_st || r < 3)) {
#pragma unroll
      for (int m = 0; m < NB; ++m)
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) {
          const int c = 32 * m + 8 * qd + 4 * h;
          uraw[m][qd] = load4_edge(urow, c < r ? c : 0, r);
        }
    } else {
#pragma unroll
      for (int m = 0; m < NB; ++m)
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) {
          const int c = 32 * m + 8 * qd + 4 * h;
          uraw[m][qd] = load4<UN>(urow + (c < r ? c : 0));
        }
    }
    const float yraw = B.y[vpt ? pt : 0];
    __builtin_amdgcn_sched_barrier(0);

    f32x16 acc[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int m = 0; m < NB; ++m) {
          const f32x4 a = *reinterpret_cast<const f32x4*>(th_s + (((ch * 4 + j) * NB + m) * 64 + lane) * 4);
          acc[m] = mfma32x32x2(a.x, xv[ch][4 * j + 0], acc[m]);
          acc[m] = mfma32x32x2(a.y, xv[ch][4 * j + 1], acc[m]);
          acc[m] = mfma32x32x2(a.z, xv[ch][4 * j + 2], acc[m]);
          acc[m] = mfma32x32x2(a.w, xv[ch][4 * j + 3], acc[m]);
        }
      __builtin_amdgcn_sched_barrier(0);
      load_x(st + 1, ch);  // this chunk of the next tile: a whole tile of lead time
      __builtin_amdgcn_sched_barrier(0);
    }

    int lds_off = 0;  // opaque zero offset: keeps the reads in LDS address space
    asm volatile("" : "+v"(lds_off));
    const float* psl = ps + lds_off;
    const float* ssl = ss + lds_off;
    float u[NB][16];
#pragma unroll
    for (int m = 0; m < NB; ++m)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        const int c = 32 * m + 8 * qd + 4 * h;
        const bool ok = vpt && c < r;
#pragma unroll
        for (int e = 0; e < 4; ++e) u[m][4 * qd + e] = (UN ? ok && c + e < r : ok) ? uraw[m][qd][e] * cf : 0.f;
      }
    float dotf = 0.f;
#pragma unroll
    for (int m = 0; m < NB; ++m)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        const f32x4 pv = *reinterpret_cast<const f32x4*>(psl + 32 * m + 8 * qd + 4 * h);
        dotf = fmaf(u[m][4 * qd + 0], pv.x, dotf);
        dotf = fmaf(u[m][4 * qd + 1], pv.y, dotf);
        dotf = fmaf(u[m][4 * qd + 2], pv.z, dotf);
        dotf = fmaf(u[m][4 * qd + 3], pv.w, dotf);
      }
    dotf += shfl_xor_f(dotf, 32);
    const float ybar = vpt ? fmaf(gam, dotf - 1.0f, yraw) : 0.f;
#pragma unroll
    for (int m = 0; m < NB; ++m) {
      float wv[16];
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        const int c = 32 * m + 8 * qd + 4 * h;
        const f32x4 pv = *reinterpret_cast<const f32x4*>(psl + c);
        const f32x4 sv = *reinterpret_cast<const f32x4*>(ssl + c);
        const float pe[4] = {pv.x, pv.y, pv.z, pv.w};
        const float se[4] = {sv.x, sv.y, sv.z, sv.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float uu = u[m][4 * qd + e];
          float t = fmaf(two_alpha, acc[m][4 * qd + e], uu);
          t = fmaf(neg_alpha, ybar * pe[e], t);
          t = fmaf(neg_alpha, se[e], t);
          float w = fmaxf(t, 0.f);
          if (!vpt || c + e >= r) w = 0.f;
          wv[4 * qd + e] = w;
          const double wd = (double)w, ud = (double)uu;
          sa = fma(wd, wd, sa);
          sb = fma(ud, ud, sb);
          sh = fma(wd, ud, sh);
        }
        if constexpr (UN) {
          store4<true>(urow, c, r, vpt && c < r, &wv[4 * qd]);
        } else {
          // unconditional store (invalid lanes write the dump slot): no branch around it
          float* dst = (vpt && c < r) ? (urow + c) : B.dump;
          f32x4 o = {wv[4 * qd + 0], wv[4 * qd + 1], wv[4 * qd + 2], wv[4 * qd + 3]};
          *reinterpret_cast<f32x4*>(dst) = o;
        }
      }
      reduce_scatter<16, 16>(wv, li);
      colacc[m] += (double)wv[0];
    }
  }

  for (int c = tid; c < 4 * r32; c += kThreads) colred[c] = 0.0;
  __syncthreads();
#pragma unroll
  for (int m = 0; m < NB; ++m) {
    const double v = colacc[m] + shfl_xor_d(colacc[m], 1);
    if ((li & 1) == 0) {
      const int col = 32 * m + 8 * (base >> 2) + 4 * h + (base & 3);
      colred[wave * r32 + col] = v;
    }
  }
  __syncthreads();
  double* out = B.b_part + (int64_t)blockIdx.x * (4 + r32);
  for (int c = tid; c < r32; c += kThreads)
    out[4 + c] = ((colred[c] + colred[r32 + c]) + colred[2 * r32 + c]) + colred[3 * r32 + c];
  const double ta = block_sum_d(sa, dred);
  const double tb2 = block_sum_d(sb, dred);
  const double th = block_sum_d(sh, dred);
  if (tid == 0) {
    out[0] = ta;
    out[1] = tb2;
    out[2] = th;
    out[3] = 0.0;
  }
}

// ---------------------------------------------------------------------------
// Control after pass B: Algorithm 2 steps (d)-(f).
// ---------------------------------------------------------------------------
// Workgroup b writes p for its columns (each forms c from the same sums), workgroup 0 the rest.
// (A breakdown, set by workgroup 0, may keep another workgroup from its columns; none are written
// on a breakdown anyway.)
// defer: as ctl_a_work.  A stop that this iteration's control after pass A set is marked 2 here: the
// Theta sums of later iterations, which share their launch with that control, go by it.
__global__ __launch_bounds__(kThreads) void k_ctl_b(Geometry g, Bufs B, StepArgs S, int defer) {
  DevCtl* ctl = B.ctl;
  if (halted_workgroup(ctl)) {
    if (blockIdx.x == 0 && threadIdx.x == 0 && ctl->stop == 1) ctl->stop = 2;
    return;
  }
  __shared__ double red[kRedDoubles];
  const int tid = threadIdx.x, blk = blockIdx.x;
  const int C = 4 + g.r32;
  const int64_t t = ctl->t_done;
  const double obj0 = ctl->objective;
  const CtlSums sm =
      ctl_sums<false, true, kThreads>(nullptr, B.b_part, g.GB, C, blk, (defer && blk == 0) ? B.th2_part : nullptr, g.RT, red);
  const float cs = norm_scale(sm.a, sm.over, S.K);
  const int pc = kCtlCols * blk + tid - 4;
  if (cs > 0.f && tid < kCtlCols && pc >= 0 && pc < g.r32)
    B.p[pc] = (pc < g.r) ? (float)((double)cs * sm.col_b) : 0.f;
  if (blk > 0) return;
  if (tid == 0) {
    const double a = sm.a, b = sm.b, h = sm.h, over = sm.over, th2 = sm.th2;
    const double nu = sqrt(a);
    nlr_iter_stats* rec = &B.hist[t % kHistCap];
    if (defer) {
      const double obj = obj0 - th2;
      ctl->objective = obj;
      ctl->theta_fro2 = th2;
      rec->objective = obj;
      rec->theta_fro2 = th2;
    }
    rec->a = a;
    rec->b = b;
    rec->h = h;
    if (over > 0.0) {
      // a split-fp16 operand of W left fp16's range (the fused pass's flag)
      ctl->breakdown = kRangeError;
      rec->breakdown = kRangeError;
    } else if (!(nu > 1e-20) || !isfinite(a)) {
      ctl->breakdown = 1;
      rec->breakdown = 1;
    } else {
      const float cf = cs;
      const double c = (double)cf;
      double D = c * c * a + b - 2.0 * c * h;
      if (D < 0.0) D = 0.0;
      const double delta = sqrt(D) / sqrt(S.K);
      const int gate = D < S.eps_d * S.eps_d * S.K;
      ctl->a = a;
      ctl->b = b;
      ctl->h = h;
      ctl->Delta = D;
      ctl->delta = delta;
      ctl->gate = gate;
      ctl->c_f = cf;
      ctl->t_done = t + 1;
      rec->c = cf;
      rec->delta = delta;
      rec->dual_step = gate;
    }
  }
}

// ---------------------------------------------------------------------------
// One-pass iteration (the eight-wave fused pass B does the row work too), control
// after the pass.  Unless the row pass ran first (rows_first: the
// previous iteration's stopping rule could fire, and k_ctl_a has decided it and
// written the record), the pass did the row work of this iteration -- the end of
// the previous one: its gated dual step, q and the objective terms -- before the
// primal step; the stopping rule could not fire then, and rho and the objective
// are recorded here.  Then as k_ctl_b, the column sums P of W and W^T ytilde for
// the next iteration's s, and whether the next iteration's row pass runs first.
// ---------------------------------------------------------------------------
// Workgroup b writes p, P and W^T ytilde for its columns, workgroup 0 the rest, as k_ctl_b.
__global__ __launch_bounds__(kThreads) void k_ctl_one(Geometry g, Bufs B, StepArgs S) {
  DevCtl* ctl = B.ctl;
  if (halted_workgroup(ctl)) return;
  __shared__ double red[kRedDoubles];
  const int tid = threadIdx.x, blk = blockIdx.x;
  const int C = 4 + g.r32;
  const int64_t t0 = ctl->t_done;
  const int rows_first = ctl->rows_first;
  const CtlSums sm =
      ctl_sums<true, true, kThreads>(B.a_part, B.b_part, g.GB, C, blk, blk == 0 ? B.th2_part : nullptr, g.RT, red);
  const float cs = norm_scale(sm.a, sm.over, S.K);
  const int pc = kCtlCols * blk + tid - 4;
  if (cs > 0.f && tid < kCtlCols && pc >= 0 && pc < g.r32) {
    const bool ok = pc < g.r;
    B.p[pc] = ok ? (float)((double)cs * sm.col_b) : 0.f;
    B.gram_vec[pc] = ok ? sm.col_b : 0.0;
    B.gram_vec[g.r32 + pc] = ok ? sm.col_a : 0.0;
  }
  if (blk > 0) return;
  if (tid == 0) {
    const int64_t t = t0;
    if (!rows_first) {
      const double qq = sm.qq, yq = sm.yq, th2 = sm.th2;
      const double rho = sqrt(qq * S.inv_n);
      ctl->rho = rho;
      if (S.end_work && t > 0) {
        nlr_iter_stats* prev = &B.hist[(t - 1) % kHistCap];
        prev->rho = rho;
        prev->stop = 0;
      }
      const double obj = -th2 + yq + 0.5 * S.beta * S.inv_n * qq;
      ctl->objective = obj;
      ctl->theta_fro2 = th2;
      nlr_iter_stats* cur = &B.hist[t % kHistCap];
      cur->t = t;
      cur->objective = obj;
      cur->theta_fro2 = th2;
      cur->rho = 0.0;
      cur->stop = 0;
    }
    const double a = sm.a, b = sm.b, h = sm.h;
    const double nu = sqrt(a);
    nlr_iter_stats* rec = &B.hist[t % kHistCap];
    rec->a = a;
    rec->b = b;
    rec->h = h;
    rec->dual_step = 0;
    rec->breakdown = 0;
    if (sm.over > 0.0) {
      // the split W operand left fp16's range: stop before Theta and s use it
      ctl->breakdown = kRangeError;
      rec->breakdown = kRangeError;
      rec->c = 0.f;
      rec->delta = 0.0;
    } else if (!(nu > 1e-20) || !isfinite(a)) {
      // W_{t+1} has overwritten the factor (Algorithm 2 order)
      ctl->breakdown = 1;
      rec->breakdown = 1;
      rec->c = 0.f;
      rec->delta = 0.0;
    } else {
      const float cf = cs;
      const double c = (double)cf;
      double D = c * c * a + b - 2.0 * c * h;
      if (D < 0.0) D = 0.0;
      const double delta = sqrt(D) / sqrt(S.K);
      const int gate = D < S.eps_d * S.eps_d * S.K;
      ctl->a = a;
      ctl->b = b;
      ctl->h = h;
      ctl->Delta = D;
      ctl->delta = delta;
      ctl->gate = gate;
      ctl->c_f = cf;
      ctl->c_gram = c;
      ctl->t_done = t + 1;
      rec->c = cf;
      rec->delta = delta;
      rec->dual_step = gate;
      // the next iteration of this call has this one's end-of-iteration work pending
      StepArgs nx = S;
      nx.end_work = 1;
      ctl->rows_first = stop_possible(ctl, nx) ? 1 : 0;
    }
  }
}

// At the start of a host call (one workgroup): s from the stored Gram terms with the
// beta of this call when they are valid, and whether the first iteration's row pass
// runs before its pass: 2 when there are no Gram terms (after nlr_init; s then comes
// from the row pass), 1 when the stopping rule of the previous iteration may fire
// under this call's arguments (eps, T_min; the row pass settles the rule, s stays
// the Gram-derived one), else 0.
__global__ __launch_bounds__(64) void k_onepass_begin(Geometry g, Bufs B, StepArgs S, int gram_valid) {
  if (B.ctl->breakdown) return;
  const int r32 = g.r32;
  const int k = threadIdx.x;
  if (k == 0) B.ctl->stop = 0;  // the stop of an earlier call
  if (k == 0) B.ctl->rows_first = !gram_valid ? 2 : (stop_possible(B.ctl, S) ? 1 : 0);
  if (!gram_valid || k >= r32) return;
  const float sk = s_from_gram(B, r32, k, B.gram_vec[2 * r32 + k], S.gamma_f);
  B.s[k] = (k < g.r) ? sk : 0.f;
}

// ---------------------------------------------------------------------------
// Row-argmax labels, lowest index on ties.  A row is read by the 16 lanes of a DPP
// row, four rows per wave and step: with 16-byte rows (VEC) lane j reads columns
// 4j .. 4j + 3, 64 + 4j .. (NCK = ceil(r / 64) pieces), so one load instruction covers
// 256 contiguous bytes of each of its four rows, and a workgroup takes 16 RPS
// consecutive rows per step, all their loads issued before any is compared (pieces
// past the last column or row read a valid address and are skipped); otherwise lane j
// reads columns
// j, j + 16, ...  Each lane keeps its first maximum (columns in increasing order,
// strict >), then the 16 candidates are reduced pairwise: the larger value, the lower
// column on equal values.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void label_reduce16(float& best, int& arg) {
  constexpr int kNone = 0x7fffffff;
#pragma unroll
  for (int m = 1; m < 16; m <<= 1) {
    const float ob = shfl_xor_f(best, m);
    const int oa = __shfl_xor(arg, m, 64);
    if (oa != kNone && (arg == kNone || ob > best || (ob == best && oa < arg))) {
      best = ob;
      arg = oa;
    }
  }
}

template <bool VEC, int NCK, int RPS>
__global__ __launch_bounds__(kThreads) void k_labels(Geometry g, const float* __restrict__ U,
                                                     int32_t* __restrict__ labels) {
  constexpr int kNone = 0x7fffffff;  // no column seen yet
  const int lane = threadIdx.x & 63;
  const int j = lane & 15;
  const int64_t n = g.n;
  const int r = g.r;
  if (VEC) {
    // a workgroup takes 16 RPS consecutive rows per step; group g its rows 16 k + g
    const int64_t bstep = (int64_t)gridDim.x * 16 * RPS;
    for (int64_t b0 = (int64_t)blockIdx.x * 16 * RPS; b0 < n; b0 += bstep) {
      const int64_t i0 = b0 + (threadIdx.x >> 4);
      f32x4 v[RPS][NCK];
#pragma unroll
      for (int k = 0; k < RPS; ++k) {
        const int64_t i = i0 + 16 * k;
        const float* row = U + (i < n ? i : 0) * (int64_t)r;
#pragma unroll
        for (int q = 0; q < NCK; ++q) {
          const int c0 = 4 * j + 64 * q;
          v[k][q] = *reinterpret_cast<const f32x4*>(row + (c0 < r ? c0 : 0));
        }
      }
#pragma unroll
      for (int k = 0; k < RPS; ++k) {
        float best = 0.f;
        int arg = kNone;
#pragma unroll
        for (int q = 0; q < NCK; ++q) {
          const int c0 = 4 * j + 64 * q;  // r % 4 == 0: c0 + 3 < r when c0 < r
          if (c0 < r) {
            const float e[4] = {v[k][q].x, v[k][q].y, v[k][q].z, v[k][q].w};
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4)
              if (arg == kNone || e[e4] > best) {
                best = e[e4];
                arg = c0 + e4;
              }
          }
        }
        label_reduce16(best, arg);
        const int64_t i = i0 + 16 * k;
        if (i < n && j == 0) labels[i] = arg;
      }
    }
  } else {
    const int64_t rows_per_step = (int64_t)gridDim.x * (kThreads / 16);
    const int64_t first = (int64_t)blockIdx.x * (kThreads / 16) + (threadIdx.x >> 4);
    for (int64_t i = first; i - (threadIdx.x >> 4) < n; i += rows_per_step) {
      const bool vrow = i < n;
      const float* row = U + (vrow ? i : 0) * (int64_t)r;
      float best = 0.f;
      int arg = kNone;
      for (int c = j; c < r; c += 16) {
        const float v = row[c];
        if (arg == kNone || v > best) {
          best = v;
          arg = c;
        }
      }
      label_reduce16(best, arg);
      if (vrow && j == 0) labels[i] = arg;
    }
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// Kernels whose dynamic LDS exceeds 64 KiB need the per-function limit raised
// (gfx950 has 160 KiB of LDS per workgroup).
template <typename F>
static hipError_t allow_lds(F* kern, size_t lds) {
  if (lds <= (64u << 10)) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)lds);
}

template <int MBG, int NBG, bool UN>
static hipError_t theta_wide_launch(const Geometry& g, const Bufs& b, hipStream_t st) {
  const size_t tiles = (size_t)kTPA * ((MBG * 32 + 4) + (NBG * 32 + 4)) * 4;
  const size_t comb = MBG < 4 ? (size_t)MBG * NBG * 16 * 64 * 4 : 0;
  const size_t lds = tiles > comb ? tiles : comb;
  hipError_t e = allow_lds(k_theta_wide<MBG, NBG, UN>, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_theta_wide<MBG, NBG, UN>), dim3(g.GA, g.mgroups * g.ngroups), dim3(kThreads), lds, st, g, b);
  return hipGetLastError();
}

template <int MBG, int NBG>
static hipError_t theta_wide_un(const Geometry& g, const Bufs& b, hipStream_t st) {
  return (g.vec_x && g.vec_u) ? theta_wide_launch<MBG, NBG, false>(g, b, st)
                              : theta_wide_launch<MBG, NBG, true>(g, b, st);
}

// (one or two blocks of columns come with more than 128 features only: narrower shapes with up to 64
// columns are register-resident)
template <int MBG>
static hipError_t theta_wide_nbg(const Geometry& g, const Bufs& b, hipStream_t st) {
  if constexpr (MBG == 4) {
    if (g.NBG == 1) return theta_wide_un<MBG, 1>(g, b, st);
    if (g.NBG == 2) return theta_wide_un<MBG, 2>(g, b, st);
  }
  switch (g.NBG) {
    case 4: return theta_wide_un<MBG, 4>(g, b, st);
    case 5: return theta_wide_un<MBG, 5>(g, b, st);
    case 7: return theta_wide_un<MBG, 7>(g, b, st);
    default: return hipErrorInvalidValue;
  }
}

static hipError_t launch_theta_wide(const Geometry& g, const Bufs& b, hipStream_t st) {
  switch (g.MBG) {
    case 1: return theta_wide_nbg<1>(g, b, st);
    case 2: return theta_wide_nbg<2>(g, b, st);
    case 4: return theta_wide_nbg<4>(g, b, st);
    default: return hipErrorInvalidValue;
  }
}

template <bool FINISH>
static hipError_t launch_rows_wide(const Geometry& g, const Bufs& b, const StepArgs& a, hipStream_t st) {
  const dim3 grid(g.GAF), blk(kThreads);
  if (g.r <= 16) {
    hipLaunchKernelGGL((k_rows_wide<16, 1, FINISH>), grid, blk, 0, st, g, b, a);
    return hipGetLastError();
  }
  if (g.r <= 32) {
    hipLaunchKernelGGL((k_rows_wide<32, 1, FINISH>), grid, blk, 0, st, g, b, a);
    return hipGetLastError();
  }
  switch ((g.r + 63) / 64) {
    case 1: hipLaunchKernelGGL((k_rows_wide<64, 1, FINISH>), grid, blk, 0, st, g, b, a); break;
    case 2: hipLaunchKernelGGL((k_rows_wide<64, 2, FINISH>), grid, blk, 0, st, g, b, a); break;
    case 3: hipLaunchKernelGGL((k_rows_wide<64, 3, FINISH>), grid, blk, 0, st, g, b, a); break;
    case 4: hipLaunchKernelGGL((k_rows_wide<64, 4, FINISH>), grid, blk, 0, st, g, b, a); break;
    case 5: hipLaunchKernelGGL((k_rows_wide<64, 5, FINISH>), grid, blk, 0, st, g, b, a); break;
    case 6: hipLaunchKernelGGL((k_rows_wide<64, 6, FINISH>), grid, blk, 0, st, g, b, a); break;
    case 7: hipLaunchKernelGGL((k_rows_wide<64, 7, FINISH>), grid, blk, 0, st, g, b, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// (the row pass belongs to the single-pass form, whose rows are whole aligned pieces)
template <int FV, int NGF, int CV, bool UN>
static hipError_t pass_a_rows_mode(const Geometry& g, const Bufs& b, const StepArgs& a, int mode, hipStream_t st) {
  const dim3 grid(g.GA), blk(kThreads);
  if (mode == kPassFinish)
    hipLaunchKernelGGL((k_pass_a_rows<FV, NGF, CV, kPassFinish, UN>), grid, blk, 0, st, g, b, a);
  else if (mode == kPassIter)
    hipLaunchKernelGGL((k_pass_a_rows<FV, NGF, CV, kPassIter, UN>), grid, blk, 0, st, g, b, a);
  else if constexpr (!UN)
    hipLaunchKernelGGL((k_pass_a_rows<FV, NGF, CV, kPassRows, UN>), grid, blk, 0, st, g, b, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

// rows that are not whole aligned pieces: the fewest pieces of up to four features a lane
static hipError_t pass_a_un_dispatch(const Geometry& g, const Bufs& b, const StepArgs& a, int mode, hipStream_t st) {
  switch (g.a_fv * 100 + g.a_ngf * 10 + g.a_cv) {
    case 111: return pass_a_rows_mode<1, 1, 1, true>(g, b, a, mode, st);
    case 112: return pass_a_rows_mode<1, 1, 2, true>(g, b, a, mode, st);
    case 114: return pass_a_rows_mode<1, 1, 4, true>(g, b, a, mode, st);
    case 211: return pass_a_rows_mode<2, 1, 1, true>(g, b, a, mode, st);
    case 212: return pass_a_rows_mode<2, 1, 2, true>(g, b, a, mode, st);
    case 214: return pass_a_rows_mode<2, 1, 4, true>(g, b, a, mode, st);
    case 411: return pass_a_rows_mode<4, 1, 1, true>(g, b, a, mode, st);
    case 412: return pass_a_rows_mode<4, 1, 2, true>(g, b, a, mode, st);
    case 414: return pass_a_rows_mode<4, 1, 4, true>(g, b, a, mode, st);
    case 421: return pass_a_rows_mode<4, 2, 1, true>(g, b, a, mode, st);
    case 422: return pass_a_rows_mode<4, 2, 2, true>(g, b, a, mode, st);
    case 424: return pass_a_rows_mode<4, 2, 4, true>(g, b, a, mode, st);
    default: return hipErrorInvalidValue;
  }
}

static hipError_t pass_a_rows_dispatch(const Geometry& g, const Bufs& b, const StepArgs& a, int finish,
                                       hipStream_t st) {
  // narrow factors in the single-Xhat-pass form: the row and finish passes (both, so
  // that their row dots agree) pack eight lanes per row; pass A with its product keeps
  // the 16-lane layout
  if (g.fused && g.r <= 16 && g.r % 2 == 0 && (finish == kPassRows || finish == kPassFinish)) {
    if (finish == kPassFinish)
      hipLaunchKernelGGL((k_rows_narrow<kPassFinish>), dim3(g.GA), dim3(kThreads), 0, st, g, b, a);
    else
      hipLaunchKernelGGL((k_rows_narrow<kPassRows>), dim3(g.GA), dim3(kThreads), 0, st, g, b, a);
    return hipGetLastError();
  }
  if (g.a_un) return pass_a_un_dispatch(g, b, a, finish, st);
  const int key = g.a_fv * 100 + g.a_ngf * 10 + g.a_cv;
  switch (key) {
    case 111: return pass_a_rows_mode<1, 1, 1, false>(g, b, a, finish, st);
    case 112: return pass_a_rows_mode<1, 1, 2, false>(g, b, a, finish, st);
    case 114: return pass_a_rows_mode<1, 1, 4, false>(g, b, a, finish, st);
    case 211: return pass_a_rows_mode<2, 1, 1, false>(g, b, a, finish, st);
    case 212: return pass_a_rows_mode<2, 1, 2, false>(g, b, a, finish, st);
    case 214: return pass_a_rows_mode<2, 1, 4, false>(g, b, a, finish, st);
    case 221: return pass_a_rows_mode<2, 2, 1, false>(g, b, a, finish, st);
    case 222: return pass_a_rows_mode<2, 2, 2, false>(g, b, a, finish, st);
    case 224: return pass_a_rows_mode<2, 2, 4, false>(g, b, a, finish, st);
    case 241: return pass_a_rows_mode<2, 4, 1, false>(g, b, a, finish, st);
    case 242: return pass_a_rows_mode<2, 4, 2, false>(g, b, a, finish, st);
    case 244: return pass_a_rows_mode<2, 4, 4, false>(g, b, a, finish, st);
    case 411: return pass_a_rows_mode<4, 1, 1, false>(g, b, a, finish, st);
    case 412: return pass_a_rows_mode<4, 1, 2, false>(g, b, a, finish, st);
    case 414: return pass_a_rows_mode<4, 1, 4, false>(g, b, a, finish, st);
    case 421: return pass_a_rows_mode<4, 2, 1, false>(g, b, a, finish, st);
    case 422: return pass_a_rows_mode<4, 2, 2, false>(g, b, a, finish, st);
    case 424: return pass_a_rows_mode<4, 2, 4, false>(g, b, a, finish, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_pass_u(const Geometry& g, const Bufs& b, const StepArgs& a, hipStream_t st) {
  if (!g.a_rows) return hipErrorInvalidValue;
  return pass_a_rows_dispatch(g, b, a, kPassRows, st);
}

hipError_t launch_pass_a(const Geometry& g, const Bufs& b, const StepArgs& a, bool finish, hipStream_t st) {
  if (g.a_rows) return pass_a_rows_dispatch(g, b, a, finish ? kPassFinish : kPassIter, st);
  if (finish) return launch_rows_wide<true>(g, b, a, st);
  const hipError_t e = launch_rows_wide<false>(g, b, a, st);
  return e != hipSuccess ? e : launch_theta_wide(g, b, st);
}

hipError_t launch_theta_sum(const Geometry& g, const Bufs& b, const StepArgs& a, int64_t rows, bool scaled,
                            float gamma_f, bool with_ctl_a, hipStream_t st) {
  // one-pass iteration (partials of its pass): workgroups after the RT of Theta form (W^T W) P; two-pass
  // form: they do the control after pass A
  const int more = (g.fused8 && scaled) ? (g.r32 * g.r32) / 64 : (with_ctl_a ? ctl_blocks(g) : 0);
  const int64_t ctl_rows = with_ctl_a ? (int64_t)(g.a_rows ? g.GA : g.GAF) : 0;
  if (g.RT >= kThetaWide)
    hipLaunchKernelGGL(k_theta_sum<true>, dim3(g.RT / 4 + more), dim3(kThreads), 0, st, g, b, a, rows, scaled ? 1 : 0,
                       gamma_f, ctl_rows);
  else
    hipLaunchKernelGGL(k_theta_sum<false>, dim3(g.RT + more), dim3(kRedThreads), 0, st, g, b, a, rows, scaled ? 1 : 0,
                       gamma_f, ctl_rows);
  return hipGetLastError();
}

hipError_t launch_ctl_a(const Geometry& g, const Bufs& b, const StepArgs& a, int64_t rows, bool finish,
                        hipStream_t st) {
  hipLaunchKernelGGL(k_ctl_a, dim3(finish ? 1 : ctl_blocks(g)), dim3(kThreads), 0, st, g, b, a, finish ? 1 : 0, rows);
  return hipGetLastError();
}

hipError_t launch_ctl_b(const Geometry& g, const Bufs& b, const StepArgs& a, bool defer, hipStream_t st) {
  hipLaunchKernelGGL(k_ctl_b, dim3(ctl_blocks(g)), dim3(kThreads), 0, st, g, b, a, defer ? 1 : 0);
  return hipGetLastError();
}

template <int CG>
static hipError_t pass_b_stream_launch(const Geometry& g, const Bufs& b, const StepArgs& a, hipStream_t st) {
  // Theta buffers, the column-sum table, p, s, the reduction
  const size_t lds = (size_t)2 * 4 * CG * 256 * 4 + (size_t)4 * g.r32 * 8 + (size_t)2 * g.r32 * 4 + 4 * 8;
  if (lds > (160u << 10)) return hipErrorInvalidValue;
  const bool un = !(g.vec_x && g.vec_u);
  hipError_t e = un ? allow_lds(k_pass_b_stream<CG, true>, lds) : allow_lds(k_pass_b_stream<CG, false>, lds);
  if (e != hipSuccess) return e;
  if (un)
    hipLaunchKernelGGL((k_pass_b_stream<CG, true>), dim3(g.GB), dim3(kThreads), lds, st, g, b, a);
  else
    hipLaunchKernelGGL((k_pass_b_stream<CG, false>), dim3(g.GB), dim3(kThreads), lds, st, g, b, a);
  return hipGetLastError();
}

template <int NB, int NCH>
static hipError_t pass_b_res_launch(const Geometry& g, const Bufs& b, const StepArgs& a, hipStream_t st) {
  if (g.vec_x && g.vec_u)
    hipLaunchKernelGGL((k_pass_b_res<NB, NCH, false>), dim3(g.GB), dim3(kThreads), g.ldsB_bytes, st, g, b, a);
  else
    hipLaunchKernelGGL((k_pass_b_res<NB, NCH, true>), dim3(g.GB), dim3(kThreads), g.ldsB_bytes, st, g, b, a);
  return hipGetLastError();
}

hipError_t launch_pass_b(const Geometry& g, const Bufs& b, const StepArgs& a, hipStream_t st) {
  if (g.split_b) return launch_pass_b_split(g, b, a, st);
  if (g.b_res) {
    switch (g.NB * 10 + g.nch) {
      case 11: return pass_b_res_launch<1, 1>(g, b, a, st);
      case 12: return pass_b_res_launch<1, 2>(g, b, a, st);
      case 13: return pass_b_res_launch<1, 3>(g, b, a, st);
      case 14: return pass_b_res_launch<1, 4>(g, b, a, st);
      case 21: return pass_b_res_launch<2, 1>(g, b, a, st);
      case 22: return pass_b_res_launch<2, 2>(g, b, a, st);
      case 23: return pass_b_res_launch<2, 3>(g, b, a, st);
      case 24: return pass_b_res_launch<2, 4>(g, b, a, st);
      case 41: return pass_b_res_launch<4, 1>(g, b, a, st);
      case 42: return pass_b_res_launch<4, 2>(g, b, a, st);
      default: return hipErrorInvalidValue;
    }
  }
  switch (g.NB) {
    case 1: return pass_b_stream_launch<1>(g, b, a, st);
    case 2: return pass_b_stream_launch<2>(g, b, a, st);
    case 10: return pass_b_stream_launch<2>(g, b, a, st);  // five exact groups of two
    default: return pass_b_stream_launch<4>(g, b, a, st);  // groups of four blocks
  }
}

hipError_t launch_ctl_one(const Geometry& g, const Bufs& b, const StepArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(k_ctl_one, dim3(ctl_blocks(g)), dim3(kThreads), 0, st, g, b, a);
  return hipGetLastError();
}

hipError_t launch_onepass_begin(const Geometry& g, const Bufs& b, const StepArgs& a, bool gram_valid,
                                hipStream_t st) {
  hipLaunchKernelGGL(k_onepass_begin, dim3(1), dim3(64), 0, st, g, b, a, gram_valid ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_labels(const Geometry& g, const Bufs& b, int32_t* labels, hipStream_t st) {
  // 16 rows per workgroup and step; enough workgroups for eight per CU
  int64_t blocks = (g.n + 15) / 16;
  if (blocks > 2048) blocks = 2048;
  const dim3 grid((unsigned)blocks), blk(kThreads);
  const float* U = b.U;
  if (!g.vec_u) {
    hipLaunchKernelGGL((k_labels<false, 1, 1>), grid, blk, 0, st, g, U, labels);
  } else {
    // rows per step so that a lane has four to eight pieces in flight
    switch ((g.r + 63) / 64) {
      case 1: hipLaunchKernelGGL((k_labels<true, 1, 4>), grid, blk, 0, st, g, U, labels); break;
      case 2: hipLaunchKernelGGL((k_labels<true, 2, 4>), grid, blk, 0, st, g, U, labels); break;
      case 3: hipLaunchKernelGGL((k_labels<true, 3, 2>), grid, blk, 0, st, g, U, labels); break;
      case 4: hipLaunchKernelGGL((k_labels<true, 4, 2>), grid, blk, 0, st, g, U, labels); break;
      case 5: hipLaunchKernelGGL((k_labels<true, 5, 1>), grid, blk, 0, st, g, U, labels); break;
      case 6: hipLaunchKernelGGL((k_labels<true, 6, 1>), grid, blk, 0, st, g, U, labels); break;
      case 7: hipLaunchKernelGGL((k_labels<true, 7, 1>), grid, blk, 0, st, g, U, labels); break;
      default: return hipErrorInvalidValue;
    }
  }
  return hipGetLastError();
}

}  // namespace nlr
