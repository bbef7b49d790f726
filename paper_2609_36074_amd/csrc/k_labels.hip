// Cluster labels from the factor by spectral embedding and K-means (Appendix D,
// "Recover cluster labels from U") for gfx950.
//
//   G = U^T U (FP64, r x r, fixed-order partial sums, fp64 matrix cores);
//   G = V Lambda V^T by Jacobi rotations: up to 64 columns in one workgroup, more as a
//   block Jacobi over pairs of 32-column blocks (one workgroup per pair);
//   P = V_K Lambda_K^{-1/2}: the embedding E = U P holds the leading K left
//   singular vectors of U (up to a rotation inside their span, which leaves all
//   distances, and so the labels, unchanged);
//   Lloyd's iteration on the rows of E from the embedded seed rows.  E is never formed:
//   with M = P cent^T (r x K) the squared distance of row i to centroid k is
//   |e_i|^2 + |cent_k|^2 - 2 u_i M_k, so a pass is one product U M with the argmin over k in
//   registers.  It runs on the fp16 matrix cores with two-term operand splits, under a bound on
//   its rounding: a row whose two smallest values lie within it is decided by the same form in
//   FP64 over its candidates, and one whose values are too close for that, or with more than four
//   candidates, by the distances themselves (FP64, lowest index on ties), so that the labels are
//   those of FP64 distances.  The
//   cluster sums S_k = sum of u_i over the rows of k are taken in 64-bit integers (below), and
//   cent_k = (S_k / count) P (a centroid without rows stays in place).
// The device notes the first pass that changes no label; passes enqueued after it return
// at entry.
#include "k_common.hpp"

namespace nlr {

constexpr int kLabUpd = 512;      // threads of the centroid kernel
constexpr int kJacLd = 65;        // LDS row stride (doubles) of the Jacobi and apply tiles

// flag slots
enum { kFlagDegenerate = 0, kFlagDone = 1, kFlagPasses = 2, kFlagEig = 3 };

// A = the sum of the Gram partials (mirrored below the 64-block diagonal), zero padded to
// r64 x r64; V = I; the power-of-two scale of each column's integer sums: sum_i |u_ic| <=
// sqrt(n G_cc) < 2^e, so sums of u 2^(61 - e) stay below 2^61.
__global__ __launch_bounds__(kThreads) void k_lab_gram_reduce(Geometry g, LabScratch L) {
  const int64_t rr = (int64_t)g.r * g.r;
  const int e = blockIdx.x * kThreads + threadIdx.x;
  if (e == 0) {
    for (int k = 0; k < 8; ++k) L.flag[k] = 0;
    *L.changed = 0;
  }
  if (e >= L.r64 * L.r64) return;
  const int i = e / L.r64, j = e - (e / L.r64) * L.r64;
  double s = 0.0;
  if (i < g.r && j < g.r) {
    const int64_t src = (i / 64 > j / 64) ? (int64_t)j * g.r + i : (int64_t)i * g.r + j;
    for (int k0 = 0; k0 < L.GU; k0 += 8) {  // eight loads in flight, added in chunk order
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = L.gpart[(int64_t)(k0 + u < L.GU ? k0 + u : 0) * rr + src];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += k0 + u < L.GU ? v[u] : 0.0;
    }
  }
  L.A[e] = s;
  L.V[e] = (i == j) ? 1.0 : 0.0;
  if (i == j && i < g.r) {
    int ex = 0;
    double sc = 0.0;
    if (s > 0.0 && isfinite(s)) {
      (void)frexp(sqrt((double)g.n * s) * 1.0001, &ex);
      sc = ldexp(1.0, 61 - ex);
    }
    L.cscale[i] = sc;
    L.cinv[i] = sc > 0.0 ? 1.0 / sc : 0.0;
    L.ubound[i] = sqrt(s) * 1.0001;
  }
}

// Round-robin pairing of m players (m even): pair a of step t, lower index first.
__device__ __forceinline__ void lab_pair(int m, int t, int a, int& lo, int& hi) {
  const int x = (t + a) % (m - 1);
  const int y = a == 0 ? m - 1 : (t + m - 1 - a) % (m - 1);
  lo = x < y ? x : y;
  hi = x < y ? y : x;
}

// Jacobi rotations of the pivot block of pair blockIdx.x (two 32-column blocks of A, a
// 64 x 64 symmetric block in LDS): up to `sweeps` cyclic sweeps over its N leading columns,
// N / 2 disjoint rotations per step, ended early once the off-diagonal mass is at rounding
// level.  The rotated block replaces the pivot block of A; the rotations go to Q[pair]
// (block form, one sweep a visit) or to V (whole = 1: r <= 64, run to the end).
// What bounds it: the chain of N - 1 steps, each two barriers, the latency of a fp64 square
// root, divide and reciprocal root, and that of the 2 x 2 updates' LDS reads.  All rotations of
// a step and both sides of the updates are taken between the barriers; the update of Q by a
// step's rotations runs on the other waves while the first one forms the next step's.
constexpr int kJacThreads = 1024;
__global__ __launch_bounds__(kJacThreads) void k_lab_sub(LabScratch L, int step, int nb, int N, int sweeps, int whole,
                                                         int check, int last) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* As = reinterpret_cast<double*>(smem_raw);
  double* Qs = As + 64 * kJacLd;
  // rotations of the current and the previous step: c, s, and the two columns
  __shared__ double cs[2][32], sn[2][32], red[2][kJacThreads / 64], tot[2];
  __shared__ int pq[2][32];
  const int tid = threadIdx.x;
  const int a = blockIdx.x, np = nb / 2;
  if (L.flag[kFlagEig]) return;
  if (check) {  // start of a sweep after the first: off-diagonal mass after the last one
    double off = 0.0, dia = 0.0;
    for (int k = 0; k < np + np * (np - 1) / 2; ++k) off += L.jpart[k];
    for (int k = 0; k < np; ++k) dia += L.jpart[kLabJacParts + k];
    if (!(off > 1e-30 * (off + dia))) {
      if (a == 0 && tid == 0) L.flag[kFlagEig] = 1;
      return;
    }
  }
  int I, J;
  lab_pair(nb, step, a, I, J);
  const int ld = L.r64;
  for (int e = tid; e < 64 * 64; e += kJacThreads) {
    const int i = e >> 6, j = e & 63;
    const int gi = i < 32 ? 32 * I + i : 32 * J + i - 32, gj = j < 32 ? 32 * I + j : 32 * J + j - 32;
    As[i * kJacLd + j] = L.A[(int64_t)gi * ld + gj];
    Qs[i * kJacLd + j] = i == j ? 1.0 : 0.0;
  }
  __syncthreads();
  const int h = N >> 1;
  // the (k, l), k <= l, pair of rotations whose 2 x 2 block this thread updates: rows ra and
  // h - 1 - ra of the triangle make one run of h + 1 (at most 16 runs of 33)
  int uk = -1, ul = 0;
  if (tid < ((h + 1) >> 1) * (h + 1)) {
    const int ra = tid / (h + 1), rb = tid - ra * (h + 1);
    if (rb < h - ra) {
      uk = ra;
      ul = ra + rb;
    } else if (h - 1 - ra != ra) {
      uk = h - 1 - ra;
      ul = uk + rb - (h - ra);
    }
  }
  auto sums = [&]() {
    double off = 0.0, dia = 0.0;
    for (int e = tid; e < 64 * 64; e += kJacThreads) {
      const double v = As[(e >> 6) * kJacLd + (e & 63)];
      if ((e >> 6) == (e & 63))
        dia += v * v;
      else
        off += v * v;
    }
    for (int m = 32; m >= 1; m >>= 1) {
      off += shfl_xor_d(off, m);
      dia += shfl_xor_d(dia, m);
    }
    if ((tid & 63) == 0) {
      red[0][tid >> 6] = off;
      red[1][tid >> 6] = dia;
    }
    __syncthreads();
    if (tid < 2) {
      double t = 0.0;
      for (int w = 0; w < kJacThreads / 64; ++w) t += red[tid][w];
      tot[tid] = t;
    }
    __syncthreads();
  };
  // Q <- Q J with the rotations in slot b: row i = lane, rotations k = first, first + every, ...
  auto rotate_q = [&](int b, int first, int every) {
    const int i = tid & 63;
    for (int k = first; k < h; k += every) {
      const int p = pq[b][k] >> 8, q = pq[b][k] & 255;
      const double c = cs[b][k], s = sn[b][k];
      const double vp = Qs[i * kJacLd + p], vq = Qs[i * kJacLd + q];
      Qs[i * kJacLd + p] = c * vp - s * vq;
      Qs[i * kJacLd + q] = s * vp + c * vq;
    }
  };
  int slot = 0;
  bool pending = false;  // the previous step's rotations are not yet in Q
  for (int sw = 0; sw < sweeps; ++sw) {
    if (whole) {
      sums();
      if (!(tot[0] > 1e-30 * (tot[0] + tot[1]))) break;
    }
    for (int t = 0; t < N - 1; ++t) {
      if (tid < 64) {
        if (tid < h) {
          // round-robin pairing, as lab_pair
          int x = t + tid, y = t + N - 1 - tid;
          x -= x >= N - 1 ? N - 1 : 0;
          y -= y >= N - 1 ? N - 1 : 0;
          if (tid == 0) y = N - 1;
          const int p = x < y ? x : y, q = x < y ? y : x;
          // tan of the angle: t = sign(d) b / (|d| + sqrt(d^2 + b^2)), d = a_qq - a_pp, b = 2 a_pq
          const double b = 2.0 * As[p * kJacLd + q], d = As[q * kJacLd + q] - As[p * kJacLd + p];
          const double hyp = d * d + b * b;
          double c = 1.0, s = 0.0;
          if (b != 0.0 && hyp > 0.0) {
            const double tt = (d >= 0.0 ? b : -b) / (fabs(d) + sqrt(hyp));
            c = rsqrt(1.0 + tt * tt);
            s = tt * c;
          }
          cs[slot][tid] = c;
          sn[slot][tid] = s;
          pq[slot][tid] = (p << 8) | q;
        }
      } else if (pending) {
        rotate_q(slot ^ 1, (tid >> 6) - 1, kJacThreads / 64 - 1);
      }
      __syncthreads();
      if (uk >= 0) {
        const int k = uk, l = ul;
        const double ck = cs[slot][k], sk = sn[slot][k], cl = cs[slot][l], sl = sn[slot][l];
        const int pk = pq[slot][k] >> 8, qk = pq[slot][k] & 255, pl = pq[slot][l] >> 8, ql = pq[slot][l] & 255;
        const double b00 = As[pk * kJacLd + pl], b01 = As[pk * kJacLd + ql];
        const double b10 = As[qk * kJacLd + pl], b11 = As[qk * kJacLd + ql];
        const double r00 = ck * b00 - sk * b10, r01 = ck * b01 - sk * b11;
        const double r10 = sk * b00 + ck * b10, r11 = sk * b01 + ck * b11;
        const double n00 = cl * r00 - sl * r01, n11 = sl * r10 + cl * r11;
        double n01 = sl * r00 + cl * r01, n10 = cl * r10 - sl * r11;
        if (k == l && sk != 0.0) n01 = n10 = 0.0;
        As[pk * kJacLd + pl] = n00;
        As[pk * kJacLd + ql] = n01;
        As[qk * kJacLd + pl] = n10;
        As[qk * kJacLd + ql] = n11;
        if (k != l) {
          As[pl * kJacLd + pk] = n00;
          As[ql * kJacLd + pk] = n01;
          As[pl * kJacLd + qk] = n10;
          As[ql * kJacLd + qk] = n11;
        }
      }
      __syncthreads();
      slot ^= 1;
      pending = true;
    }
  }
  if (pending) rotate_q(slot ^ 1, tid >> 6, kJacThreads / 64);
  __syncthreads();
  double* Qo = whole ? L.V : L.Q + (int64_t)a * 4096;
  for (int e = tid; e < 64 * 64; e += kJacThreads) {
    const int i = e >> 6, j = e & 63;
    const int gi = i < 32 ? 32 * I + i : 32 * J + i - 32, gj = j < 32 ? 32 * I + j : 32 * J + j - 32;
    L.A[(int64_t)gi * ld + gj] = As[i * kJacLd + j];
    Qo[e] = Qs[i * kJacLd + j];
  }
  if (last) {
    sums();
    if (tid == 0) {
      L.jpart[a] = tot[0];
      L.jpart[kLabJacParts + a] = tot[1];
    }
  }
}

// Rotations of one block-Jacobi step applied to the rest of A and to V: workgroup (a, b), a < b,
// takes A_ab <- Q_a^T A_ab Q_b (and its mirror); the others V rows 64 rb .. + 63, columns of pair
// b, <- times Q_b.  The pivot blocks themselves come rotated from k_lab_sub.  All operands are
// loaded into LDS at once, so one memory latency is paid (operands read from L2 inside the
// products: 15 us a step at 200 columns).
constexpr size_t kApplyLds = (64 * kJacLd + 2 * 64 * 64) * sizeof(double);
__global__ __launch_bounds__(kThreads) void k_lab_apply(LabScratch L, int step, int nb, int last) {
  if (L.flag[kFlagEig]) return;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* S = reinterpret_cast<double*>(smem_raw);
  double* Qa = S + 64 * kJacLd;
  double* Qb = Qa + 64 * 64;
  __shared__ double red[4];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, kq = lane >> 4, cl = lane & 15;
  const int np = nb / 2, nA = np * (np - 1) / 2, ld = L.r64;
  int x = blockIdx.x, a = 0, b, rb = 0;
  const bool isA = x < nA;
  if (isA) {
    while (x >= np - 1 - a) {
      x -= np - 1 - a;
      ++a;
    }
    b = a + 1 + x;
  } else {
    b = (x - nA) % np;
    rb = (x - nA) / np;
  }
  int Ia, Ja, Ib, Jb;
  lab_pair(nb, step, a, Ia, Ja);
  lab_pair(nb, step, b, Ib, Jb);
  auto row = [&](int i) { return !isA ? 64 * rb + i : (i < 32 ? 32 * Ia + i : 32 * Ja + i - 32); };
  auto col = [&](int j) { return j < 32 ? 32 * Ib + j : 32 * Jb + j - 32; };
  double* M = isA ? L.A : L.V;
  {
    double v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int e = tid + u * kThreads;
      v[u] = M[(int64_t)row(e >> 6) * ld + col(e & 63)];
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int e = tid + u * kThreads;
      Qb[e] = L.Q[(int64_t)b * 4096 + e];
      if (isA) Qa[e] = L.Q[(int64_t)a * 4096 + e];
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int e = tid + u * kThreads;
      S[(e >> 6) * kJacLd + (e & 63)] = v[u];
    }
  }
  __syncthreads();
  f64x4 acc[4];
  if (isA) {
    mm64_zero(acc);
    mm64<4>(16, [&](int k0) { return Qa[(k0 + kq) * 64 + 16 * w + cl]; },
            [&](int k0, int J) { return S[(k0 + kq) * kJacLd + 16 * J + cl]; }, acc);
    __syncthreads();
#pragma unroll
    for (int J = 0; J < 4; ++J)
#pragma unroll
      for (int v = 0; v < 4; ++v) S[(16 * w + 4 * v + kq) * kJacLd + 16 * J + cl] = acc[J][v];
    __syncthreads();
  }
  mm64_zero(acc);
  mm64<4>(16, [&](int k0) { return S[(16 * w + cl) * kJacLd + k0 + kq]; },
          [&](int k0, int J) { return Qb[(k0 + kq) * 64 + 16 * J + cl]; }, acc);
  double sq = 0.0;
#pragma unroll
  for (int J = 0; J < 4; ++J)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int gi = row(16 * w + 4 * v + kq), gj = col(16 * J + cl);
      const double t = acc[J][v];
      M[(int64_t)gi * ld + gj] = t;
      if (isA) M[(int64_t)gj * ld + gi] = t;
      sq += t * t;
    }
  if (isA && last) {
    sq = block_sum_d(sq, red);
    if (tid == 0) L.jpart[np + blockIdx.x] = 2.0 * sq;
  }
}

// P = V_K Lambda_K^{-1/2} for the K largest eigenvalues (descending, lowest index on ties):
// workgroup k finds the eigenvalue of rank k and writes column k of P (and row k of its
// transpose).  A K-th eigenvalue not above 1e-14 of the largest marks the spectrum degenerate.
__global__ __launch_bounds__(kThreads) void k_lab_basis(Geometry g, LabScratch L, int K) {
  __shared__ double lam[kMaxR];
  __shared__ int pick[2];
  const int r = g.r, tid = threadIdx.x, k = blockIdx.x;
  for (int i = tid; i < r; i += kThreads) lam[i] = L.A[(int64_t)i * L.r64 + i];
  if (tid < 2) pick[tid] = 0;
  __syncthreads();
  for (int i = tid; i < r; i += kThreads) {
    int rank = 0;
    const double li = lam[i];
    for (int j = 0; j < r; ++j) rank += (lam[j] > li || (lam[j] == li && j < i)) ? 1 : 0;
    if (rank == k) pick[0] = i;
    if (rank == 0) pick[1] = i;
  }
  __syncthreads();
  const int idx = pick[0];
  const double lk = lam[idx];
  if (k == K - 1 && tid == 0) {
    bool ok = lk > 1e-14 * lam[pick[1]];
    for (int i = 0; i < r; ++i) ok = ok && isfinite(lam[i]);
    if (!ok) L.flag[kFlagDegenerate] = 1;
    L.scal[0] = ok ? 1.0 / sqrt(lk) : 0.0;
    double ub = 0.0;  // |u| is at most its column's norm
    for (int i = 0; i < r; ++i) ub = fmax(ub, L.ubound[i]);
    L.scal[1] = (double)f16_range_scale((float)ub);
  }
  for (int c = tid; c < r; c += kThreads) {
    const double v = lk > 0.0 ? L.V[(int64_t)c * L.r64 + idx] / sqrt(lk) : 0.0;
    L.P[(int64_t)c * K + k] = v;
    L.Pt[(int64_t)k * r + c] = v;
  }
}

// One assignment pass: labels of 32 NG rows a wave, 128 NG a tile.  The product is
// taken as M^T U^T on the 32x32x16 fp16 matrix core: a 32 x 32 tile holds 32 clusters x 32 rows (lane
// l: row l % 32, clusters 32 t + 8 (v / 4) + 4 (l / 32) + v % 4 in entry v), so the argmin over the
// clusters runs over registers and then over two lanes.  A lane reads its row of U directly (8
// consecutive columns a 16-column step), splits it in two halves, and drops the product of the two
// low parts; M comes split from the centroid kernel, 32 columns at a time through one of two LDS
// buffers.  NG = 2 where one block of clusters leaves registers for it (more bytes in flight a wave),
// else 1: with 2 the accumulators spill.  Bound by reading U once and by waves in flight (two a
// SIMD): 371 us at 1e6 x 200, K = 100 (products alone 70 us, reading 160) and 55 us at 1e6 x 30,
// K = 20; the same product on the fp64 matrix cores took 1.06 to 1.27 ms and 87 us.
// Rounding: every term's error is at most 2^-20 of it (two operands to 2^-22, the dropped product) but
// for fp16 subnormals (2^-25 / scale), and each of the 3 r16 / 16 matrix instructions adds at most 16
// roundings of 2^-23 (truncation) of the sum of |u_c M_ck| <= |u| |M_k| <= |u| pmax |cent_k|.
// UN: rows not 16-byte aligned.
template <int T, int NG, bool UN>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_lab_assign(
    Geometry g, const float* __restrict__ U, LabScratch L, int K, int32_t* __restrict__ labels) {
  if (L.flag[kFlagDegenerate] | L.flag[kFlagDone]) return;
  constexpr int CH = 2 * T * 2 * 64;  // 16-byte pieces of a 32-column chunk: [step][block][hi, lo][lane]
  constexpr int PT = CH / kThreads;   // pieces a thread
  __shared__ f16x8 ms[2][CH];
  __shared__ float cnf[32 * T], cinv[32 * T];
  __shared__ double es[4][kLabMaxK];
  __shared__ unsigned wchg[4];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, h = lane >> 5, li = lane & 31;
  const int r = g.r;
  const int64_t n = g.n;
  const bool first = L.flag[kFlagPasses] == 0;
  const double pmax = L.scal[0], su = L.scal[1];
  // (a centroid that equals an earlier one takes no row, see k_lab_centroid)
  for (int k = tid; k < 32 * T; k += kThreads) {
    const bool on = k < K && L.lead[k] == k;
    cnf[k] = on ? (float)L.cn[k] : 3.0e38f;
    cinv[k] = on ? (float)(L.minv[k] / su) : 0.f;
  }
  double cnmax = 0.0;
#pragma unroll 1
  for (int k = 0; k < K; ++k) cnmax = fmax(cnmax, L.cn[k]);
  __syncthreads();
  const int np = (r + 31) >> 5;  // 32-column chunks
  const double mb = pmax * sqrt(cnmax), eps = 1.1102230246251565e-16;
  // the smallest difference of two scores that decides: fp16 form (per |u|, and fixed), FP64 form
  const float tol16u = (float)(4.0 * (96.0 * np + 64.0) * 1.1920929e-7 * mb * 1.01);
  const float tol16c = (float)((4.0 * r * mb * 2.98e-8 / su + 4.0 * 2.4e-7 * cnmax) * 1.01);
  const double tol64u = 8.0 * (r + K * sqrt((double)K) + 16.0) * eps * mb, tol64c = 4.0 * (K + 16) * eps * cnmax;
  const float suf = (float)su;
  unsigned changes = 0;
  const int64_t tiles = (n + 128 * NG - 1) / (128 * NG);
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int64_t row0 = tile * (128 * NG) + 32 * NG * w;
    const bool edge = UN && ((tile + 1) * (128 * NG) >= n || r < 3);  // (the tile that holds the last row)
    const float* up[NG];
#pragma unroll
    for (int gq = 0; gq < NG; ++gq) {
      const int64_t row = row0 + 32 * gq + li;
      up[gq] = U + (row < n ? row : n - 1) * r;
    }
    f32x16 acc[NG][T];
#pragma unroll
    for (int gq = 0; gq < NG; ++gq)
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[gq][t][v] = 0.f;
    float un2[NG] = {};
    f32x4 nx[2][NG][2];  // [step][group][half] of the next chunk
    f16x8 mr[PT];
    const f16x8* Mi = reinterpret_cast<const f16x8*>(L.Mimg);
    auto load_chunk = [&](int p) {
#pragma unroll
      for (int u = 0; u < PT; ++u) mr[u] = Mi[(int64_t)p * CH + tid + u * kThreads];
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int gq = 0; gq < NG; ++gq)
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int c = 32 * p + 16 * st + 8 * h + 4 * q;
            nx[st][gq][q] = (UN && edge) ? load4_edge(up[gq], c < r ? c : 0, r) : load4<UN>(up[gq] + (c < r ? c : 0));
          }
    };
    load_chunk(0);
    for (int p = 0; p < np; ++p) {
      const int buf = p & 1;
#pragma unroll
      for (int u = 0; u < PT; ++u) ms[buf][tid + u * kThreads] = mr[u];
      f16x8 bh[2][NG], bl[2][NG];
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int gq = 0; gq < NG; ++gq) {
          float v[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int c = 32 * p + 16 * st + 8 * h + e;
            v[e] = c < r ? nx[st][gq][e >> 2][e & 3] : 0.f;
            un2[gq] = fmaf(v[e] * suf, v[e] * suf, un2[gq]);
          }
          split_f16(v, suf, bh[st][gq], bl[st][gq]);
        }
      __syncthreads();
      if (p + 1 < np) load_chunk(p + 1);
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int t = 0; t < T; ++t) {
          const f16x8 ah = ms[buf][((st * T + t) * 2 + 0) * 64 + lane], al = ms[buf][((st * T + t) * 2 + 1) * 64 + lane];
#pragma unroll
          for (int gq = 0; gq < NG; ++gq) {
            acc[gq][t] = mfma32x32x16h(ah, bl[st][gq], acc[gq][t]);
            acc[gq][t] = mfma32x32x16h(al, bh[st][gq], acc[gq][t]);
            acc[gq][t] = mfma32x32x16h(ah, bh[st][gq], acc[gq][t]);
          }
        }
    }
    __syncthreads();  // the buffers are free for the next tile
#pragma unroll
    for (int gq = 0; gq < NG; ++gq) {
      float best = 3.0e38f, second = 3.0e38f;
      int bk = 0;
      const float *ci = cinv + 4 * h, *cf = cnf + 4 * h;
      const int Kh = K - 4 * h;
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int k0 = 32 * t + 8 * (v >> 2) + (v & 3);  // (4 h is added at the end)
          const float sc = k0 < Kh ? fmaf(-2.f * ci[k0], acc[gq][t][v], cf[k0]) : 3.0e38f;
          acc[gq][t][v] = sc;
          if (sc < best) {
            second = best;
            best = sc;
            bk = k0;
          } else {
            second = fminf(second, sc);
          }
        }
      bk += 4 * h;
      {
        const float ob = shfl_xor_f(best, 32), os = shfl_xor_f(second, 32);
        const int ok = __shfl_xor(bk, 32, 64);
        second = fminf(fminf(second, os), fmaxf(best, ob));
        if (ob < best || (ob == best && ok < bk)) {
          best = ob;
          bk = ok;
        }
      }
      const float unorm = sqrtf(un2[gq] + shfl_xor_f(un2[gq], 32)) / suf * 1.0001f;
      const float tol = tol16u * unorm + tol16c;
      const int64_t row = row0 + 32 * gq + li;
      unsigned long long close = __ballot(h == 0 && row < n && !(second - best > tol));
      if (close) {
        // candidates of every row, a bit a cluster
        unsigned long long m0 = 0, m1 = 0;
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int k0 = 32 * t + 8 * (v >> 2) + (v & 3);
            const unsigned long long bit = acc[gq][t][v] <= best + tol ? 1ull << (k0 & 63) : 0ull;
            if (k0 < 64)
              m0 |= bit;
            else
              m1 |= bit;
          }
        m0 <<= 4 * h;
        m1 <<= 4 * h;
        m0 |= __shfl_xor(m0, 32, 64);
        m1 |= __shfl_xor(m1, 32, 64);
        while (close) {  // one row a wave at a time
          const int rl = __ffsll(close) - 1;
          close &= close - 1;
          const float* u = U + (row0 + 32 * gq + rl) * r;
          unsigned long long mm[2] = {(unsigned long long)__shfl(m0, rl, 64), (unsigned long long)__shfl(m1, rl, 64)};
          const double t64 = tol64u * (double)__shfl(unorm, rl, 64) + tol64c;
          double b64 = 1e300, s64 = 1e300;
          int kb = 0;
          // a candidate costs a sum over the wave; with more than a few the distances are cheaper (a
          // third of 1e6 rows equally far from 60 centroids: a call 15.4 ms by scores, 3.3 so)
          const bool few = __popcll(mm[0]) + __popcll(mm[1]) <= 4;
#pragma unroll 1
          for (int x = 0; few && x < 2; ++x)
            while (mm[x]) {
              const int k = 64 * x + __ffsll(mm[x]) - 1;
              mm[x] &= mm[x] - 1;
              if (k >= K) break;
              double s = 0.0;
#pragma unroll 1
              for (int c = lane; c < r; c += 64) s += (double)u[c] * L.Mt[(int64_t)k * r + c];
              for (int m = 32; m >= 1; m >>= 1) s += shfl_xor_d(s, m);
              const double sc = L.cn[k] - 2.0 * s;
              if (sc < b64) {
                s64 = b64;
                b64 = sc;
                kb = k;
              } else {
                s64 = fmin(s64, sc);
              }
            }
          if (!(s64 - b64 > t64)) {
            // too close for that: the distances themselves
#pragma unroll 1
            for (int j = lane; j < K; j += 64) {
              double s = 0.0;
#pragma unroll 1
              for (int c = 0; c < r; ++c) s += (double)u[c] * L.P[(int64_t)c * K + j];
              es[w][j] = s;
            }
            __builtin_amdgcn_wave_barrier();
            double db = 1e300;
            kb = 0x7fffffff;
#pragma unroll 1
            for (int k = lane; k < K; k += 64) {
              double ds = 0.0;
#pragma unroll 1
              for (int j = 0; j < K; ++j) {
                const double t = es[w][j] - L.centT[(int64_t)j * K + k];
                ds += t * t;
              }
              if (ds < db) {
                db = ds;
                kb = k;
              }
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) {
              const double ob = __shfl_xor(db, m, 64);
              const int ok = __shfl_xor(kb, m, 64);
              if (ob < db || (ob == db && ok < kb)) {
                db = ob;
                kb = ok;
              }
            }
          }
          if (li == rl) bk = kb;
        }
      }
      if (h == 0 && row < n) {
        if (first || labels[row] != bk) ++changes;
        labels[row] = bk;
      }
    }
  }
  for (int m = 32; m >= 1; m >>= 1) changes += __shfl_xor(changes, m, 64);
  if (lane == 0) wchg[w] = changes;
  __syncthreads();
  if (tid == 0) {
    const unsigned long long c = (unsigned long long)wchg[0] + wchg[1] + wchg[2] + wchg[3];
    if (c) atomicAdd(L.changed, c);
  }
}

// Cluster sums of the rows of U over row chunk blockIdx.x, columns 64 blockIdx.y .. + 63: the sum
// of llrint(u 2^(61 - e_c)).  Integer sums do not depend on the order, so they are reproducible
// bit for bit; every term keeps 61 - log2(sqrt(n G_cc)) binary places, so a fp32 u above 2^-37 of
// that bound is summed exactly and the sum's error is n 2^-62 of it at most (FP64 sums: n 2^-53).
// The rows of a piece of the chunk are sorted by label in LDS (counting sort); G lanes take a row,
// four columns each, and a group of them the same number of consecutive sorted rows, summed in
// registers: the LDS atomics into the cluster's entry come once a run of equal labels.  (One atomic
// an element ran at the LDS unit's one 64-bit atomic a clock: 386 us at 1e6 x 200 with K = 100 and
// 69 us at 1e6 x 30 with K = 20; this way 180 and 36 us.)  Bound by reading U once (4.4 and 3.3 TB/s).
// SMALL: fewer than four columns.  UN: rows not 16-byte aligned; the last quad of a row then starts
// at column r - 4 and leaves out the columns of the quad before.
constexpr int kLabPiece = 2048;  // rows sorted at a time
template <int G, bool UN, bool SMALL>
__global__ __launch_bounds__(kThreads) void k_lab_sums(Geometry g, const float* __restrict__ U, LabScratch L, int K,
                                                       const int32_t* __restrict__ labels) {
  if (L.flag[kFlagDegenerate] | L.flag[kFlagDone]) return;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  constexpr int LPR = 4 * G, SUBS = kThreads / G, UNR = 8, RT = kLabPiece / kThreads;
  unsigned long long* S = reinterpret_cast<unsigned long long*>(smem_raw);  // K x LPR
  int* cnt = reinterpret_cast<int*>(S + K * LPR);                           // K
  __shared__ unsigned order[kLabPiece];                                     // row | label << 16, by label
  __shared__ int hist[kLabMaxK], base[kLabMaxK + 1];
  const int tid = threadIdx.x, lane = tid & 63;
  const int r = g.r;
  const int64_t n = g.n;
  for (int e = tid; e < K * LPR; e += kThreads) S[e] = 0;
  for (int e = tid; e < K; e += kThreads) cnt[e] = 0;
  const int64_t r0 = (int64_t)blockIdx.x * n / L.W, r1 = (int64_t)(blockIdx.x + 1) * n / L.W;
  const int sub = tid / G, ql = 4 * (tid & (G - 1));  // this lane's columns in the group
  const int c0 = 64 * blockIdx.y + ql;
  const int cb = SMALL ? 0 : (c0 + 4 <= r ? c0 : r - 4);  // first column loaded
  int ex[4], sl[4];                                       // exponent of the first word's scale; slot
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int c = cb + e;
    const bool on = c0 < r && c >= c0 && c < r;
    const double sc = on ? L.cscale[c] : 0.0;
    ex[e] = sc > 0.0 ? ilogb(sc) - 31 : -4000;
    sl[e] = on ? c - 64 * (int)blockIdx.y : -1;
  }
  for (int64_t s0 = r0; s0 < r1; s0 += kLabPiece) {
    const int m = (int)(r1 - s0 < kLabPiece ? r1 - s0 : kLabPiece);
    for (int k = tid; k < kLabMaxK; k += kThreads) hist[k] = 0;
    __syncthreads();
    int lb[RT], rk[RT];
#pragma unroll
    for (int u = 0; u < RT; ++u) {
      const int i = tid + u * kThreads;
      lb[u] = i < m ? labels[s0 + i] : -1;
    }
#pragma unroll
    for (int u = 0; u < RT; ++u) rk[u] = (unsigned)lb[u] < (unsigned)K ? atomicAdd(&hist[lb[u]], 1) : 0;
    __syncthreads();
    if (tid < 64) {
      const int h0 = hist[2 * lane], h1 = hist[2 * lane + 1];
      int x = h0 + h1;
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
      }
      base[2 * lane] = x - h0 - h1;
      base[2 * lane + 1] = x - h1;
      if (lane == 63) base[kLabMaxK] = x;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < RT; ++u)
      if ((unsigned)lb[u] < (unsigned)K)
        order[base[lb[u]] + rk[u]] = (unsigned)(tid + u * kThreads) | (unsigned)lb[u] << 16;
    if (tid < K) cnt[tid] += hist[tid];
    __syncthreads();
    const int mt = base[kLabMaxK];
    const int p0 = sub * mt / SUBS, p1 = (sub + 1) * mt / SUBS;
    long long acc[4] = {0, 0, 0, 0};
    int cur = -1;
    auto flush = [&]() {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (cur >= 0 && sl[e] >= 0) atomicAdd(&S[cur * LPR + sl[e]], (unsigned long long)acc[e]);
        acc[e] = 0;
      }
    };
    for (int p = p0; p < p1; p += UNR) {
      unsigned o[UNR];
      f32x4 v[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) o[u] = order[p + u < p1 ? p + u : p];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const float* row = U + (s0 + (o[u] & 0xffff)) * r + cb;
        if constexpr (SMALL) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[u][e] = row[e < r ? e : 0];
        } else {
          v[u] = load4<UN>(row);
        }
      }
#pragma unroll
      for (int u = 0; u < UNR; ++u)
        if (p + u < p1) {
          const int k = (int)(o[u] >> 16);
          if (k != cur) {
            flush();
            cur = k;
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            // v 2^(ex + 31), |.| < 2^61, as hi 2^31 + lo: both steps are exact but for lo's rounding
            const float t = ldexpf(v[u][e], ex[e]);
            const float hi = truncf(t), lo = rintf((t - hi) * 2147483648.f);
            acc[e] += (long long)(int)hi * 2147483648ll + (int)lo;
          }
        }
    }
    flush();
    __syncthreads();
  }
  for (int e = tid; e < K * LPR; e += kThreads) {
    const int k = e / LPR, cc = 64 * blockIdx.y + (e & (LPR - 1));
    if (cc < r) L.spart[((int64_t)blockIdx.x * K + k) * r + cc] = (long long)S[e];
  }
  if (blockIdx.y == 0)
    for (int k = tid; k < K; k += kThreads) L.cpart[blockIdx.x * K + k] = cnt[k];
}

// Centroid k = blockIdx.x: from the cluster sums (seed = 0) or from its seed row (seed = 1), then
// |cent_k|^2 and column k of M = P cent^T in the assignment's order (clusters beyond K, seed
// launch only: zeros).  Workgroup 0 settles the pass: the first one that changed no label ends
// the iteration.  One workgroup a centroid; the sums over chunks, columns and components are each
// shared by groups of threads (a single workgroup for all centroids: 2.7 ms at K = 100).
// Equal centroids: a centroid equal to an earlier one, bit for bit, takes no row (its distances are
// equal too, and the lowest index wins), so the assignment masks it; found tied row by row, a pass
// over 1e6 x 16 with one seed for all 16 clusters took 5.7 ms, masked 0.17 ms.  Equal seed rows give
// them.  grp: the first cluster with this seed row; lead: the first of those whose centroid is still
// the seed's (the others have no rows and keep theirs).  A cluster that is not its own lead forms
// the lead's new centroid instead of one, and passes to the next of the group when that has left.
__global__ __launch_bounds__(kLabUpd) void k_lab_centroid(Geometry g, const float* __restrict__ U, LabScratch L, int K,
                                                          int T, int seed) {
  __shared__ double sums[kMaxR], cent[kLabMaxK], part[kLabUpd];
  __shared__ long long ipart[kLabUpd];
  __shared__ long long count;
  __shared__ int eq, off;
  const int tid = threadIdx.x, r = g.r, k = blockIdx.x;
  const int r32 = (r + 31) & ~31;
  // M_ck scaled and split into the assignment's operand order: [step of 16 columns][block of 32
  // clusters][hi, lo][lane = 32 (c / 8 % 2) + k % 32][c % 8]
  auto put = [&](int c, float m) {
    const _Float16 hi = (_Float16)m;
    _Float16* o = reinterpret_cast<_Float16*>(L.Mimg) +
                  (((int64_t)((c >> 4) * T + (k >> 5)) * 2) * 64 + ((c >> 3) & 1) * 32 + (k & 31)) * 8 + (c & 7);
    o[0] = hi;
    o[512] = (_Float16)(m - (float)hi);
  };
  if (k >= K) {
    for (int c = tid; c < r32; c += kLabUpd) put(c, 0.f);
    return;
  }
  // Workgroup 0 ends the iteration at its end, so a workgroup that starts late may leave here (its
  // centroid is not read again) -- as one: its waves go by what thread 0 read.
  if (tid == 0) {
    count = seed;
    eq = k;
    off = L.flag[kFlagDegenerate] | L.flag[kFlagDone];
  }
  __syncthreads();
  if (off) return;
  const int src = seed ? k : L.lead[k];  // the cluster whose centroid is formed
  if (seed) {
    const float* u = U + L.seeds[k] * r;
    for (int c = tid; c < r; c += kLabUpd) sums[c] = (double)u[c];
    if (tid < k) {  // (K <= kLabUpd)
      const float* v = U + L.seeds[tid] * r;
      int differ = 0;
      for (int c = 0; c < r && !differ; c += 8)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int ce = c + e < r ? c + e : c;
          differ |= u[ce] != v[ce];
        }
      if (!differ) atomicMin(&eq, tid);
    }
    __syncthreads();
    if (tid == 0) L.grp[k] = L.lead[k] = eq;
  } else {
    long long nc = 0;
    for (int w = tid; w < L.W; w += kLabUpd) nc += L.cpart[w * K + src];
    if (nc) atomicAdd(reinterpret_cast<unsigned long long*>(&count), (unsigned long long)nc);
    const int cw = (r + 63) & ~63;            // r <= 448: one to eight groups of threads
    const int ng = kLabUpd / cw, gq = tid / cw, c = tid - gq * cw;
    long long s = 0;
    if (gq < ng && c < r) {
      const long long* p = L.spart + (int64_t)src * r + c;
      const int64_t st = (int64_t)K * r;
      int w = gq;
      for (; w + 7 * ng < L.W; w += 8 * ng) {
        long long v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = p[(w + u * ng) * st];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
      }
      for (; w < L.W; w += ng) s += p[w * st];
    }
    ipart[tid] = s;
    __syncthreads();
    if (gq == 0 && c < r) {
      for (int h = 1; h < ng; ++h) s += ipart[tid + h * cw];
      // the mean row: that of equal rows is the row itself (their sum is exact), so its embedding
      // is that of the row as a seed, bit for bit
      sums[c] = (double)s * L.cinv[c] / (double)count;
    }
    __syncthreads();
  }
  {  // cent_j = sum_c sums[c] P[c][j], the terms c = gq, gq + 4, ... by thread group gq
    const int j = tid & 127, gq = tid >> 7;
    double s = 0.0;
    if (j < K)
#pragma unroll 8
      for (int c = gq; c < r; c += 4) s += sums[c] * L.P[(int64_t)c * K + j];
    part[tid] = s;
    __syncthreads();
    double v = 0.0;
    if (tid < K) v = ((part[tid] + part[128 + tid]) + part[256 + tid]) + part[384 + tid];
    if (src != k) {
      const bool left = tid < K && count > 0 && v != L.centT[(int64_t)tid * K + k];
      if (__syncthreads_or(left) && tid == 0) {
        int j = src + 1;
        while (j < k && L.grp[j] != L.grp[k]) ++j;
        L.lead[k] = j;
      }
      return;
    }
    if (tid < K) {
      if (count == 0) v = L.centT[(int64_t)tid * K + k];
      cent[tid] = v;
      L.centT[(int64_t)tid * K + k] = v;
    }
    __syncthreads();
  }
  __shared__ double cn;
  if (tid == 0) {
    double s = 0.0;
    for (int j = 0; j < K; ++j) s += cent[j] * cent[j];
    cn = s;
  }
  __syncthreads();
  const double sm = (double)f16_range_scale((float)(L.scal[0] * sqrt(cn) * 1.01));  // |M_ck| <= pmax |cent_k|
  if (tid == 0) {
    L.cn[k] = cn;
    L.minv[k] = 1.0 / sm;
  }
  for (int c = tid; c < r32; c += kLabUpd) {
    double m = 0.0;
    if (c < r) {
#pragma unroll 8
      for (int j = 0; j < K; ++j) m += L.Pt[(int64_t)j * r + c] * cent[j];
      L.Mt[(int64_t)k * r + c] = m;
    }
    put(c, (float)(m * sm));
  }
  if (!seed && k == 0 && tid == 0) {
    const int passes = L.flag[kFlagPasses] + 1;
    if (passes > 1 && *L.changed == 0) L.flag[kFlagDone] = 1;
    *L.changed = 0;
    L.flag[kFlagPasses] = passes;
  }
}

hipError_t launch_lab_gram(const Geometry& g, const Bufs& b, const LabScratch& L, hipStream_t st) {
  hipError_t e = launch_gram_partials(b.U, g.n, g.r, nullptr, L.gpart, L.GU, st);
  if (e != hipSuccess) return e;
  const int rr = L.r64 * L.r64;
  hipLaunchKernelGGL(k_lab_gram_reduce, dim3((rr + kThreads - 1) / kThreads), dim3(kThreads), 0, st, g, L);
  return hipGetLastError();
}

constexpr size_t kJacLds = 2 * 64 * kJacLd * sizeof(double);

hipError_t launch_lab_sweeps(const LabScratch& L, int r, int first, int count, hipStream_t st) {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_lab_sub),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)kJacLds);
  if (e != hipSuccess) return e;
  const int nb = L.r64 / 32, np = nb / 2;
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_lab_apply), hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)kApplyLds);
  if (e != hipSuccess) return e;
  if (np == 1) {  // all columns in one pivot block: run to the end
    const int N = (r + 1) & ~1;
    hipLaunchKernelGGL(k_lab_sub, dim3(1), dim3(kJacThreads), kJacLds, st, L, 0, nb, N < 2 ? 2 : N, kLabMaxSweeps, 1, 0, 0);
    return hipGetLastError();
  }
  for (int s = first; s < first + count; ++s)
    for (int t = 0; t < nb - 1; ++t) {
      const int last = t == nb - 2;
      hipLaunchKernelGGL(k_lab_sub, dim3(np), dim3(kJacThreads), kJacLds, st, L, t, nb, 64, 1, 0, s > 0 && t == 0, last);
      hipLaunchKernelGGL(k_lab_apply, dim3(np * (np - 1) / 2 + np * np), dim3(kThreads), kApplyLds, st, L, t, nb, last);
    }
  return hipGetLastError();
}

hipError_t launch_lab_embed(const Geometry& g, const Bufs& b, const LabScratch& L, int K, hipStream_t st) {
  const int T = (K + 31) / 32;
  hipLaunchKernelGGL(k_lab_basis, dim3(K), dim3(kThreads), 0, st, g, L, K);
  hipLaunchKernelGGL(k_lab_centroid, dim3(32 * T), dim3(kLabUpd), 0, st, g, (const float*)b.U, L, K, T, 1);
  return hipGetLastError();
}

template <int T>
static void lab_assign(const Geometry& g, const Bufs& b, const LabScratch& L, int K, int32_t* labels, hipStream_t st) {
  constexpr int NG = T == 1 ? 2 : 1;
  const int64_t tiles = (g.n + 128 * NG - 1) / (128 * NG);
  const dim3 grid((unsigned)(tiles < 1024 ? tiles : 1024));
  if (g.vec_u)
    hipLaunchKernelGGL((k_lab_assign<T, NG, false>), grid, dim3(kThreads), 0, st, g, (const float*)b.U, L, K, labels);
  else
    hipLaunchKernelGGL((k_lab_assign<T, NG, true>), grid, dim3(kThreads), 0, st, g, (const float*)b.U, L, K, labels);
}

template <int G, bool UN, bool SMALL>
static hipError_t lab_sums(const Geometry& g, const Bufs& b, const LabScratch& L, int K, const int32_t* labels,
                           hipStream_t st) {
  const size_t lds = (size_t)K * 4 * G * 8 + (size_t)K * 4;
  if (lds > (48u << 10)) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_lab_sums<G, UN, SMALL>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_lab_sums<G, UN, SMALL>), dim3(L.W, (g.r + 63) / 64), dim3(kThreads), lds, st, g,
                     (const float*)b.U, L, K, labels);
  return hipGetLastError();
}

hipError_t launch_lab_pass(const Geometry& g, const Bufs& b, const LabScratch& L, int K, int32_t* labels,
                           hipStream_t st) {
  const int T = (K + 31) / 32;
  switch (T) {
    case 1: lab_assign<1>(g, b, L, K, labels, st); break;
    case 2: lab_assign<2>(g, b, L, K, labels, st); break;
    case 3: lab_assign<3>(g, b, L, K, labels, st); break;
    case 4: lab_assign<4>(g, b, L, K, labels, st); break;
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const bool v = g.vec_u;
  e = g.r < 4    ? lab_sums<4, true, true>(g, b, L, K, labels, st)
      : g.r <= 16 ? (v ? lab_sums<4, false, false>(g, b, L, K, labels, st) : lab_sums<4, true, false>(g, b, L, K, labels, st))
      : g.r <= 32 ? (v ? lab_sums<8, false, false>(g, b, L, K, labels, st) : lab_sums<8, true, false>(g, b, L, K, labels, st))
                  : (v ? lab_sums<16, false, false>(g, b, L, K, labels, st) : lab_sums<16, true, false>(g, b, L, K, labels, st));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_lab_centroid, dim3(K), dim3(kLabUpd), 0, st, g, (const float*)b.U, L, K, T, 0);
  return hipGetLastError();
}

}  // namespace nlr
