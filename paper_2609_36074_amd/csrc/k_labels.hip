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
//   |e_i|^2 + |cent_k|^2 - 2 u_i M_k, so a pass is one product U M on the fp64 matrix
//   cores with the argmin over k in registers; rows whose two smallest values lie closer
//   than the rounding of that form can resolve are decided by the distances themselves
//   (FP64, lowest index on ties).  The cluster sums S_k = sum of u_i over the rows of k
//   are taken in 64-bit integers (below), and cent_k = (S_k P) / count (a centroid
//   without rows stays in place).
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
    *L.pmax = ok ? 1.0 / sqrt(lk) : 0.0;
  }
  for (int c = tid; c < r; c += kThreads) {
    const double v = lk > 0.0 ? L.V[(int64_t)c * L.r64 + idx] / sqrt(lk) : 0.0;
    L.P[(int64_t)c * K + k] = v;
    L.Pt[(int64_t)k * r + c] = v;
  }
}

// One assignment pass: labels of 32 rows a wave (two groups of 16), 128 a tile.  The product is
// taken as M^T U^T: a 16 x 16 tile of the fp64 matrix core holds 16 clusters x 16 rows (lane l:
// row l % 16, clusters 16 t + 4 v + l / 16 in entry v), so the argmin over the clusters runs
// over registers and then over four lanes.  A step's 4 columns are 16 q + 4 (l / 16) + s for
// s = 0..3, so a lane reads its U values as 16 consecutive bytes; M comes in that order from the
// centroid kernel (32 bytes a lane, from L2 and L1).  Bound by the fp64 matrix cores: 2 n r16 K16
// flops, 0.6 ms at 1e6 x 200 with K = 100 against 0.2 ms for reading U once.
template <int T, bool VEC>
__global__ __launch_bounds__(kThreads) void k_lab_assign(Geometry g, const float* __restrict__ U, LabScratch L, int K,
                                                         int32_t* __restrict__ labels) {
  if (L.flag[kFlagDegenerate] | L.flag[kFlagDone]) return;
  __shared__ double cn[16 * T];
  __shared__ double es[4][kLabMaxK];
  __shared__ unsigned wchg[4];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, lg = lane >> 4, lr = lane & 15;
  const int r = g.r;
  const int64_t n = g.n;
  const bool first = L.flag[kFlagPasses] == 0;
  for (int k = tid; k < 16 * T; k += kThreads) cn[k] = k < K ? L.cn[k] : 0.0;
  __syncthreads();
  double cnmax = 0.0;
  for (int k = 0; k < K; ++k) cnmax = fmax(cnmax, cn[k]);
  // rounding of the scores: |M_ck| <= |P_c| |cent_k| <= pmax sqrt(cnmax), sums of r and K terms
  const double eps = 1.1102230246251565e-16;
  const double tolu = 8.0 * (r + K + 16) * eps * *L.pmax * sqrt(cnmax), tolc = 4.0 * (K + 16) * eps * cnmax;
  const int nq = (r + 15) >> 4;
  const f64x4* Mi = reinterpret_cast<const f64x4*>(L.Mimg) + lane;
  unsigned changes = 0;
  const int64_t tiles = (n + 127) / 128;
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int64_t row0 = tile * 128 + 32 * w;
    const float* up[2];
#pragma unroll
    for (int gq = 0; gq < 2; ++gq) {
      const int64_t row = row0 + 16 * gq + lr;
      up[gq] = U + (row < n ? row : n - 1) * r;
    }
    f64x4 acc[2][T];
#pragma unroll
    for (int gq = 0; gq < 2; ++gq)
#pragma unroll
      for (int t = 0; t < T; ++t) acc[gq][t] = (f64x4){0.0, 0.0, 0.0, 0.0};
    double rs[2] = {0.0, 0.0};
    float nx[2][4];
    auto load_u = [&](int q) {
      const int c0 = 16 * q + 4 * lg;
#pragma unroll
      for (int gq = 0; gq < 2; ++gq) {
        if constexpr (VEC) {
          const f32x4 t = *reinterpret_cast<const f32x4*>(up[gq] + (c0 < r ? c0 : 0));
#pragma unroll
          for (int s = 0; s < 4; ++s) nx[gq][s] = c0 < r ? t[s] : 0.f;
        } else {
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const float t = up[gq][c0 + s < r ? c0 + s : 0];
            nx[gq][s] = c0 + s < r ? t : 0.f;
          }
        }
      }
    };
    load_u(0);
    for (int q = 0; q < nq; ++q) {
      double b[2][4];
#pragma unroll
      for (int gq = 0; gq < 2; ++gq)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          b[gq][s] = (double)nx[gq][s];
          rs[gq] += fabs(b[gq][s]);
        }
      if (q + 1 < nq) load_u(q + 1);
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const f64x4 a = Mi[(int64_t)(q * T + t) * 64];
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int gq = 0; gq < 2; ++gq)
            acc[gq][t] = mfma16x16x4d(a[s], b[gq][s], acc[gq][t]);
      }
    }
#pragma unroll
    for (int gq = 0; gq < 2; ++gq) {
      double best = 1e300, second = 1e300;
      int bk = 0x7fffffff;
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int k = 16 * t + 4 * v + lg;
          const double sc = k < K ? cn[k] - 2.0 * acc[gq][t][v] : 1e300;
          if (sc < best) {
            second = best;
            best = sc;
            bk = k;
          } else {
            second = fmin(second, sc);
          }
        }
      double rsum = rs[gq];
#pragma unroll
      for (int m = 16; m <= 32; m <<= 1) {
        const double ob = __shfl_xor(best, m, 64), os = __shfl_xor(second, m, 64);
        const int ok = __shfl_xor(bk, m, 64);
        second = fmin(fmin(second, os), fmax(best, ob));
        if (ob < best || (ob == best && ok < bk)) {
          best = ob;
          bk = ok;
        }
        rsum += __shfl_xor(rsum, m, 64);
      }
      const int64_t row = row0 + 16 * gq + lr;
      // rows too close to call: the distances themselves, one row a wave at a time
      unsigned long long close =
          __ballot(lane < 16 && row < n && !(second - best > tolu * rsum + tolc)) & 0xffffull;
      while (close) {
        const int rl = __ffsll(close) - 1;
        close &= close - 1;
        const float* u = U + (row0 + 16 * gq + rl) * r;
        for (int j = lane; j < K; j += 64) {
          double s = 0.0;
          for (int c = 0; c < r; ++c) s += (double)u[c] * L.P[(int64_t)c * K + j];
          es[w][j] = s;
        }
        __builtin_amdgcn_wave_barrier();
        double db = 1e300;
        int kb = 0x7fffffff;
        for (int k = lane; k < K; k += 64) {
          double ds = 0.0;
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
        if (lr == rl) bk = kb;
      }
      if (lane < 16 && row < n) {
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

// Cluster sums of the rows of U over row chunk blockIdx.x, columns 64 blockIdx.y .. + 63: a lane
// holds column c and adds llrint(u 2^(61 - e_c)) to its cluster's entry in LDS.  Integer sums do
// not depend on the order, so LDS atomics stay reproducible bit for bit; every term keeps
// 61 - log2(sqrt(n G_cc)) binary places, so a fp32 u above 2^-37 of that bound is summed exactly
// and the sum's error is n 2^-62 of it at most (FP64 sums: n 2^-53).  LPR lanes a row (16, 32 or
// 64): narrow factors take several rows an instruction.  Bound by reading U once (0.8 GB at 1e6 x
// 200); a one-hot product on the fp64 matrix cores would take as long as the assignment.
template <int LPR>
__global__ __launch_bounds__(kThreads) void k_lab_sums(Geometry g, const float* __restrict__ U, LabScratch L, int K,
                                                       const int32_t* __restrict__ labels) {
  if (L.flag[kFlagDegenerate] | L.flag[kFlagDone]) return;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  unsigned long long* S = reinterpret_cast<unsigned long long*>(smem_raw);  // K x LPR
  int* cnt = reinterpret_cast<int*>(S + K * LPR);                           // K
  constexpr int RP = 64 / LPR, UN = 8;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int r = g.r;
  const int64_t n = g.n;
  for (int e = tid; e < K * LPR; e += kThreads) S[e] = 0;
  for (int e = tid; e < K; e += kThreads) cnt[e] = 0;
  __syncthreads();
  const int64_t r0 = (int64_t)blockIdx.x * n / L.W, r1 = (int64_t)(blockIdx.x + 1) * n / L.W;
  const int cl = lane & (LPR - 1), sub = lane / LPR;
  const int c = 64 * blockIdx.y + cl;
  const bool okc = c < r;
  const double sc = okc ? L.cscale[c] : 0.0;
  const float* up = U + (okc ? c : 0);
  for (int64_t i0 = r0 + w * RP + sub; i0 < r1; i0 += 4 * RP * UN) {
    float v[UN];
    int lb[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int64_t i = i0 + 4 * RP * u, ic = i < r1 ? i : r0;
      v[u] = up[ic * r];
      lb[u] = labels[ic];
    }
#pragma unroll
    for (int u = 0; u < UN; ++u)
      if (i0 + 4 * RP * u < r1) {
        const long long q = __double2ll_rn((double)v[u] * sc);
        if (okc) atomicAdd(&S[lb[u] * LPR + cl], (unsigned long long)q);
        if (blockIdx.y == 0 && cl == 0) atomicAdd(&cnt[lb[u]], 1);
      }
  }
  __syncthreads();
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
__global__ __launch_bounds__(kLabUpd) void k_lab_centroid(Geometry g, const float* __restrict__ U, LabScratch L, int K,
                                                          int T, int seed) {
  if (L.flag[kFlagDegenerate] | L.flag[kFlagDone]) return;
  __shared__ double sums[kMaxR], cent[kLabMaxK], part[kLabUpd];
  __shared__ long long ipart[kLabUpd];
  __shared__ long long count;
  const int tid = threadIdx.x, r = g.r, k = blockIdx.x;
  const int r16 = (r + 15) & ~15;
  auto put = [&](int c, double m) {
    const int q = c >> 4, cc = c & 15;
    L.Mimg[((int64_t)(q * T + (k >> 4)) * 64 + (cc >> 2) * 16 + (k & 15)) * 4 + (cc & 3)] = m;
  };
  if (k >= K) {
    for (int c = tid; c < r16; c += kLabUpd) put(c, 0.0);
    return;
  }
  if (tid == 0) count = seed;
  __syncthreads();
  if (seed) {
    const float* u = U + L.seeds[k] * r;
    for (int c = tid; c < r; c += kLabUpd) sums[c] = (double)u[c];
    __syncthreads();
  } else {
    long long nc = 0;
    for (int w = tid; w < L.W; w += kLabUpd) nc += L.cpart[w * K + k];
    if (nc) atomicAdd(reinterpret_cast<unsigned long long*>(&count), (unsigned long long)nc);
    const int cw = (r + 63) & ~63;            // r <= 448: one to eight groups of threads
    const int ng = kLabUpd / cw, gq = tid / cw, c = tid - gq * cw;
    long long s = 0;
    if (gq < ng && c < r) {
      const long long* p = L.spart + (int64_t)k * r + c;
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
      sums[c] = (double)s * L.cinv[c];
    }
    __syncthreads();
  }
  {  // cent_j = sum_c sums[c] P[c][j] / count, the terms c = gq, gq + 4, ... by thread group gq
    const int j = tid & 127, gq = tid >> 7;
    double s = 0.0;
    if (j < K)
#pragma unroll 8
      for (int c = gq; c < r; c += 4) s += sums[c] * L.P[(int64_t)c * K + j];
    part[tid] = s;
    __syncthreads();
    if (tid < K) {
      double v = ((part[tid] + part[128 + tid]) + part[256 + tid]) + part[384 + tid];
      v = count > 0 ? v / (double)count : L.centT[(int64_t)tid * K + k];
      cent[tid] = v;
      L.centT[(int64_t)tid * K + k] = v;
    }
    __syncthreads();
  }
  if (tid == 0) {
    double s = 0.0;
    for (int j = 0; j < K; ++j) s += cent[j] * cent[j];
    L.cn[k] = s;
  }
  for (int c = tid; c < r16; c += kLabUpd) {
    double m = 0.0;
    if (c < r)
#pragma unroll 8
      for (int j = 0; j < K; ++j) m += L.Pt[(int64_t)j * r + c] * cent[j];
    put(c, m);
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
  const int T = (K + 15) / 16;
  hipLaunchKernelGGL(k_lab_basis, dim3(K), dim3(kThreads), 0, st, g, L, K);
  hipLaunchKernelGGL(k_lab_centroid, dim3(16 * T), dim3(kLabUpd), 0, st, g, (const float*)b.U, L, K, T, 1);
  return hipGetLastError();
}

template <int T>
static void lab_assign(const Geometry& g, const Bufs& b, const LabScratch& L, int K, int32_t* labels, hipStream_t st) {
  const int64_t tiles = (g.n + 127) / 128;
  const dim3 grid((unsigned)(tiles < 2048 ? tiles : 2048));
  // 16-byte loads of U need 16-byte rows
  if (g.vec_u)
    hipLaunchKernelGGL((k_lab_assign<T, true>), grid, dim3(kThreads), 0, st, g, (const float*)b.U, L, K, labels);
  else
    hipLaunchKernelGGL((k_lab_assign<T, false>), grid, dim3(kThreads), 0, st, g, (const float*)b.U, L, K, labels);
}

template <int LPR>
static hipError_t lab_sums(const Geometry& g, const Bufs& b, const LabScratch& L, int K, const int32_t* labels,
                           hipStream_t st) {
  const size_t lds = (size_t)K * LPR * 8 + (size_t)K * 4;
  if (lds > (64u << 10)) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_lab_sums<LPR>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_lab_sums<LPR>), dim3(L.W, (g.r + 63) / 64), dim3(kThreads), lds, st, g, (const float*)b.U, L,
                     K, labels);
  return hipGetLastError();
}

hipError_t launch_lab_pass(const Geometry& g, const Bufs& b, const LabScratch& L, int K, int32_t* labels,
                           hipStream_t st) {
  const int T = (K + 15) / 16;
  switch (T) {
    case 1: lab_assign<1>(g, b, L, K, labels, st); break;
    case 2: lab_assign<2>(g, b, L, K, labels, st); break;
    case 3: lab_assign<3>(g, b, L, K, labels, st); break;
    case 4: lab_assign<4>(g, b, L, K, labels, st); break;
    case 5: lab_assign<5>(g, b, L, K, labels, st); break;
    case 6: lab_assign<6>(g, b, L, K, labels, st); break;
    case 7: lab_assign<7>(g, b, L, K, labels, st); break;
    case 8: lab_assign<8>(g, b, L, K, labels, st); break;
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = g.r <= 16 ? lab_sums<16>(g, b, L, K, labels, st)
                : (g.r <= 32 ? lab_sums<32>(g, b, L, K, labels, st) : lab_sums<64>(g, b, L, K, labels, st));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_lab_centroid, dim3(K), dim3(kLabUpd), 0, st, g, (const float*)b.U, L, K, T, 0);
  return hipGetLastError();
}

}  // namespace nlr
