// Device helpers shared by the per-iteration kernels (gfx950).
#pragma once

#include "nlr_internal.hpp"

namespace nlr {

// Forms of the row-resident pass A: with the Theta product, the finish pass
// (materialises U), and the row work alone (fused iteration).
enum PassAMode { kPassIter = 0, kPassFinish = 1, kPassRows = 2 };

__device__ __forceinline__ bool halted(const DevCtl* ctl) {
  return (ctl->stop | ctl->breakdown) != 0;
}

// The same for a whole workgroup, for kernels whose workgroup 0 sets breakdown at its end: the waves
// of a workgroup that starts late would each see it set or not, and those that go on would meet the
// barriers, and the sums in LDS, without the others.
__device__ __forceinline__ bool halted_workgroup(const DevCtl* ctl) {
  __shared__ int off;
  if (threadIdx.x == 0) off = ctl->stop | ctl->breakdown;
  __syncthreads();
  return off != 0;
}

// Whether the stopping rule of the previous iteration (Section 4.3) can still fire
// at this one: its movement is below min(eps_d, eps_c) and t >= T_min; only the
// residual rho of the current factor is then missing, which the row work computes.
// The one-pass iteration writes W over the factor it reads when this is false; when
// true, the row work runs in its own pass first and settles the rule.
__device__ __forceinline__ bool stop_possible(const DevCtl* ctl, const StepArgs& S) {
  const int64_t t = ctl->t_done;
  return S.end_work != 0 && t > 0 && ctl->Delta < S.eps_d * S.eps_d * S.K && ctl->delta < S.eps_c &&
         t >= S.T_min;
}

// Loads W consecutive floats; when !ok the (valid) address is still read and the
// values are replaced by zeros, so no branch is needed.
template <int W>
__device__ __forceinline__ void load_vec(float (&dst)[W], const float* src, bool ok) {
  if constexpr (W == 4) {
    const f32x4 t = *reinterpret_cast<const f32x4*>(src);
    dst[0] = ok ? t.x : 0.f;
    dst[1] = ok ? t.y : 0.f;
    dst[2] = ok ? t.z : 0.f;
    dst[3] = ok ? t.w : 0.f;
  } else if constexpr (W == 2) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const f32x2 t = *reinterpret_cast<const f32x2*>(src);
    dst[0] = ok ? t.x : 0.f;
    dst[1] = ok ? t.y : 0.f;
  } else {
    const float t = *src;
    dst[0] = ok ? t : 0.f;
  }
}

// Rows that are not 16-byte aligned (UN): global memory takes 16- and 8-byte accesses at any 4-byte
// address, so a row moves in pieces of four as aligned rows do; a row's last piece may run up to
// three floats into the next row (masked where used).  Past the end of the matrix there is nothing
// to read, so tiles that hold the last row -- or any, where a row is shorter than three -- load
// element by element (edge).
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));
template <bool UN>
__device__ __forceinline__ f32x4 load4(const float* p) {
  if constexpr (UN)
    return *reinterpret_cast<const f32x4u*>(p);
  else
    return *reinterpret_cast<const f32x4*>(p);
}
// W elements from column c of a row of `len` (unaligned); edge: those past its end as the last one.
template <int W>
__device__ __forceinline__ void load_piece(float (&dst)[W], const float* row, int c, int len, bool edge) {
  if (edge) {
    asm volatile("" : "+v"(c));  // as load4_edge
#pragma unroll
    for (int e = 0; e < W; ++e) dst[e] = row[c + e < len ? c + e : len - 1];
    __builtin_amdgcn_sched_barrier(0);
  } else if constexpr (W == 4) {
    const f32x4u t = *reinterpret_cast<const f32x4u*>(row + c);
#pragma unroll
    for (int e = 0; e < 4; ++e) dst[e] = t[e];
  } else if constexpr (W == 2) {
    const f32x2u t = *reinterpret_cast<const f32x2u*>(row + c);
    dst[0] = t[0];
    dst[1] = t[1];
  } else {
    dst[0] = row[c];
  }
}
// Elements c .. c + 3 of a row of `len`, those past its end as the last one.  (The opaque column
// and the barrier keep the addresses of this rare path out of registers that live across the loop.)
__device__ __forceinline__ f32x4 load4_edge(const float* row, int c, int len) {
  f32x4 t;
  asm volatile("" : "+v"(c));
#pragma unroll
  for (int e = 0; e < 4; ++e) t[e] = row[c + e < len ? c + e : len - 1];
  __builtin_amdgcn_sched_barrier(0);
  return t;
}

template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}
// Sum over the 8 lanes of each DPP half row, bitwise the same in all 8 lanes.
__device__ __forceinline__ double row8_sum_d(double v) {
  v += dpp_d<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp_d<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_d<0x141>(v);  // row_half_mirror
  return v;
}

// Sum over the 16 lanes of a DPP row with involution pairings (xor 1, xor 2,
// half-row mirror, row mirror): every step adds two equal partial sums, so all
// lanes end with the same bits.
__device__ __forceinline__ double row16_sum_d(double v) {
  v += dpp_d<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp_d<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_d<0x141>(v);  // row_half_mirror
  v += dpp_d<0x140>(v);  // row_mirror
  return v;
}

typedef float f32x4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x4v mfma16x16x4(float a, float b, f32x4v c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Reduce-scatter of LEN per-lane values across the lanes that differ in bits
// MASK, MASK/2, ...: afterwards a lane holds LEN >> steps sums, of the upper half
// when its bit is set and of the lower half otherwise.
template <int LEN, int MASK>
__device__ __forceinline__ void reduce_scatter(float* wv, int li) {
  if constexpr (LEN > 1 && MASK > 0) {
    const bool up = (li & MASK) != 0;
#pragma unroll
    for (int k = 0; k < LEN / 2; ++k) {
      const float send = up ? wv[k] : wv[k + LEN / 2];
      const float keep = up ? wv[k + LEN / 2] : wv[k];
      wv[k] = keep + shfl_xor_f(send, MASK);
    }
    reduce_scatter<LEN / 2, MASK / 2>(wv, li);
  }
}

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// D += A * B on the 32x32x16 fp16 matrix core (fp32 accumulate).  Lane l supplies
// A[l%32][8(l/32) + e] and B[8(l/32) + e][l%32] as element e; D has the layout of
// the 32x32x2 fp32 form: lane l, register v holds D[8(v/4)+4(l/32)+v%4][l%32].
__device__ __forceinline__ f32x16 mfma32x32x16h(f16x8 a, f16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// Two-term fp16 split of 8 fp32 values after scaling by the power of two s:
// v s = hi + lo + O(2^-22 |v s|), hi = fp16(v s), lo = fp16(v s - hi).  With s chosen
// so that |v s| < 2^15, hi and (for |v s| >= 2^-3) lo are normal fp16 numbers.
__device__ __forceinline__ void split_f16(const float* v, float s, f16x8& hi, f16x8& lo) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float t = v[e] * s;
    const _Float16 h = (_Float16)t;
    hi[e] = h;
    lo[e] = (_Float16)(t - (float)h);
  }
}

// Power of two s with |v| s < 2^15 for every |v| <= vmax (1 when vmax is 0 or not finite).
__device__ __forceinline__ float f16_range_scale(float vmax) {
  if (!(vmax > 0.f) || !(vmax < 3.0e38f)) return 1.0f;
  int e;
  (void)frexpf(vmax, &e);  // vmax < 2^e
  int k = 15 - e;
  if (k > 100) k = 100;
  if (k < -100) k = -100;
  return ldexpf(1.0f, k);
}

// Sum of P[off], P[off + step], ... below `limit` (count: at least the number of such terms, uniform),
// in order, UN loads in flight.  The partial rows of a pass were written by other XCDs, so a load
// takes about 2 us: all of a thread's terms go in one or two batches, with 32-bit offsets (64-bit
// products for the addresses alone took as long).
template <typename T, int UN>
__device__ __forceinline__ double batch_sum(const T* __restrict__ P, uint32_t off, uint32_t step, uint32_t limit,
                                            int count) {
  double acc = 0.0;
  for (int s0 = 0; s0 < count; s0 += UN) {
    T v[UN];
#pragma unroll
    for (int i = 0; i < UN; ++i) {
      const uint32_t o = off + (uint32_t)i * step;
      v[i] = P[o < limit ? o : 0];
    }
    __builtin_amdgcn_sched_barrier(0);  // every load is issued before the first value is used
#pragma unroll
    for (int i = 0; i < UN; ++i) acc += off + (uint32_t)i * step < limit ? (double)v[i] : 0.0;
    off += UN * step;
  }
  return acc;
}
template <typename T>
__device__ __forceinline__ double wide_sum(const T* __restrict__ P, uint32_t off, uint32_t step, uint32_t limit,
                                           int count) {
  return count <= 8 ? batch_sum<T, 8>(P, off, step, limit, count)
                    : (count <= 16 ? batch_sum<T, 16>(P, off, step, limit, count)
                                   : batch_sum<T, 32>(P, off, step, limit, count));
}

// Column sums over all rows of a partials array in one workgroup of kRedThreads: 64 consecutive
// columns, 16 groups of threads over the rows, the groups added in order.  (rows * stride < 2^32:
// the partials take at most 64 MiB or 255 rows of 768 x 256.)
// Result in the threads below 64.  `red`: kRedThreads doubles of LDS.
constexpr int kRedThreads = 1024;
__device__ __forceinline__ double part_sum64(const float* __restrict__ P, int64_t rows, int64_t stride, int64_t col,
                                             double* red) {
  const uint32_t st = (uint32_t)stride, gq = threadIdx.x >> 6;
  red[threadIdx.x] = wide_sum<float>(P, gq * st + (uint32_t)col, 16 * st, (uint32_t)rows * st, (int)((rows + 15) / 16));
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x < 64)
#pragma unroll
    for (int k = 0; k < 16; ++k) t += red[64 * k + threadIdx.x];
  return t;
}

// The same sum in one thread, in the same order (sixteen sums of every sixteenth row, added in
// order): 32 rows' loads in flight.
__device__ __forceinline__ double part_sum16(const float* __restrict__ P, int64_t rows, int64_t stride, int64_t col) {
  const uint32_t st = (uint32_t)stride, limit = (uint32_t)rows * st;
  double acc[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) acc[k] = 0.0;
  for (uint32_t off = (uint32_t)col; off < limit; off += 32 * st) {
    float v[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) {
      const uint32_t o = off + (uint32_t)i * st;
      v[i] = P[o < limit ? o : (uint32_t)col];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 32; ++i) acc[i & 15] += off + (uint32_t)i * st < limit ? (double)v[i] : 0.0;
  }
  double t = 0.0;
#pragma unroll
  for (int k = 0; k < 16; ++k) t += acc[k];
  return t;
}

// FP64 matrix core v_mfma_f64_16x16x4f64, D += A B: lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16]; entry v of D is D[4 v + l / 16][l % 16].
typedef double f64x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f64x4 mfma16x16x4d(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// v_mfma_f64_4x4x4f64: four independent 4 x 4 blocks, block b = (l >> 2) & 3; lane l supplies
// A_b[l % 4][l / 16] and B_b[l / 16][l % 4] and holds D_b[l / 16][l % 4].  It sustains 68 TFLOP/s
// on the whole chip where the 16x16x4 form stops at 47 (both measured; 35 with one wave a SIMD),
// so the long FP64 products use it: with A in the 16x16x4 layout (row l % 16) and B rotated by 4 R
// columns inside its 16 (column (l + 4 R) % 16), result R = 0..3 of a 16 x 16 tile is
// D[4 b + l / 16][4 ((b + R) % 4) + l % 4].
__device__ __forceinline__ double mfma4x4x4d(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// acc += A B over `steps` steps of 4 for a 64 x 64 result of one workgroup: wave w holds rows
// 16 w .. 16 w + 15 in four column tiles.  fa(k0): this lane's A element of row 16 w + lane % 16,
// k = k0 + lane / 16; fb(k0, J): its B element of k = k0 + lane / 16, column 16 J + lane % 16.
template <int UNROLL, class FA, class FB>
__device__ __forceinline__ void mm64(int steps, FA fa, FB fb, f64x4 (&acc)[4]) {
#pragma unroll UNROLL
  for (int st = 0; st < steps; ++st) {
    const double av = fa(4 * st);
#pragma unroll
    for (int J = 0; J < 4; ++J) acc[J] = mfma16x16x4d(av, fb(4 * st, J), acc[J]);
  }
}
__device__ __forceinline__ void mm64_zero(f64x4 (&acc)[4]) {
#pragma unroll
  for (int J = 0; J < 4; ++J) acc[J] = (f64x4){0.0, 0.0, 0.0, 0.0};
}

// Fixed-order sum over a 512-thread workgroup; result valid in thread 0.
__device__ __forceinline__ double block_sum8_d(double v, double* red) {
  for (int m = 32; m >= 1; m >>= 1) v += shfl_xor_d(v, m);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0) r = (((red[0] + red[1]) + (red[2] + red[3])) + ((red[4] + red[5]) + (red[6] + red[7])));
  __syncthreads();
  return r;
}

}  // namespace nlr
