// gdn_pull.h -- building blocks of the query pull-back on the matrix cores
// (trees above 128 slots, gdn_large.hip).
//
// For a node n the pull-back walks n's path from n to the root with
//     x <- q_n, r <- 1, acc <- 0;  for t = n, parent(n), ..., root:
//         c = beta_t k_t.x;  acc += r c v_t;  x <- x - c k_t;  r <- r alpha_t
// (Eq. 7-8 rearranged) and gives o_n = scale (S0 (r x) + acc).  A wave takes
// 16 consecutive nodes of a depth-first order.  In such an order every
// ancestor of a node of the tile is in the tile or is an ancestor of the
// tile's first node, so the tile needs its own 16 rows plus one chain, cut
// into chunks of 16, deepest first.  The walk becomes one blocked
// substitution per chunk of path nodes,
//     s = K_c x,   (I + N) c = beta s  with N_tt' = beta_t k_t.k_t' (t above t'),
//     x -= K_c^T c,   acc += V_c^T (r c),
// with the 16 nodes as matrix columns.  s and x take their fp32 operand as fp16
// hi + lo, scaled (split4 says how far off that is), acc in fp32.
//
// Layouts (v_mfma_f32_16x16x32_f16).  Lane (l16, m) = (lane % 16, lane / 16)
// of an accumulator holds rows 4 m + e (e < 4) of column l16.  An accumulator
// is fed back as a B operand without any lane move: slots e < 4 of lane group
// m are then rows 4 m + e of one 16-row tile, slots e >= 4 rows 4 m + e of
// another, and the A operand is read with the same slot order.  The rows of a
// chunk sit in the order rho = 4 (tau % 4) + tau / 4 (tau: depth order), so
// that accumulator register e of all lane groups holds the four consecutive
// rows tau = 4 e .. 4 e + 3, one k step of v_mfma_f32_16x16x4_f32: the
// substitution goes over e = 3 .. 0 with one product by the inverse of a 4 x
// 4 diagonal block and one rank-4 update each, in fp32.
#pragma once

#include "gdn_internal.h"

namespace gdn {

typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f16x8 cat(f16x4 a, f16x4 b) { return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7); }
__device__ __forceinline__ f16x4 to_h4(f32x4 x) {
  return f16x4{(_Float16)x[0], (_Float16)x[1], (_Float16)x[2], (_Float16)x[3]};
}
// x y = hi + lo, off by at most 2^-22 |x y| + 2^-25 (the last fp16 place above
// 0), with the product not rounded in between.
// For a split of x alone y is a 1.0 that the compiler cannot see (one_f):
// the remainder is then one mixed-precision FMA per value.
__device__ __forceinline__ void split4(f32x4 x, float y, f16x4& hi, f16x4& lo) {
  hi = to_h4(x * y);
#pragma unroll
  for (int e = 0; e < 4; ++e) lo[e] = (_Float16)fmaf(x[e], y, -(float)hi[e]);
}
__device__ __forceinline__ float one_f() {
  float y = 1.0f;
  asm("" : "+v"(y));
  return y;
}
__device__ __forceinline__ f32x4 mfma_h16(f16x4 a, f16x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_h(f16x8 a, f16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_f(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Transposing LDS read: within each 16 lanes, lane i names row i / 4,
// elements 4 (i % 4) .. + 3 of a 4 x 16 matrix of halves and receives column
// i (4 rows).
__device__ __forceinline__ f16x4 ld_tr(const unsigned char* p) {
  typedef __fp16 raw4 __attribute__((ext_vector_type(4)));
  typedef raw4 __attribute__((address_space(3)))* lds_p;
  return __builtin_bit_cast(f16x4, __builtin_amdgcn_ds_read_tr16_b64_v4f16((lds_p)(p)));
}

// Orders LDS accesses of one wave (no instruction besides the waits the
// compiler places for the data itself).
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// x, or 0 when it is not finite
__device__ __forceinline__ float finite(float x) { return fabsf(x) < __builtin_inff() ? x : 0.0f; }

// Depth order of operand row l16, i.e. tau(rho) at rho = l16.
__device__ __forceinline__ int tau_of(int l16) { return 4 * (l16 & 3) + (l16 >> 2); }

// This lane's entry (i, j) = (l16 / 4, m) of the 4 x 4 diagonal block of step
// e = l16 % 4 of a symmetric Gram tile g.
__device__ __forceinline__ float diag_entry(f32x4 g, int l16) {
  const int e = l16 & 3;
  return e == 0 ? g[0] : (e == 1 ? g[1] : (e == 2 ? g[2] : g[3]));
}

// Inverse of the four 4 x 4 diagonal blocks I + N (unit upper triangular in
// depth order) of a chunk: this lane's value as the k = m operand of row l16.
// n_ij: this lane's entry of N (0 on and below the diagonal); z: 64 floats of
// LDS of this wave.
__device__ __forceinline__ float block_inverse(float* z, float n_ij, int l16, int m) {
  z[16 * (l16 & 3) + 4 * (l16 >> 2) + m] = n_ij;
  wave_lds_order();
  const float* zr = z + 16 * (l16 & 3);
  const float4 r0 = *reinterpret_cast<const float4*>(zr);
  const float4 r1 = *reinterpret_cast<const float4*>(zr + 4);
  const float4 r2 = *reinterpret_cast<const float4*>(zr + 8);
  wave_lds_order();
  const float d3 = m == 3 ? 1.0f : 0.0f;
  const float d2 = (m == 2 ? 1.0f : 0.0f) - r2.w * d3;
  const float d1 = (m == 1 ? 1.0f : 0.0f) - r1.z * d2 - r1.w * d3;
  const float d0 = (m == 0 ? 1.0f : 0.0f) - r0.y * d1 - r0.z * d2 - r0.w * d3;
  const int i = l16 >> 2;
  return i == 0 ? d0 : (i == 1 ? d1 : (i == 2 ? d2 : d3));
}

// (I + N) c = b with b = bm s (bm: beta on the column's path, else 0); g: the
// chunk's Gram tile K K^T, dinv: block_inverse.
__device__ __forceinline__ f32x4 substitute(f32x4 s, f32x4 g, float dinv, f32x4 bm, int l16) {
  const f32x4 z = {0.f, 0.f, 0.f, 0.f};
  f32x4 c;
#pragma unroll
  for (int e = 3; e >= 0; --e) {
    const f32x4 d = mfma_f((l16 & 3) == e ? dinv : 0.0f, bm[e] * s[e], z);
    c[e] = d[e];
    if (e > 0) s = mfma_f(-g[e], c[e], s);
  }
  return c;
}

// Decay from each accumulator row of a chunk down to the column's node: rw
// times the alphas of the rows below it (al: alpha on the column's path, else
// 1).  rw moves up by the chunk.  Products, not sums of logarithms: alpha may
// be 0 or negative.
__device__ __forceinline__ f32x4 decays(f32x4 al, float& rw, int m) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  f32x4 lr;
#pragma unroll
  for (int e = 3; e >= 0; --e) {  // rows tau = 4 e + m: the four lane groups hold four consecutive ones
    const unsigned a = __float_as_uint(al[e]);
    u2 w = __builtin_bit_cast(u2, __builtin_amdgcn_permlane16_swap(a, a, false, false));
    const float odd = __uint_as_float(w.y);  // of this pair of groups
    const unsigned pair = __float_as_uint(__uint_as_float(w.x) * odd);
    w = __builtin_bit_cast(u2, __builtin_amdgcn_permlane32_swap(pair, pair, false, false));
    const float upper = __uint_as_float(w.y);  // groups 2 and 3
    lr[e] = rw * ((m & 1 ? 1.0f : odd) * (m < 2 ? upper : 1.0f));
    rw *= __uint_as_float(w.x) * upper;
  }
  return lr;
}

// Column of an fp16 state plane that holds channel k: within 32 channels the
// groups of 4 of the two 16-channel tiles alternate, the slot order of two
// accumulator tiles as one operand.
__device__ __forceinline__ constexpr int plane_col(int k) {
  const int j = k & 28;
  return (k & ~31) + (j < 16 ? 2 * j : 2 * (j - 16) + 4) + (k & 3);
}

}  // namespace gdn
