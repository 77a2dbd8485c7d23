// gdn_chunked.hip -- tree verification in the paper's chunked form
// (Sec. 3.4.1-3.4.2, Eq. 9-13), for trees of up to 512 slots.
//
// With positions in canonical (topological) order, a_i the product of alpha
// over the path root..i, and q~, k~, v~ the post-conv features of one
// (sequence, value head), Eq. 7-8 give for every node, in the stored
// orientation (S0 in R^{dv x dk}):
//     X_ij = [j strict ancestor of i] beta_i (a_i / a_j) k~_i.k~_j      (Eq. 9)
//     Y_ij = [j ancestor of i or i]  (a_i / a_j) q~_i.k~_j
//     (I + X) U = beta (V - a K S0^T)           (Eq. 10 with W S0 folded in)
//     O = scale (a Q S0^T + Y U)                 (Eq. 11)
// X is strictly lower triangular (ancestors come first), so U follows from a
// forward substitution over sub-blocks of B_c = 32 positions (Eq. 13):
//     U_j = (I + X_jj)^-1 (R_j - sum_{c<j} X_jc U_c),
// where the inverse of each 16 x 16 tile on the diagonal is the product
// (I - N)(I + N^2)(I + N^4)(I + N^8), N the tile of X_jj (N^16 = 0), formed by
// repeated squaring, and the tile below them is -V11 X10 V00 (V the inverses).
//
// Three launches (two up to 32 slots, see chunk_kernel):
//   features           (gdn_large.hip) fp32 rows F[B][T][C]
//   chunk_gram_kernel  one workgroup per (position block j, up to 4 blocks c <=
//                      j, key head, sequence): the Gram blocks K_j K_c^T and
//                      Q_j K_c^T, which the value heads of a key head share,
//                      for every c that holds an ancestor of a node of j; for
//                      c = j per value head the decayed, masked Y_jj and the
//                      inverse of I + X_jj, one wave each
//   chunk_kernel       one workgroup per (value head, sequence), 8 waves, each
//                      wave 16 channels of dv: U's columns are independent, so
//                      the cascade over j runs inside a wave and no U is
//                      exchanged; the waves share the decayed X_jc, Y_jc of 2
//                      blocks c at a time (LDS)
// Products are 16 x 16 MFMA tiles.  The large ones (S0 products, Gram blocks,
// block updates) take both operands as bf16 hi/lo and three
// v_mfma_f32_16x16x32_bf16 (hi*hi + hi*lo + lo*hi, fp32 accumulation, ~1e-5
// relative); the diagonal inverse and its products stay on
// v_mfma_f32_16x16x4f32.
//
// Layouts.  Lane (l16, m) = (lane % 16, lane / 16) of an accumulator holds rows
// 4 m + e (e < 4) of column l16.  Accumulators become B operands without a lane
// move: in fp32 k step e is row 4 m + e of lane group m, in bf16 slots e < 4 of
// group m are rows 4 m + e of the block's first tile, slots e >= 4 rows 4 m + e
// of its second; the A operand is laid out in the same order (slot_col).
//
// What bounds it and why this form: one workgroup per head that formed the
// Gram blocks and the inverse itself ran 28 pairs and 8 inverses one after the
// other with 3 to 7 barriers each, one workgroup per CU (150 KB): 8 chains of
// 256 slots, 16 / 48 heads of 128, took 367 us, hardly any of it in the
// products.  Now 42 us (Gram, 155 MB) + 100 us (cascade, 500 MB: the copy
// rate; U comes back from the last-level cache for every later block), two
// workgroups per CU.  Registers spilled while loads are in flight wait for
// them one by one (7 in the cascade: 120 us), and so does a branch around a
// load or store.
#include <math.h>

#include "gdn_pull.h"

namespace gdn {

constexpr int kHT = 512;      // threads per workgroup (8 waves)
constexpr int kBc = 32;       // positions per block (B_c)
constexpr int kHMaxT = 512;   // tree slots supported
constexpr int kHW = 8;        // ancestor words per node (512 / 64)
constexpr int kLs = 36;       // row stride of the 32 x 32 matrices in LDS (floats)
constexpr int kCG = 4;        // blocks c per workgroup of the Gram launch (2: 50 us instead of 47 at 8 x 256)
constexpr int kCP = 2;        // earlier blocks per group of the cascade
constexpr int kMaxNB = kHMaxT / kBc;
constexpr int kUL = kBc + 8;  // bf16 row of an X or Y plane
constexpr float kMinLog2 = -125.5f;  // floor of log2 alpha: 2^x stays a normal float

struct ChunkParams {
  int B, T, Hk, Hv, dv;
  float scale;
  const void* meta;
  const void *alpha, *beta;
  const float* S0;
  float* out;
  const float* F;  // features [B][T][C]
  float* D;        // [B][Hv][NB][2][32][32]: (I + X_jj)^-1 and Y_jj
  float* Gm;       // [B][Hk][NB (NB - 1) / 2][2][32][32]: K_j K_c^T and Q_j K_c^T, c < j
  uint32_t* mask;  // [B][NB][16][32]: per row of block j, the strict ancestors among block c's positions
  unsigned char* need;  // [B][NB][16]: 1 if block c holds an ancestor of a node of block j
  uint16_t* U;     // [B][Hv][NB][DV / 16][2][64][8]: solved rows, bf16 hi and lo, per lane
};

// Bytes of the workspace's parts, in order
struct ChunkSizes {
  size_t f, d, g, k, n, u;
  ChunkSizes(int B, int T, int Hk, int Hv, int dk, int dv) {
    const size_t NB = size_t(T + kBc - 1) / kBc, mat = size_t(2) * kBc * kBc * sizeof(float);
    f = (features_f32_bytes(B, T, Hk, Hv, dk, dv) + 255) & ~size_t(255);
    d = size_t(B) * Hv * NB * mat;
    g = size_t(B) * Hk * (NB > 1 ? NB * (NB - 1) / 2 : 1) * mat;
    k = size_t(B) * NB * kMaxNB * kBc * sizeof(uint32_t);
    n = (size_t(B) * NB * kMaxNB + 255) & ~size_t(255);
    u = size_t(B) * Hv * NB * kBc * dv * sizeof(float);
  }
  size_t total() const { return f + d + g + k + n + u; }
};

size_t chunked_workspace_bytes(int B, int T, int Hk, int Hv, int dk, int dv) {
  return ChunkSizes(B, T, Hk, Hv, dk, dv).total();
}

// x -> bf16 hi (truncation) + bf16 lo (truncation of the remainder)
__device__ __forceinline__ uint32_t hi16(float x) { return __float_as_uint(x) >> 16; }
__device__ __forceinline__ uint32_t lo16(float x) {
  return __float_as_uint(x - __uint_as_float(__float_as_uint(x) & 0xffff0000u)) >> 16;
}
// 4 consecutive floats -> hi / lo planes (8 bytes each)
__device__ __forceinline__ void st_split4(uint16_t* hi, uint16_t* lo, float4 v) {
  *reinterpret_cast<uint2*>(hi) = make_uint2(hi16(v.x) | (hi16(v.y) << 16), hi16(v.z) | (hi16(v.w) << 16));
  *reinterpret_cast<uint2*>(lo) = make_uint2(lo16(v.x) | (lo16(v.y) << 16), lo16(v.z) | (lo16(v.w) << 16));
}
__device__ __forceinline__ void st_split2(uint16_t* hi, uint16_t* lo, float x, float y) {
  *reinterpret_cast<uint32_t*>(hi) = hi16(x) | (hi16(y) << 16);
  *reinterpret_cast<uint32_t*>(lo) = lo16(x) | (lo16(y) << 16);
}
// plane column of block position c: the k slot of U's operand
__device__ __forceinline__ int slot_col(int c) { return 8 * ((c & 15) >> 2) + 4 * (c >> 4) + (c & 3); }

// acc += A (16 x K) B (K x 16) for one 16 x 16 tile from bf16 hi/lo planes:
// A[i][k] = a[i * lda + k], B[k][j] = b[j * ldb + k] (k contiguous in both);
// three v_mfma_f32_16x16x32_bf16 per 32 k.
template <int K>
__device__ __forceinline__ f32x4 mm16x3(const uint16_t* ah, const uint16_t* al, int lda, const uint16_t* bh,
                                        const uint16_t* bl, int ldb, f32x4 acc, int lane) {
  const int i = lane & 15, kk = 8 * (lane >> 4);
#pragma unroll
  for (int k0 = 0; k0 < K; k0 += 32) {
    const bf16x8 xah = *reinterpret_cast<const bf16x8*>(ah + i * lda + k0 + kk);
    const bf16x8 xal = *reinterpret_cast<const bf16x8*>(al + i * lda + k0 + kk);
    const bf16x8 xbh = *reinterpret_cast<const bf16x8*>(bh + i * ldb + k0 + kk);
    const bf16x8 xbl = *reinterpret_cast<const bf16x8*>(bl + i * ldb + k0 + kk);
    acc = mfma3(xah, xal, xbh, xbl, acc);
  }
  return acc;
}
// c + A B in fp32 for 16 x 16 tiles: at holds A's transpose, b holds B, as
// accumulators
__device__ __forceinline__ f32x4 mm_f(f32x4 at, f32x4 b, f32x4 c) {
#pragma unroll
  for (int e = 0; e < 4; ++e) c = mfma_f(at[e], b[e], c);
  return c;
}
__device__ __forceinline__ f32x4 as_x4(float4 v) { return f32x4{v.x, v.y, v.z, v.w}; }

// (I - a)^-1 of a strictly lower triangular 16 x 16 tile as (I + a)(I + a^2)
// (I + a^4)(I + a^8), the tile and its transpose as accumulators
__device__ __forceinline__ void inverse16(f32x4 a, f32x4 at, f32x4& v, f32x4& vt, int l16, int m) {
  const f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float one = 4 * m + e == l16 ? 1.0f : 0.0f;
    v[e] = a[e] + one;
    vt[e] = at[e] + one;
  }
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    const f32x4 q = mm_f(at, a, z), qt = mm_f(a, at, z);
    const f32x4 w = mm_f(vt, q, v);
    vt = mm_f(q, vt, vt);
    v = w;
    a = q;
    at = qt;
  }
}

// One wave: the decayed, masked Y_jj and the inverse of I + X_jj of a value
// head, 32 rows of stride RS each, from the Gram blocks K_j K_j^T, Q_j K_j^T in
// s_g.  ga, gb, gp: alpha, beta and the parent's row (below 0 outside the
// block) of row lane % 32; rows: rows with nodes; s_a: kDiagLds floats.
constexpr int kDiagLds = kBc * kLs + 3 * kBc;
template <int RS>
__device__ __forceinline__ void diag_block(const float* s_g, float* s_a, float ga, float gb, int gp, int rows, int lane,
                                           float* dst) {
  const int l16 = lane & 15, m = lane >> 4;
  const f32x4 z4 = {0.f, 0.f, 0.f, 0.f};
  float* s_la = s_a + kBc * kLs;
  float* s_be = s_la + kBc;
  uint32_t* s_up = reinterpret_cast<uint32_t*>(s_be + kBc);  // strict ancestors in the block, one bit each
  {  // log decay from the block's edge down to each row, and its ancestors in
     // the block, by pointer jumping over the lanes
    const int i = lane & (kBc - 1);
    const bool real = i < rows;
    // floored at the smallest normal float: a decay of 0 keeps ratios finite
    float sl = real ? fmaxf(log2f(ga), kMinLog2) : 0.0f;
    const float be = real ? gb : 0.0f;
    int nx = real ? gp : -1;
    uint32_t up = nx >= 0 ? 1u << nx : 0u;
#pragma unroll
    for (int s = 0; s < 5; ++s) {
      const int src = nx >= 0 ? nx : i;
      const float sl2 = __shfl(sl, src);
      const uint32_t up2 = __shfl(up, src);
      const int nx2 = __shfl(nx, src);
      if (nx >= 0) {
        sl += sl2;
        up |= up2;
        nx = nx2;
      }
    }
    s_la[i] = sl;
    s_be[i] = be;
    s_up[i] = up;
  }
  wave_lds_order();
  {  // A = -X_jj -> LDS, Y_jj -> workspace: 16 columns of one row per lane
    const int i = lane & (kBc - 1), cc = 16 * (lane >> 5);
    const float la = s_la[i], be = s_be[i];
    const uint32_t up = s_up[i];
    const bool real = i < rows;
#pragma unroll
    for (int q = 0; q < 16; q += 4) {
      const float4 x = *reinterpret_cast<const float4*>(s_g + i * kLs + cc + q);
      const float4 y = *reinterpret_cast<const float4*>(s_g + kBc * kLs + i * kLs + cc + q);
      const f32x4 gx = as_x4(x), gy = as_x4(y);
      f32x4 av, yv;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c = cc + q + e;
        const bool anc = (up >> c) & 1;
        const float r = __builtin_amdgcn_exp2f(la - s_la[c]);
        av[e] = anc ? -be * r * gx[e] : 0.0f;
        yv[e] = anc || (c == i && real) ? r * gy[e] : 0.0f;
      }
      *reinterpret_cast<float4*>(s_a + i * kLs + cc + q) = make_float4(av[0], av[1], av[2], av[3]);
      *reinterpret_cast<float4*>(dst + kBc * RS + i * RS + cc + q) = make_float4(yv[0], yv[1], yv[2], yv[3]);
    }
  }
  wave_lds_order();
  // (I + X_jj)^-1 from its 16 x 16 tiles: V00, V11 and V11 A10 V00
  f32x4 v[2], vt[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    f32x4 a;
#pragma unroll
    for (int e = 0; e < 4; ++e) a[e] = s_a[(16 * t + 4 * m + e) * kLs + 16 * t + l16];
    const f32x4 at = as_x4(*reinterpret_cast<const float4*>(s_a + (16 * t + l16) * kLs + 16 * t + 4 * m));
    inverse16(a, at, v[t], vt[t], l16, m);
  }
  const f32x4 at10 = as_x4(*reinterpret_cast<const float4*>(s_a + (16 + l16) * kLs + 4 * m));
  const f32x4 vt10 = mm_f(mm_f(at10, v[0], z4), vt[1], z4);
  *reinterpret_cast<float4*>(dst + l16 * RS + 4 * m) = make_float4(vt[0][0], vt[0][1], vt[0][2], vt[0][3]);
  *reinterpret_cast<float4*>(dst + (16 + l16) * RS + 4 * m) = make_float4(vt10[0], vt10[1], vt10[2], vt10[3]);
  *reinterpret_cast<float4*>(dst + (16 + l16) * RS + 16 + 4 * m) = make_float4(vt[1][0], vt[1][1], vt[1][2], vt[1][3]);
}

template <int DK>
struct GramSmem {
  static constexpr int KP = DK < 32 ? 32 : DK;  // contraction extent of the key products (zero padded)
  static constexpr int LKH = KP + 8;            // bf16 plane row (halves)
  static constexpr size_t planes = size_t(6) * kBc * LKH * 2;  // q_j, k_j, k_c (hi, lo)
  static constexpr size_t mat = size_t(kBc) * kLs * 4;
  static constexpr size_t diag = 2 * mat + (kHT / 64) * kDiagLds * 4;  // Gram, then per wave A and its rows' gates
  static constexpr size_t uni = planes > diag ? planes : diag;
  static constexpr size_t total = uni + size_t(kBc) * kHW * 8;  // ancestor words of block j
  static_assert(total <= 80 * 1024, "two workgroups per CU");
};

// Two workgroups per CU: for three (80 registers) 4 registers spill and the
// launch takes the same time (8 x 64, 8 x 256 and 8 x 512 slots: 10.1, 44.5 and
// 123 us).
template <int DK, typename TIn>
__global__ __launch_bounds__(kHT, 4) void chunk_gram_kernel(ChunkParams p) {
  using SM = GramSmem<DK>;
  constexpr int KP = SM::KP, LKH = SM::LKH;
  constexpr int NQK = (2 * kBc * (DK / 4) + kHT - 1) / kHT;  // float4 of q_j and k_j per thread
  constexpr int NKC = (kBc * (DK / 4) + kHT - 1) / kHT;      // float4 of k_c per thread
  extern __shared__ __align__(16) unsigned char smem[];
  uint16_t* s_qh = reinterpret_cast<uint16_t*>(smem);
  uint16_t* s_ql = s_qh + kBc * LKH;
  uint16_t* s_kh = s_ql + kBc * LKH;
  uint16_t* s_kl = s_kh + kBc * LKH;
  uint16_t* s_ch = s_kl + kBc * LKH;
  uint16_t* s_cl = s_ch + kBc * LKH;
  uint64_t* s_anc = reinterpret_cast<uint64_t*>(smem + SM::uni);  // [32][kHW]

  const int g = blockIdx.x, b = blockIdx.z, tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int T = p.T, Hk = p.Hk, Hv = p.Hv, NB = (T + kBc - 1) / kBc;
  // Key heads run fastest over the blocks: with 8 or 16 of them a head's groups
  // share an XCD's L2 (42 us; groups fastest: 47).
  // block j has j / kCG + 1 groups of up to kCG blocks c <= j
  int jb = 0, c0 = blockIdx.y;
  while (c0 > jb / kCG) {
    c0 -= jb / kCG + 1;
    ++jb;
  }
  c0 *= kCG;
  const MetaPtrs m_ = meta_ptrs(p.meta, p.B, T);
  const int W = m_.W;
  const size_t bt = size_t(b) * T;
  const int nval = m_.status[b] == GDN_TREE_OK ? m_.nvalid[b] : 0;
  if (kBc * jb >= nval) return;  // uniform
  const int nq = Hk * DK;
  const size_t C = size_t(2 * nq + Hv * (p.dv));
  const float* Fq = p.F + bt * C + g * DK;
  const float* Fk = Fq + nq;

  const TIn* alpha = static_cast<const TIn*>(p.alpha);
  const TIn* beta = static_cast<const TIn*>(p.beta);
  const int G = Hv / Hk;
  const bool diag = jb < c0 + kCG;
  float4 kc[NKC];
  int ndc;  // node of this thread's position of block c
  auto fetch_c = [&](int cb) {
    ndc = m_.order[bt + kBc * cb + (cb < jb ? tid % kBc : 0)];
#pragma unroll
    for (int j = 0; j < NKC; ++j) {
      const int i = j * kHT + tid < kBc * (DK / 4) ? j * kHT + tid : 0;
      kc[j] = *reinterpret_cast<const float4*>(Fk + (cb < jb ? kBc * cb + i / (DK / 4) : 0) * C + 4 * (i % (DK / 4)));
    }
  };
  // gates of a value head's rows (diagonal block), a lane per row, twice
  float ga = 0.0f, gb = 0.0f;
  int gp = -1;
  auto fetch_gates = [&](int h) {
    const int pos = kBc * jb + (lane & (kBc - 1)), pc = pos < nval ? pos : 0;
    const int nd = m_.order[bt + pc];
    ga = ld(alpha, (bt + nd) * Hv + h);
    gb = ld(beta, (bt + nd) * Hv + h);
    gp = m_.ppos[bt + pc];
  };
  {
    float4 v[NQK];
    constexpr int NAW = (kBc * kHW + kHT - 1) / kHT;
    int nd[NAW];
#pragma unroll
    for (int j = 0; j < NAW; ++j) {
      const int pos = kBc * jb + (j * kHT + tid) / kHW % kBc;
      nd[j] = m_.order[bt + (pos < nval ? pos : 0)];
    }
#pragma unroll
    for (int j = 0; j < NQK; ++j) {
      const int i = j * kHT + tid;
      const int part = i / (kBc * (DK / 4)) & 1, r = i / (DK / 4) % kBc, c4 = i % (DK / 4);
      const int pos = kBc * jb + r;
      v[j] = *reinterpret_cast<const float4*>((part ? Fk : Fq) + (pos < nval ? pos : 0) * C + 4 * c4);
    }
    fetch_c(c0);  // c0 <= jb; row clamp: block jb may end early
    if (diag && wave < G) fetch_gates(g * G + wave);
#pragma unroll
    for (int j = 0; j < NAW; ++j) {
      const int i = j * kHT + tid, r = i / kHW % kBc, w = i % kHW;
      const uint64_t a = m_.anc[(bt + nd[j]) * W + (w < W ? w : 0)];
      if (i < kBc * kHW) s_anc[i] = kBc * jb + r < nval && w < W ? a : 0ull;
    }
#pragma unroll
    for (int j = 0; j < NQK; ++j) {
      const int i = j * kHT + tid;
      if (i < 2 * kBc * (DK / 4)) {
        const int part = i / (kBc * (DK / 4)), r = i / (DK / 4) % kBc, c4 = i % (DK / 4);
        const float4 x = kBc * jb + r < nval ? v[j] : make_float4(0.f, 0.f, 0.f, 0.f);
        st_split4((part ? s_kh : s_qh) + r * LKH + 4 * c4, (part ? s_kl : s_ql) + r * LKH + 4 * c4, x);
      }
    }
    if constexpr (DK < KP) {  // zero padding of the contraction, all six planes
      for (int i = tid; i < 6 * kBc * (KP - DK); i += kHT)
        s_qh[i / (KP - DK) * LKH + DK + i % (KP - DK)] = 0;
    }
  }
  __syncthreads();
  const int kind = wave >> 2, ti = (wave >> 1) & 1, tc = wave & 1;  // this wave's tile
  const int l16 = lane & 15, m = lane >> 4;
  const f32x4 z4 = {0.f, 0.f, 0.f, 0.f};
  const int cend = jb < c0 + kCG ? jb : c0 + kCG;
  for (int cb = c0; cb < cend; ++cb) {
    // strict ancestors of the rows of j among the positions of c: half a wave per row
    bool found = false;
    const size_t jc = (size_t(b) * NB + jb) * kMaxNB + cb;
#pragma unroll
    for (int j = 0; j < kBc * kBc / kHT; ++j) {
      const int i = j * (kHT / kBc) + tid / kBc;
      const bool anc = (s_anc[i * kHW + (ndc >> 6)] >> (ndc & 63)) & 1ull;
      const uint64_t w = __ballot(anc);
      if (g == 0 && tid % kBc == 0) p.mask[jc * kBc + i] = lane < kBc ? uint32_t(w) : uint32_t(w >> 32);
      found |= anc;
    }
    const bool any = __syncthreads_or(found);  // and the planes of the block before are read
    if (g == 0 && tid == 0) p.need[jc] = any;
    if (!any) {  // uniform
      if (cb + 1 < cend) fetch_c(cb + 1);
      continue;
    }
#pragma unroll
    for (int j = 0; j < NKC; ++j) {
      const int i = j * kHT + tid;
      if (i < kBc * (DK / 4)) {
        const int r = i / (DK / 4), c4 = i % (DK / 4);
        st_split4(s_ch + r * LKH + 4 * c4, s_cl + r * LKH + 4 * c4, kc[j]);
      }
    }
    if (cb + 1 < cend) fetch_c(cb + 1);
    __syncthreads();
    const f32x4 acc = mm16x3<KP>((kind ? s_qh : s_kh) + 16 * ti * LKH, (kind ? s_ql : s_kl) + 16 * ti * LKH, LKH,
                                 s_ch + 16 * tc * LKH, s_cl + 16 * tc * LKH, LKH, z4, lane);
    float* dst = p.Gm + (((size_t(b) * Hk + g) * (size_t(NB) * (NB - 1) / 2) + size_t(jb) * (jb - 1) / 2 + cb) * 2 +
                         kind) * (kBc * kBc);
#pragma unroll
    for (int e = 0; e < 4; ++e) dst[(16 * ti + 4 * m + e) * kBc + 16 * tc + l16] = acc[e];
  }
  if (!diag) return;  // uniform

  // ---- diagonal block
  __syncthreads();
  const f32x4 gm = mm16x3<KP>((kind ? s_qh : s_kh) + 16 * ti * LKH, (kind ? s_ql : s_kl) + 16 * ti * LKH, LKH,
                              s_kh + 16 * tc * LKH, s_kl + 16 * tc * LKH, LKH, z4, lane);
  __syncthreads();  // the planes are read: LDS holds the Gram blocks from here
  float* s_g = reinterpret_cast<float*>(smem);  // [2][32][kLs]
  float* s_a = s_g + 2 * kBc * kLs + wave * kDiagLds;
#pragma unroll
  for (int e = 0; e < 4; ++e) s_g[kind * kBc * kLs + (16 * ti + 4 * m + e) * kLs + 16 * tc + l16] = gm[e];
  __syncthreads();
  for (int w = wave; w < G; w += kHT / 64) {
    const int h = g * G + w;
    if (w != wave) fetch_gates(h);
    diag_block<kBc>(s_g, s_a, ga, gb, gp - kBc * jb, nval - kBc * jb, lane,
                    p.D + ((size_t(b) * Hv + h) * NB + jb) * (2 * kBc * kBc));
    wave_lds_order();
  }
}

template <int DK, int DV>
struct ChunkSmem {
  static constexpr int KP = DK < 32 ? 32 : DK;
  static constexpr int LKH = KP + 8;
  static constexpr size_t qk = size_t(4) * kBc * LKH * 2;        // q_j, k_j planes (hi, lo)
  static constexpr size_t xy = size_t(kCP) * 4 * kBc * kUL * 2;  // -X_jc, Y_jc planes of a group
  static constexpr size_t diag = size_t(2) * kBc * kLs * 4;  // (I + X_jj)^-1 and Y_jj
  static constexpr size_t meta = size_t(kHMaxT) * (2 + 2 + 4 + 4 + 4);
  static constexpr size_t total = qk + xy + diag + meta;
};

// ONE: trees of at most 32 slots, i.e. one block.  The workgroup then forms its
// head's Gram block and diagonal matrices itself: the launch of their own took 5
// to 12 us, the work in here 2 to 8.  Whole calls: 1 x 9 slots of a toy layer
// 16.6 -> 13.6 us, 8 x 12 slots, 16 / 32 heads of 64: 19.6 -> 16.3, 8 x 32 and
// 32 x 32, 16 / 48 heads of 128: 40.4 -> 36.4 and 72.7 -> 68.1.
template <int DK, int DV, typename TIn, bool ONE>
__global__ __launch_bounds__(kHT, 4) void chunk_kernel(ChunkParams p) {
  using SM = ChunkSmem<DK, DV>;
  constexpr int KP = SM::KP, LKH = SM::LKH;
  constexpr int NKS = KP / 32;    // k steps of the S0 products
  constexpr int NTV = DV / 16;    // waves with channels
  constexpr int NQK = (2 * kBc * (DK / 4) + kHT - 1) / kHT;
  constexpr int kPl = kBc * kUL;  // halves of a plane
  static_assert(NTV <= kHT / 64 && SM::total <= 80 * 1024, "two workgroups per CU");
  extern __shared__ __align__(16) unsigned char smem[];
  uint16_t* s_qh = reinterpret_cast<uint16_t*>(smem);
  uint16_t* s_ql = s_qh + kBc * LKH;
  uint16_t* s_kh = s_ql + kBc * LKH;
  uint16_t* s_kl = s_kh + kBc * LKH;
  uint16_t* s_xy = reinterpret_cast<uint16_t*>(smem + SM::qk);  // [kCP][-X hi, -X lo, Y hi, Y lo][32][kUL]
  float* s_d = reinterpret_cast<float*>(smem + SM::qk + SM::xy);  // [2][32][kLs]
  int16_t* s_ord = reinterpret_cast<int16_t*>(s_d + 2 * kBc * kLs);
  int16_t* s_ppos = s_ord + kHMaxT;
  float* s_lal = reinterpret_cast<float*>(s_ppos + kHMaxT);
  float* s_la = s_lal + kHMaxT;
  float* s_be = s_la + kHMaxT;
  float* s_a = s_lal;  // a_p, once the partial sums are done

  // The G value heads of unit u = (sequence, key head) read the same Gram
  // blocks: blocks u % 8 + 8 j of their group of 8 G, i.e. one XCD.
  const int T = p.T, Hk = p.Hk, Hv = p.Hv;
  const int G = Hv / Hk;
  const unsigned blk = blockIdx.y * gridDim.x + blockIdx.x;  // y above 1 only past 2^22 blocks
  const int grp = blk / (8u * G), rem = blk % (8u * G);
  const int unit = 8 * grp + rem % 8;
  if (unit >= p.B * Hk) return;  // uniform
  const int b = unit / Hk, g = unit % Hk, h = g * G + rem / 8;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, m = lane >> 4;
  const int nq = Hk * DK;
  const size_t C = size_t(2 * nq + Hv * DV);
  const MetaPtrs m_ = meta_ptrs(p.meta, p.B, T);
  const size_t bt = size_t(b) * T;
  const int nval = __builtin_amdgcn_readfirstlane(m_.status[b] == GDN_TREE_OK ? m_.nvalid[b] : 0);
  const int NB = (T + kBc - 1) / kBc, NBv = (nval + kBc - 1) / kBc;
  const TIn* alpha = static_cast<const TIn*>(p.alpha);
  const TIn* beta = static_cast<const TIn*>(p.beta);
  const float* Fq = p.F + bt * C + g * DK;            // uniform
  const float* Fv = p.F + bt * C + 2 * nq + h * DV;
  const uint32_t C4 = uint32_t(C) * 4, H4 = uint32_t(Hv) * DV * 4;  // row bytes
  const int col = 16 * wave + l16;  // this lane's channel (wave < NTV)
  const bool chan = wave < NTV;
  float* outb = p.out + bt * size_t(Hv) * DV + size_t(h) * DV;
  const float* Db = p.D + (size_t(b) * Hv + h) * NB * (2 * kBc * kBc);
  const float* Gb = p.Gm + (size_t(b) * Hk + g) * (size_t(NB) * (NB - 1) / 2) * (2 * kBc * kBc);
  // this wave's U; waves without channels load the first wave's (all loads are
  // unconditional) and store nothing
  uint16_t* Uw = p.U + (((size_t(b) * Hv + h) * NB) * NTV + (chan ? wave : 0)) * (2 * 64 * 8);
  constexpr int kUB = NTV * 2 * 64 * 8;  // halves of U per block

  // ---- metadata by position: node, parent position, log2 alpha, beta
  for (int j = tid; j < T; j += kHT) {
    const int nd = m_.order[bt + j];
    const bool real = j < nval;
    s_ord[j] = int16_t(nd);
    s_ppos[j] = int16_t(real ? m_.ppos[bt + j] : -1);
    // log2 alpha, floored at the smallest normal float so that alpha = 0
    // still gives finite ratios a_i / a_j
    s_lal[j] = real ? fmaxf(log2f(ld(alpha, (bt + nd) * Hv + h)), kMinLog2) : 0.0f;
    s_be[j] = real ? ld(beta, (bt + nd) * Hv + h) : 0.0f;
  }
  for (int i = tid; i < (T - nval) * (DV / 4); i += kHT) {  // padding slots
    const int nd = m_.order[bt + nval + i / (DV / 4)];
    *reinterpret_cast<float4*>(outb + size_t(nd) * Hv * DV + 4 * (i % (DV / 4))) = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  if (nval == 0) return;  // uniform
  // block rows of q~ and k~ -> hi / lo planes, loaded a block ahead
  float4 qkv[NQK];
  auto fetch_qk = [&](int jb) {
    const int tid = opaque(threadIdx.x);
#pragma unroll
    for (int j = 0; j < NQK; ++j) {
      const int i = j * kHT + tid;
      const int part = i / (kBc * (DK / 4)) & 1, r = i / (DK / 4) % kBc, c4 = i % (DK / 4);
      const int pos = kBc * jb + r;
      // clamped rows: every load is unconditional; rows past the tree are
      // zeroed at the store
      const size_t off = size_t(uint32_t(pos < nval ? pos : 0)) * C4 + (part ? 4 * nq : 0) + 16 * c4;
      qkv[j] = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(Fq) + off);
    }
  };
  auto store_qk = [&](int jb) {
    const int tid = opaque(threadIdx.x);
#pragma unroll
    for (int j = 0; j < NQK; ++j) {
      const int i = j * kHT + tid;
      if (i < 2 * kBc * (DK / 4)) {
        const int part = i / (kBc * (DK / 4)), r = i / (DK / 4) % kBc, c4 = i % (DK / 4);
        const float4 v = kBc * jb + r < nval ? qkv[j] : make_float4(0.f, 0.f, 0.f, 0.f);
        st_split4((part ? s_kh : s_qh) + r * LKH + 4 * c4, (part ? s_kl : s_ql) + r * LKH + 4 * c4, v);
      }
    }
    if constexpr (DK < KP) {  // zero padding of the contraction
      for (int i = tid; i < 4 * kBc * (KP - DK); i += kHT)
        s_qh[i / (KP - DK) * LKH + DK + i % (KP - DK)] = 0;
    }
  };
  // top of a block, loaded a block ahead: the earlier blocks that hold an
  // ancestor of one of its nodes, its values, its diagonal matrices
  int flag;
  f32x4 vop[2];
  float4 dg;
  auto fetch_top = [&](int jb) {
    const int tid = opaque(threadIdx.x), lane = tid & 63, l16 = lane & 15, m = lane >> 4;
    if constexpr (!ONE) {
      flag = p.need[(size_t(b) * NB + jb) * kMaxNB + (lane < jb ? lane : 0)];
      dg = *reinterpret_cast<const float4*>(Db + size_t(jb) * (2 * kBc * kBc) + 4 * tid);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int pos = kBc * jb + 16 * t + 4 * m + e;
        const size_t off = size_t(uint32_t(pos < nval ? pos : 0)) * C4 + 4 * (chan ? 16 * wave + l16 : l16);
        vop[t][e] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(Fv) + off);
      }
  };
  static_assert(kHT * 4 == 2 * kBc * kBc, "a float4 of the diagonal matrices per thread");
  fetch_qk(0);
  fetch_top(0);
  constexpr int kDiagWave = kHT / 64 - 1;  // ONE: the last to have channels
  float ga = 0.0f, gb = 0.0f;
  int gp = -1;
  if constexpr (ONE) {
    if (wave == kDiagWave) {
      const int pc = (lane & (kBc - 1)) < nval ? lane & (kBc - 1) : 0, nd = m_.order[bt + pc];
      ga = ld(alpha, (bt + nd) * Hv + h);
      gb = ld(beta, (bt + nd) * Hv + h);
      gp = m_.ppos[bt + pc];
    }
  }
  // ---- this wave's rows of S0 as operands: channel 16 wave + l16, columns
  //      32 ks + 8 m .. + 7
  bf16x8 sh[NKS], sl_[NKS];
  {
    const float* S0 = p.S0 + (size_t(b) * Hv + h) * size_t(DV) * DK + size_t(chan ? col : 0) * DK;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      float x[8];
      const int k0 = DK < 32 ? 8 * (m & 1) : 32 * ks + 8 * m;
      const float4 u = *reinterpret_cast<const float4*>(S0 + k0), v = *reinterpret_cast<const float4*>(S0 + k0 + 4);
      const bool in = DK >= 32 || m < 2;
      x[0] = in ? u.x : 0.f; x[1] = in ? u.y : 0.f; x[2] = in ? u.z : 0.f; x[3] = in ? u.w : 0.f;
      x[4] = in ? v.x : 0.f; x[5] = in ? v.y : 0.f; x[6] = in ? v.z : 0.f; x[7] = in ? v.w : 0.f;
      split8(x, sh[ks], sl_[ks]);
    }
  }
  __syncthreads();
  // log2 a_p: sum of log2 alpha over the path root..p, by pointer jumping
  // (ceil(log2 T) rounds instead of a walk of depth(p) steps per position;
  // s_lal and s_ppos are rewritten to partial sums and 2^r-th ancestors)
  static_assert(kHT >= kHMaxT, "one position per thread");
  {
    float sl = tid < T ? s_lal[tid] : 0.0f;
    int nx = tid < T ? s_ppos[tid] : -1;
    for (int span = 1; span < T; span <<= 1) {
      if (nx >= 0) {
        sl += s_lal[nx];
        nx = s_ppos[nx];
      }
      __syncthreads();
      if (tid < T) {
        s_lal[tid] = sl;
        s_ppos[tid] = int16_t(nx);
      }
      __syncthreads();
    }
    s_la[tid] = sl;  // 0 past the tree
    s_a[tid] = tid < nval ? __builtin_amdgcn_exp2f(sl) : 0.0f;
    if (tid >= nval) s_be[tid] = 0.0f;
  }

  // ---- cascade over the blocks
  static_assert(kHT == kBc * kBc / 2, "two elements of a block per thread");
  const f32x4 z4 = {0.f, 0.f, 0.f, 0.f};
  for (int jb = 0; jb < NBv; ++jb) {
    // lane roles that the compiler cannot see through: addresses are formed
    // where they are used, not kept over the loop and spilled
    const int tid = opaque(threadIdx.x), lane = tid & 63, l16 = lane & 15, m = lane >> 4;
    const int col = 16 * wave + l16;
    const int xi = tid / (kBc / 2), xc = 2 * (tid % (kBc / 2));  // this thread's X, Y elements: row, columns xc, xc + 1
    uint32_t need = ONE ? 0u : uint32_t(__ballot(lane < jb && flag != 0));
    // Gram blocks of a group, two elements of each per thread
    float2 gx[kCP], gy[kCP];
    uint32_t gm[kCP];
    int cs[kCP];
    auto fetch_group = [&] {
#pragma unroll
      for (int q = 0; q < kCP; ++q) {
        cs[q] = need ? __ffs(int(need)) - 1 : -1;
        if constexpr (ONE) continue;
        need &= need - 1u;
        const int c = cs[q] >= 0 ? cs[q] : 0;  // loads without a branch, unused where there is no block
        const float* gp = Gb + (size_t(jb) * (jb - 1) / 2 + c) * (2 * kBc * kBc) + xi * kBc + xc;
        gx[q] = *reinterpret_cast<const float2*>(gp);
        gy[q] = *reinterpret_cast<const float2*>(gp + kBc * kBc);
        gm[q] = p.mask[((size_t(b) * NB + jb) * kMaxNB + c) * kBc + xi];
      }
    };
    fetch_group();
    __syncthreads();  // LDS of the block before is read (first block: s_la is written)
    store_qk(jb);
    if constexpr (!ONE) *reinterpret_cast<float4*>(s_d + tid / 8 * kLs + 4 * (tid % 8)) = dg;  // tile (0, 1) of neither is read
    __syncthreads();
    if constexpr (ONE) {
      float* s_g = reinterpret_cast<float*>(s_xy);  // the Gram blocks, then a wave's diagonal matrices
      static_assert((2 * kBc * kLs + kDiagLds) * 4 <= SM::xy, "Gram blocks in the place of X and Y");
      const int kind = wave >> 2, ti = (wave >> 1) & 1, tc = wave & 1;
      const f32x4 gm = mm16x3<KP>((kind ? s_qh : s_kh) + 16 * ti * LKH, (kind ? s_ql : s_kl) + 16 * ti * LKH, LKH,
                                  s_kh + 16 * tc * LKH, s_kl + 16 * tc * LKH, LKH, f32x4{0.f, 0.f, 0.f, 0.f}, lane);
#pragma unroll
      for (int e = 0; e < 4; ++e) s_g[kind * kBc * kLs + (16 * ti + 4 * m + e) * kLs + 16 * tc + l16] = gm[e];
      __syncthreads();
      if (wave == kDiagWave) diag_block<kLs>(s_g, s_g + 2 * kBc * kLs, ga, gb, gp, nval, lane, s_d);
    }
    // ---- O_j = a Q S0^T, R_j = beta (V - a K S0^T)
    f32x4 rr[2] = {z4, z4}, oo[2] = {z4, z4};
    if (chan) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
          const int o = (16 * t + l16) * LKH + 32 * ks + 8 * m;
          oo[t] = mfma3(*reinterpret_cast<const bf16x8*>(s_qh + o), *reinterpret_cast<const bf16x8*>(s_ql + o), sh[ks],
                        sl_[ks], oo[t]);
          rr[t] = mfma3(*reinterpret_cast<const bf16x8*>(s_kh + o), *reinterpret_cast<const bf16x8*>(s_kl + o), sh[ks],
                        sl_[ks], rr[t]);
        }
        const int p0 = kBc * jb + 16 * t + 4 * m;
        const f32x4 a = as_x4(*reinterpret_cast<const float4*>(s_a + p0));
        const f32x4 be = as_x4(*reinterpret_cast<const float4*>(s_be + p0));
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          oo[t][e] = a[e] * oo[t][e];
          rr[t][e] = be[e] * (vop[t][e] - a[e] * rr[t][e]);
        }
        if (kBc * jb + kBc > nval) {  // uniform: rows past the tree
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (p0 + e >= nval) oo[t][e] = rr[t][e] = 0.0f;
        }
      }
    }
    // ---- R_j -= X_jc U_c, O_j += Y_jc U_c, kCP blocks c at a time
    while (cs[0] >= 0) {
      bf16x8 uh[kCP], ul[kCP];
#pragma unroll
      for (int q = 0; q < kCP; ++q) {
        const uint16_t* up = Uw + size_t(cs[q] >= 0 ? cs[q] : 0) * kUB + 8 * lane;
        uh[q] = *reinterpret_cast<const bf16x8*>(up);
        ul[q] = *reinterpret_cast<const bf16x8*>(up + 64 * 8);
      }
      const int pi = kBc * jb + xi;
      const float la = s_la[pi], be = s_be[pi];  // rows past the tree: no ancestors
#pragma unroll
      for (int q = 0; q < kCP; ++q) {
        if (cs[q] < 0) break;  // uniform
        const float2 lc = *reinterpret_cast<const float2*>(s_la + kBc * cs[q] + xc);
        float x[2] = {gx[q].x, gx[q].y}, y[2] = {gy[q].x, gy[q].y};
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const bool anc = (gm[q] >> (xc + e)) & 1u;
          const float r = __builtin_amdgcn_exp2f(la - (e ? lc.y : lc.x));
          x[e] = anc ? -be * (r * x[e]) : 0.0f;
          y[e] = anc ? r * y[e] : 0.0f;
        }
        uint16_t* pl = s_xy + q * 4 * kPl + xi * kUL + slot_col(xc);
        st_split2(pl, pl + kPl, x[0], x[1]);
        st_split2(pl + 2 * kPl, pl + 3 * kPl, y[0], y[1]);
      }
      const bool second = cs[kCP - 1] >= 0;  // uniform
      fetch_group();  // the next group's loads fly during this one
      __syncthreads();
      if (chan) {
#pragma unroll
        for (int q = 0; q < kCP; ++q) {
          if (q > 0 && !second) break;  // uniform
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const uint16_t* pl = s_xy + q * 4 * kPl + (16 * t + l16) * kUL + 8 * m;
            rr[t] = mfma3(*reinterpret_cast<const bf16x8*>(pl), *reinterpret_cast<const bf16x8*>(pl + kPl), uh[q],
                          ul[q], rr[t]);
            oo[t] = mfma3(*reinterpret_cast<const bf16x8*>(pl + 2 * kPl),
                          *reinterpret_cast<const bf16x8*>(pl + 3 * kPl), uh[q], ul[q], oo[t]);
          }
        }
      }
      if (cs[0] >= 0) __syncthreads();  // uniform: the planes are read
    }
    if (jb + 1 < NBv) {
      fetch_qk(jb + 1);
      fetch_top(jb + 1);
    }
    if constexpr (ONE) __syncthreads();  // the diagonal matrices are written
    // ---- U_j = (I + X_jj)^-1 R_j, kept as operands of the later blocks
    if (chan) {
      const float* vp = s_d + l16 * kLs + 4 * m;
      const float* yp = vp + kBc * kLs;
      auto tile = [](const float* q) { return as_x4(*reinterpret_cast<const float4*>(q)); };
      const f32x4 v00 = tile(vp), v10 = tile(vp + 16 * kLs), v11 = tile(vp + 16 * kLs + 16);
      const f32x4 y00 = tile(yp), y10 = tile(yp + 16 * kLs), y11 = tile(yp + 16 * kLs + 16);
      const f32x4 u0 = mm_f(v00, rr[0], z4), u1 = mm_f(v11, rr[1], mm_f(v10, rr[0], z4));
      if constexpr (!ONE) {
        const float x[8] = {u0[0], u0[1], u0[2], u0[3], u1[0], u1[1], u1[2], u1[3]};
        bf16x8 hi, lo;
        split8(x, hi, lo);
        *reinterpret_cast<bf16x8*>(Uw + size_t(jb) * kUB + 8 * lane) = hi;
        *reinterpret_cast<bf16x8*>(Uw + size_t(jb) * kUB + 64 * 8 + 8 * lane) = lo;
      }
      // ---- O_j += Y_jj U_j, scaled and stored
      oo[0] = mm_f(y00, u0, oo[0]);
      oo[1] = mm_f(y11, u1, mm_f(y10, u0, oo[1]));
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int p0 = kBc * jb + 16 * t + 4 * m;
        const short4 nd = *reinterpret_cast<const short4*>(s_ord + p0);
        const int nn[4] = {nd.x, nd.y, nd.z, nd.w};
        // stores without a branch (a branch would make the next block wait for
        // all of them): rows past the tree are zero, those past T, in the last
        // block, go to this lane's U, which nothing reads any more
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float* o = reinterpret_cast<float*>(reinterpret_cast<char*>(outb) + size_t(uint32_t(nn[e])) * H4) + col;
          float* spare = reinterpret_cast<float*>(Uw + size_t(jb) * kUB + 8 * lane);
          *(p0 + e < T ? o : spare) = p0 + e < nval ? p.scale * oo[t][e] : 0.0f;
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Launch: features, Gram blocks, cascade
// ---------------------------------------------------------------------------
template <int DK, int DV, typename TIn>
static int launch_chunk_t(const ChunkParams& p, hipStream_t stream) {
  using SM = ChunkSmem<DK, DV>;
  using SG = GramSmem<DK>;
  const int NB = (p.T + kBc - 1) / kBc, G = p.Hv / p.Hk, units = p.B * p.Hk;
  const auto cascade = NB == 1 ? &chunk_kernel<DK, DV, TIn, true> : &chunk_kernel<DK, DV, TIn, false>;
  int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(cascade), int(SM::total), "verify_chunked");
  if (rc != GDN_OK) return rc;
  if (NB > 1) {
    rc = ensure_dynamic_lds(reinterpret_cast<const void*>(&chunk_gram_kernel<DK, TIn>), int(SG::total),
                            "verify_chunked");
    if (rc != GDN_OK) return rc;
    int groups = 0;
    for (int j = 0; j < NB; ++j) groups += j / kCG + 1;
    hipLaunchKernelGGL((chunk_gram_kernel<DK, TIn>), dim3(p.Hk, groups, p.B), dim3(kHT), SG::total, stream, p);
  }
  // whole groups of 8 G blocks; rows of the grid keep its width below the limit
  const int rows = (units + 7) / 8, wide = (1 << 19) / G > 0 ? (1 << 19) / G : 1;
  const dim3 grid(unsigned(rows < wide ? rows : wide) * 8u * G, (rows + wide - 1) / wide);
  hipLaunchKernelGGL(cascade, grid, dim3(kHT), SM::total, stream, p);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return set_error(GDN_EHIP, "verify_chunked launch: %s", hipGetErrorString(e));
  return GDN_OK;
}

template <int DK, typename TIn>
static int chunk_dv(int dv, const ChunkParams& p, hipStream_t s) {
  switch (dv) {
    case 16: return launch_chunk_t<DK, 16, TIn>(p, s);
    case 32: return launch_chunk_t<DK, 32, TIn>(p, s);
    case 64: return launch_chunk_t<DK, 64, TIn>(p, s);
    case 128: return launch_chunk_t<DK, 128, TIn>(p, s);
  }
  return set_error(GDN_EUNSUPPORTED, "verify_chunked: dv=%d unsupported", dv);
}

template <typename TIn>
static int chunk_dk(int dk, int dv, const ChunkParams& p, hipStream_t s) {
  switch (dk) {
    case 16: return chunk_dv<16, TIn>(dv, p, s);
    case 32: return chunk_dv<32, TIn>(dv, p, s);
    case 64: return chunk_dv<64, TIn>(dv, p, s);
    case 128: return chunk_dv<128, TIn>(dv, p, s);
  }
  return set_error(GDN_EUNSUPPORTED, "verify_chunked: dk=%d unsupported", dk);
}

int launch_verify_chunked(const VerifyArgs& a, void* ws, size_t ws_bytes, hipStream_t stream) {
  if (a.T > kHMaxT) return set_error(GDN_EUNSUPPORTED, "verify_chunked: T=%d exceeds %d", a.T, kHMaxT);
  if (ws_bytes < chunked_workspace_bytes(a.B, a.T, a.Hk, a.Hv, a.dk, a.dv))
    return set_error(GDN_EINVAL, "verify_chunked: workspace of %zu bytes is too small", ws_bytes);
  float* F = static_cast<float*>(ws);
  int rc = launch_features(a, F, stream);
  if (rc != GDN_OK) return rc;
  ChunkParams p;
  p.B = a.B;
  p.T = a.T;
  p.Hk = a.Hk;
  p.Hv = a.Hv;
  p.dv = a.dv;
  p.scale = a.scale;
  p.meta = a.meta;
  p.alpha = a.alpha;
  p.beta = a.beta;
  p.S0 = a.S0;
  p.out = a.out;
  p.F = F;
  const ChunkSizes z(a.B, a.T, a.Hk, a.Hv, a.dk, a.dv);
  unsigned char* w = static_cast<unsigned char*>(ws) + z.f;
  p.D = reinterpret_cast<float*>(w);
  p.Gm = reinterpret_cast<float*>(w += z.d);
  p.mask = reinterpret_cast<uint32_t*>(w += z.g);
  p.need = w += z.k;
  p.U = reinterpret_cast<uint16_t*>(w += z.n);
  if (a.in_dtype == GDN_BF16) return chunk_dk<BF16>(a.dk, a.dv, p, stream);
  return chunk_dk<float>(a.dk, a.dv, p, stream);
}

}  // namespace gdn
