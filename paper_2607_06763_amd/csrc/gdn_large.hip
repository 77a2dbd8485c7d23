// gdn_large.hip -- read-only verification of trees of 129..512 slots.
//
// The verification of one node is the query pull-back of the T <= 128
// kernel (an exact rearrangement of Eq. 7-8): walking the path of i from
// the node to the root with
//     x <- q~_i, r <- 1, acc <- 0;   for t = i, parent(i), ..., root:
//         s = k~_t.x;  acc += r beta_t s v~_t;  x <- x - beta_t s k~_t;  r <- r alpha_t
// gives o_i = scale (S0 (r x) + acc) in the stored orientation.  With up to
// 512 slots the post-conv features of a tree no longer fit in LDS, so the
// work is split in two launches:
//   feat_kernel   one workgroup per (2048 channels, 32 positions, sequence):
//                 the width-4 conv along each node's path (conv-state slots
//                 above the root), SiLU, and the per-head L2 norm of q and
//                 k; written to a workspace of fp16 features FH[B][T][C]
//                 (canonical position order, channels as in conv_w; q~
//                 and k~ have unit norm, each v~ row of a value head is
//                 scaled by the power of two that puts its largest
//                 magnitude in [1, 2), the inverse scale kept in
//                 Vs[B][T][Hv]).  The chunked form reads the same features
//                 as fp32 (launch_features).
//                 The last blocks of the launch compute each tree's
//                 depth-first order.
//   pull_kernel   one workgroup per (value head, sequence), 512 threads:
//                 the head's S0 as one fp16 plane in LDS (each row scaled by
//                 the power of two that puts its largest magnitude in [1, 2),
//                 exact, undone on the output), then tiles of 16 nodes in
//                 depth-first order, one wave each: the walks of a tile are
//                 blocked substitutions on the matrix cores (gdn_pull.h) over
//                 the tile's own 16 rows and its first node's ancestors, 16 at
//                 a time; then O^T = S0 (r X)^T on v_mfma_f32_16x16x32_f16.
//                 The value heads of one key head run on one XCD and share
//                 its k~ rows in L2.
//
// What bounds pull_kernel and why this form: walking the path of every node
// on the VALU (16 lanes per node) gathered each path row once per node below
// it, 4.4 GB per launch at 32 trees x 512 slots, 16 / 48 heads of 128, and
// spent two thirds of its instructions on it.  A tile reads the union of its
// nodes' paths, its own rows plus one chain, once.  That launch (with the
// commit of the fused step) went from 480 to 353 us, verification alone at 16
// x 250 slots, 16 / 32 heads, from 74 to 54 us (both forms in one run); bound
// by the VALU work around the MFMA and the fp32 products of the values.  128
// registers and 80 KB keep two workgroups on a CU, with 9 (fused: 11) spilled
// registers at dk = dv = 128 and none below.  With the values still in fp16,
// rows loaded whole (RowStage) instead of one per lane were 363 -> 310 us at
// 512 slots, the values' accumulators live during the substitutions 62 spills
// and 647 us, and outputs through LDS in whole 256-byte runs changed nothing (B
// = 32) or lost 3 us (B = 1).
// The fused decode step (Sec. 3.4.2) runs the conv-state shift of the
// previous step's commit first, the features on the committed conv state,
// and pull_kernel<..., FUSED>, which commits the previous accepted path into
// its head's state rows (commit_rows) and converts the committed rows
// straight into its plane.
#include <map>
#include <type_traits>
#include <mutex>

#include "gdn_commit_rows.h"
#include "gdn_pull.h"

namespace gdn {

constexpr int kLT = 512;      // threads of a pull-back workgroup (8 waves)
constexpr int kLTile = 16;    // nodes per tile (one wave each)
constexpr int kLMaxT = GDN_MAX_T;  // tree slots supported
constexpr int kFT = 256;      // threads of a feature workgroup

struct LargeParams {
  int B, T, Hk, Hv;
  float scale;
  const void* meta;
  const void *q, *k, *v, *alpha, *beta;
  const float *conv_w, *conv_state, *S0;
  float* out;
  float* F;       // fp32 features [B][T][C] (chunked form)
  _Float16* FH;   // fp16 features [B][T][C] (pull-back)
  float* Vs;      // inverse v~ row scales [B][T][Hv] (pull-back), negative: the row holds values that are not finite
  // depth-first order [B][3][large_order_stride(T)] (pull-back): canonical
  // position and end of the subtree by depth-first index; path of each 16-node
  // tile
  int16_t* ord;
  // fused step: the previous step's commit, run by the pull-back on the rows
  // it reads (conv_state above is then the conv state after the commit)
  CommitParams cp;
};

static size_t fh_bytes(int B, int T, int Hk, int Hv, int dk, int dv) {
  return (size_t(B) * size_t(T) * size_t(2 * Hk * dk + Hv * dv) * 2 + 255) & ~size_t(255);
}

size_t large_workspace_bytes(int B, int T, int Hk, int Hv, int dk, int dv) {
  return fh_bytes(B, T, Hk, Hv, dk, dv) + size_t(B) * size_t(T) * size_t(Hv) * sizeof(float);
}

size_t features_f32_bytes(int B, int T, int Hk, int Hv, int dk, int dv) {
  return size_t(B) * size_t(T) * size_t(2 * Hk * dk + Hv * dv) * sizeof(float);
}

// ---------------------------------------------------------------------------
// Features: conv taps along the path, SiLU, L2 norm (q, k).  One workgroup
// per (kFT CPT channels, block of kFP positions, sequence): each thread keeps
// the conv weights of its CPT channels in registers, the block's conv taps
// are resolved once into LDS, and the raw rows of the next positions are in
// flight while the current ones are computed.  CPT = 8 channels per thread
// for the fp16 workspace (one 16-byte row load and store per tap and
// position), 4 for the fp32 features, whose 16-byte stores then stay
// contiguous across the lanes.
// ---------------------------------------------------------------------------
constexpr int kFP = 32;  // positions per feature workgroup

// First thread (in units of CPT channels) of the value channels: the q / k
// threads come first, the value threads start on a wave boundary, so that
// every wave reads rows of one row stride (the q and k rows have Hk dk
// elements, the v rows Hv dv) and the dv / CPT lanes of a value head are
// aligned consecutive lanes of one wave.
__host__ __device__ inline int feat_vbase(int Hk, int dk, int cpt) {
  const int nqk = 2 * Hk * dk / cpt;
  return (nqk + 63) & ~63;
}

// N raw channels of one row (N = 4 or 8), kept as loaded until they are used
template <typename TIn, int N>
struct RawRow;
template <int N>
struct RawRow<BF16, N> {
  uint32_t u[N / 2];
  __device__ __forceinline__ void load(const BF16* p) {
    if constexpr (N == 8) {
      const uint4 v = *reinterpret_cast<const uint4*>(p);
      u[0] = v.x, u[1] = v.y, u[2] = v.z, u[3] = v.w;
    } else {
      const uint2 v = *reinterpret_cast<const uint2*>(p);
      u[0] = v.x, u[1] = v.y;
    }
  }
  __device__ __forceinline__ void get(float (&x)[N]) const {
#pragma unroll
    for (int j = 0; j < N / 2; ++j) {
      x[2 * j] = __uint_as_float(u[j] << 16);
      x[2 * j + 1] = __uint_as_float(u[j] & 0xffff0000u);
    }
  }
};
template <int N>
struct RawRow<float, N> {
  float4 a[N / 4];
  __device__ __forceinline__ void load(const float* p) {
#pragma unroll
    for (int h = 0; h < N / 4; ++h) a[h] = reinterpret_cast<const float4*>(p)[h];
  }
  __device__ __forceinline__ void get(float (&x)[N]) const {
#pragma unroll
    for (int h = 0; h < N / 4; ++h) x[4 * h] = a[h].x, x[4 * h + 1] = a[h].y, x[4 * h + 2] = a[h].z, x[4 * h + 3] = a[h].w;
  }
};

// Largest |x| over aligned groups of N lanes, on the bit patterns of the
// magnitudes (the same order as the floats; a NaN counts as 0, as fmaxf
// would skip it), one DPP max per step.
template <int N>
__device__ __forceinline__ float group_absmax(float v) {
  uint32_t u = __float_as_uint(v) & 0x7fffffffu;
  u = u > 0x7f800000u ? 0u : u;
  auto mx = [&](uint32_t a, uint32_t o) { return a > o ? a : o; };
  if constexpr (N >= 2) u = mx(u, uint32_t(__builtin_amdgcn_update_dpp(0, int(u), kDppQuadXor1, 0xF, 0xF, false)));
  if constexpr (N >= 4) u = mx(u, uint32_t(__builtin_amdgcn_update_dpp(0, int(u), kDppQuadXor2, 0xF, 0xF, false)));
  if constexpr (N >= 8) u = mx(u, uint32_t(__builtin_amdgcn_update_dpp(0, int(u), kDppRowHalfMirror, 0xF, 0xF, false)));
  if constexpr (N >= 16) u = mx(u, uint32_t(__builtin_amdgcn_update_dpp(0, int(u), kDppRowMirror, 0xF, 0xF, false)));
  if constexpr (N >= 32) u = mx(u, uint32_t(__shfl_xor(int(u), 16)));
  static_assert(N <= 32, "group size");
  return __uint_as_float(u);
}

// Depth-first order of tree b, children by canonical position: ord[i] is the
// canonical position of the i-th node, ord[st + i] the end of its subtree,
// ord[2 st + 16 j + tau] (st: large_order_stride(T)) the indices of the nearest 16 proper ancestors of
// node 16 j, nearest last (kLMaxT: none).  One workgroup of kFT threads; s: 5
// kLMaxT ints.  A node's index is the sum over
// its path, without the root, of 1 + the subtree sizes of the siblings before
// it (siblings share a depth, so they lie between the start of that depth and
// the node).
__device__ __forceinline__ void depth_first_order(const MetaPtrs& m, size_t bt, int T, int nval, int16_t* ord, int* s) {
  int* s_pp = s;               // parent position, -1 for the root
  int* s_size = s + kLMaxT;    // subtree size; then the path sums
  int* s_key = s + 2 * kLMaxT;  // parent position << 16 | subtree size
  int* s_nx = s + 3 * kLMaxT;  // pointer jumping: 2^r-th ancestor; then the parent's index by index
  int* s_at = s + 4 * kLMaxT;  // index by position
  constexpr int NP = kLMaxT / kFT;  // positions per thread
  const int tid = threadIdx.x, st = large_order_stride(T);
  // the last position is the deepest (depth order)
  const int last = m.pdep[bt + nval - 1], deepest = last < T ? last : T - 1;
#pragma unroll
  for (int u = 0; u < NP; ++u) {
    const int i = u * kFT + tid;
    const int pp = i < nval ? m.ppos[bt + i] : -1;
    // a parent comes first (depth order); anything else is corrupt metadata
    s_pp[i] = pp >= 0 && pp < i ? pp : -1;
    s_nx[i] = s_pp[i];
    s_size[i] = 1;
  }
  __syncthreads();
  // subtree sizes by doubling: round r adds to every node the sizes, down to
  // distance 2^r, of the nodes 2^r below it.  With one addition per (node,
  // ancestor) the launch took 51 instead of 34 us on 8 chains of 512.
  int size[NP], sum[NP];
  for (int span = 1; span <= deepest; span <<= 1) {
    int nx[NP];
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      size[u] = s_size[u * kFT + tid];
      nx[u] = s_nx[u * kFT + tid];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      if (nx[u] >= 0) {
        atomicAdd(&s_size[nx[u]], size[u]);
        nx[u] = s_nx[nx[u]];
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NP; ++u) s_nx[u * kFT + tid] = nx[u];
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < NP; ++u) {
    const int i = u * kFT + tid;
    size[u] = s_size[i];
    s_key[i] = i < nval && s_pp[i] >= 0 ? s_pp[i] << 16 | size[u] : -1;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < NP; ++u) {
    const int i = u * kFT + tid;
    const int par = s_pp[i];
    sum[u] = 0;
    if (i < nval && par >= 0) {
      sum[u] = 1;
      // positions after the parent; other depths have other parents
      for (int j = (par + 1) & ~3; j < i; j += 4) {
        const int4 k = *reinterpret_cast<const int4*>(s_key + j);
        const int kk[4] = {k.x, k.y, k.z, k.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[u] += (kk[e] >> 16) == par && j + e < i ? kk[e] & 0xffff : 0;
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < NP; ++u) {
    s_size[u * kFT + tid] = sum[u];
    s_nx[u * kFT + tid] = s_pp[u * kFT + tid];
  }
  __syncthreads();
  for (int span = 1; span <= deepest; span <<= 1) {
    int nx[NP];
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      nx[u] = s_nx[u * kFT + tid];
      if (nx[u] >= 0) {
        sum[u] += s_size[nx[u]];
        nx[u] = s_nx[nx[u]];
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      s_size[u * kFT + tid] = sum[u];
      s_nx[u * kFT + tid] = nx[u];
    }
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < NP; ++u) {
    const int i = u * kFT + tid;
    if (i < nval) {
      const int at = sum[u] < nval ? sum[u] : nval - 1;  // a permutation of 0 .. nval - 1
      s_at[i] = at;
      ord[at] = int16_t(i);
      ord[st + at] = int16_t(at + size[u] < nval ? at + size[u] : nval);
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < NP; ++u) {
    const int i = u * kFT + tid;
    if (i < nval) s_nx[s_at[i]] = s_pp[i] >= 0 ? s_at[s_pp[i]] : -1;
  }
  __syncthreads();
  if (tid < (nval + kLTile - 1) / kLTile) {
    int a = s_nx[kLTile * tid];
    for (int tau = kLTile - 1; tau >= 0; --tau) {
      a = a < kLTile * tid ? a : -1;  // ancestors come first
      ord[2 * st + kLTile * tid + tau] = int16_t(a >= 0 ? a : kLMaxT);
      a = a >= 0 ? s_nx[a] : -1;
    }
  }
}

// VG = 0: fp32 features into p.F; VG = DV / CPT: fp16 features into p.FH
// with the v~ rows of each head scaled (inverse scales into p.Vs), and, in
// the last p.B blocks, the depth-first order of each tree into p.ord.
template <typename TIn, int DK, int VG, int CPT>
__global__ __launch_bounds__(kFT) void feat_kernel(LargeParams p, int DV, int ncb) {
  constexpr bool kHalf = VG > 0;
  static_assert(CPT == 4 || CPT == 8, "channels per thread");
  // positions per register buffer: 32 registers of raw rows (4 taps each)
  constexpr int kFU = 32 / (int(sizeof(TIn)) * CPT);
  __shared__ int s_tap[kFP][4];  // node of each tap, or -1 - conv-state slot
  __shared__ __align__(16) float4 s_cs[3][CPT / 4][kFT];  // conv-state slots of the thread's channels
  // Blocks go round-robin over the 8 XCDs.  The grid is one-dimensional and
  // renumbered so that each XCD takes a contiguous range of (position block,
  // channel block, sequence) in that order: the position blocks of one
  // channel block of a sequence run on one XCD, where the rows that some of
  // them load are still in L2 when others gather them as ancestor taps
  // (measured: 1.5x fewer HBM bytes fetched).
  const int nblk = kHalf ? gridDim.x - p.B : gridDim.x, per = nblk / 8;
  const int id = blockIdx.x;
  if constexpr (kHalf) {
    static_assert(sizeof(s_cs) >= 5 * kLMaxT * sizeof(int), "order LDS");
    if (id >= nblk) {  // uniform
      const int b = id - nblk;
      const MetaPtrs m = meta_ptrs(p.meta, p.B, p.T);
      const int nval = m.status[b] == GDN_TREE_OK ? m.nvalid[b] : 0;
      if (nval > 0)
        depth_first_order(m, size_t(b) * p.T, p.T, nval < p.T ? nval : p.T, p.ord + size_t(b) * 3 * large_order_stride(p.T),
                          reinterpret_cast<int*>(s_cs));
      return;
    }
  }
  const int L = id < 8 * per ? (id % 8) * per + id / 8 : id;
  const int nyb = (p.T + kFP - 1) / kFP;
  const int yb = L % nyb, bx = (L / nyb) % ncb, b = L / (nyb * ncb);
  const int tid = threadIdx.x;
  const int p0 = yb * kFP;
  const int T = p.T, Hk = p.Hk, Hv = p.Hv;
  const MetaPtrs m = meta_ptrs(p.meta, p.B, T);
  const int nval = m.status[b] == GDN_TREE_OK ? m.nvalid[b] : 0;
  if (p0 >= nval) return;  // uniform
  const int np = nval - p0 < kFP ? nval - p0 : kFP;
  const size_t bt = size_t(b) * T;
  if (tid < np) {
    // the 4 taps of position p0 + tid (3 = the node itself): a path node's
    // raw row, or the conv-state slot d + w for taps above the root
    const int pos = p0 + tid;
    const int d = m.pdep[bt + pos];
    const int t2 = m.ppos[bt + pos];
    const int t1 = t2 >= 0 ? m.ppos[bt + t2] : -1;
    const int t0 = t1 >= 0 ? m.ppos[bt + t1] : -1;
    const int tp[4] = {t0, t1, t2, pos};
#pragma unroll
    for (int w = 0; w < 4; ++w) s_tap[tid][w] = d - 3 + w >= 0 ? m.order[bt + tp[w]] : -1 - (d + w);
  }
  const int nq = Hk * DK;
  const int C = 2 * nq + Hv * DV;
  const int vb = feat_vbase(Hk, DK, CPT);
  const int nqkt = 2 * nq / CPT, nvt = Hv * DV / CPT;
  const int ct = bx * kFT + tid;
  const bool isv = ct >= vb;  // the same for the whole wave
  const bool ok = isv ? ct - vb < nvt : ct < nqkt;
  // this thread's first channel; lanes past the channels of their kind
  // compute on the last group of that kind (in bounds) and store nothing
  const int c = isv ? 2 * nq + CPT * (ct - vb < nvt ? ct - vb : nvt - 1) : CPT * (ct < nqkt ? ct : nqkt - 1);
  const TIn* src;
  int off;
  if (c < nq) {
    src = static_cast<const TIn*>(p.q), off = c;
  } else if (c < 2 * nq) {
    src = static_cast<const TIn*>(p.k), off = c - nq;
  } else {
    src = static_cast<const TIn*>(p.v), off = c - 2 * nq;
  }
  // row stride of this wave's tensor (wave-uniform: node offsets are scalar)
  const int rs = __builtin_amdgcn_readfirstlane(isv ? Hv * DV : nq);
  src += bt * size_t(rs) + off;
  float4 wv[CPT];
#pragma unroll
  for (int j = 0; j < CPT; ++j) wv[j] = reinterpret_cast<const float4*>(p.conv_w + size_t(c) * 4)[j];
  const bool qk = !isv;
  // the conv-state slots of this thread's channels (taps above the root),
  // kept in LDS: read under a branch, an LDS load does not make the row
  // loads in flight wait
  {
    const float* cs = p.conv_state + size_t(b) * 3 * C + c;
#pragma unroll
    for (int sl = 0; sl < 3; ++sl)
#pragma unroll
      for (int h = 0; h < CPT / 4; ++h) s_cs[sl][h][tid] = ld4(cs + size_t(sl) * C + 4 * h);
  }
  float* dst = kHalf ? nullptr : p.F + (bt + p0) * size_t(C) + c;
  _Float16* dsth = kHalf ? p.FH + (bt + p0) * size_t(C) + c : nullptr;
  // the first lane of each value head writes the head's inverse scale
  const bool vs_lane = kHalf && ok && isv && (ct - vb) % (kHalf ? VG : 1) == 0;
  float* vs = vs_lane ? p.Vs + (bt + p0) * size_t(Hv) + (ct - vb) / (kHalf ? VG : 1) : nullptr;
  __syncthreads();
  // Two register buffers of kFU positions each: the rows of the next group
  // are in flight while the current one is computed.  Group indices past
  // the block are clamped to its last position (loaded again, not stored).
  RawRow<TIn, CPT> ra[kFU][4], rb[kFU][4];
  int ca[kFU], cb[kFU];  // tap 0's code: negative iff the position is within 3 of the root
  auto load_group = [&](RawRow<TIn, CPT> (&xr)[kFU][4], int (&code)[kFU], int g0) {
#pragma unroll
    for (int u = 0; u < kFU; ++u) {
      const int i = g0 + u < np ? g0 + u : np - 1;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const int nd = __builtin_amdgcn_readfirstlane(s_tap[i][w]);
        if (w == 0) code[u] = nd;
        xr[u][w].load(src + (nd >= 0 ? nd : 0) * rs);
      }
    }
  };
  auto compute_group = [&](const RawRow<TIn, CPT> (&xr)[kFU][4], const int (&code)[kFU], int g0) {
#pragma unroll
    for (int u = 0; u < kFU; ++u) {
      float x[4][CPT];
#pragma unroll
      for (int w = 0; w < 4; ++w) xr[u][w].get(x[w]);
      if (code[u] < 0) {
        // taps above the root read the conv-state slots (uniform; only near
        // the start of a tree, as the canonical order sorts by depth)
        const int i = g0 + u < np ? g0 + u : np - 1;
#pragma unroll
        for (int w = 0; w < 3; ++w) {
          const int cd = __builtin_amdgcn_readfirstlane(s_tap[i][w]);
          if (cd < 0) {
#pragma unroll
            for (int h = 0; h < CPT / 4; ++h) {
              const float4 a = s_cs[-1 - cd][h][tid];
              x[w][4 * h] = a.x, x[w][4 * h + 1] = a.y, x[w][4 * h + 2] = a.z, x[w][4 * h + 3] = a.w;
            }
          }
        }
      }
      float y[CPT];
      float ss = 0.0f;
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        y[j] = silu(fmaf(wv[j].w, x[3][j], fmaf(wv[j].z, x[2][j], fmaf(wv[j].y, x[1][j], wv[j].x * x[0][j]))));
        ss = fmaf(y[j], y[j], ss);
      }
      const bool odd = kHalf && __any(!(ss < __builtin_inff()));  // squares that overflow, or inf or NaN
      // the DK / CPT lanes of a q or k head are consecutive lanes of one wave
      ss = group_sum<DK / CPT>(ss);
      float f = qk ? rsqrt_hw(ss + 1e-6f) : 1.0f;
      const bool st = ok && g0 + u < np;
      if constexpr (kHalf) {
        // v~: one power-of-two scale per (position, head) from the row max
        float mx = 0.0f;
#pragma unroll
        for (int j = 0; j < CPT; ++j) mx = fmaxf(mx, fabsf(y[j]));
        float sc, inv;
        row_scale(group_absmax<VG>(mx), sc, inv);
        if (odd) {  // wave-uniform, rare (one branch: two cost 1 us of latency in small launches)
          float fin = 0.0f, t = 0.0f;
#pragma unroll
          for (int j = 0; j < CPT; ++j) {
            if (fabsf(y[j]) < __builtin_inff())
              fin = fmaxf(fin, fabsf(y[j]));
            else
              t = 1.0f;  // holds inf or NaN
          }
          // the row's largest finite value: an inf must not flush the rest
          row_scale(group_absmax<VG>(fin), sc, inv);
          // a q or k row with one is NaN throughout; a v row says so by the
          // sign of its scale
          if (qk && group_max<DK / CPT>(t) != 0.0f) f = __builtin_nanf("");
          if (!qk && group_max<(kHalf ? VG : 1)>(t) != 0.0f) inv = -inv;
        }
        const float g = qk ? f : sc;
        uint2 h4[CPT / 4];
#pragma unroll
        for (int h = 0; h < CPT / 4; ++h) h4[h] = to_f16x4(make_float4(y[4 * h], y[4 * h + 1], y[4 * h + 2], y[4 * h + 3]), g);
        if (st) {
          if constexpr (CPT == 8)
            *reinterpret_cast<uint4*>(dsth + size_t(g0 + u) * C) = make_uint4(h4[0].x, h4[0].y, h4[1].x, h4[1].y);
          else
            *reinterpret_cast<uint2*>(dsth + size_t(g0 + u) * C) = h4[0];
          if (vs_lane) vs[size_t(g0 + u) * Hv] = inv;
        }
      } else {
        if (st) {
          float4* d4 = reinterpret_cast<float4*>(dst + size_t(g0 + u) * C);
#pragma unroll
          for (int h = 0; h < CPT / 4; ++h)
            d4[h] = make_float4(y[4 * h] * f, y[4 * h + 1] * f, y[4 * h + 2] * f, y[4 * h + 3] * f);
        }
      }
    }
  };
  load_group(ra, ca, 0);
  for (int i0 = 0;;) {
    load_group(rb, cb, i0 + kFU);
    compute_group(ra, ca, i0);
    i0 += kFU;
    if (i0 >= np) break;
    load_group(ra, ca, i0 + kFU);
    compute_group(rb, cb, i0);
    i0 += kFU;
    if (i0 >= np) break;
  }
}

// ---------------------------------------------------------------------------
// Pull-back by tiles of 16 nodes + fp16 MFMA readout
// ---------------------------------------------------------------------------
// Two workgroups per CU: at most 80 KB each.
template <int DK, int DV>
struct PullSmem {
  static constexpr int KP = (DK < 32 ? 32 : DK) + 8;  // fp16 row of the state plane (zero beyond DK)
  static constexpr int KR = DK * 2, VR = DV * 2;       // bytes per row of a chunk
  static constexpr size_t plane = size_t(DV) * KP * 2;
  static constexpr size_t chunk = size_t(kLTile) * (KR > VR ? KR : VR);  // 16 rows of k~ or v~, one per wave
  // the plane and the chunks; in the fused step the commit's LDS first
  static constexpr size_t tiles = plane + (kLT / 64) * chunk;
  static constexpr size_t front = tiles > commit_lds_bytes<DK, DV>() ? tiles : commit_lds_bytes<DK, DV>();
  static constexpr size_t inv = size_t(DV) * 4;
  static constexpr size_t gates = size_t(kLMaxT + 1) * 16;
  static constexpr size_t solve = size_t(kLT / 64) * 64 * 4;
  static constexpr size_t order = size_t(kLMaxT + 8) * 2 * 2 + size_t(kLT / 64) * kLTile * 2;
  static constexpr size_t total = front + inv + gates + solve + order;
};

template <int N>
__device__ __forceinline__ void ld_f(const float* src, float (&x)[N]) {
  if constexpr (N % 4 == 0) {
#pragma unroll
    for (int e = 0; e < N; e += 4) {
      const float4 u = *reinterpret_cast<const float4*>(src + e);
      x[e] = u.x;
      x[e + 1] = u.y;
      x[e + 2] = u.z;
      x[e + 3] = u.w;
    }
  } else {
#pragma unroll
    for (int e = 0; e < N; ++e) x[e] = src[e];
  }
}

// 16 rows of D halves on their way to LDS: a load covers whole rows (16 bytes
// per lane, D / 8 lanes per row), which keeps the address lanes of the vector
// cache few: with a row per lane a load took 64 lookups and the launch was
// bound by them (32 x 512 slots, no commit, values in fp16: 295 us, 243 with
// whole rows).  In LDS row rho is at rho * 2 D bytes, its 32-byte granules
// swizzled by rho.
template <int D>
struct RowStage {
  static constexpr int KB = D >= 32 ? D / 32 : 1;
  static constexpr int kMask = D / 16 - 1;       // granule index mask
  static constexpr int PPR = D / 8;              // 16-byte pieces per row
  static constexpr int NI = (kLTile * PPR + 63) / 64;
  f16x8 st[NI];
  // rowoff: in lane rho (and rho + 16, ...), byte offset of row rho (rows of
  // one sequence span less than 4 GB)
  __device__ __forceinline__ void load(const _Float16* base, uint32_t rowoff, int lane) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int rho = (64 / PPR * i + lane / PPR) & (kLTile - 1);
      const uint32_t off = uint32_t(__builtin_amdgcn_ds_bpermute(4 * rho, int(rowoff))) + 16u * (lane % PPR);
      st[i] = *reinterpret_cast<const f16x8*>(reinterpret_cast<const char*>(base) + off);
    }
  }
  // values that are not finite -> 0
  __device__ __forceinline__ void keep_finite() {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int e = 0; e < 8; ++e) st[i][e] = fabsf((float)st[i][e]) < 65536.0f ? st[i][e] : (_Float16)0.0f;
  }
  __device__ __forceinline__ void store(unsigned char* buf, int lane) const {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int rho = 64 / PPR * i + lane / PPR, pc = lane % PPR;
      if (kLTile * PPR >= 64 || rho < kLTile)
        *reinterpret_cast<f16x8*>(buf + rho * 2 * D + (((pc >> 1) ^ rho) & kMask) * 32 + 16 * (pc & 1)) = st[i];
    }
  }
  // A operand in channel order: channels 32 kb + 8 m .. + 7 of row l16 (zero
  // beyond D = 16)
  __device__ static __forceinline__ unsigned char* piece(unsigned char* buf, int kb, int l16, int m) {
    return buf + l16 * 2 * D + (((2 * kb + (m >> 1)) ^ l16) & kMask) * 32 + 16 * (m & 1);
  }
  __device__ static __forceinline__ f16x8 frag(unsigned char* buf, int kb, int l16, int m) {
    f16x8 f = *reinterpret_cast<const f16x8*>(piece(buf, kb, l16, m));
    if (D < 32 && m >= 2) f = f16x8{0, 0, 0, 0, 0, 0, 0, 0};
    return f;
  }
  // 4 channels 16 t + 4 m .. of row l16 (accumulator slot order)
  __device__ static __forceinline__ f16x4 slots(const unsigned char* buf, int t, int l16, int m) {
    return *reinterpret_cast<const f16x4*>(buf + l16 * 2 * D + ((t ^ l16) & kMask) * 32 + 8 * m);
  }
  // channel 16 t + l16 of rows 4 m .. 4 m + 3
  __device__ static __forceinline__ f16x4 columns(const unsigned char* buf, int t, int l16, int m) {
    const int r = 4 * m + (l16 >> 2);
    return ld_tr(buf + r * 2 * D + ((t ^ r) & kMask) * 32 + 8 * (l16 & 3));
  }
};

// Gates of a node for one value head
struct RowGate {
  float be, al, vs;  // beta, alpha, inverse v~ row scale (sign: see LargeParams)
  int end;           // end of the subtree, 0 past the nodes
};

template <int DK, int DV, typename TIn, bool FUSED>
__global__ __launch_bounds__(kLT, 4) void pull_kernel(LargeParams p) {
  using SM = PullSmem<DK, DV>;
  using KF = RowStage<DK>;
  using VF = RowStage<DV>;
  constexpr int KP = SM::KP;
  constexpr int CK = DK / 16;                 // state columns per lane of the plane set-up
  constexpr int NX = DK / 16, NV = DV / 16;   // 16-channel tiles
  constexpr int KB = KF::KB;
  static_assert(SM::total <= 80 * 1024, "two workgroups per CU");
  extern __shared__ __align__(16) unsigned char smem[];
  _Float16* s_plane = reinterpret_cast<_Float16*>(smem);
  float* s_inv = reinterpret_cast<float*>(smem + SM::front);
  RowGate* s_g = reinterpret_cast<RowGate*>(s_inv + DV);       // by depth-first index; kLMaxT: no node
  float* s_solve = reinterpret_cast<float*>(s_g + kLMaxT + 1);  // 64 floats per wave
  int16_t* s_row = reinterpret_cast<int16_t*>(s_solve + kLT);  // canonical position
  int16_t* s_path = s_row + kLMaxT + 8;      // nearest ancestors of each tile's first node
  int16_t* s_list = s_path + kLMaxT + 8;     // 16 path nodes per wave (deeper trees)

  // Blocks go round-robin over the 8 XCDs: the G value heads of unit u =
  // (sequence, key head), which gather the same k~ rows, take blocks
  // u % 8 + 8 j of their group of 8 G, i.e. one XCD and one L2.
  const int T = p.T, Hk = p.Hk, Hv = p.Hv;
  const int G = Hv / Hk;
  const int grp = blockIdx.x / (8 * G), rem = blockIdx.x % (8 * G);
  const int unit = 8 * grp + rem % 8;
  if (unit >= p.B * Hk) return;  // uniform
  const int b = unit / Hk, g = unit % Hk, h = g * G + rem / 8;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nq = Hk * DK;
  const size_t C = size_t(2 * nq + Hv * DV);
  const MetaPtrs m_ = meta_ptrs(p.meta, p.B, T);
  const size_t bt = size_t(b) * T;
  const int nval = __builtin_amdgcn_readfirstlane(m_.status[b] == GDN_TREE_OK ? m_.nvalid[b] : 0);
  const TIn* alpha = static_cast<const TIn*>(p.alpha);
  const TIn* beta = static_cast<const TIn*>(p.beta);
  const _Float16* Fb = p.FH + bt * C;
  const _Float16* Fk = Fb + nq + g * DK;
  const _Float16* Fv = Fb + 2 * nq + h * DV;

  // ---- this thread's share of S0 (16 lanes per row), in flight first
  constexpr int NR = (DV + kLT / 16 - 1) / (kLT / 16);  // rows per thread
  float xs[FUSED ? 1 : NR][CK];
  if constexpr (!FUSED) {
    const float* S0 = p.S0 + (size_t(b) * Hv + h) * size_t(DV) * DK;
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      const int r = j * (kLT / 16) + (tid >> 4);
      ld_f<CK>(S0 + size_t(r < DV ? r : DV - 1) * DK + (tid & 15) * CK, xs[j]);
    }
  }
  // ---- order and this head's gates by depth-first index
  const int ost = large_order_stride(T);
  const int16_t* ord = p.ord + size_t(b) * 3 * ost;
  bool grows = false;
  for (int j = tid; j <= kLMaxT; j += kLT) {
    const bool real = j < nval;
    int row = nval > 0 ? ord[real ? j : nval - 1] : 0;  // past the nodes: the last one's row
    const int end = ord[ost + (real ? j : 0)];
    const bool live = j / kLTile * kLTile < nval;  // a tile with nodes
    const int a = ord[2 * ost + (live ? j : 0)];
    row = row >= 0 && row < T ? row : 0;
    RowGate g = {0.0f, 0.0f, 0.0f, 0};
    // the scale, and with it the mark, of the row that is loaded: an absent
    // row's coefficient is 0, and 0 times inf would reach the whole tile
    if (nval > 0) g.vs = p.Vs[(bt + row) * Hv + h];
    if (real) {
      const int nd = m_.order[bt + row];
      g.al = ld(alpha, (bt + nd) * Hv + h);
      g.be = ld(beta, (bt + nd) * Hv + h);
      g.end = end;
      grows = grows || g.be < 0.0f || g.be > 2.0f;
    }
    s_g[j] = g;
    s_row[j] = int16_t(row);
    if (j < kLMaxT) s_path[j] = int16_t(a >= 0 && a < kLMaxT && live ? a : kLMaxT);
  }
  if constexpr (FUSED) {
    // ---- fused step: the previous step's accepted path is committed into
    //      this head's rows (its LDS in the plane and chunk region), the rows
    //      go back to S and straight into the fp16 plane
    using CS = CommitSplit<DK, DV, kLT>;
    float srow[CS::EPT];
    const bool changed = commit_rows<DK, DV, TIn, kLT, true>(p.cp, b, h, tid, commit_lds<DK, DV>(smem), srow);
    if (changed) store_rows<DK, DV, kLT>(p.cp.S, b, h, Hv, tid, srow);
    const int row = tid / CS::LPR, col0 = (tid % CS::LPR) * CS::CPT;
#pragma unroll
    for (int i = 0; i < CS::R; ++i) {
      float mx = 0.0f;
#pragma unroll
      for (int e = 0; e < CS::CPT; ++e) mx = fmaxf(mx, fabsf(srow[i * CS::CPT + e]));
      mx = group_max<CS::LPR>(mx);
      float sc, inv;
      row_scale(mx, sc, inv);
      const int r = row + i * CS::RS;
#pragma unroll
      for (int e = 0; e < CS::CPT; ++e)
        s_plane[r * KP + plane_col(col0 + e)] = (_Float16)(srow[i * CS::CPT + e] * sc);
      if (tid % CS::LPR == 0) s_inv[r] = p.scale * inv;
    }
  } else if (nval > 0) {
    // ---- S0 -> fp16 plane
    const int ln = tid & 15;
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      const int r = j * (kLT / 16) + (tid >> 4);
      if (r < DV) {  // uniform per 16-lane group
        float mx = 0.0f;
#pragma unroll
        for (int e = 0; e < CK; ++e) mx = fmaxf(mx, fabsf(xs[j][e]));
        mx = group_max<16>(mx);
        float sc, inv;
        row_scale(mx, sc, inv);
#pragma unroll
        for (int e = 0; e < CK; ++e) s_plane[r * KP + plane_col(ln * CK + e)] = (_Float16)(xs[j][e] * sc);
        if (ln == 0) s_inv[r] = p.scale * inv;
      }
    }
  }
  if constexpr (DK < 32) {  // zero columns past DK
    for (int i = tid; i < DV * (32 - DK); i += kLT)
      s_plane[(i / (32 - DK)) * KP + plane_col(DK + i % (32 - DK))] = (_Float16)0.0f;
  }
  // q~, and with it x and c, is taken times 2^13, so that the fp16 hi + lo that
  // the products take of x and c end at 2^-38 of |q~| = 1, not at 2^-25.  For
  // beta in [0, 2] |x| does not grow, and c stays a factor of 4 below fp16's
  // largest; a node with any other beta on its path takes q~ as it is, and x has
  // all of fp16's range.
  constexpr float kUnit = 0x1p13f;
  const bool grown = __builtin_amdgcn_readfirstlane(__syncthreads_or(grows)) != 0;

  // ---- tiles of 16 nodes, one wave each: no barrier below
  unsigned char* buf = smem + SM::plane + wave * SM::chunk;
  float* z = s_solve + 64 * wave;
  int16_t* list = s_list + kLTile * wave;
  const f32x4 z4 = {0.f, 0.f, 0.f, 0.f};
  for (int n0 = kLTile * wave; n0 < T; n0 += kLT / 64 * kLTile) {
    // lane roles from values that the compiler cannot see through: addresses
    // are formed where they are used, not hoisted, kept and spilled
    const int ln = opaque(lane), l16 = ln & 15, m = ln >> 4;
    const int n = n0 + l16;  // this lane's column
    // slots of the tile's nodes; the padding ones come in canonical order
    const int slot = n < T ? m_.order[bt + (n < nval ? int(s_row[n]) : n)] : 0;
    float* outh = p.out + bt * size_t(Hv) * DV + size_t(h) * DV;  // uniform
    if (n0 >= nval) {  // uniform
      if (n < T) {
#pragma unroll
        for (int t = 0; t < NV; ++t)
          *reinterpret_cast<float4*>(outh + size_t(slot) * Hv * DV + 4 * m + 16 * t) = make_float4(0.f, 0.f, 0.f, 0.f);
      }
      continue;
    }
    // index of row tau of a chunk: the tile's own (lst null) or a list's
    auto index = [&](const int16_t* lst, int tau) { return lst ? int(lst[tau]) : n0 + tau; };
    const float y1 = one_f();
    // k~ and v~ rows of a chunk load one stage ahead: kf holds the next
    // chunk's k~ while one is solved, vf the own v~ rows while the second is.
    KF kf;
    VF vf;
    f16x8 qf[KB];   // q~ of column l16 times kUnit, channel order
    f16x4 qc[NX];   // and accumulator order
    f32x4 x[NX], acc[NV];  // x times kUnit
    const int16_t* path = s_path + n0;
    const int near = path[kLTile - 1];  // parent of the tile's first node
    auto row_off = [&](const int16_t* lst) {  // of operand row l16
      return uint32_t(s_row[index(lst, tau_of(opaque(lane) & 15))]) * uint32_t(2 * C);
    };
    auto load_k = [&](const int16_t* lst) { kf.load(Fk, row_off(lst), opaque(lane)); };
    auto load_v = [&](const int16_t* lst) { vf.load(Fv, row_off(lst), opaque(lane)); };
    {
      KF qs;
      qs.load(Fb + g * DK, uint32_t(s_row[n]) * uint32_t(2 * C), lane);
      load_k(nullptr);
#pragma unroll
      for (int i = 0; i < KF::NI; ++i) qs.st[i] *= (_Float16)kUnit;
      qs.store(buf, opaque(lane));
      wave_lds_order();
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) qf[kb] = KF::frag(buf, kb, l16, m);
#pragma unroll
      for (int t = 0; t < NX; ++t) qc[t] = KF::slots(buf, t, l16, m);
      wave_lds_order();
    }
    float rw = 1.0f / kUnit;  // decay of the rows walked, over x's unit
    if (grown) {  // uniform, rare: only the nodes below such a beta
      bool below = false;
      for (int a = 0; a < n0 + kLTile; ++a) {
        const RowGate g = s_g[a];
        below = below || (a <= n && n < g.end && (g.be < 0.0f || g.be > 2.0f));
      }
      if (below) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) qf[kb] *= (_Float16)(1.0f / kUnit);
#pragma unroll
        for (int t = 0; t < NX; ++t) qc[t] *= (_Float16)(1.0f / kUnit);
        rw = 1.0f;
      }
    }
    // The substitution over one chunk of path nodes: x and rw move up by the
    // chunk; returns the value coefficients r c / (v~ row scale) of the
    // accumulator rows.  kf: the chunk's k~ rows on entry; once they are in
    // LDS, ahead() issues later loads.  vmin: below 0 if a v~ row of this
    // lane's is marked.
    auto solve = [&](const int16_t* lst, float& vmin, auto ahead) -> f32x4 {
      const bool own = lst == nullptr;
      const int ln = opaque(lane), l16 = ln & 15, m = ln >> 4;
      const int il = index(lst, tau_of(l16));
      const RowGate gl = s_g[il];
      // ---- s = K x, Gram tile
      f32x4 s = z4, gm = z4;
      kf.store(buf, ln);
      ahead();
      wave_lds_order();
      f16x8 ka[KB];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        ka[kb] = KF::frag(buf, kb, l16, m);
        gm = mfma_h(ka[kb], ka[kb], gm);
      }
      // a key that is not finite (its row is NaN) shows on the diagonal: a
      // zero row then, and beta NaN takes it to the nodes below
      uint32_t badk = 0;  // bit rho: operand row rho
      {
        const uint64_t w = __ballot((l16 >> 2) == m && !(fabsf(diag_entry(gm, l16)) < __builtin_inff()));
        if (w) {  // uniform
          badk = uint32_t((w | w >> 16 | w >> 32 | w >> 48) & 0xffffu);
          gm = z4;
#pragma unroll
          for (int kb = 0; kb < KB; ++kb) {
            if ((badk >> l16) & 1) {
              ka[kb] = f16x8{0, 0, 0, 0, 0, 0, 0, 0};
              if (DK >= 32 || m < 2) *reinterpret_cast<f16x8*>(KF::piece(buf, kb, l16, m)) = ka[kb];
            }
            gm = mfma_h(ka[kb], ka[kb], gm);
          }
          wave_lds_order();
        }
      }
      if (own) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) s = mfma_h(ka[kb], qf[kb], s);
      }
      if (!own) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
          f16x4 h0, l0, h1 = {0, 0, 0, 0}, l1 = {0, 0, 0, 0}, a1 = {0, 0, 0, 0};
          split4(x[2 * kb], y1, h0, l0);
          const f16x4 a0 = KF::slots(buf, 2 * kb, l16, m);
          if constexpr (NX > 1) {
            split4(x[2 * kb + 1], y1, h1, l1);
            a1 = KF::slots(buf, 2 * kb + 1, l16, m);
          }
          s = mfma_h(cat(a0, a1), cat(l0, l1), s);
          s = mfma_h(cat(a0, a1), cat(h0, h1), s);
        }
      }
      // ---- gates of accumulator rows e = 0 .. 3 (rows without a node: end 0)
      f32x4 bm, al, vs;
      int ie[4];
      RowGate ge[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        ie[e] = index(lst, 4 * e + m);
        ge[e] = s_g[ie[e]];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) asm volatile("" : "+v"(ge[e].be), "+v"(ge[e].al), "+v"(ge[e].vs));  // loaded, not branched around
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const RowGate g = ge[e];
        const bool on = ie[e] <= n && n < g.end;
        bm[e] = on ? ((badk >> (4 * m + e)) & 1 ? __builtin_nanf("") : g.be) : 0.0f;
        al[e] = on ? g.al : 1.0f;
        vs[e] = fabsf(g.vs);
        vmin = fminf(vmin, g.vs);
      }
      // N_ij = beta_i k_i.k_j for i above j, in the 4 x 4 block of step l16 %
      // 4; row il is the block's row i (a chain, or an absent row, beta 0)
      const bool up = (l16 >> 2) < m && (!own || n0 + 4 * (l16 & 3) + m < gl.end);
      const float di = block_inverse(z, up ? finite(gl.be) * diag_entry(gm, l16) : 0.0f, l16, m);
      const f32x4 lr = decays(al, rw, m);
      const f32x4 c = substitute(s, gm, di, bm, l16);
      __builtin_amdgcn_sched_barrier(0);
      // ---- x -= K^T c
      f16x4 h0, l0;
      split4(-c, y1, h0, l0);
#pragma unroll
      for (int t = 0; t < NX; ++t) {
        const f16x4 a = KF::columns(buf, t, l16, m);
        if (own) x[t] = f32x4{(float)qc[t][0], (float)qc[t][1], (float)qc[t][2], (float)qc[t][3]};
        x[t] = mfma_h16(a, l0, x[t]);
        x[t] = mfma_h16(a, h0, x[t]);
      }
      wave_lds_order();
      f32x4 mm;
#pragma unroll
      for (int e = 0; e < 4; ++e) mm[e] = c[e] * lr[e] * vs[e];
      return mm;
    };
    // acc (+)= V^T mm over the chunk, whose v~ rows are in vf.  In fp32: the
    // coefficients of a path differ without bound, and a small one counts in
    // the channels where the rows of the large ones are 0.  As fp16 hi + lo
    // under one scale per node (2 products instead of 4) the call took 506
    // instead of 529 us at 32 x 512 (with the commit), 87 instead of 93 at 16 x
    // 250, and lost what was below 2^-25 of the node's largest.  The rate of
    // the fp32 products is what they cost: 2 or 4 channel tiles in turn took as
    // long.
    auto values = [&](const int16_t* lst, f32x4 mm, bool marked, auto ahead) {
      const int ln = opaque(lane), l16 = ln & 15, m = ln >> 4;
      if (marked) vf.keep_finite();
      vf.store(buf, ln);
      ahead();
      wave_lds_order();
#pragma unroll
      for (int t = 0; t < NV; ++t) {
        const f16x4 a = VF::columns(buf, t, l16, m);
        if (!lst) acc[t] = z4;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[t] = mfma_f((float)a[e], mm[e], acc[t]);
      }
      wave_lds_order();
      if (marked) {
        // values that are not finite reach the nodes whose path holds their
        // row, and no others
#pragma unroll 1
        for (int j = 0; j < kLTile; ++j) {
          const int i = index(lst, j), e = j >> 2;
          const RowGate g = s_g[i];
          const float cj = __shfl(e == 0 ? mm[0] : (e == 1 ? mm[1] : (e == 2 ? mm[2] : mm[3])), l16 + 16 * (j & 3));
          if (i <= n && n < g.end && g.vs < 0.0f) {
            const _Float16* v = Fv + size_t(s_row[i]) * C + 4 * m;
#pragma unroll
            for (int t = 0; t < NV; ++t)
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const float y = (float)v[16 * t + q];
                if (!(fabsf(y) < 65536.0f)) acc[t][q] += cj * y;
              }
          }
        }
      }
    };
    // The first two chunks' values follow both solutions: x and the solver's
    // registers are then not live together with acc (128 registers allow two
    // workgroups per CU).
    auto none = [] {};
    {
      float va = 0.0f, vb = 0.0f;
      const f32x4 ma = solve(nullptr, va, [&] {
        if (near < kLMaxT) load_k(path);
      });
      f32x4 mb = z4;
      if (near < kLMaxT)
        mb = solve(path, vb, [&] { load_v(nullptr); });
      else
        load_v(nullptr);
      values(nullptr, ma, __any(va < 0.0f), [&] {
        if (near < kLMaxT) load_v(path);
      });
      if (near < kLMaxT) values(path, mb, __any(vb < 0.0f), none);
    }
    if (path[0] < kLMaxT && path[0] > 0) {
      // more than 16 ancestors (the 16th is not the root): 16 at a time,
      // found as the nodes before the tile whose subtree reaches past its
      // first node
      const int dep = m_.pdep[bt + s_row[n0]];
      const int np = dep < nval ? dep : nval;  // corrupt metadata: the loop ends all the same
      for (int base = np - 2 * kLTile; base > -kLTile; base -= kLTile) {
        if (lane < kLTile) list[lane] = int16_t(kLMaxT);
        wave_lds_order();
        for (int a = lane; a < n0; a += 64) {
          if (s_g[a].end > n0) {
            const int d = m_.pdep[bt + s_row[a]] - base;
            if (d >= 0 && d < kLTile) list[d] = int16_t(a);
          }
        }
        wave_lds_order();
        load_k(list);
        float vb = 0.0f;
        const f32x4 mb = solve(list, vb, none);
        load_v(list);  // not ahead: acc is live here
        values(list, mb, __any(vb < 0.0f), none);
      }
    }
    // ---- O^T = S0 (r X)^T + acc.  r x enters as fp16 hi + lo: with fp16
    // features the key dims are short, and an x rounded once to 11 bits cost
    // up to 3e-4 of max|o| on 16-dim heads.
    f16x8 xh[KB], xl[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      f16x4 h0, l0, h1 = {0, 0, 0, 0}, l1 = {0, 0, 0, 0};
      split4(x[2 * kb], rw, h0, l0);
      if constexpr (NX > 1) split4(x[2 * kb + 1], rw, h1, l1);
      xh[kb] = cat(h0, h1);
      xl[kb] = cat(l0, l1);
    }
    float* dst = outh + size_t(opaque(slot)) * Hv * DV + 4 * m;
#pragma unroll
    for (int t = 0; t < NV; ++t) {
      f32x4 d = z4;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const f16x8 a = *reinterpret_cast<const f16x8*>(s_plane + (16 * t + l16) * KP + 32 * kb + 8 * m);
        d = mfma_h(a, xl[kb], d);
        d = mfma_h(a, xh[kb], d);
      }
      const float4 si = *reinterpret_cast<const float4*>(s_inv + 16 * t + 4 * m);
      const float4 o = make_float4(fmaf(d[0], si.x, acc[t][0] * p.scale), fmaf(d[1], si.y, acc[t][1] * p.scale),
                                   fmaf(d[2], si.z, acc[t][2] * p.scale), fmaf(d[3], si.w, acc[t][3] * p.scale));
      if (n < T) *reinterpret_cast<float4*>(dst + 16 * t) = n < nval ? o : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
}

// ---------------------------------------------------------------------------
// Launch
// ---------------------------------------------------------------------------
// channels per thread of the feature kernel: 8 for the fp16 workspace, 4
// for the fp32 features
constexpr int kFCHalf = 8, kFCF32 = 4;

// channel blocks of the feature kernel
static int feat_cblocks(const LargeParams& p, int dk, int dv, int cpt) {
  const int nt = feat_vbase(p.Hk, dk, cpt) + p.Hv * dv / cpt;
  return (nt + kFT - 1) / kFT;
}

static dim3 feat_grid(const LargeParams& p, int dk, int dv, int cpt) {
  return dim3(feat_cblocks(p, dk, dv, cpt) * ((p.T + kFP - 1) / kFP) * p.B + (p.ord ? p.B : 0));
}

template <int DK, int DV, typename TIn, bool FUSED>
static int launch_pull(const LargeParams& p, hipStream_t stream) {
  using SM = PullSmem<DK, DV>;
  const int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(&pull_kernel<DK, DV, TIn, FUSED>),
                                    int(SM::total), "verify (T > 128)");
  if (rc != GDN_OK) return rc;
  const int units = p.B * p.Hk, G = p.Hv / p.Hk;
  hipLaunchKernelGGL((pull_kernel<DK, DV, TIn, FUSED>), dim3((units + 7) / 8 * 8 * G), dim3(kLT), SM::total,
                     stream, p);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return set_error(GDN_EHIP, "verify (T > 128) launch: %s", hipGetErrorString(e));
  return GDN_OK;
}

// fused: the conv-state part of the previous step's commit first (the
// features read the conv state after it), the state rows inside the
// pull-back
template <int DK, int DV, typename TIn>
static int launch_large_t(const LargeParams& p, bool fused, hipStream_t stream) {
  constexpr bool kCanFuse = commit_threads(DK, DV) == kLT;
  if (fused) {
    if (!kCanFuse) return set_error(GDN_EUNSUPPORTED, "step (T > 128): dk * dv = %d below 512", DK * DV);
    const int rc = launch_commit_conv(p.cp, DK, DV, std::is_same<TIn, BF16>::value ? GDN_BF16 : GDN_F32, stream);
    if (rc != GDN_OK) return rc;
  }
  hipLaunchKernelGGL((feat_kernel<TIn, DK, DV / kFCHalf, kFCHalf>), feat_grid(p, DK, DV, kFCHalf), dim3(kFT), 0, stream,
                     p, DV, feat_cblocks(p, DK, DV, kFCHalf));
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return set_error(GDN_EHIP, "verify (T > 128) feature launch: %s", hipGetErrorString(e));
  if constexpr (kCanFuse)
    if (fused) return launch_pull<DK, DV, TIn, true>(p, stream);
  return launch_pull<DK, DV, TIn, false>(p, stream);
}

template <int DK, typename TIn>
static int large_dv(const VerifyArgs& a, const LargeParams& p, hipStream_t s) {
  switch (a.dv) {
    case 16: return launch_large_t<DK, 16, TIn>(p, a.fused, s);
    case 32: return launch_large_t<DK, 32, TIn>(p, a.fused, s);
    case 64: return launch_large_t<DK, 64, TIn>(p, a.fused, s);
    case 128: return launch_large_t<DK, 128, TIn>(p, a.fused, s);
  }
  return set_error(GDN_EUNSUPPORTED, "verify: dv=%d unsupported", a.dv);
}

template <typename TIn>
static int large_dk(const VerifyArgs& a, const LargeParams& p, hipStream_t s) {
  switch (a.dk) {
    case 16: return large_dv<16, TIn>(a, p, s);
    case 32: return large_dv<32, TIn>(a, p, s);
    case 64: return large_dv<64, TIn>(a, p, s);
    case 128: return large_dv<128, TIn>(a, p, s);
  }
  return set_error(GDN_EUNSUPPORTED, "verify: dk=%d unsupported", a.dk);
}

// ws: the pull-back workspace (fp16 features, then the v~ scales) or, for
// launch_features, the fp32 feature array
static LargeParams large_params(const VerifyArgs& a, void* ws, void* ord, bool half) {
  LargeParams p;
  p.B = a.B;
  p.T = a.T;
  p.Hk = a.Hk;
  p.Hv = a.Hv;
  p.scale = a.scale;
  p.meta = a.meta;
  p.q = a.q;
  p.k = a.k;
  p.v = a.v;
  p.alpha = a.alpha;
  p.beta = a.beta;
  p.conv_w = a.conv_w;
  p.conv_state = a.conv_state;
  p.S0 = a.S0;
  p.out = a.out;
  p.F = half ? nullptr : static_cast<float*>(ws);
  p.FH = half ? static_cast<_Float16*>(ws) : nullptr;
  p.Vs = half ? reinterpret_cast<float*>(static_cast<unsigned char*>(ws) + fh_bytes(a.B, a.T, a.Hk, a.Hv, a.dk, a.dv))
              : nullptr;
  p.ord = static_cast<int16_t*>(ord);
  p.cp = CommitParams{};
  if (a.fused) {
    p.conv_state = a.conv_state_out;  // the features see the committed conv state
    p.cp.B = a.B;
    p.cp.T = a.T;
    p.cp.Hk = a.Hk;
    p.cp.Hv = a.Hv;
    p.cp.meta = a.pmeta;
    p.cp.accepted = a.paccepted;
    p.cp.q = a.pq;
    p.cp.k = a.pk;
    p.cp.v = a.pv;
    p.cp.alpha = a.palpha;
    p.cp.beta = a.pbeta;
    p.cp.conv_w = a.conv_w;
    p.cp.cs_in = a.conv_state;
    p.cp.cs_out = a.conv_state_out;
    p.cp.S = a.S;
    p.cp.commit_status = a.commit_status;
  }
  return p;
}

static int launch_large(const VerifyArgs& a, void* ws, void* ord, hipStream_t stream) {
  const LargeParams p = large_params(a, ws, ord, true);
  if (a.in_dtype == GDN_BF16) return large_dk<BF16>(a, p, stream);
  return large_dk<float>(a, p, stream);
}

int launch_verify_large(const VerifyArgs& a, void* ws, size_t ws_bytes, hipStream_t stream) {
  if (a.T > kLMaxT) return set_error(GDN_EUNSUPPORTED, "verify: T=%d exceeds %d", a.T, kLMaxT);
  const size_t order = large_order_offset(large_workspace_bytes(a.B, a.T, a.Hk, a.Hv, a.dk, a.dv));
  if (ws_bytes < order + large_order_bytes(a.B, a.T))
    return set_error(GDN_EINVAL, "verify: workspace of %zu bytes is too small", ws_bytes);
  return launch_large(a, ws, static_cast<unsigned char*>(ws) + order, stream);
}

template <typename TIn>
static int launch_features_t(const VerifyArgs& a, const LargeParams& p, hipStream_t stream) {
  switch (a.dk) {
    case 16: hipLaunchKernelGGL((feat_kernel<TIn, 16, 0, kFCF32>), feat_grid(p, 16, a.dv, kFCF32), dim3(kFT), 0, stream,
                                  p, a.dv, feat_cblocks(p, 16, a.dv, kFCF32)); break;
    case 32: hipLaunchKernelGGL((feat_kernel<TIn, 32, 0, kFCF32>), feat_grid(p, 32, a.dv, kFCF32), dim3(kFT), 0, stream,
                                  p, a.dv, feat_cblocks(p, 32, a.dv, kFCF32)); break;
    case 64: hipLaunchKernelGGL((feat_kernel<TIn, 64, 0, kFCF32>), feat_grid(p, 64, a.dv, kFCF32), dim3(kFT), 0, stream,
                                  p, a.dv, feat_cblocks(p, 64, a.dv, kFCF32)); break;
    case 128: hipLaunchKernelGGL((feat_kernel<TIn, 128, 0, kFCF32>), feat_grid(p, 128, a.dv, kFCF32), dim3(kFT), 0, stream,
                                  p, a.dv, feat_cblocks(p, 128, a.dv, kFCF32)); break;
    default: return set_error(GDN_EUNSUPPORTED, "features: dk=%d unsupported", a.dk);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return set_error(GDN_EHIP, "feature launch: %s", hipGetErrorString(e));
  return GDN_OK;
}

int launch_features(const VerifyArgs& a, float* F, hipStream_t stream) {
  if (a.T > kLMaxT) return set_error(GDN_EUNSUPPORTED, "features: T=%d exceeds %d", a.T, kLMaxT);
  const LargeParams p = large_params(a, F, nullptr, false);
  if (a.in_dtype == GDN_BF16) return launch_features_t<BF16>(a, p, stream);
  return launch_features_t<float>(a, p, stream);
}

// ---------------------------------------------------------------------------
// Allocation-free variant: the workspace is a file-scope device array of
// GDN_NOALLOC_SCRATCH_BYTES (every device the library runs on holds one
// copy until the process ends).  In host code `scratch` only names the
// symbol; its device address is looked up once per device with
// hipGetSymbolAddress and only that address is passed to kernels.  Calls
// that overlap on one device share the array and race.  The features are
// written before they are read, so nothing needs clearing.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[GDN_NOALLOC_SCRATCH_BYTES];
// The depth-first orders of the same problems: a node takes at least 100 bytes
// above (one key and one value head of 16), and in here 6, with its tree's
// nodes rounded up to a multiple of 16: most for 129.
constexpr size_t kOrderTrees = size_t(GDN_NOALLOC_SCRATCH_BYTES) / (100 * (kSmallMaxT + 1)) + 1;
static __device__ __align__(256) unsigned char order_scratch[kOrderTrees * 6 * large_order_stride(kSmallMaxT + 1)];

static void* scratch_address(const void* symbol, int* rc) {
  static std::mutex mu;
  static std::map<std::pair<const void*, int>, void*> addr;  // (array, device) -> address of its copy
  *rc = GDN_OK;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) {
    *rc = set_error(GDN_EHIP, "verify_noalloc: hipGetDevice failed");
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(mu);
  auto it = addr.find({symbol, dev});
  if (it != addr.end()) return it->second;
  void* ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, symbol);
  if (e != hipSuccess || ptr == nullptr) {
    *rc = set_error(GDN_EHIP, "verify_noalloc: hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
    return nullptr;
  }
  addr[{symbol, dev}] = ptr;
  return ptr;
}

int launch_verify_noalloc(const VerifyArgs& a, hipStream_t stream) {
  if (a.T <= kSmallMaxT) return launch_verify(a, stream);  // uses no workspace
  const size_t bytes = large_workspace_bytes(a.B, a.T, a.Hk, a.Hv, a.dk, a.dv);
  if (bytes > size_t(GDN_NOALLOC_SCRATCH_BYTES))
    return set_error(GDN_EUNSUPPORTED,
                     "verify_noalloc: B=%d T=%d needs %zu workspace bytes, above the static %zu (call "
                     "gdn_tree_verify, or split the batch)",
                     a.B, a.T, bytes, size_t(GDN_NOALLOC_SCRATCH_BYTES));
  if (large_order_bytes(a.B, a.T) > sizeof(order_scratch))
    return set_error(GDN_EUNSUPPORTED, "verify_noalloc: B=%d T=%d: orders above the static %zu bytes", a.B, a.T,
                     sizeof(order_scratch));
  int rc = GDN_OK;
  void* ws = scratch_address(HIP_SYMBOL(scratch), &rc);
  if (!ws) return rc;
  void* ord = scratch_address(HIP_SYMBOL(order_scratch), &rc);
  if (!ord) return rc;
  if (a.T > kLMaxT) return set_error(GDN_EUNSUPPORTED, "verify: T=%d exceeds %d", a.T, kLMaxT);
  return launch_large(a, ws, ord, stream);
}

// ---------------------------------------------------------------------------
// Workspace of the T > 128 path: one device buffer per (device, stream),
// grown on demand and kept until the process ends.
// ---------------------------------------------------------------------------
void* stream_workspace(size_t bytes, hipStream_t stream, int* rc) {
  static std::mutex mu;
  static std::map<std::pair<int, hipStream_t>, std::pair<void*, size_t>> bufs;
  *rc = GDN_OK;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) {
    *rc = set_error(GDN_EHIP, "workspace: hipGetDevice failed");
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(mu);
  auto& e = bufs[{dev, stream}];
  if (e.second >= bytes) return e.first;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone) {
    *rc = set_error(GDN_EUNSUPPORTED,
                    "workspace: %zu bytes needed while the stream is captured; run the same sizes once "
                    "uncaptured first",
                    bytes);
    return nullptr;
  }
  if (e.first) {  // only this stream used it
    if (hipStreamSynchronize(stream) != hipSuccess || hipFree(e.first) != hipSuccess) {
      *rc = set_error(GDN_EHIP, "workspace: release of %zu bytes failed", e.second);
      return nullptr;
    }
    e.first = nullptr;
    e.second = 0;
  }
  if (hipMalloc(&e.first, bytes) != hipSuccess) {
    e.first = nullptr;
    *rc = set_error(GDN_EHIP, "workspace: hipMalloc of %zu bytes failed", bytes);
    return nullptr;
  }
  e.second = bytes;
  return e.first;
}

}  // namespace gdn
