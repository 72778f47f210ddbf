// blocks.hip -- the maximum vertex distances (paper Sec. 2, "Parallel diameter
// calculation") by exact pruning over blocks of vertices.
//
// The paper visits every vertex pair.  Only the four maxima are needed (all
// pairs, and the pairs on a common plane of each axis), and a set of pairs
// whose distances provably stay below a distance that some pair has can be
// skipped whole.  The mesh pass lists its vertices in blocks of 32 rows; a
// brick's rows follow its row-groups, so a block is a small patch of surface,
// and the largest distance between two blocks' boxes bounds every pair between
// them.  For the planes of axis k the bound drops axis k (the pair shares that
// coordinate) and two blocks whose extents along k do not meet hold no pair.
//
//   1. k_block_boxes: the blocks' boxes in ROI order, and the box of every 16
//      blocks (a superblock);
//   2. k_block_seed: each superblock finds, per family, the superblock whose
//      bound is largest, in that pair of superblocks the pair of blocks whose
//      bound is largest, and that pair of blocks' exact maximum: a lower bound
//      L of the family's diameter, 0.95 to 1.00 of it on unions of ellipsoids;
//   3. k_block_pairs: superblock pairs, then block pairs, whose bound reaches
//      L go to a list;
//   4. k_block_eval: the exact maximum over each listed block pair's 1,024
//      pairs, in FP64 with the oracle's operations and order;
//   5. k_block_ties: among the pairs at the maximum, the smallest id pair.
//
// Every pair at a maximum lies in a listed block pair (its bound is at least
// its distance), so the results are those of all pairs.  On a 97 x 181 x 163
// organ (52,604 vertices, 1.4e9 pairs) step 4 evaluates 1e6 to 7e6 pairs.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "s3d_device.h"
#include "s3d_launch.h"

namespace s3d {

namespace {

enum { T_STAGED = 8, T_LBLK = 9 };  // BlockBufs::totals

constexpr int kWaves = 4;  // waves per workgroup of the pair kernels

// A block's or superblock's box in half voxels (FP32, exact for binary masks,
// rounded outwards for soft ones).
struct Box {
  float lo[3], hi[3];
};

__device__ inline Box box_of(const float4& a, const float4& b) {
  Box x;
  x.lo[0] = a.x;
  x.lo[1] = a.y;
  x.lo[2] = a.z;
  x.hi[0] = a.w;
  x.hi[1] = b.x;
  x.hi[2] = b.y;
  return x;
}

// What the bounds need of a ROI: half its spacing in units of 2^ex, about the
// ROI's extent (so that squares stay in FP32's range for any spacing), and for
// soft masks the slack of a plane (a vertex lies within one half voxel of its
// plane key, so two of one plane lie at most two apart along the plane's axis).
struct Metric {
  float hs[3];
  float slack;  // half voxels: 0 binary, 2 soft
  int ex;
};

__device__ inline Metric metric_of(const RoiMeta& M, bool soft) {
  Metric m;
#pragma unroll
  for (int k = 0; k < 3; ++k) m.hs[k] = M.hs[k];
  m.slack = soft ? 2.0f : 0.0f;
  m.ex = M.ex;
  return m;
}

// Upper bounds f[0..3] on the squared distance of a vertex in a and one in b:
// over all pairs, and over the pairs on a common plane of axis 0, 1, 2 (-1
// where there is none).  Raised by 2^-18, above the FP32 rounding of the
// spacing, the products and the sums (a few 2^-24).
__device__ inline void far_bounds(const Box& a, const Box& b, const Metric& m, float* f) {
  float q[3], p[3];
  bool meet[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float d = fmaxf(a.hi[k] - b.lo[k], b.hi[k] - a.lo[k]);
    meet[k] = fmaxf(a.lo[k] - b.hi[k], b.lo[k] - a.hi[k]) <= m.slack;
    const float x = d * m.hs[k], y = fminf(d, m.slack) * m.hs[k];
    q[k] = x * x;
    p[k] = y * y;
  }
  constexpr float up = 1.0f + 3.814697265625e-06f;
  f[0] = (q[0] + q[1] + q[2]) * up;
  f[1] = meet[0] ? (p[0] + q[1] + q[2]) * up : -1.0f;
  f[2] = meet[1] ? (q[0] + p[1] + q[2]) * up : -1.0f;
  f[3] = meet[2] ? (q[0] + q[1] + p[2]) * up : -1.0f;
}

// A group's exact maximum so far in units of 2^(2 ex), rounded down to FP32:
// a bound below this cannot matter.  Less 2^-120, above the rounding of
// squares that fall out of FP32's normal range (planes whose two axes are
// 10^18 times finer than the third); 0 if the maximum left FP64's range.
__device__ inline float seen_max(const GroupRes* g, int ex) {
  const unsigned long long b = __hip_atomic_load(&g->best_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const double v = ldexp(__longlong_as_double((long long)b), -2 * ex);
  return v < 1.0e30 ? (float)(v * (1.0 - 1.1920928955078125e-07) - 7.52316384526264e-37) : 0.0f;
}

__device__ inline void raise_max(GroupRes* g, double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  if (b > __hip_atomic_load(&g->best_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(&g->best_bits, b);
}

// A staged vertex: position, and its three plane keys in 21-bit fields.
struct VRow {
  double x[3];
  unsigned long long code;
};

constexpr unsigned long long kField = (1ull << 21) - 1ull;

__device__ inline VRow vertex_row(unsigned long long k, double t, const double* s) {
  VRow v;
  key_position(k, t, s, v.x);
  const unsigned long long a = k >> 60 & 3ull;
  const unsigned long long p0 = 2ull * (k >> 40 & 0xFFFFF) + (a == 0), p1 = 2ull * (k >> 20 & 0xFFFFF) + (a == 1),
                           p2 = 2ull * (k & 0xFFFFF) + (a == 2);
  v.code = p0 | p1 << 21 | p2 << 42;
  return v;
}

struct VertexList {
  const unsigned long long* key;
  const double* t;  // null for binary masks
};

// A wave's LDS of a block pair: block b's rows, read by all lanes of a half
// wave at once (broadcast), and their keys.
struct PairStage {
  VRow row[32];
  unsigned long long key[32];
};

// Lane l holds row l % 32 of block a; the half waves take 16 rows of b each.
__device__ inline VRow stage_pair(const VertexList& L, int a, int b, const double* s, int lane, PairStage* S,
                                  unsigned long long* key_a) {
  const long long ra = 32ll * a + (lane & 31), rb = 32ll * b + (lane & 31);
  const unsigned long long ka = L.key[ra], kb = L.key[rb];
  const double ta = L.t ? L.t[ra] : 0.5, tb = L.t ? L.t[rb] : 0.5;
  __builtin_amdgcn_wave_barrier();  // the previous pair's rows have been read
  if (lane < 32) {
    S->row[lane] = vertex_row(kb, tb, s);
    S->key[lane] = kb;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  *key_a = ka;
  return vertex_row(ka, ta, s);
}

__device__ inline double wave_max_f64(double v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v = fmax(v, __shfl_xor(v, m, 64));
  return v;
}

// The exact maxima over the pairs of two blocks, for the families in `mask`
// (bit 0: all pairs, bits 1..3: pairs on a common plane of axis 0, 1, 2);
// -1 where there is no pair.  Every lane returns them.
__device__ inline void pair_max(const VertexList& L, int a, int b, const Roi& R, unsigned int mask, int lane,
                                PairStage* S, double* m) {
  unsigned long long ka;
  const VRow A = stage_pair(L, a, b, R.s, lane, S, &ka);
#pragma unroll
  for (int g = 0; g < 4; ++g) m[g] = -1.0;
  const VRow* col = S->row + (lane & 32 ? 16 : 0);
  if (mask == 1u) {
#pragma unroll 4
    for (int c = 0; c < 16; ++c) m[0] = fmax(m[0], dist2_exact(A.x, col[c].x));
  } else {
#pragma unroll 2
    for (int c = 0; c < 16; ++c) {
      const double d = dist2_exact(A.x, col[c].x);
      const unsigned long long x = A.code ^ col[c].code;
      m[0] = fmax(m[0], d);
      m[1] = fmax(m[1], (x & kField) == 0ull ? d : -1.0);
      m[2] = fmax(m[2], (x & kField << 21) == 0ull ? d : -1.0);
      m[3] = fmax(m[3], (x & kField << 42) == 0ull ? d : -1.0);
    }
  }
#pragma unroll
  for (int g = 0; g < 4; ++g)
    if (mask >> g & 1u) m[g] = wave_max_f64(m[g]);
}

// The smallest id pair among the block pairs' pairs at the families' maxima:
// with ids32 id_lo * 2^32 + id_hi at once, else PASS 0 takes the smallest
// id_lo and PASS 1 the smallest id_hi that goes with it.
__device__ inline void pair_ties(const VertexList& L, int a, int b, const Roi& R, unsigned int mask, int lane,
                                 PairStage* S, GroupRes* g4, int ids32, int pass) {
  unsigned long long ka;
  const VRow A = stage_pair(L, a, b, R.s, lane, S, &ka);
  const unsigned long long ida = key_canonical_id(ka, R.d);
  double target[4];
  unsigned long long red[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    target[g] = __longlong_as_double((long long)g4[g].best_bits);
    red[g] = ~0ull;
  }
  const int c0 = lane & 32 ? 16 : 0;
  for (int c = c0; c < c0 + 16; ++c) {
    const VRow& B = S->row[c];
    const double d = dist2_exact(A.x, B.x);
    const unsigned long long x = A.code ^ B.code;
    const bool t0 = (mask & 1u) && d == target[0];
    const bool t1 = (mask & 2u) && d == target[1] && (x & kField) == 0ull;
    const bool t2 = (mask & 4u) && d == target[2] && (x & kField << 21) == 0ull;
    const bool t3 = (mask & 8u) && d == target[3] && (x & kField << 42) == 0ull;
    if (t0 | t1 | t2 | t3) {
      const unsigned long long idb = key_canonical_id(S->key[c], R.d);
      const unsigned long long lo = min(ida, idb), hi = max(ida, idb);
      const bool hit[4] = {t0, t1, t2, t3};
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        if (!hit[g] || ida == idb) continue;
        if (ids32)
          red[g] = min(red[g], lo << 32 | hi);
        else if (pass == 0)
          red[g] = min(red[g], lo);
        else if (lo == g4[g].id_lo)
          red[g] = min(red[g], hi);
      }
    }
  }
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    if (!(mask >> g & 1u)) continue;
    for (int k = 32; k >= 1; k >>= 1) red[g] = min(red[g], (unsigned long long)__shfl_xor(red[g], k, 64));
    if (lane == 0 && red[g] != ~0ull) atomicMin(ids32 || pass == 0 ? &g4[g].id_lo : &g4[g].id_hi, red[g]);
  }
}

// The largest (value, index) key over a wave.
__device__ inline unsigned long long wave_max_u64(unsigned long long v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    const unsigned long long o = __shfl_xor(v, m, 64);
    v = o > v ? o : v;
  }
  return v;
}

__device__ inline unsigned long long bound_key(float f, int i) {
  return f > 0.0f ? (unsigned long long)__float_as_uint(f) << 32 | (unsigned int)i : 0ull;
}

__device__ inline long long staged_superblocks(const BlockBufs& B) {
  return B.totals[T_STAGED] <= B.rows_cap ? B.totals[T_LBLK] / kSuper : 0;
}

}  // namespace

// The boxes of the ROIs' blocks in ROI order (a ROI's blocks are consecutive
// and start on a superblock) and of the superblocks: a thread per block, 16
// neighbouring lanes per superblock.
__global__ __launch_bounds__(256) void k_block_boxes(BlockBufs B) {
  const long long n = staged_superblocks(B) * kSuper;
  const int lane = threadIdx.x & 63;
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += 256ll * gridDim.x) {
    const int ph = B.lphys[i];
    float lo[3] = {3.0e38f, 3.0e38f, 3.0e38f}, hi[3] = {-3.0e38f, -3.0e38f, -3.0e38f};
    if (ph >= 0) {
      const float4 a = B.pbox[2 * (long long)ph], b = B.pbox[2 * (long long)ph + 1];
      B.lbox[2 * i] = a;
      B.lbox[2 * i + 1] = make_float4(b.x, b.y, __int_as_float(ph), 0.0f);
      lo[0] = a.x;
      lo[1] = a.y;
      lo[2] = a.z;
      hi[0] = a.w;
      hi[1] = b.x;
      hi[2] = b.y;
    }
#pragma unroll
    for (int m = 1; m < kSuper; m <<= 1)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        lo[k] = fminf(lo[k], __shfl_xor(lo[k], m, 64));
        hi[k] = fmaxf(hi[k], __shfl_xor(hi[k], m, 64));
      }
    if ((lane & (kSuper - 1)) == 0) {
      const long long s = i / kSuper;
      B.sbox[2 * s] = make_float4(lo[0], lo[1], lo[2], hi[0]);
      B.sbox[2 * s + 1] = make_float4(hi[1], hi[2], __int_as_float(B.sbroi[s]), 0.0f);
    }
  }
}

// A lower bound per family and ROI: a workgroup per superblock A.  Its waves
// share the scan for the superblock with the largest bound per family; wave g
// then takes family g: the pair of blocks with the largest bound, and its
// exact maximum (unless the bound shows that it cannot raise the family's).
__global__ __launch_bounds__(64 * kWaves) void k_block_seed(BlockBufs B) {
  __shared__ unsigned long long s_best[4];
  __shared__ PairStage s_pair[kWaves];
  const long long nsb = staged_superblocks(B);
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const VertexList L{B.key, B.t};
  for (long long A = blockIdx.x; A < nsb; A += gridDim.x) {
    const float4 a0 = B.sbox[2 * A], a1 = B.sbox[2 * A + 1];
    const int r = __builtin_amdgcn_readfirstlane(__float_as_int(a1.z));
    const Roi& R = B.rois[r];
    const RoiMeta& M = B.meta[r];
    const Metric m = metric_of(M, B.t != nullptr);
    const Box ba = box_of(a0, a1);
    const long long s0 = M.blk0 / kSuper;
    const int ns = (M.nblk + kSuper - 1) / kSuper;
    unsigned long long key[4] = {0ull, 0ull, 0ull, 0ull};
    for (int j = tid; j < ns; j += 64 * kWaves) {
      const float4 b0 = B.sbox[2 * (s0 + j)], b1 = B.sbox[2 * (s0 + j) + 1];
      float f[4];
      far_bounds(ba, box_of(b0, b1), m, f);
#pragma unroll
      for (int g = 0; g < 4; ++g) key[g] = max(key[g], bound_key(f[g], j));
    }
    __syncthreads();
    if (tid < 4) s_best[tid] = 0ull;
    __syncthreads();
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const unsigned long long k = wave_max_u64(key[g]);
      if (lane == 0 && k) atomicMax(&s_best[g], k);
    }
    __syncthreads();
    const int g = wid;
    GroupRes* G = B.gres + 4ll * r + g;
    const unsigned long long sk = s_best[g];
    if (sk == 0ull) continue;
    if (__uint_as_float((unsigned int)(sk >> 32)) < seen_max(G, m.ex)) continue;
    // 16 x 16 block pairs: lane holds block lane % 16 of A, and blocks lane / 16 + 4 q of B
    const int ia = (int)(A - s0) * kSuper + (lane & 15);
    const int jb = (int)(sk & 0xffffffffull) * kSuper + (lane >> 4);
    unsigned long long bk = 0ull;
    if (ia < M.nblk) {
      const float4 p0 = B.lbox[2 * (M.blk0 + ia)], p1 = B.lbox[2 * (M.blk0 + ia) + 1];
      const Box pa = box_of(p0, p1);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = min(jb + 4 * q, M.nblk - 1);
        const float4 c0 = B.lbox[2 * (M.blk0 + j)], c1 = B.lbox[2 * (M.blk0 + j) + 1];
        float f[4];
        far_bounds(pa, box_of(c0, c1), m, f);
        const float fg = g == 0 ? f[0] : (g == 1 ? f[1] : (g == 2 ? f[2] : f[3]));
        bk = max(bk, bound_key(fg, (lane & 15) << 8 | (j & (kSuper - 1))));
      }
    }
    bk = wave_max_u64(bk);
    if (bk == 0ull || __uint_as_float((unsigned int)(bk >> 32)) < seen_max(G, m.ex)) continue;
    const long long la = M.blk0 + (A - s0) * kSuper + (int)(bk >> 8 & 15ull);
    const long long lb = M.blk0 + (long long)(sk & 0xffffffffull) * kSuper + (int)(bk & 15ull);
    double mx[4];
    pair_max(L, __builtin_amdgcn_readfirstlane(B.lphys[la]), __builtin_amdgcn_readfirstlane(B.lphys[lb]), R, 1u << g,
             lane, &s_pair[wid], mx);
    const double v = g == 0 ? mx[0] : (g == 1 ? mx[1] : (g == 2 ? mx[2] : mx[3]));
    if (lane == 0 && v > 0.0) raise_max(G, v);
  }
}

namespace {

// What a wave does with the block pairs of k_block_pairs' enumeration: list
// them (or, past the list's end, evaluate them at once), or, in the pass for
// the ties of a call whose list was too short, take their ties.
constexpr int kModeList = 0, kModeTies = 1;

constexpr int kStageItems = 320;  // block pairs a wave collects before it appends them with one atomic

// Appends a wave's collected block pairs to the list; those past its end are
// evaluated here.
__device__ inline void append_pairs(const BlockBufs& B, int lane, const int4* buf, int n, PairStage* S) {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  unsigned long long got = 0ull;
  if (lane == 0) got = atomicAdd(B.list_n, (unsigned long long)n);
  const long long first = (long long)__shfl(got, 0, 64);
  for (int e = lane; e < n; e += 64)
    if (first + e < B.list_cap) B.list[first + e] = buf[e];
  const VertexList L{B.key, B.t};
  for (int e = (int)max(0ll, min((long long)n, B.list_cap - first)); e < n; ++e) {
    const int4 E = buf[e];
    double mx[4];
    const unsigned int mask = (unsigned int)E.w & 15u;
    pair_max(L, E.x, E.y, B.rois[E.z], mask, lane, S, mx);
    if (lane == 0)
      for (int g = 0; g < 4; ++g)
        if ((mask >> g & 1u) && mx[g] > 0.0) raise_max(&B.gres[4ll * E.z + g], mx[g]);
  }
  __builtin_amdgcn_wave_barrier();
}

// Superblock A of ROI r against the superblocks A + 64 (split + nsplit i) + lane.
template <int MODE>
__device__ inline void enumerate_pairs(const BlockBufs& B, long long A, int split, int nsplit, int lane, int4* buf,
                                       int& n_buf, PairStage* S, int ids32, int pass) {
  const float4 a0 = B.sbox[2 * A], a1 = B.sbox[2 * A + 1];
  const int r = __builtin_amdgcn_readfirstlane(__float_as_int(a1.z));
  const Roi& R = B.rois[r];
  const RoiMeta& M = B.meta[r];
  const Metric m = metric_of(M, B.t != nullptr);
  const VertexList L{B.key, B.t};
  GroupRes* G = B.gres + 4ll * r;
  const long long blk0 = M.blk0;
  const int nblk = M.nblk;
  const long long s0 = blk0 / kSuper;
  const int ns = (nblk + kSuper - 1) / kSuper, ia = (int)(A - s0);
  if (ia + 64 * split >= ns) return;
  float thr[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) thr[g] = seen_max(&G[g], m.ex);
  const Box ba = box_of(a0, a1);
  // lane holds block lane % 16 of A
  const int i = ia * kSuper + (lane & 15);
  const int ic = min(i, nblk - 1);
  const float4 p0 = B.lbox[2 * (blk0 + ic)], p1 = B.lbox[2 * (blk0 + ic) + 1];
  const Box pa = box_of(p0, p1);
  const int pha = __float_as_int(p1.z);
  for (int j0 = ia + 64 * split; j0 < ns; j0 += 64 * nsplit) {
    const int j = j0 + lane;
    unsigned int um = 0u;
    if (j < ns) {
      const float4 b0 = B.sbox[2 * (s0 + j)], b1 = B.sbox[2 * (s0 + j) + 1];
      float f[4];
      far_bounds(ba, box_of(b0, b1), m, f);
#pragma unroll
      for (int g = 0; g < 4; ++g) um |= (unsigned int)(f[g] >= thr[g]) << g;
    }
    unsigned long long todo = __ballot(um != 0u);
    while (todo) {
      const int src = __ffsll((long long)todo) - 1;
      todo &= todo - 1ull;
      const int ju = j0 + src;
      const unsigned int unit = (unsigned int)__shfl((int)um, src, 64);
      unsigned int pm[4];
      float ff[4];
      int phb[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int jj = ju * kSuper + (lane >> 4) + 4 * q;
        const int jc = min(jj, nblk - 1);
        const float4 c0 = B.lbox[2 * (blk0 + jc)], c1 = B.lbox[2 * (blk0 + jc) + 1];
        float f[4];
        far_bounds(pa, box_of(c0, c1), m, f);
        pm[q] = 0u;
        ff[q] = 0.0f;
        phb[q] = __float_as_int(c1.z);
        if (i < nblk && jj < nblk && jj >= i)
#pragma unroll
          for (int g = 0; g < 4; ++g)
            if ((unit >> g & 1u) && f[g] >= thr[g]) {
              pm[q] |= 1u << g;
              ff[q] = fmaxf(ff[q], f[g]);
            }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const unsigned long long em = __ballot(pm[q] != 0u);
        if (!em) continue;
        const int k = __popcll(em);
        if (MODE == kModeList) {
          if (n_buf + k > kStageItems) {
            // append the collected pairs with one atomic
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            append_pairs(B, lane, buf, n_buf, S);
            n_buf = 0;
          }
          if (pm[q]) {
            // the largest bound of the listed families, rounded up to make room for their bits
            const unsigned int fb = (__float_as_uint(ff[q]) & ~15u) + 16u;
            buf[n_buf + __popcll(em & ((1ull << lane) - 1ull))] = make_int4(pha, phb[q], r, (int)(fb | pm[q]));
          }
          n_buf += k;
        } else {
          unsigned long long t = em;
          while (t) {
            const int s = __ffsll((long long)t) - 1;
            t &= t - 1ull;
            pair_ties(L, __shfl(pha, s, 64), __shfl(phb[q], s, 64), R, (unsigned int)__shfl((int)pm[q], s, 64), lane,
                      S, G, ids32, pass);
          }
        }
      }
    }
  }
}

}  // namespace

// Lists the block pairs whose bound reaches the lower bound of some family:
// a wave per (superblock, 1 / nsplit of its partners).
__global__ __launch_bounds__(64 * kWaves) void k_block_pairs(BlockBufs B, int nsplit) {
  __shared__ int4 s_buf[kWaves][kStageItems];
  __shared__ PairStage s_pair[kWaves];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const long long n = staged_superblocks(B) * nsplit;
  int n_buf = 0;
  int4* buf = s_buf[wid];
  for (long long w = (long long)blockIdx.x * kWaves + wid; w < n; w += (long long)gridDim.x * kWaves)
    enumerate_pairs<kModeList>(B, w / nsplit, (int)(w % nsplit), nsplit, lane, buf, n_buf, &s_pair[wid], 0, 0);
  if (n_buf) append_pairs(B, lane, buf, n_buf, &s_pair[wid]);
}

// The exact maxima of the listed block pairs, a wave each.  An entry keeps the
// families whose maximum it may hold (its own is not below the one seen).
__global__ __launch_bounds__(64 * kWaves) void k_block_eval(BlockBufs B) {
  __shared__ PairStage s_pair[kWaves];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const VertexList L{B.key, B.t};
  const long long n = min((long long)*B.list_n, B.list_cap);
  for (long long e = (long long)blockIdx.x * kWaves + wid; e < n; e += (long long)gridDim.x * kWaves) {
    const int4 E = B.list[e];
    const int r = __builtin_amdgcn_readfirstlane(E.z);
    GroupRes* G = B.gres + 4ll * r;
    unsigned int mask = (unsigned int)E.w & 15u;
    const float f = __uint_as_float((unsigned int)E.w & ~15u);
    const int ex = B.meta[r].ex;
#pragma unroll
    for (int g = 0; g < 4; ++g)
      if (f < seen_max(&G[g], ex)) mask &= ~(1u << g);
    mask = (unsigned int)__builtin_amdgcn_readfirstlane((int)mask);
    unsigned int keep = 0u;
    if (mask) {
      double mx[4];
      pair_max(L, __builtin_amdgcn_readfirstlane(E.x), __builtin_amdgcn_readfirstlane(E.y), B.rois[r], mask, lane,
               &s_pair[wid], mx);
      if (lane < 4) {
        const double v = lane == 0 ? mx[0] : (lane == 1 ? mx[1] : (lane == 2 ? mx[2] : mx[3]));
        if ((mask >> lane & 1u) && v > 0.0) {
          const unsigned long long b = (unsigned long long)__double_as_longlong(v);
          unsigned long long seen = __hip_atomic_load(&G[lane].best_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (b > seen) seen = atomicMax(&G[lane].best_bits, b);
          keep = b >= seen ? 1u << lane : 0u;
        }
      }
      keep |= __shfl_xor(keep, 1, 64);
      keep |= __shfl_xor(keep, 2, 64);
    }
    if (lane == 0) B.list[e].w = (int)keep;
  }
}

// The smallest id pair at each family's maximum, over the entries that may
// hold it; a call whose list was too short enumerates its block pairs again.
__global__ __launch_bounds__(64 * kWaves) void k_block_ties(BlockBufs B, int nsplit, int ids32, int pass) {
  __shared__ PairStage s_pair[kWaves];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const VertexList L{B.key, B.t};
  const long long n = (long long)*B.list_n;
  const long long wave = (long long)blockIdx.x * kWaves + wid, nwaves = (long long)gridDim.x * kWaves;
  if (n > B.list_cap) {
    int n_buf = 0;
    const long long nu = staged_superblocks(B) * nsplit;
    for (long long w = wave; w < nu; w += nwaves)
      enumerate_pairs<kModeTies>(B, w / nsplit, (int)(w % nsplit), nsplit, lane, nullptr, n_buf, &s_pair[wid], ids32,
                                 pass);
    return;
  }
  // 64 entries at a time, a lane each; the few that are left are visited by the wave
  for (long long e0 = wave * 64; e0 < n; e0 += nwaves * 64) {
    const long long e = e0 + lane;
    int4 E = make_int4(0, 0, 0, 0);
    if (e < n) E = B.list[e];
    unsigned int mask = (unsigned int)E.w & 15u;
    unsigned long long todo = __ballot(mask != 0u);
    while (todo) {
      const int s = __ffsll((long long)todo) - 1;
      todo &= todo - 1ull;
      const int r = __builtin_amdgcn_readfirstlane(__shfl(E.z, s, 64));
      pair_ties(L, __builtin_amdgcn_readfirstlane(__shfl(E.x, s, 64)),
                __builtin_amdgcn_readfirstlane(__shfl(E.y, s, 64)), B.rois[r],
                (unsigned int)__builtin_amdgcn_readfirstlane(__shfl((int)mask, s, 64)), lane, &s_pair[wid],
                B.gres + 4ll * r, ids32, pass);
    }
  }
}

hipError_t launch_blocks(const BlockBufs& B, hipStream_t st, hipEvent_t* ev) {
  // grids that fill the chip, or fewer workgroups where the capacity bounds the work
  auto grid = [&](long long work, long long cap) {
    return dim3((unsigned)std::max(1ll, std::min(work, cap * B.cu_count)));
  };
  hipError_t e;
  const long long nsb = B.lblk_cap / kSuper;
  // one ROI: many partners per superblock, split over waves; a batch has superblocks enough
  const int nsplit = B.n_rois == 1 ? 8 : 2;
  hipLaunchKernelGGL(k_block_boxes, grid((B.lblk_cap + 255) / 256, 8), dim3(256), 0, st, B);
  if (ev && (e = hipEventRecord(ev[0], st))) return e;
  hipLaunchKernelGGL(k_block_seed, grid(nsb, 16), dim3(64 * kWaves), 0, st, B);
  hipLaunchKernelGGL(k_block_pairs, grid((nsb * nsplit + kWaves - 1) / kWaves, 8), dim3(64 * kWaves), 0, st, B, nsplit);
  if (ev && (e = hipEventRecord(ev[1], st))) return e;
  hipLaunchKernelGGL(k_block_eval, grid((B.list_cap + kWaves - 1) / kWaves, 8), dim3(64 * kWaves), 0, st, B);
  if (ev && (e = hipEventRecord(ev[2], st))) return e;
  for (int pass = 0; pass < (B.ids32 ? 1 : 2); ++pass)
    hipLaunchKernelGGL(k_block_ties, grid((B.list_cap + 255) / 256, 4), dim3(64 * kWaves), 0, st, B, nsplit,
                       B.ids32 ? 1 : 0, pass);
  return hipGetLastError();
}

}  // namespace s3d
