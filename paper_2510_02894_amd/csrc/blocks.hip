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
//   1. k_block_boxes: the blocks' boxes in ROI order, their largest distances from
//      the ROI's centre, and both of every 16 blocks (a superblock);
//   2. k_block_seed: each superblock finds, per family, the superblock whose
//      bound is largest, in that pair of superblocks the pair of blocks whose
//      bound is largest, and that pair of blocks' exact maximum: a lower bound
//      L of the family's diameter, 0.95 to 1.00 of it on unions of ellipsoids;
//   3. k_block_pairs: superblock pairs, then block pairs, whose bound reaches
//      L go to a list (superblocks by both bounds below, blocks by their boxes);
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

constexpr float kBoundUp = 1.0f + 3.814697265625e-06f;

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
  f[0] = (q[0] + q[1] + q[2]) * kBoundUp;
  f[1] = meet[0] ? (p[0] + q[1] + q[2]) * kBoundUp : -1.0f;
  f[2] = meet[1] ? (q[0] + p[1] + q[2]) * kBoundUp : -1.0f;
  f[3] = meet[2] ? (q[0] + q[1] + p[2]) * kBoundUp : -1.0f;
}

// A second bound, from the distances |p| of a block's vertices from the centre of
// the ROI's box: |p - q|^2 = 2 |p|^2 + 2 |q|^2 - |p + q|^2, and |p + q| is at least
// the gap between one block's box and the other's mirror image.  Where the far
// pairs of a shape lie opposite each other, as on everything round, it follows the
// surface, and the boxes' corners stick out of it: a ball of radius 200 lists
// 43,000 block pairs where boxes alone list 16.5 M (the call 180 us and 7,800), 300
// balls of radii 5 to 40 take 630 us and 4,600, and of 4,096 unions of ellipsoids
// k_block_eval takes 440 us and 710.
struct Mirror {
  float o2[3];  // twice the centre (half voxels)
  float w[3];   // what the soft coordinates' rounding may add to a gap
};

__device__ inline Mirror mirror_of(const RoiMeta& M, const Roi& R, bool soft) {
  Mirror c;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    c.o2[k] = (float)(2 * (M.bb[k] + M.bb[3 + k] + 1));
    c.w[k] = soft ? 9.5367431640625e-07f * (float)(4 * (R.d[k] + 2)) : 0.0f;
  }
  return c;
}

constexpr float kBoundDown = 1.0f - 3.814697265625e-06f;

// ra, rb: the largest |p|^2 of the blocks' vertices, over all axes and without axis 0, 1, 2.
__device__ inline void mirror_bounds(const Box& a, const Box& b, const float* ra, const float* rb, const Metric& m,
                                     const Mirror& c, float* f) {
  float q[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float lo = a.lo[k] - c.o2[k] + b.lo[k], hi = a.hi[k] - c.o2[k] + b.hi[k];
    const float g = fmaxf(fmaxf(lo, -hi) - c.w[k], 0.0f) * m.hs[k], s = m.slack * m.hs[k];
    q[k] = g * g;
    f[k + 1] = s * s;
  }
  f[0] = 2.0f * (ra[0] + rb[0]) * kBoundUp - (q[0] + q[1] + q[2]) * kBoundDown;
  f[1] = (2.0f * (ra[1] + rb[1]) + f[1]) * kBoundUp - (q[1] + q[2]) * kBoundDown;
  f[2] = (2.0f * (ra[2] + rb[2]) + f[2]) * kBoundUp - (q[0] + q[2]) * kBoundDown;
  f[3] = (2.0f * (ra[3] + rb[3]) + f[3]) * kBoundUp - (q[0] + q[1]) * kBoundDown;
}

// The bound of family g alone (g the same for the whole wave).
__device__ inline float far_bound(const Box& a, const Box& b, const Metric& m, int g) {
  float sum = 0.0f;
  bool meet = true;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    float d = fmaxf(a.hi[k] - b.lo[k], b.hi[k] - a.lo[k]);
    if (g == k + 1) {
      meet = fmaxf(a.lo[k] - b.hi[k], b.lo[k] - a.hi[k]) <= m.slack;
      d = fminf(d, m.slack);
    }
    const float x = d * m.hs[k];
    sum += x * x;
  }
  return meet ? sum * kBoundUp : -1.0f;
}

// A group's exact maximum so far in units of 2^(2 ex), rounded down to FP32:
// a bound below this cannot matter.  Less 2^-120, above the rounding of
// squares that fall out of FP32's normal range (planes whose two axes are
// 10^18 times finer than the third); 0 if the maximum left FP64's range.
__device__ inline unsigned long long seen_bits(const GroupRes* g) {
  return __hip_atomic_load(&g->best_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline float bits_bound(unsigned long long b, int ex) {
  const double v = ldexp(__longlong_as_double((long long)b), -2 * ex);
  return v < 1.0e30 ? (float)(v * (1.0 - 1.1920928955078125e-07) - 7.52316384526264e-37) : 0.0f;
}

__device__ inline float seen_max(const GroupRes* g, int ex) { return bits_bound(seen_bits(g), ex); }

// Raises a group's maximum to v unless it is known to be as large: `seen` was
// read earlier, and it is read again before the atomic, since the waves of a
// ROI meet on four addresses (7,000 unconditional atomics took 50 us).  Returns
// whether v is not below the maximum.
__device__ inline bool raise_max(GroupRes* g, double v, unsigned long long seen) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  if (b < seen) return false;
  const unsigned long long now = seen_bits(g);
  return b > now ? b >= atomicMax(&g->best_bits, b) : b == now;
}

// Whether a parameter is a number, by its bits (this file is compiled for
// operands that are: its maxima would drop or keep a NaN as the instruction
// happens to treat one).
__device__ inline bool is_number(double t) {
  return ((unsigned long long)__double_as_longlong(t) & 0x7fffffffffffffffull) <= 0x7ff0000000000000ull;
}

// A staged vertex: position and the plane keys of its three axes.
struct alignas(16) VRow {
  double x[3];
  uint32_t pk[3];
  uint32_t pad_[3];
};

__device__ inline VRow vertex_row(unsigned long long k, double t, const double* s) {
  VRow v;
  key_position(k, t, s, v.x);
  const uint32_t a = (uint32_t)(k >> 60) & 3u;
  v.pk[0] = 2u * ((uint32_t)(k >> 40) & 0xFFFFFu) + (a == 0u);
  v.pk[1] = 2u * ((uint32_t)(k >> 20) & 0xFFFFFu) + (a == 1u);
  v.pk[2] = 2u * ((uint32_t)k & 0xFFFFFu) + (a == 2u);
  return v;
}

// A wave's LDS of a block pair: rows from 0 on are block b's, rows from 32 on
// block a's; and their keys.
struct PairStage {
  VRow row[64];
  unsigned long long key[64];
};

// One vertex per lane, b's rows by lanes 0..31, a's by lanes 32..63, and the box
// of the other block.
struct PairLoad {
  unsigned long long k;
  double t;
  float4 b0, b1;
};

__device__ inline PairLoad load_pair(const BlockBufs& B, int a, int b, int lane) {
  const long long mine = lane < 32 ? b : a, other = lane < 32 ? a : b;
  const long long r = 32ll * mine + (lane & 31);
  PairLoad K;
  K.k = B.key[r];
  K.t = B.t ? B.t[r] : 0.5;
  K.b0 = B.pbox[2 * other];
  K.b1 = B.pbox[2 * other + 1];
  return K;
}

__device__ inline double wave_max_f64(double v) {
  // maxima of squared distances and -1: signed integers of the same order
  const unsigned long long r = lanes_reduce<6>(
      (unsigned long long)__double_as_longlong(v),
      [](unsigned long long x, unsigned long long y) { return (long long)x > (long long)y ? x : y; });
  return __longlong_as_double((long long)r);
}

// The largest squared distance between the staged rows, n_a of block a and n_b
// of b, over all pairs (G = 0) or those on a common plane of axis G - 1 (-1 if
// there is none).  2^sh >= n_a lanes hold a row each, the groups of lanes take
// b's rows in turn.
template <int G>
__device__ inline double staged_max(const PairStage* S, int n_a, int n_b, int sh, int lane) {
  const int i = lane & ((1 << sh) - 1);
  const VRow A = S->row[32 + i];
  double m = -1.0;
  for (int c = lane >> sh; c < n_b; c += 64 >> sh) {
    const double d = dist2_exact(A.x, S->row[c].x);
    m = fmax(m, G == 0 || A.pk[G ? G - 1 : 0] == S->row[c].pk[G ? G - 1 : 0] ? d : -1.0);
  }
  return wave_max_f64(i < n_a ? m : -1.0);
}

// Stages the vertices of a block pair that can take part in a pair at or above
// thr for a family in `mask`: those whose bound to the other block's box reaches
// it (of the 1,024 pairs of a listed block pair a few dozen are left).  A vertex
// that NaN voxels leave without a position takes part in none.  n_a, n_b: their
// numbers; false if there is no pair.
__device__ inline bool stage_rows(const PairLoad& K, const Roi& R, const Metric& met, unsigned int mask,
                                  const float* thr, int lane, PairStage* S, bool keys, int& n_a, int& n_b) {
  const VRow V = vertex_row(K.k, K.t, R.s);
  bool take = false;
  {
    Box v;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      // half voxels: the plane key less the key offset, moved by the soft
      // parameter along the edge and widened by its rounding
      float c = (float)((int)V.pk[k] - 2), w = 0.0f;
      if (met.slack > 0.0f) {
        const bool along = (int)((K.k >> 60) & 3ull) == k;
        c = along ? c - 1.0f + 2.0f * (float)K.t : c;
        w = fabsf(c) * 2.384185791015625e-07f + 2.384185791015625e-07f;
      }
      v.lo[k] = c - w;
      v.hi[k] = c + w;
    }
    float f[4];
    far_bounds(v, box_of(K.b0, K.b1), met, f);
#pragma unroll
    for (int g = 0; g < 4; ++g) take |= (mask >> g & 1u) && f[g] >= thr[g];
    take &= is_number(K.t);
  }
  const unsigned long long em = __ballot(take);
  const unsigned int mb = (unsigned int)em, ma = (unsigned int)(em >> 32);
  if (!ma || !mb) return false;
  n_a = __popc(ma);
  n_b = __popc(mb);
  __builtin_amdgcn_wave_barrier();  // the previous pair's rows have been read
  if (take) {
    const int slot = (lane & 32) + __popc((lane < 32 ? mb : ma) & ((1u << (lane & 31)) - 1u));
    S->row[slot] = V;
    if (keys) S->key[slot] = K.k;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  return true;
}

// The exact maxima over the pairs of two blocks, for the families in `mask`
// (bit 0: all pairs, bits 1..3: pairs on a common plane of axis 0, 1, 2) as far
// as they reach thr (pairs below it may be left out); -1 where no pair was
// visited.  Every lane returns them.
__device__ inline void pair_max(const PairLoad& K, const Roi& R, const Metric& met, unsigned int mask,
                                const float* thr, int lane, PairStage* S, double* m) {
#pragma unroll
  for (int g = 0; g < 4; ++g) m[g] = -1.0;
  int n_a, n_b;
  if (!stage_rows(K, R, met, mask, thr, lane, S, false, n_a, n_b)) return;
  const int sh = n_a > 1 ? 32 - __clz(n_a - 1) : 0;
  if (mask & 1u) m[0] = staged_max<0>(S, n_a, n_b, sh, lane);
  if (mask & 2u) m[1] = staged_max<1>(S, n_a, n_b, sh, lane);
  if (mask & 4u) m[2] = staged_max<2>(S, n_a, n_b, sh, lane);
  if (mask & 8u) m[3] = staged_max<3>(S, n_a, n_b, sh, lane);
}

// The smallest id pair among the block pairs' pairs at the families' maxima:
// with ids32 id_lo * 2^32 + id_hi at once, else PASS 0 takes the smallest
// id_lo and PASS 1 the smallest id_hi that goes with it.
__device__ inline void pair_ties(const BlockBufs& B, int a, int b, const Roi& R, const Metric& met, unsigned int mask,
                                 int lane, PairStage* S, GroupRes* g4, int ids32, int pass) {
  double target[4];
  float thr[4];
  unsigned long long red[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const unsigned long long t = seen_bits(&g4[g]);
    target[g] = __longlong_as_double((long long)t);
    thr[g] = bits_bound(t, met.ex);
    red[g] = ~0ull;
  }
  int n_a, n_b;
  if (!stage_rows(load_pair(B, a, b, lane), R, met, mask, thr, lane, S, true, n_a, n_b)) return;
  const int sh = n_a > 1 ? 32 - __clz(n_a - 1) : 0;
  const int i = lane & ((1 << sh) - 1);
  const VRow A = S->row[32 + i];
  const unsigned long long ida = key_canonical_id(S->key[32 + i], R.d);
  for (int c = lane >> sh; c < n_b; c += 64 >> sh) {
    const VRow& C = S->row[c];
    const double d = dist2_exact(A.x, C.x);
    const bool t0 = (mask & 1u) && d == target[0];
    const bool t1 = (mask & 2u) && d == target[1] && A.pk[0] == C.pk[0];
    const bool t2 = (mask & 4u) && d == target[2] && A.pk[1] == C.pk[1];
    const bool t3 = (mask & 8u) && d == target[3] && A.pk[2] == C.pk[2];
    if (i < n_a && (t0 | t1 | t2 | t3)) {
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
    red[g] = lanes_reduce<6>(red[g], [](unsigned long long x, unsigned long long y) { return x < y ? x : y; });
    if (lane == 0 && red[g] != ~0ull) atomicMin(ids32 || pass == 0 ? &g4[g].id_lo : &g4[g].id_hi, red[g]);
  }
}

// The largest (value, index) key over a wave.
__device__ inline unsigned long long wave_max_u64(unsigned long long v) {
  return lanes_reduce<6>(v, [](unsigned long long x, unsigned long long y) { return x > y ? x : y; });
}

__device__ inline unsigned long long bound_key(float f, int i) {
  return f > 0.0f ? (unsigned long long)__float_as_uint(f) << 32 | (unsigned int)i : 0ull;
}

// The listed block pairs; 0 when the list was too short.
__device__ inline long long listed_pairs(const BlockBufs& B) {
  const long long n = (long long)*B.list_n;
  return n <= B.list_cap ? n : 0;
}

__device__ inline long long staged_superblocks(const BlockBufs& B) {
  return B.totals[T_STAGED] <= B.rows_cap ? B.totals[T_LBLK] / kSuper : 0;
}

}  // namespace

// The boxes and distances from the centre of the ROIs' blocks in ROI order (a
// ROI's blocks are consecutive and start on a superblock), and those of the
// superblocks: eight lanes per block, four vertices each, two superblocks per
// workgroup.  Bound: one read of the staged keys (50 M vertices: 132 us, 3.9 TB/s;
// 23 us for the boxes alone), a chain of three loads where there are few.
constexpr int kBoxBlocks = 32;

__global__ __launch_bounds__(8 * kBoxBlocks) void k_block_boxes(BlockBufs B) {
  __shared__ float s_v[kBoxBlocks][10];  // lo, hi, and the largest |p|^2
  const long long n = staged_superblocks(B) * kSuper;
  const int tid = threadIdx.x, j = tid >> 3, lane = tid & 7;
  for (long long i0 = (long long)blockIdx.x * kBoxBlocks; i0 < n; i0 += (long long)kBoxBlocks * gridDim.x) {
    const long long i = i0 + j;
    const int ph = i < n ? B.lphys[i] : -1;
    const int r = i < n ? B.sbroi[i / kSuper] : 0;
    float rr[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    float4 a = make_float4(3.0e38f, 3.0e38f, 3.0e38f, -3.0e38f), b = make_float4(-3.0e38f, -3.0e38f, 0.0f, 0.0f);
    if (ph >= 0) {
      a = B.pbox[2 * (long long)ph];
      b = B.pbox[2 * (long long)ph + 1];
      const RoiMeta& M = B.meta[r];
      const bool soft = B.t != nullptr;
      const long long row = 32ll * ph + 4 * lane;
      const ulonglong2 ka = *(const ulonglong2*)(B.key + row), kb = *(const ulonglong2*)(B.key + row + 2);
      const unsigned long long key[4] = {ka.x, ka.y, kb.x, kb.y};
      double t[4] = {0.5, 0.5, 0.5, 0.5};
      if (soft) {
        const double2 ta = *(const double2*)(B.t + row), tb = *(const double2*)(B.t + row + 2);
        t[0] = ta.x;
        t[1] = ta.y;
        t[2] = tb.x;
        t[3] = tb.y;
      }
      float o[3], hs[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        o[k] = (float)(M.bb[k] + M.bb[3 + k] + 1);
        hs[k] = M.hs[k];
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float q[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const int u = (int)(key[v] >> (40 - 20 * k) & 0xFFFFFull) - 1;
          const bool along = (int)(key[v] >> 60 & 3ull) == k;
          float c = (float)(2 * u + (along ? 1 : 0)), w = 0.0f;
          if (soft) {
            c = along ? (float)(2 * u) + 2.0f * (float)t[v] : c;
            w = fabsf(c) * 2.384185791015625e-07f + 2.384185791015625e-07f;
          }
          const float x = (fabsf(c - o[k]) + w) * hs[k];
          q[k] = x * x;
        }
        if (is_number(t[v])) {
          rr[0] = fmaxf(rr[0], q[0] + q[1] + q[2]);
          rr[1] = fmaxf(rr[1], q[1] + q[2]);
          rr[2] = fmaxf(rr[2], q[0] + q[2]);
          rr[3] = fmaxf(rr[3], q[0] + q[1]);
        }
      }
    }
#pragma unroll
    for (int f = 0; f < 4; ++f)
      rr[f] = __uint_as_float(
          lanes_reduce<3>(__float_as_uint(rr[f]), [](uint32_t x, uint32_t y) { return x > y ? x : y; }));
    if (lane == 0) {
      if (ph >= 0) {
        B.lbox[2 * i] = a;
        B.lbox[2 * i + 1] = make_float4(b.x, b.y, __int_as_float(ph), 0.0f);
        B.prad[ph] = make_float4(rr[0], rr[1], rr[2], rr[3]);
      }
      const float v[10] = {a.x, a.y, a.z, a.w, b.x, b.y, rr[0], rr[1], rr[2], rr[3]};
#pragma unroll
      for (int k = 0; k < 10; ++k) s_v[j][k] = v[k];
    }
    __syncthreads();
    const long long sb = i0 / kSuper + tid / kSuper;
    if (tid < kBoxBlocks && sb * kSuper < n) {
      float v[10];
#pragma unroll
      for (int k = 0; k < 10; ++k) {
        v[k] = s_v[tid][k];
#pragma unroll
        for (int m = 1; m < kSuper; m <<= 1) {
          const float x = __shfl_xor(v[k], m, 64);
          v[k] = k < 3 ? fminf(v[k], x) : fmaxf(v[k], x);
        }
      }
      if ((tid & (kSuper - 1)) == 0) {
        const int r = B.sbroi[sb];
        const RoiMeta& M = B.meta[r];
        const int left = (M.nblk + kSuper - 1) / kSuper - (int)(sb - M.blk0 / kSuper);
        B.sbox[2 * sb] = make_float4(v[0], v[1], v[2], v[3]);
        B.sbox[2 * sb + 1] = make_float4(v[4], v[5], __int_as_float(r), __int_as_float(left));
        B.srad[sb] = make_float4(v[6], v[7], v[8], v[9]);
      }
    }
    __syncthreads();
  }
}

// A lower bound per family and ROI: a workgroup per superblock A, a wave per
// family: the superblock with the largest bound, there the pair of blocks with
// the largest bound, and its exact maximum (unless a bound shows that it cannot
// raise the family's).
__global__ __launch_bounds__(64 * kWaves, 7) void k_block_seed(BlockBufs B) {
  __shared__ PairStage s_pair[kWaves];
  __shared__ unsigned long long s_best[4][kWaves];
  static_assert(kWaves == 4, "a wave per family");
  const long long nsb = staged_superblocks(B);
  const int lane = threadIdx.x & 63, g = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  // neighbouring superblocks one after another: a ROI's first ones raise its
  // maxima, and most of the others then cannot reach them (4,096 ROIs of 50 M
  // vertices: 304 us; dealt over the workgroups, all of a ROI at once, 518)
  const long long share = (nsb + gridDim.x - 1) / gridDim.x, end = min(nsb, (blockIdx.x + 1) * share);
  for (long long A = blockIdx.x * share; A < end; ++A) {
    const float4 a0 = B.sbox[2 * A], a1 = B.sbox[2 * A + 1];
    const int r = __builtin_amdgcn_readfirstlane(__float_as_int(a1.z));
    const Roi& R = B.rois[r];
    const RoiMeta& M = B.meta[r];
    const Metric m = metric_of(M, B.t != nullptr);
    const Box ba = box_of(a0, a1);
    const long long blk0 = M.blk0, s0 = blk0 / kSuper;
    const int nblk = M.nblk, ns = (nblk + kSuper - 1) / kSuper;
    // The scan costs ns^2 boxes; a large ROI's superblocks are small patches
    // whose neighbours have nearly the same partner, so every second or fourth
    // seeds.  Seed, pairs and eval together (us) with all, every second, fourth and
    // eighth, on unions of twelve ellipsoids: ns 375 32, 28, 28, 27; 490 47, 43, 44,
    // 44; 675 56, 53, 51, 61; 895 95, 91, 103, 108; 1,140 87, 79, 71, 70; 1,520 84, 75,
    // 80, 127; 2,190 108, 100, 91, 91; 3,420 172, 149, 144, 147.  ROIs of ns about 100
    // lose (eval of a batch of 256 soft ROIs 210, 226, 307), so all seed up to 512.
    if (ns > 512 && ((A - s0) & (ns > 1024 ? 3 : 1))) continue;
    // 16 x 16 block pairs later: lane holds block lane % 16 of A
    const int ia = (int)(A - s0) * kSuper + (lane & 15), ic = min(ia, nblk - 1);
    const float4 p0 = B.lbox[2 * (blk0 + ic)], p1 = B.lbox[2 * (blk0 + ic) + 1];
    GroupRes* G = B.gres + 4ll * r + g;
    const unsigned long long seen = seen_bits(G);
    unsigned long long key = 0ull;
    if (ns <= 64) {
      if (lane < ns) {
        const float4 b0 = B.sbox[2 * (s0 + lane)], b1 = B.sbox[2 * (s0 + lane) + 1];
        key = bound_key(far_bound(ba, box_of(b0, b1), m, g), lane);
      }
      key = wave_max_u64(key);
    } else {
      // the waves share the scan, each for all families (four times the reads
      // of a large ROI's superblocks would be bound by the L2)
      unsigned long long k4[4] = {0ull, 0ull, 0ull, 0ull};
      for (int j = threadIdx.x; j < ns; j += 64 * kWaves) {
        const float4 b0 = B.sbox[2 * (s0 + j)], b1 = B.sbox[2 * (s0 + j) + 1];
        float f[4];
        far_bounds(ba, box_of(b0, b1), m, f);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const unsigned long long k = bound_key(f[q], j);
          k4[q] = k > k4[q] ? k : k4[q];
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        k4[q] = wave_max_u64(k4[q]);
        if (lane == 0) s_best[q][g] = k4[q];
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < kWaves; ++q) key = s_best[g][q] > key ? s_best[g][q] : key;
      __syncthreads();
    }
    const float bar = bits_bound(seen, m.ex);
    if (key == 0ull || __uint_as_float((unsigned int)(key >> 32)) < bar) continue;
    // ... and blocks lane / 16 + 4 q of that superblock
    const int jb = (int)(key & 0xffffffffull) * kSuper + (lane >> 4);
    const Box pa = box_of(p0, p1);
    unsigned long long bk = 0ull;
    int phb[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int j = min(jb + 4 * q, nblk - 1);
      const float4 c0 = B.lbox[2 * (blk0 + j)], c1 = B.lbox[2 * (blk0 + j) + 1];
      phb[q] = __float_as_int(c1.z);
      const unsigned long long k =
          ia < nblk && jb + 4 * q < nblk
              ? bound_key(far_bound(pa, box_of(c0, c1), m, g), (lane & 15) << 8 | q << 4 | lane >> 4)
              : 0ull;
      bk = k > bk ? k : bk;
    }
    bk = wave_max_u64(bk);
    if (bk == 0ull || __uint_as_float((unsigned int)(bk >> 32)) < bar) continue;
    const int wi = __builtin_amdgcn_readfirstlane((int)(bk >> 8 & 15ull));
    const int wq = __builtin_amdgcn_readfirstlane((int)(bk >> 4 & 15ull));
    const int wl = __builtin_amdgcn_readfirstlane((int)(bk & 15ull));
    const int pha = __builtin_amdgcn_readlane(__float_as_int(p1.z), wi);
    const int sel = wq == 0 ? phb[0] : (wq == 1 ? phb[1] : (wq == 2 ? phb[2] : phb[3]));
    double mx[4];
    const float thr[4] = {bar, bar, bar, bar};
    pair_max(load_pair(B, pha, __builtin_amdgcn_readlane(sel, 16 * wl), lane), R, m, 1u << g, thr, lane, &s_pair[g],
             mx);
    const double v = g == 0 ? mx[0] : (g == 1 ? mx[1] : (g == 2 ? mx[2] : mx[3]));
    if (lane == 0 && v > 0.0) raise_max(G, v, seen);
  }
}

namespace {

// The bound and the families of a list entry: the FP32 bound rounded up to make
// room for the families' bits.
__device__ inline int entry_word(float bound, unsigned int mask) {
  return (int)(((__float_as_uint(bound) & ~15u) + 16u) | mask);
}
__device__ inline float entry_bound(int w) { return __uint_as_float((unsigned int)w & ~15u); }

// What a wave does with the block pairs it finds: list them, or, when the list
// was too short, evaluate them at once, and later take their ties.
constexpr int kModeList = 0, kModeEval = 1, kModeTies = 2;

constexpr int kStageItems = 320;  // block pairs a wave collects before it appends them with one atomic

// Appends a wave's collected block pairs to the list.  Those past its end are
// dropped: a list that was too short (*list_n counts them all) is not used,
// k_block_again then goes through the block pairs once more.
__device__ inline void append_pairs(const BlockBufs& B, int lane, const int4* buf, int n) {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  unsigned long long got = 0ull;
  if (lane == 0) got = atomicAdd(B.list_n, (unsigned long long)n);
  const long long first = (long long)__shfl(got, 0, 64);
  for (int e = lane; e < n; e += 64)
    if (first + e < B.list_cap) B.list[first + e] = buf[e];
  __builtin_amdgcn_wave_barrier();
}

// Partners of a superblock that a wave tests at once.
constexpr int kPartners = 16;

// Superblock A against every nsplit-th group of four of its ROI's superblocks
// from A on (the far partners of a superblock are neighbours: dealt out in turn
// they are shared by its waves).
template <int MODE>
__device__ inline void enumerate_pairs(const BlockBufs& B, long long A, int split, int nsplit, int lane, int4* buf,
                                       int& n_buf, PairStage* S, int ids32, int pass) {
  const float4 a0 = B.sbox[2 * A], a1 = B.sbox[2 * A + 1];
  const int left = __builtin_amdgcn_readfirstlane(__float_as_int(a1.w));  // the ROI's superblocks from A on
  if (4 * split >= left) return;
  const int r = __builtin_amdgcn_readfirstlane(__float_as_int(a1.z));
  const Roi& R = B.rois[r];
  const RoiMeta& M = B.meta[r];
  const Metric m = metric_of(M, B.t != nullptr);
  GroupRes* G = B.gres + 4ll * r;
  const long long blk0 = M.blk0;
  const int nblk = M.nblk;
  const int ia = (int)(A - blk0 / kSuper);
  unsigned long long tb[4];
  float thr[4];
  auto read_seen = [&]() {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      // (nothing raises them while the list is made: from the caches)
      tb[g] = MODE == kModeList ? G[g].best_bits : seen_bits(&G[g]);
      thr[g] = bits_bound(tb[g], m.ex);
    }
  };
  read_seen();
  const Box ba = box_of(a0, a1);
  // lane holds blocks lane / 16 + 4 q of A, and in turn block lane % 16 of each partner
  Box pa[4];
  int pha[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = min(ia * kSuper + (lane >> 4) + 4 * q, nblk - 1);
    const float4 p0 = B.lbox[2 * (blk0 + i)], p1 = B.lbox[2 * (blk0 + i) + 1];
    pa[q] = box_of(p0, p1);
    pha[q] = __float_as_int(p1.z);
  }
  // partner l of the wave's group of kPartners that starts at superblock A + j0
  auto partner = [&](int j0, int l) { return j0 + 4 * nsplit * (l >> 2) + (l & 3); };
  for (int j0 = 4 * split; j0 < left; j0 += kPartners * nsplit) {
    const int j = partner(j0, lane & (kPartners - 1));
    unsigned int um = 0u;
    if (j < left) {
      const float4 b0 = B.sbox[2 * (A + j)], b1 = B.sbox[2 * (A + j) + 1];
      float f[4];
      far_bounds(ba, box_of(b0, b1), m, f);
#pragma unroll
      for (int g = 0; g < 4; ++g) um |= (unsigned int)(f[g] >= thr[g]) << g;
      if (um) {
        const float4 ra4 = B.srad[A], rb4 = B.srad[A + j];
        const float ra[4] = {ra4.x, ra4.y, ra4.z, ra4.w}, rb[4] = {rb4.x, rb4.y, rb4.z, rb4.w};
        int rr = r;
        asm volatile("" : "+s"(rr));  // (keeps the constants out of the registers of the loop)
        mirror_bounds(ba, box_of(b0, b1), ra, rb, m, mirror_of(B.meta[rr], B.rois[rr], B.t != nullptr), f);
#pragma unroll
        for (int g = 0; g < 4; ++g) um &= ~((unsigned int)(f[g] < thr[g]) << g);
      }
    }
    unsigned int todo = (unsigned int)(__ballot(um != 0u) & ((1ull << kPartners) - 1ull));
    int src = todo ? __ffs((int)todo) - 1 : 0;
    float4 c0, c1;
    {
      const int jc = min((ia + partner(j0, src)) * kSuper + (lane & 15), nblk - 1);
      c0 = B.lbox[2 * (blk0 + jc)];
      c1 = B.lbox[2 * (blk0 + jc) + 1];
    }
    while (todo) {
      todo &= todo - 1u;
      const unsigned int unit = (unsigned int)__builtin_amdgcn_readlane((int)um, src);
      if (MODE == kModeEval) read_seen();  // once per partner: it only rises
      const Box pb = box_of(c0, c1);
      const int phb = __float_as_int(c1.z);
      const int jj = (ia + partner(j0, src)) * kSuper + (lane & 15);
      if (todo) {  // the next partner's boxes, in flight while this one's are tested
        src = __ffs((int)todo) - 1;
        const int jc = min((ia + partner(j0, src)) * kSuper + (lane & 15), nblk - 1);
        c0 = B.lbox[2 * (blk0 + jc)];
        c1 = B.lbox[2 * (blk0 + jc) + 1];
      }
      unsigned int pm[4];
      float ff[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = ia * kSuper + (lane >> 4) + 4 * q;
        float f[4];
        far_bounds(pa[q], pb, m, f);
        pm[q] = 0u;
        ff[q] = 0.0f;
#pragma unroll
        for (int g = 0; g < 4; ++g)
          if ((unit >> g & 1u) && f[g] >= thr[g]) {
            pm[q] |= 1u << g;
            ff[q] = fmaxf(ff[q], f[g]);
          }
        if (i >= nblk || jj >= nblk || jj < i) pm[q] = 0u;
        if (MODE != kModeList && pm[q]) {  // (k_block_eval sees to the list's)
          const float4 ra4 = B.prad[pha[q]], rb4 = B.prad[phb];
          const float ra[4] = {ra4.x, ra4.y, ra4.z, ra4.w}, rb[4] = {rb4.x, rb4.y, rb4.z, rb4.w};
          float h[4];
          mirror_bounds(pa[q], pb, ra, rb, m, mirror_of(M, R, B.t != nullptr), h);
#pragma unroll
          for (int g = 0; g < 4; ++g)
            if (h[g] < thr[g]) pm[q] &= ~(1u << g);
        }
      }
      unsigned long long em[4];
      int k = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        em[q] = __ballot(pm[q] != 0u);
        k += __popcll(em[q]);
      }
      if (k == 0) continue;
      if (MODE == kModeList && n_buf + k > kStageItems) {
        append_pairs(B, lane, buf, n_buf);
        n_buf = 0;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (MODE == kModeList) {
          if (pm[q])  // with the largest bound of its families
            buf[n_buf + __popcll(em[q] & ((1ull << lane) - 1ull))] =
                make_int4(pha[q], phb, r, entry_word(ff[q], pm[q]));
          n_buf += __popcll(em[q]);
          continue;
        }
        for (unsigned long long t = em[q]; t; t &= t - 1ull) {
          const int s = __ffsll((long long)t) - 1;
          const int a = __builtin_amdgcn_readlane(pha[q], s), b = __builtin_amdgcn_readlane(phb, s);
          const unsigned int mask = (unsigned int)__builtin_amdgcn_readlane((int)pm[q], s);
          if (MODE == kModeTies) {
            pair_ties(B, a, b, R, m, mask, lane, S, G, ids32, pass);
          } else {
            double mx[4];
            pair_max(load_pair(B, a, b, lane), R, m, mask, thr, lane, S, mx);
            if (lane == 0)
              for (int g = 0; g < 4; ++g)
                if (mx[g] > 0.0) raise_max(&G[g], mx[g], tb[g]);
          }
        }
      }
    }
  }
}

}  // namespace

// Lists the block pairs whose bound reaches the lower bound of some family:
// a wave per (superblock, 1 / nsplit of its partners).
__global__ __launch_bounds__(64 * kWaves, 4) void k_block_pairs(BlockBufs B, int nsplit) {
  __shared__ int4 s_buf[kWaves][kStageItems];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const long long n = staged_superblocks(B) * nsplit;
  int n_buf = 0;
  int4* buf = s_buf[wid];
  for (long long w = (long long)blockIdx.x * kWaves + wid; w < n; w += (long long)gridDim.x * kWaves)
    enumerate_pairs<kModeList>(B, w / nsplit, (int)(w % nsplit), nsplit, lane, buf, n_buf, nullptr, 0, 0);
  if (n_buf) append_pairs(B, lane, buf, n_buf);
}

// The families in which a listed block pair can hold a maximum by its boxes' and
// by its mirror bounds, a lane per entry.  The maxima may be old ones, from a
// cache (all waves of a large ROI would meet on one line of the L2).
__device__ inline unsigned int entry_families(const BlockBufs& B, const int4& E) {
  unsigned int mask = (unsigned int)E.w & 15u;
  const RoiMeta& M = B.meta[E.z];
  const bool soft = B.t != nullptr;
  const float4 a0 = B.pbox[2 * (long long)E.x], a1 = B.pbox[2 * (long long)E.x + 1], ra4 = B.prad[E.x];
  const float4 b0 = B.pbox[2 * (long long)E.y], b1 = B.pbox[2 * (long long)E.y + 1], rb4 = B.prad[E.y];
  const float ra[4] = {ra4.x, ra4.y, ra4.z, ra4.w}, rb[4] = {rb4.x, rb4.y, rb4.z, rb4.w};
  float f[4];
  mirror_bounds(box_of(a0, a1), box_of(b0, b1), ra, rb, metric_of(M, soft), mirror_of(M, B.rois[E.z], soft), f);
#pragma unroll
  for (int g = 0; g < 4; ++g)
    if (fminf(f[g], entry_bound(E.w)) < bits_bound(B.gres[4ll * E.z + g].best_bits, M.ex)) mask &= ~(1u << g);
  return mask;
}

// The exact maxima of the listed block pairs, a wave each.  An entry keeps the
// families whose maximum it may hold (its own is not below the one seen), and
// its own maximum as the new bound (none if it keeps several).
// A wave takes 16 entries of a long list at a time, four runs of four neighbours,
// the runs dealt to the waves in turn (entries that take long are neighbours),
// and drops those that their bounds rule out, a lane each; of a short one, where a
// wave has one to four in all, its neighbours.  It reads the maxima seen so far
// once for those of one ROI (the waves of a large ROI all read the same line),
// and loads the next pair's vertices while it evaluates one.
__global__ __launch_bounds__(64 * kWaves, 7) void k_block_eval(BlockBufs B) {
  __shared__ PairStage s_pair[kWaves];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const long long n = listed_pairs(B);
  const long long nwaves = (long long)gridDim.x * kWaves;
  const long long wave = (long long)blockIdx.x * kWaves + wid;
  const bool many = n >= 4 * nwaves;
  const int run = (int)max(1ll, min(4ll, (n + nwaves - 1) / nwaves)), runs = many ? 4 : 1;
  for (long long it = 0; (runs * it * nwaves + wave) * run < n; ++it) {
    const long long e = ((runs * it + (lane >> 2)) * nwaves + wave) * run + (lane & 3);
    const bool mine = lane < 4 * runs && (lane & 3) < run && e < n;
    int4 E = make_int4(0, 0, 0, 0);
    unsigned int left = 0u;
    if (mine) {
      E = B.list[e];
      left = many ? entry_families(B, E) : (unsigned int)E.w & 15u;
    }
    unsigned int todo = (unsigned int)__ballot(left != 0u);
    int r = -1, word = 0;
    if (todo) {
      int k = __ffs((int)todo) - 1;
      PairLoad K = load_pair(B, __builtin_amdgcn_readlane(E.x, k), __builtin_amdgcn_readlane(E.y, k), lane);
      unsigned long long sbits = 0ull;
      float seen = 0.0f, thr[4];
      Metric met;
      while (true) {
        const int at = k;
        const int rk = __builtin_amdgcn_readlane(E.z, at), w = __builtin_amdgcn_readlane(E.w, at);
        const unsigned int fam = (unsigned int)__builtin_amdgcn_readlane((int)left, at);
        const PairLoad K0 = K;
        todo &= todo - 1u;
        if (todo) {
          k = __ffs((int)todo) - 1;
          K = load_pair(B, __builtin_amdgcn_readlane(E.x, k), __builtin_amdgcn_readlane(E.y, k), lane);
        }
        GroupRes* G = B.gres + 4ll * rk;
        if (rk != r) {
          r = rk;
          met = metric_of(B.meta[r], B.t != nullptr);
          // lane g < 4 sees to family g; where all entries are taken at once, the maxima as
          // they were before (12,000 waves that read one line past the caches wait 20 us)
          sbits = many ? seen_bits(&G[lane & 3]) : G[lane & 3].best_bits;
          seen = bits_bound(sbits, met.ex);
#pragma unroll
          for (int g = 0; g < 4; ++g) thr[g] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(seen), g));
        }
        const bool on = lane < 4 && (fam >> (lane & 3) & 1u) && !(entry_bound(w) < seen);
        const unsigned int mask = (unsigned int)(__ballot(on) & 15ull);
        if (mask) {
          double mx[4];
          pair_max(K0, B.rois[r], met, mask, thr, lane, &s_pair[wid], mx);
          const double v = (lane & 2) ? ((lane & 1) ? mx[3] : mx[2]) : ((lane & 1) ? mx[1] : mx[0]);
          bool hold = false;
          if (on && v > 0.0) hold = raise_max(&G[lane], v, sbits);
          const unsigned int keep = (unsigned int)(__ballot(hold) & 15ull);
          if (keep) {
            int wk = entry_word(3.0e38f, keep);
            if (!(keep & (keep - 1u)))
              wk = entry_word((float)ldexp(__shfl(v, __ffs((int)keep) - 1, 64), -2 * met.ex), keep);
            if (lane == at) word = wk;
          }
        }
        if (!todo) break;
      }
    }
    if (mine) B.list[e].w = word;
  }
}

// The smallest id pair at each family's maximum, over the entries that may hold it.
__global__ __launch_bounds__(64 * kWaves) void k_block_ties(BlockBufs B, int ids32, int pass) {
  __shared__ PairStage s_pair[kWaves];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const long long n = listed_pairs(B);
  const long long wave = (long long)blockIdx.x * kWaves + wid, nwaves = (long long)gridDim.x * kWaves;
  // 64 entries at a time, a lane each, 4 neighbours to a cache line and the
  // lines dealt to the waves in turn (the entries of a shape with flat faces, all
  // ties, are neighbours); those left are visited by the wave
  for (long long it = 0; 4 * (16 * it * nwaves + wave) < n; ++it) {
    const long long e = 4 * ((16 * it + (lane >> 2)) * nwaves + wave) + (lane & 3);
    int4 E = make_int4(0, 0, 0, 0);
    if (e < n) E = B.list[e];
    unsigned int mask = (unsigned int)E.w & 15u;
    if (mask) {
      const int ex = B.meta[E.z].ex;
      for (int g = 0; g < 4; ++g)
        if ((mask >> g & 1u) && entry_bound(E.w) < seen_max(&B.gres[4ll * E.z + g], ex)) mask &= ~(1u << g);
    }
    unsigned long long todo = __ballot(mask != 0u);
    while (todo) {
      const int s = __ffsll((long long)todo) - 1;
      todo &= todo - 1ull;
      const int r = __builtin_amdgcn_readfirstlane(__shfl(E.z, s, 64));
      pair_ties(B, __builtin_amdgcn_readfirstlane(__shfl(E.x, s, 64)),
                __builtin_amdgcn_readfirstlane(__shfl(E.y, s, 64)), B.rois[r],
                metric_of(B.meta[r], B.t != nullptr), (unsigned int)__builtin_amdgcn_readfirstlane(__shfl((int)mask, s, 64)), lane, &s_pair[wid],
                B.gres + 4ll * r, ids32, pass);
    }
  }
}

// A list that was too short: the block pairs once more, evaluated where they are
// found (kModeEval), and later their ties (kModeTies).
template <int MODE>
__global__ __launch_bounds__(64 * kWaves) void k_block_again(BlockBufs B, int nsplit, int ids32, int pass) {
  __shared__ PairStage s_pair[kWaves];
  if ((long long)*B.list_n <= B.list_cap) return;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const long long n = staged_superblocks(B) * nsplit;
  int n_buf = 0;
  for (long long w = (long long)blockIdx.x * kWaves + wid; w < n; w += (long long)gridDim.x * kWaves)
    enumerate_pairs<MODE>(B, w / nsplit, (int)(w % nsplit), nsplit, lane, nullptr, n_buf, &s_pair[wid], ids32, pass);
}

hipError_t launch_blocks(const BlockBufs& B, bool again, hipStream_t st, hipEvent_t* ev) {
  // grids that fill the chip, or fewer workgroups where the capacity bounds the work
  auto grid = [&](long long work, long long cap) {
    return dim3((unsigned)std::max(1ll, std::min(work, cap * B.cu_count)));
  };
  hipError_t e;
  const long long nsb = B.lblk_cap / kSuper;
  // a few ROIs may have thousands of superblocks each, many have tens
  const int nsplit = B.n_rois <= 16 ? 16 : 2, nsplit_again = B.n_rois <= 16 ? 128 : 16;
  hipLaunchKernelGGL(k_block_boxes, grid((B.lblk_cap + kBoxBlocks - 1) / kBoxBlocks, 16), dim3(8 * kBoxBlocks), 0, st, B);
  if (ev && (e = hipEventRecord(ev[0], st))) return e;
  hipLaunchKernelGGL(k_block_seed, grid(nsb, 16), dim3(64 * kWaves), 0, st, B);
  hipLaunchKernelGGL(k_block_pairs, grid((nsb * nsplit + kWaves - 1) / kWaves, 16), dim3(64 * kWaves), 0, st, B,
                     nsplit);
  if (ev && (e = hipEventRecord(ev[1], st))) return e;
  hipLaunchKernelGGL(k_block_eval, grid((B.list_cap + kWaves - 1) / kWaves, 8), dim3(64 * kWaves), 0, st, B);
  if (again)
    hipLaunchKernelGGL(k_block_again<kModeEval>, grid((nsb * nsplit_again + kWaves - 1) / kWaves, 16),
                       dim3(64 * kWaves), 0, st, B, nsplit_again, 0, 0);
  if (ev && (e = hipEventRecord(ev[2], st))) return e;
  for (int pass = 0; pass < (B.ids32 ? 1 : 2); ++pass) {
    hipLaunchKernelGGL(k_block_ties, grid((B.list_cap + 255) / 256, 4), dim3(64 * kWaves), 0, st, B, B.ids32 ? 1 : 0,
                       pass);
    if (again)
      hipLaunchKernelGGL(k_block_again<kModeTies>, grid((nsb * nsplit_again + kWaves - 1) / kWaves, 16),
                         dim3(64 * kWaves), 0, st, B, nsplit_again, B.ids32 ? 1 : 0, pass);
  }
  return hipGetLastError();
}

}  // namespace s3d
