// mesh.hip -- the marching-cubes mesh pass (paper Sec. 2, "Marching cubes
// fused parallel kernels"): cube classification, vertex counting and
// emission, surface area and signed volume.
//
// A workgroup handles a brick: 256 row-groups (32 consecutive cubes along
// axis 2 of one cube row) times up to kTZ cube planes.  It first stages every
// voxel row-group the brick touches in LDS as 32-bit masks (all loads issued
// at once; each mask byte or float becomes one bit once), then each thread
// classifies its 32 cubes of every plane pair from LDS: crossing edges and
// active cubes come from bitwise operations on eight 32-bit corner masks, and
// only active cubes (a few percent) touch the case tables.
//
// Area and volume (binary masks): vertices sit at edge midpoints, so each
// case's area is a fixed number for the call's spacing and its volume term is
// an integer in units of s0*s1*s2/48 (see gen_mc_table.py).  The binary pass
// therefore accumulates the volume exactly in int64 and the area as FP64
// sums in a fixed order.  Soft masks evaluate every triangle in FP64.
//
// Inside-voxel moments (the principal-axis members of the Shape class, asked
// for per call): every voxel is the far corner (1, 1, 1) of exactly one cube,
// so the thread that owns that cube counts it, from the voxel-row word it
// already holds.  A word's count, sum of bit positions and sum of squared bit
// positions come from popcounts of the word under fixed bit patterns; the
// thread, brick and ROI sums are integers, so the second moments are exact
// and independent of the order of the work.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "../../include/shape3d.h"
#define MC_TABLE_QUAL __constant__ const
#include "mc_table.h"
#include "s3d_device.h"
#include "s3d_launch.h"

namespace s3d {

// ---------------------------------------------------------------------------
// Voxel bytes to inside bits, four at a time.

// Active cubes per chunk of a brick's dense enumeration (4 per thread).
constexpr int kMeshItems = 1024;
static_assert(kMeshItems == 4 * kBrickThreads, "the slot scan gives each thread 4 slots");

// Position of the r-th set bit (r = 0 for the lowest) of w; r < popc(w).
__device__ inline int nth_set_bit(uint32_t w, int r) {
  int pos = 0;
#pragma unroll
  for (int h = 16; h >= 1; h >>= 1) {
    const int up = pos | h;
    pos = __popc(w & ((1u << up) - 1u)) <= r ? up : pos;
  }
  return pos;
}

// Inclusive max-scan of s[0, n) by the workgroup, 4 consecutive slots per
// thread (slots >= n read as 0).  s_mx holds 4 words.  Contains barriers.
__device__ inline void block_max_scan(uint32_t* s, int n, uint32_t* s_mx) {
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int b = 4 * tid;
  const uint4 q = *(const uint4*)(s + b);
  const uint32_t v0 = b < n ? q.x : 0u, v1 = max(v0, b + 1 < n ? q.y : 0u), v2 = max(v1, b + 2 < n ? q.z : 0u),
                 v3 = max(v2, b + 3 < n ? q.w : 0u);
  uint32_t x = v3;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_up(x, d, 64);
    if (lane >= d) x = max(x, y);
  }
  const uint32_t prev = __shfl_up(x, 1, 64);
  if (lane == 63) s_mx[wid] = x;
  __syncthreads();
  uint32_t pre = lane > 0 ? prev : 0u;
  for (int w = 0; w < wid; ++w) pre = max(pre, s_mx[w]);
  *(uint4*)(s + b) = make_uint4(max(pre, v0), max(pre, v1), max(pre, v2), max(pre, v3));
  __syncthreads();
}

// Dense enumeration of the set bits of the brick's per-thread words: thread t
// holds NW words (their bit counts are passed, one per byte of `counts`), item
// numbers run over threads, then words, then bits, and `off` is the thread's
// first item.  For the chunk of items [c0, c0 + n), each
// nonempty word writes a marker at the slot where it begins (slot 0 for a word
// that began in an earlier chunk), (slot << 21) | (bits before the chunk << 16)
// | (t << 8) | word; the max-scan then leaves in every slot i the marker of the
// word that holds item c0 + i, which is that word's
// (i - (marker >> 21) + ((marker >> 16) & 31))-th set bit.  Every lane does
// the same amount of work however the bits fall among the threads.
template <int NW>
__device__ inline void mark_words(const uint32_t* counts, int off, int c0, int n, uint32_t* s, uint32_t* s_mx) {
  static_assert(NW <= 256, "the word index takes 8 bits");
  for (int i = threadIdx.x; i < n; i += kBrickThreads) s[i] = 0u;
  // The counts pass through an empty asm statement so that the compiler does
  // not hoist the NW word offsets out of the caller's chunk loop, which would
  // hold NW more registers through the whole kernel.
  uint32_t cc[(NW + 3) / 4];
#pragma unroll
  for (int q = 0; q < (NW + 3) / 4; ++q) {
    cc[q] = counts[q];
    asm volatile("" : "+v"(cc[q]));
  }
  __syncthreads();
  int o = off - c0;  // first item of word j, relative to the chunk
#pragma unroll
  for (int j = 0; j < NW; ++j) {
    const int c = (int)((cc[j >> 2] >> (8 * (j & 3))) & 0xffu);
    if (c > 0 && o + c > 0 && o < n) {
      const int ls = max(o, 0);
      s[ls] = ((uint32_t)ls << 21) | ((uint32_t)(ls - o) << 16) | ((uint32_t)threadIdx.x << 8) | (uint32_t)j;
    }
    o += c;
  }
  __syncthreads();
  block_max_scan(s, n, s_mx);
}

__device__ inline int marker_rank(uint32_t mk, int i) { return i - (int)(mk >> 21) + (int)((mk >> 16) & 31u); }

// The probability at (z, y, x), 0 outside the array; the load is always issued
// (at a clamped address), so that several of them are in flight together.
__device__ inline float soft_load(const Roi& R, int z, int y, int x) {
  const bool ok = (unsigned)z < (unsigned)R.d[0] && (unsigned)y < (unsigned)R.d[1] && (unsigned)x < (unsigned)R.d[2];
  const int zc = min(max(z, 0), R.d[0] - 1), yc = min(max(y, 0), R.d[1] - 1), xc = min(max(x, 0), R.d[2] - 1);
  const float v = ((const float*)R.vol)[(size_t)zc * (size_t)R.stride0 + (size_t)yc * (size_t)R.stride1 + (size_t)xc];
  return ok ? v : 0.0f;
}

// A brick is kBrickThreads consecutive row-groups (rg = cube row * G + group)
// times up to R.tz (at most kTZ) cube planes.  Its workgroup first loads, as bit masks, every
// voxel row-group it needs into LDS: planes pz0-1 .. pz1-1 and row-groups
// rg0-1 .. rg0+kBrickThreads+G-1 (the row after each cube row, and the word
// before the first group for the x-1 voxel).  All these loads are issued at
// once, each voxel row-group is converted once, and the cube classification
// then reads LDS only.
struct Tile {
  int rg0;       // first row-group of the brick
  int pz0, pz1;  // cube planes [pz0, pz1), pz = z + 1
  int np;        // voxel planes held: pz1 - pz0 + 1
  int nw;        // words per plane: kBrickThreads + 1 + G
};

__device__ inline Tile tile_of(const Roi& R, long long local_brick) {
  Tile T;
  const int bx = (int)(local_brick / R.nzc), zc = (int)(local_brick % R.nzc);
  T.rg0 = bx * kBrickThreads;
  T.pz0 = zc * R.tz;
  T.pz1 = min(T.pz0 + R.tz, R.d[0] + 1);
  T.np = T.pz1 - T.pz0 + 1;
  T.nw = kBrickThreads + 1 + R.G;
  return T;
}

// Voxel row-group vrg of voxel plane p of the tile: the address of its first
// voxel and the number of its 32 voxels that lie inside the array (0 when the
// row-group lies outside it; then the address is not used).
template <int DT>
__device__ inline const char* row_span(const Roi& R, const Tile& T, int p, int vrg, int& nvox) {
  nvox = 0;
  if (vrg < 0) return nullptr;
  const int ry = (int)fdiv((unsigned int)vrg, R.mG, R.shG);
  const int z = T.pz0 - 1 + p, y = ry - 1, x0 = 32 * (vrg - ry * R.G);
  if (z < 0 || z >= R.d[0] || y < 0 || y >= R.d[1] || x0 >= R.d[2]) return nullptr;
  nvox = min(32, R.d[2] - x0);
  const size_t off = (size_t)z * (size_t)R.stride0 + (size_t)y * (size_t)R.stride1 + (size_t)x0;
  return (const char*)R.vol + off * (DT == 0 ? 1 : 4);
}

// Stages the tile's voxel row-groups in LDS.  Each thread issues the loads of
// several row-groups before converting any of them, so a workgroup keeps its
// whole tile in flight instead of one row-group per thread at a time.  A
// row-group's voxels are read as the aligned dwords (uint8; four to a load) or
// floats (four to a load at a 16-byte aligned address) that hold them, and never
// past them, since an aligned dword holding a valid byte lies on a mapped page.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));

// The inside word of up to 32 uint8 voxels: the loads, and then the bits.
struct MaskWord {
  uint32_t d[9];
  int nvox, sh;

  __device__ inline void load(const char* ptr, int n) {
    nvox = n;
    sh = (int)((uintptr_t)ptr & 3u);
#pragma unroll
    for (int j = 0; j < 9; ++j) d[j] = 0u;
    if (n > 0) {
      const uint32_t* q = (const uint32_t*)((uintptr_t)ptr & ~(uintptr_t)3);
      const int last = (sh + n - 1) >> 2;  // last dword holding one of the voxels
#pragma unroll
      for (int h = 0; h < 8; h += 4) {
        if (last >= h + 3) {
          const u32x4 v = *(const u32x4*)(q + h);
          d[h] = v.x;
          d[h + 1] = v.y;
          d[h + 2] = v.z;
          d[h + 3] = v.w;
        } else {
#pragma unroll
          for (int j = h; j < h + 3; ++j)
            if (j <= last) d[j] = q[j];
        }
      }
      if (last == 8) d[8] = q[8];
    }
  }

  // inside: nonzero, or (with a label) no difference from it
  __device__ inline uint32_t bits(int label) const {
    uint32_t x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = __builtin_amdgcn_alignbyte(d[j + 1], d[j], (uint32_t)sh);
    if (label) {
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] ^= (uint32_t)(label & 0xff) * 0x01010101u;
    }
    uint32_t b = nz8(x[0], x[1]) >> 7 | nz8(x[2], x[3]) << 1 | nz8(x[4], x[5]) << 9 | nz8(x[6], x[7]) << 17;
    if (label) b = ~b;
    return nvox >= 32 ? b : b & ((1u << nvox) - 1u);
  }
};

template <int DT>
__device__ inline void load_tile(const Roi& R, const Tile& T, uint32_t* s_bits) {
  const int n = T.np * T.nw;
  if (DT == 0) {
    // thread t takes the word t of every plane (its row is found once), five
    // planes in flight, and then a share of the words past the 256th
    const int rg = T.rg0 - 1 + (int)threadIdx.x;
    const int ry = rg < 0 ? 0 : (int)fdiv((unsigned int)rg, R.mG, R.shG);
    const int y = ry - 1, x0 = 32 * (rg - ry * R.G);
    const int nvox = rg >= 0 && (unsigned)y < (unsigned)R.d[1] ? min(32, R.d[2] - x0) : 0;
    const char* row = (const char*)R.vol + (T.pz0 - 1) * R.stride0 + y * R.stride1 + x0;
    constexpr int kLoadBatch = 5;
#pragma unroll
    for (int p0 = 0; p0 <= kTZ; p0 += kLoadBatch) {
      MaskWord m[kLoadBatch];
#pragma unroll
      for (int u = 0; u < kLoadBatch; ++u) {
        const int p = p0 + u, z = T.pz0 - 1 + p;
        if (p <= kTZ) m[u].load(row + p * R.stride0, p < T.np && (unsigned)z < (unsigned)R.d[0] ? nvox : 0);
      }
#pragma unroll
      for (int u = 0; u < kLoadBatch; ++u)
        if (p0 + u <= kTZ && p0 + u < T.np) s_bits[(p0 + u) * T.nw + threadIdx.x] = m[u].bits(R.label);
    }
    for (int i = threadIdx.x; i < (kTZ + 1) * (T.nw - kBrickThreads); i += kBrickThreads) {
      const int w = kBrickThreads + i / (kTZ + 1), p = i % (kTZ + 1);
      if (p >= T.np) continue;
      int n;
      const char* ptr = row_span<DT>(R, T, p, T.rg0 - 1 + w, n);
      MaskWord m;
      m.load(ptr, n);
      s_bits[p * T.nw + w] = m.bits(R.label);
    }
  } else {
    // float32: a row-group is 128 B; two of them are in flight per thread
    // before either is converted
    constexpr int kLoadBatch = 2;
    for (int base = threadIdx.x; base < n; base += kBrickThreads * kLoadBatch) {
      float v[kLoadBatch][32];
      int nv[kLoadBatch];
#pragma unroll
      for (int h = 0; h < kLoadBatch; ++h) {
        const int idx = base + h * kBrickThreads;
        const char* ptr = nullptr;
        nv[h] = 0;
#pragma unroll
        for (int i = 0; i < 32; ++i) v[h][i] = 0.0f;
        if (idx < n) {
          const int p = (int)fdiv((unsigned int)idx, R.mNW, R.shNW);
          ptr = row_span<DT>(R, T, p, T.rg0 - 1 + idx - p * T.nw, nv[h]);
        }
        const float* f = (const float*)ptr;
        if (nv[h] == 32 && (((uintptr_t)ptr) & 15u) == 0) {
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const float4 q = ((const float4*)f)[i];
            v[h][4 * i] = q.x;
            v[h][4 * i + 1] = q.y;
            v[h][4 * i + 2] = q.z;
            v[h][4 * i + 3] = q.w;
          }
        } else if (nv[h] > 0) {
#pragma unroll
          for (int i = 0; i < 32; ++i)
            if (i < nv[h]) v[h][i] = f[i];
        }
      }
#pragma unroll
      for (int h = 0; h < kLoadBatch; ++h) {
        const int idx = base + h * kBrickThreads;
        if (idx >= n) continue;
        uint32_t bits = 0u;
#pragma unroll
        for (int i = 0; i < 32; ++i) bits |= (uint32_t)(v[h][i] > 0.5f) << i;
        s_bits[idx] = bits;
      }
    }
  }
}

// Thread coordinates inside a brick.
struct Lane {
  int y, l;        // cube row (voxel rows y, y+1) and 32-cube group
  uint32_t vmask;  // cubes of this group inside [-1, d2 - 1]
  bool valid;
};

// Cubes of 32-cube group l inside the ROI: cube x = 32l - 1 + k is valid iff
// k <= d2 - 32l.
__device__ inline uint32_t lane_vmask(const Roi& R, int l) {
  const int kmax = R.d[2] - 32 * l;
  return kmax >= 31 ? 0xffffffffu : ((1u << (kmax + 1)) - 1u);
}

__device__ inline Lane lane_of(const Roi& R, const Tile& T, int tid) {
  Lane L;
  const int rg = T.rg0 + tid;
  L.valid = rg < R.nrg;
  const int ry = L.valid ? (int)fdiv((unsigned int)rg, R.mG, R.shG) : 0;
  L.l = L.valid ? rg - ry * R.G : 0;
  L.y = ry - 1;
  L.vmask = lane_vmask(R, L.l);
  return L;
}

// Bits k - 1 and k of a row as bits 0 and 1 (a: shifted(r)).
__device__ inline uint32_t bit_pair(uint32_t r, uint32_t a, int k) {
  return __builtin_amdgcn_alignbit(r >> 31, a, (uint32_t)k) & 3u;
}

// Count, sum of bit positions b and sum of b^2 over the set bits of w.  With
// M_k the bits whose position has bit k set, b = sum_k 2^k [b in M_k], so
// sum b = sum_k 2^k popc(w & M_k) and sum b^2 = sum_k 4^k popc(w & M_k)
// + sum_{k<l} 2^(k+l+1) popc(w & M_k & M_l).
struct WordMom {
  int c, b1, b2;
};

__device__ inline WordMom word_moments(uint32_t w) {
  WordMom m;
  if (w == 0u) {
    m.c = m.b1 = m.b2 = 0;
    return m;
  }
  if (w == 0xffffffffu) {  // 32 bits: sum b = 496, sum b^2 = 10416
    m.c = 32;
    m.b1 = 496;
    m.b2 = 10416;
    return m;
  }
  const uint32_t M[5] = {0xaaaaaaaau, 0xccccccccu, 0xf0f0f0f0u, 0xff00ff00u, 0xffff0000u};
  m.c = __popc(w);
  int b1 = 0, b2 = 0;
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    const uint32_t wk = w & M[k];
    const int pk = __popc(wk);
    b1 += pk << k;
    b2 += pk << (2 * k);
#pragma unroll
    for (int l = k + 1; l < 5; ++l) b2 += __popc(wk & M[l]) << (k + l + 1);
  }
  m.b1 = b1;
  m.b2 = b2;
  return m;
}

// ---------------------------------------------------------------------------
// Binary masks: area of each case's triangles for each ROI's spacing (one
// workgroup per ROI, one thread per case), read by every brick of the ROI.

__device__ inline double case_area_of(const Roi& R, int c) {
  const int nt = MC_NTRI[c];
  double a = 0.0;
  for (int t = 0; t < nt; ++t) {
    const double n0 = R.s[1] * R.s[2] * MC_TRI_N[c][t][0];
    const double n1 = R.s[0] * R.s[2] * MC_TRI_N[c][t][1];
    const double n2 = R.s[0] * R.s[1] * MC_TRI_N[c][t][2];
    a += 0.125 * sqrt(n0 * n0 + n1 * n1 + n2 * n2);
  }
  return a;
}

// The small-mesh path's first launch (one workgroup): the ROI record, the
// cleared staged-row count and pair-kernel accumulators, and (binary masks)
// the per-case areas and cleared case counts.
__global__ __launch_bounds__(256) void k_small_head(Roi R, Roi* __restrict__ rois, long long* __restrict__ totals,
                                                    SmallAcc* __restrict__ acc, double* __restrict__ case_area) {
  if (threadIdx.x == 0) {
    rois[0] = R;
    totals[8] = 0;
    SmallAcc A;
    for (int g = 0; g < 4; ++g) {
      A.gmax[g] = 0ull;
      A.key[g] = ~0ull;
    }
    A.pairs2d = 0ull;
    A.ticket = 0u;
    A.pad_ = 0u;
    *acc = A;
  }
  if (case_area) {
    case_area[threadIdx.x] = case_area_of(R, (int)threadIdx.x);
    case_hist(case_area, 1)[threadIdx.x] = 0ull;
  }
}

// ---------------------------------------------------------------------------
// What the mesh pass sums in 32 bits: a wave's moments (64 threads of 32 voxels in
// kTZ planes; z' < kTZ, y' <= kBrickThreads, x <= SHAPE3D_MAX_DIM2), a brick's
// volume, and the row and group that share a word.
static_assert(64ll * 32 * (kTZ * (kTZ - 1) / 2) * SHAPE3D_MAX_DIM2 < (1ll << 32), "sum of z' x of a wave");
static_assert(64ll * 32 * kTZ * SHAPE3D_MAX_DIM2 < (1ll << 32), "sum of x of a wave");
static_assert(64ll * 32 * kTZ * kBrickThreads * kBrickThreads < (1ll << 32), "sum of y' y' of a wave");
static_assert(64ll * 32 * (kTZ * (kTZ - 1) / 2) * kBrickThreads < (1ll << 32), "sum of z' y' of a wave");
static_assert(48ll * 32 * kTZ * kBrickThreads < (1ll << 31), "volume of a brick in 1/48 voxels");
static_assert(SHAPE3D_MAX_DIM < (1 << 20) && (SHAPE3D_MAX_DIM2 + 1) / 32 < (1 << 11), "row | group << 20");

// The mesh pass: one read of the volume per brick gives its vertex and
// triangle counts, area, volume, bounding box and moments, and writes the
// canonical keys of its vertices (and soft masks' interpolation parameters)
// to a staging list, at a range of rows the brick reserves with one atomic
// (below `tmp_cap` rows; totals[8] counts them all).  Within a brick the order
// is (thread, plane, cube, axis); the row pass then places each brick's rows
// at its offset in brick order, so the final order does not depend on the
// order of the reservations.

// Bound by vector instructions (binary masks of a batch of 4,096 ROIs: 2,302 a
// wave, 622 of 777 us), so the work per voxel row and per vertex is kept small:
// rows are found once for all planes and turned into bits by dot products; only
// active cubes are enumerated, and list their edges at places the counts give
// (edges listed by an enumeration of their own took 24 markers a thread and the
// edge's words again); triangles and volume follow from the counts of the cases;
// a lane writes four rows, so that a block's box is a reduction over 8 lanes.
// Before and after: the batch 1,107 -> 777 us, 300 x 512 x 512 55 -> 44, a batch
// of 256 with moments 125 -> 85, 24 labels of 181 x 384 x 384 57 -> 38.
// Binary masks: at most 80 VGPRs, so that six bricks share a CU (a few registers
// spill; 96 VGPRs and five bricks a CU: 676 us where six took 626).  Soft masks:
// at most 128 VGPRs, four bricks per CU.
// BITS: the volumes' bit strings are there (k_volume_bits), and the tiles are
// cut from them.
template <int DT, bool BITS>
__global__ __launch_bounds__(kBrickThreads, DT == 0 ? 6 : 4) void k_mesh_pass(const Roi* __restrict__ rois, int n_rois,
                                                             long long nbricks, double* __restrict__ case_area,
                                                             BrickPart* __restrict__ part,
                                                             unsigned long long* __restrict__ tmpkey,
                                                             double* __restrict__ tmpt, long long tmp_cap,
                                                             long long* __restrict__ totals, int moments,
                                                             const int* __restrict__ bmap,
                                                             float4* __restrict__ pbox,
                                                             const uint32_t* __restrict__ bits) {
  extern __shared__ uint32_t s_bits[];
  __shared__ unsigned int s_hist[256];  // binary masks: active cubes per case
  // soft masks: the corner values of the threads' cubes and the triangle table
  // (indexed at run time: from LDS 40 cycles a triangle vertex, from constant
  // memory or by selects over registers several times that)
  __shared__ float s_p[DT == 1 ? 8 : 1][DT == 1 ? kBrickThreads : 1];
  __shared__ uint8_t s_tri[DT == 1 ? 256 * MC_MAX_TRI * 3 : 1];
  __shared__ uint8_t s_nt[DT == 1 ? 256 : 1];
  __shared__ uint32_t s_edge[DT == 1 ? 12 : 1];  // axis | corner 0 << 2 | corner 1 << 5
  // slots kMeshItems ..: the cubes of rows left over from the chunk before
  __shared__ __align__(16) uint32_t s_items[kMeshItems + kSegAlign];
  __shared__ __align__(8) uint16_t s_rows[3 * kMeshItems + kSegAlign];  // slot of the row's cube | axis << 11
  __shared__ int s_eb[kBrickThreads];                      // each thread's first row,
  __shared__ uint32_t s_ec[2][kBrickThreads];              // and its rows per plane, a byte each
  __shared__ int s_ve;
  __shared__ uint32_t s_ly[kBrickThreads];  // (y + 1) | l << 20 of each thread's row-group
  __shared__ int s_scan[4];
  __shared__ uint32_t s_mx[4];
  __shared__ double s_rd[2][4];
  __shared__ int s_rl[4];
  __shared__ int s_ri[7][4];
  __shared__ long long s_mom[10][4];
  __shared__ long long s_base;

  const long long brick = xcd_remap(blockIdx.x, nbricks);
  const int roi = bmap ? bmap[brick] : find_roi(rois, n_rois, brick);
  if (roi < 0) return;
  const Roi R = rois[roi];
  // a grid sized by a bound (ROI table planned on the device) ends past the last brick
  if (brick >= R.brick_end) return;
  const int tid = threadIdx.x;
  if (DT == 0) {
    s_hist[tid] = 0u;
  } else {
    for (int i = tid; i < 256 * MC_MAX_TRI * 3; i += kBrickThreads) s_tri[i] = (&MC_TRI[0][0][0])[i];
    s_nt[tid] = MC_NTRI[tid];
    if (tid < 12) {
      const uint32_t a = MC_EDGE_AXIS[tid], k0 = MC_EDGE_C0[tid];
      s_edge[tid] = a | k0 << 2 | (k0 | 4u >> a) << 5;
    }
  }

  const Tile T = tile_of(R, brick - R.brick_begin);
  if (BITS)
    cut_tile<kTZ + 1>(bits + R.bits_begin, volume_shift(R.vol), R.d, R.G, R.mG, R.shG, T.rg0 - 1, T.pz0 - 1, T.np,
                      T.nw, s_bits);
  else
    load_tile<DT>(R, T, s_bits);
  __syncthreads();
  const Lane L = lane_of(R, T, tid);
  s_ly[tid] = (uint32_t)(L.y + 1) | ((uint32_t)L.l << 20);  // read back by the dense loop (after a barrier)
  int nt = 0, full = 0;  // triangles; binary masks: cubes wholly inside
  double area = 0.0, vol_d = 0.0;
  int vol_i = 0;
  int bb[6] = {INT_MAX, INT_MAX, INT_MAX, INT_MIN, INT_MIN, INT_MIN};
  // origin of the soft tetrahedron sum: the array centre (as the FP64 oracle uses)
  const double o0 = 0.5 * R.d[0] * R.s[0], o1 = 0.5 * R.d[1] * R.s[1], o2 = 0.5 * R.d[2] * R.s[2];

  // All planes of the brick at once.  Each thread counts its active cubes and
  // crossing edges of every plane pair, each row word read once (bit counts of
  // plane pair p: byte p of actc and ec); a crossing edge belongs to the cube
  // that has it at its corner 0, an active one, so the brick's active cubes are
  // then enumerated densely over the workgroup (mark_words) and list their
  // edges in LDS, and the edges' rows are written from there.
  uint32_t actc[(kTZ + 3) / 4] = {}, ec[(kTZ + 3) / 4] = {};
  int cnt = 0, cnt_e = 0;
  {
    uint32_t xm = 0u, zm = 0u;  // cubes active in some plane, planes with an active cube
    uint32_t a0p = 0u, oP = 0u, nP = 0u;
    int e12 = 0;
    const uint32_t vm = L.valid ? L.vmask : 0u;
    const uint32_t* w = s_bits + tid + 1;
#pragma unroll
    for (int p = 0; p <= kTZ; ++p) {
      if (p < T.np) {
        const uint32_t r0 = w[p * T.nw], r1 = w[p * T.nw + R.G];
        const uint32_t a0 = shifted(r0, w[p * T.nw - 1]), a1 = shifted(r1, w[p * T.nw + R.G - 1]);
        const uint32_t o = r0 | a0 | r1 | a1, n = r0 & a0 & r1 & a1;
        if (p > 0) {
          const uint32_t act = (oP | o) & ~(nP & n) & vm;
          const int ca = __popc(act), ce = e12 + __popc((a0p ^ a0) & vm);
          actc[(p - 1) >> 2] |= (uint32_t)ca << (8 * ((p - 1) & 3));
          ec[(p - 1) >> 2] |= (uint32_t)ce << (8 * ((p - 1) & 3));
          cnt += ca;
          cnt_e += ce;
          xm |= act;
          zm |= act ? 1u << (p - 1) : 0u;
          if (DT == 0) full += __popc(nP & n & vm);
        }
        e12 = __popc((a0 ^ a1) & vm) + __popc((a0 ^ r0) & vm);
        a0p = a0;
        oP = o;
        nP = n;
      }
    }
    if (xm) {
      bb[0] = T.pz0 - 2 + __ffs(zm);
      bb[3] = T.pz0 - 1 + 31 - __clz(zm);
      bb[1] = bb[4] = L.y;
      bb[2] = 32 * L.l - 2 + __ffs(xm);
      bb[5] = 32 * L.l - 1 + 31 - __clz(xm);
    }
  }
  // the brick's staged rows: one reservation (of whole 32-row blocks when the
  // blocks' boxes are asked for)
  int total_e;
  s_eb[tid] = block_excl_scan256(cnt_e, s_scan, total_e);
#pragma unroll
  for (int q = 0; q < 2; ++q) s_ec[q][tid] = ec[q];
  if (tid == 0) {
    const int rows = pbox ? (total_e + kSegAlign - 1) & ~(kSegAlign - 1) : total_e;
    s_base = rows ? (long long)atomicAdd((unsigned long long*)&totals[8], (unsigned long long)rows) : 0;
  }
  int total;
  const int off = block_excl_scan256(cnt, s_scan, total);
  const long long base = s_base;
  int done = 0;  // rows written (whole blocks)
  for (int c0 = 0; c0 < total; c0 += kMeshItems) {
    const int n = min(kMeshItems, total - c0);
    mark_words<kTZ>(actc, off, c0, n, s_items, s_mx);
    for (int i = tid; i < n; i += kBrickThreads) {
      const uint32_t mk = s_items[i];
      const int p = (int)(mk & 255u), t = (int)((mk >> 8) & 255u);
      const uint32_t* w0 = s_bits + p * T.nw + t + 1;
      const uint32_t* w1 = w0 + T.nw;
      const uint32_t r00 = w0[0], r01 = w0[R.G], r10 = w1[0], r11 = w1[R.G];
      const uint32_t a00 = shifted(r00, w0[-1]), a01 = shifted(r01, w0[R.G - 1]);
      const uint32_t a10 = shifted(r10, w1[-1]), a11 = shifted(r11, w1[R.G - 1]);
      const uint32_t any = (r00 | a00 | r01) | (a01 | r10 | a10) | (r11 | a11);
      const uint32_t all = (r00 & a00 & r01) & (a01 & r10 & a10) & (r11 & a11);
      // (cubes past the row's end come after the word's last counted one)
      const int k = nth_set_bit(any & ~all, marker_rank(mk, i));
      const int cas = (int)(bit_pair(r00, a00, k) | bit_pair(r01, a01, k) << 2 | bit_pair(r10, a10, k) << 4 |
                            bit_pair(r11, a11, k) << 6);
      // the cube's rows: after those of the threads, planes and cubes before it
      const uint32_t below = (1u << k) - 1u, e0 = a00 ^ a10, e1 = a00 ^ a01, e2 = a00 ^ r00;
      const uint32_t q0 = s_ec[0][t], q1 = s_ec[1][t];
      const uint32_t h0 = p >= 4 ? q0 : q0 & ((1u << (8 * p)) - 1u), h1 = p > 4 ? q1 & ((1u << (8 * p - 32)) - 1u) : 0u;
      int at = s_eb[t] - done + (int)__builtin_amdgcn_sad_u8(h1, 0u, __builtin_amdgcn_sad_u8(h0, 0u, 0u));
      at += __popc(e0 & below) + __popc(e1 & below) + __popc(e2 & below);
      if (e0 >> k & 1u) s_rows[at++] = (uint16_t)i;
      if (e1 >> k & 1u) s_rows[at++] = (uint16_t)(i | 1 << 11);
      if (e2 >> k & 1u) s_rows[at++] = (uint16_t)(i | 2 << 11);
      if (i == n - 1) s_ve = at;
      s_items[i] = (uint32_t)p | (uint32_t)t << 3 | (uint32_t)k << 11;
      if (DT == 0) {
        atomicAdd(&s_hist[cas], 1u);
      } else {
        const uint32_t ly = s_ly[t];
        const int z = T.pz0 - 1 + p, y = (int)(ly & 0xfffffu) - 1, x = 32 * (int)(ly >> 20) - 1 + k;
        const int ntri = s_nt[cas];
        nt += ntri;
#pragma unroll
        for (int c = 0; c < 8; ++c) s_p[c][tid] = soft_load(R, z + ((c >> 2) & 1), y + ((c >> 1) & 1), x + (c & 1));
        for (int tr = 0; tr < ntri; ++tr) {
          double P[3][3];
#pragma unroll
          for (int v = 0; v < 3; ++v) {
            const uint32_t ed = s_edge[s_tri[(cas * MC_MAX_TRI + tr) * 3 + v]];
            const int ax = (int)(ed & 3u), k0 = (int)(ed >> 2 & 7u), k1 = (int)(ed >> 5);
            const double p0 = (double)s_p[k0][tid], p1 = (double)s_p[k1][tid];
            // the area and volume terms only (the vertex rows take the edge
            // pass's correctly rounded quotient): a reciprocal estimate refined
            // by Newton steps is within a unit in the last place
            const double tt = (0.5 - p0) * rcp64(p1 - p0);
            const int u0 = z + ((k0 >> 2) & 1), u1 = y + ((k0 >> 1) & 1), u2 = x + (k0 & 1);
            P[v][0] = ((double)u0 + (ax == 0 ? tt : 0.0)) * R.s[0] - o0;
            P[v][1] = ((double)u1 + (ax == 1 ? tt : 0.0)) * R.s[1] - o1;
            P[v][2] = ((double)u2 + (ax == 2 ? tt : 0.0)) * R.s[2] - o2;
          }
          const double e1x = P[1][0] - P[0][0], e1y = P[1][1] - P[0][1], e1z = P[1][2] - P[0][2];
          const double e2x = P[2][0] - P[0][0], e2y = P[2][1] - P[0][1], e2z = P[2][2] - P[0][2];
          const double nx = e1y * e2z - e1z * e2y, ny = e1z * e2x - e1x * e2z, nz = e1x * e2y - e1y * e2x;
          area += 0.5 * sqrt(nx * nx + ny * ny + nz * nz);
          const double bcx = P[1][1] * P[2][2] - P[1][2] * P[2][1];
          const double bcy = P[1][2] * P[2][0] - P[1][0] * P[2][2];
          const double bcz = P[1][0] * P[2][1] - P[1][1] * P[2][0];
          vol_d += (P[0][0] * bcx + P[0][1] * bcy + P[0][2] * bcz) / 6.0;
        }
      }
    }
    __syncthreads();
    // rows [0, m) of the list are brick rows done ..; whole blocks, unless these
    // are the last ones; with boxes, the rows that fill up the last block repeat
    // the last vertex
    const int have = s_ve;
    const bool last = c0 + kMeshItems >= total;
    const int m = last ? have : have & ~(kSegAlign - 1);
    const int n_fill = last && pbox ? (m + kSegAlign - 1) & ~(kSegAlign - 1) : m;
    // four rows per lane: a block's box is a reduction over 8 lanes
    for (int j = 4 * tid; j < n_fill; j += 4 * kBrickThreads) {
      const uint2 q = *(const uint2*)(s_rows + j);
      const uint32_t rws[4] = {q.x & 0xffffu, q.x >> 16, q.y & 0xffffu, q.y >> 16};
      const uint32_t end = s_rows[m - 1];
      const long long row = base + done + j;
      unsigned long long key[4];
      double tt[4];
      int lo[3] = {INT_MAX, INT_MAX, INT_MAX}, hi[3] = {INT_MIN, INT_MIN, INT_MIN};
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint32_t rw = j + r < m ? rws[r] : end, code = s_items[rw & 2047u];
        const int a = (int)(rw >> 11);
        const uint32_t ly = s_ly[code >> 3 & 255u];
        const int u[3] = {T.pz0 - 1 + (int)(code & 7u), (int)(ly & 0xfffffu) - 1,
                          32 * (int)(ly >> 20) - 1 + (int)(code >> 11)};
        key[r] = pack_key(u[0], u[1], u[2], a);
        tt[r] = 0.5;
        if (DT == 1) {
          const double pa = (double)soft_load(R, u[0], u[1], u[2]);
          const double pb = (double)soft_load(R, u[0] + (a == 0), u[1] + (a == 1), u[2] + (a == 2));
          tt[r] = (0.5 - pa) / (pb - pa);
        }
        // the block's box in half voxels: exact for binary masks, widened by the
        // rounding of the soft coordinate (a vertex that NaN voxels leave without
        // a position is in no box)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          if (DT == 0) {
            const int c = 2 * u[k] + (a == k);
            lo[k] = min(lo[k], c);
            hi[k] = max(hi[k], c);
          } else {
            const float c = (float)(2.0 * ((double)u[k] + (a == k ? tt[r] : 0.0))), wd = fabsf(c) * 1.1920928955078125e-07f;
            const bool ok = tt[r] == tt[r];
            lo[k] = min(lo[k], float_order(ok ? c - wd : 3.0e38f));
            hi[k] = max(hi[k], float_order(ok ? c + wd : -3.0e38f));
          }
        }
      }
      if (pbox && row + 4 <= tmp_cap) {  // (a block's rows start at a multiple of 32)
        ((ulonglong2*)(tmpkey + row))[0] = make_ulonglong2(key[0], key[1]);
        ((ulonglong2*)(tmpkey + row))[1] = make_ulonglong2(key[2], key[3]);
        if (DT == 1) {
          ((double2*)(tmpt + row))[0] = make_double2(tt[0], tt[1]);
          ((double2*)(tmpt + row))[1] = make_double2(tt[2], tt[3]);
        }
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (j + r < n_fill && row + r < tmp_cap) {
            tmpkey[row + r] = key[r];
            if (DT == 1) tmpt[row + r] = tt[r];
          }
        }
      }
      if (pbox) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          lo[k] = lanes_min_i32<3>(lo[k]);
          hi[k] = lanes_max_i32<3>(hi[k]);
        }
        if ((j & (kSegAlign - 1)) == 0 && row < tmp_cap) {
          float fl[3], fh[3];
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            fl[k] = DT == 0 ? (float)lo[k] : order_float(lo[k]);
            fh[k] = DT == 0 ? (float)hi[k] : order_float(hi[k]);
          }
          float4* bx = pbox + 2 * (row / kSegAlign);
          bx[0] = make_float4(fl[0], fl[1], fl[2], fh[0]);
          bx[1] = make_float4(fh[1], fh[2], 0.0f, 0.0f);
        }
      }
    }
    if (!last) {
      // the rows left over go to the front, their cubes to the spare slots
      uint32_t rw = 0u, code = 0u;
      if (tid < have - m) {
        rw = s_rows[m + tid];
        code = s_items[rw & 2047u];
      }
      __syncthreads();
      if (tid < have - m) {
        s_rows[tid] = (uint16_t)((rw & ~2047u) | (uint32_t)(kMeshItems + tid));
        s_items[kMeshItems + tid] = code;
      }
      done += m;
    }
  }

  // Inside-voxel moments, from the tile: voxel row (z, y) = (pz0 + p, L.y + 1),
  // x = 32 l + bit, is the tile word of plane p + 1, row-group tid + G (the far
  // corner row of plane pair p); rows past the array read as 0.  Summed with z
  // and y from the brick's first row (z' < 8, y' < 257): only the sums of x^2
  // and x y' of a wave can pass 32 bits.
  unsigned int mom[8] = {};  // n, z', y', x, z'z', y'y', z'y', z'x
  long long mxx = 0, mxy = 0;
  const int y0 = (int)(s_ly[0] & 0xfffffu);
  if (moments && L.valid) {
    unsigned int n = 0, sz = 0, szz = 0, sb1 = 0, szb = 0, sb2 = 0;
#pragma unroll
    for (int p = 0; p < kTZ; ++p) {
      if (p + 1 < T.np) {
        const uint32_t w = s_bits[(p + 1) * T.nw + tid + 1 + R.G];
        const WordMom wm = word_moments(w);
        n += wm.c;
        sz += p * wm.c;
        szz += p * p * wm.c;
        sb1 += wm.b1;
        szb += p * wm.b1;
        sb2 += wm.b2;
      }
    }
    const unsigned int y = L.y + 1 - y0, x0 = 32 * L.l;
    const unsigned int sx = x0 * n + sb1;
    mom[0] = n;
    mom[1] = sz;
    mom[2] = y * n;
    mom[3] = sx;
    mom[4] = szz;
    mom[5] = y * y * n;
    mom[6] = y * sz;
    mom[7] = x0 * sz + szb;
    mxx = (long long)x0 * (sx + sb1) + sb2;
    mxy = (long long)y * sx;
  }

  // fixed-order block reduction
  const int lane = tid & 63, wid = tid >> 6;
  if (DT == 0) {
    // triangles and volume from the case counts (the last item's barrier is past)
    const int h = (int)s_hist[tid];
    nt = h * MC_NTRI[tid];
    vol_i = lanes_sum_i32<6>(h * MC_CASE_VOLUME[tid] + 48 * full);
  }
  nt = lanes_sum_i32<6>(nt);
  if (DT == 1) {
    area = wave_sum(area);
    vol_d = wave_sum(vol_d);
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    bb[k] = lanes_min_i32<6>(bb[k]);
    bb[3 + k] = lanes_max_i32<6>(bb[3 + k]);
  }
  if (moments) {
    for (int k = 0; k < 8; ++k) mom[k] = (unsigned int)lanes_sum_i32<6>((int)mom[k]);
    mxx = wave_sum(mxx);
    mxy = wave_sum(mxy);
  }
  if (lane == 0) {
    s_ri[0][wid] = nt;
    for (int k = 0; k < 6; ++k) s_ri[1 + k][wid] = bb[k];
    s_rd[0][wid] = area;
    s_rd[1][wid] = vol_d;
    s_rl[wid] = vol_i;
    for (int k = 0; k < 8; ++k) s_mom[k][wid] = mom[k];
    s_mom[8][wid] = mxx;
    s_mom[9][wid] = mxy;
  }
  __syncthreads();
  if (tid == 0) {
    BrickPart P;
    P.nv = total_e;
    P.nt = s_ri[0][0] + s_ri[0][1] + s_ri[0][2] + s_ri[0][3];
    for (int k = 0; k < 3; ++k) {
      P.bb[k] = min(min(s_ri[1 + k][0], s_ri[1 + k][1]), min(s_ri[1 + k][2], s_ri[1 + k][3]));
      P.bb[3 + k] = max(max(s_ri[4 + k][0], s_ri[4 + k][1]), max(s_ri[4 + k][2], s_ri[4 + k][3]));
    }
    P.area = ((s_rd[0][0] + s_rd[0][1]) + s_rd[0][2]) + s_rd[0][3];
    P.vol_d = ((s_rd[1][0] + s_rd[1][1]) + s_rd[1][2]) + s_rd[1][3];
    P.vol_i = (long long)s_rl[0] + s_rl[1] + s_rl[2] + s_rl[3];
    long long m[10];
    for (int k = 0; k < 10; ++k) m[k] = s_mom[k][0] + s_mom[k][1] + s_mom[k][2] + s_mom[k][3];
    // back to the ROI's z and y: n, z, y, x, zz, yy, xx, zy, zx, yx
    const long long zo = T.pz0, yo = y0;
    P.mom[0] = m[0];
    P.mom[1] = m[1] + zo * m[0];
    P.mom[2] = m[2] + yo * m[0];
    P.mom[3] = m[3];
    P.mom[4] = m[4] + 2 * zo * m[1] + zo * zo * m[0];
    P.mom[5] = m[5] + 2 * yo * m[2] + yo * yo * m[0];
    P.mom[6] = m[8];
    P.mom[7] = m[6] + zo * m[2] + yo * m[1] + zo * yo * m[0];
    P.mom[8] = m[7] + zo * m[3];
    P.mom[9] = m[9] + yo * m[3];
    P.stage = base;
    part[brick] = P;
  }
  if (DT == 0) {
    // the area follows from the case counts (summed per ROI in a fixed order
    // later), so it does not depend on how the ROI is cut into bricks
    const unsigned int h = s_hist[tid];
    if (h) atomicAdd(&case_hist(case_area, n_rois)[(size_t)roi * 256 + tid], (unsigned long long)h);
  }
}

// ---------------------------------------------------------------------------
// Per-ROI totals: exclusive scan of brick vertex counts (each brick's first
// row within its ROI), fixed-order sums.  One 1024-thread workgroup per ROI.

// 128-bit sum over a wave (two's complement halves, carry from the low half).
__device__ inline __int128 wave_sum_i128(__int128 v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    const unsigned long long lo = (unsigned long long)v, hi = (unsigned long long)(v >> 64);
    const unsigned long long olo = __shfl_xor(lo, m, 64), ohi = __shfl_xor(hi, m, 64);
    const unsigned long long slo = lo + olo;
    const unsigned long long shi = hi + ohi + (slo < lo ? 1ull : 0ull);
    v = (__int128)(((unsigned __int128)shi << 64) | (unsigned __int128)slo);
  }
  return v;
}

// Covariance entry k (zz, yy, xx, zy, zx, yx) of the inside voxels' physical
// coordinates from exact integer moments S = (n, sums of z, y, x, of zz, yy,
// xx, of zy, zx, yx): cov_ij = s_i s_j (n S_ij - S_i S_j) / n^2, the
// numerator exact in 128 bits (n < 2^40 voxels and coordinates < 2^20 keep it
// below 2^120).
__device__ inline double cov_entry(const __int128* S, const double* sp, int k) {
  const int i = k < 3 ? k : (k == 5 ? 1 : 0);
  const int j = k < 3 ? k : (k == 3 ? 1 : 2);
  const __int128 n = S[0];
  if (n <= 0) return 0.0;
  const __int128 c = n * S[4 + k] - S[1 + i] * S[1 + j];
  return (double)c / ((double)n * (double)n) * (sp[i] * sp[j]);
}

// Exclusive prefix sum over the workgroup's NT threads; s_w: NT / 64 words of
// LDS.  Contains barriers.
template <int NT>
__device__ inline long long block_excl_scan_i64(long long v, long long* s_w, long long& total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  long long inc = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const long long t = __shfl_up(inc, d, 64);
    if (lane >= d) inc += t;
  }
  __syncthreads();  // s_w of an earlier scan has been read
  if (lane == 63) s_w[wid] = inc;
  __syncthreads();
  long long base = 0;
  total = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) {
    if (w < wid) base += s_w[w];
    total += s_w[w];
  }
  return base + inc - v;
}

// Per-ROI totals, one workgroup of NT threads per ROI: a few large ROIs take
// 1,024, a batch 256 (its ROIs have tens of bricks).  The FP64 partials of soft
// masks are summed in one order whatever NT: 1,024 slots of consecutive
// bricks, then a halving tree.  The bricks' first rows within the ROI go to
// brick_voff (the general pipeline), or, with X.lphys set, the ROI's staged
// blocks to the block list at a range that starts on a superblock.
// totals: [0] rows of all ROIs, [9] blocks (with the block list; else
// k_roi_rows writes the rows).
template <int NT>
__global__ __launch_bounds__(NT) void k_mesh_totals(const Roi* __restrict__ rois, int n_rois, int dtype,
                                                    const double* __restrict__ case_area,
                                                    const BrickPart* __restrict__ part, long long* brick_voff,
                                                    RoiMeta* __restrict__ meta, long long* __restrict__ totals,
                                                    int moments, BlockIndex X) {
  constexpr int Q = 1024 / NT, NW = NT / 64;
  __shared__ long long s_w[NW];
  __shared__ long long s_l[3][NW];
  __shared__ int s_b[6][NW];
  __shared__ double s_d[2][512];
  __shared__ __int128 s_S[10];
  __shared__ long long s_base;
  // first block, staged block and end of the ROI's first kBricks bricks
  constexpr int kBricks = 2 * NT;
  __shared__ int s_first[kBricks + 1], s_ph[kBricks];
  const int r = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const long long b0 = rois[r].brick_begin, b1 = rois[r].brick_end;
  const long long n = b1 - b0;
  const long long chunk = (n + 1023) / 1024;
  long long nv = 0, nt = 0, vi = 0, q_n[Q];
  double area[Q], vd[Q];
  int bb[6] = {INT_MAX, INT_MAX, INT_MAX, INT_MIN, INT_MIN, INT_MIN};
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const long long slot = tid + (long long)NT * q;
    const long long lo = b0 + min(n, chunk * slot), hi = b0 + min(n, chunk * (slot + 1));
    q_n[q] = 0;
    area[q] = 0.0;
    vd[q] = 0.0;
    for (long long b = lo; b < hi; ++b) {
      const BrickPart& P = part[b];
      const int pv = P.nv;
      nv += pv;
      nt += P.nt;
      vi += P.vol_i;
      area[q] += P.area;
      vd[q] += P.vol_d;
      for (int k = 0; k < 3; ++k) {
        bb[k] = min(bb[k], P.bb[k]);
        bb[3 + k] = max(bb[3 + k], P.bb[3 + k]);
      }
      q_n[q] += X.lphys ? (pv + kSegAlign - 1) / kSegAlign : pv;
    }
  }
  // where each slot's rows (or blocks) start
  long long off[Q], total = 0;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    long long t;
    off[q] = total + block_excl_scan_i64<NT>(q_n[q], s_w, t);
    total += t;
  }
  const bool fits = X.lphys == nullptr || totals[8] <= X.rows_cap;
  if (X.lphys) {
    const long long nsb = (total + kSuper - 1) / kSuper;
    if (tid == 0 && fits && total)
      s_base = (long long)atomicAdd((unsigned long long*)&totals[9], (unsigned long long)(nsb * kSuper));
    else if (tid == 0)
      s_base = 0;
    __syncthreads();
    if (fits) {
      const long long base = s_base;
      for (long long j = total + tid; j < nsb * kSuper; j += NT) X.lphys[base + j] = -1;
      for (long long j = tid; j < nsb; j += NT) X.sbroi[base / kSuper + j] = r;
    }
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const long long slot = tid + (long long)NT * q;
    const long long lo = b0 + min(n, chunk * slot), hi = b0 + min(n, chunk * (slot + 1));
    long long o = off[q];
    for (long long b = lo; b < hi; ++b) {
      const int pv = part[b].nv;
      if (!X.lphys) {
        brick_voff[b] = o;
        o += pv;
        continue;
      }
      const int nb = (pv + kSegAlign - 1) / kSegAlign;
      const int ph = (int)(part[b].stage / kSegAlign);
      if (b - b0 < kBricks) {
        s_first[b - b0] = (int)o;
        s_ph[b - b0] = ph;
        if (b + 1 == b1 || b - b0 == kBricks - 1) s_first[b - b0 + 1] = (int)(o + nb);
      } else if (fits) {
        for (int j = 0; j < nb; ++j) X.lphys[s_base + o + j] = ph + j;
      }
      o += nb;
    }
  }
  if (X.lphys) {
    // the bricks' blocks, a wave per brick
    __syncthreads();
    if (fits)
      for (int b = wid; b < (int)min(n, (long long)kBricks); b += NW) {
        const int f = s_first[b], nb = s_first[b + 1] - f, ph = s_ph[b];
        for (int j = lane; j < nb; j += 64) X.lphys[s_base + f + j] = ph + j;
      }
  }
  // integer totals: any order
  nv = wave_sum(nv);
  nt = wave_sum(nt);
  vi = wave_sum(vi);
  for (int k = 0; k < 3; ++k) {
    bb[k] = wave_min(bb[k]);
    bb[3 + k] = wave_max(bb[3 + k]);
  }
  if (lane == 0) {
    s_l[0][wid] = nv;
    s_l[1][wid] = nt;
    s_l[2][wid] = vi;
    for (int k = 0; k < 6; ++k) s_b[k][wid] = bb[k];
  }
  double sum_area = 0.0, sum_vd = 0.0;
  if (dtype == 0) {
    // binary masks: the area from the case counts
    __syncthreads();
    binary_area_tree(case_area + (size_t)r * 256, case_hist(case_area, n_rois) + (size_t)r * 256, s_d[0]);
    sum_area = s_d[0][0];
  } else {
    // the halving tree over 1,024 slots: slot v takes in slot v + w, w = 512, 256, ..., 1
    if (Q == 4) {
      area[0] += area[2 % Q];
      area[1 % Q] += area[3 % Q];
      vd[0] += vd[2 % Q];
      vd[1 % Q] += vd[3 % Q];
      area[0] += area[1 % Q];
      vd[0] += vd[1 % Q];
    }
    for (int w = NT / 2; w >= 1; w >>= 1) {
      __syncthreads();
      if (tid >= w && tid < 2 * w) {
        s_d[0][tid - w] = area[0];
        s_d[1][tid - w] = vd[0];
      }
      __syncthreads();
      if (tid < w) {
        area[0] += s_d[0][tid];
        vd[0] += s_d[1][tid];
      }
    }
    sum_area = area[0];
    sum_vd = vd[0];
  }
  if (tid == 0) {
    const Roi& R = rois[r];
    RoiMeta M;
    long long V = 0, T = 0, vol_i = 0;
    for (int w = 0; w < NW; ++w) {
      V += s_l[0][w];
      T += s_l[1][w];
      vol_i += s_l[2][w];
    }
    M.V = V;
    M.T = T;
    M.row_off = 0;
    M.prune_off = 0;
    M.V_pad = (V + kSegAlign - 1) / kSegAlign * kSegAlign;
    M.area = sum_area;
    M.vol = dtype == 0 ? (double)vol_i * (R.s[0] * R.s[1] * R.s[2] / 48.0) : sum_vd;
    double R2 = 0.0, reach = 0.0;
    for (int k = 0; k < 3; ++k) {
      M.bb[k] = s_b[k][0];
      M.bb[3 + k] = s_b[3 + k][0];
      for (int w = 1; w < NW; ++w) {
        M.bb[k] = min(M.bb[k], s_b[k][w]);
        M.bb[3 + k] = max(M.bb[3 + k], s_b[3 + k][w]);
      }
      if (V > 0) {
        M.center[k] = 0.5 * (double)(M.bb[k] + M.bb[3 + k] + 1) * R.s[k];
        const double h = 0.5 * (double)(M.bb[3 + k] - M.bb[k] + 1) * R.s[k];
        R2 += h * h;
      } else {
        M.center[k] = 0.0;
      }
      reach = fmax(reach, (double)(R.d[k] + 1) * R.s[k]);
    }
    M.R2 = R2;
    M.n_in = 0;
    for (int k = 0; k < 6; ++k) M.cov[k] = 0.0;
    M.blk0 = X.lphys ? s_base : 0;
    M.nblk = X.lphys && fits ? (int)total : 0;
    M.ex = ilogb(reach);
    for (int k = 0; k < 3; ++k) M.hs[k] = (float)ldexp(0.5 * R.s[k], -M.ex);
    meta[r] = M;
    if (X.lphys) {
      atomicAdd((unsigned long long*)&totals[0], (unsigned long long)M.V_pad);
      if (!fits) *X.overflow = 1u;
    }
  }
  if (X.lphys && tid < 4) {
    GroupRes G;
    G.best_bits = 0ull;
    G.id_lo = ~0ull;
    G.id_hi = ~0ull;
    G.row_i = -1;
    G.row_j = -1;
    G.gmax = 0.0f;
    G.n_cand = 0;
    X.gres[4ll * r + tid] = G;
  }
  if (!moments) return;
  // exact moment sums in 128 bits, a wave per moment
  for (int k = wid; k < 10; k += NW) {
    __int128 m = 0;
    for (long long b = b0 + lane; b < b1; b += 64) m += (__int128)part[b].mom[k];
    m = wave_sum_i128(m);
    if (lane == 0) s_S[k] = m;
  }
  __syncthreads();
  if (tid < 6) meta[r].cov[tid] = cov_entry(s_S, rois[r].s, tid);
  if (tid == 6) meta[r].n_in = (long long)s_S[0];
}

// Layout-0 row offsets of the ROIs (exclusive scan of V_pad) and the first
// column pair of each pruned ROI (at least prune_min_v vertices) in the 3D
// pruning pass (exclusive scan of ncol^2, ncol = ceil(V_pad / 1024)), one
// workgroup.  totals: [0] layout-0 rows, [1] largest V, [7] column pairs.
__global__ __launch_bounds__(1024) void k_roi_rows(int n_rois, RoiMeta* __restrict__ meta,
                                                   long long* __restrict__ totals, int prune_min_v) {
  __shared__ long long s[2][2][1024];
  const int tid = threadIdx.x;
  const int chunk = (n_rois + 1023) / 1024;
  const int lo = min(n_rois, chunk * tid), hi = min(n_rois, chunk * (tid + 1));
  auto npair = [&](const RoiMeta& M) -> long long {
    if (M.V < 2 || M.V < prune_min_v) return 0;
    const long long nc = (M.V_pad + kPruneSB * 32 - 1) / (kPruneSB * 32);
    return nc * nc;
  };
  long long sum = 0, np = 0, vmax = 0;
  for (int r = lo; r < hi; ++r) {
    const RoiMeta& M = meta[r];
    sum += M.V_pad;
    np += npair(M);
    vmax = max(vmax, M.V);
  }
  s[0][0][tid] = sum;
  s[1][0][tid] = np;
  __syncthreads();
  int src = 0;
  for (int d = 1; d < 1024; d <<= 1) {
    for (int q = 0; q < 2; ++q) {
      long long v = s[q][src][tid];
      if (tid >= d) v += s[q][src][tid - d];
      s[q][1 - src][tid] = v;
    }
    __syncthreads();
    src = 1 - src;
  }
  long long off = s[0][src][tid] - sum, poff = s[1][src][tid] - np;
  for (int r = lo; r < hi; ++r) {
    RoiMeta& M = meta[r];
    M.row_off = off;
    M.prune_off = poff;
    off += M.V_pad;
    poff += npair(M);
  }
  const long long rows0 = s[0][src][1023], np_total = s[1][src][1023];
  __syncthreads();
  s[0][0][tid] = vmax;
  __syncthreads();
  for (int w = 512; w >= 1; w >>= 1) {
    if (tid < w) s[0][0][tid] = max(s[0][0][tid], s[0][0][tid + w]);
    __syncthreads();
  }
  if (tid == 0) {
    totals[0] = rows0;
    totals[1] = s[0][0][0];
    totals[7] = np_total;
  }
}

// Refuses a call whose vertex rows exceed the rows the buffers were sized for
// (possible when a captured graph is replayed on new mask contents): raises
// the overflow flag and empties every ROI, so all later kernels do no work.
// Then writes each ROI's 3D segment (its layout-0 rows when it has pairs).
__global__ void k_check_capacity(int n_rois, long long rows0_cap, RoiMeta* __restrict__ meta,
                                 long long* __restrict__ totals, unsigned int* __restrict__ overflow,
                                 Seg* __restrict__ segs) {
  const bool over = totals[0] > rows0_cap;
  __syncthreads();
  for (int r = threadIdx.x; r < n_rois; r += blockDim.x) {
    if (over) {
      meta[r].V = 0;
      meta[r].V_pad = 0;
      meta[r].row_off = 0;
    }
    Seg S;
    S.row_begin = meta[r].row_off;
    S.n_rows = meta[r].V >= 2 ? (int)meta[r].V_pad : 0;
    S.group = r * 4;
    segs[r] = S;
  }
  __syncthreads();
  if (over && threadIdx.x == 0) {
    *overflow = 1u;
    totals[0] = 0;
    totals[1] = 0;
    totals[7] = 0;
  }
}

// ---------------------------------------------------------------------------
// Row layout: one workgroup per brick moves the brick's staged vertices to
// layout 0, at the ROI's first row plus the brick's offset within its ROI
// (rows in brick order, then the staging order within the brick), with the
// pair pass's operands: the position minus the ROI's centre, rounded to FP32,
// either as FP32 position blocks or as the split-f16 operand row; and the
// 16-row block tags.  The brick that holds a ROI's last vertex pads the ROI
// to a multiple of 32 rows with copies of that vertex.

__device__ inline void put_row(const Roi& R, const RoiMeta& M, long long row, unsigned long long k, double tv,
                               unsigned long long* __restrict__ key, double* __restrict__ tsoft,
                               float* __restrict__ pos, uint4* __restrict__ posh, int* __restrict__ orig,
                               long long src_row) {
  key[row] = k;
  if (tsoft) tsoft[row] = tv;
  const int u0 = (int)((k >> 40) & 0xFFFFF) - 1, u1 = (int)((k >> 20) & 0xFFFFF) - 1, u2 = (int)(k & 0xFFFFF) - 1;
  const int a = (int)((k >> 60) & 3);
  const double px = ((double)u0 + (a == 0 ? tv : 0.0)) * R.s[0] - M.center[0];
  const double py = ((double)u1 + (a == 1 ? tv : 0.0)) * R.s[1] - M.center[1];
  const double pz = ((double)u2 + (a == 2 ? tv : 0.0)) * R.s[2] - M.center[2];
  const float fx = (float)px, fy = (float)py, fz = (float)pz;
  const float fw = (float)((double)fx * fx + (double)fy * fy + (double)fz * fz);
  if (posh) {
    write_split_row(posh, row, fx, fy, fz, fw, h_scale_exp(M.R2));
  } else {
    float* blk = pos + (row >> 4) * 64 + (row & 15);
    blk[0] = fx;
    blk[16] = fy;
    blk[32] = fz;
    blk[48] = fw;
  }
  orig[row] = (int)src_row;
}

__global__ __launch_bounds__(256) void k_mesh_rows(const Roi* __restrict__ rois, int n_rois, long long nbricks,
                                                   const BrickPart* __restrict__ part,
                                                   const long long* __restrict__ brick_voff,
                                                   const RoiMeta* __restrict__ meta,
                                                   const unsigned long long* __restrict__ tmpkey,
                                                   const double* __restrict__ tmpt, long long tmp_cap,
                                                   unsigned long long* __restrict__ key, double* __restrict__ tsoft,
                                                   float* __restrict__ pos, uint4* __restrict__ posh,
                                                   int* __restrict__ orig, int* __restrict__ blkseg,
                                                   unsigned int* __restrict__ overflow, const int* __restrict__ bmap) {
  const long long brick = blockIdx.x;
  if (brick >= nbricks) return;
  const int r = bmap ? bmap[brick] : find_roi(rois, n_rois, brick);
  if (r < 0) return;
  const Roi& R = rois[r];
  if (brick >= R.brick_end) return;
  const RoiMeta& M = meta[r];
  const long long cnt = part[brick].nv, first = brick_voff[brick];
  // an emptied ROI (capacity exceeded), or a brick whose rows do not fit its ROI's count
  if (cnt == 0 || M.V == 0 || first + cnt > M.V) return;
  const long long src = part[brick].stage;
  if (src + cnt > tmp_cap) {  // staged beyond the list (a replay on larger meshes): refused
    if (threadIdx.x == 0) *overflow = 1u;
    return;
  }
  const long long dst = M.row_off + first;
  // four rows per thread at a time, their staged keys loaded together (a load
  // after a row's stores would wait for them)
  for (long long i0 = threadIdx.x; i0 < cnt; i0 += 4ll * blockDim.x) {
    unsigned long long kk[4];
    double tt[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const long long i = min(i0 + (long long)u * blockDim.x, cnt - 1);
      kk[u] = tmpkey[src + i];
      tt[u] = tsoft ? tmpt[src + i] : 0.5;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const long long i = i0 + (long long)u * blockDim.x;
      if (i >= cnt) break;
      const long long row = dst + i;
      put_row(R, M, row, kk[u], tt[u], key, tsoft, pos, posh, orig, row);
      if ((row & 15) == 0 || i == 0) blkseg[row >> 4] = r;  // a block shared with a neighbour gets the same tag
    }
  }
  if (first + cnt == M.V) {  // the ROI's last vertex: pad to V_pad rows with copies of it
    const long long last = M.row_off + M.V - 1;
    const unsigned long long k = tmpkey[src + cnt - 1];
    const double tv = tsoft ? tmpt[src + cnt - 1] : 0.5;
    for (long long row = M.row_off + M.V + threadIdx.x; row < M.row_off + M.V_pad; row += blockDim.x) {
      put_row(R, M, row, k, tv, key, tsoft, pos, posh, orig, last);
      if ((row & 15) == 0) blkseg[row >> 4] = r;
    }
  }
}

// Workgroups that write the brick -> ROI map (so that a brick's workgroup finds
// its ROI with one load instead of a search of the ROI table) past the last ROI:
// the grid of a call planned on the device is sized by a bound.
constexpr int kBrickMapTailGroups = 64;

// The call's head, one launch: clears its counters and device totals (the
// staged-row count among them); per ROI the binary masks' case areas and
// cleared case counts, and the brick -> ROI map.  Workgroup r < n_rois serves
// ROI r, the others write -1 over the bricks past the last ROI.  one: the
// ROI record of a call with one ROI, stored here instead of uploaded.
__global__ __launch_bounds__(256) void k_head(Roi* __restrict__ rois, int n_rois, long long nbricks,
                                              double* __restrict__ case_area, int* __restrict__ bmap,
                                              unsigned int* __restrict__ counters, int n_counters,
                                              long long* __restrict__ totals, int* __restrict__ bitmap,
                                              long long n_bitblks, Roi one, int use_one) {
  const int tid = threadIdx.x;
  if (blockIdx.x == 0) {
    for (int i = tid; i < n_counters; i += 256) counters[i] = 0u;
    if (tid < 16) totals[tid] = 0;
    if (use_one && tid == 0) rois[0] = one;
  }
  if ((int)blockIdx.x < n_rois && case_area) {
    const size_t i = (size_t)blockIdx.x * 256 + tid;
    case_area[i] = use_one ? case_area_of(one, tid) : case_area_of(rois[blockIdx.x], tid);
    case_hist(case_area, n_rois)[i] = 0ull;
  }
  if (!bmap) return;
  if (bitmap && (int)blockIdx.x < n_rois) {
    const long long e = (int)blockIdx.x + 1 < n_rois ? rois[blockIdx.x + 1].bitblk_begin : n_bitblks;
    for (long long b = rois[blockIdx.x].bitblk_begin + tid; b < e; b += 256) bitmap[b] = (int)blockIdx.x;
  }
  if ((int)blockIdx.x < n_rois) {
    const long long b1 = min(rois[blockIdx.x].brick_end, nbricks);
    for (long long b = rois[blockIdx.x].brick_begin + tid; b < b1; b += 256) bmap[b] = (int)blockIdx.x;
  } else {
    const long long b0 = rois[n_rois - 1].brick_end + (long long)(blockIdx.x - n_rois) * 256 + tid;
    for (long long b = b0; b < nbricks; b += (long long)kBrickMapTailGroups * 256) bmap[b] = -1;
  }
}

// ---------------------------------------------------------------------------
// The bit strings of a table of dense float volumes, a stream: 16-byte loads, 16 in
// flight a thread (256 soft ROIs of edges 48 to 160, 1.09 GB: 218 us, 5.0 TB/s).
template <int ROUNDS>
__global__ __launch_bounds__(256) void k_volume_bits(const Roi* __restrict__ rois, const int* __restrict__ map,
                                                     uint32_t* __restrict__ bits) {
  const Roi& R = rois[map ? map[blockIdx.x] : 0];
  pack_bits<ROUNDS>(R.vol, (long long)R.d[0] * R.d[1] * R.d[2],
                        (blockIdx.x - R.bitblk_begin) * (ROUNDS * 4096ll), bits + R.bits_begin);
}

// ---------------------------------------------------------------------------
// ROI tables built on the device.

// A caller's table of ROI descriptors (device memory) -> the mesh pass's ROI
// table, in one workgroup: each descriptor is validated (dims within the
// call's bounds, spacing finite and positive, strides that keep rows and
// planes apart, every voxel inside the allocation [base, base + alloc_elems)
// elements, a label only for uint8), its geometry filled as on the host, and
// brick and bucket offsets placed by exclusive scans.  A rejected descriptor
// becomes a 1x1x1 ROI with no bricks and status -1 (invalid argument).
// plan[0] receives the brick count, plan[1] the bucket count.
__global__ __launch_bounds__(1024) void k_plan_rois(const RoiDesc* __restrict__ in, int n, int dtype, long long md0,
                                                    long long md1, long long md2, const char* __restrict__ base,
                                                    long long alloc_elems, Roi* __restrict__ out,
                                                    long long* __restrict__ plan) {
  __shared__ long long s[2][2][1024];
  const int tid = threadIdx.x;
  const int chunk = (n + 1023) / 1024;
  const int lo = min(n, chunk * tid), hi = min(n, chunk * (tid + 1));
  const size_t elem = dtype == 0 ? 1 : 4;
  long long nbr = 0, nbu = 0;
  for (int r = lo; r < hi; ++r) {
    const RoiDesc D = in[r];
    bool ok = true;
    const long long dmax[3] = {md0, md1, md2};
    for (int k = 0; k < 3; ++k) {
      ok = ok && D.dims[k] >= 1 && D.dims[k] <= dmax[k];
      ok = ok && D.spacing[k] > 0.0 && isfinite(D.spacing[k]);
    }
    ok = ok && D.offset >= 0 && D.strides[0] >= 0 && D.strides[1] >= 0 && D.label >= 0 && D.label <= 255 &&
         (dtype == 0 || D.label == 0);
    long long st1 = 0, st0 = 0;
    if (ok) {
      st1 = D.strides[1] > 0 ? D.strides[1] : D.dims[2];
      st0 = D.strides[0] > 0 ? D.strides[0] : D.dims[1] * D.dims[2];
      ok = st1 >= D.dims[2] && st0 >= (D.dims[1] - 1) * st1 + D.dims[2];
      // the last voxel (products below 2^63: dims <= 2^20, strides checked against the allocation first)
      ok = ok && st0 < alloc_elems && st1 < alloc_elems &&
           D.offset + (D.dims[0] - 1) * st0 + (D.dims[1] - 1) * st1 + D.dims[2] <= alloc_elems;
    }
    Roi R;
    if (ok) {
      nbr += roi_fill(R, base + (size_t)D.offset * elem, D.dims, D.spacing, st0, st1, D.label);
    } else {
      const long long one[3] = {1, 1, 1};
      const double unit[3] = {1.0, 1.0, 1.0};
      (void)roi_fill(R, base, one, unit, 0, 0, 0);
      R.status = -1;
    }
    nbu += roi_buckets(R.d);
    out[r] = R;
  }
  s[0][0][tid] = nbr;
  s[1][0][tid] = nbu;
  __syncthreads();
  int src = 0;
  for (int d = 1; d < 1024; d <<= 1) {
    for (int q = 0; q < 2; ++q) {
      long long v = s[q][src][tid];
      if (tid >= d) v += s[q][src][tid - d];
      s[q][1 - src][tid] = v;
    }
    __syncthreads();
    src = 1 - src;
  }
  long long boff = s[0][src][tid] - nbr, uoff = s[1][src][tid] - nbu;
  for (int r = lo; r < hi; ++r) {
    Roi& R = out[r];
    const long long nb = R.status == 0 ? (long long)R.nzc * R.bpz : 0;
    R.brick_begin = boff;
    R.brick_end = boff + nb;
    roi_set_buckets(R, uoff);
    boff += nb;
    uoff += roi_buckets(R.d);
  }
  if (tid == 1023) {
    plan[0] = s[0][src][1023];
    plan[1] = s[1][src][1023];
  }
}

// One ROI descriptor passed by value (no host staging buffer).
__global__ void k_set_roi(Roi R, Roi* __restrict__ out) {
  if (threadIdx.x == 0) *out = R;
}

// ---------------------------------------------------------------------------
// Launchers.

// (rows of SHAPE3D_MAX_DIM2 voxels: 46 KB beside the soft pass's 28 KB of static
// LDS, of the 160 KB of a CU)
size_t mesh_lds_bytes(int max_G) { return sizeof(uint32_t) * (size_t)(kTZ + 1) * (kBrickThreads + 1 + max_G); }

hipError_t launch_mesh_pass(int dtype, Roi* rois, int n_rois, long long nbricks, int max_G,
                            double* case_area, BrickPart* part, unsigned int* counters, int n_counters,
                            unsigned long long* tmpkey, double* tmpt, long long tmp_cap, long long* totals,
                            int moments, int* bmap, float4* pbox, const VolumeBits* vb, const Roi* one,
                            hipStream_t st) {
  if (n_rois < 2) bmap = nullptr;  // one ROI: the search is free
  int* const bitmap = vb && n_rois > 1 ? vb->map : nullptr;
  Roi R;
  if (one)
    R = *one;
  else
    memset(&R, 0, sizeof(R));
  hipLaunchKernelGGL(k_head, dim3((unsigned)(n_rois + (bmap ? kBrickMapTailGroups : 0))), dim3(256), 0, st, rois,
                     n_rois, nbricks, dtype == 0 ? case_area : (double*)nullptr, bmap, counters, n_counters, totals,
                     bitmap, vb ? vb->n_blocks : 0ll, R, one ? 1 : 0);
  if (nbricks <= 0) return hipGetLastError();
  const size_t lds = mesh_lds_bytes(max_G);
  const uint32_t* bits = nullptr;
  if (vb) {
    const auto pack = vb->rounds == 1 ? k_volume_bits<1> : k_volume_bits<kBitRounds>;
    hipLaunchKernelGGL(pack, dim3((unsigned)vb->n_blocks), dim3(256), 0, st, (const Roi*)rois, (const int*)bitmap,
                       vb->bits);
    bits = vb->bits;
  }
  const auto pass = dtype == 0 ? k_mesh_pass<0, false> : vb ? k_mesh_pass<1, true> : k_mesh_pass<1, false>;
  hipLaunchKernelGGL(pass, dim3((unsigned)nbricks), dim3(kBrickThreads), lds, st, (const Roi*)rois, n_rois, nbricks,
                     case_area, part, tmpkey, tmpt, tmp_cap, totals, moments, (const int*)bmap, pbox, bits);
  return hipGetLastError();
}

hipError_t launch_small_head(int dtype, const Roi& R, Roi* rois, long long* totals, SmallAcc* acc,
                             double* case_area, hipStream_t st) {
  hipLaunchKernelGGL(k_small_head, dim3(1), dim3(256), 0, st, R, rois, totals, acc,
                     dtype == 0 ? case_area : (double*)nullptr);
  return hipGetLastError();
}

hipError_t launch_mesh_core(int dtype, const Roi* rois, int n_rois, long long nbricks, int max_G,
                            double* case_area, BrickPart* part, unsigned long long* tmpkey, double* tmpt,
                            long long tmp_cap, long long* totals, int moments, hipStream_t st) {
  if (nbricks <= 0) return hipGetLastError();
  const size_t lds = mesh_lds_bytes(max_G);
  const auto pass = dtype == 0 ? k_mesh_pass<0, false> : k_mesh_pass<1, false>;
  hipLaunchKernelGGL(pass, dim3((unsigned)nbricks), dim3(kBrickThreads), lds, st, rois, n_rois, nbricks, case_area, part,
                     tmpkey, tmpt, tmp_cap, totals, moments, (const int*)nullptr, (float4*)nullptr,
                     (const uint32_t*)nullptr);
  return hipGetLastError();
}

static void totals_kernel(const Roi* rois, int n_rois, int dtype, const double* case_area, const BrickPart* part,
                          long long* brick_voff, RoiMeta* meta, long long* totals, int moments, const BlockIndex& X,
                          hipStream_t st) {
  if (n_rois <= 64)
    hipLaunchKernelGGL(k_mesh_totals<1024>, dim3(n_rois), dim3(1024), 0, st, rois, n_rois, dtype, case_area, part,
                       brick_voff, meta, totals, moments, X);
  else
    hipLaunchKernelGGL(k_mesh_totals<256>, dim3(n_rois), dim3(256), 0, st, rois, n_rois, dtype, case_area, part,
                       brick_voff, meta, totals, moments, X);
}

hipError_t launch_mesh_totals(const Roi* rois, int n_rois, int dtype, const double* case_area, const BrickPart* part,
                              long long* brick_voff, RoiMeta* meta, long long* totals, int moments, int prune_min_v,
                              hipStream_t st) {
  totals_kernel(rois, n_rois, dtype, case_area, part, brick_voff, meta, totals, moments, BlockIndex{}, st);
  hipLaunchKernelGGL(k_roi_rows, dim3(1), dim3(1024), 0, st, n_rois, meta, totals, prune_min_v);
  return hipGetLastError();
}

hipError_t launch_block_totals(const Roi* rois, int n_rois, int dtype, const double* case_area, const BrickPart* part,
                               RoiMeta* meta, long long* totals, int moments, const BlockIndex& X, hipStream_t st) {
  totals_kernel(rois, n_rois, dtype, case_area, part, nullptr, meta, totals, moments, X, st);
  return hipGetLastError();
}

hipError_t launch_mesh_rows(const Roi* rois, int n_rois, long long nbricks, const BrickPart* part,
                            const long long* brick_voff, RoiMeta* meta, long long* totals, long long rows0_cap,
                            const unsigned long long* tmpkey, const double* tmpt, long long tmp_cap,
                            unsigned long long* key, double* tsoft, float* pos, uint4* posh, int* orig, int* blkseg,
                            Seg* segs, unsigned int* overflow, const int* bmap, hipStream_t st) {
  hipLaunchKernelGGL(k_check_capacity, dim3(1), dim3(1024), 0, st, n_rois, rows0_cap, meta, totals, overflow, segs);
  if (nbricks > 0)
    hipLaunchKernelGGL(k_mesh_rows, dim3((unsigned)nbricks), dim3(256), 0, st, rois, n_rois, nbricks, part,
                       brick_voff, meta, tmpkey, tmpt, tmp_cap, key, tsoft, pos, posh, orig, blkseg, overflow,
                       n_rois < 2 ? nullptr : bmap);
  return hipGetLastError();
}

hipError_t launch_plan_rois(const RoiDesc* in, int n, int dtype, const long long max_dims[3], const void* base,
                            long long alloc_elems, Roi* out, long long* plan, hipStream_t st) {
  hipLaunchKernelGGL(k_plan_rois, dim3(1), dim3(1024), 0, st, in, n, dtype, max_dims[0], max_dims[1], max_dims[2],
                     (const char*)base, alloc_elems, out, plan);
  return hipGetLastError();
}

hipError_t launch_set_roi(const Roi& R, Roi* out, hipStream_t st) {
  hipLaunchKernelGGL(k_set_roi, dim3(1), dim3(64), 0, st, R, out);
  return hipGetLastError();
}

}  // namespace s3d

