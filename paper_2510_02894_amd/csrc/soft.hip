// soft.hip -- adjoint of the soft-mask (probability) forward pass.
//
// L = sum_f g_f F_f over the six features.  The vertex on crossing edge
// (u, u + e_a) sits at x = (u + t e_a) * s with t = (0.5 - p_u) / (p_b - p_u), so
//   dL/dp_w = sum over crossing edges incident to voxel w of
//             (dL/dx_v)_a * s_a * dt/dp_w,
//   dt/dp_u = (0.5 - p_b) / (p_b - p_u)^2,  dt/dp_b = -(0.5 - p_u) / (p_b - p_u)^2.
// dL/dx_v gathers, over the triangles of the four cubes around the edge that
// contain v (a the vertex, b and c the next ones in the triangle's order):
//   area:   g_area * 1/2 * nhat x (c - b)
//   volume: g_vol * sign(SV) * (b' x c') / 6   (primes: relative to the array
//           centre, the origin of the signed sum)
// plus the diameter subgradient g_f (x_v - x_other) / D_f when v is an end
// point of the maximising pair of feature f.
//
// Passes over every ROI of a table, one of them over the volume:
//   1. k_soft_bits reads the probabilities once as inside bits and writes the
//      zeros of dL/dp (bound: HBM, 4 bytes in and 4 out per voxel, 5.1 TB/s); k_soft_scan
//      lists the active cubes and the voxels at a crossing edge from the bits; a
//      dense index gives each active cube's place in its list;
//   2. k_soft_cubes, a thread per active cube: its triangles once each, and
//      per crossing cube edge the component of their gradient along the edge.
//      Bound: FP64 VALU; a thread per edge that visits the four cubes around it
//      evaluates every triangle three times (5,440 instructions an edge);
//      k_soft_diam then adds the diameters' terms to the ends of their pairs;
//   3. k_soft_edges sums each crossing edge over its four cubes, in a fixed order,
//      into (dL/dx_v)_a s_a / (p_b - p_u)^2, three floats per active cube (sums and
//      values edge by edge, since neighbouring cubes along a row are neighbours in
//      the list: with a cube's 12 side by side this pass took 349 us);
//   4. k_soft_voxels, a thread per listed voxel: the terms of its (at most six)
//      crossing edges, the edge's value times 0.5 - p_b or -(0.5 - p_u).
//      Bound: latency of scattered reads, all of a voxel's in flight at once.
// No float atomics: the result does not depend on scheduling.
// Measured on a batch of 256 soft ROIs of edges 48 to 160 (us): bits 424, scan 360, cubes 364,
// edges 310, voxels 207, in all 1,665, against 2,408 of a wave per cube row that
// listed the edges (540), a thread per edge (1,064) and a gather over all voxels
// (804).
#include <hip/hip_runtime.h>

#include <algorithm>

#define MC_TABLE_QUAL __constant__ const
#include "mc_table.h"
#include "s3d_device.h"
#include "s3d_launch.h"

namespace s3d {

namespace {

enum { C_EDGES = 0, C_CUBES = 1, C_VOX = 2, C_BOTH = 3 };  // SoftBwdBufs::counters

struct D3 {
  double x, y, z;
};

__device__ inline D3 sub3(const D3& a, const D3& b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ inline D3 cross3(const D3& a, const D3& b) {
  return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
__device__ inline double axis_of(const D3& v, int a) { return a == 0 ? v.x : (a == 1 ? v.y : v.z); }

__device__ inline double pval(const float* p, const int* d, int z, int y, int x) {
  if (z < 0 || y < 0 || x < 0 || z >= d[0] || y >= d[1] || x >= d[2]) return 0.0;
  return (double)p[((size_t)z * d[1] + y) * (size_t)d[2] + x];
}

// Position (relative to the origin o) of the vertex on the edge from voxel u
// along axis a.
__device__ inline void vertex_pos(const float* p, const int* d, const double* s, const double* o, int u0, int u1,
                                  int u2, int a, double* x) {
  const double pa = pval(p, d, u0, u1, u2);
  const double pb = pval(p, d, u0 + (a == 0), u1 + (a == 1), u2 + (a == 2));
  const double t = (0.5 - pa) / (pb - pa);
  x[0] = ((double)u0 + (a == 0 ? t : 0.0)) * s[0] - o[0];
  x[1] = ((double)u1 + (a == 1 ? t : 0.0)) * s[1] - o[1];
  x[2] = ((double)u2 + (a == 2 ? t : 0.0)) * s[2] - o[2];
}

// p at (z, y, x), 0 outside the array; the load is always issued (at a
// clamped address) so that several of them are in flight together.
__device__ inline float pld(const float* p, const int* d, int z, int y, int x) {
  const bool ok = (unsigned)z < (unsigned)d[0] && (unsigned)y < (unsigned)d[1] && (unsigned)x < (unsigned)d[2];
  const int zc = min(max(z, 0), d[0] - 1), yc = min(max(y, 0), d[1] - 1), xc = min(max(x, 0), d[2] - 1);
  const float v = p[((size_t)zc * d[1] + yc) * (size_t)d[2] + xc];
  return ok ? v : 0.0f;
}

// Flat index of the cube with min corner u.
__device__ inline long long cube_index(const int* d, int u0, int u1, int u2) {
  return ((long long)(u0 + 1) * (d[1] + 1) + (u1 + 1)) * (long long)(d[2] + 1) + (u2 + 1);
}

// The listed cubes and voxels.
__device__ inline long long listed_cubes(const SoftBwdBufs& B) {
  return min(B.packed ? (long long)((unsigned long long)B.counters[C_BOTH] & 0xffffffffull) : B.counters[C_CUBES],
             B.cap_cubes);
}
__device__ inline long long listed_vox(const SoftBwdBufs& B) {
  return min(B.packed ? (long long)((unsigned long long)B.counters[C_BOTH] >> 32) : B.counters[C_VOX], B.cap_vox);
}

__device__ inline unsigned long long pack_vox(int u0, int u1, int u2) { return pack_key(u0, u1, u2, 0); }
__device__ inline int vox0(unsigned long long k) { return (int)(k >> 40 & 0xFFFFF) - 1; }
__device__ inline int vox1(unsigned long long k) { return (int)(k >> 20 & 0xFFFFF) - 1; }
__device__ inline int vox2(unsigned long long k) { return (int)(k & 0xFFFFF) - 1; }

// Last ROI whose first workgroup of the scan (or of the bit pass) is <= b.
#define S3D_SOFT_ROI_SEARCH(name, member)                               \
  __device__ inline int name(const SoftBwdRoi* r, int n, long long b) { \
    int lo = 0, hi = n - 1;                                             \
    while (lo < hi) {                                                   \
      const int mid = (lo + hi + 1) >> 1;                               \
      if (r[mid].member <= b)                                           \
        lo = mid;                                                       \
      else                                                              \
        hi = mid - 1;                                                   \
    }                                                                   \
    return lo;                                                          \
  }
S3D_SOFT_ROI_SEARCH(soft_roi_of, brick_begin)
S3D_SOFT_ROI_SEARCH(soft_roi_of_bits, bitblk_begin)
#undef S3D_SOFT_ROI_SEARCH

// A wave emits the set bits of its lanes' words, two words at a time, a lane
// per bit: f(bit, list position, base of the word, place of the word) for each.
// off: the lane's next list position, moved past its word.  (Loops of a lane
// over its own bits hold the wave for the fullest word.)
template <typename F>
__device__ inline void emit_words(uint32_t w, int& off, int base, int place, int lane, F&& f) {
  unsigned long long todo = __ballot(w != 0u);
  const int k = lane & 31;
  const bool low = lane < 32;
  while (todo) {
    const int s0 = __ffsll((long long)todo) - 1;
    todo &= todo - 1ull;
    const int s1 = todo ? __ffsll((long long)todo) - 1 : s0;
    const uint32_t w0 = (uint32_t)__builtin_amdgcn_readlane((int)w, s0);
    const uint32_t w1 = todo ? (uint32_t)__builtin_amdgcn_readlane((int)w, s1) : 0u;
    todo &= todo - 1ull;
    const uint32_t word = low ? w0 : w1;
    const int o = low ? __builtin_amdgcn_readlane(off, s0) : __builtin_amdgcn_readlane(off, s1);
    const int bs = low ? __builtin_amdgcn_readlane(base, s0) : __builtin_amdgcn_readlane(base, s1);
    const int pl = low ? __builtin_amdgcn_readlane(place, s0) : __builtin_amdgcn_readlane(place, s1);
    if (word >> k & 1u) f(k, o + __popc(word & ((1u << k) - 1u)), bs, pl);
  }
  off += __popc(w);
}

}  // namespace

// The inside bits of the probabilities and the zeros of dL/dp, a stream.
template <int ROUNDS>
__global__ __launch_bounds__(256) void k_soft_bits(SoftBwdBufs B) {
  const int roi = B.blk_roi ? B.blk_roi[B.n_bricks + blockIdx.x] : soft_roi_of_bits(B.rois, B.n_rois, blockIdx.x);
  const SoftBwdRoi& R = B.rois[roi];
  const long long n = (long long)R.d[0] * R.d[1] * R.d[2];
  const long long e0 = (blockIdx.x - R.bitblk_begin) * (long long)(ROUNDS * kBitRound);
  pack_bits<ROUNDS>(R.p, n, e0, B.bits + R.bits_begin);
  if (odd_floats(R.grad)) {
    const long long e1 = min(n, e0 + ROUNDS * kBitRound);
    for (long long e = e0 + threadIdx.x; e < e1; e += 256) R.grad[e] = 0.0f;
    return;
  }
  // the gradient's elements have their own 16-byte boundary
  const int shift = volume_shift(R.grad);
  float4* out = (float4*)((uintptr_t)R.grad & ~(uintptr_t)15);
#pragma unroll
  for (int u = 0; u < ROUNDS * kBitRound / 1024; ++u) {
    const long long e = e0 + 1024 * u + 4 * threadIdx.x;
    if (e >= shift && e + 4 <= n + shift) {
      out[e >> 2] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    } else {
      for (int k = 0; k < 4; ++k)
        if (e + k >= shift && e + k < n + shift) ((float*)out)[e + k] = 0.0f;
    }
  }
}

// Pass 1.  A workgroup takes 256 consecutive row-groups (rg = cube row * G +
// group of 32 cubes along axis 2) times up to R.tz cube planes, as the mesh
// pass does, and holds the inside words of their voxels and of one more row and
// plane on either side: tile word (p, i) is the row-group rg0 - 1 + i of voxel
// plane pz0 - 1 + p.
__global__ __launch_bounds__(256) void k_soft_scan(SoftBwdBufs B) {
  extern __shared__ uint32_t s_bits[];
  __shared__ int s_scan[4];
  __shared__ long long s_base[2];
  const int roi = B.blk_roi ? B.blk_roi[blockIdx.x] : soft_roi_of(B.rois, B.n_rois, blockIdx.x);
  const SoftBwdRoi& R = B.rois[roi];
  const int d0 = R.d[0], d1 = R.d[1], d2 = R.d[2], G = R.G;
  const int local = (int)(blockIdx.x - R.brick_begin);
  const int rg0 = local / R.nzc * 256, pz0 = local % R.nzc * R.tz;
  const int nz = min(R.tz, d0 + 1 - pz0);  // cube planes
  const int np = nz + 2, nw = 258 + 2 * G;
  const int tid = threadIdx.x, lane = tid & 63;
  cut_tile<kTZ + 2>(B.bits + R.bits_begin, volume_shift(R.p), R.d, G, R.mG, R.shG, rg0 - 1, pz0 - 1, np, nw, s_bits);
  __syncthreads();

  const int rg = rg0 + tid;
  const bool valid = rg < R.nrg;
  const int ry = valid ? (int)fdiv((unsigned int)rg, R.mG, R.shG) : 0;
  const int l = valid ? rg - ry * G : 0;
  const int kmax = d2 - 32 * l;  // cubes 0 .. kmax of the group, voxels 0 .. kmax - 1
  const uint32_t cmask = !valid ? 0u : (kmax >= 31 ? 0xffffffffu : (1u << (kmax + 1)) - 1u);
  const uint32_t vmask = !valid || ry >= d1 ? 0u : (kmax >= 32 ? 0xffffffffu : (1u << kmax) - 1u);
  uint32_t act[kTZ], vox[kTZ];
  int n_c = 0, n_v = 0, n_e = 0;
#pragma unroll
  for (int p = 0; p < kTZ; ++p) {
    act[p] = 0u;
    vox[p] = 0u;
    if (p >= nz || !valid) continue;
    const uint32_t* w0 = s_bits + p * nw + tid + 1;  // plane z, row y
    const uint32_t* w1 = w0 + nw;                    // plane z + 1
    const uint32_t r00 = w0[0], r01 = w0[G], r10 = w1[0], r11 = w1[G];
    const uint32_t a00 = shifted(r00, w0[-1]), a01 = shifted(r01, w0[G - 1]);
    const uint32_t a10 = shifted(r10, w1[-1]), a11 = shifted(r11, w1[G - 1]);
    act[p] = (a00 | r00 | a01 | r01 | a10 | r10 | a11 | r11) & ~(a00 & r00 & a01 & r01 & a10 & r10 & a11 & r11) & cmask;
    n_e += __popc((a00 ^ a10) & cmask) + __popc((a00 ^ a01) & cmask) + __popc((a00 ^ r00) & cmask);
    // the voxel row (z + 1, y + 1) against its six neighbours
    const uint32_t next = l + 1 < G ? w1[G + 1] << 31 : 0u;
    vox[p] = ((r11 ^ a11) | (r11 ^ (r11 >> 1 | next)) | (r11 ^ r10) | (r11 ^ w1[2 * G]) | (r11 ^ r01) |
              (r11 ^ w1[nw + G])) &
             (pz0 + p < d0 ? vmask : 0u);
    n_c += __popc(act[p]);
    n_v += __popc(vox[p]);
  }
  int total_c, total_v, total_e;
  int off_c = block_excl_scan256(n_c, s_scan, total_c);
  int off_v = block_excl_scan256(n_v, s_scan, total_v);
  (void)block_excl_scan256(n_e, s_scan, total_e);
  if (tid == 0) {
    unsigned long long* ctr = (unsigned long long*)B.counters;
    if (total_e) atomicAdd(&ctr[C_EDGES], (unsigned long long)total_e);
    // one reservation for both lists (one round trip less on the workgroup's
    // critical path), unless a count could pass 32 bits
    if (B.packed) {
      const unsigned long long both = (unsigned long long)total_v << 32 | (unsigned int)total_c;
      const unsigned long long got = both ? atomicAdd(&ctr[C_BOTH], both) : 0ull;
      s_base[0] = (long long)(got & 0xffffffffull);
      s_base[1] = (long long)(got >> 32);
    } else {
      s_base[0] = total_c ? (long long)atomicAdd(&ctr[C_CUBES], (unsigned long long)total_c) : 0;
      s_base[1] = total_v ? (long long)atomicAdd(&ctr[C_VOX], (unsigned long long)total_v) : 0;
    }
  }
  __syncthreads();
  const long long base_c = s_base[0], base_v = s_base[1];
  // a word's place, and the flat index of its first cube in plane pz0
  const int place = ry | l << 20;
  const int cube0 = (pz0 * (d1 + 1) + ry) * (d2 + 1) + 32 * l, cplane = (d1 + 1) * (d2 + 1);
  unsigned int* index = B.index + R.cube_begin;
#pragma unroll
  for (int p = 0; p < kTZ; ++p) {
    emit_words(act[p], off_c, cube0 + p * cplane, place, lane, [&](int k, int at, int cube, int pl) {
      const long long idx = base_c + at;
      if (idx >= B.cap_cubes) return;  // more cubes than the forward pass's vertices allow: the call fails
      B.cubes[idx] = pack_vox(pz0 - 1 + p, (pl & 0xfffff) - 1, 32 * (pl >> 20) - 1 + k);
      B.croi[idx] = roi;
      index[cube + k] = (unsigned int)idx;
    });
    emit_words(vox[p], off_v, 0, place, lane, [&](int k, int at, int, int pl) {
      const long long idx = base_v + at;
      if (idx >= B.cap_vox) return;
      B.vox[idx] = pack_vox(pz0 + p, pl & 0xfffff, 32 * (pl >> 20) + k);
      B.vroi[idx] = roi;
    });
  }
}

// Pass 2.  A thread per active cube; its corner values and the sums of its 12
// edges in LDS (indexed at run time).
constexpr int kCubeThreads = 256;

__global__ __launch_bounds__(kCubeThreads, 4) void k_soft_cubes(SoftBwdBufs B) {
  __shared__ double s_g[12][kCubeThreads];
  __shared__ float s_p[8][kCubeThreads];
  __shared__ uint8_t s_tri[256 * MC_MAX_TRI * 3];
  __shared__ uint8_t s_nt[256];
  __shared__ uint32_t s_edge[12];  // axis | corner 0 << 2 | corner 1 << 5
  const int tid = threadIdx.x;
  for (int i = tid; i < 256 * MC_MAX_TRI * 3; i += blockDim.x) s_tri[i] = (&MC_TRI[0][0][0])[i];
  for (int i = tid; i < 256; i += blockDim.x) s_nt[i] = MC_NTRI[i];
  if (tid < 12) {
    const uint32_t a = MC_EDGE_AXIS[tid], k0 = MC_EDGE_C0[tid];
    s_edge[tid] = a | k0 << 2 | (k0 | 4u >> a) << 5;
  }
  __syncthreads();
  const long long n = listed_cubes(B);
  for (long long i = (long long)blockIdx.x * blockDim.x + tid; i < n; i += (long long)gridDim.x * blockDim.x) {
    const unsigned long long key = B.cubes[i];
    const SoftBwdRoi& R = B.rois[B.croi[i]];
    const int u0 = vox0(key), u1 = vox1(key), u2 = vox2(key);
    float pc[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) pc[k] = pld(R.p, R.d, u0 + (k >> 2 & 1), u1 + (k >> 1 & 1), u2 + (k & 1));
    int cas = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      cas |= (int)(pc[k] > 0.5f) << k;
      s_p[k][tid] = pc[k];
    }
#pragma unroll
    for (int e = 0; e < 12; ++e) s_g[e][tid] = 0.0;
    const double ga = 0.5 * R.g_area, gv = R.g_vol_signed / 6.0;
    const double sx = R.s[0], sy = R.s[1], sz = R.s[2];
    const double bx = (double)u0 * sx - R.o[0], by = (double)u1 * sy - R.o[1], bz = (double)u2 * sz - R.o[2];
    auto vertex = [&](uint32_t ed) -> D3 {
      const int ax = (int)(ed & 3u), k0 = (int)(ed >> 2 & 7u), k1 = (int)(ed >> 5);
      const double p0 = (double)s_p[k0][tid], p1 = (double)s_p[k1][tid];
      const double t = (0.5 - p0) * rcp64(p1 - p0);
      return {bx + (ax == 0 ? t : (double)(k0 >> 2 & 1)) * sx, by + (ax == 1 ? t : (double)(k0 >> 1 & 1)) * sy,
              bz + (ax == 2 ? t : (double)(k0 & 1)) * sz};
    };
    const int nt = s_nt[cas];
    for (int t = 0; t < nt; ++t) {
      const uint8_t* tr = s_tri + (cas * MC_MAX_TRI + t) * 3;
      const int e0 = tr[0], e1 = tr[1], e2 = tr[2];
      const uint32_t d0 = s_edge[e0], d1 = s_edge[e1], d2 = s_edge[e2];
      const D3 P0 = vertex(d0), P1 = vertex(d1), P2 = vertex(d2);
      const D3 n3 = cross3(sub3(P1, P0), sub3(P2, P0));
      const double len = sqrt(n3.x * n3.x + n3.y * n3.y + n3.z * n3.z);
      // no area, or one out of range, or NaN: the area term is left out
      const bool flat = !(len > 0.0 && len < __builtin_huge_val());
      const double il = ga * rcp64(len);
      const D3 nh = {n3.x * il, n3.y * il, n3.z * il};
      // the vertex's own edge axis of ga nhat x (c - b) + gv b x c
      auto term = [&](const D3& b, const D3& c, uint32_t ed) {
        const D3 r = cross3(nh, sub3(c, b)), q = cross3(b, c);
        const int ax = (int)(ed & 3u);
        return (flat ? 0.0 : axis_of(r, ax)) + gv * axis_of(q, ax);
      };
      s_g[e0][tid] += term(P1, P2, d0);
      s_g[e1][tid] += term(P2, P0, d1);
      s_g[e2][tid] += term(P0, P1, d2);
    }
    double* out = B.cgrad + i;
#pragma unroll
    for (int e = 0; e < 12; ++e) {
      constexpr uint8_t c0[12] = {0, 1, 2, 3, 0, 1, 4, 5, 0, 2, 4, 6};
      const int k0 = c0[e], k1 = k0 | 4 >> (e >> 2);
      if ((cas >> k0 ^ cas >> k1) & 1) out[e * B.cap_cubes] = s_g[e][tid];
    }
  }
}

// The diameters' terms g_f (x_v - x_other)_a / D_f at both ends of their pairs,
// added to the cube above each end's edge (the first of its four).  Eight lanes
// per ROI, one per end; ends on one edge are summed in lane order by the first.
__global__ __launch_bounds__(64) void k_soft_diam(SoftBwdBufs B) {
  const int lane = threadIdx.x & 63, j = lane & 7, f = j >> 1;
  const int roi = (int)blockIdx.x * 8 + (lane >> 3);
  long long id = -1;
  double term = 0.0;
  long long at = -1;
  if (roi < B.n_rois) {
    const SoftBwdRoi& R = B.rois[roi];
    const double gd = R.gdiam[f];
    if (gd != 0.0) {
      id = R.pair_ids[f][j & 1];
      const long long ids[2] = {id, R.pair_ids[f][1 - (j & 1)]};
      double x[2][3];
      int u[3], a = 0;
      for (int e = 0; e < 2; ++e) {
        const long long lin = ids[e] / 3;
        const int ea = (int)(ids[e] % 3);
        const int e2 = (int)(lin % (R.d[2] + 2)) - 1;
        const long long l2 = lin / (R.d[2] + 2);
        const int e1 = (int)(l2 % (R.d[1] + 2)) - 1, e0 = (int)(l2 / (R.d[1] + 2)) - 1;
        vertex_pos(R.p, R.d, R.s, R.o, e0, e1, e2, ea, x[e]);
        if (e == 0) {
          u[0] = e0;
          u[1] = e1;
          u[2] = e2;
          a = ea;
        }
      }
      term = gd * (x[0][a] - x[1][a]);
      // (a saved context of other probabilities may name an edge outside the grid)
      if (u[0] >= -1 && u[0] < R.d[0] && u[1] >= -1 && u[1] < R.d[1] && u[2] >= -1 && u[2] < R.d[2]) {
        const unsigned int idx = B.index[R.cube_begin + cube_index(R.d, u[0], u[1], u[2])];
        if ((long long)idx < listed_cubes(B)) at = 4 * a * B.cap_cubes + idx;
      }
    }
  }
  double sum = 0.0;
  bool first = true;
  for (int k = 0; k < 8; ++k) {
    const int src = (lane & ~7) + k;
    const long long oid = __shfl(id, src, 64);
    const double ot = __shfl(term, src, 64);
    if (oid == id) {
      sum += ot;
      if (k < j) first = false;
    }
  }
  if (at >= 0 && first) B.cgrad[at] += sum;
}

// Pass 3.  Per active cube and axis, the sum over the four cubes around the
// edge from its min corner (if that edge crosses), in a fixed order.
__global__ __launch_bounds__(256) void k_soft_edges(SoftBwdBufs B) {
  const long long n = listed_cubes(B);
  const unsigned int n_cubes = (unsigned int)n;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    const unsigned long long key = B.cubes[i];
    const SoftBwdRoi& R = B.rois[B.croi[i]];
    const int u0 = vox0(key), u1 = vox1(key), u2 = vox2(key);
    const float f0 = pld(R.p, R.d, u0, u1, u2);
    const float fa[3] = {pld(R.p, R.d, u0 + 1, u1, u2), pld(R.p, R.d, u0, u1 + 1, u2), pld(R.p, R.d, u0, u1, u2 + 1)};
    const long long cs[3] = {(long long)(R.d[1] + 1) * (R.d[2] + 1), R.d[2] + 1, 1};
    const unsigned int* index = B.index + R.cube_begin + cube_index(R.d, u0, u1, u2);
    bool cross[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) cross[a] = (f0 > 0.5f) != (fa[a] > 0.5f);
    // the cubes one step back along one axis (nb[k]) and along the two others than
    // k (nb2[k]); a crossing edge lies inside the grid along its other axes, and so
    // do its cubes
    unsigned int nb[3], nb2[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int b = k == 0 ? 1 : 0, c = k == 2 ? 1 : 2;
      nb[k] = cross[b] || cross[c] ? index[-cs[k]] : ~0u;
      nb2[k] = cross[k] ? index[-cs[b] - cs[c]] : ~0u;
    }
    double part[3][4];
#pragma unroll
    for (int a = 0; a < 3; ++a)
      if (cross[a]) {
        const unsigned int around[3] = {nb[a == 2 ? 1 : 2], nb[a == 0 ? 1 : 0], nb2[a]};
        const double* g = B.cgrad + 4 * a * B.cap_cubes;
        part[a][0] = g[i];
#pragma unroll
        for (int q = 1; q < 4; ++q)
          part[a][q] = around[q - 1] < n_cubes ? g[q * B.cap_cubes + around[q - 1]] : 0.0;
      }
#pragma unroll
    for (int a = 0; a < 3; ++a)
      if (cross[a]) {
        const double den = (double)fa[a] - (double)f0;  // at least one float ulp at 0.5: the edge straddles it
        B.egrad[a * B.cap_cubes + i] =
            (float)((((part[a][0] + part[a][1]) + part[a][2]) + part[a][3]) * R.s[a] / (den * den));
      }
  }
}

// Pass 4.  A thread per voxel at a crossing edge: its edges' values times the
// rest of dt/dp.
__global__ __launch_bounds__(256) void k_soft_voxels(SoftBwdBufs B) {
  const long long n = listed_vox(B);
  const unsigned int n_cubes = (unsigned int)listed_cubes(B);
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    const unsigned long long key = B.vox[i];
    const SoftBwdRoi& R = B.rois[B.vroi[i]];
    const int w[3] = {vox0(key), vox1(key), vox2(key)};
    const size_t at = ((size_t)w[0] * R.d[1] + w[1]) * (size_t)R.d[2] + w[2];
    const size_t step[3] = {(size_t)R.d[1] * R.d[2], (size_t)R.d[2], 1};
    const float vc = R.p[at];
    float nv[6];
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      const int k = j >> 1;
      const bool ok = j & 1 ? w[k] + 1 < R.d[k] : w[k] > 0;
      const float v = R.p[ok ? (j & 1 ? at + step[k] : at - step[k]) : at];
      nv[j] = ok ? v : 0.0f;
    }
    // the cube at each edge's lower end (j & 1: the voxel itself), then the edge
    const unsigned int* index = B.index + R.cube_begin + cube_index(R.d, w[0], w[1], w[2]);
    const long long cs[3] = {(long long)(R.d[1] + 1) * (R.d[2] + 1), R.d[2] + 1, 1};
    bool cross[6], any_up = false;
    unsigned int idx[6], here = 0u;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      cross[j] = (nv[j] > 0.5f) != (vc > 0.5f);
      any_up |= cross[j] && (j & 1);
      idx[j] = ~0u;
      if (cross[j] && !(j & 1)) idx[j] = index[-cs[j >> 1]];
    }
    if (any_up) here = *index;
    float e[6];
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      e[j] = 0.0f;
      const unsigned int c = j & 1 ? here : idx[j];
      if (cross[j] && c < n_cubes) e[j] = B.egrad[(j >> 1) * B.cap_cubes + c];
    }
    double g = 0.0;
#pragma unroll
    for (int j = 0; j < 6; ++j)
      if (cross[j]) g += (double)e[j] * (j & 1 ? 0.5 - (double)nv[j] : -(0.5 - (double)nv[j]));
    R.grad[at] = (float)g;
  }
}

// The ROI of every workgroup of the scan and of the bit pass (one workgroup per
// ROI writes its ranges), and the cleared counters.
__global__ void k_soft_head(SoftBwdBufs B) {
  if (blockIdx.x == 0 && threadIdx.x < 4) B.counters[threadIdx.x] = 0;
  if (!B.blk_roi) return;
  const bool last = (int)blockIdx.x + 1 == B.n_rois;
  const SoftBwdRoi& R = B.rois[blockIdx.x];
  const long long e = last ? B.n_bricks : B.rois[blockIdx.x + 1].brick_begin;
  for (long long i = R.brick_begin + threadIdx.x; i < e; i += blockDim.x) B.blk_roi[i] = (int)blockIdx.x;
  const long long eb = last ? B.n_bitblks : B.rois[blockIdx.x + 1].bitblk_begin;
  for (long long i = R.bitblk_begin + threadIdx.x; i < eb; i += blockDim.x) B.blk_roi[B.n_bricks + i] = (int)blockIdx.x;
}

hipError_t launch_soft_backward(const SoftBwdBufs& B, hipStream_t st) {
  auto grid = [&](long long work, int threads, long long per_cu) {
    return dim3((unsigned)std::max(1ll, std::min((work + threads - 1) / threads, per_cu * B.cu_count)));
  };
  hipLaunchKernelGGL(k_soft_head, dim3((unsigned)(B.blk_roi ? B.n_rois : 1)), dim3(256), 0, st, B);
  hipLaunchKernelGGL(B.bit_rounds == 1 ? k_soft_bits<1> : k_soft_bits<kBitRounds>, dim3((unsigned)B.n_bitblks), dim3(256),
                     0, st, B);
  hipLaunchKernelGGL(k_soft_scan, dim3((unsigned)B.n_bricks), dim3(256), B.scan_lds, st, B);
  if (B.cap_cubes > 0) {
    // few cubes: waves of their own, so that they spread over the CUs
    const int threads = B.cap_cubes < 65536 ? 64 : kCubeThreads;
    hipLaunchKernelGGL(k_soft_cubes, grid(B.cap_cubes, threads, 16), dim3(threads), 0, st, B);
    hipLaunchKernelGGL(k_soft_diam, dim3((unsigned)((B.n_rois + 7) / 8)), dim3(64), 0, st, B);
    hipLaunchKernelGGL(k_soft_edges, grid(B.cap_cubes, 256, 32), dim3(256), 0, st, B);
    hipLaunchKernelGGL(k_soft_voxels, grid(B.cap_vox, 256, 32), dim3(256), 0, st, B);
  }
  return hipGetLastError();
}

}  // namespace s3d
