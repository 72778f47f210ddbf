// labels.hip -- input preprocessing on the device: the bounding box and voxel
// count of every label of a uint8 label map in one read of the map, written
// as a device ROI table (crop to the box, select the label) that the batched
// pipeline consumes directly.  The paper leaves reading and staging the
// input on the host as its open problem (Sec. 3, discussion of the results,
// and the transfer column of Table 2); this keeps that step on the GPU.
#include <climits>

#include "s3d_device.h"
#include "s3d_launch.h"

namespace s3d {

namespace {

constexpr int kLabelThreads = 1024;

// The box under construction for one label: per-thread registers first, then
// the workgroup's LDS entry, then the global one.
struct RegBox {
  int l;  // 0 = empty
  int lo[3], hi[3];
  unsigned long long n;
};

__device__ inline void flush_box(RegBox& b, int* s_lo, int* s_hi, unsigned long long* s_n) {
  if (b.l) {
    const int i = b.l - 1;
    for (int k = 0; k < 3; ++k) {
      atomicMin(&s_lo[3 * i + k], b.lo[k]);
      atomicMax(&s_hi[3 * i + k], b.hi[k]);
    }
    atomicAdd(&s_n[i], b.n);
  }
  b.l = 0;
}

__device__ inline void add_run(RegBox& b, int l, int z, int y, int x0, int x1, unsigned long long n, int* s_lo,
                               int* s_hi, unsigned long long* s_n) {
  if (l != b.l) {
    flush_box(b, s_lo, s_hi, s_n);
    b.l = l;
    b.lo[0] = z;
    b.lo[1] = y;
    b.lo[2] = x0;
    b.hi[0] = z;
    b.hi[1] = y;
    b.hi[2] = x1;
    b.n = n;
    return;
  }
  b.lo[0] = min(b.lo[0], z);
  b.lo[1] = min(b.lo[1], y);
  b.lo[2] = min(b.lo[2], x0);
  b.hi[0] = max(b.hi[0], z);
  b.hi[1] = max(b.hi[1], y);
  b.hi[2] = max(b.hi[2], x1);
  b.n += n;
}

// Row-major coordinates of voxel j (0 <= j < d0 d1 d2): floating-point
// quotients, corrected by one step either way (j < 2^53).
__device__ inline void voxel_coords(long long j, long long d12, int d1, int d2, double inv12, double inv2, int& z,
                                    int& y, int& x) {
  long long q = (long long)((double)j * inv12);
  if (q * d12 > j) --q;
  if ((q + 1) * d12 <= j) ++q;
  const long long r = j - q * d12;
  long long p = (long long)((double)r * inv2);
  if (p * d2 > r) --p;
  if ((p + 1) * d2 <= r) ++p;
  z = (int)q;
  y = (int)p;
  x = (int)(r - p * d2);
}

// The boxes under construction live in the first 32 bytes of the output
// table's entries (an 80-byte RoiDesc per label), so the pass needs no
// memory of its own; the table kernel replaces each by the finished entry.
__device__ inline LabelAcc* acc_of(RoiDesc* tab, int i) { return reinterpret_cast<LabelAcc*>(tab + i); }

}  // namespace

// Clears the boxes of labels 1..max_label.
__global__ void k_label_init(RoiDesc* __restrict__ tab, int max_label) {
  const int i = threadIdx.x;
  if (i < max_label) {
    LabelAcc* a = acc_of(tab, i);
    for (int k = 0; k < 3; ++k) {
      a->lo[k] = INT_MAX;
      a->hi[k] = -1;
    }
    a->n = 0ull;
  }
}

// Bit b set for each byte b of the chunk that differs from l.
__device__ inline uint32_t differs(const uint4& w, uint32_t l) {
  const uint32_t r = l * 0x01010101u;
  return nz8(w.x ^ r, w.y ^ r) >> 7 | nz8(w.z ^ r, w.w ^ r) << 1;
}

// One read of the map in 16-byte chunks, addressed from the 16-byte aligned
// address at or below lab (of the chunks at its ends only the map's own bytes),
// kAhead of them in flight per thread.
// A chunk is taken row by row (one row, two at a row's end) and label by label:
// its first label left, all voxels of that label at once as a 16-bit mask.  Each
// thread keeps the box of its current label in registers and folds it into the
// workgroup's LDS boxes when the label changes; the workgroup's boxes go to
// memory with atomics per label present (the minima and maxima only where they
// still move the box).  Bound: latency of the few rounds of loads, and those
// atomics (24 labels of 181 x 384 x 384, 27 MB: 33 us; 83 with 815 workgroups
// whose chunks lay all over the map, most of it their atomics on the same words).
constexpr int kAhead = 4;

__global__ __launch_bounds__(kLabelThreads) void k_label_boxes(const unsigned char* __restrict__ lab, long long n,
                                                               int mis, long long d12, int d1, int d2, double inv12,
                                                               double inv2, int max_label,
                                                               RoiDesc* __restrict__ tab) {
  __shared__ int s_lo[255 * 3], s_hi[255 * 3];
  __shared__ unsigned long long s_n[255];
  for (int i = threadIdx.x; i < max_label; i += kLabelThreads) {
    for (int k = 0; k < 3; ++k) {
      s_lo[3 * i + k] = INT_MAX;
      s_hi[3 * i + k] = -1;
    }
    s_n[i] = 0ull;
  }
  __syncthreads();
  RegBox b;
  b.l = 0;
  const unsigned char* p0 = lab - mis;
  const long long nchunks = (n + mis + 15) >> 4;
  // a contiguous share of the map per workgroup
  const long long share = (nchunks + gridDim.x - 1) / gridDim.x, end = min(nchunks, (blockIdx.x + 1) * share);
  for (long long c0 = blockIdx.x * share + threadIdx.x; c0 < end; c0 += kAhead * kLabelThreads) {
    uint4 ahead[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const long long c = c0 + u * kLabelThreads;
      const long long j0 = c * 16 - mis;
      ahead[u] = c < end && j0 >= 0 && j0 + 16 <= n ? *(const uint4*)(p0 + c * 16) : make_uint4(0u, 0u, 0u, 0u);
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const long long c = c0 + u * kLabelThreads, j0 = c * 16 - mis;
      if (c < end && (j0 < 0 || j0 + 16 > n)) {
        uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int k = 0; k < 16; ++k)
          if (j0 + k >= 0 && j0 + k < n) w[k >> 2] |= (uint32_t)p0[c * 16 + k] << (8 * (k & 3));
        ahead[u] = make_uint4(w[0], w[1], w[2], w[3]);
      }
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const uint4 w = ahead[u];
      const long long j0 = (c0 + u * kLabelThreads) * 16 - mis;  // voxel index of the chunk's first byte
      int k = j0 < 0 ? (int)(-j0) : 0;
      uint32_t live = differs(w, 0u) & (0xffffu << k);  // (nothing past the share: zeros)
      if (n - j0 < 16) live &= n > j0 ? (1u << (int)(n - j0)) - 1u : 0u;
      if (!live) continue;
      int z, y, x;
      voxel_coords(j0 + k, d12, d1, d2, inv12, inv2, z, y, x);
      for (;;) {  // bytes k .. k + len - 1 are the voxels x .. x + len - 1 of row (z, y)
        const int len = min(16 - k, d2 - x);
        const uint32_t row = ((1u << len) - 1u) << k;
        uint32_t left = live & row;
        while (left) {
          const int b0 = __ffs((int)left) - 1;
          const unsigned long long half = b0 < 8 ? (unsigned long long)w.y << 32 | w.x : (unsigned long long)w.w << 32 | w.z;
          const int l = (int)(half >> (8 * (b0 & 7)) & 0xffull);
          const uint32_t same = left & ~differs(w, (uint32_t)l);
          left &= ~same;
          if (l <= max_label)
            add_run(b, l, z, y, x + b0 - k, x + 31 - __clz((int)same) - k, (unsigned long long)__popc(same), s_lo, s_hi,
                    s_n);
        }
        live &= ~row;
        if (!live) break;
        k += len;
        x = 0;
        if (++y == d1) {
          y = 0;
          ++z;
        }
      }
    }
  }
  flush_box(b, s_lo, s_hi, s_n);
  __syncthreads();
  for (int i = threadIdx.x; i < max_label; i += blockDim.x) {
    if (s_n[i] == 0ull) continue;
    LabelAcc* a = acc_of(tab, i);
    for (int k = 0; k < 3; ++k) {
      if (s_lo[3 * i + k] < __hip_atomic_load(&a->lo[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMin(&a->lo[k], s_lo[3 * i + k]);
      if (s_hi[3 * i + k] > __hip_atomic_load(&a->hi[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(&a->hi[k], s_hi[3 * i + k]);
    }
    atomicAdd(&a->n, s_n[i]);
  }
}

// The ROI table (one workgroup): label l's entry crops the map to the label's
// box; a label with no voxel gets a 1-voxel crop at the origin (which then
// holds no voxel of it).  max_dims: the largest crop along each axis.
__global__ void k_label_table(RoiDesc* __restrict__ rois, int max_label, long long d1, long long d2, double s0,
                              double s1, double s2, long long* __restrict__ counts,
                              long long* __restrict__ max_dims) {
  __shared__ int s_max[3];
  const int i = threadIdx.x;
  if (i < 3) s_max[i] = 1;
  __syncthreads();
  if (i < max_label) {
    const LabelAcc a = *acc_of(rois, i);  // read before the entry is overwritten
    RoiDesc R;
    R.spacing[0] = s0;
    R.spacing[1] = s1;
    R.spacing[2] = s2;
    R.strides[0] = d1 * d2;
    R.strides[1] = d2;
    R.label = i + 1;
    R.reserved = 0;
    if (a.n == 0ull) {
      R.offset = 0;
      for (int k = 0; k < 3; ++k) R.dims[k] = 1;
    } else {
      R.offset = (long long)a.lo[0] * d1 * d2 + (long long)a.lo[1] * d2 + a.lo[2];
      for (int k = 0; k < 3; ++k) {
        R.dims[k] = (long long)(a.hi[k] - a.lo[k] + 1);
        atomicMax(&s_max[k], a.hi[k] - a.lo[k] + 1);
      }
    }
    rois[i] = R;
    if (counts) counts[i] = (long long)a.n;
  }
  __syncthreads();
  if (max_dims && i < 3) max_dims[i] = s_max[i];
}

hipError_t launch_label_rois(const unsigned char* lab, const long long dims[3], const double spacing[3],
                             int max_label, RoiDesc* rois, long long* counts, long long* max_dims, int cu_count,
                             hipStream_t st) {
  hipLaunchKernelGGL(k_label_init, dim3(1), dim3(256), 0, st, rois, max_label);
  const long long n = dims[0] * dims[1] * dims[2];
  const int mis = (int)((uintptr_t)lab & 15);
  const long long nchunks = (n + mis + 15) >> 4;
  // one workgroup per CU (its share's labels are few, and their boxes go to
  // memory once), or one chunk per thread of a small map
  const long long grid = std::max(1ll, std::min((nchunks + kLabelThreads - 1) / kLabelThreads, (long long)cu_count));
  const long long d12 = dims[1] * dims[2];
  hipLaunchKernelGGL(k_label_boxes, dim3((unsigned)grid), dim3(kLabelThreads), 0, st, lab, n, mis, d12,
                     (int)dims[1], (int)dims[2], 1.0 / (double)d12, 1.0 / (double)dims[2], max_label, rois);
  hipLaunchKernelGGL(k_label_table, dim3(1), dim3(256), 0, st, rois, max_label, dims[1], dims[2], spacing[0],
                     spacing[1], spacing[2], counts, max_dims);
  return hipGetLastError();
}

}  // namespace s3d
