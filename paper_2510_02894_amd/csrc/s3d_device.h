// s3d_device.h -- device helpers shared by the HIP translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "s3d_internal.h"

namespace s3d {

// Maps a workgroup index to a work index so that each of the 8 XCDs (which
// receive workgroups round-robin) walks one contiguous range of work indices:
// neighbouring bricks then share that XCD's L2.  A bijection on [0, n).
__device__ inline long long xcd_remap(long long bid, long long n) {
  const long long per = n / 8, rem = n % 8;
  const long long x = bid % 8, idx = bid / 8;
  return x * per + (x < rem ? x : rem) + idx;
}

// floor(n / d) for 0 <= n < 2^31 from the precomputed pair m = floor(2^sh / d) + 1,
// sh = 31 + ceil(log2 d): (n * m) >> sh (the error term n (m - 2^sh / d) / 2^sh
// stays below 1 / d, so the floor is exact).
__device__ inline unsigned int fdiv(unsigned int n, unsigned int m, int sh) {
  return (unsigned int)(((unsigned long long)n * m) >> sh);
}

// Index of the last ROI whose first brick is <= b (ROIs are sorted by brick_begin).
__device__ inline int find_roi(const Roi* rois, int n, long long b) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (rois[mid].brick_begin <= b)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

template <typename T>
__device__ inline T wave_sum(T v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
  return v;
}

__device__ inline int wave_min(int v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v = min(v, __shfl_xor(v, m, 64));
  return v;
}

__device__ inline int wave_max(int v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v = max(v, __shfl_xor(v, m, 64));
  return v;
}

// Reductions across lanes without LDS traffic (a __shfl_xor is an LDS permute):
// step STEP combines a lane's value with that of another lane of its 2^(STEP+1)
// group, after steps 0 .. STEP - 1 have made the smaller groups uniform: DPP
// quad permutes and row mirrors within 16 lanes, then the row swaps of gfx950.
template <int STEP, typename Op>
__device__ inline uint32_t lane_step(uint32_t v, Op op) {
  static_assert(STEP >= 0 && STEP < 6, "64 lanes");
  if constexpr (STEP < 4) {
    constexpr int ctrl[4] = {0xB1, 0x4E, 0x141, 0x140};  // lane ^ 1, lane ^ 2, half-row mirror, row mirror
    return op(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, ctrl[STEP], 0xf, 0xf, true));
  } else if constexpr (STEP == 4) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return op((uint32_t)r[0], (uint32_t)r[1]);
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return op((uint32_t)r[0], (uint32_t)r[1]);
  }
}

template <int STEP, typename Op>
__device__ inline unsigned long long lane_step(unsigned long long v, Op op) {
  const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  if constexpr (STEP < 4) {
    constexpr int ctrl[4] = {0xB1, 0x4E, 0x141, 0x140};
    const uint32_t ol = (uint32_t)__builtin_amdgcn_mov_dpp((int)lo, ctrl[STEP], 0xf, 0xf, true);
    const uint32_t oh = (uint32_t)__builtin_amdgcn_mov_dpp((int)hi, ctrl[STEP], 0xf, 0xf, true);
    return op(v, (unsigned long long)oh << 32 | ol);
  } else if constexpr (STEP == 4) {
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return op((unsigned long long)(uint32_t)h[0] << 32 | (uint32_t)l[0],
              (unsigned long long)(uint32_t)h[1] << 32 | (uint32_t)l[1]);
  } else {
    const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return op((unsigned long long)(uint32_t)h[0] << 32 | (uint32_t)l[0],
              (unsigned long long)(uint32_t)h[1] << 32 | (uint32_t)l[1]);
  }
}

// Reduction over groups of 2^STEPS consecutive lanes (all lanes active); every
// lane receives its group's value.
template <int STEPS, typename T, typename Op>
__device__ inline T lanes_reduce(T v, Op op) {
  v = lane_step<0>(v, op);
  if constexpr (STEPS > 1) v = lane_step<1>(v, op);
  if constexpr (STEPS > 2) v = lane_step<2>(v, op);
  if constexpr (STEPS > 3) v = lane_step<3>(v, op);
  if constexpr (STEPS > 4) v = lane_step<4>(v, op);
  if constexpr (STEPS > 5) v = lane_step<5>(v, op);
  return v;
}

template <int STEPS>
__device__ inline int lanes_min_i32(int v) {
  return (int)lanes_reduce<STEPS>((uint32_t)v, [](uint32_t a, uint32_t b) { return (uint32_t)min((int)a, (int)b); });
}
template <int STEPS>
__device__ inline int lanes_max_i32(int v) {
  return (int)lanes_reduce<STEPS>((uint32_t)v, [](uint32_t a, uint32_t b) { return (uint32_t)max((int)a, (int)b); });
}

template <int STEPS>
__device__ inline int lanes_sum_i32(int v) {
  return (int)lanes_reduce<STEPS>((uint32_t)v, [](uint32_t a, uint32_t b) { return a + b; });
}

// A float as an integer of the same order (NaN apart), and back.
__device__ inline int float_order(float f) {
  const int b = __float_as_int(f);
  return b ^ ((b >> 31) & 0x7fffffff);
}
__device__ inline float order_float(int b) { return __int_as_float(b ^ ((b >> 31) & 0x7fffffff)); }

// Exclusive prefix sum over a 256-thread block; `total` receives the block sum.
// `sh` must hold 4 ints of shared memory.  Contains barriers.
__device__ inline int block_excl_scan256(int v, int* sh, int& total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  int inc = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    int t = __shfl_up(inc, d, 64);
    if (lane >= d) inc += t;
  }
  if (lane == 63) sh[wid] = inc;
  __syncthreads();
  int base = 0;
  for (int w = 0; w < wid; ++w) base += sh[w];
  total = sh[0] + sh[1] + sh[2] + sh[3];
  __syncthreads();
  return base + inc - v;
}

// 1 / x in FP64 from the hardware reciprocal estimate and two Newton steps
// (each squares the relative error, which ends far below a unit in the last
// place of a double for the estimate's accuracy; the result may differ from the
// correctly rounded quotient in its last bit); x != 0.
__device__ inline double rcp64(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  r = fma(r, fma(-x, r, 1.0), r);
  return r;
}

// Exact FP64 squared distance in a fixed operation order (no contraction).
__device__ inline double dist2_exact(const double* p, const double* q) {
  double dx = __dsub_rn(p[0], q[0]), dy = __dsub_rn(p[1], q[1]), dz = __dsub_rn(p[2], q[2]);
  return __dadd_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)), __dmul_rn(dz, dz));
}

// Physical FP64 position of a vertex from its key and interpolation parameter,
// ((double)u_k + [k == a] * t) * s_k, in that operation order.
__device__ inline void key_position(uint64_t key, double t, const double* s, double* x) {
  const int u2 = (int)(key & 0xFFFFF) - 1;
  const int u1 = (int)((key >> 20) & 0xFFFFF) - 1;
  const int u0 = (int)((key >> 40) & 0xFFFFF) - 1;
  const int a = (int)((key >> 60) & 3);
  x[0] = __dmul_rn(__dadd_rn((double)u0, a == 0 ? t : 0.0), s[0]);
  x[1] = __dmul_rn(__dadd_rn((double)u1, a == 1 ? t : 0.0), s[1]);
  x[2] = __dmul_rn(__dadd_rn((double)u2, a == 2 ? t : 0.0), s[2]);
}

// Binary exponent e of the scale 2^e applied to a ROI's centred coordinates
// before the split-f16 pair pass: with R2 a bound on |x|^2, 64 <= 2^e R < 128,
// so scaled coordinates and |x|^2 (< 2^14) are far inside the f16 range.
__host__ __device__ inline int h_scale_exp(double R2) {
  if (!(R2 > 0.0)) return 0;
  int k;
  (void)frexp(R2, &k);                                  // 2^(k-1) <= R2 < 2^k
  const int half = k >= 0 ? (k + 1) / 2 : -((-k) / 2);  // ceil(k / 2)
  const int e = 7 - half;
  return e < -120 ? -120 : (e > 120 ? 120 : e);
}

// Split-f16 B operand of a row (the pair pass's kernel 1): the centred FP32
// position (x, y, z) and w = |p|^2, scaled by 2^e and 2^(2e), each split into
// h = f16(v) and l = f16(v - h).  A row is 32 contiguous bytes: K entries 0-7
// [h, l, h0, h1] (read by lane row % 32 of the MFMA) and then K entries 8-15
// [h2, 1, 1, w_hi, w_lo, 0, 0, 0] (read by lane 32 + row % 32), so lane l of
// a wave reads uint4 2 (l % 32) + l / 32 of the 32-row block: one contiguous
// 1 KB load per block, and one 32-byte record per row to copy.
typedef _Float16 v8h __attribute__((ext_vector_type(8)));

__device__ inline void write_split_row(uint4* __restrict__ posh, long long row, float fx, float fy, float fz,
                                       float fw, int e) {
  const float x[3] = {ldexpf(fx, e), ldexpf(fy, e), ldexpf(fz, e)};
  const float w = ldexpf(fw, 2 * e);
  _Float16 h[3], l[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    h[c] = (_Float16)x[c];
    l[c] = (_Float16)(x[c] - (float)h[c]);
  }
  const _Float16 wh = (_Float16)w, wl = (_Float16)(w - (float)wh);
  const _Float16 one = (_Float16)1.0f, zero = (_Float16)0.0f;
  const v8h b0 = {h[0], h[1], h[2], l[0], l[1], l[2], h[0], h[1]};
  const v8h b1 = {h[2], one, one, wh, wl, zero, zero, zero};
  uint4* r = posh + 2 * row;
  r[0] = *(const uint4*)&b0;
  r[1] = *(const uint4*)&b1;
}

// uint4 index, within a 32-row block of split-f16 operand rows, that lane l
// passes to the MFMA.
__device__ inline int split_lane_index(int lane) { return 2 * (lane & 31) + (lane >> 5); }

// Copies the pair-pass operands of row src to row dst: the split-f16 B
// operand when posh is set, else the FP32 position block entries.
__device__ inline void copy_row_operands(float* __restrict__ pos, uint4* __restrict__ posh, long long src,
                                         long long dst) {
  if (posh) {
    const uint4* s = posh + 2 * src;
    uint4* d = posh + 2 * dst;
    const uint4 a = s[0], b = s[1];
    d[0] = a;
    d[1] = b;
  } else {
    const float* s = pos + (src >> 4) * 64 + (src & 15);
    float* d = pos + (dst >> 4) * 64 + (dst & 15);
    const float a = s[0], b = s[16], c = s[32], w = s[48];
    d[0] = a;
    d[16] = b;
    d[32] = c;
    d[48] = w;
  }
}

// Canonical id 3 * lin_pad(u) + a of a vertex key for a ROI of dims d.
__device__ inline unsigned long long key_canonical_id(uint64_t key, const int* d) {
  const unsigned long long p2 = key & 0xFFFFF, p1 = (key >> 20) & 0xFFFFF, p0 = (key >> 40) & 0xFFFFF;
  const unsigned long long a = (key >> 60) & 3;
  const unsigned long long lin = (p0 * (unsigned long long)(d[1] + 2) + p1) * (unsigned long long)(d[2] + 2) + p2;
  return 3ull * lin + a;
}

// Bits 7..14 set for the nonzero bytes of x (low four) and y.
__device__ inline uint32_t nz8(uint32_t x, uint32_t y) {
  // high bit of each byte set iff the byte is nonzero, then gathered by dot products
  const uint32_t s = (((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x) & 0x80808080u;
  const uint32_t t = (((y & 0x7f7f7f7fu) + 0x7f7f7f7fu) | y) & 0x80808080u;
  return __builtin_amdgcn_udot4(s, 0x08040201u, __builtin_amdgcn_udot4(t, 0x80402010u, 0u, false), false);
}

// ---------------------------------------------------------------------------
// Inside bits of dense float volumes as one bit string (bit i: element i), written by
// a streaming pass, from which the passes over cubes cut the 32-voxel words of
// their rows: a brick that reads the volume itself waits for its own few loads
// and reads its neighbours' rows again, in four bytes a voxel.

// The string starts at the 16-byte boundary at or before the volume: bit
// shift + i is element i, shift = volume_shift(), so that the loads are whole
// aligned 16 bytes, but for the elements before the first and after the last of
// those.  Floats that are not aligned themselves are read one by one, with no shift.

__host__ __device__ inline bool odd_floats(const void* vol) { return ((uintptr_t)vol & 3u) != 0; }
__host__ __device__ inline int volume_shift(const void* vol) {
  return odd_floats(vol) ? 0 : (int)((uintptr_t)vol & 15u) / 4;
}

// 32-bit words of the string of n elements (whatever its shift), one more for
// the last cut and even, and its workgroups of `block` elements.
__host__ __device__ inline long long bit_words(long long n) { return (n + 3 + 63) / 64 * 2 + 2; }
__host__ __device__ inline long long bit_blocks(long long n, int block) { return (n + 3 + block - 1) / block; }

// The word of the bits pos .. pos + left - 1 (at most 32 of them; 0 if left <= 0).
__device__ inline uint32_t cut_word(const uint32_t* __restrict__ bits, unsigned int pos, int left) {
  if (left <= 0) return 0u;
  const uint32_t w = __builtin_amdgcn_alignbit(bits[(pos >> 5) + 1], bits[pos >> 5], pos & 31u);
  return left >= 32 ? w : w & ((1u << left) - 1u);
}

// The bits one voxel before those of row word r (prev: the word before it;
// bit 31 of a row's last word lies past the array, so it is 0 before a row).
__device__ inline uint32_t shifted(uint32_t r, uint32_t prev) { return __builtin_amdgcn_alignbit(r, prev, 31u); }

// The words of voxel planes z0 .. z0 + np - 1 (at most MAXP), row-groups rg0 ..
// rg0 + nw - 1 (row-group = cube row * G + group; 0 outside the array) of a
// dense volume of dims d into tile[plane * nw + word].  Thread t (of 256) takes
// words t, t + 256, ... of every plane: the rows are found once, and the planes'
// words are read together.
template <int MAXP>
__device__ inline void cut_tile(const uint32_t* __restrict__ bits, int shift, const int* d, int G, unsigned int mG,
                                int shG, int rg0, int z0, int np, int nw, uint32_t* tile) {
  const int d0 = d[0], d1 = d[1], d2 = d[2];
  for (int i = threadIdx.x; i < nw; i += 256) {
    const int rg = rg0 + i;
    const int ry = rg < 0 ? 0 : (int)fdiv((unsigned int)rg, mG, shG);
    const int y = ry - 1, x = 32 * (rg - ry * G);
    const int left = rg >= 0 && (unsigned)y < (unsigned)d1 ? d2 - x : 0;
    const unsigned int at = (unsigned int)shift + (unsigned int)y * (unsigned int)d2 + (unsigned int)x;
    const unsigned int plane = (unsigned int)d1 * (unsigned int)d2;
#pragma unroll
    for (int p = 0; p < MAXP; ++p) {
      const int z = z0 + p;
      if (p < np)
        tile[p * nw + i] = cut_word(bits, (unsigned int)z * plane + at, (unsigned)z < (unsigned)d0 ? left : 0);
    }
  }
}

// A workgroup's (256 threads) bits [e0, e0 + ROUNDS * 4096) of the string of n
// elements, a wave's ROUNDS * 1024 together.
template <int ROUNDS>
__device__ inline void pack_bits(const void* __restrict__ vol, long long n, long long e0,
                                 uint32_t* __restrict__ bits) {
  if (odd_floats(vol)) {
    const float* f = (const float*)vol;
    for (long long w = e0 / 32 + threadIdx.x; w < e0 / 32 + ROUNDS * 128 && 32 * w < n; w += 256) {
      uint32_t b = 0u;
      for (int k = 0; k < 32 && 32 * w + k < n; ++k) b |= (uint32_t)(f[32 * w + k] > 0.5f) << k;
      bits[w] = b;
    }
    return;
  }
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int shift = volume_shift(vol);
  const long long end = n + shift;
  const long long w0 = e0 + (long long)wid * (ROUNDS * 1024);
  const uint4* src = (const uint4*)((uintptr_t)vol & ~(uintptr_t)15);
  constexpr int J = ROUNDS > 1 ? 8 : 4;  // 16-byte loads in flight per thread
#pragma unroll
  for (int g = 0; g < ROUNDS * 4; g += J) {
    uint4 v[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const long long e = w0 + 256 * (g + j) + 4 * lane;
      v[j] = e >= shift && e + 4 <= end ? src[e >> 2] : make_uint4(0u, 0u, 0u, 0u);
    }
    // the volume's ends: the elements of a 16-byte word that is not all its own
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const long long e = w0 + 256 * (g + j) + 4 * lane;
      if (e < end && (e < shift || e + 4 > end)) {
        const uint32_t* w = (const uint32_t*)(src + (e >> 2));
        v[j].x = e >= shift ? w[0] : 0u;
        v[j].y = e + 1 >= shift && e + 1 < end ? w[1] : 0u;
        v[j].z = e + 2 >= shift && e + 2 < end ? w[2] : 0u;
        v[j].w = e + 3 >= shift && e + 3 < end ? w[3] : 0u;
      }
    }
    uint32_t mine = 0u;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const uint32_t b = (uint32_t)(__uint_as_float(v[j].x) > 0.5f) | (uint32_t)(__uint_as_float(v[j].y) > 0.5f) << 1 |
                         (uint32_t)(__uint_as_float(v[j].z) > 0.5f) << 2 | (uint32_t)(__uint_as_float(v[j].w) > 0.5f) << 3;
      const uint32_t w = lanes_reduce<3>(b << (4 * (lane & 7)), [](uint32_t a, uint32_t c) { return a | c; });
      mine = (lane & 7) == j ? w : mine;
    }
    const long long e = w0 + 256 * (g + (lane & 7)) + 32 * (lane >> 3);
    if ((lane & 7) < J && e < end) bits[e >> 5] = mine;
  }
}

}  // namespace s3d
