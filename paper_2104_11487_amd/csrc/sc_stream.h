// Streaming helpers shared by the gate kernel and the fused gate+conv kernel:
// canonical per-pixel statistic, vector loads/copies, XCD-aware tile order.
#pragma once

#include "sc_device.h"

#pragma clang fp contract(off)

namespace sc {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kUnroll = 4;  // staging chunks whose loads are issued together

__device__ __forceinline__ float term(float r, int norm_p) {
  return norm_p == 2 ? mul_rn(r, r) : fabsf(r);
}

// Canonical order of the per-pixel statistic: channels in chunks of kChunk
// consecutive channels; within a chunk the terms are added in ascending
// order from +0; the chunk sums are then added in ascending chunk order.
constexpr int kChunk = 8;

// Ordered sum of the terms of up to kChunk consecutive channels (one chunk).
template <int N>
__device__ __forceinline__ float chunk_sum(const float* r, int norm_p) {
  float part = 0.0f;
#pragma unroll
  for (int i = 0; i < N; ++i) part = add_rn(part, term(r[i], norm_p));
  return part;
}

template <typename T, int VEC>
__device__ __forceinline__ void load_vec(const T* p, size_t off, float* v) {
  if (VEC == 8) {
    Elem<T>::load8(p, off, v);
  } else if (VEC == 4) {
    Elem<T>::load4(p, off, v);
  } else {
    v[0] = Elem<T>::load1(p, off);
  }
}

template <typename T, int VEC>
__device__ __forceinline__ void copy_vec(T* dst, const T* src, size_t off) {
  if (VEC * sizeof(T) == 16) {
    *reinterpret_cast<uint4*>(dst + off) = *reinterpret_cast<const uint4*>(src + off);
  } else if (VEC * sizeof(T) == 8) {
    *reinterpret_cast<uint2*>(dst + off) = *reinterpret_cast<const uint2*>(src + off);
  } else {
#pragma unroll
    for (int j = 0; j < VEC; ++j) dst[off + j] = src[off + j];
  }
}

// floor(n / d) for 0 <= n < 2^20 and d >= 1, given inv_d = 1 / d rounded to
// fp32 (within 2.5 ulp): (n + 1/2) / d is at least 1 / (2d) away from an
// integer, and the fp32 product lies within (n + 1/2) / d * 2^-21 < 1 / (2d)
// of it, so truncation gives the exact quotient. A few VALU operations instead
// of the long integer-division sequence.
__device__ __forceinline__ int qdiv(int n, float inv_d) {
  return (int)(((float)n + 0.5f) * inv_d);
}

// Value of lane (this lane + J) of the same 16-lane row (DPP row_shl:J).
template <int J>
__device__ __forceinline__ float row_shl(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x100 + J, 0xf, 0xf, false));
}

template <int NC, int J>
__device__ __forceinline__ float group_sum_from(float acc, float v) {
  if constexpr (J < NC) {
    return group_sum_from<NC, J + 1>(add_rn(acc, row_shl<J>(v)), v);
  } else {
    return acc;
  }
}

// Ordered sum (from +0, ascending lanes) of the NC values held by lanes
// l .. l + NC - 1 of one 16-lane row, valid in lane l (NC <= 16; the group
// must not cross a row boundary). Lane-to-lane moves only, no LDS traffic.
template <int NC>
__device__ __forceinline__ float group_sum(float v) {
  return group_sum_from<NC, 1>(add_rn(0.0f, v), v);
}

// Workgroup barrier that orders LDS accesses only: outstanding global loads
// and stores stay in flight. (A global_load_lds still in flight makes the
// compiler wait for it here.)
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Raw buffer resource over `bytes` bytes at `base`: a load at an offset at or
// beyond `bytes` returns zeros and a store there is dropped, without a memory
// access (range-checked buffer addressing of the CDNA ISA).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t frame_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}
constexpr uint32_t kOutOfRange = 0x80000000u;  // byte offset past every frame resource

// Copy the pixels [y0, y1) x [x0, x1) of one image from `src` to `dst` (frame
// resources; px16 16-byte words a pixel, w pixels a row), by `threads` threads
// of a workgroup: the owned pixels of a tile whose halo does not hold them all
// (strides larger than the kernel).
template <typename R>
__device__ __forceinline__ void copy_pixels(R src, R dst, int y0, int y1, int x0, int x1, int w, int px16, int threads) {
  const int per_row = max(x1 - x0, 0) * px16, total = max(y1 - y0, 0) * per_row;
  for (int i = threadIdx.x; i < total; i += threads) {
    const int yy = i / per_row, e = i - yy * per_row;
    const uint32_t off = (uint32_t)(((y0 + yy) * w + x0) * px16 + e) * 16u;
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_amdgcn_raw_buffer_load_b128(src, off, 0, 0), dst, off, 0, 2);
  }
}

// Workgroup b runs tile remap(b): XCD b % 8 (workgroups go to the XCDs
// round-robin) receives a contiguous range of tiles, so neighbouring tiles
// share their halo rows through one L2.
__device__ __forceinline__ int xcd_tile(int b, int g) {
  const int per = g >> 3, rem = g & 7, x = b & 7;
  return x * per + min(x, rem) + (b >> 3);
}

// Workgroup b runs tile xcd_deal(b): runs of G tiles are dealt to the XCDs in
// turn. Neighbours within a run share an L2, and a cluster of active tiles (a
// moving object) is spread over every XCD, where a contiguous range would leave
// its products to one XCD's CUs.
template <int G>
__device__ __forceinline__ int xcd_deal(int b, int g) {
  const int full = g / (8 * G) * (8 * G);
  if (b >= full) return b;
  const int i = b >> 3;
  return (i / G * 8 + (b & 7)) * G + i % G;
}

// Chained steps with a norm gate: the residual is zero outside the upstream
// layer's active blocks, so a tile whose input region meets none of them has a
// zero statistic and every gate off. Then true (uniform over the workgroup), with
// the tile's statistics and block flags written by the threads of `lead`. A tile
// has oh x ow sites at (oy0, ox0), its rows 1 << lw sites wide and `sites` in all
// when it is whole; its halo starts at (iy0, ix0). No more sites than threads.
template <typename G>
__device__ __forceinline__ bool quiet_tile(const G& g, int n, int iy0, int ix0, int oy0, int ox0, int oh, int ow, int lw,
                                           int sites, int threads, bool lead) {
  const int y0 = max(iy0, 0), y1 = min(iy0 + (oh - 1) * g.stride + g.k, g.h);
  const int x0 = max(ix0, 0), x1 = min(ix0 + (ow - 1) * g.stride + g.k, g.w);
  const int by0 = y0 / g.up_block, bx0 = x0 / g.up_block;
  const int nbx = (x1 - 1) / g.up_block - bx0 + 1, cnt = ((y1 - 1) / g.up_block - by0 + 1) * nbx;
  int any = 0;
  for (int i = threadIdx.x; i < cnt; i += threads)
    any |= g.up_mask[((size_t)n * g.up_hb + by0 + i / nbx) * g.up_wb + bx0 + i % nbx] != 0;
  if (__syncthreads_or(any)) return false;
  if (!lead) return true;
  if (g.keep_stats && threadIdx.x < sites) {
    const int ly = threadIdx.x >> lw, lx = threadIdx.x & ((1 << lw) - 1);
    const size_t o = ((size_t)n * g.h_out + oy0 + ly) * g.w_out + ox0 + lx;
    if (ly < oh && lx < ow) {
      g.stat[o] = 0.0f;
      g.site_mask[o] = 0;
    }
  }
  const int lblk = __ffs(g.block) - 1, nb = 1 << (lw - lblk), by = threadIdx.x / nb, bx = threadIdx.x - by * nb;
  if ((by << lblk) < oh && (bx << lblk) < ow)
    g.block_mask[((size_t)n * g.hb + (oy0 >> lblk) + by) * g.wb + (ox0 >> lblk) + bx] = 0;
  return true;
}

}  // namespace sc
