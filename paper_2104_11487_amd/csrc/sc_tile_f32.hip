// One launch per step for fp32 layers (Eq. 2-5; C_in % 8 == 0, 24..128): the
// gate of an 8 x 8-site tile and the product of its active blocks in one
// workgroup, as sc_tile.hip does for bf16.
//
// The fp32 matrix rate (157 TFLOP/s, 1/16 of bf16) makes one tile's product
// long for one CU: 64 sites x 64 channels x K = 576 take 7.7 us. So the output
// channels of a tile are split over several workgroups, each with NS 16-column
// tiles: all of them load the halo and evaluate the gate, the first writes what
// every one would write alike (x_{t-1} copy, statistics, block flags). NS is
// the largest that still leaves two workgroups per CU (one where no more fit).
//
//   1. halo: 8-channel chunks (two 16-byte words of each frame), KI in flight
//      per thread; r = x_t - x_{t-1} to LDS in fp32, the canonical statistic of
//      a pixel in one lane group;
//   2. support sums, threshold, block flags;
//   3. product of an active tile: wave w takes M-tile w (16 sites). A lane reads
//      16 bytes of r (4 channels) and of the weights (packed to match, channels
//      padded to 16 per tap) for four v_mfma_f32_16x16x4_f32, weights
//      kRing - 1 such groups ahead; the sums are added to z_{t-1}, loaded with
//      the first weights.
// 128 x 96, 64 -> 64, 3 x 3, 8 x 8 blocks, 38 % active: the gate kernel (6.2 us)
// and the gathering convolution (20-26 us, a memory round trip per 8 k-steps of
// 4-byte loads) before.
#include "sc_device.h"
#include "sc_kernels.h"
#include "sc_stream.h"

#pragma clang fp contract(off)

namespace sc {

namespace {

constexpr int kF32Threads = 256;
constexpr int kSide = 8;  // sites per tile side
constexpr int kItems = 4;
constexpr int kNonTemporal = 2;

// kParts: partial sums per output
template <int NS, int kParts>
__global__ void __launch_bounds__(kF32Threads) __attribute__((amdgpu_waves_per_eu(kParts == 2 ? 4 : 3)))
tile_f32_kernel(GateParams g, ConvParams c, TileF32Params tp) {
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  __shared__ uint32_t blk_flag[kSide * kSide];
  constexpr int kRing = NS == 4 ? 3 : (NS == 2 ? 4 : 6);  // weight groups in registers
  constexpr int kJoins = 8 / kParts;                      // times that the partial sums join the total
  const int hh = tp.hh, hw = tp.hw;
  float* a_halo = reinterpret_cast<float*>(lds + hh * hw * tp.pstride);

  // A tile's shares run on one XCD (its halo comes from HBM once: 128 x 96 x 64
  // 14.8 us, on several 18.8). The tiles are dealt to the XCDs one by one, so
  // that a cluster of active tiles has every CU (2 x 256 x 256 x 64, 3 % covered,
  // 49 -> 35 us), or in contiguous ranges while there is not one per CU (16.6 -> 14.8 us).
  const int per_img = g.tiles_y * g.tiles_x;
  const int slot = tp.deal ? (int)blockIdx.x >> 3 : xcd_tile(blockIdx.x, gridDim.x);
  const int tile = tp.deal ? slot / tp.shares * 8 + (int)(blockIdx.x & 7) : slot / tp.shares, share = slot % tp.shares;
  if (tile >= g.n * per_img) return;
  const bool lead = share == 0;
  const int n = tile / per_img, trem = tile - n * per_img;
  const int ty = trem / g.tiles_x, tx = trem - ty * g.tiles_x;
  const int oy0 = ty * kSide, ox0 = tx * kSide;
  const int oh = min(kSide, g.h_out - oy0), ow = min(kSide, g.w_out - ox0);
  const int s = g.stride, k = g.k;
  const int iy0 = oy0 * s - g.pad, ix0 = ox0 * s - g.pad;
  const int own_y0 = oy0 * s, own_x0 = ox0 * s;
  const int own_y1 = ty == g.tiles_y - 1 ? g.h : min(g.h, (oy0 + kSide) * s);
  const int own_x1 = tx == g.tiles_x - 1 ? g.w : min(g.w, (ox0 + kSide) * s);
  const int lblk = __ffs(g.block) - 1, tb_w = kSide >> lblk;
  if (threadIdx.x < kSide * kSide) blk_flag[threadIdx.x] = 0u;
  // chained: a tile far from every change stops before its loads, as in the gate
  // of the split pipeline (2 x 256 x 256, 128 -> 64: 6.1 us where nothing changed,
  // 21.1 with the loads; 47.6 against 54.1 where 2 % did)
  if (g.up_mask && quiet_tile(g, n, iy0, ix0, oy0, ox0, oh, ow, 3, kSide * kSide, kF32Threads, lead)) return;

  // ---- halo ----
  const uint32_t img_bytes = (uint32_t)((size_t)g.h * g.w * g.c * 4);
  const size_t img = (size_t)n * g.h * g.w * g.c;
  const auto rt = frame_rsrc(static_cast<const float*>(g.x_t) + img, img_bytes);
  const auto rp = frame_rsrc(static_cast<const float*>(g.no_prev ? g.x_t : g.x_prev) + img, img_bytes);
  const bool keep_on = g.x_keep != nullptr && lead;
  const auto rk = frame_rsrc(keep_on ? static_cast<float*>(g.x_keep) + img : nullptr, keep_on ? img_bytes : 0u);
  const int lg = tp.lg_group, group = 1 << lg, nchk = g.c >> 3;
  const int total = (hh * hw) << lg;
  const float inv_hw = 1.0f / (float)hw;
  const int wave0 = threadIdx.x & ~63;
  for (int base = 0; base < total; base += kF32Threads * kItems) {
    u32x4 vt[kItems][2], vp[kItems][2];
    uint32_t koff[kItems];
    int tid = threadIdx.x;  // opaque: the per-item terms are recomputed each round
    asm volatile("" : "+v"(tid));
#pragma unroll
    for (int u = 0; u < kItems; ++u) {
      const int idx = base + u * kF32Threads + tid;
      const int q = idx >> lg, ch = idx & (group - 1);
      const int hy = qdiv(q, inv_hw), hx = q - hy * hw;
      const int y = iy0 + hy, x = ix0 + hx;
      // (a group's lanes past the chunks load nothing and add +0 at the end)
      const bool in = idx < total && ch < nchk && y >= 0 && y < g.h && x >= 0 && x < g.w;
      const uint32_t off = in ? (uint32_t)(((y * g.w + x) * g.c + ch * kChunk) * 4) : kOutOfRange;
      const bool own = in && keep_on && g.copy_in_halo && y >= own_y0 && y < own_y1 && x >= own_x0 && x < own_x1;
      koff[u] = own ? off : kOutOfRange;
#pragma unroll
      for (int wd = 0; wd < 2; ++wd) {
        vt[u][wd] = __builtin_amdgcn_raw_buffer_load_b128(rt, off + 16 * wd, 0, 0);
        vp[u][wd] = __builtin_amdgcn_raw_buffer_load_b128(rp, (g.no_prev ? kOutOfRange : off) + 16 * wd, 0, 0);
      }
    }
#pragma unroll
    for (int u = 0; u < kItems; ++u) {
      if (base + u * kF32Threads + wave0 >= total) break;  // wave-uniform
      const int idx = base + u * kF32Threads + tid;
      const int q = idx >> lg, ch = idx & (group - 1);
      float r[kChunk];
      float sum = 0.0f;
#pragma unroll
      for (int j = 0; j < kChunk; ++j) {
        r[j] = __fsub_rn(__uint_as_float(vt[u][j >> 2][j & 3]), __uint_as_float(vp[u][j >> 2][j & 3]));
        sum = add_rn(sum, term(r[j], g.norm_p));
      }
      float acc;
      if (lg == 3) acc = group_sum<8>(sum);
      else if (lg == 2) acc = group_sum<4>(sum);
      else acc = group_sum<16>(sum);
      if (idx < total && ch == 0) a_halo[q] = acc;
      // channels past C, up to the padding of the weights, are zeros
      if (idx < total && ch * kChunk < tp.cpad) {
        float4* d = reinterpret_cast<float4*>(lds + q * tp.pstride + ch * 32);
        d[0] = make_float4(r[0], r[1], r[2], r[3]);
        d[1] = make_float4(r[4], r[5], r[6], r[7]);
      }
    }
#pragma unroll
    for (int u = 0; u < kItems; ++u)
#pragma unroll
      for (int wd = 0; wd < 2; ++wd)
        __builtin_amdgcn_raw_buffer_store_b128(vt[u][wd], rk, koff[u] + 16 * wd, 0, kNonTemporal);
  }
  if (!g.copy_in_halo && keep_on) copy_pixels(rt, rk, own_y0, own_y1, own_x0, own_x1, g.w, g.c >> 2, kF32Threads);
  lds_barrier();

  // ---- gate ----
  if (threadIdx.x < kSide * kSide) {
    const int ly = threadIdx.x >> 3, lx = threadIdx.x & 7;
    if (ly < oh && lx < ow) {
      float sv = 0.0f;
      if (g.support == 0) {
        const float* base = a_halo + (ly * s) * hw + lx * s;
        for (int kh = 0; kh < k; ++kh)
          for (int kw = 0; kw < k; ++kw) sv = add_rn(sv, base[kh * hw + kw]);
      } else {
        sv = a_halo[(ly * s + g.pad) * hw + lx * s + g.pad];
      }
      const bool on = g.reference || g.force_dense || ((double)sv * g.wnorm > g.thr) || (sv != sv);
      if (g.keep_stats && lead) {
        const size_t o = ((size_t)n * g.h_out + oy0 + ly) * g.w_out + ox0 + lx;
        g.stat[o] = sv;
        g.site_mask[o] = on ? 1 : 0;
      }
      if (on) blk_flag[(ly >> lblk) * tb_w + (lx >> lblk)] = 1u;
    }
  }
  lds_barrier();
  if (lead && threadIdx.x < kSide * kSide) {
    const int by = threadIdx.x / tb_w, bx = threadIdx.x - by * tb_w;
    if ((by << lblk) < oh && (bx << lblk) < ow)
      g.block_mask[((size_t)n * g.hb + (oy0 >> lblk) + by) * g.wb + (ox0 >> lblk) + bx] =
          (uint8_t)blk_flag[by * tb_w + bx];
  }

  // ---- product: this wave's 16 sites (two rows), NS x 16 channels ----
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r16 = lane & 15, kq = lane >> 4;
  const int ly = wave * 2 + (r16 >> 3), lx = r16 & 7;
  const bool live = ly < oh && lx < ow && blk_flag[(ly >> lblk) * tb_w + (lx >> lblk)] != 0u;
  if (__ballot(live) == 0ull) return;
  const int nt0 = share * NS, groups = tp.groups;  // groups of 16 k indices
  const auto wrs = frame_rsrc(tp.wpack, (uint32_t)(groups * c.ntiles_n * 1024));
  floatx4 wq[kRing][NS];
  auto load_w = [&](floatx4* dst, int j) {
#pragma unroll
    for (int i = 0; i < NS; ++i)
      dst[i] = __builtin_bit_cast(
          floatx4, __builtin_amdgcn_raw_buffer_load_b128(wrs, lane * 16, (j * c.ntiles_n + nt0 + i) * 1024, 0));
  };
#pragma unroll
  for (int j = 0; j < kRing - 1; ++j) load_w(wq[j], min(j, groups - 1));
  const size_t zimg = (size_t)g.h_out * g.w_out * c.c_out;
  const auto zrs = frame_rsrc(c.z + (size_t)n * zimg, (uint32_t)(zimg * 4));
  uint32_t zoff[NS];
  // kParts partial sums per output, K taken in turn: independent MFMA chains, and
  // fewer roundings behind each other. They join the total kJoins times on the
  // way through K, so z is no further from the exact sums than by the gathering
  // convolution's four sums over a quarter of K each (relative 2-norm, 2 x 160 x 160,
  // 128 -> 64: 2.3e-7 against 3.1e-7; two parts without joins 4.6e-7). Four column
  // tiles take two parts and four joins where K is long enough for them: four
  // parts leave registers for three waves per SIMD (256 x 256, 64 -> 64, 3 x 3, 3 %
  // covered: 33.0 against 25.5 us, 30 % 43.8 against 50.6; the other sizes and
  // reference frames 1 to 3 % slower on average)
  floatx4 zo[NS], acc[kParts][NS], tot[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    const int col = (nt0 + i) * 16 + kq * 4;
    zoff[i] = live && col < c.c_out ? (uint32_t)((((oy0 + ly) * g.w_out + ox0 + lx) * c.c_out + col) * 4) : kOutOfRange;
    zo[i] = __builtin_bit_cast(
        floatx4, __builtin_amdgcn_raw_buffer_load_b128(zrs, g.reference ? kOutOfRange : zoff[i], 0, 0));
#pragma unroll
    for (int e = 0; e < kParts; ++e) acc[e][i] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    tot[i] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  auto sum_of_parts = [&](int i, int v) {
    const float u = __fadd_rn(acc[0][i][v], acc[1][i][v]);
    if constexpr (kParts == 4) return __fadd_rn(u, __fadd_rn(acc[2][i][v], acc[3][i][v]));
    return u;
  };
  auto join = [&]() {
#pragma unroll
    for (int i = 0; i < NS; ++i) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
        tot[i][v] = __fadd_rn(tot[i][v], sum_of_parts(i, v));
#pragma unroll
      for (int e = 0; e < kParts; ++e) acc[e][i] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    }
  };
  const uint8_t* abase = lds + (ly * s * hw + lx * s) * tp.pstride + kq * 16;
  const int per_tap = tp.cpad >> 4;
  int aoff = 0, cc = 0, kw = 0, jn = 0;  // halo offset of the next group (kh, kw, cc)
  auto read_a = [&]() {
    const floatx4 a = *reinterpret_cast<const floatx4*>(abase + aoff);
    const bool more = ++jn < groups;
    const bool wrap = cc + 1 == per_tap, wrap2 = wrap && kw + 1 == k;
    int step = 64;
    step += wrap ? tp.pstride - per_tap * 64 : 0;
    step += wrap2 ? (hw - k) * tp.pstride : 0;
    aoff += more ? step : 0;
    cc = wrap ? 0 : cc + 1;
    kw = wrap2 ? 0 : (wrap ? kw + 1 : kw);
    return a;
  };
  floatx4 a = read_a();
  auto use = [&](const floatx4* w) {
    const floatx4 an = read_a();
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < NS; ++i)
        acc[e % kParts][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[i][e], a[e], acc[e % kParts][i], 0, 0, 0);
    a = an;
  };
  int j = 0;
  const int run = max(groups / kJoins / kRing, 1) * kRing;  // groups between joins
  int next = run;
  for (; j + kRing <= groups; j += kRing) {
    if (j == next) {
      join();
      next += run;
    }
#pragma unroll
    for (int r = 0; r < kRing; ++r) {
      load_w(wq[(r + kRing - 1) % kRing], min(j + r + kRing - 1, groups - 1));
      use(wq[r]);
    }
  }
  if (j == next) join();
#pragma unroll
  for (int r = 0; r < kRing - 1; ++r)
    if (r < groups - j) use(wq[r]);
  join();

#pragma unroll
  for (int i = 0; i < NS; ++i) {
    floatx4 nv;
#pragma unroll
    for (int v = 0; v < 4; ++v) nv[v] = __fadd_rn(zo[i][v], tot[i][v]);
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, nv), zrs, zoff[i], 0, 0);
    if (c.act && zoff[i] != kOutOfRange) {
      float4* y = reinterpret_cast<float4*>(static_cast<float*>(c.y) + (size_t)n * zimg + zoff[i] / 4);
      *y = c.act == 2 ? make_float4(relu_f32(nv[0]), relu_f32(nv[1]), relu_f32(nv[2]), relu_f32(nv[3]))
                      : make_float4(nv[0], nv[1], nv[2], nv[3]);
    }
  }
}

// Weights for it: [tap][16-channel group][16-column tile][lane][4], lane l and
// element e holding channel 16 * group + 4 * (l / 16) + e of output column
// l % 16; channels past C_in and columns past C_out are zero.
__global__ void pack_tile_f32_kernel(const float* w, float* out, int c_out, int c_in, int k, int per_tap, int ntn,
                                     int total) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int e = i & 3, lane = (i >> 2) & 63, q = i >> 8;
  const int nt = q % ntn, grp = q / ntn;
  const int tap = grp / per_tap, ci = (grp - tap * per_tap) * 16 + (lane >> 4) * 4 + e, co = nt * 16 + (lane & 15);
  out[i] = ci < c_in && co < c_out ? w[((size_t)co * c_in + ci) * k * k + tap] : 0.0f;
}

using Kernel = void (*)(GateParams, ConvParams, TileF32Params);
Kernel kernel_of(const TileF32Params& t) {
  // two parts: at least one turn of the weight ring between joins
  if (t.ns == 4) return t.groups >= 12 ? tile_f32_kernel<4, 2> : tile_f32_kernel<4, 4>;
  return t.ns == 1 ? tile_f32_kernel<1, 4> : (t.ns == 2 ? tile_f32_kernel<2, 4> : nullptr);
}
int lds_of(const TileF32Params& t) { return t.hh * t.hw * t.pstride + (t.hh * t.hw * 4 + 15) / 16 * 16; }

}  // namespace

bool tile_f32_shape(TileF32Params& t, int c, int k, int stride, int ntn, long tiles, int num_cu, long lds_limit) {
  if (c % 8 || c < 24 || c > 128 || (ntn != 1 && ntn != 2 && ntn != 4 && ntn != 8)) return false;
  t.hh = t.hw = (kSide - 1) * stride + k;
  t.cpad = (c + 15) / 16 * 16;
  t.pstride = t.cpad * 4 + 16;
  t.groups = k * k * t.cpad / 16;
  t.lg_group = 2;
  while (c >> 3 > 1 << t.lg_group || t.cpad >> 3 > 1 << t.lg_group) ++t.lg_group;
  t.ns = ntn < 4 ? ntn : 4;
  // two workgroups per CU, or the one whose halo fits (128 channels at stride 2:
  // shares past the first round only load the halo again; 160 x 160, 128 -> 128,
  // reference 76.0 -> 48.7 us, 30 % covered 62.8 -> 49.3; 200 x 200, 128 -> 64, 60.4 -> 49.9)
  const long per_cu = lds_of(t) > lds_limit / 2 ? 1 : 2;
  while (t.ns > 1 && tiles * (ntn / t.ns) < per_cu * num_cu) t.ns >>= 1;
  t.shares = ntn / t.ns;
  t.deal = tiles >= num_cu;
  return lds_of(t) <= lds_limit;
}

int tile_f32_occupancy(const TileF32Params& t) {
  const Kernel f = kernel_of(t);
  int blocks = 0;
  if (!f || hipFuncSetAttribute(reinterpret_cast<const void*>(f), hipFuncAttributeMaxDynamicSharedMemorySize, lds_of(t)) !=
                hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, f, kF32Threads, lds_of(t)) != hipSuccess)
    return 0;
  return blocks;
}

hipError_t launch_tile_f32(const GateParams& g, const ConvParams& c, const TileF32Params& t, hipStream_t st) {
  const Kernel f = kernel_of(t);
  if (!f) return hipErrorInvalidValue;
  const int tiles = g.n * g.tiles_y * g.tiles_x;
  hipLaunchKernelGGL(f, dim3((unsigned)((t.deal ? (tiles + 7) / 8 * 8 : tiles) * t.shares)), dim3(kF32Threads), lds_of(t), st, g, c, t);
  return hipGetLastError();
}

hipError_t launch_pack_tile_f32(const void* w, void* out, int c_out, int c_in, int k, const TileF32Params& t, int ntn,
                                hipStream_t st) {
  const int total = t.groups * ntn * 256;
  hipLaunchKernelGGL(pack_tile_f32_kernel, dim3((total + 255) / 256), dim3(256), 0, st, static_cast<const float*>(w),
                     static_cast<float*>(out), c_out, c_in, k, t.cpad / 16, ntn, total);
  return hipGetLastError();
}

}  // namespace sc
