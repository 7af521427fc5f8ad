// One launch per step for mid-size frames of dense bf16 layers (Eq. 2-5): the
// gate of a tile of up to 16 x 16 output sites and the convolution of its
// active blocks in one workgroup.
//
// On frames of a few tiles per CU the split pipeline's two kernels are mostly
// latency: each pays its launch, and the convolution then reads counters and
// list (two dependent round trips), loads the residual halo that the gate has
// just had in registers, and waits for its first weights. Here the gate's
// halo pass leaves rho = bf16(x_t - x_{t-1}) in LDS, so an active tile goes on
// to the product at once, on weights whose first k-steps were fetched before
// the halo; a tile with no active block stops after its block flags.
//
//   1. first kR - 1 k-steps of weights, then the halo: 16-byte chunks of both
//      frames, KI in flight per thread; residual, canonical statistic (chunk
//      sums of a pixel in one lane group, see halo_lane_sums of sc_gate.hip),
//      rho to LDS, x_t of owned pixels to the spare x_{t-1} slot;
//   2. support sums, threshold, block flags in LDS and in memory;
//   3. product of the tile's 16 * WM * WAVES_M sites in one pass (a wave whose
//      sites are all off skips it), z_{t-1} added, then the stores.
//      One pass, because loads issued after a store wait for it: two passes of
//      128 sites took 3 us more on 2 x 256 x 256 x 64.
// On a reference frame every block is on and x_{t-1} is not read: the frame
// is read once for state, statistic and product alike.
//
// Translated steps (TRANS): x_{t-1} and z_{t-1} are read at shifted places;
// blocks with an exposed line are computed by a second product over the x_t
// halo (border tiles only), and the tile moves the state of its off blocks.
//
// Chained steps (CHAIN): the input is the upstream layer's fp32 residual; the
// same arithmetic from there on, so z is that of a plain step bit for bit.
//
// The kernel is instantiated in sc_tile.hip (32, 64 or 128 input channels),
// sc_tile_parts.hip (those whose K is summed in short chains: FL) and
// sc_tile_tab.hip (other multiples of 8).
#pragma once

#include <type_traits>

#include "sc_device.h"
#include "sc_halo_conv.h"
#include "sc_kernels.h"
#include "sc_stream.h"

#pragma clang fp contract(off)

namespace sc {

namespace {

constexpr int kNonTemporal = 2;

// Ordered sum over the 1 << lg lanes of a pixel's group (lg is uniform).
__device__ __forceinline__ float group_sum_lg(float v, int lg) {
  if (lg == 3) return group_sum<8>(v);
  if (lg == 2) return group_sum<4>(v);
  if (lg == 4) return group_sum<16>(v);
  return group_sum<2>(v);
}

// OCC: waves per SIMD the register budget aims for. z_{t-1} is added after the
// product (one rounding of the update on the state: 1.1e-7 from the exact
// sums at 48 -> 128 channels, 1.3e-7 when the sums start from z_{t-1}). LATE: it
// is loaded after the product too, where it would not fit the registers beside
// the sums (2 x 280 x 280, 48 -> 128: 46.5 us, started from z_{t-1} 41.4, by the
// gathering convolution 79.7; 2 x 256 x 256 x 64 translated 31.1, 31.2 and 66.2).
template <int WAVES_M, int WAVES_N, int WM, int WN, int KR, int OCC, int KI, bool LATE, bool TRANS, bool CHAIN, int LEARN,
          bool TAB, int FL = 0>
__global__ void __launch_bounds__(64 * WAVES_M * WAVES_N) __attribute__((amdgpu_waves_per_eu(OCC)))
tile_kernel(GateParams g, ConvParams c, HaloParams hp) {
  constexpr int kTileThreads = 64 * WAVES_M * WAVES_N;
  static_assert(!TRANS || (!LEARN && !CHAIN), "learned and chained translated steps take the split pipeline");
  typedef HaloConv<WAVES_M, WAVES_N, WM, WN, KR, 1, 1, TRANS, true, TAB, FL> HC;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  __shared__ uint32_t blk_flag[kMaxTileBlocks];
  float* a_halo = reinterpret_cast<float*>(lds + hp.lds_bytes);
  float* part = reinterpret_cast<float*>(lds + hp.part_off);

  // runs of four tiles dealt to the XCDs: active tiles cluster, so contiguous
  // ranges leave XCDs idle (512 x 512 x 64, per-site, 15 % covered, caller's frames:
  // 38.3 -> 35.8 us; 2 x 256 x 256 x 64, reference 23.2 -> 22.7, learned 31.3 -> 30.9;
  // 108 tiles of 135 x 181 11.85 -> 12.0)
  const int tile = xcd_deal<4>(blockIdx.x, gridDim.x);
  const int per_img = g.tiles_y * g.tiles_x;
  const int n = tile / per_img, trem = tile - n * per_img;
  const int ty = trem / g.tiles_x, tx = trem - ty * g.tiles_x;
  const int th = hp.rows, tw = hp.side;  // tile extent in sites
  const int oy0 = ty * th, ox0 = tx * tw;
  const int oh = min(th, g.h_out - oy0), ow = min(tw, g.w_out - ox0);
  const int s = g.stride, k = g.k, hh = hp.hh, hw = hp.hw;
  const int iy0 = oy0 * s - g.pad, ix0 = ox0 * s - g.pad;
  const int own_y0 = oy0 * s, own_x0 = ox0 * s;
  const int own_y1 = ty == g.tiles_y - 1 ? g.h : min(g.h, (oy0 + th) * s);
  const int own_x1 = tx == g.tiles_x - 1 ? g.w : min(g.w, (ox0 + tw) * s);
  const int lw = __ffs(tw) - 1, lblk = __ffs(g.block) - 1;

  HC H(c, hp, lds);
  typename HC::Ring bq;
  if constexpr (!LEARN) H.start_b(bq);
  if constexpr (TAB) H.make_tab(reinterpret_cast<int*>(lds + hp.tab_off), kTileThreads);
  if (threadIdx.x < kMaxTileBlocks) blk_flag[threadIdx.x] = 0u;

  if constexpr (CHAIN && !LEARN) {
    if (g.up_mask && quiet_tile(g, n, iy0, ix0, oy0, ox0, oh, ow, lw, th * tw, kTileThreads, true)) return;
  }

  // ---- halo ----
  constexpr int kE = CHAIN ? 4 : 2;  // bytes per input element
  const uint32_t img_bytes = (uint32_t)((size_t)g.h * g.w * g.c * kE);
  const size_t img = (size_t)n * g.h * g.w * g.c;
  const auto rt = frame_rsrc(static_cast<const uint8_t*>(g.x_t) + img * kE, img_bytes);
  const auto rp = frame_rsrc(static_cast<const uint8_t*>(g.no_prev ? g.x_t : g.x_prev) + img * kE, img_bytes);
  const bool keep_on = g.x_keep != nullptr;
  const auto rk = frame_rsrc(keep_on ? static_cast<uint16_t*>(g.x_keep) + img : nullptr, keep_on ? img_bytes : 0u);
  const int lg = hp.lg_group, group = 1 << lg, nchk = g.c >> 3;
  const int total = (hh * hw) << lg;
  const float inv_hw = 1.0f / (float)hw;
  const int wave0 = threadIdx.x & ~63;
  // the residual of a chunk from its two words: of x_t and x_{t-1}, or (CHAIN)
  // the fp32 residual's halves
  auto residual = [&](const u32x4& wt, const u32x4& wp, float (&r)[kChunk]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {  // channels 2e (low half) and 2e + 1 (high half)
      if constexpr (CHAIN) {
        r[e] = __uint_as_float(wt[e]);
        r[4 + e] = __uint_as_float(wp[e]);
      } else {
        r[2 * e] = __fsub_rn(__uint_as_float(wt[e] << 16), __uint_as_float(wp[e] << 16));
        r[2 * e + 1] = __fsub_rn(__uint_as_float(wt[e] & 0xffff0000u), __uint_as_float(wp[e] & 0xffff0000u));
      }
    }
  };
  // FIRST: residual, statistic and state; otherwise only rho = x_t
  auto halo = [&](auto first) {
    constexpr bool kFirst = decltype(first)::value;
    for (int base = 0; base < total; base += kTileThreads * KI) {
      u32x4 vt[KI], vp[KI];
      uint32_t koff[KI];
      int tid = threadIdx.x;  // opaque: the per-item terms are recomputed each round
      asm volatile("" : "+v"(tid));
#pragma unroll
      for (int u = 0; u < KI; ++u) {
        const int idx = base + u * kTileThreads + tid;
        const int q = idx >> lg, ch = idx & (group - 1);
        const int hy = qdiv(q, inv_hw), hx = q - hy * hw;
        const int y = iy0 + hy, x = ix0 + hx;
        // (TAB: a group may have more lanes than the pixel has chunks; the spare
        // ones load nothing and add +0 after the last chunk)
        const bool in = idx < total && (!TAB || ch < nchk) && y >= 0 && y < g.h && x >= 0 && x < g.w;
        const uint32_t off = (uint32_t)(((y * g.w + x) * g.c + ch * kChunk) * kE);
        vt[u] = __builtin_amdgcn_raw_buffer_load_b128(rt, in ? off : kOutOfRange, 0, 0);
        if constexpr (kFirst) {
          bool pin = in && (CHAIN || !g.no_prev);
          uint32_t po = CHAIN ? off + 16 : off;
          if constexpr (TRANS) {
            const int yp = y - g.sy, xq = x - g.sx;
            pin = pin && yp >= 0 && yp < g.h && xq >= 0 && xq < g.w;
            po = (uint32_t)(((yp * g.w + xq) * g.c + ch * kChunk) * 2);
          }
          vp[u] = __builtin_amdgcn_raw_buffer_load_b128(rp, pin ? po : kOutOfRange, 0, 0);
          const bool own = in && keep_on && g.copy_in_halo && y >= own_y0 && y < own_y1 && x >= own_x0 && x < own_x1;
          koff[u] = own ? off : kOutOfRange;
        }
      }
#pragma unroll
      for (int u = 0; u < KI; ++u) {
        if (base + u * kTileThreads + wave0 >= total) break;  // wave-uniform
        const int idx = base + u * kTileThreads + tid;
        const int q = idx >> lg, ch = idx & (group - 1);
        u32x4 rho = vt[u];
        if constexpr (kFirst) {
          float sum = 0.0f;
          float r[kChunk];
          residual(vt[u], vp[u], r);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            sum = add_rn(sum, term(r[2 * e], g.norm_p));
            sum = add_rn(sum, term(r[2 * e + 1], g.norm_p));
            rho[e] = pack_bf16(r[2 * e], r[2 * e + 1]);
          }
          if (TAB && hp.part_off) {
            if (idx < total && ch < nchk) part[q * (nchk | 1) + ch] = sum;
          } else {
            const float acc = group_sum_lg(sum, lg);
            if (idx < total && ch == 0) a_halo[q] = acc;
          }
        }
        if (idx < total && (!TAB || ch < nchk)) *reinterpret_cast<u32x4*>(lds + q * hp.pstride + ch * 16) = rho;
      }
      if constexpr (kFirst) {
#pragma unroll
        for (int u = 0; u < KI; ++u)
          __builtin_amdgcn_raw_buffer_store_b128(vt[u], rk, koff[u], 0, kNonTemporal);
      }
    }
  };
  const int tb_w = tw >> lblk;
  // the gate of one site: statistic or score sv
  auto decide = [&](int ly, int lx, float sv, bool above) {
    const int oy = oy0 + ly, ox = ox0 + lx;
    bool on = g.reference || g.force_dense || above || (sv != sv);
    if constexpr (TRANS) on = on || oy < c.ey.lo || oy >= c.ey.hi || ox < c.ex.lo || ox >= c.ex.hi;
    if (g.keep_stats) {
      const size_t o = ((size_t)n * g.h_out + oy) * g.w_out + ox;
      g.stat[o] = sv;
      g.site_mask[o] = on ? 1 : 0;
    }
    if (on) blk_flag[(ly >> lblk) * tb_w + (lx >> lblk)] = 1u;
  };
  const int ly = (threadIdx.x >> lw) & (th - 1), lx = threadIdx.x & (tw - 1);  // this thread's site
  if constexpr (LEARN) {
    // ---- learned gate (Eq. 8): one thread per site and share of the taps ----
    // A score takes 2 k^2 C_in rounded operations a site in a fixed order, so
    // the work is VALU issue: every (site, tap) pair is formed once, by the
    // thread of that site (the halo pixels' terms of every tap, formed per
    // pixel and exchanged through LDS, took 1.56 x the products on 8 x 8 tiles
    // and most of their time in the exchange). phi comes through the scalar
    // cache, two 8-channel chunks of the residual at a time through LDS (20
    // floats a pixel: 16 sites of a row read distinct banks), and the frames'
    // chunks stay in registers, from which an active tile then writes rho.
    constexpr int K2 = LEARN * LEARN, kSites = 16 * WM * WAVES_M, kSplit = kTileThreads / kSites;
    constexpr int TPT = (K2 + kSplit - 1) / kSplit;  // taps per thread
    constexpr int RS = 20;                           // floats of a pixel in the residual buffer
    float* rbuf = reinterpret_cast<float*>(lds);
    u32x4 vt[KI], vp[KI];
    const int ch = threadIdx.x & (group - 1);  // the same for every item of the thread
    auto each = [&](auto body) {
#pragma unroll
      for (int u = 0; u < KI; ++u) {
        int tid = threadIdx.x;  // opaque: recomputed, not held
        asm volatile("" : "+v"(tid));
        const int idx = u * kTileThreads + tid;
        body(u, idx >> lg, idx < total);
      }
    };
    each([&](int u, int q, bool valid) {
      const int hy = qdiv(q, inv_hw), hx = q - hy * hw;
      const int y = iy0 + hy, x = ix0 + hx;
      const bool in = valid && y >= 0 && y < g.h && x >= 0 && x < g.w;
      const uint32_t off = in ? (uint32_t)(((y * g.w + x) * g.c + ch * kChunk) * kE) : kOutOfRange;
      vt[u] = __builtin_amdgcn_raw_buffer_load_b128(rt, off, 0, 0);
      vp[u] = __builtin_amdgcn_raw_buffer_load_b128(rp, CHAIN ? off + 16 : (g.no_prev ? kOutOfRange : off), 0, 0);
    });
    float acc[TPT];
#pragma unroll
    for (int i = 0; i < TPT; ++i) acc[i] = 0.0f;
    const int tg = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kSites);  // share of the taps (whole waves)
    const bool score = !g.reference || g.keep_stats;
    typedef const __attribute__((address_space(4))) float const_f32;
    const const_f32* phi = (const const_f32*)g.phi;
    for (int c0 = 0; c0 < nchk && score; c0 += 2) {
      if ((ch >> 1) == (c0 >> 1))
        each([&](int u, int q, bool valid) {
          float r[kChunk];
          residual(vt[u], vp[u], r);
          float4* d = reinterpret_cast<float4*>(rbuf + q * RS + (ch & 1) * kChunk);
          if (valid) {
            d[0] = make_float4(r[0], r[1], r[2], r[3]);
            d[1] = make_float4(r[4], r[5], r[6], r[7]);
          }
        });
      lds_barrier();
#pragma unroll
      for (int i = 0; i < TPT; ++i) {
        const int t = tg * TPT + i, kh = t / LEARN, kw = t - kh * LEARN;  // uniform
        if (t < K2) {
          const float4* rr = reinterpret_cast<const float4*>(rbuf + ((ly * s + kh) * hw + lx * s + kw) * RS);
#pragma unroll
          for (int cc = 0; cc < 2; ++cc) {
            const const_f32* ph = phi + t * g.c + (c0 + cc) * kChunk;
            const float4 a = rr[2 * cc], b = rr[2 * cc + 1];
            const float r[kChunk] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
            // (the chunk sum's own first addition to +0 is left out: a sum of
            // -0 terms becomes +0 in the next one)
            float part = mul_rn(ph[0], r[0]);
#pragma unroll
            for (int j = 1; j < kChunk; ++j) part = add_rn(part, mul_rn(ph[j], r[j]));
            acc[i] = add_rn(acc[i], part);
          }
        }
      }
      lds_barrier();  // the next chunks overwrite the buffer
    }
    // without a score no barrier has passed since the block flags were cleared
    if (kSplit == 1 && !score) lds_barrier();
    // the owned pixels' state copy, past the loads that the scores waited for
    each([&](int u, int q, bool valid) {
      const int hy = qdiv(q, inv_hw), hx = q - hy * hw;
      const int y = iy0 + hy, x = ix0 + hx;
      const bool own = valid && keep_on && g.copy_in_halo && y >= own_y0 && y < own_y1 && x >= own_x0 && x < own_x1;
      __builtin_amdgcn_raw_buffer_store_b128(
          vt[u], rk, own ? (uint32_t)(((y * g.w + x) * g.c + ch * kChunk) * kE) : kOutOfRange, 0, kNonTemporal);
    });
    // the taps' sums of a site meet in tap order, then the bias; out-of-frame taps
    // add +0 (their own sums, zeros times phi, are NaN where phi is not finite)
    if constexpr (kSplit > 1) {
      if (tg > 0) {
#pragma unroll
        for (int i = 0; i < TPT; ++i)
          if (tg * TPT + i < K2) rbuf[(tg * TPT + i) * kSites + (threadIdx.x & (kSites - 1))] = acc[i];
      }
      lds_barrier();
    }
    if (threadIdx.x < kSites && ly < oh && lx < ow) {
      float sv = 0.0f;
#pragma unroll
      for (int t = 0; t < K2; ++t) {
        const int y = iy0 + ly * s + t / LEARN, x = ix0 + lx * s + t % LEARN;
        const float v = t < TPT ? acc[t < TPT ? t : 0] : rbuf[t * kSites + threadIdx.x];
        sv = add_rn(sv, y >= 0 && y < g.h && x >= 0 && x < g.w ? v : 0.0f);
      }
      sv = add_rn(sv, g.gate_bias);
      decide(ly, lx, sv, sv > 0.0f);
    }
    lds_barrier();
    // an active tile writes rho and fetches its first weights; the others end
    uint32_t any = 0u;
    for (int i = threadIdx.x & 63; i < (th >> lblk) * tb_w; i += 64) any |= blk_flag[i];
    const bool active = __ballot(any != 0u) != 0ull;  // every wave sees all flags: uniform
    if (active) {
      H.start_b(bq);
      each([&](int u, int q, bool valid) {
        float r[kChunk];
        residual(vt[u], vp[u], r);
        if (valid)
          *reinterpret_cast<u32x4*>(lds + q * hp.pstride + ch * 16) =
              u32x4{pack_bf16(r[0], r[1]), pack_bf16(r[2], r[3]), pack_bf16(r[4], r[5]), pack_bf16(r[6], r[7])};
      });
    }
  } else {
    halo(std::true_type{});
    lds_barrier();
    if (TAB && hp.part_off) {  // more than 16 chunks a pixel: their sums meet in LDS
      for (int q = threadIdx.x; q < hh * hw; q += kTileThreads) {
        float a = 0.0f;
        for (int i = 0; i < nchk; ++i) a = add_rn(a, part[q * (nchk | 1) + i]);
        a_halo[q] = a;
      }
      lds_barrier();
    }

    // ---- gate: support statistic, threshold, block flags ----
    if (threadIdx.x < th * tw && ly < oh && lx < ow) {
      float sv = 0.0f;
      if (g.support == 0) {
        const float* base = a_halo + (ly * s) * hw + lx * s;
        for (int kh = 0; kh < k; ++kh)
          for (int kw = 0; kw < k; ++kw) sv = add_rn(sv, base[kh * hw + kw]);
      } else {
        sv = a_halo[(ly * s + g.pad) * hw + lx * s + g.pad];
      }
      decide(ly, lx, sv, (double)sv * g.wnorm > g.thr);
    }
  }
  if (!g.copy_in_halo && keep_on) copy_pixels(rt, rk, own_y0, own_y1, own_x0, own_x1, g.w, nchk, kTileThreads);
  lds_barrier();
  const int bi0 = oy0 >> lblk, bj0 = ox0 >> lblk;
  {
    const int by = threadIdx.x / tb_w, bx = threadIdx.x - by * tb_w;  // one block per thread (<= 256)
    if ((by << lblk) < oh && (bx << lblk) < ow)
      g.block_mask[((size_t)n * g.hb + bi0 + by) * g.wb + bj0 + bx] = (uint8_t)blk_flag[by * tb_w + bx];
  }

  // ---- product ----
  // the sites in active blocks (exposed: those that need, or need not, be computed from x_t)
  auto product = [&](bool exposed) {
    HaloTile T = H.tile(n, oy0, ox0, g.reference || exposed);
    T.live = 0u;
#pragma unroll
    for (int i = 0; i < WM; ++i) {
      const int m = (H.wm * WM + i) * 16 + H.r16;
      const int ly = m >> lw, lx = m & (tw - 1);
      const int by = ly >> lblk, bx = lx >> lblk;
      bool on = ly < oh && lx < ow && blk_flag[by * tb_w + bx] != 0u;
      if constexpr (TRANS) on = on && block_exposed(c, bi0 + by, bj0 + bx) == exposed;
      T.live |= (uint32_t)on << i;
    }
    if (__ballot(T.live != 0u) == 0ull) return;
    if (exposed) H.start_b(bq);
    typename HC::Acc zo, acc;
    if constexpr (!LATE) H.load_z(zo, T, false);
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int jn = 0; jn < WN; ++jn) acc[i][jn] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    H.product(acc, bq);
    if constexpr (LATE) {
      asm volatile("" ::: "memory");  // not moved up into the product's registers
      H.load_z(zo, T, false);
    }
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int jn = 0; jn < WN; ++jn)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[i][jn][v] = __fadd_rn(zo[i][jn][v], acc[i][jn][v]);
    H.store(T, acc);
  };
  product(false);
  if constexpr (TRANS) {
    // does the tile touch an exposed line's block? (uniform)
    const int y1 = min((oy0 + oh + g.block - 1) >> lblk << lblk, g.h_out);
    const int x1 = min((ox0 + ow + g.block - 1) >> lblk << lblk, g.w_out);
    if (oy0 < c.ey.lo || y1 > c.ey.hi || ox0 < c.ex.lo || x1 > c.ex.hi) {
      lds_barrier();  // every wave is done with the residual halo
      halo(std::false_type{});
      lds_barrier();
      product(true);
    }
    // the state of the off blocks moves to the new slot
    const int cg = c.c_out >> 2, pieces = oh * ow * cg;
    const size_t zimg = (size_t)g.h_out * g.w_out * c.c_out;
    const auto zs = frame_rsrc(c.zsrc + (size_t)n * zimg, (uint32_t)(zimg * 4));
    const auto zd = frame_rsrc(c.z + (size_t)n * zimg, (uint32_t)(zimg * 4));
    const auto yd = frame_rsrc(c.act ? static_cast<uint16_t*>(c.y) + (size_t)n * zimg : nullptr,
                               c.act ? (uint32_t)(zimg * 2) : 0u);
    constexpr int kMove = 4;  // pieces per thread whose loads are in flight together
    const float inv_cg = 1.0f / (float)cg, inv_ow = 1.0f / (float)ow;
    for (int base = 0; base < pieces; base += kTileThreads * kMove) {
      u32x4 v[kMove];
      uint32_t dst[kMove];
#pragma unroll
      for (int u = 0; u < kMove; ++u) {
        const int e = base + u * kTileThreads + threadIdx.x;
        const int site = qdiv(e, inv_cg), ch = (e - site * cg) * 4;
        const int ly = qdiv(site, inv_ow), lx = site - ly * ow;
        const bool off = e < pieces && blk_flag[e < pieces ? (ly >> lblk) * tb_w + (lx >> lblk) : 0] == 0u;
        const int sy = oy0 + ly - c.zdy, sx = ox0 + lx - c.zdx;
        dst[u] = off ? (uint32_t)((((oy0 + ly) * g.w_out + ox0 + lx) * c.c_out + ch) * 4) : kOutOfRange;
        v[u] = __builtin_amdgcn_raw_buffer_load_b128(
            zs, off && sy >= 0 && sy < g.h_out && sx >= 0 && sx < g.w_out
                    ? (uint32_t)(((sy * g.w_out + sx) * c.c_out + ch) * 4) : kOutOfRange, 0, 0);
      }
#pragma unroll
      for (int u = 0; u < kMove; ++u) {
        __builtin_amdgcn_raw_buffer_store_b128(v[u], zd, dst[u], 0, 0);
        if (c.act) {
          uint32_t q[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) q[j] = f32_to_bf16(activate(__uint_as_float(v[u][j]), c.act));
          typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
          __builtin_amdgcn_raw_buffer_store_b64(u32x2v{q[0] | (q[1] << 16), q[2] | (q[3] << 16)}, yd,
                                                dst[u] == kOutOfRange ? kOutOfRange : dst[u] / 2, 0, 0);
        }
      }
    }
  }
}

// Builds by tile extent (16 x 16, 8 x 16 or 8 x 8 sites) and 16-column output
// tiles: rows, columns, ntn, WAVES_M, WAVES_N, WM, WN, KR and LATE of plain
// steps, KR of translated steps (all LATE: with z beside the sums the
// 128-register builds spill), OCC, KI.
#define SC_TILE_BUILDS(X)                                                                                 \
  X(16, 16, 1, 4, 1, 4, 1, 4, false, 4, 3, 6) X(16, 16, 2, 4, 2, 4, 1, 4, false, 4, 4, 3)                 \
  X(16, 16, 4, 4, 2, 4, 2, 2, false, 4, 4, 3) X(16, 16, 8, 4, 2, 4, 4, 2, true, 2, 2, 3)                  \
  X(8, 16, 1, 4, 1, 2, 1, 4, false, 4, 4, 4) X(8, 16, 2, 4, 1, 2, 2, 4, false, 4, 4, 4)                   \
  X(8, 16, 4, 2, 2, 4, 2, 2, false, 4, 4, 3) X(8, 16, 8, 2, 4, 4, 2, 2, false, 4, 4, 3)

// learned gate: halo chunks per thread, all in registers: (rows + 2) x 18
// pixels of up to 64 channels
constexpr int kLearnItems(int rows, int waves) { return ((rows + 2) * 18 * 8 + waves * 64 - 1) / (waves * 64); }

}  // namespace

using TileKernel = void (*)(GateParams, ConvParams, HaloParams);
struct TileBuild {
  int rows, cols, ntn, threads;
  TileKernel plain, trans, chain, learned1, learned3, chain1, chain3;  // (chain: norm gates; chain1, chain3: learned)
};

// the builds of sc_tile_tab.hip and sc_tile_parts.hip
const TileBuild* tile_tab_builds(int* count);
const TileBuild* tile_parts_builds(int* count);

}  // namespace sc
