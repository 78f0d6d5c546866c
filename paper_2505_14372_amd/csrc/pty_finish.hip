// pty_finish.hip -- the last sums of the adjoint, independent of each other and
// taken in one launch: object gradient, probe-spectrum gradient, loss and
// position gradients.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "pty_device.hpp"
#include "pty_internal.h"

namespace pty {

constexpr int kTY = kFinishTY;    // rows of an object-gradient tile
constexpr int kProbeSplit = 16;   // interleaved sums of the probe-spectrum gradient

// The work is split over workgroup ranges, each request's by its own sizes (by
// the largest of a group's the product of all the maxima can exceed what a launch
// takes); every sum has a fixed order, so repeated calls give the same bits.
//   - object gradient (stored contributions), where sum_in_strips does not hold: one
//     workgroup per 4 x 64 tile and slice (object_sum). The chain kernels leave one contribution per mode, the
//     two-pass kernels one per position (already scaled). With one list of
//     positions per workgroup behind barriers, 8 x 64 tiles and 4 waves, this
//     launch took 36 us at 64 x 64, 1 slice, 256 positions (now 15), 53 us at 2
//     modes, 8 slices (35; 118 MB of contributions) and 1.15 ms at 128 x 128, 4
//     modes, 8 slices, 1024 positions (1.10; 4.3 GB of contributions, 5.6 GB of counted
//     traffic at 5.1 TB/s);
//   - probe-spectrum gradient: gphat_m(u) = scale sum_b h_hat_{b,m}(u) conj(R_b(u)),
//     16 interleaved sums over the items, added in order (finish_pixels); for the
//     requests whose final pass kept these sums (chain_final), the 16 tiles it
//     left are added the same way;
//   - loss; position gradients.
// CHAIN: spectra are transposed, as the chain kernels hold them.
template <int N, bool CHAIN>
__global__ __launch_bounds__(512) void k_finish(const Item* __restrict__ items, const ReqTable reqs,
                                                const float2* __restrict__ ws, const float2* __restrict__ ck,
                                                const float2* __restrict__ ramps, const float* __restrict__ loss_part,
                                                const float* __restrict__ pos_part, int n_items, float scale,
                                                FinishRun p) {
  constexpr int NBLK = N / 32;
  __shared__ float2 part[7 * kTY * 64];
  static_assert(7 * kTY * 64 >= 512, "one value per thread");
  const int t = threadIdx.x;
  const FinishWork work = finish_work(p, blockIdx.x + p.first);
  const int q = work.req;
  const unsigned g = work.index;
  if (q == p.n_reqs) {
    // per item: dL/dX = 2 pi scale times the sum over modes (and column blocks) of
    // the partials; to g_pos[local] and / or added to a dense [J][2] gradient
    const int b = (int)g * 512 + t;
    if (b >= n_items) return;
    const Item it = items[b];
    const ReqDev& r = reqs.r[it.req];
    float g0 = 0.f, g1 = 0.f;
    if (it.valid)
      for (int m = 0; m < r.M; ++m)
        for (int k = 0; k < (CHAIN ? 1 : NBLK); ++k) {
          const float* pp = pos_part + ((size_t)(it.tile0 + m) * NBLK + k) * 2;
          g0 += pp[0];
          g1 += pp[1];
        }
    const float f = 6.283185307179586f * adj_scale(r, scale);
    g0 *= f;
    g1 *= f;
    const int local = b - r.item0;
    if (r.gpos) {
      if (r.accumulate) { r.gpos[2 * local] += g0; r.gpos[2 * local + 1] += g1; }
      else { r.gpos[2 * local] = g0; r.gpos[2 * local + 1] = g1; }
    }
    if (r.gpos_dense && it.valid) {
      atomicAdd(r.gpos_dense + 2 * it.j, g0);
      atomicAdd(r.gpos_dense + 2 * it.j + 1, g1);
    }
    return;
  }
  const ReqDev& r = reqs.r[q];
  const FinishParts parts = finish_parts(p, r, q, N);
  if (work.tile) {
    const int i = p.lo + (int)(g / (parts.tx * parts.ty)), x0 = (int)(g % parts.tx) * 64;
    const int y0 = (int)((g / parts.tx) % parts.ty) * kTY, x = x0 + (t & 63);
    const bool sg = p.seg && i % r.ck_every != 0;
    const float2* src = sg ? p.seg + (size_t)(i - p.seg_base) * N * N
                           : ck + (size_t)(i / r.ck_every) * r.n_items * r.M * N * N;
    float2 acc[kTY];
    float none[kTY];
    if (!object_sum<N, kTY, false>(items, r.item0, r.item0, r.item0 + r.n_items, y0, x0, src, nullptr,
                                   (size_t)(sg ? p.seg_len : 1) * N * N, CHAIN ? r.M : 1,
                                   [&](int, const Item& it) { return sg ? it.tile0 : (int)it.ck0; }, acc, none, part,
                                   nullptr) ||
        x >= r.W)
      return;
    const float sc = CHAIN ? adj_scale(r, scale) : 1.f;
    float2* go = r.gobj + (size_t)i * r.H * r.W;
#pragma unroll
    for (int e = 0; e < kTY; ++e) {
      const int y = y0 + e;
      if (y >= r.H) continue;
      const float2 z = CHAIN ? cscale(acc[e], sc) : acc[e];
      go[(size_t)y * r.W + x] = r.accumulate ? cadd(go[(size_t)y * r.W + x], z) : z;
    }
    return;
  }
  if (g < parts.probe) {
    const int per = N * N / finish_pixels(p.wide), m = (int)g / per;
    const int px = p.wide ? (int)g % per * 512 + t : (int)g % per * 32 + (t & 31), s = t >> 5;
    const int ux = CHAIN ? px / N : mem_column<N>(px % N), uy = CHAIN ? px % N : px / N;
    const bool sums = !CHAIN && r.chain_final;
    auto term = [&](int b) {
      const Item it = items[b];
      const float2 R = xmul(ramps[(size_t)b * 2 * N + uy], ramps[(size_t)b * 2 * N + N + ux]);
      const float2 h = ws[(size_t)(it.tile0 + m) * N * N + px];
      return it.valid ? xmul(h, cconj(R)) : make_float2(0.f, 0.f);
    };
    float2 z = make_float2(0.f, 0.f);
    if (p.wide) {
      for (int s0 = 0; s0 < kProbeSplit; s0 += 4) {
        float2 a[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) a[k] = make_float2(0.f, 0.f);
        if (sums) {
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (s0 + k < r.n_items) a[k] = ws[(size_t)(items[r.item0 + s0 + k].tile0 + m) * N * N + px];
        } else {
          for (int b = s0; b < r.n_items; b += kProbeSplit) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
              if (b + k < r.n_items) a[k] = cadd(a[k], term(r.item0 + b + k));
          }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) z = s0 + k == 0 ? a[0] : cadd(z, a[k]);
      }
    } else {
      float2 acc = make_float2(0.f, 0.f);
      if (sums) {
        if (s < r.n_items) acc = ws[(size_t)(items[r.item0 + s].tile0 + m) * N * N + px];
      } else {
#pragma unroll 4
        for (int b = r.item0 + s; b < r.item0 + r.n_items; b += kProbeSplit) acc = cadd(acc, term(b));
      }
      part[t] = acc;
      __syncthreads();
      if (s > 0) return;
      z = part[t];
#pragma unroll
      for (int k = 1; k < kProbeSplit; ++k) z = cadd(z, part[32 * k + t]);
    }
    r.gphat[(size_t)m * N * N + (CHAIN ? px : uy * N + ux)] = cscale(z, adj_scale(r, scale));
    return;
  }
  // the loss
  double* red = reinterpret_cast<double*>(part);
  double acc = 0.0;
  const float* lp = loss_part + (size_t)r.item0 * NBLK;
  for (int e = t; e < r.n_items * NBLK; e += 512) acc += (double)lp[e];
  red[t] = acc;
  __syncthreads();
  for (int s = 256; s > 0; s >>= 1) {
    if (t < s) red[t] += red[t + s];
    __syncthreads();
  }
  if (t == 0) *r.loss_out = red[0];
}

// Object gradient of a large object under few windows: one wave per strip of 16 x 64
// values of a slice. A strip that no window touches costs a look at the items and
// its zeros; for the others the wave lists the items of the strip and adds, tile
// by tile of 4 rows, what a workgroup of k_finish adds, in the same order (the
// items b = item0 + w mod 8 in batch order for each w, then the eight sums), so
// that a pixel's bits are those of object_sum.
template <int N, bool WS>
__global__ __launch_bounds__(256) void k_object_strips(const Item* __restrict__ items, const ReqDev r, const StripRun p,
                                                       unsigned tx, unsigned ty) {
  constexpr int TY = kTY, MOST = 64;
  __shared__ int list_[4][MOST];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned g = blockIdx.x * 4 + wave;
  if (g >= (unsigned)p.slices * tx * ty) return;
  int* list = list_[wave];
  const int i = p.lo + (int)(g / (tx * ty)), x0 = (int)(g % tx) * 64, x = x0 + lane;
  const int top = (int)((g / tx) % ty) * kStripRows, end = min(top + kStripRows, r.H);
  const size_t slice = (size_t)i * r.H * r.W;
  auto covers = [&](const Item& it, int y0, int rows) {
    return it.valid && it.ny < y0 + rows && it.ny + N > y0 && it.nx < x0 + 64 && it.nx + N > x0;
  };
  int n = 0;
  for (int b0 = p.item_lo; b0 < p.item_hi; b0 += 64) {
    const int b = b0 + lane;
    const bool hit = b < p.item_hi && covers(items[b], top, end - top);
    const unsigned long long m = __ballot(hit);
    const int at = n + __popcll(m & ((1ull << lane) - 1ull));
    if (hit && at < MOST) list[at] = b;
    n += __popcll(m);
  }
  if (n == 0) {
    if (!p.add && x < r.W)
      for (int y = top; y < end; ++y) r.gobj[slice + (size_t)y * r.W + x] = make_float2(0.f, 0.f);
    return;
  }
  WaveSync{}();
  const bool sg = p.seg && i % r.ck_every != 0;
  const float2* src = p.scratch ? p.src
                      : sg      ? p.seg + (size_t)(i - p.seg_base) * N * N
                                : p.src + (size_t)(i / r.ck_every) * r.n_items * r.M * N * N;
  const size_t step = (size_t)(sg ? p.seg_len : 1) * N * N;
  // a block of up to 64 items in the lanes: the listed ones, or all in turn
  int ny = 0, nx = 0, t0 = 0, cls = 0;
  bool here = false;
  auto take = [&](int b, bool on) {
    here = on;
    if (!on) return;
    const Item it = items[b];
    ny = it.ny;
    nx = it.nx;
    t0 = p.scratch ? b : sg ? it.tile0 : (int)it.ck0;
    cls = (b - r.item0) & 7;
    here = covers(it, top, end - top);
  };
  const float sc = p.scaled ? adj_scale(r, p.scale) : 1.f;
  const bool listed = n <= MOST;
  if (listed) take(list[min(lane, n - 1)], lane < n);
  for (int y0 = top; y0 < end; y0 += TY) {
    float2 sum[TY], acc[TY];
    float wsum[TY], wacc[TY];
#pragma unroll
    for (int e = 0; e < TY; ++e) {
      sum[e] = acc[e] = make_float2(0.f, 0.f);
      wsum[e] = wacc[e] = 0.f;
    }
    // the contributions in turn: class w, item in lane l, part m
    int w = -1, l = 0, m = p.parts, b0 = p.item_hi;
    unsigned long long todo = 0;
    auto next = [&]() {
      if (++m < p.parts) return true;
      m = 0;
      while (!todo) {
        if (listed) {
          ++w;
        } else if ((b0 += 64) >= p.item_hi) {
          b0 = p.item_lo;
          ++w;
        }
        if (w == 8) return false;
        if (!listed) take(b0 + lane, b0 + lane < p.item_hi);
        todo = __ballot(here && cls == w && ny < y0 + TY && ny + N > y0);
      }
      l = __builtin_ctzll(todo);
      todo &= todo - 1;
      return true;
    };
    auto fold = [&]() {
#pragma unroll
      for (int e = 0; e < TY; ++e) {
        sum[e] = cadd(sum[e], acc[e]);
        acc[e] = make_float2(0.f, 0.f);
        if constexpr (WS) {
          wsum[e] += wacc[e];
          wacc[e] = 0.f;
        }
      }
    };
    // up to four at a time, the loads of all issued before the additions
    int of = 0, got = 4;   // class of the sum in acc (a class without items adds zero)
    while (got == 4) {
      float2 z[4][TY];
      float zw[4][TY];
      int c[4];
      got = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (got < k || !next()) continue;
        const int wx = x - __builtin_amdgcn_readlane(nx, l), wy0 = y0 - __builtin_amdgcn_readlane(ny, l);
        const size_t at = ((size_t)__builtin_amdgcn_readlane(t0, l) + (size_t)m) * step;
#pragma unroll
        for (int e = 0; e < TY; ++e) {
          const int wy = wy0 + e;
          const bool in = wy >= 0 && wy < N && wx >= 0 && wx < N;
          z[k][e] = in ? src[at + wy * N + wx] : make_float2(0.f, 0.f);
          if constexpr (WS) zw[k][e] = in ? p.wsrc[at + wy * N + wx] : 0.f;
        }
        c[k] = w;
        ++got;
      }
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (k < got) {
          if (c[k] != of) {
            fold();
            of = c[k];
          }
#pragma unroll
          for (int e = 0; e < TY; ++e) {
            acc[e] = cadd(acc[e], z[k][e]);
            if constexpr (WS) wacc[e] += zw[k][e];
          }
        }
    }
    fold();
    if (x >= r.W) continue;
#pragma unroll
    for (int e = 0; e < TY; ++e) {
      if (y0 + e >= r.H) continue;
      const size_t at = slice + (size_t)(y0 + e) * r.W + x;
      const float2 z = p.scaled ? cscale(sum[e], sc) : sum[e];
      r.gobj[at] = p.add ? cadd(r.gobj[at], z) : z;
      if constexpr (WS) {
        if (r.wsum) r.wsum[at] += wsum[e];
      }
    }
  }
}

template <int N>
static void object_strips(hipStream_t s, const Item* items, const ReqDev& r, const StripRun& p) {
  const unsigned tx = (unsigned)(r.W + 63) / 64, ty = (unsigned)(r.H + kStripRows - 1) / kStripRows;
  const unsigned blocks = ((unsigned)p.slices * tx * ty + 3) / 4;
  if (p.wsrc) hipLaunchKernelGGL((k_object_strips<N, true>), dim3(blocks), dim3(256), 0, s, items, r, p, tx, ty);
  else hipLaunchKernelGGL((k_object_strips<N, false>), dim3(blocks), dim3(256), 0, s, items, r, p, tx, ty);
}
void launch_object_strips(hipStream_t s, int N, const Item* items, const ReqDev& r, StripRun p) {
  switch (N) {
    case 64: object_strips<64>(s, items, r, p); break;
    case 128: object_strips<128>(s, items, r, p); break;
    case 192: object_strips<192>(s, items, r, p); break;
    default: object_strips<256>(s, items, r, p); break;
  }
}

template <int N, bool CHAIN>
static void finish(const LaunchCtx& L, FinishRun p, bool rest, float scale) {
  const unsigned blocks = finish_layout(p, L.reqs, L.n_reqs, L.n_items, N, CHAIN, rest);
  for (int q = 0; q < L.n_reqs; ++q) {
    const ReqDev& r = L.reqs.r[q];
    if (!((p.strips >> q) & 1u)) continue;
    StripRun o{};
    o.src = static_cast<const float2*>(L.ck);
    o.seg = p.seg;
    o.seg_len = p.seg_len;
    o.seg_base = p.seg_base;
    o.parts = CHAIN ? r.M : 1;
    o.lo = p.lo;
    o.slices = std::min(r.S - p.lo, p.slices);
    o.item_lo = r.item0;
    o.item_hi = r.item0 + r.n_items;
    o.add = r.accumulate;
    o.scaled = CHAIN;
    o.scale = scale;
    launch_object_strips(L.stream, N, L.items, r, o);
  }
  for (p.first = 0; p.first < blocks; p.first += kFinishBlocks)
    hipLaunchKernelGGL((k_finish<N, CHAIN>), dim3(std::min(blocks - p.first, kFinishBlocks)), dim3(512), 0, L.stream,
                       L.items, L.reqs, L.ws, static_cast<const float2*>(L.ck), L.ramps, L.loss_part, L.pos_part,
                       L.n_items, scale, p);
}

void launch_finish(const LaunchCtx& L, int N, FinishRun p, bool rest, float scale) {
  if (L.chain) {
    if (N == 64) finish<64, true>(L, p, rest, scale);
    else finish<128, true>(L, p, rest, scale);
    return;
  }
  switch (N) {
    case 64: finish<64, false>(L, p, rest, scale); break;
    case 128: finish<128, false>(L, p, rest, scale); break;
    case 192: finish<192, false>(L, p, rest, scale); break;
    default: finish<256, false>(L, p, rest, scale); break;
  }
}

}  // namespace pty
