// pty_finish.hip -- the last sums of the adjoint, independent of each other and
// taken in one launch: object gradient, probe-spectrum gradient, loss and
// position gradients.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "pty_device.hpp"
#include "pty_internal.h"

namespace pty {

constexpr int kTY = 4;            // rows of an object-gradient tile
constexpr int kProbeSplit = 16;   // interleaved sums of the probe-spectrum gradient

// The work is split over workgroup ranges; every sum has a fixed order, so
// repeated calls give the same bits.
//   - object gradient (stored contributions): one workgroup per 4 x 64 tile and
//     slice (object_sum). The chain kernels leave one contribution per mode, the
//     two-pass kernels one per position (already scaled). With one list of
//     positions per workgroup behind barriers, 8 x 64 tiles and 4 waves, this
//     launch took 36 us at 64 x 64, 1 slice, 256 positions (now 15), 53 us at 2
//     modes, 8 slices (35; 118 MB of contributions) and 1.15 ms at 128 x 128, 4
//     modes, 8 slices, 1024 positions (1.07; 4.3 GB, read at 4.0 TB/s);
//   - probe-spectrum gradient: gphat_m(u) = scale sum_b h_hat_{b,m}(u) conj(R_b(u)),
//     32 pixels x 16 interleaved sums over the items, added in order; for the
//     requests whose final pass kept these sums (chain_final), the 16 tiles it
//     left are added the same way;
//   - loss; position gradients.
// CHAIN: spectra are transposed, as the chain kernels hold them.
template <int N, bool CHAIN>
__global__ __launch_bounds__(512) void k_finish(const Item* __restrict__ items, const ReqTable reqs,
                                                const float2* __restrict__ ws, const float2* __restrict__ ck,
                                                const float2* __restrict__ ramps, const float* __restrict__ loss_part,
                                                const float* __restrict__ pos_part, int n_items, int max_modes,
                                                float scale, FinishRun p) {
  constexpr int NBLK = N / 32;
  __shared__ float2 part[7 * kTY * 64];
  static_assert(7 * kTY * 64 >= 512, "one value per thread");
  const int t = threadIdx.x;
  int g = blockIdx.x;
  const int n_gather = p.n_reqs * p.slices * p.ty * p.tx;
  if (g < n_gather) {
    const int tx = g % p.tx, ty = (g / p.tx) % p.ty, s = (g / (p.tx * p.ty)) % p.slices, q = g / (p.tx * p.ty * p.slices);
    const ReqDev& r = reqs.r[q];
    const int i = p.lo + s, x0 = tx * 64, y0 = ty * kTY, x = x0 + (t & 63);
    if (i >= r.S || !r.gobj || x0 >= r.W || y0 >= r.H) return;
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
  g -= n_gather;
  const int n_probe = p.n_reqs * max_modes * (N * N / 32);
  if (g < n_probe) {
    const ReqDev& r = reqs.r[g / (max_modes * (N * N / 32))];
    const int m = (g / (N * N / 32)) % max_modes;
    if (m >= r.M || !r.gphat) return;
    const int px = (g % (N * N / 32)) * 32 + (t & 31), s = t >> 5;
    const int ux = CHAIN ? px / N : mem_column<N>(px % N), uy = CHAIN ? px % N : px / N;
    float2 acc = make_float2(0.f, 0.f);
    if (!CHAIN && r.chain_final) {
      if (s < r.n_items) acc = ws[(size_t)(items[r.item0 + s].tile0 + m) * N * N + px];
    } else {
#pragma unroll 4
      for (int b = r.item0 + s; b < r.item0 + r.n_items; b += kProbeSplit) {
        const Item it = items[b];
        const float2 R = xmul(ramps[(size_t)b * 2 * N + uy], ramps[(size_t)b * 2 * N + N + ux]);
        const float2 h = ws[(size_t)(it.tile0 + m) * N * N + px];
        if (it.valid) acc = cadd(acc, xmul(h, cconj(R)));
      }
    }
    part[t] = acc;
    __syncthreads();
    if (s == 0) {
      float2 z = part[t];
#pragma unroll
      for (int k = 1; k < kProbeSplit; ++k) z = cadd(z, part[32 * k + t]);
      r.gphat[(size_t)m * N * N + (CHAIN ? px : uy * N + ux)] = cscale(z, adj_scale(r, scale));
    }
    return;
  }
  g -= n_probe;
  if (g < p.n_reqs) {
    const ReqDev& r = reqs.r[g];
    if (!r.loss_out) return;
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
    return;
  }
  // per item: dL/dX = 2 pi scale times the sum over modes (and column blocks) of
  // the partials; to g_pos[local] and / or added to a dense [J][2] gradient
  g -= p.n_reqs;
  const int b = g * 512 + t;
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
}

template <int N, bool CHAIN>
static void finish(const LaunchCtx& L, FinishRun p, bool gather, bool rest, float scale) {
  p.n_reqs = L.n_reqs;
  p.tx = p.ty = 0;
  if (gather)
    for (int q = 0; q < L.n_reqs; ++q) {
      if (!L.reqs.r[q].gobj) continue;
      p.tx = std::max(p.tx, (L.reqs.r[q].W + 63) / 64);
      p.ty = std::max(p.ty, (L.reqs.r[q].H + kTY - 1) / kTY);
    }
  size_t blocks = (size_t)p.n_reqs * p.slices * p.ty * p.tx;
  if (rest) blocks += (size_t)p.n_reqs * L.max_modes * (N * N / 32) + p.n_reqs + (L.n_items + 511) / 512;
  if (blocks == 0) return;
  hipLaunchKernelGGL((k_finish<N, CHAIN>), dim3((unsigned)blocks), dim3(512), 0, L.stream, L.items, L.reqs, L.ws,
                     static_cast<const float2*>(L.ck), L.ramps, L.loss_part, L.pos_part, L.n_items, L.max_modes, scale,
                     p);
}

void launch_finish(const LaunchCtx& L, int N, const FinishRun& p, bool gather, bool rest, float scale) {
  if (L.chain) {
    if (N == 64) finish<64, true>(L, p, gather, rest, scale);
    else finish<128, true>(L, p, gather, rest, scale);
    return;
  }
  switch (N) {
    case 64: finish<64, false>(L, p, gather, rest, scale); break;
    case 128: finish<128, false>(L, p, gather, rest, scale); break;
    case 192: finish<192, false>(L, p, gather, rest, scale); break;
    default: finish<256, false>(L, p, gather, rest, scale); break;
  }
}

}  // namespace pty
