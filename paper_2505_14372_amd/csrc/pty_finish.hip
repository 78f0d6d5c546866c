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
                                                const float* __restrict__ pos_part, int n_items, float scale,
                                                FinishRun p) {
  constexpr int NBLK = N / 32;
  __shared__ float2 part[7 * kTY * 64];
  static_assert(7 * kTY * 64 >= 512, "one value per thread");
  const int t = threadIdx.x;
  unsigned g = blockIdx.x + p.first;
  const int q = finish_request(p, g);
  g -= p.at[q];
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
  const FinishParts parts = finish_parts(p, r, N);
  if (g < parts.gather) {
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
  g -= parts.gather;
  if (g < parts.probe) {
    const int m = (int)(g / (N * N / kFinishPX));
    const int px = (int)(g % (N * N / kFinishPX)) * kFinishPX + (t & 31), s = t >> 5;
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

template <int N, bool CHAIN>
static void finish(const LaunchCtx& L, FinishRun p, bool rest, float scale) {
  const unsigned blocks = finish_layout(p, L.reqs, L.n_reqs, L.n_items, N, rest);
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
