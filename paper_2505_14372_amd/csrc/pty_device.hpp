// pty_device.hpp -- device functions shared by the two-pass kernels and the
// chain kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "pty_fft.hpp"
#include "pty_internal.h"

namespace pty {

__device__ __forceinline__ void raise_flag(int* flags, int bit) {
  if (flags) atomicOr(flags, bit);
}

// Row spectra of the two-pass kernels in memory. A row pass holds columns l and
// l + 8 of every 16 in neighbouring registers where a line has 8 lanes (N = 64,
// 128, 192); in memory the two halves of each 16 columns are interleaved there,
// so that a lane moves both in one 16-byte access and 8 lanes cover a whole
// 128-byte line. Per step at 192 x 192, 6 modes, 20 slices and 256 positions, with
// two 64-byte halves by separate instructions -> so: adjoint row passes 5.20 ->
// 4.64 ms, forward ones 3.34 -> 2.77 ms. Everything else about a row spectrum is
// in plain column order.
template <int N>
__host__ __device__ __forceinline__ constexpr bool row_pairs() { return Cfg<N>::L == 8; }
// column at position p of a row, and the position of column x
template <int N>
__host__ __device__ __forceinline__ int mem_column(int p) {
  return row_pairs<N>() ? (p & ~15) | ((p & 1) << 3) | ((p >> 1) & 7) : p;
}
template <int N>
__host__ __device__ __forceinline__ int mem_position(int x) {
  return row_pairs<N>() ? (x & ~15) | ((x & 7) << 1) | ((x >> 3) & 1) : x;
}

// Sum over a request's items lo .. hi - 1, in a fixed order, of their
// contributions to the TY x 64 tile of an object slice at (y0, x0), by a
// workgroup of 8 waves: wave w adds, in batch order, those of the items
// b = item0 + w mod 8 whose windows cover the tile (an item that does not cover
// a pixel adds nothing to it, so a pixel's sum does not depend on the tile's
// shape), and wave 0 adds the eight sums in wave order. Contribution `p` of item
// b is tile index(b, item) + p of `src` (tiles `step` apart, parts per item);
// with WS the floats of wsrc are summed alike. part / wpart: LDS for 7 waves.
// Returns whether this thread (of wave 0, column x0 + lane) holds the sums.
template <int N, int TY, bool WS, typename INDEX>
__device__ __forceinline__ bool object_sum(const Item* __restrict__ items, int item0, int lo, int hi, int y0, int x0,
                                           const float2* __restrict__ src, const float* __restrict__ wsrc, size_t step,
                                           int parts, INDEX&& index, float2 (&acc)[TY], float (&wacc)[TY], float2* part,
                                           float* wpart) {
  constexpr int W = 8;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), x = x0 + lane;
#pragma unroll
  for (int k = 0; k < TY; ++k) {
    acc[k] = make_float2(0.f, 0.f);
    wacc[k] = 0.f;
  }
  for (int b0 = item0 + (lo - item0) / (64 * W) * (64 * W); b0 < hi; b0 += 64 * W) {
    const int b = b0 + lane * W + w;
    int ny = 0, nx = 0, t0 = 0;
    bool hit = false;
    if (b >= lo && b < hi) {
      const Item it = items[b];
      ny = it.ny;
      nx = it.nx;
      t0 = index(b, it);
      hit = it.valid && ny < y0 + TY && ny + N > y0 && nx < x0 + 64 && nx + N > x0;
    }
    unsigned long long todo = __ballot(hit);
    // up to four contributions at a time, the loads of all issued before the additions
    int l = -1, m = parts;
    while (todo || m < parts) {
      float2 z[4][TY];
      float zw[4][TY];
      int got = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (m >= parts) {
          if (!todo) break;
          l = __builtin_ctzll(todo);
          todo &= todo - 1;
          m = 0;
        }
        const int wx = x - __builtin_amdgcn_readlane(nx, l), wy0 = y0 - __builtin_amdgcn_readlane(ny, l);
        const size_t at = ((size_t)__builtin_amdgcn_readlane(t0, l) + (size_t)m) * step;
        const float2* c = src + at;
#pragma unroll
        for (int e = 0; e < TY; ++e) {
          const int wy = wy0 + e;
          const bool in = wy >= 0 && wy < N && wx >= 0 && wx < N;
          z[k][e] = in ? c[wy * N + wx] : make_float2(0.f, 0.f);
          if constexpr (WS) zw[k][e] = in ? (wsrc + at)[wy * N + wx] : 0.f;
        }
        ++m;
        ++got;
      }
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (k < got) {
#pragma unroll
          for (int e = 0; e < TY; ++e) {
            acc[e] = cadd(acc[e], z[k][e]);
            if constexpr (WS) wacc[e] += zw[k][e];
          }
        }
    }
  }
  if (w > 0) {
#pragma unroll
    for (int e = 0; e < TY; ++e) {
      part[((w - 1) * TY + e) * 64 + lane] = acc[e];
      if constexpr (WS) wpart[((w - 1) * TY + e) * 64 + lane] = wacc[e];
    }
  }
  __syncthreads();
  if (w != 0) return false;
#pragma unroll
  for (int e = 0; e < TY; ++e)
#pragma unroll
    for (int k = 0; k < W - 1; ++k) {
      acc[e] = cadd(acc[e], part[(k * TY + e) * 64 + lane]);
      if constexpr (WS) wacc[e] += wpart[(k * TY + e) * 64 + lane];
    }
  return true;
}

// One real component of an update.
//   SGD:  th -= lr g
//   Adam: m = b1 m + (1 - b1) g ; v = b2 v + (1 - b2) g^2 ;
//         th -= step_size m / (sqrt(v) inv_sqrt_bc2 + eps), step_size = lr / (1 - b1^t)
// The complements c1 = 1 - b1 and c2 = 1 - b2 are formed in double: 1 - 0.999f in
// float would be off by 1.3e-5 relative.
struct OptCoef {
  float lr, step_size, inv_sqrt_bc2, b1, c1, b2, c2, eps;
};
__device__ __forceinline__ void opt_element(int kind, const OptCoef& k, float& th, float g, float& mo, float& ve) {
  if (kind == OPT_SGD) {
    th -= k.lr * g;
    return;
  }
  const float m = k.b1 * mo + k.c1 * g;
  const float v = k.b2 * ve + k.c2 * g * g;
  mo = m;
  ve = v;
  th -= k.step_size * m / (sqrtf(v) * k.inv_sqrt_bc2 + k.eps);
}

__device__ __forceinline__ OptCoef opt_coef(const OptSeg& s, const OptPar& p) {
  if (s.kind != OPT_ADAM) return OptCoef{(float)s.lr, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  AdamFactors f = s.f;
  if (p.t_dev) f = adam_factors(s.lr, p.b1, p.b2, *p.t_dev + 1);
  return OptCoef{0.f, f.step_size, f.inv_sqrt_bc2, (float)p.b1, (float)(1.0 - p.b1), (float)p.b2, (float)(1.0 - p.b2),
                 p.eps};
}

// Updates a segment: thread `start` of `step`, 4 consecutive elements at a time.
__device__ __forceinline__ void opt_update(const OptSeg& s, const OptPar& p, long long start, long long step) {
  const OptCoef k = opt_coef(s, p);
  const long long hi = s.n;
  for (long long i = 4 * start; i < hi; i += 4 * step) {
    if (s.wide && i + 4 <= hi) {
      float4 th = *reinterpret_cast<float4*>(s.th + i), mo{}, ve{};
      const float4 g = *reinterpret_cast<const float4*>(s.g + i);
      if (s.kind == OPT_ADAM) {
        mo = *reinterpret_cast<float4*>(s.m + i);
        ve = *reinterpret_cast<float4*>(s.v + i);
      }
      opt_element(s.kind, k, th.x, g.x, mo.x, ve.x);
      opt_element(s.kind, k, th.y, g.y, mo.y, ve.y);
      opt_element(s.kind, k, th.z, g.z, mo.z, ve.z);
      opt_element(s.kind, k, th.w, g.w, mo.w, ve.w);
      if (s.kind == OPT_ADAM) {
        *reinterpret_cast<float4*>(s.m + i) = mo;
        *reinterpret_cast<float4*>(s.v + i) = ve;
      }
      *reinterpret_cast<float4*>(s.th + i) = th;
    } else {
      for (long long j = i; j < hi && j < i + 4; ++j) {
        float mo = 0.f, ve = 0.f;
        if (s.kind == OPT_ADAM) {
          mo = s.m[j];
          ve = s.v[j];
        }
        opt_element(s.kind, k, s.th[j], s.g[j], mo, ve);
        if (s.kind == OPT_ADAM) {
          s.m[j] = mo;
          s.v[j] = ve;
        }
      }
    }
  }
}

// Segment and parameters of this workgroup.
__device__ __forceinline__ int opt_segment(const OptTable& t, int& par) {
  int q = -1;
  unsigned at = 0;
#pragma unroll
  for (int k = 0; k < kMaxOpt; ++k) {
    const bool in = t.at[k] <= blockIdx.x * kMaxReqs + (kMaxReqs - 1);
    q += in ? 1 : 0;
    at = in ? t.at[k] : at;
  }
  par = (int)(at % kMaxReqs);
  return q;
}

// Descriptor of batch entry b, written by nt threads (t: this one's index):
// its request, integer window offset and
// subpixel remainder (in double, so n = floor(X + 0.5) is exact for float32
// positions), bounds check, workspace offsets, and the two 1D shift ramps
// exp(-2 pi i f(u) d) with f(u) = fftfreq(N).
__device__ __forceinline__ void make_item(const ReqTable& reqs, int n_reqs, Item* __restrict__ items,
                                          float2* __restrict__ ramps, int b, int N, int* flags, int t, int nt) {
  int q = 0;
  for (int k = 0; k < n_reqs; ++k)
    if (b >= reqs.r[k].item0 && b < reqs.r[k].item0 + reqs.r[k].n_items) q = k;
  const ReqDev& r = reqs.r[q];
  const int local = b - r.item0;
  const int j = r.batch_idx[local];
  const bool ok_idx = (j >= 0 && j < r.J);
  const double X0 = ok_idx ? (double)r.positions[2 * j] : 0.0;
  const double X1 = ok_idx ? (double)r.positions[2 * j + 1] : 0.0;
  const double n0 = floor(X0 + 0.5), n1 = floor(X1 + 0.5);
  const bool ok = ok_idx && (n0 >= 0.0) && (n1 >= 0.0) && (n0 + N <= (double)r.H) &&
                  (n1 + N <= (double)r.W);
  const float d0 = ok ? (float)(X0 - n0) : 0.f, d1 = ok ? (float)(X1 - n1) : 0.f;
  if (t == 0) {
    Item it;
    it.req = q;
    it.j = ok_idx ? j : 0;
    it.ny = ok ? (int)n0 : 0;
    it.nx = ok ? (int)n1 : 0;
    it.dy = d0;
    it.dx = d1;
    it.valid = ok ? 1 : 0;
    it.tile0 = r.tile_base + local * r.M;
    it.ck0 = r.ck_base + (long long)local * r.M;
    items[b] = it;
    if (!ok) raise_flag(flags, kFlagBounds);
  }
  for (int u = t; u < N; u += nt) {
    const int k = (u < (N + 1) / 2) ? u : u - N;
    const float f = (float)k / (float)N;
    float s0, c0, s1, c1;
    sincospif(2.f * f * d0, &s0, &c0);
    sincospif(2.f * f * d1, &s1, &c1);
    ramps[(size_t)b * 2 * N + u] = make_float2(c0, -s0);
    ramps[(size_t)b * 2 * N + N + u] = make_float2(c1, -s1);
  }
}

__device__ __forceinline__ void loss_weight(int kind, float I, float Ie, float eps, float inv_sigma2,
                                            float& ell, float& w) {
  if (kind == PTY_LOSS_POISSON) {
    if (Ie == 0.f) {
      ell = I;
      w = 2.f;
    } else {
      // I - Ie - Ie (ln(I+eps) - ln(Ie+eps)). Near I = Ie the log ratio is
      // log1p of the relative difference (no cancellation); away from it the
      // difference of the two logs, since for I + eps below about 6e-8 of
      // Ie + eps the relative difference rounds to -1 and log1p would return
      // -inf for a finite loss. Invalid counts (negative, NaN) and I + eps = 0
      // give a non-finite loss and raise the flag.
      const float den = Ie + eps;
      const float x = (I - Ie) / den;
      const float lr = fabsf(x) < 0.5f ? log1pf(x) : logf(I + eps) - logf(den);
      ell = (I - Ie) - Ie * lr;
      w = 2.f * (1.f - Ie / (I + eps));
    }
  } else if (kind == PTY_LOSS_GAUSSIAN) {
    float d = I - Ie;
    ell = 0.5f * d * d * inv_sigma2;
    w = 2.f * d * inv_sigma2;
  } else {
    float c = (kind == PTY_LOSS_ANSCOMBE) ? 0.375f : 0.f;
    float a = sqrtf(I + c), ae = sqrtf(Ie + c);
    ell = 0.5f * (a - ae) * (a - ae);
    float den = eps + a;
    w = (den > 0.f) ? 1.f - ae / den : 0.f;
  }
}

}  // namespace pty
