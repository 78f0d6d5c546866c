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
