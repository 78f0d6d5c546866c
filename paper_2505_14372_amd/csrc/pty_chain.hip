// pty_chain.hip -- chain kernels: every slice of one (position, mode) tile in
// one launch, the tile held in registers (pty_chain.hpp), for N = 64, 128.
//
// A slice step is F^-1 H F between two products with the object, all of it
// local to a workgroup, so the tile itself never travels to memory between
// slices: the forward chain writes the entry waves (checkpoints, real space,
// row-major), the adjoint chain reads each one and leaves the mode's object-
// gradient contribution conj(psi_i) g in its place, and one launch over all
// slices sums the contributions tile by tile in batch order (no atomics).
// Spectra between the launches (probe, far field, h_hat) are stored
// transposed, [k_x][k_y], the order in which the lanes hold them.
//
// A step is: k_chain_begin (probe spectra, item descriptors, zeroed position
// gradient), k_chain (forward and adjoint; with several modes a launch each and
// k_chain_far, the noise model, between them), k_finish (object gradient,
// probe-spectrum sum, loss, position gradient: independent of each other, one
// launch) and k_chain_plain (probe gradient), where the two-pass kernels take
// 4 S + 11 launches.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "pty_chain.hpp"
#include "pty_device.hpp"
#include "pty_internal.h"

namespace pty {

namespace {

// Constant tables read at wave-uniform addresses: loaded through the constant
// address space, so that the values sit in scalar registers.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef const f32x2 __attribute__((address_space(4))) * ConstTab;
__device__ __forceinline__ ConstTab const_tab(const float2* p) { return (ConstTab)(uintptr_t)p; }
__device__ __forceinline__ float2 as_f2(f32x2 v) { return make_float2(v.x, v.y); }
// The same table, for a use inside a loop: its loads stay where they are used
// (hoisted out of the slice loop, the roots of both stages would fill the
// scalar registers and spill).
__device__ __forceinline__ ConstTab here(ConstTab p) {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" : "+s"(p));
  return p;
}

enum Side { A1, B1, B2, C2 };
template <int N, int SIDE>
__device__ __forceinline__ constexpr int xoff(int e) {
  return SIDE == A1 ? off_a1<N>(e) : SIDE == B1 ? off_b1<N>(e) : SIDE == B2 ? off_b2<N>(e) : off_c2<N>(e);
}

// Exchange: register e goes to wb + xoff<W>(e) and comes from rb + xoff<R>(e).
// The first barrier waits for the readers of the exchange before.
template <int N, int W, int R>
__device__ __forceinline__ void exchange(float2 (&v)[Ch<N>::EL], typename Ch<N>::Elem* lds, int wb, int rb) {
  constexpr int EL = Ch<N>::EL;
  __syncthreads();
  if constexpr (Ch<N>::SPLIT) {
    // (volatile: merged in pairs, the accesses would need a base register for
    // each pair, more than there are)
    typedef volatile float __attribute__((address_space(3))) Lds;
    Lds* put = (Lds*)(lds + wb);
    Lds* get = (Lds*)(lds + rb);
    float u[EL];
#pragma unroll
    for (int e = 0; e < EL; ++e) put[xoff<N, W>(e)] = v[e].x;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < EL; ++e) u[e] = get[xoff<N, R>(e)];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < EL; ++e) put[xoff<N, W>(e)] = v[e].y;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < EL; ++e) v[e] = make_float2(u[e], get[xoff<N, R>(e)]);
  } else {
#pragma unroll
    for (int e = 0; e < EL; ++e) lds[wb + xoff<N, W>(e)] = v[e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < EL; ++e) v[e] = lds[rb + xoff<N, R>(e)];
  }
}

// The transform of one workgroup's tile.
template <int N>
struct Fft2 {
  using Elem = typename Ch<N>::Elem;
  const ChThread<N> th;
  Elem* lds;
  ConstTab ta, tc;
  __device__ __forceinline__ Fft2(Elem* l, const float2* tab)
      : th(threadIdx.x & 63, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)), lds(l),
        ta(const_tab(tab) + th.yl * Ch<N>::EL), tc(const_tab(tab) + N + th.j1 * 16) {}

  __device__ __forceinline__ void forward(float2 (&v)[Ch<N>::EL]) const {   // A -> C
    constexpr int EL = Ch<N>::EL;
    float2 w[EL > 16 ? EL : 16];
    const ConstTab a = here(ta);
#pragma unroll
    for (int k = 1; k < EL; ++k) w[k] = as_f2(a[k]);
    ch_stage_a<N, false>(v, w);
    exchange<N, A1, B1>(v, lds, th.a1(), th.b1());
    ch_stage_b<N, false>(v);
    exchange<N, B2, C2>(v, lds, th.b2(), th.c2());
    const ConstTab c = here(tc);
#pragma unroll
    for (int k = 1; k < 16; ++k) w[k] = as_f2(c[k]);
    ch_stage_c<N, false>(v, w);
  }
  __device__ __forceinline__ void inverse(float2 (&v)[Ch<N>::EL]) const {   // C -> A
    constexpr int EL = Ch<N>::EL;
    float2 w[EL > 16 ? EL : 16];
    const ConstTab c = here(tc);
#pragma unroll
    for (int k = 1; k < 16; ++k) w[k] = as_f2(c[k]);
    ch_stage_c<N, true>(v, w);
    exchange<N, C2, B2>(v, lds, th.c2(), th.b2());
    ch_stage_b<N, true>(v);
    exchange<N, B1, A1>(v, lds, th.b1(), th.a1());
    const ConstTab a = here(ta);
#pragma unroll
    for (int k = 1; k < EL; ++k) w[k] = as_f2(a[k]);
    ch_stage_a<N, true>(v, w);
  }
  __device__ __forceinline__ void load_spec(float2 (&v)[Ch<N>::EL], const float2* s) const {
#pragma unroll
    for (int e = 0; e < Ch<N>::EL; ++e) v[e] = s[th.kx(e & 15) * N + th.ky(e >> 4)];
  }
  __device__ __forceinline__ void store_spec(const float2 (&v)[Ch<N>::EL], float2* s, float scale) const {
#pragma unroll
    for (int e = 0; e < Ch<N>::EL; ++e) s[th.kx(e & 15) * N + th.ky(e >> 4)] = cscale(v[e], scale);
  }
  // Real-space rows through a raw buffer: one lane offset, and the row as a
  // scalar offset (64-bit row addresses would take two scalar registers each
  // and, kept across the slice loop, spill). W: row length in values.
  struct Rows {
    __amdgpu_buffer_rsrc_t r;
    unsigned v;
    int step;   // bytes from register to register (four rows)
    __device__ __forceinline__ Rows(const float2* s, int W, const ChThread<N>& th)
        : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<float2*>(s), (short)0, ((N - 1) * W + N) * 8, 0x00020000)),
          v((unsigned)th.x * 8u + (unsigned)(th.yl * W) * 8u), step(32 * W) {}
    __device__ __forceinline__ float2 ld(int k) const {
      const u32x2 z = __builtin_amdgcn_raw_buffer_load_b64(r, v, k * step, 0);
      return make_float2(__uint_as_float(z.x), __uint_as_float(z.y));
    }
    __device__ __forceinline__ void st(int k, float2 x) const {
      const u32x2 z = {__float_as_uint(x.x), __float_as_uint(x.y)};
      __builtin_amdgcn_raw_buffer_store_b64(z, r, v, k * step, 0);
    }
  };
  __device__ __forceinline__ void load_real(float2 (&v)[Ch<N>::EL], const float2* s) const {
    const Rows row(s, N, th);
#pragma unroll
    for (int r = 0; r < Ch<N>::EL; ++r) v[r] = row.ld(r);
  }
  __device__ __forceinline__ void store_real(const float2 (&v)[Ch<N>::EL], float2* s) const {
    const Rows row(s, N, th);
#pragma unroll
    for (int r = 0; r < Ch<N>::EL; ++r) row.st(r, v[r]);
  }
  // v <- v s (or conj(s) v) with s in real space, 16 loads in flight at a time
  template <bool CONJ>
  __device__ __forceinline__ void times_real(float2 (&v)[Ch<N>::EL], const float2* s, int W) const {
    asm volatile("" : "+s"(W));   // row offsets formed here, not kept across the slice loop
    const Rows row(s, W, th);
#pragma unroll
    for (int r0 = 0; r0 < Ch<N>::EL; r0 += 16) {
      float2 o[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) o[r] = row.ld(r0 + r);
#pragma unroll
      for (int r = 0; r < 16; ++r) v[r0 + r] = CONJ ? xjmul(o[r], v[r0 + r]) : xmul(v[r0 + r], o[r]);
      if (r0 + 16 < Ch<N>::EL) __builtin_amdgcn_sched_barrier(0);
    }
  }
  // s <- conj(s) v
  __device__ __forceinline__ void contribute(const float2 (&v)[Ch<N>::EL], float2* s) const {
    const Rows row(s, N, th);
#pragma unroll
    for (int r0 = 0; r0 < Ch<N>::EL; r0 += 16) {
      float2 o[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) o[r] = row.ld(r0 + r);
#pragma unroll
      for (int r = 0; r < 16; ++r) row.st(r0 + r, xjmul(o[r], v[r0 + r]));
      sched_fence();
    }
  }
};

// times H (or conj H) of a gap, rebuilt from its separable factors:
// H = [|k_x| <= K_y] Hy(k_y) Hx(k_x); Hx is wave-uniform
template <int N, bool CONJ>
__device__ __forceinline__ void propagate(float2 (&v)[Ch<N>::EL], const ReqDev& r, int gap, const ChThread<N>& th) {
  asm volatile("" : "+s"(gap));   // table rows addressed here, not by pointers kept across the slice loop
  const ConstTab px = const_tab(r.prop_x) + (size_t)gap * N;
  const float4* py = r.prop_y + (size_t)gap * N;
#pragma unroll
  for (int kb = 0; kb < Ch<N>::KB; ++kb) {
    const float4 q = py[th.ky(kb)];
    const int K = __float_as_int(q.z);
#pragma unroll
    for (int j2 = 0; j2 < 16; ++j2) {
      if (j2 % 4 == 0) sched_fence();   // (all 16 factors and row tests at once would spill)
      const int ux = th.kx(j2);
      const int akx = abs(ux < N / 2 ? ux : ux - N);
      const float2 hx = as_f2(px[ux]), hy = make_float2(q.x, q.y), z = v[16 * kb + j2];
      const float2 w = CONJ ? xjmul(hy, xjmul(hx, z)) : xmul(xmul(z, hx), hy);
      v[16 * kb + j2] = akx > K ? make_float2(0.f, 0.f) : w;
    }
  }
}

// Does the chain take the far field and the noise model too? With one mode
// nothing has to be summed between workgroups (one launch instead of three:
// 64 x 64, 1 slice, 256 positions, 49 -> 31 us). Several modes in one workgroup,
// summing far fields and object-gradient contributions through LDS, measured
// slower: the tiles then wait for each other at every barrier (64 x 64, 2 modes,
// 8 slices: 155 -> 185 us; 128 x 128, 2 modes, 5 slices: 254 -> 439 us).
constexpr bool far_in_chain_at(int N) { return N == 64; }
template <int N>
__host__ __device__ __forceinline__ bool far_in_chain(int M) { return far_in_chain_at(N) && M == 1; }

// (item, mode) of a workgroup: consecutive workgroups go to the 8 XCDs in
// turn, so the modes of one item, which read the same object patch, take every
// eighth workgroup (one XCD's L2).
__device__ __forceinline__ bool chain_tile(int n_items, int max_modes, bool reverse, int& b, int& m) {
  const int g = blockIdx.x >> 3;
  b = (blockIdx.x & 7) + 8 * (g / max_modes);
  m = g % max_modes;
  if (b >= n_items) return false;
  if (reverse) b = n_items - 1 - b;
  return true;
}

}  // namespace

// ============================================================ kernels

// First launch of a step, its work split over workgroup ranges: the spectra
// of the probe modes (transposed), the item descriptors and ramps (one wave
// per item), zeros for the dense position gradients.
template <int N>
__global__ __launch_bounds__(Ch<N>::T) void k_chain_begin(const ReqTable reqs, int n_reqs, int max_modes, int n_items,
                                                          int item_blocks, int fill, Item* __restrict__ items,
                                                          float2* __restrict__ ramps, const float2* __restrict__ tab,
                                                          int* flags) {
  __shared__ typename Ch<N>::Elem lds[Ch<N>::SIZE];
  const int ffts = n_reqs * max_modes;
  int blk = blockIdx.x;
  if (blk < ffts) {
    const ReqDev& r = reqs.r[blk / max_modes];
    const int m = blk % max_modes;
    if (m >= r.M) return;
    const Fft2<N> fft(lds, tab);
    float2 v[Ch<N>::EL];
    fft.load_real(v, r.probe + (size_t)m * N * N);
    fft.forward(v);
    fft.store_spec(v, const_cast<float2*>(r.phat) + (size_t)m * N * N, 1.f / (float)N);
    return;
  }
  blk -= ffts;
  if (blk < item_blocks) {
    const int b = blk * (Ch<N>::T / 64) + (threadIdx.x >> 6);
    if (b < n_items) make_item(reqs, n_reqs, items, ramps, b, N, flags, threadIdx.x & 63, 64);
    return;
  }
  blk -= item_blocks;
  const ReqDev& r = reqs.r[blk / fill];
  if (!r.gpos_dense || r.accumulate) return;
  for (int e = (blk % fill) * Ch<N>::T + threadIdx.x; e < 2 * r.J; e += fill * Ch<N>::T) r.gpos_dense[e] = 0.f;
}

// The chains: one workgroup per (item, mode) tile. p.what selects, in this order:
//   kForward    shifted probe, every slice, far field; entry waves go to the
//               checkpoint slots (p.store);
//   kRecompute  instead: from the checkpoint of slice p.from, the entry waves
//               of slices p.from + 1 .. p.to go to the segment buffer;
//   kFar        (far_in_chain) noise model, intensities, and with kSeed the
//               detector gradient w Psi / N;
//   kAdjoint    g = gradient with respect to the exit wave, from slice p.hi (with
//               kFirst the last one, from the detector gradient) down to p.lo
//               (or 0): the entry wave psi_i is read from its checkpoint (or
//               segment) slot, conj(psi_i) g, the mode's contribution to the
//               object gradient, is stored in its place, and g <-
//               F^-1 conj(H) F conj(O) g. Slice 0 ends with h_hat = F(conj(O) g) / N
//               in the work tile and the sums of Im(conj(h_hat) phat R) u for the
//               position gradient. Between two segments g waits in the work
//               tile (real space).
// A far field or detector gradient that the next launch takes over waits in
// the work tile (transposed).
// With few tiles bound by too few waves to hide barriers and loads: 8 and 10 us a slice
// with 450 tiles of 64 x 64 (6 of 16 waves a CU, vector issue 0.5 of the time), 26 and 34
// us with 277 of 128 x 128 (6 waves, 0.36 and 0.30). With many, by vector issue and the
// checkpoints' traffic together: 128 x 128, 4 modes, 8 slices, 1024 positions forward
// 1.9 ms (14 waves, issue 0.73, 4.2 TB/s), adjoint 2.7 ms (0.55, 4.7 TB/s); the two passes
// took 2.6 and 3.7.
template <int N, int WHAT>
__global__ __launch_bounds__(Ch<N>::T, 4) void k_chain(
    const Item* __restrict__ items, const ReqTable reqs, float2* __restrict__ ws, float2* __restrict__ ck,
    const float2* __restrict__ ramps, const float2* __restrict__ tab, float* __restrict__ loss_part,
    float* __restrict__ pos_part, int* flags, int item_off, int n_items, int max_modes,
    ChainRun p) {
  using Elem = typename Ch<N>::Elem;
  constexpr int EL = Ch<N>::EL, T = Ch<N>::T, NBLK = N / 32;
  __shared__ Elem lds[Ch<N>::SIZE];
  __shared__ double red[2][Ch<N>::WAVES];
  int b, m;
  if (!chain_tile(n_items, max_modes, (WHAT & kAdjoint) != 0, b, m)) return;
  b += item_off;
  const Item it = items[b];
  const ReqDev& r = reqs.r[it.req];
  if (m >= r.M) return;
  const bool far = (WHAT & kFar) && far_in_chain<N>(r.M);
  if (!it.valid) {
    if (far) {
      if (r.I_out)
        for (int e = threadIdx.x; e < N * N; e += T) r.I_out[(size_t)(b - r.item0) * N * N + e] = 0.f;
      if (threadIdx.x < NBLK) loss_part[(size_t)b * NBLK + threadIdx.x] = 0.f;
    }
    return;
  }
  const Fft2<N> fft(lds, tab);
  const ChThread<N>& th = fft.th;
  const float inv = 1.f / (float)N;
  float2* tile = ws + (size_t)(it.tile0 + m) * N * N;
  float2 v[EL];

  if constexpr ((WHAT & (kForward | kRecompute)) != 0) {
    constexpr bool rec = (WHAT & kRecompute) != 0;
    int i = 0;
    if constexpr (!rec) {
      const float2* ph = r.phat + (size_t)m * N * N;
      const float2* ry = ramps + (size_t)b * 2 * N;
      const ConstTab rx = const_tab(ry + N);
#pragma unroll
      for (int kb = 0; kb < Ch<N>::KB; ++kb) {
        const float2 y = cscale(ry[th.ky(kb)], inv);
#pragma unroll
        for (int j2 = 0; j2 < 16; ++j2)
          v[16 * kb + j2] = xmul(xmul(ph[th.kx(j2) * N + th.ky(kb)], y), as_f2(rx[th.kx(j2)]));
      }
      fft.inverse(v);
    } else {
      i = p.from;
      fft.load_real(v, ck + ck_tile(it, r, m, i / r.ck_every) * N * N);
    }
    for (;; ++i) {
      if constexpr (rec) {
        if (i > p.from) fft.store_real(v, p.seg + ((size_t)(it.tile0 + m) * p.seg_len + (i - p.from - 1)) * N * N);
        if (i == p.to) return;
      } else if (p.store && i % r.ck_every == 0) {
        fft.store_real(v, ck + ck_tile(it, r, m, i / r.ck_every) * N * N);
      }
      fft.template times_real<false>(v, r.obj + ((size_t)i * r.H + it.ny) * r.W + it.nx, r.W);
      fft.forward(v);
      if (i == r.S - 1) break;
      propagate<N, false>(v, r, i, th);
      fft.inverse(v);
    }
  }

  if (far) {
    // the lanes hold the spectrum transposed: patterns and intensities, which
    // are row-major, go through LDS
    float* sh = reinterpret_cast<float*>(lds);
    static_assert(N * (N + 1) * 4 <= (int)sizeof(lds), "a pattern fits the space");
    const int t = threadIdx.x;
    auto at = [&](int e) { return th.ky(e >> 4) * (N + 1) + th.kx(e & 15); };
    float w[EL];
#pragma unroll
    for (int e = 0; e < EL; ++e) {
      v[e] = cscale(v[e], inv);
      w[e] = xabs2(v[e]);
    }
    if (r.I_out) {
      __syncthreads();
#pragma unroll
      for (int e = 0; e < EL; ++e) sh[at(e)] = w[e];
      __syncthreads();
      float* out = r.I_out + (size_t)(b - r.item0) * N * N;
#pragma unroll 4
      for (int e = t; e < N * N; e += T) out[e] = sh[(e / N) * (N + 1) + e % N];
    }
    float l = 0.f;
    if (r.patterns) {
      const float* pt = r.patterns + (size_t)it.j * N * N;
      __syncthreads();
#pragma unroll 4
      for (int e = t; e < N * N; e += T) sh[(e / N) * (N + 1) + e % N] = pt[e];
      __syncthreads();
      bool bad = false;
#pragma unroll
      for (int e = 0; e < EL; ++e) {
        float ell = 0.f, wt = 0.f;
        loss_weight(r.loss, w[e], sh[at(e)], r.eps, r.inv_sigma2, ell, wt);
        w[e] = wt;
        l += ell;
        bad |= !isfinite(ell) || !isfinite(wt);
      }
      if (bad) raise_flag(flags, kFlagNonFinite);
    }
    double lsum = (double)l;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) lsum += __shfl_xor(lsum, off);
    if (th.lane == 0) red[0][th.wave] = lsum;
    __syncthreads();
    if (t < NBLK) {
      double s = 0.0;
      if (t == 0)
        for (int q = 0; q < Ch<N>::WAVES; ++q) s += red[0][q];
      loss_part[(size_t)b * NBLK + t] = (float)s;   // (one sum for the item)
    }
    if (!(p.what & kSeed)) return;
#pragma unroll
    for (int e = 0; e < EL; ++e) {
      v[e] = cscale(v[e], w[e] * inv);
      // rounded here, as where the value is stored for a later launch (the
      // transform's first additions must not be fused with this product)
      asm volatile("" : "+v"(v[e].x), "+v"(v[e].y));
    }
    if constexpr (!(WHAT & kAdjoint)) fft.store_spec(v, tile, 1.f);
  } else if (WHAT & kForward) {
    fft.store_spec(v, tile, inv);
    return;
  }
  if constexpr (!(WHAT & kAdjoint)) return;

  if (!(p.what & kFirst)) {
    fft.load_real(v, tile);
  } else {
    if (!far) fft.load_spec(v, tile);
    fft.inverse(v);
  }
  for (int i = (p.what & kFirst) ? r.S - 1 : p.hi;; --i) {
    if (r.gobj)
      fft.contribute(v, p.seg && i % r.ck_every != 0
                            ? p.seg + ((size_t)(it.tile0 + m) * p.seg_len + (i - p.seg_base)) * N * N
                            : ck + ck_tile(it, r, m, i / r.ck_every) * N * N);
    fft.template times_real<true>(v, r.obj + ((size_t)i * r.H + it.ny) * r.W + it.nx, r.W);
    fft.forward(v);
    if (i == 0) break;
    propagate<N, true>(v, r, i - 1, th);
    fft.inverse(v);
    if (i == p.lo) {
      fft.store_real(v, tile);
      return;
    }
  }
  const float2* ph = r.phat + (size_t)m * N * N;
  const float2* ry = ramps + (size_t)b * 2 * N;
  const ConstTab rx = const_tab(ry + N);
  // the terms cancel to about a hundredth of their size: summed in double (in
  // float the sum's rounding would be the largest error of the result)
  double sy = 0.0, sx = 0.0;
#pragma unroll
  for (int kb = 0; kb < Ch<N>::KB; ++kb) {
    const int uy = th.ky(kb);
    const float2 ryk = ry[uy];
    const double fy = (double)(uy < N / 2 ? uy : uy - N) / (double)N;
#pragma unroll
    for (int j2 = 0; j2 < 16; ++j2) {
      const int ux = th.kx(j2);
      const double fx = (double)(ux < N / 2 ? ux : ux - N) / (double)N;
      float2& h = v[16 * kb + j2];
      h = cscale(h, inv);
      const float2 A = xmul(xmul(ph[ux * N + uy], ryk), as_f2(rx[ux]));
      const double z = (double)xjmul(h, A).y;   // Im(conj(h_hat) A)
      sy += fy * z;
      sx += fx * z;
    }
  }
  fft.store_spec(v, tile, 1.f);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    sy += __shfl_xor(sy, off);
    sx += __shfl_xor(sx, off);
  }
  __syncthreads();
  if (th.lane == 0) { red[0][th.wave] = sy; red[1][th.wave] = sx; }
  __syncthreads();
  if (threadIdx.x < 2) {
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < Ch<N>::WAVES; ++q) s += red[threadIdx.x][q];
    pos_part[(size_t)(it.tile0 + m) * NBLK * 2 + threadIdx.x] = (float)s;
  }
}

// Far field of the requests whose chains do not take it: mode sum, noise
// model and detector gradient of the Psi_m in the work tiles: I = sum_m |Psi_m|^2, loss partials per 32 columns, intensities
// if asked for and, with GRAD, tile_m = w Psi_m / N. Patterns and intensities
// are row-major; the tiles are transposed, so both go through LDS.
template <int N, bool GRAD>
__global__ __launch_bounds__(256) void k_chain_far(const Item* __restrict__ items, const ReqTable reqs,
                                                   float2* __restrict__ ws, float* __restrict__ loss_part, int* flags,
                                                   int item_off) {
  constexpr int PX = N * 32 / 256;
  __shared__ float pat[N * 33];
  __shared__ float red[4];
  const int b = item_off + gridDim.y - 1 - blockIdx.y;
  const Item it = items[b];
  const ReqDev& r = reqs.r[it.req];
  if (far_in_chain<N>(r.M)) return;
  const int t = threadIdx.x, x0 = blockIdx.x * 32;
  float* Io = r.I_out ? r.I_out + (size_t)(b - r.item0) * N * N : nullptr;
  if (!it.valid) {
    if (Io)
      for (int q = 0; q < PX; ++q) { const int e = t + 256 * q; Io[(e >> 5) * N + x0 + (e & 31)] = 0.f; }
    if (t == 0) loss_part[(size_t)b * (N / 32) + blockIdx.x] = 0.f;
    return;
  }
  float2* tile = ws + (size_t)it.tile0 * N * N + (size_t)x0 * N;
  const float* pt = r.patterns ? r.patterns + (size_t)it.j * N * N + x0 : nullptr;
  if (pt) {
#pragma unroll
    for (int q = 0; q < PX; ++q) { const int e = t + 256 * q; pat[(e >> 5) * 33 + (e & 31)] = pt[(e >> 5) * N + (e & 31)]; }
  }
  float I[PX];
#pragma unroll
  for (int q = 0; q < PX; ++q) I[q] = 0.f;
  for (int m = 0; m < r.M; ++m) {
    const float2* s = tile + (size_t)m * N * N;
#pragma unroll
    for (int q = 0; q < PX; ++q) I[q] += xabs2(s[t + 256 * q]);
  }
  __syncthreads();
  float w[PX];
  float lsum = 0.f;
  bool bad = false;
#pragma unroll
  for (int q = 0; q < PX; ++q) {
    const int e = t + 256 * q;
    float* c = pat + (e % N) * 33 + e / N;
    float ell = 0.f, wt = 0.f;
    if (pt) loss_weight(r.loss, I[q], *c, r.eps, r.inv_sigma2, ell, wt);
    w[q] = wt;
    lsum += ell;
    bad |= !isfinite(ell) || !isfinite(wt);
    if (Io) *c = I[q];
  }
  if (bad) raise_flag(flags, kFlagNonFinite);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) lsum += __shfl_xor(lsum, off);
  if ((t & 63) == 0) red[t >> 6] = lsum;
  __syncthreads();
  if (t == 0) loss_part[(size_t)b * (N / 32) + blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
  if (Io) {
#pragma unroll
    for (int q = 0; q < PX; ++q) { const int e = t + 256 * q; Io[(e >> 5) * N + x0 + (e & 31)] = pat[(e >> 5) * 33 + (e & 31)]; }
  }
  if constexpr (GRAD) {
    const float inv = 1.f / (float)N;
    for (int m = 0; m < r.M; ++m) {
      float2* s = tile + (size_t)m * N * N;
#pragma unroll
      for (int q = 0; q < PX; ++q) s[t + 256 * q] = cscale(s[t + 256 * q], w[q] * inv);
    }
  }
}

// dst = scale F^-1(src) of probe-sized tiles (src transposed), added to dst if
// accumulate; the probes of every request of a step in one launch.
template <int N>
__global__ __launch_bounds__(Ch<N>::T) void k_chain_plain(const PlainTable t, const float2* __restrict__ tab,
                                                          float scale, int accumulate) {
  __shared__ typename Ch<N>::Elem lds[Ch<N>::SIZE];
  int q = 0, tile = blockIdx.x;
  while (tile >= t.n[q]) tile -= t.n[q++];
  const Fft2<N> fft(lds, tab);
  float2 v[Ch<N>::EL];
  fft.load_spec(v, t.src[q] + (size_t)tile * N * N);
  fft.inverse(v);
  float2* out = t.dst[q] + (size_t)tile * N * N;
#pragma unroll
  for (int e = 0; e < Ch<N>::EL; ++e) v[e] = cscale(v[e], scale);
  if (accumulate) {
    float2 u[Ch<N>::EL];
    fft.load_real(u, out);
#pragma unroll
    for (int e = 0; e < Ch<N>::EL; ++e) v[e] = cadd(v[e], u[e]);
  }
  fft.store_real(v, out);
}

// ============================================================ launchers

namespace {

template <int N>
struct Chain {
  static const float2* tab(const LaunchCtx& L) { return L.tw + N; }
  static void begin(const LaunchCtx& L) {
    constexpr int W = Ch<N>::T / 64;
    const int item_blocks = (L.n_items + W - 1) / W;
    int J = 0;
    for (int q = 0; q < L.n_reqs; ++q)
      if (L.reqs.r[q].gpos_dense && !L.reqs.r[q].accumulate) J = std::max(J, L.reqs.r[q].J);
    const int fill = J ? std::min(64, (2 * J + Ch<N>::T - 1) / Ch<N>::T) : 0;
    hipLaunchKernelGGL((k_chain_begin<N>), dim3(L.n_reqs * L.max_modes + item_blocks + L.n_reqs * fill), dim3(Ch<N>::T),
                       0, L.stream, L.reqs, L.n_reqs, L.max_modes, L.n_items, item_blocks, fill, L.items, L.ramps,
                       tab(L), L.flags);
  }
  template <int WHAT>
  static void run_as(const LaunchCtx& L, const ChainRun& p) {
    const int most = chain_items(L.max_modes, Ch<N>::T);
    for (int at = 0; at < L.n_items; at += most) {
      const int n = std::min(L.n_items - at, most);
      hipLaunchKernelGGL((k_chain<N, WHAT>), dim3(8 * ((n + 7) / 8) * L.max_modes), dim3(Ch<N>::T), 0, L.stream,
                         L.items, L.reqs, L.ws, static_cast<float2*>(L.ck), L.ramps, tab(L), L.loss_part, L.pos_part,
                         L.flags, L.item_off + at, n, L.max_modes, p);
    }
  }
  static void run(const LaunchCtx& L, ChainRun p) {
    bool far = false;   // a far-field launch between the chains
    if (p.what & kFar)
      for (int q = 0; q < L.n_reqs; ++q) far |= !far_in_chain<N>(L.reqs.r[q].M);
    const int later = far ? p.what & (kAdjoint | kFirst) : 0;
    p.what &= ~later;
    if (p.what & kRecompute) run_as<kRecompute>(L, p);
    else if (!(p.what & kForward)) run_as<kAdjoint>(L, p);
    else if constexpr (far_in_chain_at(N)) {
      if (p.what & kAdjoint) run_as<kForward | kFar | kAdjoint>(L, p);
      else run_as<kForward | kFar>(L, p);
    } else {
      run_as<kForward>(L, p);
    }
    if (far) {
      const dim3 g(N / 32, L.n_items);
      if (p.what & kSeed)
        hipLaunchKernelGGL((k_chain_far<N, true>), g, dim3(256), 0, L.stream, L.items, L.reqs, L.ws, L.loss_part,
                           L.flags, L.item_off);
      else
        hipLaunchKernelGGL((k_chain_far<N, false>), g, dim3(256), 0, L.stream, L.items, L.reqs, L.ws, L.loss_part,
                           L.flags, L.item_off);
    }
    if (later) {
      p.what = later;
      run_as<kAdjoint>(L, p);
    }
  }
  static void plain_inv(hipStream_t s, const float2* tw, const PlainTable& t, float scale, bool acc) {
    int n = 0;
    for (int k = 0; k < t.count; ++k) n += t.n[k];
    if (n) hipLaunchKernelGGL((k_chain_plain<N>), dim3(n), dim3(Ch<N>::T), 0, s, t, tw + N, scale, acc ? 1 : 0);
  }
};

}  // namespace

bool chain_size(int N) { return N == 64 || N == 128; }

#define CHAIN_DISPATCH(N, CALL)          \
  switch (N) {                           \
    case 64: Chain<64>::CALL; break;     \
    default: Chain<128>::CALL; break;    \
  }

void launch_chain_begin(const LaunchCtx& L, int N) { CHAIN_DISPATCH(N, begin(L)); }
void launch_chain(const LaunchCtx& L, int N, const ChainRun& p) { CHAIN_DISPATCH(N, run(L, p)); }
void launch_chain_plain_inv(int N, hipStream_t s, const float2* tw, const PlainTable& t, float scale, bool acc) {
  CHAIN_DISPATCH(N, plain_inv(s, tw, t, scale, acc));
}

}  // namespace pty
