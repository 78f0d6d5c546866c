// pty_chain.hpp -- 2D transform of an N x N tile held in the registers of one
// workgroup (N = 64, 128), the building block of the chain kernels. (At N = 192
// the same tile, 768 threads and 157 KB of LDS, one workgroup per CU, measured
// slower than the two passes: 15.1 -> 17.9 ms at 6 modes, 20 slices, 256
// positions.)
//
// A workgroup of 4 N threads holds the tile as EL = N / 4 complex values per
// thread and goes through three layouts; indices: y = yl + 4 r, x = xl + 16 xh,
// k_y = k1 + EL k2, k_x = j1 + XH j2, XH = N / 16:
//   A (real space)   thread (yl, x), register r            -- x runs over the lanes, yl is wave-uniform
//   B (in between)   thread (k1, xl), registers (yl | k2, xh | j1)
//   C (spectrum)     thread (j1, k2, k1 mod 16), registers (k1 / 16, xl | j2)  -- j1 is wave-uniform
// Forward: EL-point DFT over r and twiddle w_N^{yl k1} in A; 4-point DFT over
// yl and XH-point DFT over xh in B; twiddle w_N^{xl j1} and 16-point DFT over xl
// in C. The inverse runs the same steps backwards with conjugated roots. Both
// twiddles have a wave-uniform factor and a register index, so they are scalar
// operands read from a table laid out per wave; the only traffic between
// threads is one exchange through LDS between A and B and one between B and C.
//
// Exchange addresses (in units of the exchanged element): A<->B element
// (k1, yl, x) at P1 k1 + N yl + x; B<->C element (j1, k1, k2, xl) at
// JS (j1 + XH (k1 / 16)) + XLS xl + 16 k2 + k1 mod 16. The pads P1 = 4 N + 16
// and XLS let the 64 lanes of a wave hit distinct banks on both sides. For
// N = 64 a whole complex value is exchanged at once (34 KB a tile); for N = 128
// the real parts go first, then the imaginary ones, through half the space
// (68 KB), which leaves room for two tiles per CU.
// Transforms are unnormalised.
#pragma once

#include <cmath>

#include "pty_fft.hpp"

namespace pty {

template <int N>
struct Ch {
  static_assert(N == 64 || N == 128, "register tiles exist for these sizes");
  static constexpr int EL = N / 4, T = 4 * N, XH = N / 16, KB = N / 64, WAVES = T / 64;
  static constexpr bool SPLIT = N > 64;
  static constexpr int P1 = 4 * N + 16;
  static constexpr int XLS = SPLIT ? 68 : 66;
  static constexpr int JS = 16 * XLS;
  static constexpr int SIZE1 = P1 * (EL - 1) + 4 * N, SIZE2 = JS * XH * KB;
  static constexpr int SIZE = SIZE1 > SIZE2 ? SIZE1 : SIZE2;
  using Elem = typename std::conditional<SPLIT, float, float2>::type;
  static constexpr int TW = 2 * N;   // chain_table
};

// exp(-2 pi i k / n) as the pair of floats near it whose modulus is closest to
// one, a direction error weighted with 0.1: the chain applies a table root and
// later its conjugate to the same value, so the direction mostly cancels and
// the modulus counts twice. At most 3 spacings from the nearest floats.
inline float2 near_root(long k, long n) {
  const CosSin e = unit_root(k, n);
  const double c = e.c, s = -e.s;
  const float c0 = (float)c, s0 = (float)s;
  if (c0 == 0.f || s0 == 0.f) return make_float2(c0, s0);
  const float uc = std::nextafter(std::fabs(c0), 2.f) - std::fabs(c0), us = std::nextafter(std::fabs(s0), 2.f) - std::fabs(s0);
  float2 best = make_float2(c0, s0);
  double least = 1.0;
  for (int i = -3; i <= 3; ++i)
    for (int j = -3; j <= 3; ++j) {
      const float a = c0 + (float)i * uc, b = s0 + (float)j * us;
      const double da = (double)a - c, db = (double)b - s, r = c * da + s * db, t = c * db - s * da;
      const double q = r * r + 0.1 * t * t;
      if (q < least) { least = q; best = make_float2(a, b); }
    }
  return best;
}
// Both twiddle tables, Ch<N>::TW roots: [4][N / 4] w_N^{yl k1}, [N / 16][16] w_N^{j1 xl}.
inline void chain_table(int N, float2* t) {
  for (int k = 0; k < N; ++k) {
    t[k] = near_root((long)(k / (N / 4)) * (k % (N / 4)), N);
    t[N + k] = near_root((long)(k / 16) * (k % 16), N);
  }
}

// Indices of one thread in the three layouts (wave: threadIdx.x / 64, uniform).
template <int N>
struct ChThread {
  int lane, wave;
  int x, yl;        // A
  int xl, k1;       // B
  int k1a, k2, j1;  // C
  __host__ __device__ __forceinline__ ChThread(int lane_, int wave_) : lane(lane_), wave(wave_) {
    yl = wave / (N / 64);
    x = (wave % (N / 64)) * 64 + lane;
    xl = lane & 15;
    k1 = wave * 4 + (lane >> 4);
    k1a = lane & 15;
    k2 = lane >> 4;
    j1 = wave;
  }
  __host__ __device__ __forceinline__ int a1() const { return N * yl + x; }
  __host__ __device__ __forceinline__ int b1() const { return Ch<N>::P1 * k1 + xl; }
  __host__ __device__ __forceinline__ int b2() const {
    return (k1 & 15) + Ch<N>::XLS * xl + Ch<N>::JS * Ch<N>::XH * (k1 >> 4);
  }
  __host__ __device__ __forceinline__ int c2() const { return lane + Ch<N>::JS * j1; }
  // spectrum position of register (kb, j2)
  __host__ __device__ __forceinline__ int ky(int kb) const { return k1a + 16 * kb + Ch<N>::EL * k2; }
  __host__ __device__ __forceinline__ int kx(int j2) const { return j1 + Ch<N>::XH * j2; }
};

// Offsets of register e from the thread's base in each layout's exchange.
template <int N> __host__ __device__ __forceinline__ constexpr int off_a1(int e) { return Ch<N>::P1 * e; }
template <int N> __host__ __device__ __forceinline__ constexpr int off_b1(int e) {   // e = yl XH + xh
  return N * (e / Ch<N>::XH) + 16 * (e % Ch<N>::XH);
}
template <int N> __host__ __device__ __forceinline__ constexpr int off_b2(int e) {   // e = k2 XH + j1
  return 16 * (e / Ch<N>::XH) + Ch<N>::JS * (e % Ch<N>::XH);
}
template <int N> __host__ __device__ __forceinline__ constexpr int off_c2(int e) {   // e = 16 kb + xl
  return Ch<N>::JS * Ch<N>::XH * (e / 16) + Ch<N>::XLS * (e % 16);
}

// ---- register stages

// A: EL-point DFT over r and the twiddle (tw: the wave's EL roots)
template <int N, bool INV>
__host__ __device__ __forceinline__ void ch_stage_a(float2 (&v)[Ch<N>::EL], const float2* tw) {
  constexpr int EL = Ch<N>::EL;
  if (INV) {
#pragma unroll
    for (int k = 1; k < EL; ++k) v[k] = xjmul(tw[k], v[k]);
    Dft<EL, true, true>::run(v);
  } else {
    Dft<EL, false, true>::run(v);
#pragma unroll
    for (int k = 1; k < EL; ++k) v[k] = xmul(v[k], tw[k]);
  }
}

// B: 4-point DFTs over yl and XH-point DFTs over xh
template <int N, bool INV>
__host__ __device__ __forceinline__ void ch_stage_b(float2 (&v)[Ch<N>::EL]) {
  constexpr int XH = Ch<N>::XH;
  auto over_y = [&]() {
#pragma unroll
    for (int h = 0; h < XH; ++h) {
      float2 t[4] = {v[h], v[XH + h], v[2 * XH + h], v[3 * XH + h]};
      Dft<4, INV>::run(t);
      v[h] = t[0]; v[XH + h] = t[1]; v[2 * XH + h] = t[2]; v[3 * XH + h] = t[3];
    }
  };
  auto over_x = [&]() {
#pragma unroll
    for (int k = 0; k < 4; ++k) Dft<XH, INV, true>::run(&v[k * XH]);
  };
  if (INV) { over_x(); over_y(); }
  else { over_y(); over_x(); }
}

// C: twiddle (tw: the wave's 16 roots) and 16-point DFTs over xl
template <int N, bool INV>
__host__ __device__ __forceinline__ void ch_stage_c(float2 (&v)[Ch<N>::EL], const float2* tw) {
#pragma unroll
  for (int kb = 0; kb < Ch<N>::KB; ++kb) {
    if (kb > 0) sched_fence();
    if (INV) {
      Dft<16, true, true>::run(&v[16 * kb]);
#pragma unroll
      for (int k = 1; k < 16; ++k) v[16 * kb + k] = xjmul(tw[k], v[16 * kb + k]);
    } else {
#pragma unroll
      for (int k = 1; k < 16; ++k) v[16 * kb + k] = xmul(v[16 * kb + k], tw[k]);
      Dft<16, false, true>::run(&v[16 * kb]);
    }
  }
}

}  // namespace pty
