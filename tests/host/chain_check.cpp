// Host emulation of the register-held 2D transform of the chain kernels
// (pty_chain.hpp): every thread's registers and the exchange buffer of a
// workgroup, stage by stage. Checks that each exchange writes every element
// to an address of its own inside the buffer, reads only what was written,
// that 64 lanes of a wave spread over the LDS banks, and that forward and
// inverse transforms match a direct 2D DFT in double.
#include <array>
#include <cmath>
#include <complex>
#include <cstdio>
#include <random>
#include <set>
#include <vector>

#include "pty_chain.hpp"

using cd = std::complex<double>;

static int bad = 0;
static void need(bool ok, const char* what, int n) {
  if (!ok) { std::printf("N=%d: %s\n", n, what); ++bad; }
}

template <int N>
struct Tile {
  using C = pty::Ch<N>;
  std::vector<std::array<float2, C::EL>> reg{std::vector<std::array<float2, C::EL>>(C::T)};
  std::vector<float2> lds = std::vector<float2>(C::SIZE);

  // one exchange: thread t puts register e at wb(t) + wo(e) and takes it from rb(t) + ro(e)
  template <typename WB, typename WO, typename RB, typename RO>
  void exchange(WB wb, WO wo, RB rb, RO ro) {
    std::vector<char> used(C::SIZE, 0);
    for (int t = 0; t < C::T; ++t) {
      pty::ChThread<N> th(t & 63, t >> 6);
      for (int e = 0; e < C::EL; ++e) {
        const int a = wb(th) + wo(e);
        need(a >= 0 && a < C::SIZE, "write outside the buffer", N);
        need(!used[a], "two elements at one address", N);
        used[a] = 1;
        lds[a] = reg[t][e];
      }
    }
    for (int t = 0; t < C::T; ++t) {
      pty::ChThread<N> th(t & 63, t >> 6);
      for (int e = 0; e < C::EL; ++e) {
        const int a = rb(th) + ro(e);
        need(a >= 0 && a < C::SIZE && used[a], "read of an address nothing was written to", N);
        reg[t][e] = lds[a];
      }
    }
    // lanes of a wave: 64 four-byte elements over 64 banks, or 32 eight-byte ones at a time
    const int group = C::SPLIT ? 64 : 32;
    for (int t0 = 0; t0 < C::T; t0 += group) {
      std::set<int> w, r;
      for (int t = t0; t < t0 + group; ++t) {
        pty::ChThread<N> th(t & 63, t >> 6);
        w.insert((wb(th) + wo(0)) % group);
        r.insert((rb(th) + ro(0)) % group);
      }
      need((int)w.size() == group && (int)r.size() == group, "bank conflict", N);
    }
  }
  void ab() {
    exchange([](auto& h) { return h.a1(); }, [](int e) { return pty::off_a1<N>(e); }, [](auto& h) { return h.b1(); },
             [](int e) { return pty::off_b1<N>(e); });
  }
  void ba() {
    exchange([](auto& h) { return h.b1(); }, [](int e) { return pty::off_b1<N>(e); }, [](auto& h) { return h.a1(); },
             [](int e) { return pty::off_a1<N>(e); });
  }
  void bc() {
    exchange([](auto& h) { return h.b2(); }, [](int e) { return pty::off_b2<N>(e); }, [](auto& h) { return h.c2(); },
             [](int e) { return pty::off_c2<N>(e); });
  }
  void cb() {
    exchange([](auto& h) { return h.c2(); }, [](int e) { return pty::off_c2<N>(e); }, [](auto& h) { return h.b2(); },
             [](int e) { return pty::off_b2<N>(e); });
  }
};

template <int N>
double check(unsigned seed) {
  using C = pty::Ch<N>;
  std::mt19937 rng(seed);
  std::normal_distribution<float> nd;
  std::vector<float2> x((size_t)N * N), ta(N), tc(N);
  for (auto& z : x) z = make_float2(nd(rng), nd(rng));
  std::vector<float2> tab(C::TW);
  pty::chain_table(N, tab.data());
  for (int k = 0; k < N; ++k) {
    ta[k] = tab[k];
    tc[k] = tab[N + k];
  }
  auto each = [](Tile<N>& t, auto f) {
    for (int i = 0; i < C::T; ++i) {
      pty::ChThread<N> th(i & 63, i >> 6);
      f(th, *reinterpret_cast<float2(*)[C::EL]>(t.reg[i].data()));
    }
  };
  Tile<N> t;
  for (int i = 0; i < C::T; ++i) {
    pty::ChThread<N> th(i & 63, i >> 6);
    for (int r = 0; r < C::EL; ++r) t.reg[i][r] = x[(size_t)(th.yl + 4 * r) * N + th.x];
  }
  each(t, [&](auto& h, auto& v) { pty::ch_stage_a<N, false>(v, &ta[h.yl * C::EL]); });
  t.ab();
  each(t, [&](auto&, auto& v) { pty::ch_stage_b<N, false>(v); });
  t.bc();
  each(t, [&](auto& h, auto& v) { pty::ch_stage_c<N, false>(v, &tc[h.j1 * 16]); });
  // direct 2D DFT (separable, double)
  std::vector<cd> w(N), rows((size_t)N * N), ref((size_t)N * N);
  for (int k = 0; k < N; ++k) w[k] = std::polar(1.0, -2.0 * M_PI * k / N);
  for (int y = 0; y < N; ++y)
    for (int k = 0; k < N; ++k) {
      cd acc = 0;
      for (int n = 0; n < N; ++n) acc += cd(x[(size_t)y * N + n].x, x[(size_t)y * N + n].y) * w[(long)n * k % N];
      rows[(size_t)y * N + k] = acc;
    }
  double err = 0, mx = 0;
  for (int k = 0; k < N; ++k)
    for (int c = 0; c < N; ++c) {
      cd acc = 0;
      for (int n = 0; n < N; ++n) acc += rows[(size_t)n * N + c] * w[(long)n * k % N];
      ref[(size_t)k * N + c] = acc;
      mx = std::max(mx, std::abs(acc));
    }
  for (int i = 0; i < C::T; ++i) {
    pty::ChThread<N> th(i & 63, i >> 6);
    for (int e = 0; e < C::EL; ++e) {
      const float2 g = t.reg[i][e];
      err = std::max(err, std::abs(ref[(size_t)th.ky(e / 16) * N + th.kx(e % 16)] - cd(g.x, g.y)));
    }
  }
  std::printf("N%d forward %.3e\n", N, err / mx);
  double worst = err / mx;
  // and back: N^2 times the input
  each(t, [&](auto& h, auto& v) { pty::ch_stage_c<N, true>(v, &tc[h.j1 * 16]); });
  t.cb();
  each(t, [&](auto&, auto& v) { pty::ch_stage_b<N, true>(v); });
  t.ba();
  each(t, [&](auto& h, auto& v) { pty::ch_stage_a<N, true>(v, &ta[h.yl * C::EL]); });
  double e2 = 0;
  for (int i = 0; i < C::T; ++i) {
    pty::ChThread<N> th(i & 63, i >> 6);
    for (int r = 0; r < C::EL; ++r) {
      const float2 g = t.reg[i][r], z = x[(size_t)(th.yl + 4 * r) * N + th.x];
      e2 = std::max(e2, std::hypot(g.x / ((double)N * N) - z.x, g.y / ((double)N * N) - z.y));
    }
  }
  std::printf("N%d round trip %.3e\n", N, e2);
  return std::max(worst, e2 / 4);   // inputs reach about 4
}

int main() {
  double worst = std::max(check<64>(1), check<128>(2));
  return worst < 1e-5 && bad == 0 ? 0 : 1;
}
