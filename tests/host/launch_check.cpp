// Workgroups of the launches whose grids grow with the requests of a group
// (finish_layout, chain_items), taken through every workgroup on the host: each
// request gets those of its own sizes, every launch stays under the threads a
// grid dimension takes, and together they cover the work once.
#include <cstdio>
#include <vector>

#include "pty_internal.h"

using namespace pty;

static int bad = 0;
static void need(bool ok, const char* what) {
  if (!ok) { std::printf("%s\n", what); ++bad; }
}

static ReqDev request(int M, int S, int H, int W, int n_items) {
  static float2 some;
  static double loss;
  ReqDev r{};
  r.M = M;
  r.S = S;
  r.H = H;
  r.W = W;
  r.n_items = n_items;
  r.gobj = r.gphat = &some;
  r.loss_out = &loss;
  return r;
}

// Walks the launches; returns how many there were.
static int walk(const std::vector<ReqDev>& rs, int N, int lo, int slices, bool rest, unsigned long long want) {
  ReqTable t{};
  int n_items = 0;
  for (size_t q = 0; q < rs.size(); ++q) {
    t.r[q] = rs[q];
    t.r[q].item0 = n_items;
    n_items += rs[q].n_items;
  }
  FinishRun p{};
  p.lo = lo;
  p.slices = slices;
  const unsigned blocks = finish_layout(p, t, (int)rs.size(), n_items, N, true, rest);
  need(blocks == want, "workgroups of the request sizes");
  int launches = 0;
  unsigned next = 0;
  std::vector<unsigned> tiles(rs.size()), others(rs.size());
  for (p.first = 0; p.first < blocks; p.first += kFinishBlocks, ++launches) {
    const unsigned n = blocks - p.first < kFinishBlocks ? blocks - p.first : kFinishBlocks;
    need((unsigned long long)n * 512 < (1ull << 32), "threads of a launch");
    for (unsigned g = p.first; g < p.first + n; ++g) {
      const FinishWork w = finish_work(p, g);
      const int q = w.req;
      if (q < 0 || q > (int)rs.size()) { need(false, "a workgroup of no request"); return launches; }
      need(g == next++, "workgroups in turn");
      if (q == (int)rs.size()) {
        need(rest && !w.tile && (int)w.index * 512 < n_items, "positions");
        continue;
      }
      const FinishParts f = finish_parts(p, t.r[q], q, N);
      if (w.index >= (w.tile ? f.gather : f.probe + f.loss)) { need(false, "past the request's work"); return launches; }
      (w.tile ? tiles : others)[q] += 1;
    }
  }
  for (size_t q = 0; q < rs.size(); ++q) {
    const FinishParts f = finish_parts(p, t.r[q], (int)q, N);
    need(tiles[q] == f.gather && others[q] == f.probe + f.loss, "all of a request's work");
  }
  need(next == blocks, "the last workgroup");
  return launches;
}

int main() {
  auto tiles = [](unsigned long long S, unsigned long long H, unsigned long long W) { return S * ((H + 3) / 4) * ((W + 63) / 64); };
  // sixteen requests, one with a large object: by the largest of each size they
  // would need 16 * 30 * 529 * 34 = 8633280 workgroups for the object alone
  std::vector<ReqDev> group{request(1, 30, 2116, 2116, 9)};
  unsigned long long small = 0, modes = 1;
  for (int q = 1; q < 16; ++q) {
    group.push_back(request(q % 3 + 1, 1 + q % 2, 64 + q, 70, 4 + q));
    small += tiles(1 + q % 2, 64 + q, 70);
    modes += q % 3 + 1;
  }
  need(sum_in_strips(64, 9, 1, 2116, 2116, 30), "few windows on a large object");
  // (its sum is taken in strips; 31 modes of 64 x 64 pixels, at most 19 items: 512 pixels a workgroup)
  need(walk(group, 64, 0, 30, true, small + 8 * modes + 16 + 1) == 1, "one launch for the group");
  need(walk(group, 64, 0, 30, false, small) == 1, "the objects alone");
  // the same object under many windows, and 3 x 10^9 values
  group[0].n_items = 20000;
  need(walk(group, 64, 0, 30, true, tiles(30, 2116, 2116) + small + 128 * modes + 16 + (20000 + 15 * 12 + 511) / 512) == 1,
       "one launch for the group");
  need(walk({request(5, 3, 32000, 32000, 65535)}, 256, 0, 3, true, tiles(3, 32000, 32000) + 5 * 128 + 1 + 128) == 2,
       "two launches");
  // the line between 32 and 512 probe pixels
  need(!finish_wide(32767, 1) && finish_wide(32768, 8) && !finish_wide(32768, 9) && finish_wide(262144, 65535), "probe pixels");
  // the line between tiles and strips: enough strips; contributions over a value
  const int H = 3000 * 16, values = H * 64;
  need(!sum_in_strips(64, 8, 1, H - 16, 64, 1) && sum_in_strips(64, 8, 1, H, 64, 1), "3000 strips");
  need(sum_in_strips(64, values / 4096 * 4, 1, H, 64, 1) && !sum_in_strips(64, values / 4096 * 5, 1, H, 64, 1) &&
           !sum_in_strips(64, values / 4096, 5, H, 64, 1),
       "3000 / 700 contributions over a value");
  need(sum_in_strips(256, 65535, 1, 17000, 17000, 2) && !sum_in_strips(256, 65535, 1, 16000, 16000, 2), "sixteen");
  // a segment of slices, past the end of a shallower request; nothing to sum
  need(walk({request(2, 7, 200, 300, 5)}, 128, 6, 3, false, tiles(1, 200, 300)) == 1, "the last segment");
  need(walk({request(2, 7, 200, 300, 5)}, 128, 0, 0, true, 2 * 32 + 1 + 1) == 1, "no object gradient");
  ReqDev no = request(1, 3, 100, 100, 600);
  no.gobj = no.gphat = nullptr;
  no.loss_out = nullptr;
  need(walk({no}, 64, 0, 3, true, 2) == 1, "positions alone");
  for (int T : {256, 512})
    for (int M : {1, 3, 8, 127, 128, 300, 65535}) {
      const int n = chain_items(M, T);
      need(n >= 8 && n % 8 == 0 && (unsigned long long)n * M * T < (1ull << 32), "threads of a chain launch");
      need(n > kMaxItems || (unsigned long long)(n + 8) * M * T >= (1ull << 32), "no more chain launches than needed");
    }
  if (!bad) std::printf("ok\n");
  return bad ? 1 : 0;
}
