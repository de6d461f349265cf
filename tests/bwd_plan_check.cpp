// Host check of the dK/dV division (bwd_plan.h): random masks and head counts,
// every plan walked as the kernels walk it.  Prints one line per shape named on
// the command line (tokens per trajectory, trajectories, Hq, Hkv, D: shares,
// partial tiles of the shares and of the items).
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "bwd_plan.h"

namespace mv {
void set_error(const std::string&) {}
}  // namespace mv
using namespace mv;

#define CHECK(c)                                              \
  do {                                                        \
    if (!(c)) {                                               \
      std::printf("line %d: %s\n", __LINE__, #c);             \
      std::exit(1);                                           \
    }                                                         \
  } while (0)

// The steps of every worker's runs (bwd_dkdv_kernel), then the partial tiles
// that the blocks of every first cut sum (bwd_reduce_kernel).
static void walk(const mv_view_mask& m, const SharePlan& p, int G, int Hkv) {
  const int NT = p.n_kt * Hkv;
  auto steps_of = [&](int tile) {
    return (m.bwd_cum[tile % p.n_kt + 1] - m.bwd_cum[tile % p.n_kt]) * G;
  };
  std::vector<std::vector<int>> parts(NT);
  std::vector<int> done(NT, 0);
  int next = 0;
  for (int w = 0; w < p.n; ++w) {
    int tile = p.tile(w), st0 = p.st[w], part = p.part(w);
    const int tile1 = p.tile(w + 1), st1 = p.st[w + 1];
    CHECK(part == next);
    CHECK(tile < tile1 || st0 < st1);
    while (tile < tile1 || (tile == tile1 && st0 < st1)) {
      CHECK(tile < NT && done[tile] == st0);
      const int steps = steps_of(tile), n = (tile < tile1 ? steps : st1) - st0;
      CHECK(n > 0 && st0 + n <= steps);
      done[tile] += n;
      if (n != steps) parts[tile].push_back(part++);
      ++tile;
      st0 = 0;
    }
    next = part;
  }
  CHECK(next == p.part(p.n) && p.tile(p.n) == NT && p.st[p.n] == 0);
  for (int t = 0; t < NT; ++t) CHECK(done[t] == steps_of(t));
  std::vector<char> summed(NT, 0);
  for (int w = 1; w < p.n; ++w) {
    if (p.st[w] == 0) continue;
    const int tile = p.tile(w);
    if (p.tile(w - 1) == tile && p.st[w - 1] > 0) continue;
    int n = 2;
    for (; p.tile(w + n - 1) == tile; ++n) CHECK(w + n - 1 < p.n);
    CHECK(!summed[tile]++ && int(parts[tile].size()) == n);
    for (int i = 0; i < n; ++i) CHECK(parts[tile][i] == p.part(w) - 1 + i);
  }
  for (int t = 0; t < NT; ++t) CHECK(summed[t] == !parts[t].empty());
}

int main(int argc, char** argv) {
  std::mt19937 rng(1);
  const int hkvs[] = {1, 2, 4, 8, 12}, groups[] = {1, 2, 3, 4, 7, 8};
  const size_t scratch = MV_ATTN_BWD_NOALLOC_SCRATCH_BYTES;
  int shares = 0, items = 0, capped = 0;
  for (int it = 0; it < 600; ++it) {
    const int nt = 1 + rng() % 6;
    std::vector<mv_trajectory> tr;
    std::vector<std::vector<mv_edit>> ed(nt);
    std::vector<std::vector<mv_span>> sp(nt);
    int T = 0;
    for (int t = 0; t < nt; ++t) {
      const int len = 1 + rng() % (it % 3 == 0 ? 300 : 9000), b = T;
      T += len;
      sp[t].reserve(8);
      for (int j = b, lo = b, e = int(rng() % 6); e > 0; --e) {
        j += 1 + rng() % (len / 4 + 1);
        if (j >= T) break;
        mv_edit x{};
        x.junction = j;
        if (j - lo > 2) {   // evict a run of [lo, j)
          const int s = lo + rng() % (j - lo - 1), f = s + 1 + rng() % (j - s - 1);
          sp[t].push_back({s, f});
          x.n_evict = 1;
          x.evict = &sp[t].back();
          lo = f;
        }
        ed[t].push_back(x);
      }
      tr.push_back({b, T, int32_t(ed[t].size()), ed[t].data()});
    }
    mv_view_mask* m = nullptr;
    CHECK(mv_build_view_mask(tr.data(), nt, T, &m) == MV_OK);
    for (int q = 0; q < 4; ++q) {
      const int Hkv = hkvs[rng() % 5], G = groups[rng() % 6], D = rng() % 2 ? 64 : 128;
      const size_t items_ws = bwd_ws_bytes(*m, Hkv * G, D, size_t(m->n_slots) * Hkv);
      const BwdPlan p = bwd_plan(*m, Hkv * G, Hkv, D);
      CHECK(p.ws_bytes >= items_ws && (p.ws_bytes <= scratch || items_ws > scratch ||
                                       p.share.n == 0));
      if (p.share.n == 0) {
        CHECK(p.ws_bytes == items_ws);
        ++items;
      } else {
        CHECK(p.share.n > 1 && p.share.n <= kNumCu && p.share.part(p.share.n) < 2 * kNumCu);
        CHECK(p.ws_bytes >= bwd_ws_bytes(*m, Hkv * G, D, p.share.part(p.share.n)));
        capped += p.share.n < kNumCu * 7 / 8;
        walk(*m, p.share, G, Hkv);
        ++shares;
      }
      // any number of workers, whether the rule takes it or not
      if (int64_t(m->stats.bwd_items) * Hkv <= kShareMaxGroups)
        walk(*m, share_plan(*m, G, Hkv, 1 + int(rng() % kNumCu)), G, Hkv);
    }
    mv_view_mask_free(m);
  }
  CHECK(shares > 100 && items > 100 && capped > 10);
  for (int i = 1; i + 4 < argc; i += 5) {
    const int L = std::atoi(argv[i]), n = std::atoi(argv[i + 1]), Hq = std::atoi(argv[i + 2]),
              Hkv = std::atoi(argv[i + 3]), D = std::atoi(argv[i + 4]);
    std::vector<mv_trajectory> tr;
    for (int t = 0; t < n; ++t) tr.push_back({t * L, (t + 1) * L, 0, nullptr});
    mv_view_mask* m = nullptr;
    CHECK(mv_build_view_mask(tr.data(), n, n * L, &m) == MV_OK);
    const BwdPlan p = bwd_plan(*m, Hq, Hkv, D);
    std::printf("%d %d %d\n", p.share.n, p.share.n ? p.share.part(p.share.n) : 0,
                m->n_slots * Hkv);
    mv_view_mask_free(m);
  }
  return 0;
}
