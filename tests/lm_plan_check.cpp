// Host check of the LM head's workspace sizes (lm_plan.h): the partials of the
// dH product that a call of n tokens takes fit what is reserved for it, and the
// reserved bytes never shrink with n.
#include <cstdio>

#include "lm_plan.h"

using namespace mv;

int main() {
  const int shapes[][2] = {{1024, 32000}, {2048, 50257}, {3584, 152064}, {4096, 128256},
                           {896, 151936}, {64, 1000},    {8192, 128256}, {320, 4133}};
  for (const auto& hv : shapes) {
    const int H = hv[0], V = hv[1];
    size_t before = 0;
    for (int n = 1; n <= 40000; n += n < 6000 ? 1 : 41) {
      const int s = dh_splits(n, H, V);
      const size_t room = g_and_part_bytes(n, H, V);
      const size_t part = s > 1 ? lm_align256(size_t(s) * n * H * 4) : 0;
      if (g_bytes(n, V) + part > room || room < before) {
        std::printf("n %d H %d V %d: splits %d, G %zu, partials %zu, room %zu, before %zu\n", n, H,
                    V, s, g_bytes(n, V), part, room, before);
        return 1;
      }
      before = room;
    }
  }
  return 0;
}
