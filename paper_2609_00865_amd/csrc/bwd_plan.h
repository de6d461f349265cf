// How the attention backward's dK/dV pass is divided among the CUs: the mask's
// work items, or equal shares, one per CU.  Host code; the kernels read the
// SharePlan.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

#include "mv_internal.h"

#if defined(__HIPCC__)
#define MV_PLAN_HD __host__ __device__
#else
#define MV_PLAN_HD
#endif

namespace mv {

// The dK/dV pass cut into n equal shares: worker w takes the steps from cut w
// to cut w + 1 of all steps laid end to end (KV head, key tile, query head,
// query block).  Cut w: step st[w] of tile tile(w) = hk * n_kt + kt, with
// st < the tile's steps (the last cut: tile n_kt * Hkv, step 0); cuts are
// strictly increasing.  A run that is part of a tile goes to an fp32 partial
// tile; these are numbered in the order of the steps, worker w's from part(w)
// on, so that the partial tiles of one key tile follow one another.
struct SharePlan {
  int n, n_kt;
  uint32_t cut[kNumCu + 1];   // tile | partial tiles of the workers before << 16
  int st[kNumCu + 1];
  MV_PLAN_HD int tile(int w) const { return int(cut[w] & 0xffffu); }
  MV_PLAN_HD int part(int w) const { return int(cut[w] >> 16); }
};

// Shares are considered only while the work items (times KV heads) are at most
// kShareMaxGroups: shares lose the items' grouping by XCD (the L2 hit rate
// falls from 46% to 15%), which costs more than any balance beyond (whole
// layer at 3992 items 7453 -> 7296 us, at 6048 items 11778 -> 11888 us).
constexpr int kShareMaxGroups = 4096;
constexpr int kShareMinSteps = 4;
// With no more items than CUs the longest item bounds the pass; shares then
// have to be this many steps shorter (the reduce launch and a run's start and
// end take 8 steps' time: on 512 tokens, one head of 64, items of 8 steps and
// 19 us became shares of 4 steps with 17 + 6 us, and stay items).
constexpr int kShareExtra = 8;
// Costs in eighths of a fully visible step (2.1 - 2.5 us at head size 128); a
// step that applies the mask costs 0.3 us more, and a run 10 us (its K and V,
// the first blocks' latency, its stores).
constexpr int64_t kStepCost = 8, kMaskCost = 1, kRunCost = 32;

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// D [Hq, T] | LSE * log2 e [Hq, T] | fp32 partial tiles [n_partials, 2, 128, D]
inline size_t bwd_ws_bytes(const mv_view_mask& m, int Hq, int D, size_t n_partials) {
  return 2 * align256(size_t(Hq) * m.T * sizeof(float)) +
         align256(n_partials * 2 * kBwdTileK * D * sizeof(float)) + 256;
}

// Cost of the key tiles before kt of one KV head, each in one run.
inline int64_t tiles_cost(const mv_view_mask& m, int G, int kt) {
  return m.bwd_cost[kt] * G + kRunCost * kt;
}

inline SharePlan share_plan(const mv_view_mask& m, int G, int Hkv, int workers) {
  SharePlan p;
  p.n_kt = m.n_kt128;
  auto cost = [&](int kt) { return tiles_cost(m, G, kt); };
  const int64_t per_kv = cost(p.n_kt);
  int n = 0, kt = 0, hk = 0, last = 0;
  p.cut[0] = p.st[0] = 0;
  for (int w = 1; w < workers; ++w) {
    const int64_t pos = int64_t(w) * per_kv * Hkv / workers;
    for (; (hk + 1) * per_kv <= pos; ++hk) kt = 0;
    const int64_t r = pos - hk * per_kv;
    while (cost(kt + 1) <= r) ++kt;
    const int64_t steps = int64_t(m.bwd_cum[kt + 1] - m.bwd_cum[kt]) * G;
    int tile = hk * p.n_kt + kt;
    int st = int(((r - cost(kt)) * steps * 2 / (cost(kt + 1) - cost(kt)) + 1) / 2);   // nearest
    if (st == steps) {
      ++tile;
      st = 0;
    }
    // a cut that falls on the one before it, or on the end, is dropped
    if (tile == p.n_kt * Hkv || (tile == last && st == p.st[n])) continue;
    ++n;
    p.cut[n] = last = tile;
    p.st[n] = st;
  }
  p.n = n + 1;
  p.cut[p.n] = p.n_kt * Hkv;
  p.st[p.n] = 0;
  uint32_t parts = 0;
  for (int w = 0; w <= p.n; ++w) {
    const uint32_t tile = p.cut[w];
    p.cut[w] |= parts << 16;
    if (w == p.n) break;
    // a worker that stays inside one tile has one run of it; any other has
    // the end of a tile if it starts inside, and the start of one if the next
    // worker does
    parts += p.cut[w + 1] == tile ? 1 : (p.st[w] > 0) + (p.st[w + 1] > 0);
  }
  return p;
}

struct BwdPlan {
  SharePlan share;   // n = 0: the mask's work items, one workgroup each
  size_t ws_bytes;   // of the backward's workspace
};

// Equal shares while the work items are few (kShareMaxGroups): few items of
// uneven length leave CUs idle.  dK/dV at 8192 tokens, 16 / 4 heads (388
// items): 441 -> 335 us; 9500-token stream, 28 / 4 heads: 1121 -> 1018 us;
// 16384 tokens, 28 / 4 heads (1208): whole layer 4820 -> 4446 us.
inline BwdPlan bwd_plan(const mv_view_mask& m, int Hq, int Hkv, int D) {
  const int G = Hq / Hkv;
  const size_t items_ws = bwd_ws_bytes(m, Hq, D, size_t(m.n_slots) * Hkv);
  BwdPlan p;
  p.share.n = 0;
  p.ws_bytes = items_ws;
  const int64_t groups = int64_t(m.stats.bwd_items) * Hkv;
  if (groups > kShareMaxGroups) return p;
  const int64_t steps = int64_t(m.bwd_cum.back()) * Hq;
  int n = int(std::min<int64_t>(kNumCu, (steps + kShareMinSteps - 1) / kShareMinSteps));
  // The allocation-free form takes the same calls, with the same bits, either
  // way: where the items' partial tiles fit its static scratch, as many shares
  // as do too (a cut less takes away at most two partial tiles).
  const size_t limit = MV_ATTN_BWD_NOALLOC_SCRATCH_BYTES;
  SharePlan s;
  size_t ws;
  for (;;) {
    if (n < 2) return p;
    s = share_plan(m, G, Hkv, n);
    ws = bwd_ws_bytes(m, Hq, D, s.part(s.n));
    if (ws <= limit || items_ws > limit) break;
    n -= std::max(1, int((ws - limit) / (size_t(4) * kBwdTileK * D * sizeof(float))));
  }
  if (s.n < 2) return p;
  if (n * 8 < std::min<int64_t>(kNumCu, groups) * 7) return p;
  if (groups <= kNumCu && steps / n + kShareExtra > int64_t(m.bwd_max_blocks) * G) return p;
  p.share = s;
  p.ws_bytes = std::max(items_ws, ws);
  return p;
}

}  // namespace mv
