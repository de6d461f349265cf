// How the attention backward's dK/dV pass is divided among the CUs: the mask's
// work items, or equal shares, one per CU.  Host code; the kernels read the
// SharePlan.
#pragma once

#include <algorithm>
#include <array>
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
// Costs in eighths of a fully visible step (2.1 - 2.5 us at head size 128); a
// step that applies the mask costs 0.3 us more, a run 10 us (its K and V, the
// first blocks' latency, its stores), a work item that leaves a partial tile
// as much again, and a reduce pass of P partial tiles 16 + P / 10.
constexpr int64_t kStepCost = 8, kMaskCost = 1, kRunCost = 32, kPartCost = 32;
inline double reduce_cost(int64_t parts) { return parts > 0 ? 16 + parts * 0.1 : 0.0; }

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

// Cost of the longest share.
inline double share_time(const mv_view_mask& m, const SharePlan& p, int G) {
  const double per_kv = double(tiles_cost(m, G, p.n_kt));
  double most = 0, from = 0;
  for (int w = 1, hk = 0; w <= p.n; ++w) {
    // cost of the steps before cut w and of the runs they make
    while (p.tile(w) >= (hk + 1) * p.n_kt) ++hk;
    const int kt = p.tile(w) - hk * p.n_kt;
    double to = hk * per_kv + double(tiles_cost(m, G, kt));
    if (p.st[w] > 0)
      to += kRunCost + double((m.bwd_cost[kt + 1] - m.bwd_cost[kt]) * p.st[w]) /
                           (m.bwd_cum[kt + 1] - m.bwd_cum[kt]);
    most = std::max(most, to - from + (p.st[w - 1] > 0 ? kRunCost : 0));
    from = to;
  }
  return most;
}

// Cost of the pass as work items: the dispatcher deals items to the XCDs
// round-robin and each XCD gives the next to its first free CU.  Of the XCD
// with the most work.
inline double items_time(const mv_view_mask& m, int G, int Hkv) {
  const int n = int(m.bwd_item_cost.size());
  auto cost = [&](int w) {
    return int64_t(m.bwd_item_cost[w]) * G + kRunCost + (m.bwd_items[4 * w + 3] < 0 ? 0 : kPartCost);
  };
  int64_t most = -1;
  int xcd = 0;
  for (int x = 0; x < std::min(n, kNumXcd); ++x) {
    int64_t sum = 0;
    for (int w = x; w < n; w += kNumXcd) sum += cost(w);
    if (sum > most) {
      most = sum;
      xcd = x;
    }
  }
  std::array<int64_t, kNumCu / kNumXcd> free_at{};   // a heap, the earliest first
  constexpr int N = int(free_at.size());
  int64_t end = 0;
  for (int w = xcd; w < n; w += kNumXcd)
    for (int hk = 0; hk < Hkv; ++hk) {
      const int64_t t = free_at[0] + cost(w);
      end = std::max(end, t);
      int i = 0;
      for (int c; (c = 2 * i + 1) < N; i = c) {
        if (c + 1 < N && free_at[c + 1] < free_at[c]) ++c;
        if (free_at[c] >= t) break;
        free_at[i] = free_at[c];
      }
      free_at[i] = t;
    }
  return double(end);
}

struct BwdPlan {
  SharePlan share;   // n = 0: the mask's work items, one workgroup each
  size_t ws_bytes;   // of the backward's workspace
};

// Whether equal shares beat the work items by the costs above.  Shares make
// less of L2 and cannot even out what the costs miss: they have to be 10%
// shorter, with interval lists 25% (a step's cost then varies with its lists).
// dK/dV and reduce, items -> shares, with the items' cost over the share's:
// 8192 tokens, 16 / 4 heads (1.38): 428 -> 333 us; 2048 tokens, 32 / 8 heads
// (3.0): 202 -> 91; 4 x 3000 tokens, 32 / 8 heads (1.35): 687 -> 590; 18230
// tokens, 28 / 4 heads (1.13): 2144 -> 1963.  But 16 x 2048 tokens, 28 / 4
// heads (1.08): 962 -> 1031, 32 x 1024 (1.01): 557 -> 594, 8 x 1024, 32 / 8
// heads (0.99): 160 -> 180, 878 tokens, 12 / 12 heads (147 against 105 and 192
// partial tiles): 34 -> 38, and 23286 tokens in three trajectories with
// restores, 8 / 2 heads of 64 (1.12): 1760 -> 2088.  Over 126 shapes the better
// form is missed by 0.2% on average and 5% at most.
inline bool shares_pay(const mv_view_mask& m, const SharePlan& p, int G, int Hkv) {
  const double lead = m.iv.empty() ? 1.1 : 1.25;
  return items_time(m, G, Hkv) + reduce_cost(int64_t(m.n_slots) * Hkv) >
         share_time(m, p, G) * lead + reduce_cost(p.part(p.n));
}

inline BwdPlan bwd_plan(const mv_view_mask& m, int Hq, int Hkv, int D) {
  const int G = Hq / Hkv;
  const size_t items_ws = bwd_ws_bytes(m, Hq, D, size_t(m.n_slots) * Hkv);
  BwdPlan p;
  p.share.n = 0;
  p.ws_bytes = items_ws;
  if (int64_t(m.stats.bwd_items) * Hkv > kShareMaxGroups) return p;
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
  if (!shares_pay(m, s, G, Hkv)) return p;
  p.share = s;
  p.ws_bytes = std::max(items_ws, ws);
  return p;
}

}  // namespace mv
