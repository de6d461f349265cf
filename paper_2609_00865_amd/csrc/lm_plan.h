// Sizes of the LM head's passes: vocabulary tiles, splits of the dH product,
// and the workspaces that follow from them.  Host code.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

#include "mv_internal.h"

namespace mv {

constexpr int kLmTileA = 256, kLmTileT = 256, kLmSliceK = 64;
// dH reads W itself up to this many tokens: the transposed copy costs its one
// pass over W whatever the tokens (0.40 ms at 152064 x 3584), the product on
// it runs 13% faster (4001 tokens: 3.09 against 3.53 ms; 1384 leaves: 1.12
// against 1.30 ms; 32768 tokens: 22.7 against 25.9 ms).
constexpr int kMaxDirectDh = 3072;
constexpr int kMaxDhBlocks = 2048;   // output tiles times splits
constexpr int kMaxDhSplits = 32;     // fp32 partials of a dH product split over the vocabulary

inline size_t lm_align256(size_t x) { return (x + 255) & ~size_t(255); }
inline int vocab_pad(int V) { return (V + kLmTileA - 1) / kLmTileA * kLmTileA; }
inline int token_tiles(int n) { return (n + kLmTileT - 1) / kLmTileT; }
// rows of a panel-layout matrix
inline int panel_rows(int R) { return (R + 255) / 256 * 256; }

// Vocabulary splits for a dH product: none when the output tiles already
// cover the CUs several times, otherwise the count with the least time, of
// rounds of 256 resident blocks at 1.4 us a slice (a block's slice measured
// 1.35 - 1.45 us) and the fp32 partials' way out and back at 4 TB/s; a larger
// count has to gain 3% on the one it replaces.  (With at most 8 splits,
// whatever they left idle, 777 tokens x 1024 x 32000 ran 128 blocks: dH 87 us.)
inline int dh_splits(int n_tokens, int H, int V, double gain = 0.97) {
  const int tiles = ((H + kLmTileA - 1) / kLmTileA) * token_tiles(n_tokens);
  if (tiles >= 4 * kNumCu || tiles == 0) return 1;
  const int nk = (V + kLmSliceK - 1) / kLmSliceK;
  const double part_us = double(n_tokens) * H * 8 / 4e6;   // one split's partial, both ways
  int best = 1;
  double best_t = 0;
  for (int s = 1; s <= kMaxDhSplits && s <= nk && tiles * s <= kMaxDhBlocks; ++s) {
    const double t = double((int64_t(tiles) * s + kNumCu - 1) / kNumCu) * ((nk + s - 1) / s) * 1.4 +
                     (s > 1 ? s * part_us : 0.0);
    if (s == 1 || t < gain * best_t) {
      best_t = t;
      best = s;
    }
  }
  return best;
}

// Bytes of G [n, Vp] and of the dH partials that follow it: no fewer than for
// any smaller n, so that a workspace sized for some tokens serves any fewer,
// and no more than some n' <= n takes.
//
// Within a token tile the split count depends on n through the partials' cost,
// which rises with n and, per token, with the count: a count chosen for some n
// of the tile beats every smaller one there, so it beats them at the tile's
// first n too, and the best count at that n (with no gain asked for) is at
// least as large.  Only the tiles shortly before n's can need more than n
// itself: G grows by 512 Vp bytes a tile, and the partials have a limit.
inline size_t g_bytes(int n, int V) {
  return lm_align256(size_t(panel_rows(n)) * vocab_pad(V) * sizeof(uint16_t));
}
inline size_t g_and_part_bytes(int n, int H, int V) {
  constexpr size_t most = size_t(kMaxDhBlocks) * kLmTileA * kLmTileT * sizeof(float);
  size_t need = g_bytes(n, V);
  for (int t = token_tiles(n); t > 0; --t) {
    const int last = std::min(n, t * kLmTileT);
    const size_t Gt = g_bytes(last, V);
    if (Gt + std::min(most, size_t(kMaxDhSplits) * last * H * sizeof(float)) <= need) break;
    const int s = dh_splits((t - 1) * kLmTileT + 1, H, V, 1.0);
    if (s > 1) need = std::max(need, Gt + lm_align256(size_t(s) * last * H * sizeof(float)));
  }
  return need;
}

// Whether the products over the hidden dimension take 128-row vocabulary
// tiles instead of 256: only when twice as many tiles still run at once.  A
// tile of half the rows takes 0.73 of the time (it has half the bytes of W in
// flight): 100 tokens x 1024 x 32000 (125 tiles), training step: 141 -> 130
// us, 100 leaves: 94 -> 84 us; but 201 tokens x 3584 x 152064 (594 tiles, 3
// rounds of resident blocks against 5 half ones), scoring: 273 -> 320 us.
inline bool half_tiles(int n_tokens, int V) {
  return 2 * int64_t(vocab_pad(V) / kLmTileA) * token_tiles(n_tokens) <= kNumCu;
}
// vocabulary tiles (each holds some row < V: a tile clamps its rows to V - 1)
inline int tiles_a(int n_tokens, int V) {
  const int rows = half_tiles(n_tokens, V) ? 128 : kLmTileA;
  return (V + rows - 1) / rows;
}
// partials of the logits pass at most where its tiles are 128 rows (KL: half)
constexpr size_t kHalfPartials = size_t(kLmTileT) * 2 * kNumCu;
// per-token partials of the logits and KL passes: one per tile and wave row
inline int n_chunks_of(int n_tokens, int V) { return 2 * tiles_a(n_tokens, V); }

// Whether the dH product reads W as it is, with transposing LDS reads, instead
// of a transposed copy that the call first makes of it.
inline bool dh_direct(int n_tokens) { return n_tokens <= kMaxDirectDh; }
inline size_t wT_bytes(int n_tokens, int H, int V) {
  return dh_direct(n_tokens) ? 0
                             : lm_align256(size_t(panel_rows(H)) * vocab_pad(V) * sizeof(uint16_t));
}

}  // namespace mv
