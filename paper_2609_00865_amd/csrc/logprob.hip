// Fused LM-head token log-prob, ratio and clip on gfx950.
//
// Forward: z = W h is produced 256 vocab rows x 256 tokens at a time by a bf16
// MFMA tile engine and reduced in registers to a per-token (max, sum of exp)
// over each wave's 128 (or 64) vocab rows; the full logits are never stored.  A
// combine pass (one wave per token) takes the target logit z_{t,y_t} as an
// fp32 dot product, merges the partials into logsumexp and writes logp,
// ratio and the clipped ratio (the GRPO ratio of Appendix C, "Pitfall A, RL
// view"); its fused variant also evaluates the GRPO loss of each token and
// its gradient, and reduces the drift statistics (Eq. "logdiff") in the same
// pass.
//
// Backward: the logits tile is recomputed and turned into
// G_tv = g_t (onehot(y_t)_v - softmax(z_t)_v), stored once in bf16 (the tile
// writes -g_t softmax(z_t)_v everywhere, the per-token pass then rewrites the
// target entry), and a second pass of the same engine computes dH = G W from
// a transposed copy of W, so that both operands run along the vocabulary (for
// few tokens, where that copy is a large part of the call, from W itself,
// read across its rows).
// dW = G^T H contracts over tokens, along which neither operand is
// contiguous: it has an engine of its own that stages both operands k-major
// and reads them with the transposing LDS read.
//
// Tile engine (logits, G, the KL passes, dH): 512 threads = 8 waves (two per
// SIMD) in a 2 x 4 grid over a 256 A-row x 256 token tile; each wave owns 128
// A rows x 64 tokens and runs MFMA 16x16x32.  64-wide k slices go from HBM
// straight into LDS (global_load_lds: no register staging and no LDS store
// instructions), two slices deep.  The two waves of a SIMD take turns: one
// runs the MFMAs of a quarter of its tile while the other reads its next
// fragments from LDS and issues its share of a later slice's loads, so the
// matrix pipe is not waiting behind LDS reads, and quarter by quarter the
// slice's LDS regions are free for the slice after next (a load has 1.5
// slices to land).  Bound by the matrix pipe at the clock the chip holds
// under it: at 32768 tokens x 3584 x 152064, on two boxes, the pipe is busy
// 81-82% (logits), 73-75% (G) and 93% (dH) of the cycles at 1.76-1.81,
// 1.78-1.87 and 1.59-1.64 GHz, where the earlier loop (both waves reading, then
// both in MFMAs; one barrier per slice) had 56-64%.  Both timed in turn: at 4001 tokens logits 3.54 -> 3.22 ms, G 3.73 ->
// 3.20, dH 3.50 -> 3.11; at 32768: 26.7 -> 24.5, 28.6 -> 26.0, 26.0 -> 23.1.  An
// operand slice sits in LDS as [256 rows][64] bf16 without padding, with
// 16-byte chunk c of row r at chunk position c ^ (r & 7): the fragment reads
// (16 lanes = 16 consecutive rows at one chunk) hit distinct banks.  Tiles are
// ordered so that the blocks resident on one XCD at a time form a compact 2-D
// patch (a few token tiles x several A tiles) and share operand slices in that
// XCD's L2.
#include <algorithm>
#include <type_traits>

#include "lm_plan.h"
#include "mv_grpo_dev.h"

namespace mv {

namespace {
constexpr int BA = kLmTileA, BT = kLmTileT, BKK = kLmSliceK;
constexpr int NWAVES = 8;                  // waves per tile (2 x 4 grid)
// token tiles per raster group: 8 x 4 A tiles run side by side on an XCD
// for the products over the hidden dimension (measured ~1% faster than
// 4 x 8), 4 x 8 for dH and dW
constexpr int GROUP_T_H = 8, GROUP_T_V = 4;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.69314718055994531f;
// tile engine
constexpr int SLICE_B = 256 * BKK * 2;             // bytes of one operand's k slice

// Panel layout of a bf16 matrix [R][K] (R padded to a multiple of 256, K a
// multiple of 64), used for G and W^T, the operands of the dH product whose
// k runs along the vocabulary: the 64-wide k slice of a 256-row block is one
// contiguous 32 KiB panel of 128-byte rows, so each slice load of a tile is
// one linear read instead of 256 rows a vocabulary row (~300 KB) apart.
constexpr int PANEL = 256 * 64;
__host__ __device__ inline size_t panel_index(int r, int k, int K) {
  return (size_t(r >> 8) * (K >> 6) + (k >> 6)) * PANEL + (r & 255) * 64 + (k & 63);
}
constexpr int FB = 4;                              // 16-row MFMA blocks per wave: tokens
static_assert(4 * NWAVES * 1024 == SLICE_B, "two regions of two 1 KiB loads per wave");
size_t align256(size_t x) { return lm_align256(x); }
}  // namespace

enum { kModeLogits = 0, kModeGrad = 1, kModeDh = 2, kModeKL = 3, kModeKLGrad = 4, kModeDhW = 5 };

hipError_t launch_grpo_fused_finish(const float* part, int n_blocks, int stride, int n_traj,
                                    const float* adv, float* stats, hipStream_t stream);

struct LmArgs {
  const u16* h;       // [T, H]
  const u16* w;       // [V, H]
  const u16* wT;      // [H, Vp] (dH mode: W transposed, zero past V)
  const int32_t* tgt; // [T]
  const float* lse;   // [T] (grad mode)
  const float* g;     // [T] upstream dlogp (grad mode)
  const u16* G;       // [T, Vp] (dH and dW modes)
  u16* Gout;          // [T, Vp] (grad modes)
  u16* dh;            // [T, H] (dH mode)
  float2* part;       // [T, n_chunks] (logits mode)
  // KL modes: token row 2i is leaf i's teacher row, 2i + 1 its student row
  const u16* zero_row; // [H] zeros: the row read for an out-of-range leaf row index
  const u16* hT;      // teacher hidden states [*, H]
  const u16* hS;      // student hidden states [*, H]
  const int32_t* rowsT;
  const int32_t* rowsS;
  float4* partT;      // [n, n_chunks] (max, sum, cross, -) of the teacher
  float2* partS;      // [n, n_chunks] (max, sum) of the student
  const float* lseT;  // [n] (KL grad mode)
  const float* lseS;
  const float* dkl;   // [n] upstream gradient of each leaf's KL
  int n_leaves, n_rows_T, n_rows_S;
  int T, H, V, Vp, n_chunks;
  int nA, nT;         // tiles along the A side and along tokens
  // dH mode split over the vocabulary (K) when there are too few output
  // tiles to fill the chip: split s covers k slices [s*nk_split, ...) and
  // writes fp32 partials dh_part[s][t][H], summed in order by dh_reduce_kernel
  int k_split, nk_split;
  float* dh_part;
  float* dw;          // [V, H] fp32 (dW)
  int* bad_targets;   // count of target ids outside [-1, V) met by this call
};

// Output tile (a0, t0) and k split of this block.  Blocks are dealt to XCDs
// round-robin; each XCD gets a contiguous range of the rasterised tile order
// (groups of GT token tiles x all A tiles).  False: no tile (grid tail).
template <int GT, int TA = BA>
__device__ __forceinline__ bool tile_of(const LmArgs& a, int n_splits, int& a0, int& t0,
                                        int& split) {
  const int n_out = a.nA * a.nT;
  const int n_tiles = n_out * n_splits;
  const int per_xcd = (n_tiles + kNumXcd - 1) / kNumXcd;
  int xcd, local;
  xcd_split(xcd, local);
  const int Lx = xcd * per_xcd + local;
  if (local >= per_xcd || Lx >= n_tiles) return false;
  split = Lx / n_out;
  const int L = Lx % n_out;
  const int grp = L / (GT * a.nA);
  const int rem = L % (GT * a.nA);
  const int t_in = min(GT, a.nT - grp * GT);
  a0 = (rem / t_in) * TA;
  t0 = (grp * GT + rem % t_in) * BT;
  return true;
}

// The k loop of a 256 x 256 tile over nk >= 1 slices of 64.  Waves w and w + 4
// share a SIMD and take turns: between two barriers one runs the MFMAs of a
// quarter of its tile (mma(ha, hb): half ha of its A fragments x half hb of
// its B fragments, 256 cycles), the other loads: the fragments of its next
// quarter from LDS (read_a / read_b of a half, from the current buffer) and
// its share of a region of the slice after next (issue_a /
// issue_b(half, slice)).  A region is the part of an operand slice that the
// waves' fragments of one half come from.  The quarters of a slice go (0,0)
// (0,1) (1,1) (1,0); before them are read B0, B1, A1 and the next slice's A0
// (flip(d) moves the fragment addresses to the other buffer), so a region is
// free for its next load one or two turns after it is read, and each load has
// about 12 turns (1.5 slices) to land.  late: this wave runs one turn behind.
// On return every load has landed and every wave is done with the LDS reads.
// LA, LB: loads per region and wave of either operand.
template <int LA, int LB, class IA, class IB, class RA, class RB, class FL, class MM>
__device__ __forceinline__ void tile_pipeline(int nk, bool late, IA issue_a, IB issue_b, RA read_a,
                                              RB read_b, FL flip, MM mma) {
  auto turn = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  // before the barrier that ends a load turn: the wave's LDS reads are done
  // (their region may be overwritten), the loads the next turns read landed
  auto read_done = [&]() { __builtin_amdgcn_s_waitcnt(0xC07F); };   // lgkmcnt(0)
  auto quarter = [&](int ha, int hb) {
    turn();
    __builtin_amdgcn_s_setprio(1);
    mma(ha, hb);
    __builtin_amdgcn_s_setprio(0);
    turn();
  };
  // order of the loads: A0 B0 B1 A1 of slice 0, of slice 1, ...; each wait
  // keeps the six regions younger than the one it waits for in flight
  auto issue_slice = [&](int kk) {
    issue_a(0, kk);
    issue_b(0, kk);
    issue_b(1, kk);
    issue_a(1, kk);
  };
  issue_slice(0);
  if (nk > 1) {
    issue_slice(1);
    wait_vmcnt<3 * LA + 3 * LB>();   // A0, B0 of slice 0
  } else {
    wait_vmcnt<0>();
  }
  __syncthreads();
  read_a(0);
  read_done();
  turn();
  if (late) turn();
  // one slice; MORE: slice kk + 2 exists; w0 .. w3: loads that may stay in
  // flight at each turn
  auto slice = [&](int kk, auto more_tag, auto last_tag, auto w0, auto w1, auto w2, auto w3) {
    constexpr bool MORE = decltype(more_tag)::value, LAST = decltype(last_tag)::value;
    if (MORE) issue_a(0, kk + 2);
    read_b(0);
    wait_vmcnt<decltype(w0)::value>();
    read_done();
    quarter(0, 0);
    if (MORE) issue_b(0, kk + 2);
    read_b(1);
    wait_vmcnt<decltype(w1)::value>();
    read_done();
    quarter(0, 1);
    if (MORE) issue_b(1, kk + 2);
    read_a(1);
    wait_vmcnt<decltype(w2)::value>();
    read_done();
    quarter(1, 1);
    flip((kk & 1) ? uint32_t(-SLICE_B) : uint32_t(SLICE_B));
    if (MORE) issue_a(1, kk + 2);
    if (!LAST) read_a(0);
    wait_vmcnt<decltype(w3)::value>();
    read_done();
    quarter(1, 0);
  };
  using std::integral_constant;
  using T = std::true_type;
  using F = std::false_type;
  constexpr int R = LA + LB;   // loads of half a slice
  for (int kk = 0; kk + 2 < nk; ++kk)
    slice(kk, T{}, F{}, integral_constant<int, 2 * R + 2 * LA>{}, integral_constant<int, 3 * R>{},
          integral_constant<int, 2 * R + 2 * LB>{}, integral_constant<int, 3 * R>{});
  if (nk > 1)
    slice(nk - 2, F{}, F{}, integral_constant<int, 2 * R + LA>{}, integral_constant<int, 2 * R>{},
          integral_constant<int, R + LB>{}, integral_constant<int, R>{});
  slice(nk - 1, F{}, T{}, integral_constant<int, LA>{}, integral_constant<int, 0>{},
        integral_constant<int, 0>{}, integral_constant<int, 0>{});
  if (!late) turn();
}

// TA: A rows of the tile, 256 or 128 (each wave half as many rows; see
// half_tiles).
template <int MODE, int TA = BA>
__global__ __launch_bounds__(NWAVES * 64, 1) void lm_tile_kernel(LmArgs a) {
  __shared__ __align__(1024) u16 smem[2 * 2 * SLICE_B / 2];   // 2 slices x 2 operands

  // the call's status block (256 bytes), for the passes after this one
  if ((MODE == kModeLogits || MODE == kModeGrad) && blockIdx.x == 0 && threadIdx.x < 64)
    a.bad_targets[threadIdx.x] = 0;

  constexpr int FA = TA / 32;      // 16-row MFMA blocks per wave along A
  constexpr int WR = TA / 2;       // A rows per wave
  constexpr int NQA = TA / 128;    // loads per A region and wave
  int a0, t0, split;
  constexpr bool DH = MODE == kModeDh || MODE == kModeDhW;
  constexpr int GT = DH ? GROUP_T_V : GROUP_T_H;
  if (!tile_of<GT, TA>(a, DH ? a.k_split : 1, a0, t0, split)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wa = wave >> 2, wt = wave & 3;

  // A [a_rows][K] and B [T][K], both contiguous along k; kModeDhW: A is W
  // itself, [K][a_rows]
  constexpr bool TRA = MODE == kModeDhW;
  const int K = DH ? a.Vp : a.H;
  const int a_rows = DH ? a.H : a.V;
  const u16* A = MODE == kModeDh ? a.wT : a.w;
  const int kbeg = DH ? split * a.nk_split : 0;
  const int nk = DH ? min((a.V + BKK - 1) / BKK - kbeg, a.nk_split) : K / BKK;

  // Slice loads.  Each operand slice is loaded in two regions of 128 rows,
  // the rows that every wave's first (region 0) and second (1) half of its
  // fragments come from: A rows 64 of each 128 (128-row tiles: 32 of each 64,
  // one load), token rows 32 of each 64.
  // Load q of this wave fills rows rowX(h, q) + lane / 8, whose 16-byte chunk
  // position lane % 8 holds chunk (lane % 8) ^ (row % 8).  Rows past the
  // operands are read from clamped (valid) rows; their products land in
  // output rows or columns that the epilogues skip.  The dH product reads
  // G (and W^T) in the panel layout, the others row-major.
  // kModeDhW: the regions of A are sub-tiles of 64 vocabulary rows x 64
  // hidden columns, h and h + 2, in 128-byte rows with chunk c of row r at
  // position c ^ ((r & 2) | (r & 8) / 2): a transposing fragment read (rows 0-3
  // and 8-11 x 32 bytes per 32 lanes) hits distinct banks.
  constexpr bool PANELS = DH;
  constexpr bool GATHER = MODE == kModeKL || MODE == kModeKLGrad;
  constexpr uint32_t SSTEP = (PANELS ? PANEL : BKK) * 2;   // bytes from a row's k slice to the next
  auto row_a = [&](int h, int q) {
    return TA == 256 ? q * 128 + h * 64 + wave * 8
                     : (wave >> 2) * 64 + h * 32 + (wave & 3) * 8;
  };
  auto row_b = [&](int h, int q) { return q * 128 + (wave >> 2) * 64 + h * 32 + (wave & 3) * 8; };
  const size_t tile_a = TRA ? size_t(0) : PANELS ? panel_index(a0, kbeg * BKK, K) : size_t(a0) * K;
  const size_t tile_b = PANELS ? panel_index(t0, kbeg * BKK, K) : size_t(t0) * K;
  const char* baseA = reinterpret_cast<const char*>(uniform_ptr(A + tile_a));
  const char* baseB =
      GATHER ? nullptr : reinterpret_cast<const char*>(uniform_ptr((PANELS ? a.G : a.h) + tile_b));
  uint32_t offA[2][2], offB[2][2];
  const u16* rowB[2][2];   // gathered token rows
  const uint32_t row_bytes = PANELS ? BKK * 2 : uint32_t(K) * 2;
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const uint32_t ch = ((lane & 7) ^ (lane >> 3)) * 16;
      const int ra = min(row_a(h, q) + (lane >> 3), a_rows - 1 - a0);
      const int rb = min(row_b(h, q) + (lane >> 3), a.T - 1 - t0);
      offA[h][q] = uint32_t(ra) * row_bytes + ch;
      offB[h][q] = uint32_t(rb) * row_bytes + ch;
      if (GATHER) {
        // a row index outside its matrix reads as a zero hidden state
        const int t = t0 + rb;
        const int r = (t & 1) ? a.rowsS[t >> 1] : a.rowsT[t >> 1];
        const int n_rows = (t & 1) ? a.n_rows_S : a.n_rows_T;
        rowB[h][q] = ((r >= 0 && r < n_rows) ? ((t & 1) ? a.hS : a.hT) + size_t(r) * a.H
                                             : a.zero_row) + ch / 2;
      }
    }
  const int lrow = wave * 8 + (lane >> 3);   // kModeDhW: this lane's row of a sub-tile
  const uint32_t wch = ((lane & 7) ^ ((lrow & 2) | ((lrow & 8) >> 1))) * 16;
  // LDS: A slice in buffer b at b * 32 KiB, B at 64 KiB + b * 32 KiB, rows of
  // 128 bytes
  const uint32_t lds0 = lds_addr(smem);
  auto issue_a = [&](int h, int kk) {
    const uint32_t st = lds0 + (kk & 1) * SLICE_B;
    if (TRA) {
      // vocabulary rows past V read row V - 1 and meet zeros of G; hidden
      // columns past H (whole sub-tiles) the last ones: outputs skipped
      const int k0 = (kbeg + kk) * BKK;   // < V
      const uint32_t off = uint32_t(min(lrow, a.V - 1 - k0)) * (uint32_t(a.H) * 2) + wch;
#pragma unroll
      for (int q = 0; q < 2; ++q)
        lds_load16s(baseA + (size_t(k0) * a.H + min(a0 + (h + 2 * q) * 64, a.H - 64)) * 2, off,
                    st + row_a(h, q) * 128);
      return;
    }
    const char* b = baseA + size_t(kk) * SSTEP;
#pragma unroll
    for (int q = 0; q < NQA; ++q) lds_load16s(b, offA[h][q], st + row_a(h, q) * 128);
  };
  auto issue_b = [&](int h, int kk) {
    const uint32_t st = lds0 + 2 * SLICE_B + (kk & 1) * SLICE_B;
    if (GATHER) {
      lds_load16(rowB[h][0] + size_t(kk) * BKK, st + row_b(h, 0) * 128);
      lds_load16(rowB[h][1] + size_t(kk) * BKK, st + row_b(h, 1) * 128);
    } else {
      const char* b = baseB + size_t(kk) * SSTEP;
      lds_load16s(b, offB[h][0], st + row_b(h, 0) * 128);
      lds_load16s(b, offB[h][1], st + row_b(h, 1) * 128);
    }
  };

  // Fragments of half h: 16 consecutive rows at one chunk per read
  const int frow = lane & 15, fk = lane >> 4;
  uint32_t pa = lds0 + (wa * WR + frow) * 128 + ((fk ^ (frow & 7)) * 16);
  if (TRA) {   // lane j of a 16-lane group: row fk * 8 + j / 4 (and + 4), columns 4 (j % 4)
    const int r = fk * 8 + (frow >> 2);
    pa = lds0 + wa * 128 * 128 + r * 128 +
         ((((frow & 3) >> 1) ^ ((r & 2) | ((r & 8) >> 1))) * 16) + (frow & 1) * 8;
  }
  uint32_t pb = lds0 + 2 * SLICE_B + (wt * 64 + frow) * 128 + ((fk ^ (frow & 7)) * 16);
  bf16x8 fa[2][2][FA / 2], fb[2][2][FB / 2];   // [half][k step][block]
  auto read_a = [&](int h, uint32_t p) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < FA / 2; ++i)
        fa[h][ks][i] = TRA ? lds_frag_tr((p ^ (i * 32)) + h * 8192 + ks * 32 * 128, 4 * 128)
                           : lds_frag((p ^ (ks * 64)) + h * (WR / 2) * 128 + i * 2048);
  };
  auto read_b = [&](int h, uint32_t p) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int j = 0; j < FB / 2; ++j)
        fb[h][ks][j] = lds_frag((p ^ (ks * 64)) + h * 4096 + j * 2048);
  };

  f32x4 acc[FA][FB];
#pragma unroll
  for (int i = 0; i < FA; ++i)
#pragma unroll
    for (int j = 0; j < FB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto mma = [&](int ha, int hb) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < FA / 2; ++i)
#pragma unroll
        for (int j = 0; j < FB / 2; ++j)
          acc[ha * (FA / 2) + i][hb * (FB / 2) + j] =
              mfma16(fa[ha][ks][i], fb[hb][ks][j], acc[ha * (FA / 2) + i][hb * (FB / 2) + j]);
  };
  auto flip = [&](uint32_t d) {
    pa += d;
    pb += d;
  };
  tile_pipeline<NQA, 2>(nk, wa == 1, issue_a, issue_b, [&](int h) { read_a(h, pa); },
                        [&](int h) { read_b(h, pb); }, flip, mma);

  // acc[i][j][r]: A row rb + i*16 + r, token tb + j*16
  const int rb = a0 + wa * WR + (lane >> 4) * 4;
  const int tb = t0 + wt * 64 + (lane & 15);
  const bool full_v = a0 + TA <= a.V;  // block-uniform: no vocabulary padding in this tile
  const int chunk = (a0 + wa * WR) / WR;
  if (MODE == kModeLogits) {
#pragma unroll
    for (int j = 0; j < FB; ++j) {
      const int t = tb + j * 16;
      float mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < FA; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (!full_v && rb + i * 16 + r >= a.V) acc[i][j][r] = -INFINITY;
          mx = fmaxf(mx, acc[i][j][r]);
        }
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float m2 = mx * kLog2e;                // -inf for a chunk of padding only
      const float mu = mx == -INFINITY ? 0.f : m2;
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < FA; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) s += fast_exp2(fmaf(acc[i][j][r], kLog2e, -mu));
      s += __shfl_xor(s, 16);
      s += __shfl_xor(s, 32);
      if (lane < 16 && t < a.T) a.part[size_t(t) * a.n_chunks + chunk] = make_float2(m2, s);
    }
  } else if (MODE == kModeGrad) {
    // -g_t softmax(z_t)_v everywhere (zero from V to the tile's end; rows
    // past T, which pad the dW product's k, are zeros too); the target
    // entry gets its one-hot term from lm_target_kernel afterwards.  The
    // tile's block of G is one contiguous run of TA / 64 panels (128 or 64
    // KiB): it is assembled in LDS in that order (the 16-byte chunks of each
    // 128-byte row permuted by the row's low bits, against bank conflicts) and
    // written with 16-byte stores that cover whole lines.
    char* sg = reinterpret_cast<char*>(smem);
    __syncthreads();   // every wave has read its last operand fragments
#pragma unroll
    for (int j = 0; j < FB; ++j) {
      const int t = tb + j * 16;
      const int tl = t - t0;                       // row within the tile's panels
      const int tc = min(t, a.T - 1);
      const int y = a.tgt[tc];
      // an id outside [0, V) carries no loss (-1 by convention; any other is
      // counted by lm_target_kernel)
      const float ng = (uint32_t(y) < uint32_t(a.V) && t < a.T) ? -a.g[tc] : 0.f;
      const float l2 = a.lse[tc] * kLog2e;
#pragma unroll
      for (int i = 0; i < FA; ++i) {
        const int vl = rb + i * 16 - a0;             // 4 consecutive entries vl ..
        float vals[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          vals[r] = ng * fast_exp2(fmaf(acc[i][j][r], kLog2e, -l2));
          if (!full_v && rb + i * 16 + r >= a.V) vals[r] = 0.f;
        }
        uint2 wv;
        wv.x = pack2(vals[0], vals[1]);
        wv.y = pack2(vals[2], vals[3]);
        const int c = vl & 63;
        *reinterpret_cast<uint2*>(sg + (vl >> 6) * 32768 + tl * 128 +
                                  ((((c >> 3) ^ (tl & 7)) << 4) | ((c & 7) * 2))) = wv;
      }
    }
    __syncthreads();
    uint4* gt = reinterpret_cast<uint4*>(a.Gout + panel_index(t0, a0, a.Vp));
#pragma unroll 4
    for (int k = tid; k < TA * BT * 2 / 16; k += NWAVES * 64) {
      const int q = k >> 11, r = (k >> 3) & 255, c16 = k & 7;
      gt[k] = *reinterpret_cast<const uint4*>(sg + (q << 15) + (r << 7) + ((c16 ^ (r & 7)) << 4));
    }
  } else if (MODE == kModeKL) {
    // lanes c (even, teacher) and c ^ 1 (student) hold the same vocabulary
    // rows of one leaf; each lane keeps its own (max, sum of exp) and the
    // teacher also accumulates sum exp(zT - mT) * (zT - zS)
#pragma unroll
    for (int j = 0; j < FB; ++j) {
      const int t = tb + j * 16;
      const int leaf = t >> 1;
      float mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < FA; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (full_v || rb + i * 16 + r < a.V) mx = fmaxf(mx, acc[i][j][r]);
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float m2 = mx * kLog2e;
      const float mu = mx == -INFINITY ? 0.f : m2;
      float sm = 0.f, cross = 0.f;
#pragma unroll
      for (int i = 0; i < FA; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float z = acc[i][j][r];
          const float zo = __shfl_xor(z, 1);  // the partner row's logit
          const bool ok = full_v || rb + i * 16 + r < a.V;
          const float e = ok ? fast_exp2(fmaf(z, kLog2e, -mu)) : 0.f;
          sm += e;
          cross += e * (z - zo);
        }
      sm += __shfl_xor(sm, 16);
      sm += __shfl_xor(sm, 32);
      cross += __shfl_xor(cross, 16);
      cross += __shfl_xor(cross, 32);
      if (lane < 16 && leaf < a.n_leaves) {
        const size_t o = size_t(leaf) * a.n_chunks + chunk;
        if (t & 1)
          a.partS[o] = make_float2(m2, sm);
        else
          a.partT[o] = make_float4(m2, sm, cross, 0.f);
      }
    }
  } else if (MODE == kModeKLGrad) {
    // student lanes write G = dkl * (q - p) for their leaf
#pragma unroll
    for (int j = 0; j < FB; ++j) {
      const int t = tb + j * 16;
      const int leaf = t >> 1;
      const bool student = (t & 1) && leaf < a.n_leaves;
      const int lc = leaf < a.n_leaves ? leaf : 0;
      const float gl = a.dkl[lc];
      const float lS = a.lseS[lc] * kLog2e, lT = a.lseT[lc] * kLog2e;
#pragma unroll
      for (int i = 0; i < FA; ++i) {
        u16* out = a.Gout + panel_index(lc, rb + i * 16, a.Vp);
        float vals[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float zS = acc[i][j][r];
          const float zT = __shfl_xor(zS, 1);
          const float q = fast_exp2(fmaf(zS, kLog2e, -lS));
          const float pt = fast_exp2(fmaf(zT, kLog2e, -lT));
          vals[r] = (full_v || rb + i * 16 + r < a.V) ? gl * (q - pt) : 0.f;
        }
        if (student) {
          uint2 wv;
          wv.x = pack2(vals[0], vals[1]);
          wv.y = pack2(vals[2], vals[3]);
          *reinterpret_cast<uint2*>(out) = wv;
        }
      }
    }
  } else {  // dH: A rows are hidden columns
#pragma unroll
    for (int j = 0; j < FB; ++j) {
      const int t = tb + j * 16;
      if (t >= a.T) continue;
      if (a.k_split > 1) {
        float* out = a.dh_part + (size_t(split) * a.T + t) * a.H;
#pragma unroll
        for (int i = 0; i < FA; ++i) {
          const int hcol = rb + i * 16;
          if (hcol < a.H)
            *reinterpret_cast<float4*>(out + hcol) =
                make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
        }
      } else {
        u16* out = a.dh + size_t(t) * a.H;
#pragma unroll
        for (int i = 0; i < FA; ++i) {
          const int hcol = rb + i * 16;
          if (hcol < a.H) {
            uint2 wv;
            wv.x = pack2(acc[i][j][0], acc[i][j][1]);
            wv.y = pack2(acc[i][j][2], acc[i][j][3]);
            *reinterpret_cast<uint2*>(out + hcol) = wv;
          }
        }
      }
    }
  }
}

// dW[v][c] = sum_t G[t][v] H[t][c] (fp32 out).  Same tile shape and pipeline
// as the tile engine (256 vocabulary rows x 256 hidden columns, 8 waves) with
// MFMA 32x32x16; k = tokens, along which neither operand is contiguous.  Both
// k slices (64 tokens x 256 columns) go from HBM straight into LDS as four
// sub-tiles of 64 columns: 128-byte token rows, with 16-byte chunk c of row r
// at position c ^ ((r & 2) << 1), so that a transposing operand read (four
// token rows x 64 bytes per 32 lanes) hits distinct banks.  A wave owns 128
// vocabulary rows (two sub-tiles, its two halves) and the columns wt * 32 of
// each 128 (its two halves).  G's rows past T are zeros up to a multiple of
// 256 (the grad pass writes them), so the last slice needs no masking: H rows
// past T are read clamped and meet zero G rows.  Bound as the tile engine: at
// 32768 tokens x 3584 x 152064 the loop in which both waves of a SIMD read and
// multiplied together took 31.7 ms with the pipe 64% busy, this one 28.3 ms
// with 85%.
__global__ __launch_bounds__(NWAVES * 64, 1) void lm_dw_kernel(LmArgs a) {
  __shared__ __align__(1024) u16 smem[2 * 2 * SLICE_B / 2];   // (G, H) x 2 slices
  constexpr int SUB = 64 * 128;   // bytes of a sub-tile

  int a0, t0, split;
  if (!tile_of<GROUP_T_V>(a, 1, a0, t0, split)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wa = wave >> 2, wt = wave & 3;
  const int nk = (a.T + BKK - 1) / BKK;

  // Region h of G: the sub-tiles h and h + 2 (half h of the waves' rows), of H:
  // the sub-tiles 2 h and 2 h + 1 (half h of their columns).  Load q of this
  // wave fills rows wave * 8 + lane / 8 of the region's sub-tile q.
  const uint32_t lds0 = lds_addr(smem);
  const int lrow = wave * 8 + (lane >> 3);
  const uint32_t lch = ((lane & 7) ^ ((lrow & 2) << 1)) * 16;
  const uint32_t goff = lrow * 128 + lch;
  const uint32_t hrow_bytes = uint32_t(a.H) * 2;
  const char* Gb = reinterpret_cast<const char*>(uniform_ptr(a.G + panel_index(0, a0, a.Vp)));
  const size_t gstep = size_t(a.Vp >> 6) * PANEL * 2;   // bytes from 256 token rows to the next
  const char* Hb = reinterpret_cast<const char*>(uniform_ptr(a.h));
  auto issue_a = [&](int h, int kk) {
    const char* b = Gb + size_t(kk >> 2) * gstep + (kk & 3) * SUB;
    const uint32_t st = lds0 + (kk & 1) * SLICE_B + wave * 1024;
    lds_load16s(b + size_t(h) * (PANEL * 2), goff, st + h * SUB);
    lds_load16s(b + size_t(h + 2) * (PANEL * 2), goff, st + (h + 2) * SUB);
  };
  auto issue_b = [&](int h, int kk) {
    const int k0 = kk * BKK;   // < T
    const uint32_t off = uint32_t(min(lrow, a.T - 1 - k0)) * hrow_bytes + lch;
    const uint32_t st = lds0 + 2 * SLICE_B + (kk & 1) * SLICE_B + wave * 1024;
    // hidden columns past H (whole sub-tiles) read the last ones: outputs skipped
#pragma unroll
    for (int q = 0; q < 2; ++q)
      lds_load16s(Hb + size_t(k0) * hrow_bytes + min(t0 + (2 * h + q) * 64, a.H - 64) * 2, off,
                  st + (2 * h + q) * SUB);
  };

  // Transposing operand read in natural k order (rows g*8 + 0..7 of a k step
  // of 16): lane l of a 16-lane group reads token rows (lane/32)*8 + l/4 and +
  // 4, columns col0 + ((lane/16) % 2)*16 + 4 (l % 4); the swizzle term of a
  // lane is fixed (row & 2 = (l / 4) & 2), and col0 = 32 is chunk bit 2.
  const int l = lane & 15;
  const int rl = (lane >> 5) * 8 + (l >> 2);
  const uint32_t fr = rl * 128 +
                      (((((lane >> 4) & 1) * 2 + ((l & 3) >> 1)) ^ ((rl & 2) << 1)) << 4) +
                      (l & 1) * 8;
  uint32_t pa = lds0 + wa * 2 * SUB + fr;
  uint32_t pb = lds0 + 2 * SLICE_B + (wt >> 1) * SUB + (fr ^ ((wt & 1) * 64));
  auto tr = [&](uint32_t p) { return lds_frag_tr(p, 4 * 128); };
  bf16x8 fa[2][4][2], fb[2][4];   // [half][k step](block)
  auto read_a = [&](int h) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int i = 0; i < 2; ++i) fa[h][ks][i] = tr((pa ^ (i * 64)) + h * SUB + ks * 16 * 128);
  };
  auto read_b = [&](int h) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) fb[h][ks] = tr(pb + h * 2 * SUB + ks * 16 * 128);
  };
  auto flip = [&](uint32_t d) {
    pa += d;
    pb += d;
  };

  f32x16 acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  auto mma = [&](int ha, int hb) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int i = 0; i < 2; ++i)
        acc[ha * 2 + i][hb] = mfma32(fa[ha][ks][i], fb[hb][ks], acc[ha * 2 + i][hb]);
  };
  tile_pipeline<2, 2>(nk, wa == 1, issue_a, issue_b, read_a, read_b, flip, mma);

  // acc[i][j][r]: vocabulary row a0 + wa*128 + i*32 + (r/4)*8 + g*4 + r%4,
  //               hidden column t0 + j*128 + wt*32 + c
  const int c = lane & 31, g = lane >> 5;
  const int arow0 = a0 + wa * 128;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int hc = t0 + j * 128 + wt * 32 + c;
    if (hc >= a.H) continue;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int v = arow0 + i * 32 + (r >> 2) * 8 + g * 4 + (r & 3);
        if (v < a.V) a.dw[size_t(v) * a.H + hc] = acc[i][j][r];
      }
  }
}

// Target logit z_{t,y_t} = h_t . W[y_t] in fp32 by one wave (lane k takes
// 16-byte chunks k, k + 64, ...; a fixed shuffle tree sums the lanes), so
// that the forward's combine and the backward's fix-up see the same value.
__device__ __forceinline__ float target_dot(const LmArgs& a, int t, int y, int lane) {
  const u16* hp = a.h + size_t(t) * a.H;
  const u16* wp = a.w + size_t(y) * a.H;
  float s = 0.f;
  for (int k = lane * 8; k < a.H; k += 512) {
    const uint4 hv = ld16(hp + k), wv = ld16(wp + k);
    const uint32_t hw[4] = {hv.x, hv.y, hv.z, hv.w}, ww[4] = {wv.x, wv.y, wv.z, wv.w};
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      s = fmaf(bf16_to_f32(u16(hw[u])), bf16_to_f32(u16(ww[u])), s);
      s = fmaf(bf16_to_f32(u16(hw[u] >> 16)), bf16_to_f32(u16(ww[u] >> 16)), s);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  return s;
}

// Backward fix-up, one wave per token: rewrites G[t][y_t], which the grad
// tile left at -g_t p, to g_t (1 - p) with p = softmax(z_t)_{y_t} from the
// forward's lse.  An id outside [-1, V) is never used as an index: the token
// is treated as one without loss and counted in *bad_targets (this kernel
// sees every token exactly once per call).
__global__ __launch_bounds__(256) void lm_target_kernel(LmArgs a) {
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (t >= a.T) return;
  const int y = a.tgt[t];
  if (uint32_t(y) >= uint32_t(a.V)) {
    if (lane == 0 && y != -1) atomicAdd(a.bad_targets, 1);
    return;
  }
  const float s = target_dot(a, t, y, lane);
  if (lane != 0) return;
  const float p = fast_exp2(fmaf(s, kLog2e, -a.lse[t] * kLog2e));
  a.Gout[panel_index(t, y, a.Vp)] = u16(bf16_bits(a.g[t] * (1.f - p)));
}

// wT[h][v] = w[v][h] for v < V and 0 for V <= v < Vp, in the panel layout;
// 64 x 64 tiles through LDS.
__global__ __launch_bounds__(256) void transpose_w_kernel(const u16* w, u16* wT, int V, int H,
                                                          int Vp) {
  __shared__ u16 tile[64][72];
  const int v0 = blockIdx.x * 64, h0 = blockIdx.y * 64;
  const int tid = threadIdx.x;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int idx = tid + q * 256;
    const int r = idx >> 3, c = (idx & 7) * 8;
    const uint4 val = v0 + r < V ? ld16(w + size_t(v0 + r) * H + h0 + c) : make_uint4(0, 0, 0, 0);
    st16(&tile[r][c], val);
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int idx = tid + q * 256;
    const int r = idx >> 3, c = (idx & 7) * 8;   // wT row h0 + r, columns v0 + c .. + 8
    uint32_t e[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      e[u] = uint32_t(tile[c + 2 * u][r]) | (uint32_t(tile[c + 2 * u + 1][r]) << 16);
    st16(wT + panel_index(h0 + r, v0 + c, Vp), make_uint4(e[0], e[1], e[2], e[3]));
  }
}

// Outputs of the forward's combine pass; the GRPO fields are used only by the
// fused variant (mv_token_logprob_grpo).
struct CombineOut {
  const float* logp_old;
  float* logp;
  float* ratio;
  float* clipped;
  float* lse;
  float eps_lo, eps_hi;
  // GRPO loss fused into the pass
  const int32_t* traj_ptr;
  const float* reward;
  const float* logp_ref;     // null: no reference KL
  const uint8_t* mask;       // null: every token carries loss
  const float* adv;          // [n_traj] advantages from the preparation pass
  const int* n_loss_count;   // loss tokens counted by the preparation pass (mask given)
  int n_loss_fixed;          // the count when there is no mask (-1 otherwise)
  float* dlogp;
  float* part;               // [kGrpoParts][part_stride] (one column per block)
  int part_stride;
  int n_traj, G;
  float g_eps_lo, g_eps_hi, beta, adv_eps;
};

// One wave per token: the target logit, the merge of the per-chunk (max,
// sum) pairs into logsumexp, and the epilogue (logp, ratio, clip).  An id
// outside [-1, V) is never used as an index: the token is treated as one
// without loss and counted in *bad_targets.  GRPO: the wave finds the
// token's trajectory, lane 0 evaluates the token's loss terms and its
// gradient (already divided by the number of loss tokens), and the block's
// four tokens are summed in wave order into one column of per-block
// partials.
// HELD: partials a lane holds, as many as there are up to 32 (as 24 for every
// size, the pass took 1 us more on 256 tokens x 512 x 8000, 2 us on 250000).
template <bool GRPO, int HELD>
__global__ __launch_bounds__(256) void lm_combine_kernel(LmArgs a, CombineOut o) {
  __shared__ float red[4][kGrpoParts];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int t = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + wave);   // wave-uniform
  float v[kGrpoParts] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (t < a.T) {
    // GRPO: the token's inputs and trajectory first, so that their loads
    // land while the merge below runs
    bool on = false;
    float old_t = 0.f, ref_t = 0.f, adv_t = 0.f;
    if (GRPO) {
      on = o.mask == nullptr || o.mask[t] != 0;
      old_t = o.logp_old[t];
      if (o.logp_ref != nullptr) ref_t = o.logp_ref[t];
      adv_t = o.adv[grpo_traj_of_wave(o.traj_ptr, o.n_traj, t, lane)];
    }
    const int y = a.tgt[t];
    const bool scored = uint32_t(y) < uint32_t(a.V);
    float tl = 0.f;
    if (scored)
      tl = target_dot(a, t, y, lane);
    else if (lane == 0 && y != -1)
      atomicAdd(a.bad_targets, 1);
    const float2* p = a.part + size_t(t) * a.n_chunks;
    // The lane's first partials are read once and held until the wave's
    // maximum is known, so that no sum is rescaled (a running maximum, with a
    // rescaled sum every eight partials, cost two roundings in the last place
    // more); vocabularies past 64 * 32 chunks (262144) read the rest twice.
    constexpr int kMerge = 8;
    const int n = a.n_chunks;
    float2 x[HELD];
    float m = -INFINITY;
#pragma unroll
    for (int u0 = 0; u0 < HELD; u0 += kMerge) {
#pragma unroll
      for (int u = u0; u < u0 + kMerge; ++u) x[u] = make_float2(-INFINITY, 0.f);
      if (64 * u0 < n) {   // wave-uniform
#pragma unroll
        for (int u = u0; u < u0 + kMerge; ++u) {
          const int i = lane + 64 * u;
          const float2 v = p[min(i, n - 1)];
          x[u] = i < n ? v : x[u];
        }
      }
    }
#pragma unroll
    for (int u = 0; u < HELD; ++u) m = fmaxf(m, x[u].x);
    for (int i = lane + 64 * HELD; i < n; i += 64) m = fmaxf(m, p[i].x);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    float s = 0.f;
#pragma unroll
    for (int u = 0; u < HELD; ++u)
      if (64 * u < n) s += x[u].y * fast_exp2(x[u].x - m);   // no partial: + 0
    for (int i = lane + 64 * HELD; i < n; i += 64) s += p[i].y * fast_exp2(p[i].x - m);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if (lane == 0) {
      const float l = (m + __log2f(s)) * kLn2;
      o.lse[t] = l;
      const float lp = scored ? tl - l : 0.f;
      o.logp[t] = lp;
      if (o.logp_old != nullptr) {
        const float r = scored ? expf(lp - o.logp_old[t]) : 1.f;
        o.ratio[t] = r;
        o.clipped[t] = fminf(fmaxf(r, 1.f - o.eps_lo), 1.f + o.eps_hi);
      }
      if (GRPO) {
        float g = 0.f;
        if (on) {
          g = grpo_token_terms(lp, old_t, o.logp_ref != nullptr ? &ref_t : nullptr, adv_t,
                               o.g_eps_lo, o.g_eps_hi, o.beta, v);
          const float n = o.n_loss_fixed >= 0 ? float(o.n_loss_fixed) : float(*o.n_loss_count);
          g = g / n;   // n >= 1: this token is a loss token
        }
        o.dlogp[t] = g;
      }
    }
  }
  if (GRPO) {
    if (lane == 0)
#pragma unroll
      for (int k = 0; k < kGrpoParts; ++k) red[wave][k] = v[k];
    __syncthreads();
    if (threadIdx.x < kGrpoParts) {   // partials stored counter-major: [k][block]
      const int k = threadIdx.x;
      o.part[size_t(k) * o.part_stride + blockIdx.x] =
          ((red[0][k] + red[1][k]) + red[2][k]) + red[3][k];
    }
  }
}

// Merge one leaf's per-chunk teacher and student partials into both LSEs and
// KL(p || q) = sum_v p_v (zT_v - zS_v) - lseT + lseS.
__global__ __launch_bounds__(256) void kl_combine_kernel(LmArgs a, float* kl, float* lseT,
                                                         float* lseS) {
  const int leaf = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (leaf >= a.n_leaves) return;
  const float4* pt = a.partT + size_t(leaf) * a.n_chunks;
  const float2* ps = a.partS + size_t(leaf) * a.n_chunks;
  float mt = -INFINITY, ms = -INFINITY;
  for (int i = lane; i < a.n_chunks; i += 64) {
    mt = fmaxf(mt, pt[i].x);
    ms = fmaxf(ms, ps[i].x);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    mt = fmaxf(mt, __shfl_xor(mt, off));
    ms = fmaxf(ms, __shfl_xor(ms, off));
  }
  float st = 0.f, cr = 0.f, ss = 0.f;
  for (int i = lane; i < a.n_chunks; i += 64) {
    const float wt = fast_exp2(pt[i].x - mt);
    st += pt[i].y * wt;
    cr += pt[i].z * wt;
    ss += ps[i].y * fast_exp2(ps[i].x - ms);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    st += __shfl_xor(st, off);
    cr += __shfl_xor(cr, off);
    ss += __shfl_xor(ss, off);
  }
  if (lane != 0) return;
  const float l2t = __log2f(st), l2s = __log2f(ss);
  lseT[leaf] = (mt + l2t) * kLn2;
  lseS[leaf] = (ms + l2s) * kLn2;
  // lseS - lseT from the differences of its parts: no cancellation between
  // two terms of size log V, and exactly zero when both sides agree
  kl[leaf] = cr / st + ((ms - mt) + (l2s - l2t)) * kLn2;
}

size_t kl_fwd_ws_bytes(int n, int H, int V) {
  const size_t np = std::max(size_t(n) * n_chunks_of(2 * n, V), kHalfPartials / 2);
  return align256(np * sizeof(float4)) + align256(np * sizeof(float2)) +
         align256(size_t(H) * sizeof(u16)) + 256;
}

// G [n, Vp] | dH partials | zero row [H] | W^T [H, Vp] unless direct (G and W^T in panels)
size_t kl_bwd_ws_bytes(int n, int H, int V) {
  return g_and_part_bytes(n, H, V) + align256(size_t(H) * sizeof(u16)) + wT_bytes(n, H, V) + 256;
}

__global__ __launch_bounds__(256) void zero_u16_kernel(u16* p, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0;
}

static hipError_t zero_row(u16* p, int H, hipStream_t stream) {
  hipLaunchKernelGGL(zero_u16_kernel, dim3((H + 255) / 256), dim3(256), 0, stream, p, H);
  return hipGetLastError();
}

// Both log-prob workspaces start (at their first 256-byte aligned address)
// with a 256-byte status block: word 0 counts the target ids outside
// [-1, V) the last call met, word 1 the loss tokens of a fused GRPO forward.
// The call's own buffers follow it.
constexpr size_t kStatusBytes = 256;

// status | per-(token, chunk) (max, sum)
size_t logprob_fwd_ws_bytes(int T, int H, int V) {
  (void)H;
  // (at least what any 128-row tiling takes: a workspace sized for some tokens
  // serves any fewer)
  return kStatusBytes +
         align256(std::max(size_t(T) * n_chunks_of(T, V), kHalfPartials) * sizeof(float2)) + 256;
}

// the forward's workspace | GRPO per-block partials (4 tokens a block) |
// advantages
static int combine_blocks(int T) { return (T + 3) / 4; }
// row stride of the counter-major partials (16-byte rows for the finish)
static int part_stride(int T) { return (combine_blocks(T) + 3) / 4 * 4; }
size_t logprob_grpo_ws_bytes(int T, int H, int V, int n_traj) {
  return logprob_fwd_ws_bytes(T, H, V) +
         align256(size_t(part_stride(T)) * kGrpoParts * sizeof(float)) +
         align256(size_t(n_traj) * sizeof(float));
}

// status | G [T up to a multiple of 256, Vp] | dH partials | W^T [H, Vp] unless direct (G and W^T in panels)
size_t logprob_bwd_ws_bytes(int T, int H, int V) {
  return kStatusBytes + g_and_part_bytes(T, H, V) + wT_bytes(T, H, V) + 256;
}

static char* align_ptr(void* p) {
  return reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(p) + 255) & ~uintptr_t(255));
}

__global__ __launch_bounds__(64) void clear_status_kernel(int* status) {
  status[threadIdx.x] = 0;   // the whole 256-byte block
}

int* logprob_status_word(const void* ws) {
  return reinterpret_cast<int*>(align_ptr(const_cast<void*>(ws)));
}

static dim3 gemm_grid(const LmArgs& a) {
  const int splits = a.k_split > 1 ? a.k_split : 1;
  const int per_xcd = (a.nA * a.nT * splits + kNumXcd - 1) / kNumXcd;
  return dim3(per_xcd * kNumXcd);
}

template <int MODE>
static void launch_tile(const LmArgs& a, hipStream_t stream) {
  if (half_tiles(a.T, a.V))
    hipLaunchKernelGGL((lm_tile_kernel<MODE, 128>), gemm_grid(a), dim3(NWAVES * 64), 0, stream, a);
  else
    hipLaunchKernelGGL((lm_tile_kernel<MODE, 256>), gemm_grid(a), dim3(NWAVES * 64), 0, stream, a);
}

static hipError_t transpose_w(const u16* w, u16* wT, int V, int H, const char* name,
                              hipStream_t stream) {
  ProfScope p(name, stream);
  hipLaunchKernelGGL(transpose_w_kernel, dim3(vocab_pad(V) / 64, H / 64), dim3(256), 0, stream, w,
                     wT, V, H, vocab_pad(V));
  return hipGetLastError();
}

// dH[t][h] = sum over splits of the fp32 partials, in split order (the
// result does not depend on scheduling), rounded once to bf16.
__global__ __launch_bounds__(256) void dh_reduce_kernel(const float* part, u16* dh, int splits,
                                                        size_t n4) {
  const size_t i = size_t(blockIdx.x) * 256 + threadIdx.x;
  if (i >= n4) return;
  const float4* p = reinterpret_cast<const float4*>(part) + i;
  float4 acc = p[0];
  auto add = [&](const float4& v) {
    acc.x += v.x;
    acc.y += v.y;
    acc.z += v.z;
    acc.w += v.w;
  };
  int s = 1;
  for (; s + 4 <= splits; s += 4) {   // four loads in flight
    float4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = p[size_t(s + u) * n4];
#pragma unroll
    for (int u = 0; u < 4; ++u) add(v[u]);
  }
  for (; s < splits; ++s) add(p[size_t(s) * n4]);
  uint2 w;
  w.x = pack2(acc.x, acc.y);
  w.y = pack2(acc.z, acc.w);
  reinterpret_cast<uint2*>(dh)[i] = w;
}

// dh[T, H] = G[T, Vp] W[Vp, H] (bf16 out) with b.wT = W^T [H, Vp], split over
// the vocabulary when the output alone would leave CUs idle; `part` is the
// fp32 partial area of the workspace (g_and_part_bytes).
static hipError_t launch_dh(LmArgs b, float* part, const char* name, hipStream_t stream) {
  // G is written (zero from V on) up to a multiple of the tile height, 128 or
  // 256: readers take no column past the last slice that holds one below V
  const int nk_total = (b.V + BKK - 1) / BKK;
  int splits = dh_splits(b.T, b.H, b.V);
  b.nk_split = (nk_total + splits - 1) / splits;
  splits = (nk_total + b.nk_split - 1) / b.nk_split;  // no empty split
  b.k_split = splits;
  b.dh_part = part;
  b.nA = (b.H + BA - 1) / BA;
  b.nT = (b.T + BT - 1) / BT;
  {
    ProfScope p(name, stream);
    if (dh_direct(b.T))
      hipLaunchKernelGGL(lm_tile_kernel<kModeDhW>, gemm_grid(b), dim3(NWAVES * 64), 0, stream, b);
    else
      hipLaunchKernelGGL(lm_tile_kernel<kModeDh>, gemm_grid(b), dim3(NWAVES * 64), 0, stream, b);
    if (splits > 1) {
      const size_t n4 = size_t(b.T) * b.H / 4;
      hipLaunchKernelGGL(dh_reduce_kernel, dim3(unsigned((n4 + 255) / 256)), dim3(256), 0, stream,
                         part, b.dh, splits, n4);
    }
  }
  return hipGetLastError();
}

// Preparation pass of the fused GRPO forward: the advantage of every
// trajectory (thread i < n_traj) and the loss tokens (the mask's nonzero
// entries, 1024 per block, added with one integer atomic per block: exact in
// any order).
__global__ __launch_bounds__(256) void grpo_prep_kernel(const uint8_t* mask, int T, int* count,
                                                        const float* reward, int n_traj, int G,
                                                        float adv_eps, float* adv) {
  __shared__ int wsum[4];
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n_traj) adv[i] = grpo_advantage(reward, G, i, adv_eps);
  if (mask == nullptr) return;   // block-uniform
  const int i0 = i * 4;
  int c = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) c += (i0 + k < T && mask[i0 + k] != 0) ? 1 : 0;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    const int tot = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    if (tot) atomicAdd(count, tot);
  }
}

static hipError_t logprob_fwd_common(LmArgs& a, void* ws, const CombineOut& o, bool grpo,
                                     const uint8_t* grpo_mask, hipStream_t stream) {
  a.bad_targets = logprob_status_word(ws);
  a.part = reinterpret_cast<float2*>(align_ptr(ws) + kStatusBytes);
  a.nA = tiles_a(a.T, a.V);
  a.nT = (a.T + BT - 1) / BT;
  // the status block is cleared by the logits pass (by a kernel, not a
  // memset, so that the call can be captured in a graph)
  if (a.T > 0) {
    ProfScope p("lm_logits", stream);
    launch_tile<kModeLogits>(a, stream);
  } else {
    hipLaunchKernelGGL(clear_status_kernel, dim3(1), dim3(64), 0, stream, a.bad_targets);
  }
  if (grpo) {
    const int blocks = std::max((a.T + 1023) / 1024, (o.n_traj + 255) / 256);
    ProfScope p("grpo_prep", stream);
    hipLaunchKernelGGL(grpo_prep_kernel, dim3(unsigned(blocks)), dim3(256), 0, stream, grpo_mask,
                       a.T, a.bad_targets + 1, o.reward, o.n_traj, o.G, o.adv_eps,
                       const_cast<float*>(o.adv));
  }
  if (a.T == 0) return hipGetLastError();
  {
    ProfScope p("lm_combine", stream);
    auto combine = [&](auto grpo_tag) {
      constexpr bool GRPO = decltype(grpo_tag)::value;
      auto* kernel = a.n_chunks <= 64 * 8    ? lm_combine_kernel<GRPO, 8>
                     : a.n_chunks <= 64 * 24 ? lm_combine_kernel<GRPO, 24>
                                             : lm_combine_kernel<GRPO, 32>;
      hipLaunchKernelGGL(kernel, dim3(combine_blocks(a.T)), dim3(256), 0, stream, a, o);
    };
    if (grpo)
      combine(std::true_type{});
    else
      combine(std::false_type{});
  }
  return hipGetLastError();
}

static LmArgs fwd_args(int T, int H, int V, const void* hidden, const void* weight,
                       const int32_t* target) {
  LmArgs a{};
  a.h = static_cast<const u16*>(hidden);
  a.w = static_cast<const u16*>(weight);
  a.tgt = target;
  a.T = T;
  a.H = H;
  a.V = V;
  a.Vp = vocab_pad(V);
  a.n_chunks = n_chunks_of(T, V);
  return a;
}

hipError_t launch_logprob_fwd(int T, int H, int V, float eps_lo, float eps_hi, const void* hidden,
                              const void* weight, const int32_t* target, const float* logp_old,
                              float* logp, float* ratio, float* clipped, float* lse, void* ws,
                              hipStream_t stream) {
  LmArgs a = fwd_args(T, H, V, hidden, weight, target);
  CombineOut o{};
  o.logp_old = logp_old;
  o.logp = logp;
  o.ratio = ratio;
  o.clipped = clipped;
  o.lse = lse;
  o.eps_lo = eps_lo;
  o.eps_hi = eps_hi;
  return logprob_fwd_common(a, ws, o, false, nullptr, stream);
}

// The forward with the GRPO loss fused into its combine pass: the logits GEMM
// (which clears the status block, so it comes first), the advantages and the
// count of the loss tokens (mask given; a word of that block), the combine with
// the per-token loss terms and gradient, one block for the statistics.
hipError_t launch_logprob_grpo(int T, int H, int V, float eps_lo, float eps_hi,
                               const void* hidden, const void* weight, const int32_t* target,
                               const float* logp_old, int n_traj, int G, float g_eps_lo,
                               float g_eps_hi, float beta, float adv_eps, const int32_t* traj_ptr,
                               const float* reward, const float* logp_ref, const uint8_t* mask,
                               float* logp, float* ratio, float* clipped, float* lse,
                               float* adv_out, float* dlogp, float* stats, void* ws,
                               hipStream_t stream) {
  LmArgs a = fwd_args(T, H, V, hidden, weight, target);
  CombineOut o{};
  o.logp_old = logp_old;
  o.logp = logp;
  o.ratio = ratio;
  o.clipped = clipped;
  o.lse = lse;
  o.eps_lo = eps_lo;
  o.eps_hi = eps_hi;
  o.traj_ptr = traj_ptr;
  o.reward = reward;
  o.logp_ref = logp_ref;
  o.mask = mask;
  o.n_loss_count = reinterpret_cast<const int*>(align_ptr(ws)) + 1;
  o.n_loss_fixed = mask == nullptr ? T : -1;
  o.dlogp = dlogp;
  o.part = reinterpret_cast<float*>(align_ptr(ws) + kStatusBytes +
                                    align256(size_t(T) * a.n_chunks * sizeof(float2)));
  o.part_stride = part_stride(T);
  o.adv = adv_out != nullptr
              ? adv_out
              : reinterpret_cast<float*>(reinterpret_cast<char*>(o.part) +
                                         align256(size_t(part_stride(T)) * kGrpoParts *
                                                  sizeof(float)));
  o.n_traj = n_traj;
  o.G = G;
  o.g_eps_lo = g_eps_lo;
  o.g_eps_hi = g_eps_hi;
  o.beta = logp_ref != nullptr ? beta : 0.f;
  o.adv_eps = adv_eps;
  if (hipError_t e = logprob_fwd_common(a, ws, o, true, mask, stream); e != hipSuccess) return e;
  ProfScope p("grpo_finish", stream);
  return launch_grpo_fused_finish(o.part, combine_blocks(T), o.part_stride, n_traj, o.adv, stats,
                                  stream);
}

hipError_t launch_logprob_bwd(int T, int H, int V, const void* hidden, const void* weight,
                              const int32_t* target, const float* lse, const float* dlogp,
                              void* dhidden, void* ws, hipStream_t stream) {
  LmArgs a{};
  a.h = static_cast<const u16*>(hidden);
  a.w = static_cast<const u16*>(weight);
  a.tgt = target;
  a.lse = lse;
  a.g = dlogp;
  a.T = T;
  a.H = H;
  a.V = V;
  a.Vp = vocab_pad(V);
  a.bad_targets = logprob_status_word(ws);   // cleared by the G pass
  char* base = align_ptr(ws) + kStatusBytes;
  u16* G = reinterpret_cast<u16*>(base);
  float* part = reinterpret_cast<float*>(base + g_bytes(T, V));
  u16* wT = reinterpret_cast<u16*>(base + g_and_part_bytes(T, H, V));
  a.Gout = G;
  a.G = G;
  a.wT = wT;
  a.dh = static_cast<u16*>(dhidden);
  a.nA = tiles_a(a.T, a.V);
  a.nT = (T + BT - 1) / BT;
  if (!dh_direct(T))
    if (hipError_t e = transpose_w(a.w, wT, V, H, "lm_wt", stream); e != hipSuccess) return e;
  {
    ProfScope p("lm_grad", stream);
    launch_tile<kModeGrad>(a, stream);
  }
  {
    ProfScope p("lm_target", stream);
    hipLaunchKernelGGL(lm_target_kernel, dim3((T + 3) / 4), dim3(256), 0, stream, a);
  }
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  return launch_dh(a, part, "lm_dh", stream);
}

// dW = G^T H from the G that launch_logprob_bwd left in its workspace.
hipError_t launch_logprob_dweight(int T, int H, int V, const void* hidden, const void* ws,
                                  float* dw, hipStream_t stream) {
  LmArgs a{};
  a.h = static_cast<const u16*>(hidden);
  a.G = reinterpret_cast<const u16*>(align_ptr(const_cast<void*>(ws)) + kStatusBytes);
  a.dw = dw;
  a.T = T;
  a.H = H;
  a.V = V;
  a.Vp = vocab_pad(V);
  a.nA = a.Vp / BA;
  a.nT = (H + BT - 1) / BT;
  ProfScope p("lm_dw", stream);
  hipLaunchKernelGGL(lm_dw_kernel, gemm_grid(a), dim3(NWAVES * 64), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_kl_fwd(int n, int H, int V, const void* hT, int nT, const int32_t* rowsT,
                         const void* hS, int nS, const int32_t* rowsS, const void* weight,
                         float* kl, float* lseT, float* lseS, void* ws, hipStream_t stream) {
  LmArgs a{};
  a.n_rows_T = nT;
  a.n_rows_S = nS;
  a.w = static_cast<const u16*>(weight);
  a.hT = static_cast<const u16*>(hT);
  a.hS = static_cast<const u16*>(hS);
  a.rowsT = rowsT;
  a.rowsS = rowsS;
  a.n_leaves = n;
  a.T = 2 * n;
  a.H = H;
  a.V = V;
  a.Vp = vocab_pad(V);
  a.n_chunks = n_chunks_of(a.T, V);
  char* base = align_ptr(ws);
  a.partT = reinterpret_cast<float4*>(base);
  a.partS = reinterpret_cast<float2*>(base + align256(size_t(n) * a.n_chunks * sizeof(float4)));
  u16* zrow = reinterpret_cast<u16*>(base + align256(size_t(n) * a.n_chunks * sizeof(float4)) +
                                     align256(size_t(n) * a.n_chunks * sizeof(float2)));
  a.zero_row = zrow;
  if (hipError_t e = zero_row(zrow, H, stream); e != hipSuccess) return e;
  a.nA = tiles_a(a.T, a.V);
  a.nT = (a.T + BT - 1) / BT;
  {
    ProfScope p("kl_logits", stream);
    launch_tile<kModeKL>(a, stream);
  }
  {
    ProfScope p("kl_combine", stream);
    hipLaunchKernelGGL(kl_combine_kernel, dim3((n + 3) / 4), dim3(256), 0, stream, a, kl, lseT,
                       lseS);
  }
  return hipGetLastError();
}

hipError_t launch_kl_bwd(int n, int H, int V, const void* hT, int nT, const int32_t* rowsT,
                         const void* hS, int nS, const int32_t* rowsS, const void* weight,
                         const float* lseT, const float* lseS, const float* dkl, void* dh,
                         void* ws, hipStream_t stream) {
  LmArgs a{};
  a.n_rows_T = nT;
  a.n_rows_S = nS;
  a.w = static_cast<const u16*>(weight);
  a.hT = static_cast<const u16*>(hT);
  a.hS = static_cast<const u16*>(hS);
  a.rowsT = rowsT;
  a.rowsS = rowsS;
  a.lseT = lseT;
  a.lseS = lseS;
  a.dkl = dkl;
  a.n_leaves = n;
  a.T = 2 * n;
  a.H = H;
  a.V = V;
  a.Vp = vocab_pad(V);
  char* base = align_ptr(ws);
  u16* G = reinterpret_cast<u16*>(base);
  float* part = reinterpret_cast<float*>(base + g_bytes(n, V));
  u16* zrow = reinterpret_cast<u16*>(base + g_and_part_bytes(n, H, V));
  u16* wT = reinterpret_cast<u16*>(reinterpret_cast<char*>(zrow) + align256(size_t(H) * sizeof(u16)));
  a.Gout = G;
  a.nA = tiles_a(a.T, a.V);
  a.nT = (a.T + BT - 1) / BT;
  a.zero_row = zrow;
  if (hipError_t e = zero_row(zrow, H, stream); e != hipSuccess) return e;
  if (!dh_direct(n))
    if (hipError_t e = transpose_w(a.w, wT, V, H, "kl_wt", stream); e != hipSuccess) return e;
  {
    ProfScope p("kl_grad", stream);
    launch_tile<kModeKLGrad>(a, stream);
  }
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  // dh = G W over the leaves
  LmArgs b{};
  b.w = a.w;
  b.wT = wT;
  b.G = G;
  b.dh = static_cast<u16*>(dh);
  b.T = n;
  b.H = H;
  b.V = V;
  b.Vp = a.Vp;
  return launch_dh(b, part, "kl_dh", stream);
}

}  // namespace mv
