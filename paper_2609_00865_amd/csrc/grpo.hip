// GRPO token loss, its gradient into the per-token log-probs, and the drift
// diagnostics, on the outputs of the fused LM head (the same loss also runs
// inside the LM head's combine pass: mv_token_logprob_grpo; both use the
// per-token arithmetic of mv_grpo_dev.h).
//
// Two small launches (HBM-trivial next to the LM-head GEMMs; bound by launches
// and their latency: as four, advantage / token / statistics / scale, 64 x 512
// tokens took 23.4 us a call):
//   1. per token: the trajectory by binary search of the packed offsets, its
//      group-normalised advantage (once per trajectory and block), the ratio,
//      the clipped surrogate and its gradient, the k3 reference KL and the
//      drift |logp - logp_old|; unnormalised gradient out, per-block partial
//      sums to the workspace (fixed-order tree in LDS); the advantages;
//   2. the gradient scaled by 1 / (number of loss tokens), which every block
//      sums for itself from the partials (whole numbers: exact in any order);
//      the first block sums all partials in block order (fp64) into the
//      statistics.
// The blocks of the second pass are at most kScaleBlocks, so that what they
// read of the partials grows with the tokens and not with their square.
// Every reduction has a fixed order, so results are bitwise reproducible.
#include <algorithm>

#include "mv_grpo_dev.h"

namespace mv {

namespace {
constexpr int kTok = 256;          // threads (= tokens) per block of the token pass
constexpr int kRatioPart = 6;
constexpr int kNP = kGrpoParts;
size_t al256(size_t x) { return (x + 255) & ~size_t(255); }
}  // namespace

struct GrpoArgs {
  const int32_t* traj_ptr;   // [n_traj + 1]
  const float* reward;       // [n_traj]
  const float* logp;
  const float* logp_old;
  const float* logp_ref;     // null when beta == 0
  const uint8_t* mask;       // null: every token carries loss
  float* adv;                // [n_traj]
  float* dlogp;              // [T]
  float* part;               // [kNP][n_blocks] (counter-major)
  float* stats;              // 8 floats
  int T, n_traj, G;
  float eps_lo, eps_hi, beta, adv_eps;
};

__global__ __launch_bounds__(kTok) void grpo_token_kernel(GrpoArgs a, int n_blocks) {
  __shared__ float red[kNP][kTok];
  __shared__ float adv_of[kTok];   // at a trajectory's first token in the block
  const int b0 = blockIdx.x * kTok, t = b0 + threadIdx.x;
  if (t < a.n_traj) a.adv[t] = grpo_advantage(a.reward, a.G, t, a.adv_eps);
  if (blockIdx.x >= n_blocks) return;   // a block of advantages only
  float v[kNP] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  int first = 0;
  bool on = false;
  float lp = 0.f, old = 0.f, ref = 0.f;
  if (t < a.T) {
    // the token's inputs first: they land while its trajectory is looked up
    on = a.mask == nullptr || a.mask[t] != 0;
    lp = a.logp[t];
    old = a.logp_old[t];
    if (a.logp_ref != nullptr) ref = a.logp_ref[t];
    const int tr = grpo_traj_of(a.traj_ptr, a.n_traj, t);
    first = min(max(a.traj_ptr[tr] - b0, 0), kTok - 1);
    if (first == int(threadIdx.x)) adv_of[first] = grpo_advantage(a.reward, a.G, tr, a.adv_eps);
  }
  __syncthreads();
  if (t < a.T) {
    float g = 0.f;
    if (on)
      g = grpo_token_terms(lp, old, a.logp_ref != nullptr ? &ref : nullptr, adv_of[first],
                           a.eps_lo, a.eps_hi, a.beta, v);
    a.dlogp[t] = g;
  }
#pragma unroll
  for (int k = 0; k < kNP; ++k) red[k][threadIdx.x] = v[k];
  __syncthreads();
  for (int s = kTok / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
#pragma unroll
      for (int k = 0; k < kNP; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x < kNP) a.part[size_t(threadIdx.x) * n_blocks + blockIdx.x] = red[threadIdx.x][0];
}

// One block: the per-block partials (counter-major: counter k of block b at
// part[k * stride + b]) summed in fp64, thread-strided (16-byte loads where
// the rows allow them) then a fixed tree, into the statistics.
constexpr int kFinish = 512;
__device__ __forceinline__ void grpo_finish(const GrpoArgs& a, int n_blocks, int stride,
                                            double (&red)[kNP + 1][kFinish]) {
  double v[kNP + 1] = {0, 0, 0, 0, 0, 0, 0, 0};
  const bool vec = (stride & 3) == 0 && (reinterpret_cast<uintptr_t>(a.part) & 15) == 0;
  const int n4 = vec ? n_blocks / 4 : 0;
#pragma unroll
  for (int k = 0; k < kNP; ++k) {
    const float* row = a.part + size_t(k) * stride;
    for (int b = threadIdx.x; b < n4; b += kFinish) {
      const float4 x = reinterpret_cast<const float4*>(row)[b];
      v[k] += x.x;
      v[k] += x.y;
      v[k] += x.z;
      v[k] += x.w;
    }
    for (int b = 4 * n4 + threadIdx.x; b < n_blocks; b += kFinish) v[k] += row[b];
  }
  for (int i = threadIdx.x; i < a.n_traj; i += kFinish) v[kNP] += fabs(double(a.adv[i]));
#pragma unroll
  for (int k = 0; k <= kNP; ++k) red[k][threadIdx.x] = v[k];
  __syncthreads();
  for (int s = kFinish / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
#pragma unroll
      for (int k = 0; k <= kNP; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  const double n = red[0][0];
  const double inv = n > 0 ? 1.0 / n : 0.0;
  a.stats[0] = float(red[1][0] * inv);               // loss
  a.stats[1] = float(red[2][0] * inv);               // logdiff
  a.stats[2] = float(red[3][0] * inv);               // clip fraction, low side
  a.stats[3] = float(red[4][0] * inv);               // clip fraction, high side
  a.stats[4] = float(red[5][0] * inv);               // mean k3
  a.stats[5] = float(red[kRatioPart][0] * inv);      // mean ratio
  a.stats[6] = float(n);                             // loss tokens
  a.stats[7] = a.n_traj > 0 ? float(red[kNP][0] / a.n_traj) : 0.f;  // mean |advantage|
}

__global__ __launch_bounds__(kFinish) void grpo_finish_kernel(GrpoArgs a, int n_blocks,
                                                              int stride) {
  __shared__ double red[kNP + 1][kFinish];
  grpo_finish(a, n_blocks, stride, red);
}

// The first block: the statistics; the others: the gradients, in strides of
// their number times kFinish tokens.  A block reads every token block's count
// once.  A call of 4M tokens takes 76 us, of 1M 23 (each wave reading the
// counts, a block per kFinish tokens: 313 and 47; as separate advantage, token,
// statistics and scale passes 81 and 24).
constexpr int kScaleBlocks = 512;
__global__ __launch_bounds__(kFinish) void grpo_scale_kernel(GrpoArgs a, int n_blocks) {
  __shared__ double red[kNP + 1][kFinish];
  if (blockIdx.x == 0) {
    grpo_finish(a, n_blocks, n_blocks, red);
    return;
  }
  double c = 0.0;   // loss tokens
  for (int b = threadIdx.x; b < n_blocks; b += kFinish) c += a.part[b];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
  if ((threadIdx.x & 63) == 0) red[0][threadIdx.x >> 6] = c;
  __syncthreads();
  c = 0.0;
#pragma unroll
  for (int w = 0; w < kFinish / 64; ++w) c += red[0][w];
  const float n = float(c);
  const int64_t stride = int64_t(gridDim.x - 1) * kFinish;
  for (int64_t t = int64_t(blockIdx.x - 1) * kFinish + threadIdx.x; t < a.T; t += stride)
    a.dlogp[t] = n > 0.f ? a.dlogp[t] / n : 0.f;
}

size_t grpo_ws_bytes(int T, int n_traj) {
  const size_t n_blocks = (size_t(T) + kTok - 1) / kTok;
  return al256(n_blocks * kNP * sizeof(float)) + al256(size_t(n_traj) * sizeof(float)) + 256;
}

hipError_t launch_grpo(int T, int n_traj, int G, float eps_lo, float eps_hi, float beta,
                       float adv_eps, const int32_t* traj_ptr, const float* reward,
                       const float* logp, const float* logp_old, const float* logp_ref,
                       const uint8_t* mask, float* adv_out, float* dlogp, float* stats, void* ws,
                       hipStream_t stream) {
  GrpoArgs a{};
  char* base = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(ws) + 255) & ~uintptr_t(255));
  const int n_blocks = (T + kTok - 1) / kTok;
  a.part = reinterpret_cast<float*>(base);
  a.adv = adv_out != nullptr
              ? adv_out
              : reinterpret_cast<float*>(base + al256(size_t(n_blocks) * kNP * sizeof(float)));
  a.traj_ptr = traj_ptr;
  a.reward = reward;
  a.logp = logp;
  a.logp_old = logp_old;
  a.logp_ref = logp_ref;
  a.mask = mask;
  a.dlogp = dlogp;
  a.stats = stats;
  a.T = T;
  a.n_traj = n_traj;
  a.G = G;
  a.eps_lo = eps_lo;
  a.eps_hi = eps_hi;
  a.beta = logp_ref != nullptr ? beta : 0.f;
  a.adv_eps = adv_eps;
  ProfScope prof("grpo", stream);
  // a block per kTok tokens, and as many as give every trajectory a thread
  // (256 tokens of 100000 trajectories, most of them empty, with the token
  // blocks alone: 545 us a call instead of 66)
  const int adv_blocks = (n_traj + kTok - 1) / kTok;
  hipLaunchKernelGGL(grpo_token_kernel, dim3(std::max(adv_blocks, n_blocks)), dim3(kTok), 0,
                     stream, a, n_blocks);
  const int scale_blocks = std::min((T + kFinish - 1) / kFinish, kScaleBlocks);
  hipLaunchKernelGGL(grpo_scale_kernel, dim3(1 + scale_blocks), dim3(kFinish), 0, stream, a,
                     n_blocks);
  return hipGetLastError();
}

// Statistics of the GRPO loss that the LM head's combine pass evaluated per
// token (part: its per-block partials, counter k of block b at part[k *
// stride + b]; adv: the advantages its preparation pass wrote).
hipError_t launch_grpo_fused_finish(const float* part, int n_blocks, int stride, int n_traj,
                                    const float* adv, float* stats, hipStream_t stream) {
  GrpoArgs a{};
  a.part = const_cast<float*>(part);
  a.adv = const_cast<float*>(adv);
  a.stats = stats;
  a.n_traj = n_traj;
  hipLaunchKernelGGL(grpo_finish_kernel, dim3(1), dim3(kFinish), 0, stream, a, n_blocks, stride);
  return hipGetLastError();
}

}  // namespace mv
