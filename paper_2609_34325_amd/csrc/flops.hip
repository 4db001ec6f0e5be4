// FLOP accounting of realised token trajectories.
// DORA (arXiv 2609.34325), App. E.4: two FLOPs per multiply-accumulate over
// the complete forward (patch embedding, backbone, classifier and the actor),
// following each image's own token trajectory: at block l the attention runs
// over the N_l + 1 tokens that enter it and the MLP over the N_l - k_l + 1 it
// keeps.  Actor shapes from App. A.1: gate (d + 16 + 3) -> 64 -> 1 on the CLS
// key at every block with a legal budget; where tokens were removed the
// controller ran: input projection d -> 128 of every key and 3 -> 128 of the
// history, one width-128 Transformer block (4 heads, FFN 128 -> 256 -> 128),
// budget head 128 -> 128 -> M, the 1 -> 128 projection of k / N, selector
// 128 -> 64 -> 1 on the visual tokens.
//
// One thread per image, walking its L blocks in exact int64 arithmetic.  The
// token counts of a block do not depend on the block before, so a thread loads
// kAhead of them at once (one memory round trip per kAhead blocks instead of
// one per block).  Up to kOneGroupB images one workgroup does it all and writes
// the total; it is bound by latency at few images and by the 64-bit multiplies
// of one compute unit at many.  Past that the images spread over workgroups,
// which add their sums to a total cleared by the launch before (integer
// additions: the result does not depend on their order).  12 blocks, before
// -> now: 64 images 4.0 -> 3.5 us, 2048 images 9.2 -> 5.5, 50,000 images
// 176 -> 7.4, 1,000,000 images 4870 -> 27.5.
#include <algorithm>

#include "dora_internal.h"

namespace dora {
namespace {

constexpr int kFlopThreads = 1024;      // one workgroup
constexpr int kFlopWideThreads = 256;   // several workgroups
constexpr int kFlopMaxGroups = 1024;    // atomics on the total
// The second launch costs about as much as 700 images on one compute unit:
// at 1000 images one workgroup takes 5.7 us, at 1500 6.9 against 5.4 spread.
constexpr int kOneGroupB = 1024;
constexpr int kAhead = 8;
constexpr int64_t kActW = 128, kActFfn = 256, kGateHidden = 64, kGateEmbed = 16, kHist = 3, kSelHidden = 64;

__device__ __forceinline__ int64_t block_attn_macs(int64_t n, int64_t d) {
  return n * d * 3 * d + 2 * n * n * d + n * d * d;
}

struct FlopParams {
  const int32_t* tokens;  // [L+1][B]
  int32_t B;
  dora_flops_config c;
  int64_t* flops;
  int64_t* total;
  int32_t* status;
};

__global__ void clear_total_kernel(int64_t* total) { *total = 0; }

template <int THREADS, bool WIDE>
__global__ __launch_bounds__(THREADS) void trajectory_flops_kernel(FlopParams p) {
  __shared__ long long s_red[THREADS / 64];
  const int64_t d = p.c.d;
  const int64_t fixed = static_cast<int64_t>(p.c.N0) * p.c.in_chans * p.c.patch * p.c.patch * d +
                        static_cast<int64_t>(p.c.head_inputs) * d * p.c.classes;
  const int64_t mlp_tok = 2 * d * (static_cast<int64_t>(p.c.mlp_ratio) * d);
  const int64_t gate = (d + kGateEmbed + kHist) * kGateHidden + kGateHidden;
  long long sum = 0;
  bool bad = false;
  const int stride = WIDE ? static_cast<int>(gridDim.x) * THREADS : THREADS;
  for (int b = (WIDE ? static_cast<int>(blockIdx.x) * THREADS : 0) + threadIdx.x; b < p.B; b += stride) {
    int64_t macs = fixed;
    int64_t n = p.tokens[b];
    bool ok = n == p.c.N0 + 1;
    for (int l0 = 0; l0 < p.c.L; l0 += kAhead) {
      // Blocks past the last re-read its count (in bounds) and are not used.
      int32_t next[kAhead];
#pragma unroll
      for (int i = 0; i < kAhead; ++i) next[i] = p.tokens[static_cast<int64_t>(min(l0 + i, p.c.L - 1) + 1) * p.B + b];
#pragma unroll
      for (int i = 0; i < kAhead; ++i) asm volatile("" : "+v"(next[i]));  // all loads before the first use
#pragma unroll
      for (int i = 0; i < kAhead; ++i) {
        if (l0 + i >= p.c.L) break;
        const int64_t m = next[i];
        ok = ok && m >= 1 && m <= n;
        macs += block_attn_macs(n, d) + m * mlp_tok;
        if (p.c.actor) {
          if (n - 1 >= 6) macs += gate;
          if (m < n) {
            macs += n * d * kActW + kHist * kActW;                                    // input projections
            macs += block_attn_macs(n, kActW) + n * 2 * kActW * kActFfn;              // encoder block
            macs += kActW * kActW + kActW * static_cast<int64_t>(p.c.M);              // budget head
            macs += kActW + (n - 1) * (kActW * kSelHidden + kSelHidden);              // k / N projection, selector
          }
        }
        n = m;
      }
    }
    p.flops[b] = ok ? 2 * macs : -1;
    if (ok) sum += 2 * macs;
    bad |= !ok;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
  if (lane == 0) s_red[wave] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    long long t = 0;
    for (int w = 0; w < THREADS / 64; ++w) t += s_red[w];
    if (WIDE) atomicAdd(reinterpret_cast<unsigned long long*>(p.total), static_cast<unsigned long long>(t));
    else *p.total = t;
  }
  if (bad) atomicOr(p.status, DORA_DEV_KEEP_RANGE);
}

}  // namespace
}  // namespace dora

extern "C" int dora_trajectory_flops(const int32_t* tokens, int32_t B, const dora_flops_config* config,
                                     int64_t* flops_out, int64_t* total_out, int32_t* dev_status, void* stream) {
  using namespace dora;
  if (!tokens || !config || !flops_out || !total_out || !dev_status) return DORA_ERR_NULL;
  const dora_flops_config& c = *config;
  if (B < 1 || B > (1 << 24) || c.d < 1 || c.d > 65536 || c.L < 1 || c.L > 1024 || c.N0 < 1 ||
      c.N0 > DORA_MAX_ROW_TOKENS || c.patch < 1 || c.patch > 64 || c.in_chans < 1 || c.in_chans > 16 ||
      c.classes < 1 || c.classes > (1 << 20) || c.head_inputs < 1 || c.head_inputs > 8 || c.mlp_ratio < 1 ||
      c.mlp_ratio > 16 || c.M < 1 || c.M > DORA_MAX_ROW_TOKENS || (c.actor != 0 && c.actor != 1))
    return DORA_ERR_SHAPE;
  FlopParams p{tokens, B, c, flops_out, total_out, dev_status};
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (B <= kOneGroupB) {
    hipLaunchKernelGGL((trajectory_flops_kernel<kFlopThreads, false>), dim3(1), dim3(kFlopThreads), 0, st, p);
  } else {
    const int groups = std::min((B + kFlopWideThreads - 1) / kFlopWideThreads, kFlopMaxGroups);
    hipLaunchKernelGGL(clear_total_kernel, dim3(1), dim3(1), 0, st, total_out);
    hipLaunchKernelGGL((trajectory_flops_kernel<kFlopWideThreads, true>), dim3(groups), dim3(kFlopWideThreads), 0, st,
                       p);
  }
  return hipGetLastError() == hipSuccess ? DORA_OK : DORA_ERR_HIP;
}
