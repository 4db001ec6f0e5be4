// Decode of the deterministic actor's outputs into the inputs of
// select/pack, on the device, with no host synchronisation.
// DORA (arXiv 2609.34325): Sec. 3.2 "Gate", "Budget head and selector" and
// "Sampling and deployment"; App. A.2 (budget grid {2, 4, ..., N0 - 4} with
// M = (N0 - 4) / 2 outputs; legal budgets leave at least four visual tokens);
// App. A.3 (deployment: gate at probability >= 0.5 when a budget is legal,
// the legal budget with the largest logit, the k highest removal scores go).
//
//   actor_gate_kernel    one workgroup: gate decision per image and the
//                        ordered compaction of the gate-on images (ballot +
//                        mbcnt within a wave, wave counts through LDS), so
//                        the controller can run on gate-on images only.
//   actor_decode_kernel  one wave per image: argmax over the legal budget
//                        logits (the first maximum; NaN above every number),
//                        keep = tokens - budget; all threads also negate the
//                        selector's removal scores into keep-scores.
#include "dora_internal.h"

namespace dora {
namespace {

constexpr int kGateThreads = 1024;
constexpr int kDecodeThreads = 256;
constexpr int kDecodeWaves = kDecodeThreads / 64;
constexpr int32_t kActorMaxB = 1 << 24;  // images per call (keeps every index in int32)

// Legal budgets 2(m+1), m < M, with 2(m+1) <= (n_tok - 1) - 4: their count.
__device__ __forceinline__ int legal_budgets(int n_tok, int M) {
  const int c = n_tok >= 5 ? (n_tok - 5) >> 1 : 0;
  return c < M ? c : M;
}

// Token count of image b (CLS included); 0 when its segment is invalid.
__device__ __forceinline__ int image_tokens(const int32_t* cu_in, int b, int N) {
  if (!cu_in) return N;
  const int lo = cu_in[b], hi = cu_in[b + 1];
  const int n = hi - lo;
  return (lo >= 0 && n >= 1 && n <= N) ? n : 0;
}

struct GateParams {
  const float* p_gate;
  const int32_t* cu_in;
  int32_t B, N, M;
  int32_t* on_rank;
  int32_t* on_list;
  int32_t* n_on;
  int32_t* status;
};

__global__ __launch_bounds__(kGateThreads) void actor_gate_kernel(GateParams p) {
  __shared__ int s_count[kGateThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int ranked = 0;  // gate-on images before the current chunk
  bool bad = false;
  for (int base = 0; base < p.B; base += kGateThreads) {
    const int b = base + tid;
    bool open = false;
    if (b < p.B) {
      const int n = image_tokens(p.cu_in, b, p.N);
      bad |= n == 0;
      open = n > 0 && p.p_gate[b] >= 0.5f && legal_budgets(n, p.M) > 0;
    }
    const uint64_t mask = __ballot(open);
    if (lane == 0) s_count[wave] = __popcll(mask);
    __syncthreads();
    int before = 0, chunk = 0;
#pragma unroll
    for (int w = 0; w < kGateThreads / 64; ++w) {
      const int c = s_count[w];
      before += w < wave ? c : 0;
      chunk += c;
    }
    if (b < p.B) {
      const int r = ranked + before + lanes_below(mask);
      p.on_rank[b] = open ? r : -1;
      if (open) p.on_list[r] = b;
    }
    ranked += chunk;
    __syncthreads();  // s_count is rewritten by the next chunk
  }
  for (int i = ranked + tid; i < p.B; i += kGateThreads) p.on_list[i] = -1;
  if (tid == 0) *p.n_on = ranked;
  if (bad) atomicOr(p.status, DORA_DEV_CU_IN);
}

struct DecodeParams {
  const float* logits;
  int64_t rows;
  int32_t M;
  const float* removal;
  float* keep_scores;
  int64_t n_scores;
  const int32_t* cu_in;
  int32_t B, N;
  const int32_t* on_rank;
  int32_t* keep;
  int32_t* status;
};

// Argmax word of logit x at index m: larger for larger x (NaN above every
// number, -0 equal to +0), and among equal values larger for the lower index.
__device__ __forceinline__ unsigned long long argmax_word(float x, int m) {
  uint32_t u = __float_as_uint(x == 0.0f ? 0.0f : x);
  u = x != x ? 0xFFFFFFFFu : (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return (static_cast<unsigned long long>(u) << 32) | ~static_cast<uint32_t>(m);
}

// Largest word of the wave: register exchanges (DPP inside 16-lane rows, then
// the row swaps), no trip through the LDS crossbar.
__device__ __forceinline__ unsigned long long wave_max_word(unsigned long long v) {
  auto larger = [](unsigned long long a, uint32_t hi, uint32_t lo) {
    const unsigned long long b = (static_cast<unsigned long long>(hi) << 32) | lo;
    return a > b ? a : b;
  };
  auto hi = [](unsigned long long x) { return static_cast<uint32_t>(x >> 32); };
  auto lo = [](unsigned long long x) { return static_cast<uint32_t>(x); };
  v = larger(v, __builtin_amdgcn_update_dpp(0u, hi(v), 0xB1, 0xF, 0xF, false),   // quad_perm 1,0,3,2
             __builtin_amdgcn_update_dpp(0u, lo(v), 0xB1, 0xF, 0xF, false));
  v = larger(v, __builtin_amdgcn_update_dpp(0u, hi(v), 0x4E, 0xF, 0xF, false),   // quad_perm 2,3,0,1
             __builtin_amdgcn_update_dpp(0u, lo(v), 0x4E, 0xF, 0xF, false));
  v = larger(v, __builtin_amdgcn_update_dpp(0u, hi(v), 0x141, 0xF, 0xF, false),  // row_half_mirror
             __builtin_amdgcn_update_dpp(0u, lo(v), 0x141, 0xF, 0xF, false));
  v = larger(v, __builtin_amdgcn_update_dpp(0u, hi(v), 0x140, 0xF, 0xF, false),  // row_mirror
             __builtin_amdgcn_update_dpp(0u, lo(v), 0x140, 0xF, 0xF, false));
  {
    const auto h = __builtin_amdgcn_permlane16_swap(hi(v), hi(v), false, false);
    const auto l = __builtin_amdgcn_permlane16_swap(lo(v), lo(v), false, false);
    v = larger((static_cast<unsigned long long>(h[0]) << 32) | l[0], h[1], l[1]);
  }
  {
    const auto h = __builtin_amdgcn_permlane32_swap(hi(v), hi(v), false, false);
    const auto l = __builtin_amdgcn_permlane32_swap(lo(v), lo(v), false, false);
    v = larger((static_cast<unsigned long long>(h[0]) << 32) | l[0], h[1], l[1]);
  }
  return v;
}

__global__ __launch_bounds__(kDecodeThreads) void actor_decode_kernel(DecodeParams p) {
  const int lane = threadIdx.x & 63;
  const int b = blockIdx.x * kDecodeWaves + (threadIdx.x >> 6);
  // This thread's first removal score, in flight while the image's wave
  // follows its own chain of loads.
  const int64_t i0 = static_cast<int64_t>(blockIdx.x) * kDecodeThreads + threadIdx.x;
  const bool negates = p.removal != nullptr && i0 < p.n_scores;
  float first = 0.0f;
  if (negates) first = p.removal[i0];
  asm volatile("" : "+v"(first));
  if (b < p.B) {
    const int n = image_tokens(p.cu_in, b, p.N);
    const int r = p.on_rank[b];
    int keep = n, flag = 0;
    if (n == 0) {
      flag = DORA_DEV_CU_IN;
    } else if (r >= 0) {
      const int legal = legal_budgets(n, p.M);
      if (legal == 0 || r >= p.rows) {
        flag = DORA_DEV_ACTOR;  // left unpruned
      } else {
        const float* row = p.logits + static_cast<int64_t>(r) * p.M;
        unsigned long long best = 0ull;
        for (int m = lane; m < legal; m += 64) {
          const unsigned long long w = argmax_word(row[m], m);
          best = w > best ? w : best;
        }
        const int ib = static_cast<int>(~static_cast<uint32_t>(wave_max_word(best)));
        keep = n - 2 * (ib + 1);
      }
    }
    if (lane == 0) {
      p.keep[b] = keep;
      if (flag) atomicOr(p.status, flag);
    }
  }
  if (negates) {
    p.keep_scores[i0] = -first;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kDecodeThreads;
    for (int64_t i = i0 + stride; i < p.n_scores; i += stride) p.keep_scores[i] = -p.removal[i];
  }
}

}  // namespace
}  // namespace dora

extern "C" int dora_actor_gate(const float* p_gate, const int32_t* cu_in, int32_t B, int32_t N, int32_t M,
                               int32_t* on_rank, int32_t* on_list, int32_t* n_on, int32_t* dev_status,
                               void* stream) {
  using namespace dora;
  if (!p_gate || !on_rank || !on_list || !n_on || !dev_status) return DORA_ERR_NULL;
  if (B < 1 || B > kActorMaxB || N < 1 || M < 1 || N > DORA_MAX_ROW_TOKENS) return DORA_ERR_SHAPE;
  GateParams p{p_gate, cu_in, B, N, M, on_rank, on_list, n_on, dev_status};
  hipLaunchKernelGGL(actor_gate_kernel, dim3(1), dim3(kGateThreads), 0, static_cast<hipStream_t>(stream), p);
  return hipGetLastError() == hipSuccess ? DORA_OK : DORA_ERR_HIP;
}

extern "C" int dora_actor_decode(const float* budget_logits, int64_t logit_rows, int32_t M,
                                 const float* removal_scores, const int32_t* cu_in, int64_t total_in, int32_t B,
                                 int32_t N, const int32_t* on_rank, int32_t* keep_out, float* scores_out,
                                 int32_t* dev_status, void* stream) {
  using namespace dora;
  if (!on_rank || !keep_out || !dev_status) return DORA_ERR_NULL;
  if ((removal_scores == nullptr) != (scores_out == nullptr)) return DORA_ERR_NULL;
  if (!budget_logits && logit_rows > 0) return DORA_ERR_NULL;
  if (B < 1 || B > kActorMaxB || N < 1 || M < 1 || N > DORA_MAX_ROW_TOKENS || logit_rows < 0 ||
      logit_rows > 0x7FFFFFFF)
    return DORA_ERR_SHAPE;
  const int64_t n_scores = cu_in ? total_in : static_cast<int64_t>(B) * N;
  if (n_scores < 0) return DORA_ERR_SHAPE;
  DecodeParams p{budget_logits, logit_rows, M, removal_scores, scores_out, n_scores, cu_in, B, N,
                 on_rank, keep_out, dev_status};
  // One wave per image; the score negation strides over whatever grid that
  // gives, widened to a score per thread (at most 2048 workgroups).  197
  // tokens, before (four scores per thread after the argmax, shuffles through
  // LDS) -> now: 64 images 3.2 -> 2.3 us, 2048 images 3.6 -> 2.7.
  const int64_t for_images = (static_cast<int64_t>(B) + kDecodeWaves - 1) / kDecodeWaves;
  int64_t for_scores = removal_scores ? (n_scores + kDecodeThreads - 1) / kDecodeThreads : 0;
  if (for_scores > 2048) for_scores = 2048;
  const int64_t grid = for_images > for_scores ? for_images : for_scores;
  hipLaunchKernelGGL(actor_decode_kernel, dim3(static_cast<unsigned>(grid)), dim3(kDecodeThreads), 0,
                     static_cast<hipStream_t>(stream), p);
  return hipGetLastError() == hipSuccess ? DORA_OK : DORA_ERR_HIP;
}
