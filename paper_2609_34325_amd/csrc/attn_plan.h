// The attention plan from sequence boundaries, by one workgroup: shared by the
// plan kernel and by select/pack, where one workgroup of a large launch makes
// the plan while the others copy rows.
//
// Three passes: count the sequences by length (1024 bins), turn the counts
// into positions of the longest-first order and into the item bases of each
// class (sequences of equal chunk count), and give every sequence its position
// (an LDS atomic on its bin) and with it its items' slots.  Nothing but the
// bins and class tables lives in LDS (about 6 KB), so a workgroup that makes a
// plan does not crowd out copying ones.  Latency bound: a few memory round
// trips and, for many sequences, the item stores of one compute unit.
#pragma once

#include "dora_internal.h"

namespace dora {

constexpr int kPlanMaxChunks = (DORA_MAX_SEQLEN + kAttnQTile - 1) / kAttnQTile;  // chunks of the longest sequence
constexpr int kPlanBins = 1024;

struct PlanParams {
  const int32_t* cu;
  int32_t B, H, max_seqlen;
  int32_t min_len;  // shortest valid sequence (0; 1 for the plan of a select/pack output)
  int64_t total;
  AttnPlanHeader* hdr;
  int2* items;
  int32_t* status;
};

inline PlanParams make_plan_params(const int32_t* cu, int32_t B, int32_t H, int32_t max_seqlen, int64_t total,
                                   int32_t min_len, void* workspace, int32_t* dev_status) {
  PlanParams p;
  p.cu = cu;
  p.B = B;
  p.H = H;
  p.max_seqlen = max_seqlen;
  p.min_len = min_len;
  p.total = total;
  p.hdr = static_cast<AttnPlanHeader*>(workspace);
  p.items = reinterpret_cast<int2*>(static_cast<char*>(workspace) +
                                    attn_workspace_layout(B, H, max_seqlen).items_off);
  p.status = dev_status;
  return p;
}

template <int THREADS>
struct PlanLds {
  int bins[kPlanBins];               // counts, then next position of the longest-first order
  int wave_sums[THREADS / 64];
  int count[kPlanMaxChunks + 1];     // per chunk count: sequences,
  int first[kPlanMaxChunks + 1];     // first position
  int item0[kPlanMaxChunks + 1];     // and first item
  int bad;
};

// Called by every thread of a workgroup of THREADS.
template <int THREADS>
__device__ __forceinline__ void attn_plan_body(const PlanParams& p, PlanLds<THREADS>& s) {
  constexpr int kPer = kPlanBins / THREADS;  // bins per thread
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // Length bins: bin 0 for empty sequences, then (len - 1) >> shift + 1.
  // The smallest shift that fits is at most 5 (max_seqlen <= 16384), and
  // 2^shift divides kAttnQTile, so a bin never straddles a chunk boundary and
  // the sequences of equal chunk count stay contiguous in the sorted order.
  int shift = 0;
  while (((p.max_seqlen - 1) >> shift) + 1 >= kPlanBins) ++shift;
  auto bin_of = [shift](int len) { return len == 0 ? 0 : ((len - 1) >> shift) + 1; };
  const int max_ch = attn_chunks(p.max_seqlen);

  for (int i = tid; i < kPlanBins; i += THREADS) s.bins[i] = 0;
  for (int i = tid; i <= max_ch; i += THREADS) s.count[i] = 0;
  if (tid == 0) s.bad = 0;
  __syncthreads();
  // The bounds of a thread's next sequence are loaded before the current one's
  // atomic (past the last: the last again).
  int nlo = p.cu[min(tid, p.B - 1)], nhi = p.cu[min(tid, p.B - 1) + 1];
  for (int b = tid; b < p.B; b += THREADS) {
    const long long a = nlo, e = nhi, len = e - a;
    const int nb = min(b + THREADS, p.B - 1);
    nlo = p.cu[nb];
    nhi = p.cu[nb + 1];
    if (a < 0 || e > p.total || len < p.min_len || len > p.max_seqlen || (b == 0 && a != 0)) s.bad = 1;
    else atomicAdd(&s.bins[bin_of(static_cast<int>(len))], 1);
  }
  __syncthreads();
  if (s.bad) {
    if (tid == 0) {
      atomicOr(p.status, DORA_DEV_CU_SEQLENS);
      write_plan_header(p.hdr, 0, p.B, p.H, p.max_seqlen, p.total);
    }
    return;
  }

  // Positions, longest bin first: thread t holds bins kPlanBins - 1 - t kPer
  // and the kPer - 1 below it.
  int n[kPer], sum = 0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int bin = kPlanBins - 1 - (tid * kPer + i);
    n[i] = s.bins[bin];
    sum += n[i];
    const int len = bin == 0 ? 0 : ((bin - 1) << shift) + 1;  // a length of the bin
    if (n[i] > 0) atomicAdd(&s.count[attn_chunks(len)], n[i]);
  }
  int incl = sum;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int t = __shfl_up(incl, off, 64);
    if (lane >= off) incl += t;
  }
  if (lane == 63) s.wave_sums[wave] = incl;
  __syncthreads();
  int run = incl - sum;
  for (int w = 0; w < wave; ++w) run += s.wave_sums[w];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    s.bins[kPlanBins - 1 - (tid * kPer + i)] = run;
    run += n[i];
  }
  // Classes of more chunks come first.  At most 8192 x 256 x 86 items: int32.
  for (int ch = tid; ch <= max_ch; ch += THREADS) {
    int before = 0, items = 0;
    for (int c = max_ch; c > ch; --c) {
      before += s.count[c];
      items += s.count[c] * c;
    }
    s.first[ch] = before;
    s.item0[ch] = items * p.H;
    if (ch == 0) write_plan_header(p.hdr, items * p.H, p.B, p.H, p.max_seqlen, p.total);
  }
  if (tid < 32) p.hdr->zero_row[tid] = 0u;
  __syncthreads();

  // One lane per sequence where a sequence has few items; where it has more
  // than 64 (long sequences), a wave writes those of its sequences one after
  // the other, and the sequences are dealt over all waves.  One sequence of
  // 16384 tokens with 12 heads: 41 us by one lane, 9.2 by a wave; groups of 16
  // lanes for 12 items each took 143 us for 8192 sequences, a lane each 60.
  const bool together = p.H * max_ch > 64;
  const int b_first = together ? lane * (THREADS / 64) + wave : tid;
  nlo = p.cu[min(b_first, p.B - 1)];
  nhi = p.cu[min(b_first, p.B - 1) + 1];
#pragma unroll 1
  for (int b0 = 0; b0 < p.B; b0 += THREADS) {
    const int b = b0 + b_first, nb = min(b + THREADS, p.B - 1);
    const int lo = nlo, len = b < p.B ? nhi - nlo : 0;
    nlo = p.cu[nb];
    nhi = p.cu[nb + 1];
    int pos = 0;
    if (len > 0) pos = atomicAdd(&s.bins[bin_of(len)], 1);
    if (together) {
      for (uint64_t left = __ballot(len > 0); left != 0; left &= left - 1) {
        const int l = __ffsll(static_cast<unsigned long long>(left)) - 1;
        const int l_lo = __builtin_amdgcn_readlane(lo, l), l_len = __builtin_amdgcn_readlane(len, l);
        const int ch = attn_chunks(l_len), groups = s.count[ch] * p.H, base = s.item0[ch];
        const int g0 = (__builtin_amdgcn_readlane(pos, l) - s.first[ch]) * p.H;
        for (int j = lane; j < p.H * ch; j += 64)
          p.items[attn_item_slot(base, groups, ch, g0 + j / ch, j % ch)] = encode_item(l_lo, l_len, j / ch, j % ch);
      }
    } else if (len > 0) {
      const int ch = attn_chunks(len), groups = s.count[ch] * p.H, base = s.item0[ch];
      const int g0 = (pos - s.first[ch]) * p.H;
      for (int h = 0; h < p.H; ++h)
        for (int c = 0; c < ch; ++c)
          p.items[attn_item_slot(base, groups, ch, g0 + h, c)] = encode_item(lo, len, h, c);
    }
  }
}

}  // namespace dora
