// The attention plan from sequence boundaries, by one workgroup: shared by the
// plan kernel and by select/pack, where one workgroup of a large launch makes
// the plan while the others copy rows.
//
// Three passes: count the sequences by length (1024 bins), turn the counts
// into positions of the longest-first order and into the item bases of each
// class (sequences of equal chunk count), and give every sequence its position
// (an LDS atomic on its bin) and with it its items' slots.  Latency bound: a few
// memory round trips and, for many sequences, the item stores of one compute
// unit.
//
// ORDER (the plan kernel) sorts more sequences than the workgroup has threads
// in LDS first, so that the lanes of a wave write neighbouring slots: 8192
// sequences of 20 to 197 tokens with 12 heads 61 us by input order, 55 sorted (3
// heads 19.7 and 14.6); up to 1024 sequences the extra pass costs more than it
// gives.  Beside copying workgroups nothing but the bins and class tables is
// held in LDS (about 6 KB), so that the plan's workgroup does not crowd them out.
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

template <int THREADS, bool ORDER>
struct PlanLds {
  int bins[kPlanBins];               // counts, then next position of the longest-first order
  int wave_sums[THREADS / 64];
  int count[kPlanMaxChunks + 1];     // per chunk count: sequences,
  int first[kPlanMaxChunks + 1];     // first position
  int item0[kPlanMaxChunks + 1];     // and first item
  int bad;
  uint32_t order[ORDER ? kPlanMaxB : 1];  // ORDER: sequence | length << 13, by position
};
static_assert(kPlanMaxB == 1 << 13 && DORA_MAX_SEQLEN < 1 << 19, "order");

// Called by every thread of a workgroup of THREADS.
template <int THREADS, bool ORDER>
__device__ __forceinline__ void attn_plan_body(const PlanParams& p, PlanLds<THREADS, ORDER>& s) {
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

  // A sequence of few items is written by its lane, one of more than 64 (a long
  // one) by its wave, and where there is such a one the sequences are dealt over
  // all waves.  One sequence of 16384 tokens with 12 heads: 49 us by one lane, 10
  // by a wave.  By the lengths, not by max_seqlen: 8192 sequences of 20 to 197
  // tokens under max_seqlen 4096 took 263 us written by waves, 55 by lanes.
  const bool ordered = ORDER && p.B > THREADS;
  if (ordered) {
    for (int b = tid; b < p.B; b += THREADS) {
      const int len = p.cu[b + 1] - p.cu[b];
      s.order[atomicAdd(&s.bins[bin_of(len)], 1)] = static_cast<uint32_t>(b) | (static_cast<uint32_t>(len) << 13);
    }
    __syncthreads();
  }
  const bool any_many = s.first[min(64 / p.H, max_ch)] > 0;
  const int i_first = any_many ? lane * (THREADS / 64) + wave : tid;
  int next_lo, next_len, next_pos = 0;
  auto load = [&](int i) {  // past the last: the last again, as an empty one
    const int at = min(i, p.B - 1);
    if (ordered) {
      next_pos = at;
      next_len = static_cast<int>(s.order[at] >> 13);
      next_lo = p.cu[s.order[at] & (kPlanMaxB - 1)];
    } else {
      next_lo = p.cu[at];
      next_len = p.cu[at + 1] - next_lo;
    }
    if (i >= p.B) next_len = 0;
  };
  load(i_first);
#pragma unroll 1
  for (int i0 = 0; i0 < p.B; i0 += THREADS) {
    const int lo = next_lo, len = next_len;
    int pos = next_pos;
    load(i0 + THREADS + i_first);
    const int ch = attn_chunks(len);  // 0 for an empty sequence
    const int groups = s.count[ch] * p.H, base = s.item0[ch];
    if (!ordered && len > 0) pos = atomicAdd(&s.bins[bin_of(len)], 1);
    const int g0 = (pos - s.first[ch]) * p.H;
    const bool many = p.H * ch > 64;
    for (uint64_t left = __ballot(many); left != 0; left &= left - 1) {
      const int l = __ffsll(static_cast<unsigned long long>(left)) - 1;
      const int l_lo = __builtin_amdgcn_readlane(lo, l), l_len = __builtin_amdgcn_readlane(len, l);
      const int l_ch = attn_chunks(l_len), l_groups = s.count[l_ch] * p.H, l_base = s.item0[l_ch];
      const int l_g0 = __builtin_amdgcn_readlane(g0, l);
      for (int j = lane; j < p.H * l_ch; j += 64)
        p.items[attn_item_slot(l_base, l_groups, l_ch, l_g0 + j / l_ch, j % l_ch)] =
            encode_item(l_lo, l_len, j / l_ch, j % l_ch);
    }
    if (!many)
      for (int h = 0; h < p.H; ++h)
        for (int c = 0; c < ch; ++c)
          p.items[attn_item_slot(base, groups, ch, g0 + h, c)] = encode_item(lo, len, h, c);
  }
}

}  // namespace dora
