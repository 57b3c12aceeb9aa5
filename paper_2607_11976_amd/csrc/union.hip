// LiteDSA's group union and per-query membership masks (sec. 3.3). One
// block per group of consecutive queries, in one of two ways chosen by the
// block from the span of its group's keys:
//  * bitmap (the span fits the block's bitmap, about 2^20 keys in wide blocks
//    and 218000 in narrow ones): every entry
//    sets its key's bit in LDS; a prefix sum of the population counts per 128
//    keys gives each key its union slot, so the union comes out ascending and
//    distinct, and each entry finds the bit of its query's mask with two LDS
//    reads. Every step is O(1) per entry.
//  * sort (wider spans): the group's keys are sorted ascending in LDS (bitonic
//    sort of the descending order of ~key, which sends the dropped entries,
//    mapped to 0, last), the first of each run of equal keys takes the next
//    union slot, and every key finds its slot by binary search. LDS is bounded
//    by the group's entries, whatever the span.
// A query's mask is built in LDS with atomic ORs and then written out.
#include <algorithm>

#include "internal.hpp"
#include "select_dev.hpp"

namespace lt {

constexpr int kUnionThreads = 1024;
// groups of at most kUnionSmall entries, in launches of more than
// kUnionManyGroups of them, run narrow blocks, several per CU
constexpr int kUnionThreadsSmall = 256;
constexpr int kUnionSmall = 4096, kUnionManyGroups = 512;
constexpr size_t kUnionLds = 152 * 1024, kUnionLdsSmall = 38 * 1024;  // dynamic LDS the bitmap may take
constexpr int kUnionMaskWords = 2048;  // mask words built in LDS at a time (a query's at least: W <= 1024)

// The bitmap way; false (with nothing written) when the span of the keys
// exceeds the `ng` groups of 128 keys that the block's LDS holds.
// LDS: bitmap [ng * 4], mask words [kUnionMaskWords], prefix [ng] (16 bits: a
// union has at most LT_UNION_MAX keys before its last).
// Bound by the latency of its few passes over LDS and its stores: 128 groups of
// eight lists of 2048 take 22 us a call, where the sort took 162.
template <int NTH, int EPT>
__device__ __forceinline__ bool union_bits(const int32_t* idx, int64_t ld, int t0, int nt, int k, int n, int ng,
                                           int32_t* urow, int32_t* ucount, uint32_t* mask, uint32_t* lds,
                                           uint32_t* tmp) {
  constexpr int NW = NTH / kWave;
  const int tid = threadIdx.x, l = lane_id(), wave = tid / kWave, W = (n + 31) / 32;
  uint32_t* bits = lds;
  uint32_t* mw = lds + 4 * (size_t)ng;
  uint16_t* pre = reinterpret_cast<uint16_t*>(mw + kUnionMaskWords);
  // the thread's entries: tid, tid + NTH, ... of the group's nt * k, as (row
  // r, column c) advanced without a division per entry
  const int m = nt * k, dr = NTH / k, dc = NTH % k;
  int v[EPT];
  int lo = INT_MAX, hi = -1;
  {
    int r = tid / k, c = tid - r * k;
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
      v[j] = -1;
      if (tid + j * NTH < m) v[j] = idx[(int64_t)(t0 + r) * ld + c];
      r += dr;
      c += dc;
      if (c >= k) {
        c -= k;
        ++r;
      }
    }
  }
#pragma unroll
  for (int j = 0; j < EPT; ++j)
    if (v[j] >= 0) {
      lo = min(lo, v[j]);
      hi = max(hi, v[j]);
    }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    lo = min(lo, __shfl_xor(lo, o, kWave));
    hi = max(hi, __shfl_xor(hi, o, kWave));
  }
  if (l == 0) {
    tmp[wave] = (uint32_t)lo;
    tmp[NW + wave] = (uint32_t)hi;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    lo = min(lo, (int)tmp[w]);
    hi = max(hi, (int)tmp[NW + w]);
  }
  const int base = hi < 0 ? 0 : lo & ~127;
  const int used = hi < 0 ? 0 : ((hi - base) >> 7) + 1;  // groups of 128 keys
  if (used > ng) return false;  // block-uniform
  for (int i = tid; i < used * 4; i += NTH) bits[i] = 0u;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < EPT; ++j)
    if (v[j] >= 0) atomicOr(&bits[(v[j] - base) >> 5], 1u << (v[j] & 31));
  __syncthreads();
  // exclusive prefix of the population counts, per group
  auto popc4 = [](const uint4& q) { return __popc(q.x) + __popc(q.y) + __popc(q.z) + __popc(q.w); };
  const uint4* b4 = reinterpret_cast<const uint4*>(bits);
  const int per = (used + NTH - 1) / NTH, g0 = min(tid * per, used), g1 = min(g0 + per, used);
  uint32_t own = 0, total;
  for (int g = g0; g < g1; ++g) own += (uint32_t)popc4(b4[g]);
  uint32_t at = block_scan_excl<NTH>(own, tmp, &total);
  for (int g = g0; g < g1; ++g) {
    pre[g] = (uint16_t)at;
    at += (uint32_t)popc4(b4[g]);
  }
  __syncthreads();
  // slot of the key at bit o (an offset from base)
  auto slot = [&](int o) {
    const uint4 q = b4[o >> 7];
    const int w = (o >> 5) & 3;
    const uint32_t x = w == 0 ? q.x : w == 1 ? q.y : w == 2 ? q.z : q.w;
    uint32_t s = (uint32_t)pre[o >> 7] + (uint32_t)__popc(x & ((1u << (o & 31)) - 1u));
    s += w > 0 ? (uint32_t)__popc(q.x) : 0u;
    s += w > 1 ? (uint32_t)__popc(q.y) : 0u;
    s += w > 2 ? (uint32_t)__popc(q.z) : 0u;
    return s;
  };
  for (int i = tid; i < used * 4; i += NTH) {
    uint32_t x = bits[i];
    if (x == 0u) continue;
    uint32_t s = slot(32 * i);
    for (; x; x &= x - 1) urow[s++] = base + 32 * i + __builtin_ctz(x);
  }
  for (int i = (int)total + tid; i < n; i += NTH) urow[i] = -1;
  if (tid == 0) *ucount = (int32_t)total;
  // membership masks, kUnionMaskWords / W queries at a time
  const int rows = kUnionMaskWords / W;
  for (int r0 = 0; r0 < nt; r0 += rows) {
    const int nr = min(rows, nt - r0);
    for (int i = tid; i < nr * W; i += NTH) mw[i] = 0u;
    __syncthreads();
    // (an opaque copy: the compiler would keep every (r, c) of the load above)
    int ot = tid;
    asm volatile("" : "+v"(ot));
    int r = ot / k, c = ot - r * k;
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
      if (v[j] >= 0 && r >= r0 && r < r0 + nr) {
        const uint32_t s = slot(v[j] - base);
        atomicOr(&mw[(r - r0) * W + (int)(s >> 5)], 1u << (s & 31));
      }
      r += dr;
      c += dc;
      if (c >= k) {
        c -= k;
        ++r;
      }
    }
    __syncthreads();
    for (int i = tid; i < nr * W; i += NTH) mask[(int64_t)(t0 + r0) * W + i] = mw[i];
    __syncthreads();
  }
  return true;
}

// EPT: entries per thread, group * k <= NTH * EPT
template <int NTH, int EPT>
__global__ __launch_bounds__(NTH) void k_dsa_union(const int32_t* idx, int64_t ld, int nq, int k, int group, int ng,
                                                   int32_t* uidx, int32_t* ucount, uint32_t* mask) {
  extern __shared__ __align__(16) uint32_t lds_u[];
  __shared__ uint32_t tmp[2 * NTH / kWave];
  const int g = blockIdx.x, t0 = g * group, nt = min(group, nq - t0);
  const int n = group * k, P = next_pow2(n), W = (n + 31) / 32;
  uint32_t* a = lds_u;          // [P] sort buffer, then the union
  uint32_t* mw = lds_u + P;     // [W] mask of one query
  const int tid = threadIdx.x;
  int32_t* urow = uidx + (int64_t)g * n;
  if (union_bits<NTH, EPT>(idx, ld, t0, nt, k, n, ng, urow, ucount + g, mask, lds_u, tmp)) return;
  __syncthreads();

  // 1. load (rows past the last query and negative entries are dropped)
  for (int i = tid; i < P; i += NTH) {
    int v = -1;
    if (i < n) {
      const int r = i / k, j = i - r * k;
      if (r < nt) v = idx[(int64_t)(t0 + r) * ld + j];
    }
    a[i] = v >= 0 ? ~(uint32_t)v : 0u;
  }
  __syncthreads();
  bitonic_sort_desc<NTH>(a, P);

  // 2. ordered compaction of the first entry of every run; a[] is rewritten
  //    in place: a round writes slots <= its positions, after all its reads,
  //    and the one earlier position a round reads (i0 - 1, which the round
  //    before may have overwritten) is carried in `carry`
  __shared__ uint32_t carry;
  uint32_t base = 0;
  for (int i0 = 0; i0 < P; i0 += NTH) {
    const int i = i0 + tid;
    const uint32_t x = i < P ? a[i] : 0u;
    const uint32_t prev = (i == 0 || i >= P) ? 0u : (tid == 0 ? carry : a[i - 1]);
    const bool first = x != 0u && x != prev;
    uint32_t total;
    const uint32_t ex = block_scan_excl<NTH>(first ? 1u : 0u, tmp, &total);
    __syncthreads();  // every read of this round precedes any write
    if (tid == NTH - 1) carry = x;
    if (first) a[base + ex] = ~x;  // the key itself
    base += total;
    __syncthreads();
  }
  const int count = (int)base;
  for (int i = tid; i < n; i += NTH) urow[i] = i < count ? (int32_t)a[i] : -1;
  if (tid == 0) ucount[g] = count;

  // 3. membership masks, one query at a time
  for (int r = 0; r < nt; ++r) {
    for (int w = tid; w < W; w += NTH) mw[w] = 0u;
    __syncthreads();
    for (int j = tid; j < k; j += NTH) {
      const int v = idx[(int64_t)(t0 + r) * ld + j];
      if (v < 0) continue;
      // lower bound of v in the ascending union a[0, count); v is present
      int lo = 0, hi = count;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if ((int)a[mid] < v) lo = mid + 1;
        else hi = mid;
      }
      atomicOr(&mw[lo >> 5], 1u << (lo & 31));
    }
    __syncthreads();
    uint32_t* mrow = mask + (int64_t)(t0 + r) * W;
    for (int w = tid; w < W; w += NTH) mrow[w] = mw[w];
    __syncthreads();
  }
}

// LDS of the sort way.
static size_t union_sort_lds(int group, int k) {
  const int n = group * k;
  return ((size_t)next_pow2(n) + (size_t)(n + 31) / 32) * 4;
}

hipError_t launch_dsa_union(const int32_t* idx, int64_t ld, int nq, int k, int group, int32_t* uidx, int32_t* ucount,
                            uint32_t* mask, hipStream_t st) {
  const int groups = (nq + group - 1) / group;
  if (groups == 0) return hipSuccess;
  auto go = [&](auto kernel, int nth, size_t room) {
    const size_t lds = std::max(union_sort_lds(group, k), room);
    // 16 bytes of bitmap and 2 of prefix per group of 128 keys
    const int ng = (int)((lds - kUnionMaskWords * 4) / 18);
    if (lds > 65536)
      (void)hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kernel, dim3(groups), dim3(nth), lds, st, idx, ld, nq, k, group, ng, uidx, ucount, mask);
  };
  // small groups leave most of a wide block idle: 2048 lists of 256 keys alone
  // take 24 us in narrow blocks and 70 us in wide ones, 1024 pairs of lists of
  // 1024 keys 20 us and 43 us. Where few groups are that small, wide blocks
  // with one entry per thread: 512 lists of 1024 keys 13.2 us (20.2 in the
  // blocks of 16 entries), 16 of 64 13.2 (16.0). The host does not know the
  // span: 1024 pairs of lists of 2048 keys take 23 us in narrow blocks within
  // their bitmap and 122 to 125 past it, in the sort (164 to 172 in the wide
  // blocks' sort alone)
  const int n = group * k;
  if (n <= kUnionSmall && groups > kUnionManyGroups)
    go(k_dsa_union<kUnionThreadsSmall, kUnionSmall / kUnionThreadsSmall>, kUnionThreadsSmall, kUnionLdsSmall);
  else if (n <= kUnionThreads)
    go(k_dsa_union<kUnionThreads, 1>, kUnionThreads, kUnionLds);
  else if (n <= LT_UNION_MAX / 2)
    go(k_dsa_union<kUnionThreads, LT_UNION_MAX / 2 / kUnionThreads>, kUnionThreads, kUnionLds);
  else
    go(k_dsa_union<kUnionThreads, LT_UNION_MAX / kUnionThreads>, kUnionThreads, kUnionLds);
  return hipGetLastError();
}

}  // namespace lt
