// Selection-side kernels: per-row range from the sample, the scores-in
// filter scan, the final select, the exact fallback and plain radix select.
#include <type_traits>

#include "internal.hpp"
#include "select_dev.hpp"

namespace lt {

// ---------------------------------------------------------------------------
// Zero the queue counters, the fallback cursor and its chunk counters, where
// no sample list is made that would do it.
// ---------------------------------------------------------------------------
__global__ void k_init(uint32_t* qctl) {
  for (int i = threadIdx.x; i < kQctlWords; i += blockDim.x) qctl[i] = 0u;
}

// ---------------------------------------------------------------------------
// Range and initial threshold (sec. 3.2 "Sampling"). One block per row.
// s_min / s_max over the row's visible, finite sample scores; delta = m /
// (s_max - s_min); tau0 = bin of the k-th largest visible sample score, found
// with the sample's histogram. The sample histogram is NOT carried into the
// scan: every sampled key is scanned again, and counting it twice could
// raise the threshold above the true k-th score.
// The sample is the key list `list` (holes < 0 skipped; NULL: every sample key
// is visible to every row, and the list need not be read). FROM_SCORES: its
// scores are read from a score matrix (scores-in entry); otherwise from the
// [nq, ns] matrix of sample scores the sample kernel wrote. Each thread keeps
// kRangeUnroll loads in flight: the kernel is bound by load latency.
// ---------------------------------------------------------------------------
constexpr int kRangeThreads = 256;
constexpr int kRangeThreadsLarge = 1024;  // samples of kRangeLargeSample keys or more, or few rows
constexpr int kRangeLargeSample = 16384;
constexpr int kRangeUnroll = 8;
constexpr int kRangeThreadsMid = 512;  // two blocks of them fit a CU with kRangeHold * 2 scores a thread
constexpr int kRangeHold = 32, kRangeHoldFew = 8;  // sample scores a thread keeps in registers

template <int NTH, bool FROM_SCORES>
__device__ __forceinline__ void range_load(const float* rp, const int32_t* list, int ns, RowRange rr, int base,
                                           float (&s)[kRangeUnroll], bool (&vis)[kRangeUnroll]) {
  int key[kRangeUnroll];
#pragma unroll
  for (int u = 0; u < kRangeUnroll; ++u) {
    const int i = base + u * NTH + (int)threadIdx.x;
    key[u] = -1;
    if (i < ns) key[u] = list ? list[i] : rr.s;
  }
#pragma unroll
  for (int u = 0; u < kRangeUnroll; ++u) {
    const int i = base + u * NTH + (int)threadIdx.x;
    vis[u] = key[u] >= rr.s && key[u] < rr.e;
    s[u] = vis[u] ? (FROM_SCORES ? rp[key[u]] : rp[i]) : 0.0f;
  }
}

// HOLD: sample scores per thread kept in registers (ns <= NTH * HOLD), or 0:
// read twice. The histogram of held scores takes only what tau0 needs of it: the bins from
// 3m/4 up where they hold k sample keys, else from m/2 up, else all (LDS
// atomics on the few bins that most scores fall in cost more than the reads).
template <int NTH, bool FROM_SCORES, int HOLD>
__global__ __launch_bounds__(NTH) void k_range(const float* src, int64_t stride, int nq, int nk,
                                                         const int32_t* offs, const int32_t* starts,
                                                         const int32_t* list, int ns, int m, int k,
                                                         RowParam* params, int32_t* stats, int32_t* rflag,
                                                         uint64_t* pub) {
  constexpr int NW = NTH / kWave, U = kRangeUnroll, STEP = NTH * U;
  static_assert(HOLD % U == 0, "whole steps");
  __shared__ uint32_t hist[kMaxBins];
  __shared__ float red_mn[NW], red_mx[NW];
  __shared__ uint32_t red_n[NW];
  __shared__ uint32_t sel[2];
  const int row = blockIdx.x, wave = threadIdx.x / kWave, l = lane_id();
  const RowRange rr = row_range(offs, starts, row, nk);
  const float* rp = src + (int64_t)row * stride;

  for (int b = threadIdx.x; b < kMaxBins; b += NTH) hist[b] = 0u;
  if (threadIdx.x < 2) sel[threadIdx.x] = 0u;
  // the row's flags of the second filter pass (rflag[row]) and of the dense
  // fallback (rflag[nq + row])
  if (rflag && threadIdx.x == 0) {
    rflag[row] = 0;
    rflag[nq + row] = 0;
  }
  // step j of the sample: its visible scores, NaN for the others and past ns
  // (a NaN score is counted as visible and otherwise left out too)
  uint32_t nvis = 0;
  auto fetch = [&](int base, float* v, bool count) {
    float s[U];
    bool vis[U];
    range_load<NTH, FROM_SCORES>(rp, list, ns, rr, base, s, vis);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (count) nvis += vis[u];
      v[u] = vis[u] ? s[u] : __builtin_nanf("");
    }
  };
  constexpr int KEEP = HOLD > 0 ? HOLD : U;
  float v[KEEP];
  // every sample key visible: the whole row's loads go out at once, through a
  // descriptor whose range check needs no branch
  bool held = false;
  if constexpr (HOLD > 0 && !FROM_SCORES) {
    if (!list) {
      held = true;
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)rp, 0, ns * 4, kBufferRaw);
#pragma unroll
      for (int j = 0; j < HOLD; ++j)
        v[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)threadIdx.x * 4 + j * NTH * 4, 0, 0));
#pragma unroll
      for (int j = 0; j < HOLD; ++j) {
        const bool in = (int)threadIdx.x + j * NTH < ns;
        nvis += in;
        v[j] = in ? v[j] : __builtin_nanf("");
      }
    }
  }
  auto each = [&](bool first, auto&& body) {
    if constexpr (HOLD > 0) {
#pragma unroll
      for (int j = 0; j < HOLD; j += U) {
        if (j * NTH < ns) {
          if (first && !held) fetch(j * NTH, v + j, true);
          body(v + j);
        }
      }
    }
  };
  float mn = __builtin_inff(), mx = -__builtin_inff();
  if constexpr (HOLD > 0) {
    each(true, [&](const float* x) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (__builtin_isfinite(x[u])) {
          mn = fminf(mn, x[u]);
          mx = fmaxf(mx, x[u]);
        }
      }
    });
  } else {
    for (int base = 0; base < ns; base += STEP) {
      float s[U];
      bool vis[U];
      range_load<NTH, FROM_SCORES>(rp, list, ns, rr, base, s, vis);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        nvis += vis[u];
        if (vis[u] && __builtin_isfinite(s[u])) {
          mn = fminf(mn, s[u]);
          mx = fmaxf(mx, s[u]);
        }
      }
    }
  }
  mn = wave_min(mn);
  mx = wave_max(mx);
  nvis = wave_sum(nvis);
  if (l == 0) {
    red_mn[wave] = mn;
    red_mx[wave] = mx;
    red_n[wave] = nvis;
  }
  __syncthreads();
  mn = red_mn[0];
  mx = red_mx[0];
  nvis = red_n[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) {
    mn = fminf(mn, red_mn[w]);
    mx = fmaxf(mx, red_mx[w]);
    nvis += red_n[w];
  }
  float delta = 1.0f, c = 0.0f;
  if (mx > mn) delta = (float)m / (mx - mn);
  if (!(delta > 0.0f) || !__builtin_isfinite(delta)) delta = 1.0f;
  if (__builtin_isfinite(mn)) c = -mn * delta;
  if (!__builtin_isfinite(c)) c = 0.0f;

  // the lowest bin that the histogram takes
  int from = 0;
  if constexpr (HOLD > 0) {
    // (bins end at m - 1: the greatest scores, at m and above, are clamped to it)
    const int b_hi = min(m - m / 4, m - 1), b_mid = m / 2;
    const float hi = (float)b_hi, mid = (float)b_mid;
    uint32_t n_hi = 0, n_mid = 0;
    each(false, [&](const float* x) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float t = bin_x(x[u], delta, c);
        n_hi += t >= hi;
        n_mid += t >= mid;
      }
    });
    n_hi = wave_sum(n_hi);
    n_mid = wave_sum(n_mid);
    if (l == 0) {
      atomicAdd(&sel[0], n_hi);
      atomicAdd(&sel[1], n_mid);
    }
    __syncthreads();
    from = sel[0] >= (uint32_t)k ? b_hi : sel[1] >= (uint32_t)k ? b_mid : 0;
  }
  if constexpr (HOLD > 0) {
    each(false, [&](const float* x) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int b = bin_of(bin_x(x[u], delta, c), m);
        if (b >= from) atomicAdd(&hist[b], 1u);
      }
    });
  } else {
    for (int base = 0; base < ns; base += STEP) {
      float s[U];
      bool vis[U];
      range_load<NTH, FROM_SCORES>(rp, list, ns, rr, base, s, vis);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int b = bin_of(bin_x(s[u], delta, c), m);
        if (vis[u] && b >= 0) atomicAdd(&hist[b], 1u);
      }
    }
  }
  __syncthreads();
  if (wave == 0) {
    const int tau0 = wave_threshold(hist, m, (uint32_t)k, nullptr);
    if (l == 0) params[row] = RowParam{delta, c, tau0, (int)nvis};
    if (pub && l == 0) pub[row] = pub_word(tau0);
    if (stats && l == 0) {
      int32_t* sr = stats + (int64_t)row * LT_ROW_STATS;
      sr[4] = tau0;
      sr[6] = (int32_t)__float_as_uint(delta);
      sr[7] = (int32_t)__float_as_uint(c);
      sr[8] = m;
      sr[9] = (int32_t)nvis;
      sr[10] = 0;
      sr[11] = 0;
    }
  }
  if (!stats) return;
  // The sample's k-th score under the total order (for the invariant
  // kth(sample) <= kth(row) of sec. 3.2 "Sampling"): most-significant-digit
  // radix selection over the order keys of the visible sample scores, four
  // 8-bit digits, the bins reused as the digit histogram.
  uint32_t prefix = 0, pmask = 0, want = (uint32_t)k;
  for (int shift = 24; shift >= 0 && nvis >= (uint32_t)k; shift -= 8) {
    __syncthreads();
    for (int b = threadIdx.x; b < kMaxBins; b += NTH) hist[b] = 0u;
    __syncthreads();
    for (int base = 0; base < ns; base += NTH * kRangeUnroll) {
      float sv[kRangeUnroll];
      bool vis[kRangeUnroll];
      range_load<NTH, FROM_SCORES>(rp, list, ns, rr, base, sv, vis);
#pragma unroll
      for (int u = 0; u < kRangeUnroll; ++u) {
        const uint32_t o = ord_key(sv[u]);
        if (vis[u] && (o & pmask) == prefix) atomicAdd(&hist[(o >> shift) & 0xFFu], 1u);
      }
    }
    __syncthreads();
    if (wave == 0) {
      uint32_t above = 0;
      const int dg = wave_threshold(hist, kMaxBins, want, &above);
      if (l == 0) {
        sel[0] = (uint32_t)dg;
        sel[1] = above;
      }
    }
    __syncthreads();
    const uint32_t dg = sel[0], above = sel[1];
    prefix |= dg << shift;
    pmask |= 0xFFu << shift;
    want -= above;
  }
  if (threadIdx.x == 0)
    stats[(int64_t)row * LT_ROW_STATS + 5] =
        nvis >= (uint32_t)k ? (int32_t)__float_as_uint(ord_inv(prefix)) : (int32_t)0xFF800000u;
}

// ---------------------------------------------------------------------------
// Scores-in filter scan (sec. 3.2 "Filtering" + "Threshold Refresh"). One
// block owns one (row, key split): it streams its scores once in steps of
// NTH * U keys, wave w of a step taking the w-th run of kWave * U
// consecutive keys, gates them with the row's current
// threshold bin, appends the passing ones to the split's candidate list in
// key order (a ballot per 64 keys; the waves exchange their step totals
// through LDS, one barrier a step) and counts them in the block's LDS
// histogram. A list that reaches `cap` stops storing but keeps counting, so
// the final select can detect the overflow.
// Threshold refresh: a step counts its passing keys in the histogram first.
// Once kRefreshShare-th of k new ones have been counted, every wave walks the
// histogram to the new threshold and the step's keys are gated again before
// they are written, so that a step as long as a short row keeps no more than
// a fine-grained scan would.
// The splits of a row cut its visible range into even parts and keep their
// own thresholds: reading each other's from global memory stalled every
// refresh (128 rows x 131072 in two splits: 158 us a call against 76) and
// came too late in short splits, so the host makes few and long ones
// (resolve_scores).
// Bound by HBM: the loads of the next step (4 U bytes a thread) are in flight
// while the current one is gated, and the block is as wide as it takes to keep
// four waves per SIMD resident (launch_filter).
// 1024 rows of 262144 scores (1.07 GB), k = 2048: 1078 us with one wave per
// row and one load in flight, 282 us so (3.8 TB/s).
// ---------------------------------------------------------------------------
constexpr int kRefreshShare = 4;
constexpr int kFilterShort = 1024;  // splits of so many keys are one wave's
constexpr int kFilterLong = 32768;  // splits of this many keys take 16 keys per thread and step, shorter ones 8

template <int NTH, int U>
__global__ __launch_bounds__(NTH) void k_filter(const float* scores, int64_t stride, int nq, int nk,
                                                const int32_t* offs, const int32_t* starts, const RowParam* params,
                                                int S, int L, int cap, int m, int k, uint32_t* cnt,
                                                uint32_t* hist_out, int2* cand) {
  constexpr int NW = NTH / kWave, STEP = NTH * U;
  __shared__ uint32_t hist[kMaxBins];
  __shared__ uint32_t wtot[3][NW];  // the waves' passing keys: steps in turn, a step gated again
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), l = lane_id();
  const int unit = blockIdx.x, row = unit / S, split = unit - row * S;
  const RowRange rr = row_range(offs, starts, row, nk);
  // the split's share of the row's range (at most L keys; positions unsigned,
  // here and below: a row may have up to 2^31 - 1 keys)
  const uint32_t range = rr.e - rr.s;
  const uint32_t part = min((uint32_t)L, ((range + S - 1) / S + 255) & ~255u);
  const int lo = rr.s + (int)min(split * part, range), hi = lo + (int)min(part, (uint32_t)(rr.e - lo));
  const RowParam p = params[row];
  float thr = gate_thr(p.tau0);
  for (int b = threadIdx.x; b < kMaxBins; b += NTH) hist[b] = 0u;
  __syncthreads();

  int2* out = cand + (int64_t)unit * cap;
  uint32_t tail = 0, fresh = 0;
  const uint32_t refresh_at = max((uint32_t)k / kRefreshShare, 8u);
  const uint32_t len = hi - lo;
  // a descriptor per step whose range check turns the keys past hi into
  // zeros without a branch (they are masked below)
  const uint64_t base = (uint64_t)(scores + (int64_t)row * stride + lo);
  const float* ubase = (const float*)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)base) |
                                      (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(base >> 32)) << 32);
  const uint32_t ulen = __builtin_amdgcn_readfirstlane(len);
  const uint32_t woff = wave * kWave * U;  // the wave's keys of a step: [step + woff, + kWave * U)
  auto load = [&](uint32_t off, float (&v)[U]) {
    const uint32_t at = off + woff;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(ubase + at), 0, at < ulen ? (int)(min(ulen - at, (uint32_t)(kWave * U)) * 4u) : 0, kBufferRaw);
#pragma unroll
    for (int u = 0; u < U; ++u)
      v[u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, l * 4 + u * kWave * 4, 0, 0));
  };
  int par = 0;
  // the waves' totals: this wave's offset in the step and the step's total
  uint32_t before = 0, total = 0;
  auto exchange = [&](uint32_t* tot, uint32_t mine) {
    if (l == 0) tot[wave] = mine;
    __syncthreads();
    before = total = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const uint32_t t = (uint32_t)__builtin_amdgcn_readfirstlane((int)tot[w]);
      before += w < wave ? t : 0u;
      total += t;
    }
  };
  auto step = [&](uint32_t off, const float (&v)[U]) {
    const uint32_t rel = off + woff + l;  // position of item 0 in the split
    uint32_t bits = 0, mine = 0;     // bit u: item u passes; the wave's passing keys
    auto gate = [&]() {
      bits = mine = 0;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool ps = (rel + u * kWave < ulen) & !(bin_x(v[u], p.delta, p.c) < thr);
        mine += (uint32_t)__popcll(__ballot(ps));
        bits |= (uint32_t)ps << u;
      }
    };
    gate();
    if (mine != 0) {  // wave-uniform
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int b = bin_of(bin_x(v[u], p.delta, p.c), m);
        if (((bits >> u) & 1u) && b >= 0) atomicAdd(&hist[b], 1u);
      }
    }
    exchange(wtot[par], mine);
    par ^= 1;
    fresh += total;
    if (fresh >= refresh_at) {  // block-uniform; no wave counts again before the exchange below
      fresh = 0;
      thr = fmaxf(thr, gate_thr(wave_threshold(hist, m, (uint32_t)k, nullptr)));
      gate();
      exchange(wtot[2], mine);
    }
    if (mine != 0) {
      uint32_t at = tail + before;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool ps = (bits >> u) & 1u;
        const uint64_t mask = __ballot(ps);
        const uint32_t pos = at + mbcnt64(mask);
        if (ps && pos < (uint32_t)cap) out[pos] = make_int2(lo + (int)(rel + u * kWave), __float_as_int(v[u]));
        at += (uint32_t)__popcll(mask);
      }
    }
    tail += total;
  };
  if (ulen > 0) {
    float va[U], vb[U];
    load(0, va);
    for (uint32_t off = 0; off < ulen; off += 2 * STEP) {
      load(off + STEP, vb);
      step(off, va);
      load(off + 2 * STEP, va);
      step(off + STEP, vb);
    }
  }
  __syncthreads();
  for (int b = threadIdx.x; b < m; b += NTH) hist_out[(int64_t)unit * m + b] = hist[b];
  if (threadIdx.x == 0) cnt[unit] = tail;
}

// ---------------------------------------------------------------------------
// Final select (sec. 3.2 "Top-k Selection"). One block per row.
//  1. Sum the row's HS histograms; the final threshold bin tau is the largest
//     bin whose suffix count reaches k (bins >= tau are complete: every key in
//     them passed the gate, which never exceeded tau).
//  2. Candidates in bins above tau (fewer than k) go straight to the output,
//     in list order.
//  3. Candidates in bin tau are collected in LDS and only they are sorted;
//     the best k - (count above) complete the row.
// The row's S lists are walked as one sequence, NTH lists at a time (their
// counts prefix-summed in LDS) and PER entries per thread per step, so many
// short lists cost no more than one long one. Keyed rows (few rows with
// hundreds of thousands of candidates each) run 1024 threads with 8 entries
// per thread; the others 256 threads with 4.
// Rows whose buffer overflowed, whose threshold bin does not fit in LDS,
// whose counts disagree with their lists, whose final bin lies below the
// sample's initial bin, or that are forced, are queued for the exact fallback
// instead.
// ---------------------------------------------------------------------------
constexpr int kSelThreads = 256;
constexpr int kSelPer = 4;         // list entries per thread per step
constexpr int kSelThreadsWide = 1024;  // keyed rows, and launches of few rows
constexpr int kSelPerWide = 8;
constexpr int kSelFewRows = 512;     // launches of at most this many rows use the wide blocks
constexpr int kSecondSelectGrid = 512;  // blocks of the second select (persistent over its queue)

// Threshold bins of at most this many keys are ranked by counting instead of
// sorted.
constexpr int kRankMax = 512;

constexpr int kHistUnroll = 8;  // split histograms a thread reads at once

// LDS byte offset of the sort entries of k_select with NTH threads.
constexpr size_t select_ent_offset(int nth) { return ((size_t)kMaxBins + 32 + nth + 16) * 4; }

// Sorted rows. Their final order does not depend on the order in which the
// candidates arrive, so the keys at or above bin tau (k plus part of one bin)
// are gathered into LDS by independent waves and ordered there by
// order_entries, where a gather in list order, block-wide step by step, and a
// bitonic sort took twice as long (4096 rows of 8.7 K candidates, k = 2048:
// 314 -> 149 us; 10000 rows of 1.1 K, k = 100: 231 -> 125 us).
// Rows with more than sort_slots(E) keys take the general path.
//
// nmax: keys at or above bin tau by the histograms. Returns 0 when the row is
// written, 1 when the lists disagree with the histograms (the fallback's), -1
// for the general path. tmp[26] ends as the keys gathered, tmp[27] as those
// above bin tau.
template <int NTH, int PER>
__device__ __forceinline__ int select_sorted(int row, const RowParam& p, const uint32_t* cnt, const int2* cand, int nq,
                                             int S, int cap, int m, int k, int E, bool keyed, bool ilv, int tau,
                                             uint32_t c_above, uint32_t nmax, uint32_t* tmp, uint32_t* off,
                                             uint64_t* ent, int32_t* oi, float* os) {
  constexpr int NW = NTH / kWave, EPT = 12;  // entries per thread: sort_slots(E) / NTH at most (launch_select)
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), l = lane_id();
  const uint32_t slots = (uint32_t)sort_slots(E);
  const int NB = bucket_count<NTH>(nmax, E);
  int2* e2 = reinterpret_cast<int2*>(ent);
  uint32_t* bk = reinterpret_cast<uint32_t*>(ent + slots);  // [NB]
  float* red = reinterpret_cast<float*>(off);               // [2 * NW]
  for (int b = tid; b < NB; b += NTH) bk[b] = 0u;
  if (tid == 0) {
    tmp[26] = 0u;
    tmp[27] = 0u;
  }
  __syncthreads();

  // ---- gather ----
  float mn = __builtin_inff(), mx = -__builtin_inff();
  uint32_t wab = 0;  // the wave's keys above bin tau
  // positions p0 + u * ll + lo (u < PER) of list li, of c entries
  auto take = [&](int64_t li, uint32_t c, uint32_t p0, int ll, int lo) {
    int2 ce[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const uint32_t pos = p0 + (uint32_t)(u * ll + lo);
      ce[u] = make_int2(0, 0);
      if (pos < c) ce[u] = cand[ilv ? ilv_index(li, pos, (int64_t)nq * S) : li * cap + pos];
    }
    uint32_t in = 0u, nin = 0u;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const bool v = p0 + (uint32_t)(u * ll + lo) < c;
      const float sc = __int_as_float(ce[u].y);
      const int b = bin_of(bin_x(sc, p.delta, p.c), m);
      const bool i1 = v & (b >= tau);
      in |= (uint32_t)i1 << u;
      nin += (uint32_t)__popcll(__ballot(i1));
      wab += (uint32_t)__popcll(__ballot(v & (b > tau)));
      if (i1 & (bool)__builtin_isfinite(sc)) {
        mn = fminf(mn, sc);
        mx = fmaxf(mx, sc);
      }
    }
    if (nin == 0) return;
    uint32_t r0 = 0u;
    if (l == 0) r0 = atomicAdd(&tmp[26], nin);
    r0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)r0);
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const bool i1 = (in >> u) & 1u;
      const uint64_t mk = __ballot(i1);
      const uint32_t r = r0 + mbcnt64(mk);
      if (i1 && r < slots) e2[r] = ce[u];
      r0 += (uint32_t)__popcll(mk);
    }
  };
  if (S >= 4 * NW) {
    // whole lists per wave, four at a time (16 lanes on 16 consecutive
    // positions of each, one 128-byte chunk)
    constexpr int ll = kWave / 4;
    const int sub = l / ll, lo = l - sub * ll;
    for (int s0 = wave * 4; s0 < S; s0 += NW * 4) {
      const int64_t li = (int64_t)row * S + s0 + sub;
      const uint32_t c = s0 + sub < S ? min(cnt[li], (uint32_t)cap) : 0u;
      uint32_t cmax = 0u;
#pragma unroll
      for (int g = 0; g < 4; ++g) cmax = max(cmax, (uint32_t)__builtin_amdgcn_readlane((int)c, g * ll));
      for (uint32_t p0 = 0; p0 < cmax; p0 += (uint32_t)(PER * ll)) take(li, c, p0, ll, lo);
    }
  } else {
    // few lists (at most a wave's lanes), of any lengths: their runs of
    // PER * 64 entries go round the waves
    static_assert(4 * NW <= kWave, "one list per lane");
    const uint32_t cl = l < S ? min(cnt[(int64_t)row * S + l], (uint32_t)cap) : 0u;
    uint32_t turn = 0;  // runs handed out so far
    for (int s = 0; s < S; ++s) {
      const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)cl, s);
      const uint32_t runs = (c + PER * kWave - 1) / (PER * kWave);
      for (uint32_t r = (uint32_t)(wave - (int)turn) & (NW - 1); r < runs; r += NW)
        take((int64_t)row * S + s, c, r * (PER * kWave), kWave, l);
      turn += runs;
    }
  }
  mn = wave_min(mn);
  mx = wave_max(mx);
  if (l == 0) {
    red[wave] = mn;
    red[NW + wave] = mx;
    if (wab) atomicAdd(&tmp[27], wab);
  }
  __syncthreads();
  const uint32_t n = tmp[26];
  if (n > slots) return -1;
  if (tmp[27] != c_above) return 1;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    mn = fminf(mn, red[w]);
    mx = fmaxf(mx, red[NW + w]);
  }

  order_entries<NTH, EPT>(e2, n, mn, mx, bk, NB, off);
  for (int i = tid; i < k; i += NTH) {
    const bool v = (uint32_t)i < n;
    const int2 x = v ? e2[i] : make_int2(-1, __float_as_int(-__builtin_inff()));
    oi[i] = x.x;
    // keyed rows report canonical scores (a zero as +0, a NaN as the quiet one)
    const float sc = __int_as_float(x.y);
    os[i] = keyed && v ? ord_inv(ord_key(sc)) : sc;
  }
  return 0;
}

template <int NTH, int PER>
__device__ __forceinline__ void select_row(int row, RowParam* params, const uint32_t* cnt, const uint32_t* hist,
                           const int2* cand, int nq, int S, int HS, int cap, int m, int k, int E, uint32_t flags,
                           int32_t* out_i, float* out_s, uint32_t* qctl, int32_t* queue, int32_t* rqueue,
                           int32_t* rflag, uint64_t* pub, int32_t* stats) {
  extern __shared__ __align__(16) uint8_t lds[];
  uint32_t* hsum = reinterpret_cast<uint32_t*>(lds);          // [256]
  uint32_t* tmp = hsum + kMaxBins;                             // [32]
  uint32_t* off = tmp + 32;                                    // [NTH + 1]: list offsets of a group
  uint64_t* ent = reinterpret_cast<uint64_t*>(lds + select_ent_offset(NTH));  // [E]
  const int tid = threadIdx.x;
  // keyed: the lists are not in key order, so the tie-break position is the
  // key itself, the sorted scores are rebuilt from the sort entries, and
  // every row is sorted (the order of arrival would make it vary between
  // calls)
  const bool keyed = flags & kSelKeyed;
  const bool ilv = flags & kSelIlv;
  const bool sorted = (flags & LT_SORTED_OUTPUT) || keyed;
  int32_t* oi = out_i + (int64_t)row * k;
  float* os = out_s + (int64_t)row * k;

  // ---- overflow / forced ----
  uint32_t total_c = 0;
  int reason = (flags & LT_FORCE_FALLBACK) ? 3 : 0;
  {
    uint32_t my = 0;
    bool ovf = false;
    for (int s = tid; s < S; s += NTH) {
      const uint32_t c = cnt[(int64_t)row * S + s];
      my += c;
      ovf |= c > (uint32_t)cap;
    }
    (void)block_scan_excl<NTH>(my, tmp, &total_c);
    if (__syncthreads_or(ovf) && reason == 0) reason = 1;
  }
  auto enqueue = [&](int why, int tau, uint32_t nt) {
    if (tid == 0) {
      uint32_t slot = atomicAdd(&qctl[0], 1u);
      queue[slot] = row;
      if (rflag) rflag[nq + row] = 1;  // queued for the dense fallback
      if (stats) {
        int32_t* st = stats + (int64_t)row * LT_ROW_STATS;
        if (!(flags & kSelSecond)) st[0] = (int32_t)total_c;
        st[1] = tau;
        st[2] = why;
        st[3] = (int32_t)nt;
      }
    }
  };
  if (reason == 3) {
    enqueue(reason, -2, 0);
    return;
  }

  // ---- 1. final threshold bin ----
  // The sum of the row's HS histograms: thread (b, g) adds every
  // (NTH / kMaxBins)-th of them, kHistUnroll loads in flight (a row of a few
  // queries has up to 256: one load after the other, 64 and 256 splits of two
  // rows took 40 and 84 us in this kernel).
  {
    constexpr int G = NTH / kMaxBins;
    static_assert(G >= 1, "one thread per bin at least");
    const int b = tid & (kMaxBins - 1), g = tid / kMaxBins;
    const uint32_t* hp = hist + (int64_t)row * HS * m + b;
    uint32_t h = 0;
    if (b < m) {
      for (int s = g; s < HS; s += kHistUnroll * G) {
        uint32_t x[kHistUnroll];
#pragma unroll
        for (int u = 0; u < kHistUnroll; ++u) x[u] = s + u * G < HS ? hp[(int64_t)(s + u * G) * m] : 0u;
#pragma unroll
        for (int u = 0; u < kHistUnroll; ++u) h += x[u];
      }
    }
    if constexpr (G == 1) {
      hsum[b] = h;
    } else {
      if (g == 0) hsum[b] = 0u;
      __syncthreads();
      if (h) atomicAdd(&hsum[b], h);
    }
  }
  __syncthreads();
  if (tid < kWave) {
    uint32_t above = 0;
    int tau = wave_threshold(hsum, m, (uint32_t)k, &above);
    if (tid == 0) {
      tmp[24] = (uint32_t)tau;
      tmp[25] = above;
    }
  }
  __syncthreads();
  const int tau = (int)tmp[24];
  const uint32_t c_above = tmp[25];
  const uint32_t c_tie = tau >= 0 ? hsum[tau] : 0u;
  __syncthreads();
  if (reason == 1) {
    // The lists overflowed, but the histograms kept counting: bins >= tau
    // are complete and tau is the row's exact final bin. A second filter
    // pass gated at tau from its first key writes exactly the c_above +
    // c_tie keys of those bins; when they fit in one list (and the sort
    // buffer) the row is queued for that pass, else for the dense fallback.
    if ((flags & kSelRefilter) && tau >= 0 && c_above + c_tie <= (uint32_t)cap && c_tie <= (uint32_t)E) {
      if (tid == 0) {
        params[row].tau0 = tau;
        if (pub) pub[row] = pub_word(tau);
        rflag[row] = 1;
        rqueue[atomicAdd(&qctl[1], 1u)] = row;
        if (stats) {
          int32_t* st = stats + (int64_t)row * LT_ROW_STATS;
          st[0] = (int32_t)total_c;
          st[1] = tau;
          st[2] = 6;
          st[3] = (int32_t)c_tie;
        }
      }
      return;
    }
    enqueue(1, tau, c_tie);
    return;
  }
  const RowParam p = params[row];
  // Every visible sample key in a bin >= tau0 passes the gate or is
  // outranked by k counted keys, so an exact scan ends with tau >= tau0. A
  // lower bin means the sample's scores and the scan's disagree; the bins
  // between were gated and are incomplete, so the row is recomputed.
  if (p.tau0 >= 0 && tau < p.tau0) {
    enqueue(5, tau, 0);
    return;
  }

  // ---- sorted rows: the keys at or above bin tau in one gather ----
  // (see select_sorted); a row that it does not take goes on
  // with the steps below
  const uint32_t nmax = tau >= 0 ? c_above + c_tie : total_c;
  if (sorted && nmax <= (uint32_t)sort_slots(E)) {
    const int done = select_sorted<NTH, PER>(row, p, cnt, cand, nq, S, cap, m, k, E, keyed, ilv, tau, c_above, nmax,
                                             tmp, off, ent, oi, os);
    if (done >= 0) {
      if (done == 0 && stats && tid == 0) {
        int32_t* st = stats + (int64_t)row * LT_ROW_STATS;
        if (!(flags & kSelSecond)) st[0] = (int32_t)total_c;
        st[1] = tau;
        st[2] = (flags & kSelSecond) ? 6 : 0;
        st[3] = (int32_t)(tmp[26] - tmp[27]);
      }
      if (done == 1) enqueue(4, tau, tmp[26] - tmp[27]);
      return;
    }
    __syncthreads();
  }

  // ---- 2./3. one pass over the candidates ----
  uint32_t run_above = 0, run_tie = 0;
  bool tie_ovf = false;
  if (keyed) {
    // The final sort puts the keys above bin tau in order and bin tau's
    // entries carry their keys, so no position needs the list order: each
    // wave takes whole lists, four at a time when there are enough (16 lanes
    // on 16 consecutive positions of each, one 128-byte chunk), with PER
    // loads in flight per lane, and reserves output slots with one LDS
    // atomic per kind and step. No block-wide step, no search for a
    // position's list.
    constexpr int NW = NTH / kWave;
    const int wave = tid / kWave, l = lane_id();
    const int lpw = S >= 4 * NW ? 4 : 1;  // lists a wave takes at once
    const int ll = kWave / lpw, sub = l / ll, lo = l - sub * ll;
    if (tid == 0) {
      tmp[26] = 0u;
      tmp[27] = 0u;
    }
    __syncthreads();
    for (int s0 = wave * lpw; s0 < S; s0 += NW * lpw) {
      const int s = s0 + sub;
      const int64_t li = (int64_t)row * S + s;
      const uint32_t c = s < S ? min(cnt[li], (uint32_t)cap) : 0u;
      // the wave steps through the longest of its lists
      uint32_t cmax = 0u;
      for (int g = 0; g < lpw; ++g) cmax = max(cmax, (uint32_t)__builtin_amdgcn_readlane((int)c, g * ll));
      for (uint32_t p0 = 0; p0 < cmax; p0 += (uint32_t)(PER * ll)) {
        int2 ce[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          const uint32_t pos = p0 + (uint32_t)(u * ll + lo);
          ce[u] = make_int2(0, 0);
          if (pos < c) ce[u] = cand[ilv ? ilv_index(li, pos, (int64_t)nq * S) : li * cap + pos];
        }
        // bit u: entry u is above bin tau (ab) / in it (ti); the wave masks
        // are taken again where they are used, to keep few of them live
        uint32_t ab = 0u, ti = 0u, na = 0u, nt = 0u;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          const bool v = p0 + (uint32_t)(u * ll + lo) < c;
          const int b = bin_of(bin_x(__int_as_float(ce[u].y), p.delta, p.c), m);
          const bool a1 = v & (b > tau), t1 = v & (b == tau);
          ab |= (uint32_t)a1 << u;
          ti |= (uint32_t)t1 << u;
          na += (uint32_t)__popcll(__ballot(a1));
          nt += (uint32_t)__popcll(__ballot(t1));
        }
        uint32_t ba = 0u, bt = 0u;
        if (l == 0) {
          if (na) ba = atomicAdd(&tmp[26], na);
          if (nt) bt = atomicAdd(&tmp[27], nt);
        }
        ba = (uint32_t)__builtin_amdgcn_readfirstlane((int)ba);
        bt = (uint32_t)__builtin_amdgcn_readfirstlane((int)bt);
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          const bool a1 = (ab >> u) & 1u, t1 = (ti >> u) & 1u;
          const uint64_t ma = __ballot(a1), mt = __ballot(t1);
          if (a1) {
            const uint32_t r = ba + mbcnt64(ma);
            if (r < (uint32_t)k) {
              oi[r] = ce[u].x;
              os[r] = __int_as_float(ce[u].y);
            }
          }
          if (t1) {
            const uint32_t r = bt + mbcnt64(mt);
            if (r < (uint32_t)E) ent[r] = comp_key(__int_as_float(ce[u].y), (uint32_t)ce[u].x);
          }
          ba += (uint32_t)__popcll(ma);
          bt += (uint32_t)__popcll(mt);
        }
      }
    }
    __syncthreads();
    run_above = tmp[26];
    run_tie = tmp[27];
  }
  // lists in key order: one block-wide pass in list order, so that a
  // position in the concatenated lists orders equal scores by key
  for (int g0 = 0; g0 < (keyed ? 0 : S); g0 += NTH) {
    // offsets of the group's lists in their concatenation
    const int sg = g0 + tid;
    const uint32_t cg = sg < S ? min(cnt[(int64_t)row * S + sg], (uint32_t)cap) : 0u;
    uint32_t gtot;
    const uint32_t ex = block_scan_excl<NTH>(cg, tmp, &gtot);
    off[tid] = ex;
    if (tid == 0) off[NTH] = gtot;
    __syncthreads();
    const int ng = min(NTH, S - g0);
    for (uint32_t base = 0; base < gtot; base += NTH * PER) {
      int2 ce[PER];
      uint32_t gpos[PER];
      bool ab[PER], ti[PER];
      uint32_t na = 0, nt = 0;
      // the PER positions of a thread are consecutive: one binary search for
      // the list holding the first (the last list whose offset is <= i), a
      // forward walk for the others; then every load goes out before any is
      // used, so a step costs one load latency, not PER of them
      const uint32_t i0 = base + (uint32_t)(tid * PER);
      int lst[PER];
      {
        int lo = 0, hi = ng - 1;
        const uint32_t i = i0 < gtot ? i0 : gtot - 1;
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (off[mid] <= i) lo = mid;
          else hi = mid - 1;
        }
#pragma unroll
        for (int j = 0; j < PER; ++j) {
          while (lo + 1 < ng && off[lo + 1] <= i0 + (uint32_t)j) ++lo;
          lst[j] = lo;
        }
      }
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        const uint32_t i = i0 + (uint32_t)j;
        ce[j] = make_int2(0, 0);
        if (i < gtot) {
          const int64_t li = (int64_t)row * S + g0 + lst[j];
          const uint32_t pos = i - off[lst[j]];
          ce[j] = cand[ilv ? ilv_index(li, pos, (int64_t)nq * S) : li * cap + pos];
        }
      }
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        const uint32_t i = i0 + (uint32_t)j;
        ab[j] = ti[j] = false;
        gpos[j] = 0;
        if (i < gtot) {
          // the list position, which increases with the key index
          gpos[j] = (uint32_t)(g0 + lst[j]) * (uint32_t)cap + (i - off[lst[j]]);
          const int b = bin_of(bin_x(__int_as_float(ce[j].y), p.delta, p.c), m);
          ab[j] = b > tau;
          ti[j] = b == tau;
        }
        na += ab[j];
        nt += ti[j];
      }
      uint32_t tot;
      const uint32_t ex2 = block_scan_excl<NTH>((na << 16) | nt, tmp, &tot);
      uint32_t ra = run_above + (ex2 >> 16), rt = run_tie + (ex2 & 0xFFFFu);
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        if (ab[j] && ra < (uint32_t)k) {
          oi[ra] = ce[j].x;
          os[ra] = __int_as_float(ce[j].y);
        }
        if (ti[j] && rt < (uint32_t)E) ent[rt] = comp_key(__int_as_float(ce[j].y), gpos[j]);
        ra += ab[j];
        rt += ti[j];
      }
      run_above += tot >> 16;
      run_tie += tot & 0xFFFFu;
    }
    __syncthreads();  // off[] is rewritten by the next group
  }
  const uint32_t nent = run_tie;
  tie_ovf = nent > (uint32_t)E;
  if (tie_ovf || run_above != c_above) {
    enqueue(tie_ovf ? 2 : 4, tau, run_tie);
    return;
  }
  // the need = k - c_above best keys of bin tau, after the keys above it
  const uint32_t need = (uint32_t)k - c_above;
  const uint32_t take = min(need, nent);
  // the bin's i-th best key goes to slot c_above + i
  auto emit = [&](uint32_t i, uint64_t e) {
    const uint32_t gp = comp_pos(e);
    if (keyed) {
      oi[c_above + i] = (int32_t)gp;
      os[c_above + i] = ord_inv((uint32_t)(e >> 32));
      return;
    }
    const uint32_t s = gp / (uint32_t)cap, j = gp - s * (uint32_t)cap;
    const int2 ce = cand[((int64_t)row * S + s) * cap + j];
    oi[c_above + i] = ce.x;
    os[c_above + i] = __int_as_float(ce.y);
  };
  if (nent <= (uint32_t)kRankMax) {
    // a small bin: each key's rank is the number of keys above it (the sort
    // entries are distinct), one pass over the bin per key and no barrier
    // per sorting stage
    __syncthreads();
    for (uint32_t i = tid; i < nent; i += NTH) {
      const uint64_t e = ent[i];
      uint32_t r = 0;
      for (uint32_t j = 0; j < nent; ++j) r += ent[j] > e;
      if (r < take) emit(r, e);
    }
  } else {
    const int P = next_pow2((int)nent);
    for (int i = tid; i < P; i += NTH)
      if ((uint32_t)i >= nent) ent[i] = 0ull;
    __syncthreads();
    bitonic_sort_desc_fast<NTH>(ent, P);
    for (uint32_t i = tid; i < take; i += NTH) emit(i, ent[i]);
  }
  for (uint32_t i = c_above + take + tid; i < (uint32_t)k; i += NTH) {
    oi[i] = -1;
    os[i] = -__builtin_inff();
  }
  if (sorted) {
    // Sort the row's nout kept keys in place. Equal scores lie in one bin, and
    // within a bin the row already holds them in key order (the list order,
    // or the bin's sort), so (score, slot) is the total order; keyed rows,
    // whose keys above bin tau came in arrival order, sort by (score, key)
    // and take canonical scores from the sort entries. The slots' pairs wait
    // in the upper half of the sort buffer (k <= E / 2).
    const uint32_t nout = c_above + take;
    int2* pair = reinterpret_cast<int2*>(ent + E / 2);
    __threadfence_block();
    __syncthreads();
    for (uint32_t i = tid; i < nout; i += NTH) {
      const int32_t x = oi[i];
      const float y = os[i];
      pair[i] = make_int2(x, __float_as_int(y));
      ent[i] = comp_key(y, keyed ? (uint32_t)x : i);
    }
    const int P = next_pow2((int)nout < 1 ? 1 : (int)nout);
    for (int i = tid; i < P; i += NTH)
      if ((uint32_t)i >= nout) ent[i] = 0ull;
    __syncthreads();
    bitonic_sort_desc_fast<NTH>(ent, P);
    for (uint32_t i = tid; i < nout; i += NTH) {
      const uint32_t g = comp_pos(ent[i]);
      if (keyed) {
        oi[i] = (int32_t)g;
        os[i] = ord_inv((uint32_t)(ent[i] >> 32));
      } else {
        const int2 pr = pair[g];
        oi[i] = pr.x;
        os[i] = __int_as_float(pr.y);
      }
    }
  }
  if (stats && tid == 0) {
    int32_t* st = stats + (int64_t)row * LT_ROW_STATS;
    // a row finished by the second filter pass keeps its candidates written
    // by the first pass (field 0) and reports reason 6
    if (!(flags & kSelSecond)) st[0] = (int32_t)total_c;
    st[1] = tau;
    st[2] = (flags & kSelSecond) ? 6 : 0;
    st[3] = (int32_t)run_tie;
  }
}

// One block per row.
template <int NTH, int PER>
__global__ __launch_bounds__(NTH) void k_select(
    RowParam* params, const uint32_t* cnt, const uint32_t* hist, const int2* cand, int nq,
    int S, int HS, int cap, int m, int k, int E, uint32_t flags, int32_t* out_i, float* out_s,
    uint32_t* qctl, int32_t* queue, int32_t* rqueue, int32_t* rflag, uint64_t* pub, int32_t* stats) {
  select_row<NTH, PER>(blockIdx.x, params, cnt, hist, cand, nq, S, HS, cap, m, k, E, flags, out_i, out_s, qctl,
                       queue, rqueue, rflag, pub, stats);
}

// The rows of the second filter pass (queue rqueue, length qctl[1]);
// persistent: block b takes entries b, b + grid, ...
template <int NTH, int PER>
__global__ __launch_bounds__(NTH) void k_select_second(
    RowParam* params, const uint32_t* cnt, const uint32_t* hist, const int2* cand, int nq,
    int S, int HS, int cap, int m, int k, int E, uint32_t flags, int32_t* out_i, float* out_s,
    uint32_t* qctl, int32_t* queue, int32_t* rqueue, int32_t* rflag, int32_t* stats) {
  const uint32_t n = qctl[1];
  for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
    select_row<NTH, PER>(rqueue[i], params, cnt, hist, cand, nq, S, HS, cap, m, k, E, flags | kSelSecond, out_i,
                         out_s, qctl, queue, rqueue, rflag, nullptr, stats);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Exact fallback for the scores-in entry: the queued rows go through plain
// radix selection over all their visible scores. Persistent: block b handles
// queue entries b, b + grid, ...; the queue length is read on the device.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kSelThreads) void k_fallback_scores(
    const float* scores, int64_t stride, int nk, const int32_t* offs, const int32_t* starts, int k,
    uint32_t flags, uint32_t* qctl, const int32_t* queue, int32_t* cidx, float* cscore, int32_t* out_i,
    float* out_s) {
  extern __shared__ __align__(16) uint8_t lds[];
  __shared__ int last;
  const uint32_t n = qctl[0];
  // split mode (few rows: up to kFallbackGrid blocks over the rows' chunks,
  // no scratch rows needed), else one block per queued row
  const int chunks = fallback_chunks(n, min((int)gridDim.x, kFallbackGrid), INT_MAX, nk);
  if (chunks > 1) {
    if (blockIdx.x >= n * (uint32_t)chunks) return;  // block-uniform
    const int e = blockIdx.x / chunks, c = blockIdx.x - e * chunks;
    const int row = queue[e];
    const RowRange rr = row_range(offs, starts, row, nk);
    const int len = rr.e > rr.s ? rr.e - rr.s : 0, per = (int)(((uint32_t)len + chunks - 1) / chunks);
    const int kb = rr.s + (int)min((int64_t)c * per, (int64_t)len), ke = kb + min(per, rr.s + len - kb);
    const int64_t cb = (int64_t)e * chunks * k;
    split_fallback_select<kSelThreads>(scores + (int64_t)row * stride, rr.s, len, per, chunks, c, kb, ke, k,
                                       cidx + cb, cscore + cb, &qctl[kQctlDone + e], out_i + (int64_t)row * k,
                                       out_s + (int64_t)row * k, flags & LT_SORTED_OUTPUT, lds, &last);
    return;
  }
  for (uint32_t r = blockIdx.x; r < n; r += gridDim.x) {
    const int row = queue[r];
    const RowRange rr = row_range(offs, starts, row, nk);
    radix_select_row<kSelThreads>(scores + (int64_t)row * stride + rr.s, rr.e - rr.s, k,
                                  out_i + (int64_t)row * k, out_s + (int64_t)row * k,
                                  flags & LT_SORTED_OUTPUT, lds, rr.s);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Plain radix selection of every row (no sampling, no filtering), one block
// per row. The digits are taken over the row's own span of order keys, 12 bits
// at a time: after the least and greatest key are known, a histogram of 4096
// equal parts of the span gives the part that holds the k-th key, and that
// part is cut again until it and the keys above it fit in LDS (one histogram,
// usually), or until it is one key, whose copies are then cut by index. What
// is kept is gathered in LDS and ordered by order_entries: three passes over
// the row, the later ones from the caches.
// Bound by those passes at one block per CU and by the histogram's LDS atomics:
// 255 rows of 65501 scores, k = 2048, take 49 us, against 224 us with four
// 8-bit digits in 256-thread blocks. 512 rows of 65536, k = 2048: 94 us of
// normal scores, 101 of scores spread over 50 octaves, 172 of multiples of
// 1/8, 193 of zeros but for one in 500 (228, 271 and 813 when such rows were
// given up and done again by radix_select_row, which takes 147, 184 and 457
// from the start).
// ---------------------------------------------------------------------------
constexpr int kRadixBits = 12;
constexpr int kRadixThreads = 1024, kRadixThreadsSmall = 256;
constexpr int kRadixShort = 16384;  // keys of a row that a narrow block takes

// The block's keys row[0, n) in steps of kRadixUnroll per thread: x[u] of the
// step at i0 is key i0 + u * NTH + tid (zero past n).
template <int NTH>
struct RadixRow {
  static constexpr int U = kRadixUnroll, STEP = NTH * U;
  const float* row;  // wave-uniform
  int n;             // wave-uniform
  __device__ __forceinline__ void load(int i0, float* v) const {
    const int left = n - i0;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(row + i0), 0, left > 0 ? (int)((uint32_t)min(left, STEP) * 4u) : 0, kBufferRaw);
#pragma unroll
    for (int u = 0; u < U; ++u)
      v[u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)threadIdx.x * 4 + u * NTH * 4, 0, 0));
  }
  __device__ __forceinline__ void init(const float* r, int len) {
    const uint64_t b = (uint64_t)r;
    row = (const float*)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b) |
                         (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32)) << 32);
    n = __builtin_amdgcn_readfirstlane(len);
  }
  template <class Body>
  __device__ __forceinline__ void each(Body&& body) const {
    float a[U], b[U];
    load(0, a);
    for (int i0 = 0; i0 < n; i0 += 2 * STEP) {
      load(i0 + STEP, b);
      body(i0, a);
      load(i0 + 2 * STEP, a);
      body(i0 + STEP, b);
    }
  }
};

// LDS of the kernel: a buffer of E entries (the histogram while it is built,
// then the sort slots and buckets) and 64 words of exchange; at least what
// radix_select_row needs.
constexpr size_t kRadixExchange = 64 * 4;
static size_t radix_row_lds(int nth, int k, int E) {
  const size_t a = kRadixExchange + (size_t)E * 8, b = radix_lds_bytes(nth, k);
  return a > b ? a : b;
}

// False (nothing written, block-uniform) for the rows that it does not take.
template <int NTH>
__device__ __forceinline__ bool radix_row(const float* rowp, int n, int k, int E, int32_t* oi, float* os,
                                          uint8_t* lds) {
  constexpr int NW = NTH / kWave, U = kRadixUnroll, EPT = 12, BINS = 1 << kRadixBits, Q = BINS / NTH;
  uint32_t* tmp = reinterpret_cast<uint32_t*>(lds);  // [64]
  uint32_t* hist = reinterpret_cast<uint32_t*>(lds + kRadixExchange);
  int2* e2 = reinterpret_cast<int2*>(lds + kRadixExchange);
  const uint32_t slots = (uint32_t)sort_slots(E);
  uint32_t* bk = reinterpret_cast<uint32_t*>(e2 + slots);
  const int tid = threadIdx.x, l = lane_id(), wave = tid / kWave;
  // (the loads run up to two steps past the row's end, in 32-bit positions)
  if (n <= k || n > INT_MAX - 2 * RadixRow<NTH>::STEP) return false;
  RadixRow<NTH> rr;
  rr.init(rowp, n);
  // ---- span of the order keys ----
  uint32_t lo = 0xFFFFFFFFu, hi = 0u;
  rr.each([&](int i0, const float* x) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool v = i0 + u * NTH + tid < rr.n;
      const uint32_t o = ord_key(x[u]);
      lo = min(lo, v ? o : 0xFFFFFFFFu);
      hi = max(hi, v ? o : 0u);
    }
  });
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, kWave));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, o, kWave));
  }
  if (l == 0) {
    tmp[wave] = lo;
    tmp[NW + wave] = hi;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    lo = min(lo, tmp[w]);
    hi = max(hi, tmp[NW + w]);
  }
  // ---- the part that holds the k-th key ----
  // (the parts lie above the least key, which is not counted but left over: a
  // masked row's -inf, or the zeros of a sparse one, would all wait for one LDS
  // word, and a row whose k-th key it is ends here)
  uint32_t remaining = (uint32_t)k, above = 0, count, part = (uint32_t)n;  // part: keys in [lo, hi]
  // thread t owns Q bins, from the top (the histogram of keys) or the bottom
  uint32_t sum, tot;
  auto scan_bins = [&](const uint32_t* first, int dir) {
    sum = 0;
#pragma unroll
    for (int i = 0; i < Q; ++i) sum += first[dir * i];
    return block_scan_excl<NTH>(sum, tmp, &tot);
  };
  auto clear_bins = [&]() {
    __syncthreads();  // the exchange words and the histogram have been read
    for (int b = tid; b < BINS; b += NTH) hist[b] = 0u;
    __syncthreads();
  };
  for (;;) {
    const uint32_t low = lo + 1u, span = hi - lo;
    const int shift = span <= (uint32_t)BINS ? 0 : 32 - kRadixBits - __builtin_clz(span - 1u);
    clear_bins();
    if (span > 0)
      rr.each([&](int i0, const float* x) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const uint32_t o = ord_key(x[u]) - low;
          if ((i0 + u * NTH + tid < rr.n) & (o < span)) atomicAdd(&hist[o >> shift], 1u);
        }
      });
    __syncthreads();
    const uint32_t* own = hist + BINS - 1 - tid * Q;
    uint32_t at = scan_bins(own, -1);
    if (remaining > tot) {  // block-uniform
      above += tot;
      remaining -= tot;
      count = above + part - tot;
      break;
    }
    if (at < remaining && remaining <= at + sum) {  // one thread
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        const uint32_t c = own[-i];
        if (at < remaining && remaining <= at + c) {
          tmp[48] = (uint32_t)(BINS - 1 - (tid * Q + i));
          tmp[49] = at;
          tmp[50] = c;
        }
        at += c;
      }
    }
    __syncthreads();
    above += tmp[49];
    remaining -= tmp[49];
    part = tmp[50];
    count = above + part;
    lo = low + (tmp[48] << shift);
    if (count <= slots || shift == 0) break;
    hi = lo + ((1u << shift) - 1u);
  }
  // More keys equal to the k-th than there is room for: those of the lowest
  // indices, up to the end of the 64 (or n / 4096) that hold the last of them.
  uint32_t limit = UINT_MAX;
  if (count > slots) {
    const uint32_t last = (uint32_t)rr.n - 1u;
    const int shift = max(6, 32 - kRadixBits - __builtin_clz(last | 1u));
    clear_bins();
    rr.each([&](int i0, const float* x) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t i = (uint32_t)(i0 + u * NTH + tid);
        const uint64_t eq = __ballot((i <= last) & (ord_key(x[u]) == lo));
        if (l == 0 && eq != 0) atomicAdd(&hist[i >> shift], (uint32_t)__popcll(eq));
      }
    });
    __syncthreads();
    const uint32_t* own = hist + tid * Q;
    uint32_t at = scan_bins(own, 1);
    if (at < remaining && remaining <= at + sum) {  // one thread
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        const uint32_t c = own[i];
        if (at < remaining && remaining <= at + c) {
          tmp[48] = (uint32_t)(tid * Q + i + 1) << shift;
          tmp[49] = at + c;
        }
        at += c;
      }
    }
    __syncthreads();
    limit = tmp[48];
    count = above + tmp[49];
    if (count > slots) return false;
  }
  // ---- the keys from `lo` up ----
  const int NB = bucket_count<NTH>(count, E);
  __syncthreads();  // tmp and the histogram have been read
  for (int b = tid; b < NB; b += NTH) bk[b] = 0u;
  if (tid == 0) tmp[48] = 0u;
  __syncthreads();
  float mn = __builtin_inff(), mx = -__builtin_inff();
  auto gather = [&]<bool CUT>(int i0, const float* x) {
    uint32_t in = 0u, nin = 0u;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t o = ord_key(x[u]);
      const int i = i0 + u * NTH + tid;
      const bool i1 = (i < rr.n) & (CUT ? (o > lo) | ((o == lo) & ((uint32_t)i < limit)) : o >= lo);
      in |= (uint32_t)i1 << u;
      nin += (uint32_t)__popcll(__ballot(i1));
    }
    if (nin == 0) return;
    uint32_t r = 0u;
    if (l == 0) r = atomicAdd(&tmp[48], nin);
    r = (uint32_t)__builtin_amdgcn_readfirstlane((int)r);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool i1 = (in >> u) & 1u;
      const uint64_t mk = __ballot(i1);
      const uint32_t at = r + mbcnt64(mk);
      if (i1 & (at < slots)) {
        e2[at] = make_int2(i0 + u * NTH + tid, __float_as_int(x[u]));
        if (__builtin_isfinite(x[u])) {
          mn = fminf(mn, x[u]);
          mx = fmaxf(mx, x[u]);
        }
      }
      r += (uint32_t)__popcll(mk);
    }
  };
  if (limit == UINT_MAX) rr.each([&](int i0, const float* x) { gather.template operator()<false>(i0, x); });
  else rr.each([&](int i0, const float* x) { gather.template operator()<true>(i0, x); });
  mn = wave_min(mn);
  mx = wave_max(mx);
  float* red = reinterpret_cast<float*>(tmp);
  if (l == 0) {
    red[wave] = mn;
    red[NW + wave] = mx;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    mn = fminf(mn, red[w]);
    mx = fmaxf(mx, red[NW + w]);
  }
  order_entries<NTH, EPT>(e2, count, mn, mx, bk, NB, tmp);
  for (int i = tid; i < k; i += NTH) {
    oi[i] = e2[i].x;
    os[i] = __int_as_float(e2[i].y);
  }
  return true;
}

template <int NTH>
__global__ __launch_bounds__(NTH, 4) void k_radix(const float* scores, int64_t stride, int nk, const int32_t* offs, int k,
                                               int E, uint32_t flags, int32_t* out_i, float* out_s) {
  extern __shared__ __align__(16) uint8_t lds[];
  const int row = blockIdx.x;
  int e = offs ? offs[row] : nk;
  e = e < 0 ? 0 : (e > nk ? nk : e);
  if (radix_row<NTH>(scores + (int64_t)row * stride, e, k, E, out_i + (int64_t)row * k, out_s + (int64_t)row * k, lds))
    return;
  __syncthreads();
  radix_select_row<NTH>(scores + (int64_t)row * stride, e, k, out_i + (int64_t)row * k, out_s + (int64_t)row * k,
                        flags & LT_SORTED_OUTPUT, lds);
}

// The same by radix_select_row alone, in narrow blocks (radix_digits). It sorts
// no more than kRadixCollect keys of a digit's prefix: one pass more over such
// rows costs less (3000 rows of 4096, k = 3000: 61 us, and 332 with up to 4096
// keys sorted; 600 of 16384, k = 8192, scores around 10, 67 and 90).
constexpr int kRadixCollect = 256;
__global__ __launch_bounds__(kSelThreads) void k_radix_digits(const float* scores, int64_t stride, int nk,
                                                              const int32_t* offs, int k, int32_t* out_i,
                                                              float* out_s) {
  extern __shared__ __align__(16) uint8_t lds[];
  const int row = blockIdx.x;
  int e = offs ? offs[row] : nk;
  e = e < 0 ? 0 : (e > nk ? nk : e);
  radix_select_row<kSelThreads, kRadixCollect>(scores + (int64_t)row * stride, e, k, out_i + (int64_t)row * k,
                                               out_s + (int64_t)row * k, false, lds);
}

// The fused path's dense fallback mode, second half: queued row t (flag 1)
// was re-scored into scratch row t; one block selects it.
__global__ __launch_bounds__(kSelThreads) void k_fallback_rows(const uint32_t* qctl, const int32_t* fbflag,
                                                               const float* scratch, int nq, int nk,
                                                               const int32_t* offs, const int32_t* starts, int k,
                                                               uint32_t flags, int slots, int qt, int32_t* out_i,
                                                               float* out_s) {
  extern __shared__ __align__(16) uint8_t lds[];
  const int row = blockIdx.x;
  if (!fallback_dense(qctl[0], nq, kFallbackGrid, slots, nk, qt) || fbflag[row] != 1) return;  // block-uniform
  const RowRange rr = row_range(offs, starts, row, nk);
  radix_select_row<kSelThreads>(scratch + (int64_t)row * nk + rr.s, rr.e - rr.s, k, out_i + (int64_t)row * k,
                                out_s + (int64_t)row * k, flags & LT_SORTED_OUTPUT, lds, rr.s);
}

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------
hipError_t launch_init(uint32_t* qctl, hipStream_t st) {
  hipLaunchKernelGGL(k_init, dim3(1), dim3(64), 0, st, qctl);
  return hipGetLastError();
}

hipError_t launch_range(bool from_scores, const float* src, int64_t stride, int nq, int nk,
                        const int32_t* offs, const int32_t* starts, const int32_t* list, int ns, int m, int k,
                        RowParam* params, int32_t* stats, int32_t* rflag, uint64_t* pub, hipStream_t st) {
  dim3 grid(nq);
  auto go = [&](auto kernel, int nth) {
    hipLaunchKernelGGL(kernel, grid, dim3(nth), 0, st, src, stride, nq, nk, offs, starts, list, ns, m, k, params,
                       stats, rflag, pub);
  };
  // a long sample is read in fewer, wider steps (the kernel waits on loads);
  // so are the rows of a launch of few rows, which otherwise leaves most of
  // the GPU idle. The scores stay in registers as long as they fit (12288
  // samples of 3000 rows: 40 us, 51 us read twice), but 64 of them in 1024
  // threads take a whole CU: many rows whose list is read too (40000 samples
  // of 1500 rows, causal: 106 us held, 88 us read twice) read them twice
  const bool large = ns >= kRangeLargeSample || nq <= kSelFewRows;
  auto by_size = [&](auto FROM) {
    constexpr bool F = decltype(FROM)::value;
    if (!large && ns <= kRangeThreads * kRangeHold) go(k_range<kRangeThreads, F, kRangeHold>, kRangeThreads);
    else if (!large) go(k_range<kRangeThreads, F, 2 * kRangeHold>, kRangeThreads);
    else if (ns <= kRangeThreadsLarge * kRangeHoldFew) go(k_range<kRangeThreadsLarge, F, kRangeHoldFew>, kRangeThreadsLarge);
    else if (nq > kSelFewRows && ns <= kRangeThreadsMid * 2 * kRangeHold) go(k_range<kRangeThreadsMid, F, 2 * kRangeHold>, kRangeThreadsMid);
    else if (ns <= kRangeThreadsLarge * kRangeHold) go(k_range<kRangeThreadsLarge, F, kRangeHold>, kRangeThreadsLarge);
    else if (ns <= kRangeThreadsLarge * 2 * kRangeHold && (F || !list || nq <= kSelFewRows))
      go(k_range<kRangeThreadsLarge, F, 2 * kRangeHold>, kRangeThreadsLarge);
    else go(k_range<kRangeThreadsLarge, F, 0>, kRangeThreadsLarge);
  };
  if (from_scores) by_size(std::true_type{});
  else by_size(std::false_type{});
  return hipGetLastError();
}

hipError_t launch_filter(const float* scores, int64_t stride, int nq, int nk, const int32_t* offs,
                         const int32_t* starts, const RowParam* params, int S, int L, int cap, int m, int k,
                         uint32_t* cnt, uint32_t* hist, int2* cand, hipStream_t st) {
  auto go = [&](auto kernel, int nth) {
    hipLaunchKernelGGL(kernel, dim3(nq * S), dim3(nth), 0, st, scores, stride, nq, nk, offs, starts, params, S, L,
                       cap, m, k, cnt, hist, cand);
  };
  // 16 waves per CU: one block of 1024 threads, two of 512 or four of 256; a
  // split of at most two steps of one wave is a wave's alone, for its block's
  // barriers and empty waves cost more than its keys (unsorted: 100000 rows of
  // 256 keys 1022 us a call in blocks of 256 threads, 855 in single waves; 300
  // rows of 1024, 42 in blocks of 1024 and 36; 1200 rows of 2048, 29.7 and 32.8)
  const int units = nq * S;
  if (units == 0) return hipSuccess;
  if (L <= kFilterShort) {
    go(k_filter<kWave, 8>, kWave);
    return hipGetLastError();
  }
  auto by_len = [&](auto U) {
    constexpr int u = decltype(U)::value;
    if (units >= 1024) go(k_filter<256, u>, 256);
    else if (units >= 512) go(k_filter<512, u>, 512);
    else go(k_filter<1024, u>, 1024);
  };
  if (L >= kFilterLong) by_len(std::integral_constant<int, 16>{});
  else by_len(std::integral_constant<int, 8>{});
  return hipGetLastError();
}

size_t select_lds_bytes(int E) { return select_ent_offset(kSelThreadsWide) + (size_t)E * 8; }

hipError_t launch_select(RowParam* params, const uint32_t* cnt, const uint32_t* hist, const int2* cand, int nq,
                         int S, int HS, int cap, int m, int k, int E, uint32_t flags, int32_t* out_i, float* out_s,
                         uint32_t* qctl, int32_t* queue, int32_t* rqueue, int32_t* rflag, uint64_t* pub,
                         int32_t* stats, hipStream_t st) {
  auto go = [&](auto kernel, int nth) {
    const size_t lds = select_ent_offset(nth) + (size_t)E * 8;
    if (lds > 65536) (void)hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kernel, dim3(nq), dim3(nth), lds, st, params, cnt, hist, cand, nq, S, HS, cap, m, k, E, flags,
                       out_i, out_s, qctl, queue, rqueue, rflag, pub, stats);
  };
  // one block per row: a launch of few rows (a short chunk) fills the GPU
  // only with wide blocks, whose more loads in flight also shorten the walk
  // over the lists; many rows fill it with narrow ones. A call at 1024 and 256
  // threads: 256 rows of 65536 scores, k = 2048, sorted, 59 and 65 us; 4096 of
  // 16384, k = 100, 240 and 117. From 257 to 512 rows either may win: 512 rows
  // of 16384, k = 100, 47 and 36; but 300 queries of 65536 keys, k = 2048, no
  // sample, 892 and 1018, 300 of 100000 (inner product), k = 1000, 316 and 335,
  // and 512 rows of 131072 multiples of 1/8, k = 2048, 211 and 231
  // (and a sort buffer past 4096 entries leaves room for one block per CU)
  if ((flags & kSelIlv) || nq <= kSelFewRows || E > 4096) go(k_select<kSelThreadsWide, kSelPerWide>, kSelThreadsWide);
  else go(k_select<kSelThreads, kSelPer>, kSelThreads);
  return hipGetLastError();
}

hipError_t launch_select_second(RowParam* params, const uint32_t* cnt, const uint32_t* hist, const int2* cand,
                                int nq, int S, int HS, int cap, int m, int k, int E, uint32_t flags, int32_t* out_i,
                                float* out_s, uint32_t* qctl, int32_t* queue, int32_t* rqueue, int32_t* rflag,
                                int32_t* stats,
                                hipStream_t st) {
  const int grid = nq < kSecondSelectGrid ? nq : kSecondSelectGrid;
  if (grid == 0) return hipSuccess;
  auto go = [&](auto kernel, int nth) {
    const size_t lds = select_ent_offset(nth) + (size_t)E * 8;
    if (lds > 65536) (void)hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(nth), lds, st, params, cnt, hist, cand, nq, S, HS, cap, m, k, E,
                       flags & ~kSelRefilter, out_i, out_s, qctl, queue, rqueue, rflag, stats);
  };
  if ((flags & kSelIlv) || E > 4096) go(k_select_second<kSelThreadsWide, kSelPerWide>, kSelThreadsWide);
  else go(k_select_second<kSelThreads, kSelPer>, kSelThreads);
  return hipGetLastError();
}

hipError_t launch_fallback_scores(const float* scores, int64_t stride, int nk, const int32_t* offs,
                                  const int32_t* starts, int k, uint32_t flags, uint32_t* qctl,
                                  const int32_t* queue, int32_t* cidx, float* cscore, int32_t* out_i, float* out_s,
                                  int grid, hipStream_t st) {
  const size_t lds = radix_lds_bytes(kSelThreads, k);
  if (lds > 65536)
    (void)hipFuncSetAttribute((const void*)k_fallback_scores, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(k_fallback_scores, dim3(grid), dim3(kSelThreads), lds, st, scores,
                     stride, nk, offs, starts, k, flags, qctl, queue, cidx, cscore, out_i, out_s);
  return hipGetLastError();
}

hipError_t launch_fallback_rows(const uint32_t* qctl, const int32_t* fbflag, const float* scratch, int nq, int nk,
                                const int32_t* offs, const int32_t* starts, int k, uint32_t flags, int slots,
                                int qt, int32_t* out_i, float* out_s, hipStream_t st) {
  if (!may_dense(nq, slots, qt)) return hipSuccess;
  const size_t lds = radix_lds_bytes(kSelThreads, k);
  if (lds > 65536)
    (void)hipFuncSetAttribute((const void*)k_fallback_rows, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(k_fallback_rows, dim3(nq), dim3(kSelThreads), lds, st, qctl, fbflag, scratch, nq, nk, offs,
                     starts, k, flags, slots, qt, out_i, out_s);
  return hipGetLastError();
}

// Unsorted rows that radix_select_row takes from the start. Past k = 2048 the
// buffer that orders them leaves room for one wide block per CU, and rows that
// need no order are better off several to a CU, as long as they are short
// against that ordering. us a call, k_radix and k_radix_digits, k = 4096, normal
// scores (scores around 10): 3000 rows of 8192, 297 (298) and 78 (102); of
// 16384, 319 (318) and 135 (142); of 32768, 366 (357) and 244 (264); of 65536,
// 560 (547) and 502 (593); 512 rows of 16384, 57 (56) and 36 (40); of 32768, 65
// (64) and 64 (79); 256 rows of 16384, 28 (28) and 33 (46).
static bool radix_digits(int nq, int nk, int k) {
  return k > 2048 &&
         (nq > kSelFewRows ? nk <= 2 * kRadixShort : nq > 256 && nk <= kRadixShort);
}

hipError_t launch_radix(const float* scores, int64_t stride, int nq, int nk, const int32_t* offs,
                        int k, uint32_t flags, int32_t* out_i, float* out_s, hipStream_t st) {
  const int E = max(4096, 2 * next_pow2(k));
  if (!(flags & LT_SORTED_OUTPUT) && radix_digits(nq, nk, k)) {
    const size_t lds = radix_lds_bytes(kSelThreads, k);
    if (lds > 65536)
      (void)hipFuncSetAttribute((const void*)k_radix_digits, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(k_radix_digits, dim3(nq), dim3(kSelThreads), lds, st, scores, stride, nk, offs, k, out_i,
                       out_s);
    return hipGetLastError();
  }
  auto go = [&](auto kernel, int nth) {
    const size_t lds = radix_row_lds(nth, k, E);
    if (lds > 65536) (void)hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kernel, dim3(nq), dim3(nth), lds, st, scores, stride, nk, offs, k, E, flags, out_i, out_s);
  };
  // many short rows: narrow blocks, several per CU; their 3072 sort slots
  // serve k <= 2048
  if (nq > kSelFewRows && nk <= kRadixShort && E <= 4096)
    go(k_radix<kRadixThreadsSmall>, kRadixThreadsSmall);
  else
    go(k_radix<kRadixThreads>, kRadixThreads);
  return hipGetLastError();
}

}  // namespace lt
