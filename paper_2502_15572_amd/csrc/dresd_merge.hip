// gfx950 merge + gather kernel: one workgroup per query turns the scan's
// per-wave candidate lists into the exact k best keys of that query
// (DReSD Section 3.5, Eq. 3 taken as top-k for batch verification,
// Section 3.6), then gathers the winners' continuations -- the value map of
// the key -> next-tokens datastore.  For a sampled pass it instead emits the
// k-th best key, a lower bound that prunes the next pass.
//
// Latency matters more than throughput here (one short kernel per pass), so
// every step is one round of independent loads followed by a few barriers:
// list summaries, then all listed keys at once (8 lanes per 8 keys of a kept
// list, so no thread searches for its key), and radix selections that start
// at the highest bit where the keys differ.  The bound over the lists' best
// keys stops after two digits, or later where that would keep more than twice
// the lists that the exact k-th best would (and 64 more): opening a few lists
// more costs less than another digit's barriers.  Empty lists take no part in
// it: their key, 0, would make the highest differing bit the sign, and two
// digits would end at steps of 0.004 for scores in [0.5, 1).
// Measured, against one key per thread found by binary search and an exact
// bound: 13 queries, k = 30, 768 lists 18 -> 10 us; one query, k = 100, 4,096
// lists of 64 keys 24 -> 20 us.  Searches over tight clusters, with the bound
// over all lists after two digits and as it is now: 262,144 x 64 fp32 keys, k =
// 100, two queries 124 -> 41 us, with the next-token filter 130 -> 35; one query
// grouped by first token over 4,194,304 x 128 f16 keys 59 -> 30.
#include "dresd_device.h"
#include "dresd_ops.h"

namespace dresd {

// Candidate counts up to this are ordered whole (no selection first).
constexpr int kSmallMerge = 256;
// Winner counts up to this are ordered by rank, larger ones by a bitonic
// network over the workgroup.
constexpr int kRankSortMax = 512;
// Each thread looks at this many lists.
constexpr int kListsPerThread = kMergeLists / kMergeThreads;
// Work items of the gather (8, 16 or 64 keys of a kept list each) held in LDS.
constexpr uint32_t kMergeItems = kMergeLists;
static_assert(kMergeLists <= 4096, "items of 8 keys of all lists (at most 2,048 each) fit 21 bits");

struct MergeShared {
  uint32_t hist[kMergeItems];  // radix histogram (256 bins); the gather's work items
  alignas(16) uint64_t cache[kMergeCap];
  alignas(16) uint64_t win[DRESD_K_MAX_INTERNAL];
  uint64_t sel_prefix, sel_mask, bound, v_and, v_or, items;
  uint32_t sel_krem, sel_done, win_cnt, ncand, known;
};

__device__ inline uint64_t wave_and(uint64_t v) {
  for (int off = 32; off > 0; off >>= 1) v &= __shfl_xor(v, off, kWaveSize);
  return v;
}
__device__ inline uint64_t wave_or(uint64_t v) {
  for (int off = 32; off > 0; off >>= 1) v |= __shfl_xor(v, off, kWaveSize);
  return v;
}
__device__ inline uint64_t wave_max(uint64_t v) {
  for (int off = 32; off > 0; off >>= 1) {
    const uint64_t o = __shfl_xor(v, off, kWaveSize);
    v = o > v ? o : v;
  }
  return v;
}

typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));

// Descending order of n distinct keys src[0..n) (every key names its own
// row): key i goes to dst[number of keys greater than it] when that is below
// `keep`.  T adjacent lanes (a power of two, as many as the workgroup allows
// up to a wave) share a key's count, so every wave takes part; keys are read
// as LDS broadcasts and there is no barrier inside.  src and dst are 16-byte
// aligned LDS arrays; src is not written.
__device__ inline void rank_sort_desc(const uint64_t *src, uint32_t n, uint64_t *dst,
                                      uint32_t keep, int tid, int nth) {
  int T = 1;
  while (T < kWaveSize && n * (uint32_t)(2 * T) <= (uint32_t)nth) T <<= 1;
  const int sub = tid & (T - 1);
  const uint32_t per = (uint32_t)(nth / T), n2 = n & ~1u;
  for (uint32_t i0 = 0; i0 < n; i0 += per) {
    const uint32_t i = i0 + (uint32_t)(tid / T);
    const bool valid = i < n;
    const uint64_t x = valid ? src[i] : ~0ull;
    uint32_t r = 0;
#pragma unroll 4
    for (uint32_t j = 2u * (uint32_t)sub; j < n2; j += 2u * (uint32_t)T) {
      const u64x2 v = *reinterpret_cast<const u64x2 *>(src + j);
      r += (uint32_t)(v.x > x) + (uint32_t)(v.y > x);
    }
    if ((n & 1u) && sub == 0) r += (uint32_t)(src[n - 1] > x);
    for (int o = 1; o < T; o <<= 1) r += __shfl_xor(r, o, kWaveSize);
    if (valid && sub == 0 && r < keep) dst[r] = x;
  }
}

// Largest value v such that at least kk of the nonzero values among the M
// values src(i) are >= v (1 <= kk <= their number; the kk-th largest value, or a
// lower boundary of the digit bin holding exactly the kk largest values).
// Radix selection 8 bits at a time from the highest bit in which the values
// differ: every thread adds its values to the 256-bin histogram, then one wave
// finds the bin holding the kk-th largest (and clears the histogram), two
// barriers per digit.
// Called by the whole workgroup.  After `digits` digits it also stops at the
// lower boundary of a bin at or above which no more than kk + slack values lie.
template <class Src>
__device__ uint64_t radix_kth(MergeShared &sh, Src src, uint32_t M, uint32_t kk,
                              int digits = 8, uint32_t slack = 0) {
  constexpr int kDigit = 8, kBins = 1 << kDigit, kBinsPerLane = kBins / kWaveSize;
  const int tid = threadIdx.x, nth = blockDim.x;
  const int lane = tid & (kWaveSize - 1), wid = tid / kWaveSize;
  if (tid == 0) {
    sh.v_and = ~0ull;
    sh.v_or = 0ull;
    sh.sel_done = 0u;
  }
  if (tid < kBins) sh.hist[tid] = 0;
  __syncthreads();
  uint64_t va = ~0ull, vo = 0ull;
  for (uint32_t i = tid; i < M; i += nth) {
    const uint64_t key = src(i);
    va &= key ? key : ~0ull;
    vo |= key;
  }
  va = wave_and(va);
  vo = wave_or(vo);
  if (lane == 0) {
    atomicAnd((unsigned long long *)&sh.v_and, (unsigned long long)va);
    atomicOr((unsigned long long *)&sh.v_or, (unsigned long long)vo);
  }
  __syncthreads();
  const uint64_t diff = sh.v_and ^ sh.v_or;
  if (diff == 0) return sh.v_or;  // one distinct value
  int top = 63 - __clzll((long long)diff);
  uint64_t pm = (top == 63) ? 0ull : ~((2ull << top) - 1ull);  // bits fixed so far
  uint64_t pre = sh.v_and & pm;                                 // their values
  uint32_t krem = kk;  // rank of the answer among the values matching pre
  // Every thread follows the same (pre, pm, top, krem), published by wave 0.
  for (;;) {
    const int w = top + 1 < kDigit ? top + 1 : kDigit;
    const int s = top + 1 - w;
    const uint32_t wmask = (1u << w) - 1u;
    for (uint32_t i = tid; i < M; i += nth) {
      const uint64_t key = src(i);
      if (key && (key & pm) == pre) atomicAdd(&sh.hist[(uint32_t)(key >> s) & wmask], 1u);
    }
    __syncthreads();
    if (wid == 0) {
      // lane l owns bins [kBinsPerLane l, kBinsPerLane (l + 1)); count the
      // values in the bins of all higher lanes
      uint32_t h[kBinsPerLane], mine = 0;
#pragma unroll
      for (int j = 0; j < kBinsPerLane; ++j) {
        h[j] = sh.hist[lane * kBinsPerLane + j];
        mine += h[j];
      }
      uint32_t incl = mine;
      for (int off = 1; off < kWaveSize; off <<= 1) {
        const uint32_t v = __shfl_down(incl, off, kWaveSize);
        if (lane + off < kWaveSize) incl += v;
      }
      const uint32_t cnt_above = incl - mine;
      if (cnt_above < krem && krem <= cnt_above + mine) {
        uint32_t cum = cnt_above;
        for (int j = kBinsPerLane - 1; j >= 0; --j) {
          if (cum + h[j] >= krem) {
            const uint32_t dg = (uint32_t)(lane * kBinsPerLane + j);
            sh.sel_prefix = pre | ((uint64_t)dg << s);
            sh.sel_mask = pm | ((uint64_t)wmask << s);
            sh.sel_krem = krem - cum;
            // the whole bin is in, or few enough values too many
            sh.sel_done = h[j] <= krem - cum + (digits <= 1 ? slack : 0u) ? 1u : 0u;
            break;
          }
          cum += h[j];
        }
      }
#pragma unroll
      for (int j = 0; j < kBinsPerLane; ++j) sh.hist[lane * kBinsPerLane + j] = 0;
    }
    __syncthreads();
    pre = sh.sel_prefix;
    pm = sh.sel_mask;
    krem = sh.sel_krem;
    top = s - 1;
    --digits;
    if (sh.sel_done || top < 0) break;
    // wave 0 rewrites the state only after the next histogram's barrier,
    // which every thread reaches after reading it
  }
  return pre;
}

// Output of one query from its sorted winners win[0..kk): the k-th best key
// (sampled pass) or indices, scores and gathered continuations (final pass).
// Each thread issues all of its continuation loads before its first store,
// so the gather costs one memory latency rather than one per token.  A
// winner that names no row of the value table (only an upstream fault could
// produce one) is written as index -1, score -inf and zero tokens instead of
// being dereferenced.
__device__ inline void write_result(const MergeParams &p, int b, const uint64_t *win,
                                    uint32_t kk, int tid, int nth) {
  if (!p.final_mode) {
    // The k-th best key of any subset of the rows is a lower bound of the
    // k-th best of all of them; a pass that found fewer than k keys at or
    // above its (speculative) threshold keeps the bound it started from.
    // The speculative key for the next pass is the spec_rank-th best found,
    // never below the bound.
    if (tid == 0) {
      const uint64_t fb = p.tau_fb ? p.tau_fb[b] : 0ull;
      uint64_t v = (kk >= (uint32_t)p.k) ? win[p.k - 1] : 0ull;
      v = v > fb ? v : fb;
      p.tau_out[b] = v;
      if (p.spec_out) {
        const uint64_t s = (kk >= (uint32_t)p.spec_rank) ? win[p.spec_rank - 1] : 0ull;
        p.spec_out[b] = s > v ? s : v;
      }
    }
    return;
  }
  for (int r = tid; r < p.k; r += nth) {
    const size_t o = (size_t)b * p.k + r;
    const uint32_t row = r < (int)kk ? ~(uint32_t)win[r] : 0xFFFFFFFFu;
    if ((int64_t)row < p.N) {
      p.idx[o] = (int64_t)row;
      p.score[o] = order_value((uint32_t)(win[r] >> 32));
    } else {  // past the candidates (cannot happen when N >= k), or no row
      p.idx[o] = -1;
      p.score[o] = -__builtin_inff();
    }
  }
  if (p.tokens) {
    constexpr int R = 8;  // tokens per thread per round, loaded together
    const int L = p.L, n = p.k * L;
    int32_t *out = p.tokens + (size_t)b * p.k * L;
    for (int i0 = tid; i0 < n; i0 += R * nth) {
      int32_t v[R];
#pragma unroll
      for (int u = 0; u < R; ++u) {
        const int i = i0 + u * nth;
        const int r = i / L;
        v[u] = 0;
        if (i < n && r < (int)kk) {
          const uint32_t row = ~(uint32_t)win[r];
          if ((int64_t)row < p.N) v[u] = p.cont[(size_t)row * L + (i - r * L)];
        }
      }
#pragma unroll
      for (int u = 0; u < R; ++u)
        if (i0 + u * nth < n) out[i0 + u * nth] = v[u];
    }
  }
}

// 1. A lower bound on the query's k-th best key: the larger of (a) the best
//    k-th key published by any list holding k sorted keys and (b) the k-th
//    largest of the lists' known best keys -- k distinct listed keys reach
//    each, and the answer is among the listed keys.
// 2. Candidates: listed keys at or above the bound; lists whose best key is
//    below it are not opened.  All kept lists' keys are loaded at once.
// 3. The k best candidates: ordered by rank when few, else a radix select
//    finds the k-th and the keys at or above it are ordered.
__global__ void __launch_bounds__(kMergeThreads) dresd_merge(MergeParams p) {
  __shared__ MergeShared sh;
  const int b = blockIdx.x;
  const int tid = threadIdx.x;
  const int nth = blockDim.x;
  const int lane = tid & (kWaveSize - 1), wid = tid / kWaveSize;
  const int G = p.G;
  const uint32_t *lcnt = p.lcnt + (size_t)b * G;
  const uint64_t *lkth = p.lkth + (size_t)b * G;
  const uint64_t *lfirst = p.lfirst + (size_t)b * G;
  const uint64_t *lists = p.lists + (size_t)b * G * p.C;
  uint64_t *spill = p.spill + (size_t)b * p.spill_cap;
  if (tid == 0) {
    sh.bound = 0;
    sh.ncand = 0;
    sh.win_cnt = 0;
    sh.known = 0;
    sh.items = 0;
  }
  __syncthreads();
  // Thread t looks at lists t, t + 1024, ...
  uint32_t cnt[kListsPerThread];
  uint64_t first[kListsPerThread];
  uint64_t mb = 0;
  uint32_t known = 0;  // non-empty lists of the wave whose best key is known
#pragma unroll
  for (int j = 0; j < kListsPerThread; ++j) {
    const int w = tid + j * kMergeThreads;
    cnt[j] = 0;
    first[j] = 0;
    if (w < G) {
      cnt[j] = min(lcnt[w] & ~kSortedFlag, (uint32_t)p.C);
      first[j] = lfirst[w];
      const uint64_t v = lkth[w];
      mb = v > mb ? v : mb;
    }
  }
#pragma unroll
  for (int j = 0; j < kListsPerThread; ++j) {
    const int w = tid + j * kMergeThreads;
    const uint64_t f = first[j] == ~0ull ? 0ull : first[j];
    if (w < G) sh.cache[w] = f;
    known += (uint32_t)__popcll(__ballot(f != 0ull));
  }
  mb = wave_max(mb);
  if (lane == 0 && mb) atomicMax((unsigned long long *)&sh.bound, (unsigned long long)mb);
  if (lane == 0 && known) atomicAdd(&sh.known, known);
  __syncthreads();
  // (b), where that many best keys are known
  if (sh.known >= (uint32_t)p.k) {
    const uint64_t t1 = radix_kth(sh, [&](uint32_t i) { return sh.cache[i]; }, (uint32_t)G,
                                  (uint32_t)p.k, 2, (uint32_t)p.k + 64u);
    if (tid == 0 && t1 > sh.bound) sh.bound = t1;
  }
  __syncthreads();
  const uint64_t bnd = sh.bound;

  // 2. work items: 8 keys of a kept list (one whose best key reaches the
  //    bound) for 8 lanes, so that short lists fill the loads too; 16 keys, or 64
  //    for a wave, where smaller items would be too many.  In any order, eight
  //    rounds of the workgroup in flight.
  uint64_t items = 0;  // of 8, 16 and 64 keys, 21 bits each
#pragma unroll
  for (int j = 0; j < kListsPerThread; ++j) {
    if (first[j] < bnd) cnt[j] = 0;
    items += (uint64_t)((cnt[j] + 7u) / 8u) | (uint64_t)((cnt[j] + 15u) / 16u) << 21 |
             (uint64_t)((cnt[j] + 63u) / 64u) << 42;
  }
  uint64_t incl = items;
  for (int off = 1; off < kWaveSize; off <<= 1) {
    const uint64_t v = __shfl_up(incl, off, kWaveSize);
    if (lane >= off) incl += v;
  }
  uint64_t base = 0;
  if (lane == kWaveSize - 1 && incl)
    base = atomicAdd((unsigned long long *)&sh.items, (unsigned long long)incl);
  base = __shfl(base, kWaveSize - 1, kWaveSize) + incl - items;
  __syncthreads();
  const uint64_t all = sh.items;
  const int level = ((uint32_t)all & 0x1fffffu) <= kMergeItems ? 0
                    : ((uint32_t)(all >> 21) & 0x1fffffu) <= kMergeItems ? 1 : 2;
  const uint32_t total = (uint32_t)(all >> (21 * level)) & 0x1fffffu;
  const int lg = level == 0 ? 3 : level == 1 ? 4 : 6;  // keys per item, as a power of two
  const uint32_t per = 1u << lg;
  if (total <= kMergeItems) {
    uint32_t at = (uint32_t)(base >> (21 * level)) & 0x1fffffu;
#pragma unroll
    for (int j = 0; j < kListsPerThread; ++j)
      for (uint32_t c = 0; c < cnt[j]; c += per, ++at)
        // list (12 bits), item of it (8), keys of the item - 1 (6)
        sh.hist[at] = (uint32_t)(tid + j * kMergeThreads) | (c >> lg) << 12 |
                      (min(cnt[j] - c, per) - 1u) << 20;
  }
  __syncthreads();
  // a key at or above the bound becomes a candidate
  auto offer = [&](uint64_t key) {
    const bool take = key >= bnd && key != 0ull;
    const uint64_t mk = __ballot(take);
    if (!mk) return;
    uint32_t at = 0;
    if (lane == 0) at = atomicAdd(&sh.ncand, (uint32_t)__popcll(mk));
    at = __builtin_amdgcn_readfirstlane(at) + (uint32_t)__popcll(mk & ((1ull << lane) - 1ull));
    if (take) {
      if (at < (uint32_t)kMergeCap) sh.cache[at] = key;
      else if ((int64_t)(at - kMergeCap) < p.spill_cap) spill[at - kMergeCap] = key;
    }
  };
  constexpr uint32_t NW = kMergeThreads / kWaveSize;
  if (total <= kMergeItems) {
    constexpr int R = 8;
    const uint32_t round = (uint32_t)kMergeThreads >> lg;  // items of one round
    const uint32_t mine = (uint32_t)tid >> lg, e = (uint32_t)tid & (per - 1u);
    // (whole waves stay together: the loop bound is the workgroup's)
    for (uint32_t i0 = 0; i0 < total; i0 += R * round) {
      uint64_t key[R];
#pragma unroll
      for (int u = 0; u < R; ++u) {
        const uint32_t i = i0 + (uint32_t)u * round + mine;
        key[u] = 0ull;
        if (i < total) {
          const uint32_t it = sh.hist[i];
          if (e <= it >> 20)
            key[u] = lists[(size_t)(it & 4095u) * p.C + (((it >> 12) & 255u) << lg) + e];
        }
      }
#pragma unroll
      for (int u = 0; u < R; ++u) offer(key[u]);
    }
  } else {  // more keys than items fit: every list in turn
    for (int w = wid; w < G; w += (int)NW) {
      if (lfirst[w] < bnd) continue;
      const uint32_t n = min(lcnt[w] & ~kSortedFlag, (uint32_t)p.C);
      for (uint32_t c = 0; c < n; c += kWaveSize)
        offer(c + (uint32_t)lane < n ? lists[(size_t)w * p.C + c + lane] : 0ull);
    }
  }
  // Winner slots start empty (key 0 names no row), so that a slot no key
  // reaches is written as a missing result rather than as stale LDS.
  for (int i = tid; i < p.k; i += nth) sh.win[i] = 0ull;
  __threadfence_block();
  __syncthreads();
  const uint32_t M = sh.ncand;
  const uint32_t kk = M < (uint32_t)p.k ? M : (uint32_t)p.k;

  // 3. the k best
  if (M <= (uint32_t)kSmallMerge) {
    rank_sort_desc(sh.cache, M, sh.win, kk, tid, nth);
    __syncthreads();
    write_result(p, b, sh.win, kk, tid, nth);
    return;
  }
  auto cand = [&](uint32_t i) {
    return i < (uint32_t)kMergeCap ? sh.cache[i] : spill[i - kMergeCap];
  };
  const uint64_t cut = (kk == M) ? 0ull : radix_kth(sh, cand, M, kk);
  for (uint32_t i = tid; i < M; i += nth) {
    const uint64_t key = cand(i);
    if (key >= cut) {
      const uint32_t at = atomicAdd(&sh.win_cnt, 1u);
      if (at < (uint32_t)DRESD_K_MAX_INTERNAL) sh.win[at] = key;
    }
  }
  __syncthreads();
  if (kk <= (uint32_t)kRankSortMax) {  // the winners, ordered into the free cache
    for (uint32_t i = tid; i < kk; i += nth) sh.cache[i] = 0ull;
    __syncthreads();
    rank_sort_desc(sh.win, kk, sh.cache, kk, tid, nth);
    __syncthreads();
    write_result(p, b, sh.cache, kk, tid, nth);
    return;
  }
  int n = 1;
  while (n < (int)kk) n <<= 1;
  for (int i = (int)kk + tid; i < n; i += nth) sh.win[i] = 0ull;
  __syncthreads();
  block_bitonic_desc(sh.win, n);
  write_result(p, b, sh.win, kk, tid, nth);
}

void *merge_kernel_ptr() { return (void *)dresd_merge; }

}  // namespace dresd
