// gfx950 draft assembly for batch verification (DReSD Section 3.6): the
// retrieved continuations become the rows of a [r, length] draft matrix
// padded with the EOS id.  A draft is the first `length` tokens of a
// continuation with every token after its first EOS replaced by EOS; drafts
// that start with EOS (nothing to propose) and repeats of an earlier draft
// are dropped, and the first r remaining drafts, in rank order, fill the rows.
//
// One workgroup (1024 threads) per query.  What bounds it is latency: one read
// of the tokens, then LDS.  The tokens are staged in LDS (up to 48 KiB of them;
// beyond that they are read where they are), one thread per retrieved rank
// hashes its draft and finds its end, T adjacent threads per rank (as many as
// the workgroup has) compare the hash with those of all earlier ranks (exact
// comparison on a hash match), a workgroup prefix sum over the kept flags
// gives every kept draft its row, and its T threads write it.  k = 100, L = 10:
// 5.4 us (18.1 with one thread per rank and the tokens in global memory).
#include "dresd_device.h"
#include "dresd_ops.h"

namespace dresd {

namespace {

constexpr int kDraftThreads = 1024;
constexpr int kDraftStage = 12288;  // tokens staged in LDS

template <bool STAGED>
__global__ void __launch_bounds__(kDraftThreads) dresd_pack(DraftParams p) {
  extern __shared__ int32_t stage[];
  __shared__ uint64_t hash[DRESD_K_MAX_INTERNAL];
  __shared__ uint16_t len[DRESD_K_MAX_INTERNAL];  // tokens before the first EOS
  __shared__ uint32_t wsum[kDraftThreads / kWaveSize];
  const int b = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int k = p.k, L = p.L, length = p.length;
  const int32_t *src = p.tokens + (size_t)b * k * L;
  if constexpr (STAGED) {
    for (int e = tid; e < k * L; e += kDraftThreads) stage[e] = src[e];
    __syncthreads();
  }
  auto token = [&](int i, int j) -> int32_t {
    if constexpr (STAGED) return stage[i * L + j];
    else return src[(size_t)i * L + j];
  };

  // 1. hash of the normalised draft (64-bit FNV-1a over the tokens up to and
  //    with the first EOS: what follows is EOS) and its length
  if (tid < k) {
    uint64_t h = 1469598103934665603ull;
    int n = 0;
    for (; n < length; ++n) {
      const int32_t x = token(tid, n);
      h = (h ^ (uint32_t)x) * 1099511628211ull;
      if (x == p.eos) break;
    }
    hash[tid] = h;
    len[tid] = (uint16_t)n;
  }
  __syncthreads();

  // 2. drop empty drafts and repeats of an earlier one (exact check on equal
  //    hash); threads T i .. T i + T - 1 share rank i
  int T = 1;
  while (T < kWaveSize && k * 2 * T <= kDraftThreads) T <<= 1;
  const int i = tid / T, sub = tid & (T - 1);
  bool dup = false;
  const int n = i < k ? len[i] : 0;
  if (n > 0) {
    const uint64_t h = hash[i];
#pragma unroll 4
    for (int j = sub; j < i; j += T) {
      if (hash[j] != h || len[j] != n || dup) continue;
      bool same = true;
      for (int c = 0; c < n && same; ++c) same = token(i, c) == token(j, c);
      dup = same;
    }
  }
  int any = dup;
  for (int o = 1; o < T; o <<= 1) any |= __shfl_xor(any, o, kWaveSize);
  const bool keep = n > 0 && !any;

  // 3. row of each kept draft: workgroup prefix sum of the kept flags
  const uint64_t m = __ballot(keep && sub == 0);
  // (all T threads of a rank count the ranks before it)
  const uint32_t before = __popcll(m & ((1ull << (lane & ~(T - 1))) - 1ull));
  if (lane == 0) wsum[wid] = (uint32_t)__popcll(m);
  __syncthreads();
  uint32_t base = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kDraftThreads / kWaveSize; ++w) {
    const uint32_t c = wsum[w];
    if (w < wid) base += c;
    total += c;
  }
  const uint32_t row = base + before;
  int32_t *out = p.drafts + (size_t)b * p.r * length;
  if (keep && row < (uint32_t)p.r)
    for (int j = sub; j < length; j += T)
      out[(size_t)row * length + j] = j < n ? token(i, j) : p.eos;
  // 4. rows past the kept drafts are all EOS
  const int rows = total < (uint32_t)p.r ? (int)total : p.r;
  for (int e = rows * length + tid; e < p.r * length; e += kDraftThreads) out[e] = p.eos;
  if (tid == 0) p.count[b] = rows;
}

}  // namespace

hipError_t launch_pack_drafts(const DraftParams &p, hipStream_t st) {
  if (p.B == 0) return hipSuccess;
  DraftParams q = p;
  void *args[] = {&q};
  const int64_t tokens = (int64_t)p.k * p.L;
  const bool staged = tokens <= kDraftStage;
  return hipLaunchKernel(staged ? (const void *)dresd_pack<true> : (const void *)dresd_pack<false>,
                         dim3((unsigned)p.B), dim3(kDraftThreads), args,
                         staged ? (size_t)tokens * 4 : 0, st);
}

}  // namespace dresd
