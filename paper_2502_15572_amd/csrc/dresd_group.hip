// Grouping of a datastore's rows into partitions on the GPU (one-time, at
// the build of a partitioned index): a stable least-significant-digit radix
// sort of (key, row) pairs, where the key is the row's partition or the first
// token of its value (Section 3.5's next-token filter as a partitioning),
// then the partitions' starts and the slot table of the tiled layout.
//
// A pass over an 8-bit digit is three launches: counts per block of 4,096
// rows, one workgroup per digit that turns its counts into positions (the
// lower digits' totals come from one histogram of all digits, taken when the
// keys are made), and the scatter.  In the scatter a wave owns 1,024
// consecutive rows and takes them 64 at a time: lanes with equal digits find
// each other by eight ballots, so ranks need no atomics and equal keys keep
// their row order.  Digits in which all keys agree are skipped (the host
// reads the histogram once).
//
// What bounds it: the strided read of the first tokens, the scattered 8-byte
// writes and a dozen launches.  4,194,304 rows by first token: 0.26 ms of
// kernels (keys 46 us, two passes 90 and 47 us, distinct tokens 24 us, slots
// 53 us), against 200 ms for the read-back and host sort it replaces.
#include "dresd_device.h"
#include "dresd_ops.h"

namespace dresd {

namespace {

constexpr int kGT = 256;                       // threads per workgroup
constexpr int kGRounds = 16;                   // rows per thread
constexpr int kGTile = kGroupTile;             // rows per workgroup
constexpr int kGWaves = kGT / kWaveSize;
static_assert(kGT * kGRounds == kGTile, "tile");

__device__ __forceinline__ uint32_t wave_scan_incl(uint32_t v, int lane) {
#pragma unroll
  for (int off = 1; off < kWaveSize; off <<= 1) {
    const uint32_t o = __shfl_up(v, off, kWaveSize);
    if (lane >= off) v += o;
  }
  return v;
}

// Keys of all rows, and the histogram of each of their four digits.  By
// token (cont set): the first token, its sign bit turned over so that
// unsigned order is token order.  Else the assignment; *bad is set when one
// lies outside [0, P).
__global__ void __launch_bounds__(kGT) dresd_group_keys(GroupParams p) {
  __shared__ uint32_t h[4][256];
  const int tid = threadIdx.x, lane = tid & 63;
  for (int i = tid; i < 1024; i += kGT) (&h[0][0])[i] = 0;
  __syncthreads();
  bool bad = false;
  const int64_t step = (int64_t)gridDim.x * kGT;
  for (int64_t i0 = (int64_t)blockIdx.x * kGT; i0 < p.n; i0 += step) {
    const int64_t i = i0 + tid;
    const bool in = i < p.n;
    uint32_t key = 0;
    if (in) {
      if (p.cont) {
        key = (uint32_t)p.cont[i * p.L] ^ 0x80000000u;
      } else {
        const int32_t a = p.assign[i];
        bad |= a < 0 || a >= p.P;
        key = (uint32_t)a;
      }
      p.key[0][i] = key;
    }
    const uint64_t act = __ballot(in);
    if (act == 0) continue;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const uint32_t v = (key >> (8 * d)) & 255u;
      // high digits mostly agree: one lane then adds for the wave
      const int lead = __ffsll((long long)act) - 1;
      const uint32_t v0 = __builtin_amdgcn_readlane(v, lead);
      if (__ballot(in && v == v0) == act) {
        if (lane == lead) atomicAdd(&h[d][v0], (uint32_t)__popcll(act));
      } else if (in) {
        atomicAdd(&h[d][v], 1u);
      }
    }
  }
  if (__syncthreads_or(bad) && tid == 0) *p.bad = 1;
  for (int i = tid; i < 1024; i += kGT)
    if ((&h[0][0])[i]) atomicAdd(p.hist + i, (&h[0][0])[i]);
}

// counts[digit][block] of one pass.
__global__ void __launch_bounds__(kGT) dresd_group_count(GroupParams p) {
  __shared__ uint32_t h[256];
  const int tid = threadIdx.x;
  h[tid] = 0;
  __syncthreads();
  const int64_t b0 = (int64_t)blockIdx.x * kGTile;
#pragma unroll
  for (int r = 0; r < kGRounds; ++r) {
    const int64_t i = b0 + r * kGT + tid;
    if (i < p.n) atomicAdd(&h[(p.key[p.src][i] >> p.shift) & 255u], 1u);
  }
  __syncthreads();
  p.counts[(int64_t)tid * p.nblk + blockIdx.x] = h[tid];
}

// One workgroup per digit: exclusive positions of its blocks' runs, after
// all rows of lower digits.
__global__ void __launch_bounds__(kGT) dresd_group_scan(GroupParams p) {
  __shared__ uint32_t part[kGWaves];
  __shared__ uint32_t carry;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, dg = blockIdx.x;
  // rows of lower digits
  uint32_t v = tid < dg ? p.hist[(p.shift / 8) * 256 + tid] : 0;
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWaveSize);
  if (lane == 0) part[w] = v;
  __syncthreads();
  if (tid == 0) {
    uint32_t s = 0;
    for (int i = 0; i < kGWaves; ++i) s += part[i];
    carry = s;
  }
  __syncthreads();
  uint32_t *row = p.counts + (int64_t)dg * p.nblk;
  for (int64_t b = 0; b < p.nblk; b += kGT) {
    const uint32_t c = b + tid < p.nblk ? row[b + tid] : 0;
    const uint32_t incl = wave_scan_incl(c, lane);
    if (lane == kWaveSize - 1) part[w] = incl;
    __syncthreads();
    uint32_t base = carry;
    for (int i = 0; i < w; ++i) base += part[i];
    if (b + tid < p.nblk) row[b + tid] = base + incl - c;
    __syncthreads();
    if (tid == kGT - 1) carry = base + incl;
    __syncthreads();
  }
}

// Stable scatter of one pass.
__global__ void __launch_bounds__(kGT) dresd_group_scatter(GroupParams p) {
  __shared__ uint32_t wh[kGWaves][256];  // per wave: rows seen of each digit, then its base
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int i = lane; i < 256; i += kWaveSize) wh[w][i] = 0;
  wave_sync_lds();
  const int64_t w0 = (int64_t)blockIdx.x * kGTile + w * (kWaveSize * kGRounds);
  const uint32_t *src = p.key[p.src];
  uint32_t key[kGRounds], rank[kGRounds];
#pragma unroll
  for (int r = 0; r < kGRounds; ++r) {
    const int64_t i = w0 + r * kWaveSize + lane;
    key[r] = i < p.n ? src[i] : 0u;
  }
#pragma unroll
  for (int r = 0; r < kGRounds; ++r) {
    const bool in = w0 + r * kWaveSize + lane < p.n;
    const uint32_t dg = (key[r] >> p.shift) & 255u;
    uint64_t same = __ballot(in);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bool bit = (dg >> b) & 1u;
      const uint64_t m = __ballot(bit);
      same &= bit ? m : ~m;
    }
    // (a lane past the end is in no other lane's set and writes nothing)
    const uint32_t before = (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
    const uint32_t seen = wh[w][dg];
    wave_sync_lds();
    rank[r] = seen + before;
    if (in && before == 0) wh[w][dg] = seen + (uint32_t)__popcll(same);
    wave_sync_lds();
  }
  __syncthreads();
  {
    uint32_t base = p.counts[(int64_t)tid * p.nblk + blockIdx.x];
#pragma unroll
    for (int i = 0; i < kGWaves; ++i) {
      const uint32_t c = wh[i][tid];
      wh[i][tid] = base;
      base += c;
    }
  }
  __syncthreads();
  const int to = p.src ^ 1;
#pragma unroll
  for (int r = 0; r < kGRounds; ++r) {
    const int64_t i = w0 + r * kWaveSize + lane;
    if (i < p.n) {
      const uint32_t at = wh[w][(key[r] >> p.shift) & 255u] + rank[r];
      p.key[to][at] = key[r];
      p.row[to][at] = p.first ? (uint32_t)i : p.row[p.src][i];
    }
  }
}

// Distinct keys of the sorted sequence.  Pass 1: first occurrences per block.
__global__ void __launch_bounds__(kGT) dresd_group_heads(GroupParams p) {
  __shared__ uint32_t part[kGWaves];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const uint32_t *key = p.key[p.src];
  const int64_t b0 = (int64_t)blockIdx.x * kGTile;
  uint32_t c = 0;
#pragma unroll
  for (int r = 0; r < kGRounds; ++r) {
    const int64_t i = b0 + r * kGT + tid;
    if (i < p.n) c += (uint32_t)(i == 0 || key[i] != key[i - 1]);
  }
  for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, kWaveSize);
  if (lane == 0) part[w] = c;
  __syncthreads();
  if (tid == 0) {
    uint32_t s = 0;
    for (int i = 0; i < kGWaves; ++i) s += part[i];
    p.counts[blockIdx.x] = s;
  }
}

// Pass 2 (one workgroup): their positions, and how many there are.
__global__ void __launch_bounds__(kGT) dresd_group_heads_scan(GroupParams p) {
  __shared__ uint32_t part[kGWaves];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  uint32_t carry = 0;
  for (int64_t b = 0; b < p.nblk; b += kGT) {
    const uint32_t c = b + tid < p.nblk ? p.counts[b + tid] : 0;
    const uint32_t incl = wave_scan_incl(c, lane);
    if (lane == kWaveSize - 1) part[w] = incl;
    __syncthreads();
    uint32_t base = carry;
    for (int i = 0; i < w; ++i) base += part[i];
    if (b + tid < p.nblk) p.counts[b + tid] = base + incl - c;
    for (int i = 0; i < kGWaves; ++i) carry += part[i];
    __syncthreads();
  }
  if (tid == 0) *p.distinct = carry;
}

// Pass 3: start[j] and token of the j-th distinct key.
__global__ void __launch_bounds__(kGT) dresd_group_starts(GroupParams p) {
  __shared__ uint32_t part[kGWaves];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const uint32_t *key = p.key[p.src];
  const int64_t b0 = (int64_t)blockIdx.x * kGTile;
  uint32_t carry = p.counts[blockIdx.x];
  for (int r = 0; r < kGRounds; ++r) {
    const int64_t i = b0 + r * kGT + tid;
    const bool head = i < p.n && (i == 0 || key[i] != key[i - 1]);
    const uint64_t mk = __ballot(head);
    if (lane == 0) part[w] = (uint32_t)__popcll(mk);
    __syncthreads();
    uint32_t at = carry;
    for (int q = 0; q < w; ++q) at += part[q];
    at += (uint32_t)__popcll(mk & ((1ull << lane) - 1ull));
    if (head) {
      p.start[at] = (uint32_t)i;
      p.tok[at] = (int32_t)(key[i] ^ 0x80000000u);
    }
    for (int q = 0; q < kGWaves; ++q) carry += part[q];
    __syncthreads();
  }
  if (blockIdx.x == 0 && tid == 0) p.start[*p.distinct] = (uint32_t)p.n;
}

// start[q] of partition q in [0, P]: the first sorted position with a key of
// at least q (empty partitions start where the next one does).
__global__ void __launch_bounds__(kGT) dresd_group_bounds(GroupParams p) {
  const int64_t q = (int64_t)blockIdx.x * kGT + threadIdx.x;
  if (q > p.P) return;
  const uint32_t *key = p.key[p.src];
  int64_t lo = 0, hi = p.n;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if ((int64_t)key[mid] < q) lo = mid + 1;
    else hi = mid;
  }
  p.start[q] = (uint32_t)lo;
}

// Slot table: one thread per slot.  Tile t belongs to the last partition
// whose first tile is <= t (empty partitions have none); its slots take that
// partition's rows in order, the rest of its last tile is padding.
__global__ void __launch_bounds__(kGT) dresd_group_slots(GroupParams p) {
  for (int64_t s = (int64_t)blockIdx.x * kGT + threadIdx.x; s < p.nslot;
       s += (int64_t)gridDim.x * kGT) {
    const int32_t t = (int32_t)(s / kTileRows);
    int32_t lo = 0, hi = p.P;  // part_tile[lo] <= t < part_tile[hi]
    while (hi - lo > 1) {
      const int32_t mid = (int32_t)(((int64_t)lo + hi) >> 1);
      if (p.part_tile[mid] <= t) lo = mid;
      else hi = mid;
    }
    const int64_t at = (int64_t)p.start[lo] + (s - (int64_t)p.part_tile[lo] * kTileRows);
    const bool pad = at >= (int64_t)p.start[lo + 1];
    const uint32_t row = pad ? kPadRow : p.row[p.src][at];
    p.slot_row[s] = row;
    p.ftok_slot[s] = pad ? 0 : p.by_token ? (int32_t)(p.key[p.src][at] ^ 0x80000000u)
                                          : p.values[(int64_t)row * p.L];
  }
}

__global__ void __launch_bounds__(kGT) dresd_group_iota(int32_t *out, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * kGT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kGT)
    out[i] = (int32_t)i;
}

// (a kernel and not a memset: also the flag and the count)
__global__ void __launch_bounds__(kGT) dresd_group_clear(GroupParams p) {
  for (int i = threadIdx.x; i < 1024; i += kGT) p.hist[i] = 0;
  if (threadIdx.x == 0) {
    *p.bad = 0;
    *p.distinct = 0;
  }
}

hipError_t go(const void *f, int64_t blocks, GroupParams &p, hipStream_t st) {
  void *args[] = {&p};
  return hipLaunchKernel(f, dim3((unsigned)blocks), dim3(kGT), args, 0, st);
}

int64_t some(int64_t work) {
  const int64_t b = (work + kGT - 1) / kGT;
  return b < 1 ? 1 : b < 16384 ? b : 16384;
}

}  // namespace

hipError_t launch_group_keys(GroupParams &p, hipStream_t st) {
  hipError_t e = go((const void *)dresd_group_clear, 1, p, st);
  const int64_t b = some(p.n);
  if (e == hipSuccess) e = go((const void *)dresd_group_keys, b < 512 ? b : 512, p, st);
  return e;
}

hipError_t launch_group_pass(GroupParams &p, int digit, bool first, hipStream_t st) {
  p.shift = 8 * digit;
  p.first = first ? 1 : 0;
  hipError_t e = go((const void *)dresd_group_count, p.nblk, p, st);
  if (e == hipSuccess) e = go((const void *)dresd_group_scan, 256, p, st);
  if (e == hipSuccess) e = go((const void *)dresd_group_scatter, p.nblk, p, st);
  p.src ^= 1;
  return e;
}

hipError_t launch_group_distinct(GroupParams &p, hipStream_t st) {
  hipError_t e = go((const void *)dresd_group_heads, p.nblk, p, st);
  if (e == hipSuccess) e = go((const void *)dresd_group_heads_scan, 1, p, st);
  if (e == hipSuccess) e = go((const void *)dresd_group_starts, p.nblk, p, st);
  return e;
}

hipError_t launch_group_bounds(GroupParams &p, hipStream_t st) {
  return go((const void *)dresd_group_bounds, ((int64_t)p.P + 1 + kGT - 1) / kGT, p, st);
}

hipError_t launch_group_slots(GroupParams &p, hipStream_t st) {
  return go((const void *)dresd_group_slots, some(p.nslot), p, st);
}

hipError_t launch_iota(int32_t *out, int64_t n, hipStream_t st) {
  void *args[] = {&out, &n};
  return hipLaunchKernel((const void *)dresd_group_iota, dim3((unsigned)some(n)), dim3(kGT), args,
                         0, st);
}

}  // namespace dresd
