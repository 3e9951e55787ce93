// One-time copy of an index's rows into the scans' layout (dresd_layout) and
// of the first tokens of its values into a column (dresd_first_tokens).
//
// Layout: a wave writes one tile (16 rows, KB blocks of 1 KiB) at a time, lane
// c the 16-byte chunk c of every block: row c % 16, so a lane looks its row up
// once per tile and then walks along it, four blocks in flight.  Rows are read
// with the widest loads that their pitch allows (16, 4 or one element's
// bytes).  What bounds it: HBM, one read and one write of the keys; in the
// partitioned layout the rows are gathered, whole rows of at least 64 bytes.
// The tiles are stored past the caches: 8.6 GB of dirty lines made the first
// search after a build wait 90 us for their way out.
// Measured: 4,194,304 x 128 f16 rows gathered by first token 0.98 -> 0.42 ms
// (5.2 TB/s read and written) against one chunk per thread with element loads.
#include "dresd_device.h"
#include "dresd_ops.h"

namespace dresd {

namespace {

// The 16 bytes of one chunk: dims [dim, dim + EPC) of `row`, zero past d.  VB:
// bytes per load.
template <typename T, int VB>
__device__ __forceinline__ u4 row_chunk(const T *row, int dim, int d) {
  constexpr int EPC = 16 / sizeof(T);
  if constexpr (VB == 16) {
    // d is a multiple of EPC here: a chunk lies inside the row or past it
    return dim < d ? *reinterpret_cast<const u4 *>(row + dim) : u4{0, 0, 0, 0};
  } else if constexpr (VB == 4) {
    constexpr int EPV = 4 / sizeof(T);  // d is a multiple of it
    u4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      v[i] = dim + i * EPV < d ? *reinterpret_cast<const uint32_t *>(row + dim + i * EPV) : 0u;
    return v;
  } else {
    union {
      T e[EPC];
      u4 v;
    } u;
#pragma unroll
    for (int e = 0; e < EPC; ++e) u.e[e] = dim + e < d ? row[dim + e] : T(0);
    return u.v;
  }
}

template <typename T, int VB>
__global__ void __launch_bounds__(256) dresd_layout(LayoutParams p) {
  constexpr int EPC = 16 / sizeof(T);  // elements per 16-byte chunk
  const T *src = static_cast<const T *>(p.src);
  const int lane = threadIdx.x & 63;
  const int64_t nw = (int64_t)gridDim.x * (blockDim.x >> 6);
  const int d = p.d, KB = p.KB;
  for (int64_t t = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); t < p.tiles;
       t += nw) {
    int64_t row = t * kTileRows + (lane & 15);
    if (p.slot_row) {  // partitioned layout: the slot's row, or padding
      const uint32_t r = p.slot_row[row];
      row = r == kPadRow ? p.N : (int64_t)r;
    }
    const bool in = row < p.N;
    const T *s = src + (in ? row : 0) * d;
    const int dim0 = (lane >> 4) * EPC;
    u4 *dst = static_cast<u4 *>(p.dst) + t * KB * 64 + lane;
    const int dl = in ? d : 0;
    int kb = 0;
    for (; kb + 4 <= KB; kb += 4) {
      u4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = row_chunk<T, VB>(s, (kb + u) * 4 * EPC + dim0, dl);
#pragma unroll
      for (int u = 0; u < 4; ++u) __builtin_nontemporal_store(v[u], dst + (int64_t)(kb + u) * 64);
    }
    for (; kb < KB; ++kb)
      __builtin_nontemporal_store(row_chunk<T, VB>(s, kb * 4 * EPC + dim0, dl), dst + (int64_t)kb * 64);
  }
}

// out[i] = cont[i][0] for rows below n, zero for the slots past them.
__global__ void __launch_bounds__(256) dresd_first_tokens(const int32_t *cont, int L, int64_t n,
                                                          int64_t nslot, int32_t *out) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < nslot;
       i += (int64_t)gridDim.x * blockDim.x)
    out[i] = i < n ? cont[i * L] : 0;
}

template <typename T>
const void *layout_kernel(const LayoutParams &p) {
  const size_t pitch = (size_t)p.d * sizeof(T);
  const size_t align = (uintptr_t)p.src | pitch;
  if (align % 16 == 0) return (const void *)dresd_layout<T, 16>;
  if (align % 4 == 0) return (const void *)dresd_layout<T, 4>;
  return (const void *)dresd_layout<T, (int)sizeof(T)>;
}

}  // namespace

hipError_t launch_layout(const LayoutParams &pin, int dtype, int cus, hipStream_t st) {
  LayoutParams p = pin;
  const int64_t want = (p.tiles + 3) / 4, most = (int64_t)cus * 32;
  void *args[] = {&p};
  return hipLaunchKernel(dtype == kF32 ? layout_kernel<float>(p) : layout_kernel<uint16_t>(p),
                         dim3((unsigned)(want < most ? want : most)), dim3(256), args, 0, st);
}

hipError_t launch_first_tokens(const int32_t *cont, int L, int64_t n, int64_t nslot, int32_t *out,
                               hipStream_t st) {
  const int64_t want = (nslot + 255) / 256;
  const unsigned blocks = (unsigned)(want < 65536 ? want : 65536);
  hipLaunchKernelGGL(dresd_first_tokens, dim3(blocks), dim3(256), 0, st, cont, L, n, nslot, out);
  return hipGetLastError();
}

}  // namespace dresd
