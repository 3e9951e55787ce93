// gfx950 assignment step of spherical k-means on the 16-bit matrix cores: the
// contraction of dresd_kmeans_assign (dresd_kmeans.hip) for rows of at most
// 256 dims.  The fp32 matrix cores run 16x slower than the 16-bit ones, so
// the fp32 centroids are split into three 16-bit parts that sum to them and
// every product is formed exactly:
//   f16 keys : hi, mid, lo in f16 of the centroid scaled by a power of two
//              that brings its largest element to [2^14, 2^15) (all three
//              parts at one scale, so one accumulator takes them; what is cut
//              off is at most 2^-25 there: 2^-39 of the largest element); 3
//              products.
//   bf16 keys: hi, mid, lo in bf16 (8 + 8 + 8 bits: the fp32 centroid); 3
//              products.
//   fp32 keys: rows split the same way; the six products of parts whose
//              orders of magnitude add up to more than 2^-24 (the other
//              three are below 2^-26 of the product).
// The sums stay in fp32, in d / 32 x 3 (or 6) steps instead of d / 4: the
// error against 64-bit sums is smaller than the fp32 contraction's.
//
// What bounds it: the matrix cores (6 n d P flops for 16-bit keys).  Rows stay
// in registers (a wave holds RT tiles of 16 rows, all dims), centroids stream
// through an LDS ring shared by the workgroup's 4 waves, so a 1 KiB LDS read
// feeds RT matrix instructions; the argmax of 16 centroids x 16 rows is six
// VALU instructions per lane, and only a wave with a new best does more.
// Measured on 524,288 x 128 rows against 8,192
// centroids: 2.23 ms for f16 and bf16 rows, 4.04 ms for fp32 rows (1.48 and 1.63
// PFLOP/s of 16-bit products), against 15.2 ms on the fp32 matrix cores.
//
// Rows or centroids that the split does not represent (non-finite values,
// fp32 beyond bf16's rounding range, centroids of vanishing size) are left to
// the fp32 contraction: a row without a finite best score is marked with id
// -1, and dresd_kmeans_assign then computes the marked rows.
#include "dresd_device.h"
#include "dresd_ops.h"
#include "dresd_split.h"

namespace dresd {

namespace {

constexpr int kAT = 16;          // centroids per tile
constexpr int kAPad = 64;        // centroids are padded to whole groups of 64
constexpr int kAWaves = 4;

template <int DT>
__device__ __forceinline__ f4 mfma16(u4 a, u4 b, f4 acc) {
  if constexpr (DT == kF16)
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, a),
                                                  __builtin_bit_cast(h8, b), acc, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8, a),
                                                   __builtin_bit_cast(b8, b), acc, 0, 0, 0);
}

// Centroid operands: one workgroup per tile of 16 centroids, 16 threads per
// centroid.  Writes [tile][block of 32 dims][part][64 lanes] 16-byte chunks
// (lane (g, m): centroid m, dims 8 g .. + 8 of the block), the factor that
// takes a centroid's scores back to their scale (+inf past P: 0 * inf is NaN,
// which wins no comparison) and whether the tile holds a centroid that the
// split does not represent.  Also clears the packed results of a split search.
template <bool F16>
__global__ void __launch_bounds__(256) dresd_assign_operand(AssignParams p) {
  __shared__ float mx[kAT][17];
  __shared__ int bad;
  const int tid = threadIdx.x, tile = blockIdx.x;
  const int m = tid >> 4, j = tid & 15;
  const int c = tile * kAT + m, d = p.d;
  const float *src = p.centroids + (int64_t)c * d;
  if (tid == 0) bad = 0;
  float v = 0.f;
  bool fin = true;
  if (c < p.P)
    for (int k = j; k < d; k += 16) {
      const float a = fabsf(src[k]);
      fin = fin && a < __builtin_inff();  // false for NaN as well
      v = fmaxf(v, a);
    }
  mx[m][j] = fin ? v : __builtin_inff();
  __syncthreads();
  v = mx[m][0];
#pragma unroll
  for (int i = 1; i < 16; ++i) v = fmaxf(v, mx[m][i]);
  // representable: zero, or a largest element in [2^-60, 2^120)
  const bool ok = v == 0.f || (v >= 0x1p-60f && v < 0x1p120f);
  if (!ok) bad = 1;
  int e = 0;  // scale 2^e
  if (F16 && ok && v > 0.f) e = 14 - (int)((__float_as_uint(v) >> 23) - 127u);
  const float up = __uint_as_float((uint32_t)(127 + e) << 23);
  const float down = __uint_as_float((uint32_t)(127 - e) << 23);
  if (j == 0) p.scale[c] = c < p.P ? down : __builtin_inff();
  uint16_t *dst = static_cast<uint16_t *>(p.op) + (int64_t)tile * p.KB * 3 * 512;
  for (int k = j * 8; k < p.KB * 32; k += 128) {
    us8 part[3];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float x = (ok && c < p.P && k + i < d) ? src[k + i] * up : 0.f;
      uint16_t a, b, l;
      split3<F16>(x, a, b, l);
      part[0][i] = a;
      part[1][i] = b;
      part[2][i] = l;
    }
    const int kb = k >> 5, g = (k >> 3) & 3;
#pragma unroll
    for (int q = 0; q < 3; ++q)
      *reinterpret_cast<us8 *>(dst + ((int64_t)(kb * 3 + q) * 64 + g * 16 + m) * 8) = part[q];
  }
  __syncthreads();
  if (tid == 0) p.special[tile] = bad;
  if (p.packed)
    for (int64_t i = (int64_t)tile * 256 + tid; i < p.n; i += (int64_t)gridDim.x * 256)
      p.packed[i] = 0ull;
}

// Shape of a variant: KB blocks of 32 dims; XP parts per row (1, or 3 for
// fp32 rows).  RT row tiles per wave (at most 32 chunks of 16 bytes, 24 for
// fp32 rows whose parts take three), TS centroid tiles per ring stage.
template <int DT, int KB>
struct AssignShape {
  static constexpr int XP = DT == kF32 ? 3 : 1;
  static constexpr int RT = DT == kF32 ? (KB <= 1 ? 8 : KB <= 2 ? 4 : KB <= 4 ? 2 : 1)
                                       : (KB <= 4 ? 8 : 4);
  static constexpr int TS = KB == 1 ? 4 : KB == 2 ? 2 : 1;
  static constexpr int NB = TS * KB * 3;                     // blocks per stage
  static constexpr int CPW = (NB + kAWaves - 1) / kAWaves;   // copies per wave and stage
  static constexpr int S = KB <= 4 ? 4 : 3;                  // ring stages
  static constexpr int kStage = CPW * kAWaves * kBlockBytes + 256;  // blocks, then 64 scales
  static constexpr int ROWS = kAWaves * RT * 16;
};

template <int DT, int KB>
__global__ void __launch_bounds__(256, 2) dresd_assign_split(AssignParams p) {
  using Sh = AssignShape<DT, KB>;
  constexpr int RT = Sh::RT, TS = Sh::TS, S = Sh::S, CPW = Sh::CPW, XP = Sh::XP;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, m = lane & 15;
  const int64_t r0 = (int64_t)blockIdx.x * Sh::ROWS + wv * (RT * 16);
  const int d = p.d;
  const int ntile = p.ppad / kAT;

  // A centroid that the split does not hold: every row goes to the fp32 path.
  int any = 0;
  for (int i = tid; i < ntile; i += 256) any |= p.special[i];
  if (__syncthreads_or(any)) {
    if (blockIdx.y == 0 && lane < 16)
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        const int64_t row = r0 + r * 16 + lane;
        if (row < p.n) p.assign[row] = -1;
      }
    if (p.packed && lane < 16)
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        const int64_t row = r0 + r * 16 + lane;
        if (row < p.n) p.packed[row] = ~0ull;
      }
    return;
  }

  // Rows: lane (g, m) holds dims 8 g .. + 8 of every block of row m of every tile.
  u4 x[RT][KB * XP];
  uint32_t tiny = 0;  // fp32 rows: bit r, row m of tile r is nonzero and below 2^-100
  {
    const int es = DT == kF32 ? 4 : 2;
    const bool vec = (((uintptr_t)p.x & 15u) == 0) && ((int64_t)d * es) % 16 == 0;
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      const int64_t row = r0 + r * 16 + m;
      const bool in = row < p.n;
      float big = 0.f;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const int k = kb * 32 + g * 8;
        if constexpr (DT == kF32) {
          float v[8];
          const float *src = static_cast<const float *>(p.x) + (in ? row : 0) * d;
          if (in && vec && k + 8 <= d) {
            const float4 lo = *reinterpret_cast<const float4 *>(src + k);
            const float4 hi = *reinterpret_cast<const float4 *>(src + k + 4);
            v[0] = lo.x, v[1] = lo.y, v[2] = lo.z, v[3] = lo.w;
            v[4] = hi.x, v[5] = hi.y, v[6] = hi.z, v[7] = hi.w;
          } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = (in && k + i < d) ? src[k + i] : 0.f;
          }
          us8 part[3];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            uint16_t a, b, c;
            split3<false>(v[i], a, b, c);
            part[0][i] = a;
            part[1][i] = b;
            part[2][i] = c;
            big = fmaxf(big, fabsf(v[i]));
          }
#pragma unroll
          for (int q = 0; q < 3; ++q) x[r][kb * 3 + q] = __builtin_bit_cast(u4, part[q]);
        } else {
          const uint16_t *src = static_cast<const uint16_t *>(p.x) + (in ? row : 0) * d;
          if (in && vec && k + 8 <= d) {
            x[r][kb] = *reinterpret_cast<const u4 *>(src + k);
          } else {
            us8 v;
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = (in && k + i < d) ? src[k + i] : (uint16_t)0;
            x[r][kb] = __builtin_bit_cast(u4, v);
          }
        }
      }
      if constexpr (DT == kF32) {
        big = fmaxf(big, __shfl_xor(big, 16, kWaveSize));
        big = fmaxf(big, __shfl_xor(big, 32, kWaveSize));
        if (big > 0.f && big < 0x1p-100f) tiny |= 1u << r;
      }
    }
  }
  // Wait for the rows here: left to the compiler, the wait lands at their
  // first use inside the loop, where it would drain the copy ring each time.
  asm volatile("" : : : "memory");
  __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);

  const int nst = ntile / TS;  // whole: ppad is a multiple of 64 centroids
  const int s0 = (int)((int64_t)nst * blockIdx.y / gridDim.y);
  const int s1 = (int)((int64_t)nst * (blockIdx.y + 1) / gridDim.y);
  const uint32_t ring = (uint32_t)(uintptr_t)smem;
  const unsigned char *op = static_cast<const unsigned char *>(p.op);
  // Copies of stage s into slot s mod S: this wave's CPW blocks (the last
  // block again past the stage) and the stage's scales (all four waves the
  // same).  Past the last stage the last one is read again, so that every
  // stage issues the same number of copies.
  auto issue = [&](int s, int slot) {
    s = s < s1 ? s : s1 - 1;
    const unsigned char *src = op + (int64_t)s * Sh::NB * kBlockBytes;
    const uint32_t base = ring + (uint32_t)slot * Sh::kStage;
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
      const int b = wv * CPW + i;
      const int bb = b < Sh::NB ? b : Sh::NB - 1;
      copy16_to_lds(src, (uint32_t)(bb * kBlockBytes + lane * 16),
                        base + (uint32_t)(b * kBlockBytes));
    }
    // (64 floats from the stage's first centroid; the array ends 64 past ppad)
    copy1_to_lds(p.scale + (int64_t)s * (TS * kAT) + lane,
                 base + (uint32_t)(CPW * kAWaves * kBlockBytes));
  };
  float best[RT];
  int bid[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    best[r] = -__builtin_inff();
    bid[r] = -1;
  }
#pragma unroll
  for (int i = 0; i < S - 1; ++i) issue(s0 + i, i);
  int slot = 0;
#pragma unroll 1
  for (int s = s0; s < s1; ++s) {
    wait_vmcnt<(S - 2) * (CPW + 1)>();  // this wave's copies of stage s have landed
    __syncthreads();                    // everyone's have, and stage s - 1 is read
    issue(s + S - 1, slot == 0 ? S - 1 : slot - 1);
    const unsigned char *st = smem + (size_t)slot * Sh::kStage;
    const float *scl = reinterpret_cast<const float *>(st + CPW * kAWaves * kBlockBytes);
#pragma unroll
    for (int t = 0; t < TS; ++t) {
      const u4 *blk = reinterpret_cast<const u4 *>(st + (size_t)t * KB * 3 * kBlockBytes) + lane;
      f4 acc[RT];
#pragma unroll
      for (int r = 0; r < RT; ++r) acc[r] = f4{0.f, 0.f, 0.f, 0.f};
      // Smallest products first, so that only the last KB sums (of the high
      // parts) round at the scores' own magnitude.  fp32 rows: part q of the
      // centroid meets the row's parts 0 .. 2 - q.
      auto multiply = [&](int q, int h0, int h1) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
          const u4 c = blk[(kb * 3 + q) * 64];
#pragma unroll
          for (int h = h0; h >= h1; --h)
#pragma unroll
            for (int r = 0; r < RT; ++r)
              acc[r] = mfma16<DT == kF16 ? kF16 : kBF16>(c, x[r][kb * XP + h], acc[r]);
        }
      };
      multiply(2, 0, 0);
      if constexpr (XP == 3) {
        multiply(1, 1, 0);
        multiply(0, 2, 1);
      } else {
        multiply(1, 0, 0);
      }
      multiply(0, 0, 0);
      // D layout: lane (g, m), register i -> centroid 4 g + i, row m.
      const float4 sc = *reinterpret_cast<const float4 *>(scl + t * kAT + g * 4);
      const int c0 = (s * TS + t) * kAT + g * 4;
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        const float v0 = acc[r][0] * sc.x, v1 = acc[r][1] * sc.y, v2 = acc[r][2] * sc.z,
                    v3 = acc[r][3] * sc.w;
        const float mx = fmaxf(fmaxf(fmaxf(v0, v1), v2), v3);
        if (__ballot(mx > best[r])) {
          const int i = v0 == mx ? 0 : v1 == mx ? 1 : v2 == mx ? 2 : 3;
          const bool up = mx > best[r];
          bid[r] = up ? c0 + i : bid[r];
          best[r] = up ? mx : best[r];
        }
      }
    }
    slot = slot == S - 1 ? 0 : slot + 1;
  }
  wait_vmcnt<0>();  // no LDS copy may land after the workgroup ends

  // The four lane groups hold the same 16 rows.
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    float b = best[r];
    int id = bid[r];
#pragma unroll
    for (int off = 16; off < 64; off <<= 1) {
      const float ob = __shfl_xor(b, off, kWaveSize);
      const int oid = __shfl_xor(id, off, kWaveSize);
      if (ob > b || (ob == b && (uint32_t)oid < (uint32_t)id)) {
        b = ob;
        id = oid;
      }
    }
    const int64_t row = r0 + r * 16 + m;
    // fp32 rows lose lower parts where their elements or scores vanish (bf16
    // ends at 2^-133, a score of size 2^-80 has parts down to 2^-104): left to fp32
    const bool fine = id >= 0 && fabsf(b) < __builtin_inff() &&
                      (DT != kF32 || (!((tiny >> r) & 1u) && (b == 0.f || fabsf(b) >= 0x1p-80f)));
    if (g == (r & 3) && row < p.n) {
      if (p.packed) {
        atomicMax(reinterpret_cast<unsigned long long *>(p.packed + row),
                  (unsigned long long)(fine ? make_key(b, (uint32_t)id) : ~0ull));
      } else {
        p.assign[row] = fine ? id : -1;
        if (p.score) p.score[row] = b;
      }
    }
  }
}

template <int DT, int KB>
hipError_t launch_split(AssignParams &p, hipStream_t st) {
  using Sh = AssignShape<DT, KB>;
  const int64_t rows = (p.n + Sh::ROWS - 1) / Sh::ROWS;
  constexpr size_t lds = (size_t)Sh::S * Sh::kStage;
  static_assert(lds <= 81920, "two workgroups per CU");
  void *args[] = {&p};
  if (lds > 65536)
    (void)hipFuncSetAttribute((const void *)dresd_assign_split<DT, KB>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  return hipLaunchKernel((const void *)dresd_assign_split<DT, KB>,
                         dim3((unsigned)rows, (unsigned)p.splits), dim3(256), args, lds, st);
}

template <int DT>
int rows_per_wg(int KB) {
  return KB == 1 ? AssignShape<DT, 1>::ROWS : KB == 2 ? AssignShape<DT, 2>::ROWS
       : KB == 3 ? AssignShape<DT, 3>::ROWS : KB == 4 ? AssignShape<DT, 4>::ROWS
       : KB == 6 ? AssignShape<DT, 6>::ROWS : AssignShape<DT, 8>::ROWS;
}

template <int DT>
hipError_t launch_dt(AssignParams &p, hipStream_t st) {
  switch (p.KB) {
    case 1: return launch_split<DT, 1>(p, st);
    case 2: return launch_split<DT, 2>(p, st);
    case 3: return launch_split<DT, 3>(p, st);
    case 4: return launch_split<DT, 4>(p, st);
    case 6: return launch_split<DT, 6>(p, st);
    default: return launch_split<DT, 8>(p, st);
  }
}

}  // namespace

bool assign_split_plan(int64_t n, int d, int dtype, int P, int cus, AssignParams *out) {
  AssignParams &p = *out;
  p = AssignParams{};
  const int kb = (d + 31) / 32;
  if (kb > 8) return false;  // rows wider than a wave's registers hold
  p.KB = kb <= 4 ? kb : kb <= 6 ? 6 : 8;
  const int64_t ppad = ((int64_t)P + kAPad - 1) / kAPad * kAPad;
  const int64_t op = ppad * p.KB * 32 * 6;
  if (op > kAssignMaxOperand) return false;
  p.ppad = (int)ppad;
  p.n = n;
  p.d = d;
  p.dtype = dtype;
  p.P = P;
  const int rows = dtype == kF32 ? rows_per_wg<kF32>(p.KB)
                   : dtype == kF16 ? rows_per_wg<kF16>(p.KB) : rows_per_wg<kBF16>(p.KB);
  // Two workgroups per CU run at once.  Fewer than four such rounds of row
  // blocks leave CUs idle (or a last round nearly empty): the centroids are
  // then split over workgroups too, at least one 64-centroid group each.
  const int64_t wgs = (n + rows - 1) / rows;
  int64_t splits = wgs >= 8LL * cus ? 1 : (8LL * cus + wgs - 1) / wgs;
  const int64_t most = ppad / kAPad;
  splits = splits < most ? splits : most;
  p.splits = (int)(splits < 1 ? 1 : splits);
  auto up = [](int64_t b) { return (b + 255) / 256 * 256; };
  p.off_scale = up(op);
  p.off_special = p.off_scale + up((ppad + 64) * 4);
  p.off_packed = p.off_special + up(ppad / kAT * 4);
  p.bytes = p.off_packed + (p.splits > 1 ? up(n * 8) : 0);
  return true;
}

hipError_t launch_assign_split(AssignParams &p, void *ws, hipStream_t st) {
  unsigned char *b = static_cast<unsigned char *>(ws);
  p.op = b;
  p.scale = reinterpret_cast<float *>(b + p.off_scale);
  p.special = reinterpret_cast<int32_t *>(b + p.off_special);
  p.packed = p.splits > 1 ? reinterpret_cast<uint64_t *>(b + p.off_packed) : nullptr;
  void *args[] = {&p};
  hipError_t e = hipLaunchKernel(
      p.dtype == kF16 ? (const void *)dresd_assign_operand<true>
                      : (const void *)dresd_assign_operand<false>,
      dim3((unsigned)(p.ppad / kAT)), dim3(256), args, 0, st);
  if (e != hipSuccess) return e;
  if (p.dtype == kF32) return launch_dt<kF32>(p, st);
  if (p.dtype == kF16) return launch_dt<kF16>(p, st);
  return launch_dt<kBF16>(p, st);
}

}  // namespace dresd
