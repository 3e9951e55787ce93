// gfx950 projection of datastore-sized batches (Algorithm 1 steps 4-6, see
// dresd_transform.hip) on the 16-bit matrix cores, which run 16x faster than
// the fp32 ones: z-scored inputs and weights are split into three bf16 parts
// each (8 + 8 + 8 bits: the fp32 value), and of the nine products the six
// whose parts reach 2^-24 of the whole are formed (the others are below
// 2^-26).  The products of the two high parts have an accumulator of their own:
// it rounds D / 32 times at the result's magnitude, not D / 4 times as the
// fp32 contraction, and the error against 64 bits is about half of that one's.
//
// A workgroup computes 256 rows (8 waves of 32) x NT tiles of 16 columns.
// Weights come as ready operands (dresd_project_operand, once per call)
// through a two-stage LDS ring shared by the waves; every wave copies its own
// rows of x into a three-stage ring (they come from HBM and need the longer
// lead), 16 bytes per lane where rows are 16-byte aligned and 4 elsewhere,
// with the 16-byte pieces of a row swapped by its number so that the reads
// of 16 rows spread over the banks.  Each wave z-scores and splits its rows
// once for all columns.  Few row blocks split D over workgroups, as in
// dresd_transform.hip.  Up to 128 columns without such a split, the
// workgroup holds whole rows and normalises them itself.
//
// What bounds it: the matrix cores (12 M D l flops; at l <= 32 HBM).
// Measured: 65,536 x 4,096 -> 128 in 0.38-0.46 ms (0.9-1.1 PFLOP/s of bf16
// products; 0.86-0.92 ms on the fp32 matrix cores), -> 32 in 0.21 ms (5.1 TB/s; 0.45 ms), 8,192
// rows -> 1,024 in 0.48 ms (0.81 ms).  Back to back the clock falls under the
// matrix load (0.34 ms for a launch on its own).
//
// What the split does not hold (values that are not finite or past bf16's
// rounding range, rows so small beside the weights that lower parts are lost,
// weights of such sizes) shows in a row's sum of squares: the workgroup that
// holds the row computes it again on the fp32 matrix cores, for its columns
// and its slice of D.  65,536 x 4,096 -> 128 with 65 / 6,553 / all rows in
// doubt: 0.53 / 0.78 / 1.96 ms (the whole batch in fp32 0.93 ms; each wave one
// of its rows after another 3.4 / 21 / 65 ms).
#include "dresd_device.h"
#include "dresd_ops.h"
#include "dresd_split.h"

namespace dresd {

namespace {

constexpr int kPWaves = 8, kPRows = 32 * kPWaves;  // rows per workgroup
constexpr int kXWave = 32 * 128 + 256;  // a wave's rows of a 32-dim block, its means and factors

// Weight operands [group][block of 32 dims][tile][part][64 lanes] x 16 bytes
// (lane (g, m): column m of the tile, dims 8 g .. + 8; zero past D and l), and
// per block of dims 32 means and 32 factors 1 / sqrt(var + eps_z) (Eq. 1;
// zero past D), and per workgroup the largest size of its weights (infinity
// where one is not finite).  One wave per (tile, block).
__global__ void __launch_bounds__(256) dresd_project_operand(ProjectParams p) {
  __shared__ float top[4];
  const int lane = threadIdx.x & 63, g = lane >> 4, m = lane & 15;
  const int tiles = p.groups * p.NT;
  const int64_t last = (int64_t)tiles * p.KB - 1, mine = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int64_t i = mine < last ? mine : last;  // (waves past the end write the last one again)
  const int kb = (int)(i / tiles), tile = (int)(i - (int64_t)kb * tiles);
  const int c = tile * 16 + m;
  us8 part[3];
  float big = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int k = kb * 32 + g * 8 + e;
    const float x = (k < p.t.D && c < p.t.l) ? p.t.W[(int64_t)k * p.t.l + c] : 0.f;
    big = fabsf(x) <= big ? big : x == x ? fabsf(x) : __builtin_inff();
    uint16_t a, b, l;
    split3<false>(x, a, b, l);
    part[0][e] = a;
    part[1][e] = b;
    part[2][e] = l;
  }
#pragma unroll
  for (int o = 1; o < kWaveSize; o <<= 1) big = fmaxf(big, __shfl_xor(big, o, kWaveSize));
  if (lane == 0) top[threadIdx.x >> 6] = big;
  __syncthreads();
  if (threadIdx.x == 0) p.wmax[blockIdx.x] = fmaxf(fmaxf(fmaxf(top[0], top[1]), top[2]), top[3]);
  const int gr = tile / p.NT, t = tile - gr * p.NT;
  us8 *dst = static_cast<us8 *>(p.op) +
             (((int64_t)gr * p.KB + kb) * p.NT + t) * 3 * 64 + lane;
#pragma unroll
  for (int q = 0; q < 3; ++q) dst[q * 64] = part[q];
  if (tile == 0) {
    const int k = kb * 32 + (lane & 31);
    float v = 0.f;
    if (k < p.t.D) v = lane < 32 ? p.t.mean[k] : 1.0f / sqrtf(p.t.var[k] + p.t.eps_z);
    p.norm[kb * 64 + lane] = v;
  }
}

// As copy16_to_lds, 16 or 4 bytes per lane, streamed past the cache.
__device__ __forceinline__ void copy16_nt_to_lds(const void *base, uint32_t off, uint32_t lds) {
  asm volatile(
      "s_mov_b32 m0, %2\n\t"
      "global_load_lds_dwordx4 %0, %1 nt"
      :
      : "v"(off), "s"(base), "s"(lds)
      : "memory");
}
__device__ __forceinline__ void copy4_nt_to_lds(const void *base, uint32_t off, uint32_t lds) {
  asm volatile(
      "s_mov_b32 m0, %2\n\t"
      "global_load_lds_dword %0, %1 nt"
      :
      : "v"(off), "s"(base), "s"(lds)
      : "memory");
}

// WHOLE: the workgroup holds whole rows (one column group, D not split) and
// writes unit rows; else unnormalised sums, to y or the slice's partials.
template <int NT, bool VEC, bool WHOLE>
__global__ void __launch_bounds__(64 * kPWaves, 2) dresd_project_split(ProjectParams p) {
  constexpr int CPW = (NT * 3 + kPWaves - 1) / kPWaves;  // weight copies per wave and stage
  constexpr int kWSlot = CPW * kPWaves * kBlockBytes;
  constexpr int XC = VEC ? 4 : 16;                       // copies of x per wave and stage
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, m = lane & 15;
  const int64_t r0 = (int64_t)blockIdx.x * kPRows + wv * 32;
  const int gr = blockIdx.y;
  const int kb0 = (int)((int64_t)p.KB * blockIdx.z / p.t.splits);
  const int kb1 = (int)((int64_t)p.KB * (blockIdx.z + 1) / p.t.splits);
  const int D = p.t.D;
  const uint32_t lds = (uint32_t)(uintptr_t)smem;
  const unsigned char *op = static_cast<const unsigned char *>(p.op) +
                            (int64_t)gr * p.KB * (NT * 3 * kBlockBytes);

  // x: copy i of a stage takes rows 8 i + lane / 8 (16 bytes per lane) or
  // 2 i + lane / 32 (4 bytes).  LDS is filled in lane order; the lane at piece
  // position c of row r reads the row's piece c ^ (r mod 8).  Rows past M are
  // the last one again.
  constexpr int RPC = VEC ? 8 : 2;             // rows per copy
  const int lr = VEC ? lane >> 3 : lane >> 5;  // this lane's row of them
  constexpr int NV = VEC ? 1 : 4;              // copies until the pieces' order repeats
  const bool full = r0 + 32 <= p.t.M;
  const int64_t rb = r0 < p.t.M ? r0 : p.t.M - 1;
  const float *xr = p.t.x + rb * D;
  int xdim[NV];  // this lane's first dim within a block
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int r7 = (RPC * v + lr) & 7;
    xdim[v] = VEC ? ((lane & 7) ^ r7) * 4 : ((((lane & 31) >> 2) ^ r7) * 4 + (lane & 3));
  }
  // Past the slice's last block that block is read again; past D a row's
  // last dims are (their factor and weights are zero).
  auto issue_w = [&](int kb, int slot) {
    kb = kb < kb1 ? kb : kb1 - 1;
    const unsigned char *src = op + (int64_t)kb * (NT * 3 * kBlockBytes);
    const uint32_t base = lds + (uint32_t)slot * kWSlot;
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
      const int b = wv * CPW + i;
      const int bb = b < NT * 3 ? b : NT * 3 - 1;
      copy16_to_lds(src, (uint32_t)(bb * kBlockBytes + lane * 16),
                    base + (uint32_t)(b * kBlockBytes));
    }
  };
  const uint32_t xbase = lds + 2u * kWSlot + (uint32_t)(wv * kXWave);
  auto issue_x = [&](int kb, int slot) {
    kb = kb < kb1 ? kb : kb1 - 1;
    const uint32_t base = xbase + (uint32_t)slot * (kPWaves * kXWave);
    const float *src = xr + kb * 32;
    const bool tail = kb * 32 + 32 > D;
#pragma unroll
    for (int i = 0; i < XC; ++i) {
      int k = xdim[i % NV];
      if (tail) {
        const int last = (VEC ? D - 4 : D - 1) - kb * 32;
        k = k < last ? k : last;
      }
      // rows i RPC .. of the wave from a scalar base, unless some lie past M
      int r = lr;
      const float *from = src;
      if (full) {
        from += (int64_t)(i * RPC) * D;
      } else {
        const int64_t most = p.t.M - 1 - rb;
        r = i * RPC + lr < most ? i * RPC + lr : (int)most;
      }
      const uint32_t off = ((uint32_t)r * (uint32_t)D + (uint32_t)k) * 4u;
      if constexpr (VEC) copy16_nt_to_lds(from, off, base + (uint32_t)(i * kBlockBytes));
      else copy4_nt_to_lds(from, off, base + (uint32_t)(i * 256));
    }
    copy1_to_lds(p.norm + kb * 64 + lane, base + 4096u);
  };
  // z-scores (Eq. 1) of this wave's two tiles of 16 rows, in three parts.
  auto scores = [&](int slot, u4 (&z)[2][3]) {
    const unsigned char *xp =
        smem + 2 * kWSlot + (size_t)slot * (kPWaves * kXWave) + wv * kXWave;
    const float *nm = reinterpret_cast<const float *>(xp + 4096) + g * 8;
    float mu[8], inv[8];
#pragma unroll
    for (int e = 0; e < 8; e += 4) {
      const float4 a = *reinterpret_cast<const float4 *>(nm + e);
      const float4 b = *reinterpret_cast<const float4 *>(nm + 32 + e);
      mu[e] = a.x, mu[e + 1] = a.y, mu[e + 2] = a.z, mu[e + 3] = a.w;
      inv[e] = b.x, inv[e + 1] = b.y, inv[e + 2] = b.z, inv[e + 3] = b.w;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const unsigned char *rp = xp + (h * 16 + m) * 128;
      const int sw = m & 7;
      const float4 a = *reinterpret_cast<const float4 *>(rp + (((2 * g) ^ sw) * 16));
      const float4 b = *reinterpret_cast<const float4 *>(rp + (((2 * g + 1) ^ sw) * 16));
      const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
      us8 part[3];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        uint16_t pa, pb, pc;
        split3<false>((v[e] - mu[e]) * inv[e], pa, pb, pc);
        part[0][e] = pa;
        part[1][e] = pb;
        part[2][e] = pc;
      }
#pragma unroll
      for (int q = 0; q < 3; ++q) z[h][q] = __builtin_bit_cast(u4, part[q]);
    }
  };

  f4 hi[2][NT], lo[2][NT];  // sums of the high parts' products, and of the others
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int t = 0; t < NT; ++t) hi[h][t] = lo[h][t] = f4{0.f, 0.f, 0.f, 0.f};
  issue_x(kb0, 0);
  issue_x(kb0 + 1, 1);
  issue_w(kb0, 0);
  issue_x(kb0 + 2, 2);
  // the largest weight's size
  float wtop = 0.f;
  for (int i = lane; i < (p.groups * NT * p.KB + 3) / 4; i += kWaveSize)
    wtop = fmaxf(wtop, p.wmax[i]);
  wait_vmcnt<2 * (XC + 1) + CPW>();
  u4 z[2][3];
  scores(0, z);
  int xs = 0, ws = 0;  // slots of block kb
#pragma unroll 1
  for (int kb = kb0; kb < kb1; ++kb) {
    // All but the rows of block kb + 2 (the newest copies) have landed: the
    // weights of kb and the rows of kb + 1; after the barrier everyone's
    // weights have, and the other slot is read.
    wait_vmcnt<XC + 1>();
    __syncthreads();
    issue_w(kb + 1, ws ^ 1);
    issue_x(kb + 3, xs);  // its rows are in z
    xs = xs == 2 ? 0 : xs + 1;
    const u4 *wb = reinterpret_cast<const u4 *>(smem + (size_t)ws * kWSlot) + lane;
    ws ^= 1;
    // The next block's scores are made between this block's products.
    u4 zn[2][3];
    scores(xs, zn);
    // A = rows (lane (g, m): row m), B = weights: D lane (g, m), register i
    // holds row 4 g + i, column m.
    auto mul = [](const u4 &a, const u4 &b, f4 c) {
      return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8, a),
                                                     __builtin_bit_cast(b8, b), c, 0, 0, 0);
    };
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const u4 w0 = wb[(t * 3) * 64], w1 = wb[(t * 3 + 1) * 64], w2 = wb[(t * 3 + 2) * 64];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        lo[h][t] = mul(z[h][0], w2, lo[h][t]);
        hi[h][t] = mul(z[h][0], w0, hi[h][t]);
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) lo[h][t] = mul(z[h][1], w1, lo[h][t]);
#pragma unroll
      for (int h = 0; h < 2; ++h) lo[h][t] = mul(z[h][2], w0, lo[h][t]);
#pragma unroll
      for (int h = 0; h < 2; ++h) lo[h][t] = mul(z[h][0], w1, lo[h][t]);
#pragma unroll
      for (int h = 0; h < 2; ++h) lo[h][t] = mul(z[h][1], w0, lo[h][t]);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int q = 0; q < 3; ++q) z[h][q] = zn[h][q];
  }
  wait_vmcnt<0>();  // no LDS copy may land after the workgroup ends

  // Sums of squares of this wave's rows: a row's columns lie in the 16 lanes of
  // a group (columns past l are zero).
  const int l = p.t.l, c0 = gr * NT * 16;
  float ss[2][4];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int t = 0; t < NT; ++t) hi[h][t] += lo[h][t];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float s = 0.f;
#pragma unroll
      for (int t = 0; t < NT; ++t) s += hi[h][t][i] * hi[h][t][i];
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) s += __shfl_xor(s, o, kWaveSize);
      ss[h][i] = s;
    }
  }
  // Rows in doubt: not finite; or a norm below 2^-60 or below largest weight x
  // D x 2^-100, which lets a row's largest z-score lie below 2^-100, where its
  // parts end (bf16: 2^-133) less than 33 bits further down; or any row if
  // that is so of the weights.  A row of zero z-scores is none.
#pragma unroll
  for (int o = 1; o < kWaveSize; o <<= 1) wtop = fmaxf(wtop, __shfl_xor(wtop, o, kWaveSize));
  const bool odd = wtop > 0.f && !(wtop >= 0x1p-100f && wtop <= 0x1p100f);
  const float low = wtop > 0.f ? fmaxf(0x1p-60f, wtop * (float)D * 0x1p-100f) : 0.f;
  const int kbeg = kb0 * 32, kend = kb1 * 32 < D ? kb1 * 32 : D;
  uint32_t again = 0;  // bit 4 h + i: row 16 h + 4 g + i is in doubt
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool bad = odd || !(ss[h][i] < __builtin_inff()) || sqrtf(ss[h][i]) < low;
      if (bad && r0 + 16 * h + 4 * g + i < p.t.M) again |= 1u << (4 * h + i);
    }
  if (__ballot(again != 0)) {
    for (int r = 0; r < 32; ++r) {
      const int bit = 4 * (r >> 4) + (r & 3), of = (r >> 2) & 3;
      if (!((__builtin_amdgcn_readlane(again, of * 16) >> bit) & 1u)) continue;
      const float *row = p.t.x + (r0 + r) * D;
      bool nz = false;
      for (int k = kbeg + lane; k < kend && !nz; k += kWaveSize) {
        const float *nm = p.norm + (k >> 5) * 64 + (k & 31);
        nz = !((row[k] - nm[0]) * nm[32] == 0.f);
      }
      if (!__ballot(nz) && g == of) again &= ~(1u << bit);
    }
  }

  // Sums; WHOLE: unit rows (Eq. 2).
  float *out = p.t.splits > 1 ? p.t.part + (size_t)blockIdx.z * p.t.M * l : p.t.y;
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t row = r0 + 16 * h + 4 * g + i;
      const bool write = row < p.t.M && !((again >> (4 * h + i)) & 1u);
      const float inv = WHOLE ? 1.0f / fmaxf(sqrtf(ss[h][i]), p.t.eps_n) : 1.f;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int c = c0 + t * 16 + m;
        if (write && c < l) out[row * l + c] = WHOLE ? hi[h][t][i] * inv : hi[h][t][i];
      }
    }
  if (!__syncthreads_or(again != 0)) return;

  // The workgroup's rows in doubt, 32 at a time, one tile of columns per wave:
  // list of the rows (any order: each has sums of its own), then their sums.
  int32_t *list = reinterpret_cast<int32_t *>(smem), *nlist = list + kPRows;
  float *sums = reinterpret_cast<float *>(smem) + 512;  // [32][NT * 16]
  if (tid == 0) *nlist = 0;
  __syncthreads();
  if (m == 0)
    for (uint32_t left = again; left; left &= left - 1) {
      const int bit = __ffs((int)left) - 1;
      list[atomicAdd(nlist, 1)] = wv * 32 + 16 * (bit >> 2) + 4 * g + (bit & 3);
    }
  __syncthreads();
  const int total = *nlist;
  for (int b0 = 0; b0 < total; b0 += 32) {
    const float *xa[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int at = b0 + 16 * h + m < total ? b0 + 16 * h + m : total - 1;
      xa[h] = p.t.x + ((int64_t)blockIdx.x * kPRows + list[at]) * D;
    }
    if (wv < NT) {
      // Step e of a block of 32 dims multiplies dims 8 g + e, so that a lane's x
      // and norms are eight in a row; four blocks' loads are in flight.
      const int c = c0 + wv * 16 + m;
      const float *wc = p.t.W + (c < l ? c : l - 1);
      f4 acc[2] = {f4{0.f, 0.f, 0.f, 0.f}, f4{0.f, 0.f, 0.f, 0.f}};
      constexpr int U = 4;
#pragma unroll 1
      for (int kb = kb0; kb < kb1; kb += U) {
        float xv[U][2][8], w[U][8];
        float4 nm[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int k0 = (kb + u < kb1 ? kb + u : kb1 - 1) * 32 + g * 8;
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            if constexpr (VEC) {
#pragma unroll
              for (int e = 0; e < 8; e += 4) {
                const float4 v =
                    *reinterpret_cast<const float4 *>(xa[h] + (k0 + e < D ? k0 + e : D - 4));
                xv[u][h][e] = v.x, xv[u][h][e + 1] = v.y;
                xv[u][h][e + 2] = v.z, xv[u][h][e + 3] = v.w;
              }
            } else {
#pragma unroll
              for (int e = 0; e < 8; ++e) xv[u][h][e] = xa[h][k0 + e < D ? k0 + e : D - 1];
            }
          }
#pragma unroll
          for (int e = 0; e < 8; ++e) w[u][e] = wc[(int64_t)(k0 + e < D ? k0 + e : D - 1) * l];
          const float *n0 = p.norm + (k0 >> 5) * 64 + g * 8;
#pragma unroll
          for (int e = 0; e < 4; ++e)
            nm[u][e] = *reinterpret_cast<const float4 *>(n0 + (e & 1) * 4 + (e >> 1) * 32);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int k0 = (kb + u) * 32 + g * 8;
          if (kb + u < kb1) {
            const float mu[8] = {nm[u][0].x, nm[u][0].y, nm[u][0].z, nm[u][0].w,
                                 nm[u][1].x, nm[u][1].y, nm[u][1].z, nm[u][1].w};
            const float inv[8] = {nm[u][2].x, nm[u][2].y, nm[u][2].z, nm[u][2].w,
                                  nm[u][3].x, nm[u][3].y, nm[u][3].z, nm[u][3].w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const bool in = k0 + e < D;
              const float wv1 = in && c < l ? w[u][e] : 0.f;
#pragma unroll
              for (int h = 0; h < 2; ++h) {
                const float z1 = in ? (xv[u][h][e] - mu[e]) * inv[e] : 0.f;
                acc[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(z1, wv1, acc[h], 0, 0, 0);
              }
            }
          }
        }
      }
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r = 16 * h + 4 * g + i;
          if constexpr (WHOLE) {
            sums[r * (NT * 16) + wv * 16 + m] = acc[h][i];
          } else if (b0 + r < total && c < l) {
            out[((int64_t)blockIdx.x * kPRows + list[b0 + r]) * l + c] = acc[h][i];
          }
        }
    }
    if constexpr (WHOLE) {
      __syncthreads();
      for (int r = wv; r < 32 && b0 + r < total; r += kPWaves) {
        float v[2], s = 0.f;  // NT * 16 <= 128 columns, zero past l
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          v[j] = lane + 64 * j < NT * 16 ? sums[r * (NT * 16) + lane + 64 * j] : 0.f;
          s += v[j] * v[j];
        }
        for (int o = 1; o < kWaveSize; o <<= 1) s += __shfl_xor(s, o, kWaveSize);
        const float inv = 1.0f / fmaxf(sqrtf(s), p.t.eps_n);
#pragma unroll
        for (int j = 0; j < 2; ++j)
          if (lane + 64 * j < l)
            out[((int64_t)blockIdx.x * kPRows + list[b0 + r]) * l + lane + 64 * j] = v[j] * inv;
      }
      __syncthreads();
    }
  }
}

template <int NT>
constexpr size_t project_lds() {
  return 2 * (size_t)((NT * 3 + kPWaves - 1) / kPWaves * kPWaves * kBlockBytes) +
         3 * (size_t)kPWaves * kXWave;
}

template <int NT>
hipError_t launch_nt(ProjectParams &p, hipStream_t st) {
  const bool vec = (p.t.D & 3) == 0 && ((uintptr_t)p.t.x & 15u) == 0;
  const bool whole = p.groups == 1 && p.t.splits == 1;
  const void *f = vec ? (whole ? (const void *)dresd_project_split<NT, true, true>
                               : (const void *)dresd_project_split<NT, true, false>)
                      : (whole ? (const void *)dresd_project_split<NT, false, true>
                               : (const void *)dresd_project_split<NT, false, false>);
  hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)project_lds<NT>());
  if (e != hipSuccess) return e;
  void *args[] = {&p};
  return hipLaunchKernel(f,
                         dim3((unsigned)((p.t.M + kPRows - 1) / kPRows), (unsigned)p.groups,
                              (unsigned)p.t.splits),
                         dim3(64 * kPWaves), args, project_lds<NT>(), st);
}

}  // namespace

bool project_split_plan(int64_t M, int D, int l, int cus, ProjectParams *out) {
  ProjectParams &p = *out;
  p = ProjectParams{};
  // Its three launches cost more than the fp32 kernels below about 2^30
  // multiply-adds (2,000 x 4,096 -> 128: 35 against 39 us; 1,024 rows: 30
  // against 25), half of that where those take their scalar loads (1,465 x
  // 4,096 -> 108: 32 against 71 us); few rows leave most of a 256-row block
  // empty.
  const bool even = D % 4 == 0 && l % 64 == 0;
  if (M < 512 || D < 32 || M * (double)D * l < (even ? 0x1p30 : 0x1p29) * 0.95) return false;
  p.KB = (D + 31) / 32;
  const int tiles = (l + 15) / 16;
  p.groups = (tiles + 7) / 8;
  p.NT = (tiles + p.groups - 1) / p.groups;
  const int64_t op = (int64_t)p.groups * p.KB * p.NT * 3 * kBlockBytes;
  const int64_t most = (int64_t)256 << 20;
  if (op > most) return false;
  // One workgroup per CU runs at once.  D is split where that shortens the
  // rounds of workgroups times a slice's blocks of dims (and about 6 blocks'
  // time to start and end), into slices of at least 4 blocks whose partial sums
  // take at most 256 MiB.
  const int64_t wgs = (M + kPRows - 1) / kPRows * p.groups;
  int64_t best = 0;
  for (int s = 1; s <= 64 && (s == 1 || (s * 4 <= p.KB && wgs < 2 * cus &&
                                         s * M * l * 4 <= most)); ++s) {
    const int64_t cost = (wgs * s + cus - 1) / cus * ((p.KB + s - 1) / s + 6);
    if (s == 1 || cost < best) {
      best = cost;
      p.t.splits = s;
    }
  }
  p.off_norm = (op + 255) / 256 * 256;
  p.off_wmax = p.off_norm + (int64_t)p.KB * 256;
  p.off_part = p.off_wmax + ((int64_t)p.groups * p.NT * p.KB * 4 + 255) / 256 * 256;
  p.bytes = p.off_part + (p.t.splits > 1 ? (int64_t)p.t.splits * M * l * 4 : 0);
  return true;
}

hipError_t launch_project_split(ProjectParams &p, void *ws, hipStream_t st) {
  unsigned char *b = static_cast<unsigned char *>(ws);
  p.op = b;
  p.norm = reinterpret_cast<float *>(b + p.off_norm);
  p.wmax = reinterpret_cast<float *>(b + p.off_wmax);
  p.t.part = reinterpret_cast<float *>(b + p.off_part);
  void *args[] = {&p};
  const int64_t waves = (int64_t)p.groups * p.NT * p.KB;
  hipError_t e = hipLaunchKernel((const void *)dresd_project_operand,
                                 dim3((unsigned)((waves + 3) / 4)), dim3(256), args, 0, st);
  if (e != hipSuccess) return e;
  switch (p.NT) {
    case 1: e = launch_nt<1>(p, st); break;
    case 2: e = launch_nt<2>(p, st); break;
    case 3: e = launch_nt<3>(p, st); break;
    case 4: e = launch_nt<4>(p, st); break;
    case 5: e = launch_nt<5>(p, st); break;
    case 6: e = launch_nt<6>(p, st); break;
    case 7: e = launch_nt<7>(p, st); break;
    default: e = launch_nt<8>(p, st); break;
  }
  if (e != hipSuccess || (p.groups == 1 && p.t.splits == 1)) return e;
  return launch_finish_rows(p.t, st);
}

}  // namespace dresd
