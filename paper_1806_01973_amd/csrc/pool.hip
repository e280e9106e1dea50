// Neighbourhood pooling on gfx950 (Algorithm 1, line 1 applied as a gather
// over the once-per-node projections of Sec. 3.4). Importance pooling
// (Sec. 3.2: gamma is the weighted mean of the transformed neighbour vectors,
// weighted by the L1-normalised visit counts):
//   n[r] = sum_t alpha[r][t] * P[idx[r][t]];
// and the gamma = mean and gamma = max variants compared in Sec. 4.
//
// One wavefront per output row (grid-stride). The row's idx/weights are
// wave-uniform and come through the scalar cache; each lane owns VEC
// consecutive columns of every 64*VEC-column slab, so one load instruction of
// the wave reads a contiguous 64*VEC-element span of a gathered row. Rows are
// fetched in groups of U neighbours before they are accumulated, which
// keeps several row reads in flight per wave. The sum runs in rank order t in
// fp32; the result is stored in the storage dtype.
#include "device_util.h"
#include "kernels.h"

namespace pinsage {
namespace {

constexpr int kWavesPerBlock = 4;

template <bool BF16>
struct Vec;
template <>
struct Vec<false> {  // 4 x fp32 = 16 B per lane
  static constexpr int kN = 4;
  using Raw = float4;
  __device__ static void to_f32(const Raw& r, float (&o)[4]) {
    o[0] = r.x; o[1] = r.y; o[2] = r.z; o[3] = r.w;
  }
  __device__ static Raw from_f32(const float (&o)[4]) { return make_float4(o[0], o[1], o[2], o[3]); }
};
template <>
struct Vec<true> {  // 8 x bf16 = 16 B per lane
  static constexpr int kN = 8;
  using Raw = uint4;
  __device__ static void to_f32(const Raw& r, float (&o)[8]) {
    const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[2 * i] = __uint_as_float(w[i] << 16);
      o[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
    }
  }
  __device__ static Raw from_f32(const float (&o)[8]) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      w[i] = (uint32_t)f32_to_bf16(o[2 * i]) | ((uint32_t)f32_to_bf16(o[2 * i + 1]) << 16);
    return make_uint4(w[0], w[1], w[2], w[3]);
  }
};

// Per-row setup shared by both kernels: the weight sum S of a row without
// stored weights (importance pooling derives alpha = count / S) or the number
// of neighbours (mean pooling), counted by the lanes in parallel; integers, so
// the order does not matter.
__device__ __forceinline__ int row_total(const PoolLaunch& a, int64_t row, int lane) {
  const int T = a.T;
  int part = 0;
  if (a.mode == kPoolMean) {
    for (int t = lane; t < T; t += kWave) {
      const int32_t v = a.idx[row * T + t];
      part += ((uint64_t)(int64_t)v < (uint64_t)a.n_transform) ? 1 : 0;
    }
  } else if (a.mode == kPoolImportance && !a.weights) {
    for (int t = lane; t < T; t += kWave) part += a.counts[row * T + t];
  } else {
    return 0;
  }
  return wave_sum_i32(part);
}

// One past the last slot of the row that holds a neighbour (0 for an empty
// row): the loops stop there, so short rows of a wide table cost little.
// Skipped slots hold no neighbour and would contribute nothing.
__device__ __forceinline__ int row_end(const PoolLaunch& a, int64_t row, int lane) {
  const int T = a.T;
  int last = -1;
  for (int t = lane; t < T; t += kWave) {
    const int32_t v = a.idx[row * T + t];
    if ((uint64_t)(int64_t)v < (uint64_t)a.n_transform) last = t;
  }
  return __builtin_amdgcn_readfirstlane(wave_max_i32(last)) + 1;
}

// Weight of neighbour slot t of a row (importance or mean pooling).
template <int MODE>
__device__ __forceinline__ float slot_alpha(const PoolLaunch& a, int64_t row, int t, int total) {
  if constexpr (MODE == kPoolMean) return 1.0f / (float)total;
  if (a.weights) return a.weights[row * a.T + t];
  return (float)a.counts[row * a.T + t] / (float)total;
}

// J = number of 64*VEC-column slabs per row (compile time); U neighbour rows
// are in flight per wave (U*J 16-byte loads per lane). MODE: importance
// (weighted sum), mean (uniform weights 1/#neighbours) or max (element-wise,
// skipped slots do not take part; an empty row gives zeros).
template <bool BF16, int MODE, int J, int U = (J <= 2 ? 8 : (J <= 4 ? 4 : (J <= 8 ? 2 : 1)))>
__global__ __launch_bounds__(256) void pool_kernel(PoolLaunch a) {
  using V = Vec<BF16>;
  using Raw = typename V::Raw;
  constexpr int VN = V::kN;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (a.slabbed && *a.slabbed) return;  // pool_slab_kernel has pooled the rows
  const int m = a.m;
  const int T = a.T;
  const Raw* __restrict__ P = static_cast<const Raw*>(a.P);
  Raw* __restrict__ out = static_cast<Raw*>(a.out);
  const int vec_per_row = m / VN;

  for (int64_t row0 = (int64_t)blockIdx.x * kWavesPerBlock + wave; row0 < a.rows;
       row0 += (int64_t)gridDim.x * kWavesPerBlock) {
    const int64_t row = row0;
    const int32_t* __restrict__ ridx = a.idx + row * T;
    const int total = row_total(a, row, lane);
    const int tend = row_end(a, row, lane);
    float acc[J][VN];
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
      for (int v = 0; v < VN; ++v) acc[j][v] = MODE == kPoolMax ? -INFINITY : 0.0f;
    bool any = false;

    for (int t0 = 0; t0 < tend; t0 += U) {
      Raw buf[U][J];
      float alpha[U];
      bool ok[U];
#pragma unroll
      for (int i = 0; i < U; ++i) {
        const int t = t0 + i;
        int32_t v = t < tend ? ridx[t] : -1;
        if ((uint64_t)(int64_t)v >= (uint64_t)a.n_transform) v = -1;
        ok[i] = v >= 0;
        alpha[i] = 0.0f;
        if constexpr (MODE != kPoolMax)
          if (v >= 0) alpha[i] = slot_alpha<MODE>(a, row, t, total);
#pragma unroll
        for (int j = 0; j < J; ++j) {
          const int c = j * kWave + lane;
          if (v >= 0 && c < vec_per_row) buf[i][j] = P[(int64_t)v * vec_per_row + c];
          else buf[i][j] = Raw{};
        }
      }
#pragma unroll
      for (int i = 0; i < U; ++i) {
        any = any || ok[i];
#pragma unroll
        for (int j = 0; j < J; ++j) {
          float f[VN];
          V::to_f32(buf[i][j], f);
#pragma unroll
          for (int v = 0; v < VN; ++v) {
            if constexpr (MODE == kPoolMax) acc[j][v] = ok[i] ? fmaxf(acc[j][v], f[v]) : acc[j][v];
            else acc[j][v] = fmaf(alpha[i], f[v], acc[j][v]);
          }
        }
      }
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int c = j * kWave + lane;
      if constexpr (MODE == kPoolMax)
#pragma unroll
        for (int v = 0; v < VN; ++v) acc[j][v] = any ? acc[j][v] : 0.0f;
      if (c < vec_per_row) out[row * vec_per_row + c] = V::from_f32(acc[j]);
    }
  }
}

// Rows narrower than one wave slab (at most 64 / RG vectors): the wave splits
// into RG lane groups of 64 / RG lanes, group g gathering neighbours
// t = g, g + RG, ... of the row, so one load instruction reads RG rows. Each
// group reduces its neighbours in rank order; the RG partial results are then
// combined by a fixed butterfly over the groups (the same order on every
// lane). U = 4 loads in flight per lane: on 512-byte rows, 8 and 16 measured
// 5% and 40% slower (fewer resident waves).
template <bool BF16, int MODE, int RG, int U = 4>
__global__ __launch_bounds__(256) void pool_narrow_kernel(PoolLaunch a) {
  using V = Vec<BF16>;
  using Raw = typename V::Raw;
  constexpr int VN = V::kN;
  constexpr int GL = kWave / RG;  // lanes per group
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int grp = lane / GL, c = lane % GL;
  const int T = a.T;
  const Raw* __restrict__ P = static_cast<const Raw*>(a.P);
  Raw* __restrict__ out = static_cast<Raw*>(a.out);
  const int vec_per_row = a.m / VN;
  const bool col_ok = c < vec_per_row;

  for (int64_t row = (int64_t)blockIdx.x * kWavesPerBlock + wave; row < a.rows;
       row += (int64_t)gridDim.x * kWavesPerBlock) {
    const int32_t* __restrict__ ridx = a.idx + row * T;
    const int total = row_total(a, row, lane);
    const int tend = row_end(a, row, lane);
    float acc[VN];
#pragma unroll
    for (int v = 0; v < VN; ++v) acc[v] = MODE == kPoolMax ? -INFINITY : 0.0f;
    bool any = false;
    for (int t0 = 0; t0 < tend; t0 += U * RG) {
      Raw buf[U];
      float alpha[U];
      bool ok[U];
#pragma unroll
      for (int i = 0; i < U; ++i) {
        const int t = t0 + i * RG + grp;
        int32_t v = t < tend ? ridx[t] : -1;
        if ((uint64_t)(int64_t)v >= (uint64_t)a.n_transform) v = -1;
        ok[i] = v >= 0;
        alpha[i] = 0.0f;
        if constexpr (MODE != kPoolMax)
          if (v >= 0) alpha[i] = slot_alpha<MODE>(a, row, t, total);
        buf[i] = (v >= 0 && col_ok) ? P[(int64_t)v * vec_per_row + c] : Raw{};
      }
#pragma unroll
      for (int i = 0; i < U; ++i) {
        any = any || ok[i];
        float f[VN];
        V::to_f32(buf[i], f);
#pragma unroll
        for (int v = 0; v < VN; ++v) {
          if constexpr (MODE == kPoolMax) acc[v] = ok[i] ? fmaxf(acc[v], f[v]) : acc[v];
          else acc[v] = fmaf(alpha[i], f[v], acc[v]);
        }
      }
    }
#pragma unroll
    for (int o = GL; o < kWave; o <<= 1)
#pragma unroll
      for (int v = 0; v < VN; ++v) {
        const float other = __shfl_xor(acc[v], o);
        acc[v] = MODE == kPoolMax ? fmaxf(acc[v], other) : acc[v] + other;
      }
    if constexpr (MODE == kPoolMax) {
      // `any` of the whole row: some group saw a neighbour.
      const bool row_any = __builtin_amdgcn_readfirstlane(wave_sum_i32(any ? 1 : 0)) > 0;
#pragma unroll
      for (int v = 0; v < VN; ++v) acc[v] = row_any ? acc[v] : 0.0f;
    }
    if (grp == 0 && col_ok) out[row * vec_per_row + c] = V::from_f32(acc);
  }
}

// Rows of at most 64 / RG vectors with at most 64 neighbour slots (every
// workload's pooled width in the dense-then-pool order): the row's header --
// neighbour ids and the weights, counts or neighbour count alpha needs -- is
// one coalesced vector load (lane t holds slot t), alpha is formed per lane
// with the same fp32 division as the batched kernels, and every live slot's
// gather is issued before the first one is summed: NB slots per lane group
// per batch (one batch when the row has at most RG * NB slots), slot ids and
// alphas passed to the groups by lane permutes. Group g sums slots g, g + RG,
// ... in rank order and the groups are combined by the same butterfly as in
// pool_narrow_kernel, so the result is the same bits. Measured on random 512-byte rows from a 41 GB
// table: as fast as a gather with no header reads at all (+16% over the
// batched kernel).
template <bool BF16, int MODE, int RG, int NB>
__global__ __launch_bounds__(256) void pool_head_kernel(PoolLaunch a) {
  using V = Vec<BF16>;
  using Raw = typename V::Raw;
  constexpr int VN = V::kN;
  constexpr int GL = kWave / RG;  // lanes per group
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int grp = lane / GL, c = lane % GL;
  const int T = a.T;
  const Raw* __restrict__ P = static_cast<const Raw*>(a.P);
  Raw* __restrict__ out = static_cast<Raw*>(a.out);
  const int vec_per_row = a.m / VN;
  const bool col_ok = c < vec_per_row;

  for (int64_t row = (int64_t)blockIdx.x * kWavesPerBlock + wave; row < a.rows;
       row += (int64_t)gridDim.x * kWavesPerBlock) {
    // Header: slot `lane` of the row.
    int32_t v = -1;
    float w = 0.0f;
    int cnt = 0;
    if (lane < T) {
      v = a.idx[row * T + lane];
      if constexpr (MODE == kPoolImportance) {
        if (a.weights) w = a.weights[row * T + lane];
        else cnt = a.counts[row * T + lane];
      }
    }
    const bool valid = (uint64_t)(int64_t)v < (uint64_t)a.n_transform;
    if (!valid) v = -1;
    float alpha = 0.0f;
    if constexpr (MODE == kPoolMean) {
      const int total = wave_sum_i32(valid ? 1 : 0);
      alpha = valid ? 1.0f / (float)total : 0.0f;
    } else if constexpr (MODE == kPoolImportance) {
      if (a.weights) {
        alpha = valid ? w : 0.0f;
      } else {
        const int total = wave_sum_i32(cnt);  // every slot, as the walk kernel's S
        alpha = valid ? (float)cnt / (float)total : 0.0f;
      }
    }
    const int tend = __builtin_amdgcn_readfirstlane(wave_max_i32(valid ? lane : -1)) + 1;

    float acc[VN];
#pragma unroll
    for (int k = 0; k < VN; ++k) acc[k] = MODE == kPoolMax ? -INFINITY : 0.0f;
    bool any = false;
    for (int b0 = 0; b0 < tend; b0 += RG * NB) {
      Raw buf[NB];
      float al[NB];
      bool ok[NB];
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int t = b0 + i * RG + grp;
        int32_t vt;
        float at;
        if constexpr (RG == 1) {
          vt = __builtin_amdgcn_readlane(v, t & 63);
          at = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(alpha), t & 63));
        } else {
          vt = __shfl(v, t & 63);
          at = __shfl(alpha, t & 63);
        }
        ok[i] = t < tend && vt >= 0;
        al[i] = ok[i] ? at : 0.0f;
        buf[i] = (ok[i] && col_ok) ? P[(int64_t)vt * vec_per_row + c] : Raw{};
      }
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        any = any || ok[i];
        float f[VN];
        V::to_f32(buf[i], f);
#pragma unroll
        for (int k = 0; k < VN; ++k) {
          if constexpr (MODE == kPoolMax) acc[k] = ok[i] ? fmaxf(acc[k], f[k]) : acc[k];
          else acc[k] = fmaf(al[i], f[k], acc[k]);
        }
      }
    }
#pragma unroll
    for (int o = GL; o < kWave; o <<= 1)
#pragma unroll
      for (int k = 0; k < VN; ++k) {
        const float other = __shfl_xor(acc[k], o);
        acc[k] = MODE == kPoolMax ? fmaxf(acc[k], other) : acc[k] + other;
      }
    if constexpr (MODE == kPoolMax) {
      const bool row_any = __builtin_amdgcn_readfirstlane(wave_sum_i32(any ? 1 : 0)) > 0;
#pragma unroll
      for (int k = 0; k < VN; ++k) acc[k] = row_any ? acc[k] : 0.0f;
    }
    if (grp == 0 && col_ok) out[row * vec_per_row + c] = V::from_f32(acc);
  }
}

// Decides between whole rows and column slabs (below) from kProbes sampled slots:
// slabs pay when the neighbourhoods are deep (a header is read per slab) and when
// enough gathers go to rows that are gathered again and again, so that their slices
// stay in the L2s: the share of samples whose id was sampled more than once. Slabs
// against whole rows at T = 50, by that share: tables beyond the last-level cache, 700K
// rows of 1 KB in fp32 0.03 1.07x the time, 0.07 1.04, 0.11 1.01, 0.19 0.97, 0.23 0.93,
// 0.50 0.82, in bf16 1.12, 1.08, 1.05, 1.00, 0.98 and 0.88; 1.5M 1.02 at 0.07 and 0.97
// at 0.18; the 1.2M-node graph's pins 0.79 at 0.19. Tables inside it, 200K rows of 1 KB
// 0.99 at 0.05 and 0.86 at 0.32, 100K of 2 KB 0.89 at 0.10. (The pairs of equal ids
// among 2,048 samples, tried before, do not tell a few very popular rows from many
// popular ones: 77 at 1.08x, 64 at 0.79x.)
constexpr int kProbes = 8192;
__global__ __launch_bounds__(1024) void pool_probe_kernel(PoolLaunch a, int min_live) {
  constexpr int kSlots = 2 * kProbes;
  constexpr int kEach = kProbes / 1024;
  __shared__ uint32_t keys[kSlots], seen[kSlots];
  __shared__ int live, repeated;
  for (int i = threadIdx.x; i < kSlots; i += 1024) {
    keys[i] = 0xFFFFFFFFu;
    seen[i] = 0u;
  }
  if (threadIdx.x == 0) live = repeated = 0;
  int32_t ids[kEach];
#pragma unroll
  for (int e = 0; e < kEach; ++e) {
    const uint32_t x = (uint32_t)(e * 1024 + (int)threadIdx.x) * 0x9E3779B9u;
    const int64_t row = (int64_t)(((uint64_t)x * (uint64_t)a.rows) >> 32);
    const int t = (int)(((uint64_t)(x * 0x85EBCA6Bu) * (uint64_t)a.T) >> 32);
    ids[e] = a.idx[row * a.T + t];
  }
  __syncthreads();
  int n = 0;
#pragma unroll
  for (int e = 0; e < kEach; ++e) {
    const uint32_t v = (uint32_t)ids[e];
    if ((uint64_t)(int64_t)ids[e] >= (uint64_t)a.n_transform) continue;
    ++n;
    uint32_t h = (v * 0x9E3779B9u) >> (32 - 14);
    static_assert(kSlots == 1 << 14, "home slot");
    for (;;) {  // half full at most, so a free slot is found
      const uint32_t k = atomicCAS(&keys[h], 0xFFFFFFFFu, v);
      if (k == 0xFFFFFFFFu || k == v) break;
      h = (h + 1) & (kSlots - 1);
    }
    atomicAdd(&seen[h], 1u);
  }
  __syncthreads();
  int again = 0;
  for (int i = threadIdx.x; i < kSlots; i += 1024) again += seen[i] > 1u ? (int)seen[i] : 0;
  n = wave_sum_i32(n);
  again = wave_sum_i32(again);
  if ((threadIdx.x & 63) == 0) {
    atomicAdd(&live, n);
    atomicAdd(&repeated, again);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const int64_t table = a.n_transform * (int64_t)a.m * (a.bf16 ? 2 : 4);
    const int least = table <= (256ll << 20) ? 5 : 12;  // percent
    *a.slabbed = (int64_t)live * a.T >= (int64_t)min_live * kProbes && repeated * 100 >= live * least;
  }
}

// Tables of wide rows beyond the L2s: the pool runs over column slabs of GL
// 16-byte vectors, all rows of one slab before the next (blocks are dispatched in
// order), so that an L2 holds the slices of 8 or 4 times as many popular rows as
// it holds whole rows, and the last-level cache a slab of the whole table. An item
// is one row of one slab: RG = 64 / GL lane groups gather its slots, every slot in
// flight at once, each group summing slots g, g + RG, ... in rank order. A narrow
// item costs issue slots as much as bytes, so: the next row's header is loaded
// under the current row's gathers; a slot's byte offset and weight pass through
// LDS (two lane permutes and a 64-bit multiply per slot otherwise); and the groups
// are added by halving (each step exchanges half of the values a lane still
// holds), in the same tree as a butterfly. pool_probe_kernel decides; this kernel
// and pool_kernel (whole rows, launched behind it) each end at once if not chosen
// (with the probe about 35 us where whole rows are).
// What bounds it: cache bandwidth, about 13 TB/s of gathered bytes, and at 128
// bytes an item the issue slots. T = 50, pin degree Zipf(2): 1M rows of 1 KB
// (fp32) 6.60 -> 5.19 ms; 300K of 1 KB (bf16) 1.72 -> 1.36; 100K of 2 KB, max
// 1.09 -> 0.82. Where popularity is uniform, 800K rows of 1 KB took 6.67 ms whole
// and 7.03 in slabs; with 10 neighbours a row 1.06 and 1.51 (whence the probe).
constexpr int kSlabBlockRows = 32 * kWavesPerBlock;  // 64 per wave: 3-5% slower
template <bool BF16, int MODE, int GL>
__global__ __launch_bounds__(256, GL == 8 ? 7 : 4) void pool_slab_kernel(PoolLaunch a) {
  using V = Vec<BF16>;
  using Raw = typename V::Raw;
  constexpr int VN = V::kN;
  constexpr int RG = kWave / GL;
  constexpr int NB = kWave / RG;  // slots per lane group: T <= 64 in one batch
  constexpr int ESZ = BF16 ? 2 : 4;
  __shared__ uint2 slots_all[kWavesPerBlock][kWave];  // byte offset, weight per slot
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (!*a.slabbed) return;
  uint2* const slots = slots_all[wave];
  const int T = a.T;
  const int grp = lane / GL, c = lane % GL;
  const uint32_t row_bytes = (uint32_t)a.m * ESZ;
  // Block b: slab b / blocks per slab, kSlabBlockRows of its rows.
  const uint32_t per_slab = (uint32_t)((a.rows + kSlabBlockRows - 1) / kSlabBlockRows);
  const uint32_t slab = blockIdx.x / per_slab;
  const uint32_t col = slab * GL * 16 + c * 16;  // byte of the row
  const bool col_ok = col < row_bytes;
  const unsigned char* const P = static_cast<const unsigned char*>(a.P);
  struct Head {
    int32_t v = -1;
    float w = 0.0f;
    int cnt = 0;
  };
  auto load_head = [&](int64_t row) __attribute__((always_inline)) {
    Head h;
    if (lane < T) {
      h.v = a.idx[row * T + lane];
      if constexpr (MODE == kPoolImportance) {
        if (a.weights) h.w = a.weights[row * T + lane];
        else h.cnt = a.counts[row * T + lane];
      }
    }
    return h;
  };

  int64_t row = (int64_t)(blockIdx.x % per_slab) * kSlabBlockRows;
  const int64_t end = row + kSlabBlockRows < a.rows ? row + kSlabBlockRows : a.rows;
  row += wave;
  Head head;
  if (row < end) head = load_head(row);
  for (; row < end; row += kWavesPerBlock) {
    const Head cur = head;
    if (row + kWavesPerBlock < end) head = load_head(row + kWavesPerBlock);

    const bool valid = (uint64_t)(int64_t)cur.v < (uint64_t)a.n_transform;
    float alpha = 0.0f;
    if constexpr (MODE == kPoolMean) {
      const int total = wave_sum_i32(valid ? 1 : 0);
      alpha = valid ? 1.0f / (float)total : 0.0f;
    } else if constexpr (MODE == kPoolImportance) {
      if (a.weights) {
        alpha = valid ? cur.w : 0.0f;
      } else {
        const int total = wave_sum_i32(cur.cnt);  // every slot, as the walk kernel's S
        alpha = valid ? (float)cur.cnt / (float)total : 0.0f;
      }
    }
    slots[lane] = make_uint2(valid ? (uint32_t)cur.v * row_bytes : 0xFFFFFFFFu,
                             __float_as_uint(alpha));
    wave_lds_sync();
    Raw buf[NB];
    bool ok[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const uint32_t at = slots[i * RG + grp].x;
      ok[i] = at != 0xFFFFFFFFu && col_ok;
      buf[i] = ok[i] ? *reinterpret_cast<const Raw*>(P + (at + col)) : Raw{};
    }
    float acc[VN];
#pragma unroll
    for (int k = 0; k < VN; ++k) acc[k] = MODE == kPoolMax ? -INFINITY : 0.0f;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      float f[VN];
      V::to_f32(buf[i], f);
      const float al = MODE == kPoolMax ? 0.0f : __uint_as_float(slots[i * RG + grp].y);
#pragma unroll
      for (int k = 0; k < VN; ++k) {
        // Absent slots: weight 0 and zeros; for the max they take no part.
        if constexpr (MODE == kPoolMax) acc[k] = ok[i] ? fmaxf(acc[k], f[k]) : acc[k];
        else acc[k] = fmaf(al, f[k], acc[k]);
      }
    }
    wave_lds_sync();  // the slots are rewritten for the next row
    // Sum (or max) over the groups; the lane ends with elements [e0, e0 + left)
    // of its vector, the same in `copies` lanes.
    int left = VN, e0 = 0;
    bool first = true;
#pragma unroll
    for (int o = kWave / 2; o >= GL; o >>= 1) {
      const bool up = (lane & o) != 0;
      if (left > 1) {
        left /= 2;
#pragma unroll
        for (int k = 0; k < VN / 2; ++k) {
          if (k >= left) continue;
          const float give = up ? acc[k] : acc[k + left];
          const float keep = up ? acc[k + left] : acc[k];
          const float got = __shfl_xor(give, o);
          acc[k] = MODE == kPoolMax ? fmaxf(keep, got) : keep + got;
        }
        e0 += up ? left : 0;
      } else {
        const float got = __shfl_xor(acc[0], o);
        acc[0] = MODE == kPoolMax ? fmaxf(acc[0], got) : acc[0] + got;
        first = first && !up;
      }
    }
    if constexpr (MODE == kPoolMax) {
      const bool row_any = __ballot(valid) != 0ull;
#pragma unroll
      for (int k = 0; k < VN; ++k) acc[k] = row_any ? acc[k] : 0.0f;
    }
    constexpr int LEFT = VN > RG ? VN / RG : 1;
    if (first && col_ok) {
      unsigned char* const o =
          static_cast<unsigned char*>(a.out) + row * (int64_t)row_bytes + col + e0 * ESZ;
      if constexpr (!BF16) {
        *reinterpret_cast<float*>(o) = acc[0];
      } else if constexpr (LEFT == 2) {
        *reinterpret_cast<uint32_t*>(o) =
            (uint32_t)f32_to_bf16(acc[0]) | ((uint32_t)f32_to_bf16(acc[1]) << 16);
      } else {
        *reinterpret_cast<uint16_t*>(o) = f32_to_bf16(acc[0]);
      }
      static_assert(BF16 ? LEFT <= 2 : LEFT == 1, "elements left per lane");
    }
  }
}

// Fewest live slots per row (on average) that pay for a header per slab: at 27 of
// T = 27, fp32 rows gained (396 -> 352 us, 150K of 1 KB) and bf16 rows lost (891 ->
// 1166, 300K of 1 KB: twice the values per lane to add over the groups).
inline int min_live(bool bf16) { return bf16 ? 40 : 22; }

// Bytes of a row per slab, 0 for whole rows. 256 while a slab takes at most half
// of the last-level cache (256 MB), 128 up to all of it. Measured, whole / 256 / 128
// (us): 20K rows of 2 KB 146 / 153 / 149; 50K of 1 KB 218 / 182 / 187; 150K of 1 KB
// 724 / 542 / 553; 300K of 1 KB in bf16 1722 / 1336 / 1611; 700K of 1 KB 4427 / 3683
// / 3384; 1.6M 10855 / 9812 / 9641; 2M in bf16 14339 / 13441 / 13073.
inline int slab_bytes(const PoolLaunch& a) {
  if (!a.slabbed || a.T > kWave || a.T < min_live(a.bf16)) return 0;
  if (a.n_transform * 256 <= (128ll << 20)) return 256;
  return a.n_transform * 128 <= (256ll << 20) ? 128 : 0;
}

template <bool BF16, int MODE>
hipError_t launch_slabs(const PoolLaunch& a, int bytes, hipStream_t s) {
  const int64_t slabs = ((int64_t)a.m * (BF16 ? 2 : 4) + bytes - 1) / bytes;
  const int64_t blocks = slabs * ((a.rows + kSlabBlockRows - 1) / kSlabBlockRows);
  if (blocks > 0x7FFFFFFFll) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks), block(256);
  hipLaunchKernelGGL(pool_probe_kernel, dim3(1), dim3(1024), 0, s, a, min_live(BF16));
  if (bytes == 256) hipLaunchKernelGGL((pool_slab_kernel<BF16, MODE, 16>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((pool_slab_kernel<BF16, MODE, 8>), grid, block, 0, s, a);
  return hipGetLastError();
}

template <bool BF16, int MODE>
hipError_t launch_batched(const PoolLaunch& a, dim3 grid, dim3 block, int slabs, int vec_per_row,
                          hipStream_t s);

template <bool BF16, int MODE>
hipError_t launch_mode(PoolLaunch a, hipStream_t s) {
  constexpr int VN = BF16 ? 8 : 4;
  const int slabs = (a.m / VN + kWave - 1) / kWave;
  const int64_t blocks_needed = (a.rows + kWavesPerBlock - 1) / kWavesPerBlock;
  int64_t cap = 1ll << 22;
  if (const int bytes = slab_bytes(a)) {
    const hipError_t e = launch_slabs<BF16, MODE>(a, bytes, s);
    if (e != hipSuccess) return e;
    // Whole rows behind it. Ending 2^18 blocks takes up to 50 us of a pool in slabs
    // (1.2M rows of 1 KB, T = 50: 5.06 -> 5.11 ms); in 2^15 blocks whole rows that were
    // chosen take 4% longer (9.51 -> 9.89 ms, evenly spread).
    cap = 1ll << 18;
  } else {
    a.slabbed = nullptr;
  }
  const dim3 grid((unsigned)(blocks_needed < cap ? blocks_needed : cap));
  const dim3 block(256);
  const int vec_per_row = a.m / VN;
  // The header-in-registers kernel for rows narrower than a wave slab (it gathers
  // 1 KB per load instruction from two or four rows at once). Rows of a full
  // slab measured as fast or faster in the batched kernel (1.2M- and 12M-node
  // graphs: 6.49 against 6.61 ms, 25.1 against 25.3 ms), and much faster on
  // short neighbourhoods (graph neighbourhoods of about 3 pins: 0.84 against
  // 1.58 ms), where the header's round trip is most of a row's work.
  if (a.T <= kWave && vec_per_row <= kWave / 2) {
    if (vec_per_row <= kWave / 4)
      hipLaunchKernelGGL((pool_head_kernel<BF16, MODE, 4, 16>), grid, block, 0, s, a);
    else
      hipLaunchKernelGGL((pool_head_kernel<BF16, MODE, 2, 32>), grid, block, 0, s, a);
    return hipGetLastError();
  }
  return launch_batched<BF16, MODE>(a, grid, block, slabs, vec_per_row, s);
}

// Neighbourhoods of more than 64 slots, or rows wider than one slab.
template <bool BF16, int MODE>
hipError_t launch_batched(const PoolLaunch& a, dim3 grid, dim3 block, int slabs, int vec_per_row,
                          hipStream_t s) {
  if (vec_per_row <= kWave / 4)
    hipLaunchKernelGGL((pool_narrow_kernel<BF16, MODE, 4>), grid, block, 0, s, a);
  else if (vec_per_row <= kWave / 2)
    hipLaunchKernelGGL((pool_narrow_kernel<BF16, MODE, 2>), grid, block, 0, s, a);
  else if (slabs <= 1) hipLaunchKernelGGL((pool_kernel<BF16, MODE, 1>), grid, block, 0, s, a);
  else if (slabs <= 2) hipLaunchKernelGGL((pool_kernel<BF16, MODE, 2>), grid, block, 0, s, a);
  else if (slabs <= 4) hipLaunchKernelGGL((pool_kernel<BF16, MODE, 4>), grid, block, 0, s, a);
  else if (slabs <= 8) hipLaunchKernelGGL((pool_kernel<BF16, MODE, 8>), grid, block, 0, s, a);
  else if (slabs <= 16) hipLaunchKernelGGL((pool_kernel<BF16, MODE, 16>), grid, block, 0, s, a);
  else if (slabs <= 32) hipLaunchKernelGGL((pool_kernel<BF16, MODE, 32>), grid, block, 0, s, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

template <bool BF16>
hipError_t launch_typed(const PoolLaunch& a, hipStream_t s) {
  switch (a.mode) {
    case kPoolImportance: return launch_mode<BF16, kPoolImportance>(a, s);
    case kPoolMean: return launch_mode<BF16, kPoolMean>(a, s);
    case kPoolMax: return launch_mode<BF16, kPoolMax>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// Pools the slabs are for: tables of rows of 1 KB and more, 48 MB and more (byte
// offsets are 32 bits), and 8 GB or more to gather (about 1.2 ms), beside which the
// probe and the empty launch, about 35 us, count little.
bool pool_slabs_wanted(int64_t n_transform, int64_t row_bytes, int64_t rows, int T) {
  const int64_t table = n_transform * row_bytes;
  return row_bytes >= 1024 && table >= (48ll << 20) && table < (1ll << 32) - 16 &&
         rows * row_bytes * T >= (8ll << 30);
}

hipError_t launch_pool(const PoolLaunch& a, hipStream_t s) {
  if (a.rows <= 0) return hipSuccess;
  ProfileScope prof(kKPool, s);
  return a.bf16 ? launch_typed<true>(a, s) : launch_typed<false>(a, s);
}

}  // namespace pinsage
