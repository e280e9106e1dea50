// Minibatch forward support on gfx950 (Algorithm 2 and Sec. 3.3):
//  * frontier sets S^(k): the ids of a level are marked in a node-flag array,
//    and an exclusive scan over the flags yields, in one pass, the sorted
//    unique set and the global -> local position map used to re-index
//    neighbour ids and self rows into the compact sets (the re-indexing of
//    Sec. 3.3, done on the device);
//  * the max-margin loss of Eq. 1 over a shared negative set.
// Everything is integer or fixed-order fp32, hence deterministic.
#include <type_traits>

#include "device_util.h"
#include "kernels.h"
#include "split_device.h"

namespace pinsage {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kScanThreads = 256;
constexpr int kScanPerThread = 16;
constexpr int kScanTile = kScanThreads * kScanPerThread;  // flags per tile

__global__ void fill_u8_kernel(uint8_t* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0;
}

// Element i of up to four id lists one after another.
__device__ __forceinline__ int32_t list_at(const IdLists& l, int64_t i) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    if (i < l.n[k]) return l.ids[k][i];
    i -= l.n[k];
  }
  return l.ids[3][i];
}

__global__ void mark_kernel(IdLists ids, int64_t n, int64_t N, uint8_t* flags) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int32_t v = list_at(ids, i);
    if (v >= 0 && (int64_t)v < N) flags[v] = 1;
  }
}

// A thread's kScanPerThread flags (0 past N), 16 bytes in one load where all exist.
__device__ __forceinline__ void load_flags(const uint8_t* flags, int64_t base, int64_t N,
                                           uint8_t (&f)[kScanPerThread]) {
  static_assert(kScanPerThread == 16, "one 16-byte load");
  if (base + kScanPerThread <= N) {
    const uint4 v = *reinterpret_cast<const uint4*>(flags + base);
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < kScanPerThread; ++e) f[e] = (uint8_t)(w[e >> 2] >> (8 * (e & 3)));
  } else {
#pragma unroll
    for (int e = 0; e < kScanPerThread; ++e) f[e] = base + e < N ? flags[base + e] : 0;
  }
}

// Block-wide exclusive scan of one int per thread (blockDim.x a multiple of 64).
__device__ int block_exclusive_scan(int v, int* lds_waves, int* block_total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nwaves = blockDim.x >> 6;
  const int incl = wave_inclusive_sum(v, lane);
  if (lane == 63) lds_waves[wave] = incl;
  __syncthreads();
  if (wave == 0) {
    const int t = lane < nwaves ? lds_waves[lane] : 0;
    const int ti = wave_inclusive_sum(t, lane);
    if (lane < nwaves) lds_waves[lane] = ti - t;  // exclusive wave offsets
    if (lane == 63) lds_waves[64] = ti;
  }
  __syncthreads();
  const int res = lds_waves[wave] + incl - v;
  *block_total = lds_waves[64];
  __syncthreads();
  return res;
}

__global__ __launch_bounds__(kScanThreads) void scan_tile_sums_kernel(const uint8_t* flags,
                                                                      int64_t N, int32_t* sums) {
  __shared__ int lds[65];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPerThread;
  uint8_t f[kScanPerThread];
  load_flags(flags, base, N, f);
  int s = 0;
#pragma unroll
  for (int e = 0; e < kScanPerThread; ++e) s += f[e];
  int total = 0;
  block_exclusive_scan(s, lds, &total);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// counts[0] = flagged ids, and with all_below counts[1] as well.
__global__ __launch_bounds__(1024) void scan_tile_offsets_kernel(int32_t* sums, int64_t ntiles,
                                                                 long long* counts,
                                                                 bool all_below) {
  __shared__ int lds[65];
  long long carry = 0;
  for (int64_t c = 0; c < ntiles; c += blockDim.x) {
    const int64_t i = c + threadIdx.x;
    const int v = i < ntiles ? sums[i] : 0;
    int chunk = 0;
    const int ex = block_exclusive_scan(v, lds, &chunk);
    if (i < ntiles) sums[i] = (int32_t)(carry + ex);
    carry += chunk;
  }
  if (threadIdx.x == 0) {
    counts[0] = carry;
    if (all_below) counts[1] = carry;
  }
}

// set, pos; counts[1] = flagged ids below `bound` (when bound < N); the flags are
// left zero for the next level.
__global__ __launch_bounds__(kScanThreads) void scan_tile_finish_kernel(
    uint8_t* flags, int64_t N, const int32_t* offsets, int32_t* pos, int32_t* set, int64_t cap,
    int64_t bound, long long* counts) {
  __shared__ int lds[65];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPerThread;
  uint8_t f[kScanPerThread];
  load_flags(flags, base, N, f);
  int s = 0;
#pragma unroll
  for (int e = 0; e < kScanPerThread; ++e) s += f[e];
  int total = 0;
  int p = offsets[blockIdx.x] + block_exclusive_scan(s, lds, &total);
#pragma unroll
  for (int e = 0; e < kScanPerThread; ++e) {
    if (base + e == bound && base + e < N) counts[1] = p;
    if (f[e]) {
      pos[base + e] = p;
      if (p < cap) set[p] = (int32_t)(base + e);
      ++p;
      flags[base + e] = 0;
    }
  }
}

__global__ void remap_kernel(IdLists in, int64_t n, int64_t N, const int32_t* pos, int32_t* out) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int32_t v = list_at(in, i);
    out[i] = (v >= 0 && (int64_t)v < N) ? pos[v] : -1;
  }
}

template <bool BF16>
__device__ __forceinline__ float load_elem(const void* base, int64_t i) {
  if constexpr (BF16) return bf16_to_f32(static_cast<const uint16_t*>(base)[i]);
  else return static_cast<const float*>(base)[i];
}

// The 16-byte vector at element i, and s + the dot product of two in index order.
template <bool BF16>
__device__ __forceinline__ u32x4 load_vec(const void* base, int64_t i) {
  return *reinterpret_cast<const u32x4*>(static_cast<const unsigned char*>(base) +
                                         i * (BF16 ? 2 : 4));
}
template <bool BF16>
__device__ __forceinline__ float dot_vec(const u32x4& x, const u32x4& y, float s) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if constexpr (BF16) {
      s = fmaf(__uint_as_float(x[q] << 16), __uint_as_float(y[q] << 16), s);
      s = fmaf(__uint_as_float(x[q] & 0xFFFF0000u), __uint_as_float(y[q] & 0xFFFF0000u), s);
    } else {
      s = fmaf(__uint_as_float(x[q]), __uint_as_float(y[q]), s);
    }
  }
  return s;
}

// Elements k0 .. k0 + 7 of row `row` of a [rows][d] table as MFMA operand
// parts: the bf16 values themselves, or fp32 values split exactly into three
// bf16 parts (key: their least magnitude so far). Zeros for row < 0 and past d.
// VEC: rows are whole 16-byte vectors.
template <bool BF16, bool VEC>
__device__ __forceinline__ auto load_parts(const void* table, int64_t row, int d, int k0,
                                           uint32_t& key) {
  if constexpr (BF16) {
    u32x4 v = {0u, 0u, 0u, 0u};
    if (row < 0 || k0 >= d) return v;
    const uint16_t* src = static_cast<const uint16_t*>(table) + row * d + k0;
    if constexpr (VEC) {
      v = *reinterpret_cast<const u32x4*>(src);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (k0 + e < d) v[e >> 1] |= (uint32_t)src[e] << (16 * (e & 1));
    }
    return v;
  } else {
    u32x4 u = {0u, 0u, 0u, 0u}, v = u;
    if (row >= 0 && k0 < d) {
      const float* src = static_cast<const float*>(table) + row * d + k0;
      if constexpr (VEC) {  // d % 4 == 0
        u = *reinterpret_cast<const u32x4*>(src);
        if (k0 + 4 < d) v = *reinterpret_cast<const u32x4*>(src + 4);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (k0 + e < d) u[e] = __float_as_uint(src[e]);
          if (k0 + 4 + e < d) v[e] = __float_as_uint(src[4 + e]);
        }
      }
    }
    return split3(u, v, key);
  }
}

// fp32 elements k0 .. k0 + 3 of row `row`, zeros as above.
template <bool VEC>
__device__ __forceinline__ u32x4 load4_f32(const void* table, int64_t row, int d, int k0) {
  u32x4 u = {0u, 0u, 0u, 0u};
  if (row < 0 || k0 >= d) return u;
  const float* src = static_cast<const float*>(table) + row * d + k0;
  if constexpr (VEC) {
    u = *reinterpret_cast<const u32x4*>(src);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (k0 + e < d) u[e] = __float_as_uint(src[e]);
  }
  return u;
}

// Eq. (1) per pair. A block of 8 waves scores 16 queries against all the
// negatives on the matrix cores (v_mfma_f32_16x16x32_bf16; fp32 storage as
// split triples, eight MFMAs per product): the queries' operand parts sit in LDS,
// wave w takes negatives 16 (w + 8 i) .. + 15 and reads their rows straight
// from memory as operands (the negatives are shared by every block and stay in
// L2). A lane then holds one query's scores of 4 negatives; it adds its hinge
// terms in order, the 4 lanes of a query are summed by a fixed butterfly and
// the waves in order. The positive is a dot product of 32 threads, the pair's own
// hard negatives of 8 each, summed by fixed butterflies.
// What bounds it: the latency of the rows' reads. 2,048 pairs, 500 negatives,
// d = 256, with the mean's launch: 15.8 us in bf16 and 26.1 in fp32, where fp32
// FMAs from LDS took 47.0 and 49.7; with 4 hard negatives per pair 16.4 (50.6), with
// 64 28.6 (56.2); 256 pairs with 1,000 each 157 (183, fp32 246 and 287);
// 4,096 pairs, 1,000 + 16 negatives, d = 512: 50 (345).
// KS: most k-steps of 32 columns; TPQ threads per query.
template <bool BF16, bool VEC, int KS>
__global__ __launch_bounds__(512) void loss_pairs_kernel(LossLaunch a) {
  constexpr int QB = 16, WAVES = 8, TPQ = 32;
  constexpr int PARTS = BF16 ? 1 : 3;
  constexpr int U = BF16 ? 8 : 4;  // k-steps in flight; KS is a multiple
  __shared__ u32x4 qf[KS * PARTS * 64];
  __shared__ float pos_s[QB], hard_s[QB], sum_s[WAVES][QB];
  __shared__ int count_s[QB];
  __shared__ uint32_t key_s[QB];  // fp32: least magnitude of each query
  const int d = a.d, ksteps = (d + 31) / 32;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int64_t b0 = (int64_t)blockIdx.x * QB;
  auto row_of = [](const int32_t* map, int64_t i) { return map ? (int64_t)map[i] : i; };

  if (!BF16 && t < QB) key_s[t] = ~0u;
  if constexpr (!BF16) __syncthreads();
  // Queries as operands: lane l of k-step ks holds row l % 16, columns
  // 32 ks + 8 (l / 16) .. + 7 (zeros for missing pairs or ids).
  for (int i = t; i < (ksteps + U - 1) / U * U * 64; i += 512) {
    const int64_t b = b0 + (i & 15);
    const int64_t row = b < a.B ? row_of(a.q_rows, b) : -1;
    uint32_t key = ~0u;
    const auto f = load_parts<BF16, VEC>(a.zq, row, d, 32 * (i >> 6) + 8 * ((i >> 4) & 3), key);
    if constexpr (BF16) {
      qf[i] = f;
    } else {
      atomicMin(&key_s[i & 15], key);
#pragma unroll
      for (int p = 0; p < 3; ++p) qf[((i >> 6) * 3 + p) * 64 + (i & 63)] = f.p[p];
    }
  }
  // Positive score and hard negatives of query t / 32.
  {
    const int q = t / TPQ, c = t % TPQ;
    const int64_t b = b0 + q;
    const int64_t qr = b < a.B ? row_of(a.q_rows, b) : -1;
    auto dot = [&](const void* table, int64_t row) {
      float s = 0.0f;
      if (qr >= 0 && row >= 0)
        for (int k = c; k < d; k += TPQ)
          s = fmaf(load_elem<BF16>(a.zq, qr * d + k), load_elem<BF16>(table, row * d + k), s);
#pragma unroll
      for (int o = TPQ / 2; o >= 1; o >>= 1) s += __shfl_xor(s, o);
      return s;
    };
    const float pos = dot(a.zpos, b < a.B ? row_of(a.pos_rows, b) : -1);
    // Hard negatives: 8 threads per row, 4 U rows of the query at a time, all their
    // reads in flight at once (absent rows read row 0, so that no read waits for a
    // branch). One row after another by 32 threads each, 1,000 per pair took 2.1-3.3
    // ms in 256 pairs; one row per thread, 0.29-0.58.
    float hh = 0.0f;
    int hv = 0;
    auto hard = [&](auto rows_per_group, auto vectors) __attribute__((always_inline)) {
      constexpr int U = decltype(rows_per_group)::value;
      const int gl = c & 7, gr = c >> 3;
      for (int64_t j0 = gr; j0 - gr < a.k_hard; j0 += 4 * U) {
        int64_t rows[U], at[U];
        float s[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int64_t j = j0 + 4 * u;
          rows[u] = b < a.B && j < a.k_hard ? row_of(a.hard_rows, b * a.k_hard + j) : -1;
          at[u] = (rows[u] < 0 ? 0 : rows[u]) * d;
          s[u] = 0.0f;
        }
        if (qr >= 0) {
          if constexpr (decltype(vectors)::value) {
            constexpr int VE = BF16 ? 8 : 4;
#pragma unroll 2
            for (int k = VE * gl; k < d; k += 8 * VE) {
              u32x4 y[U];
#pragma unroll
              for (int u = 0; u < U; ++u) y[u] = load_vec<BF16>(a.zhard, at[u] + k);
              const u32x4 x = load_vec<BF16>(a.zq, qr * d + k);
#pragma unroll
              for (int u = 0; u < U; ++u) s[u] = dot_vec<BF16>(x, y[u], s[u]);
            }
          } else {
#pragma unroll 2
            for (int k = gl; k < d; k += 8) {
              float y[U];
#pragma unroll
              for (int u = 0; u < U; ++u) y[u] = load_elem<BF16>(a.zhard, at[u] + k);
              const float x = load_elem<BF16>(a.zq, qr * d + k);
#pragma unroll
              for (int u = 0; u < U; ++u) s[u] = fmaf(x, y[u], s[u]);
            }
          }
        }
#pragma unroll
        for (int o = 4; o >= 1; o >>= 1)
#pragma unroll
          for (int u = 0; u < U; ++u) s[u] += __shfl_xor(s[u], o);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const float h = s[u] - pos + a.margin;
          hh += rows[u] >= 0 && h > 0.0f ? h : 0.0f;
          hv += rows[u] >= 0 ? 1 : 0;
        }
      }
#pragma unroll
      for (int o = TPQ / 2; o >= 8; o >>= 1) {
        hh += __shfl_xor(hh, o);
        hv += __shfl_xor(hv, o);
      }
    };
    // Whole vectors where both tables start on one; these rows may come from anywhere.
    const uintptr_t starts = reinterpret_cast<uintptr_t>(a.zq) | reinterpret_cast<uintptr_t>(a.zhard);
    const std::integral_constant<int, 1> few{};
    const std::integral_constant<int, 4> many{};
    if (VEC && starts % 16 == 0) {
      if (a.k_hard > 4) hard(many, std::integral_constant<bool, VEC>{});
      else if (a.k_hard > 0) hard(few, std::integral_constant<bool, VEC>{});
    } else {
      if (a.k_hard > 4) hard(many, std::false_type{});
      else if (a.k_hard > 0) hard(few, std::false_type{});
    }
    if (c == 0) {
      pos_s[q] = pos;
      hard_s[q] = hh;
      count_s[q] = hv;
    }
  }
  __syncthreads();

  const float shift = a.margin - pos_s[lane & 15];
  uint32_t key_q = ~0u;  // of the block's queries
  if constexpr (!BF16) key_q = wave_min_key(key_s[lane & 15]);
  float acc = 0.0f;
  for (int64_t n0 = 16 * wave; n0 < a.n_neg; n0 += 16 * WAVES) {
    const int64_t n = n0 + (lane & 15);
    const int64_t row = n < a.n_neg ? row_of(a.neg_rows, n) : -1;
    f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f}, small = s;
    uint32_t key = ~0u;
    // U k-steps' rows in flight before the first is multiplied.
    for (int ks0 = 0; ks0 < ksteps; ks0 += U) {
      decltype(load_parts<BF16, VEC>(a.zneg, row, d, 0, key)) f[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        f[u] = load_parts<BF16, VEC>(a.zneg, row, d, 32 * (ks0 + u) + 8 * (lane >> 4), key);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const u32x4* q = qf + (ks0 + u) * PARTS * 64 + lane;
        if constexpr (BF16) {
          s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f[u]),
                                                      __builtin_bit_cast(bf16x8, q[0]), s, 0, 0,
                                                      0);
        } else {
#pragma unroll
          for (int i = 0; i < kSplitProducts; ++i) {
            f32x4& c = i < kSplitProducts - 1 ? small : s;
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, f[u].p[split_b(i)]),
                __builtin_bit_cast(bf16x8, q[64 * split_a(i)]), c, 0, 0, 0);
          }
        }
      }
    }
    if constexpr (!BF16) {
      s += small;
      // Scores whose rows the parts do not cover, and those that are not finite, are
      // taken from the same 16 x 16 scores in fp32 MFMAs (step e of 16 columns pairs
      // lane group l / 16 with column 4 (l / 16) + e).
      float probe = 0.0f;
#pragma unroll
      for (int r = 0; r < 4; ++r) probe = fmaf(s[r], 0.0f, probe);
      if (!split_covers(key_q, wave_min_key(key)) || __ballot(probe != 0.0f) != 0ull) {
        const int64_t bq = b0 + (lane & 15);
        const int64_t rq = bq < a.B ? row_of(a.q_rows, bq) : -1;
        f32x4 full = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
        for (int k0 = 4 * (lane >> 4); k0 - 4 * (lane >> 4) < d; k0 += 16) {
          const u32x4 y = load4_f32<VEC>(a.zneg, row, d, k0), x = load4_f32<VEC>(a.zq, rq, d, k0);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            full = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(y[e]),
                                                        __uint_as_float(x[e]), full, 0, 0, 0);
        }
        key = umin(key, (uint32_t)__shfl_xor((int)key, 16));
        key = umin(key, (uint32_t)__shfl_xor((int)key, 32));  // of negative n0 + l % 16
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const uint32_t kn = (uint32_t)__shfl((int)key, 4 * (lane >> 4) + r);
          const bool keep = split_covers(key_s[lane & 15], kn) && fabsf(s[r]) < INFINITY;
          s[r] = keep ? s[r] : full[r];
        }
      }
    }
    // Lane l: query l % 16, negatives n0 + 4 (l / 16) + 0..3.
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t nr = n0 + 4 * (lane >> 4) + r;
      const float x = s[r];
      const float h = x + shift;
      acc += (nr < a.n_neg && h > 0.0f) ? h : 0.0f;
    }
  }
  acc += __shfl_xor(acc, 16);
  acc += __shfl_xor(acc, 32);
  if (lane < QB) sum_s[wave][lane] = acc;
  __syncthreads();
  if (t < QB && b0 + t < a.B) {
    float total = 0.0f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) total += sum_s[w][t];
    a.per_pair[b0 + t] = (total + hard_s[t]) / (float)(a.n_neg + count_s[t]);
  }
}

// Mean over pairs in a fixed order: strided per-thread sums, then a fixed tree.
__global__ __launch_bounds__(256) void loss_mean_kernel(const float* per_pair, int64_t B,
                                                        float* loss) {
  __shared__ float part[256];
  float s = 0.0f;
  for (int64_t i = threadIdx.x; i < B; i += 256) s += per_pair[i];
  part[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w >= 1; w >>= 1) {
    if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *loss = part[0] / (float)B;
}

// out[i][:] = table[rows[i]][:] (zero row for rows[i] < 0); 16-byte vectors.
__global__ void gather_rows_kernel(const uint4* table, const int32_t* rows, int64_t n,
                                   int vec_per_row, uint4* out) {
  const int64_t total = n * vec_per_row;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / vec_per_row;
    const int c = (int)(i % vec_per_row);
    const int32_t src = rows[r];
    out[i] = src >= 0 ? table[(int64_t)src * vec_per_row + c] : make_uint4(0, 0, 0, 0);
  }
}

inline dim3 grid_for(int64_t n, int threads = 256) {
  int64_t b = (n + threads - 1) / threads;
  if (b < 1) b = 1;
  if (b > 65536) b = 65536;
  return dim3((unsigned)b);
}

}  // namespace

hipError_t launch_fill_zero_u8(uint8_t* p, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_u8_kernel, grid_for(n), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

static int64_t list_size(const IdLists& l) { return l.n[0] + l.n[1] + l.n[2] + l.n[3]; }

hipError_t launch_mark(const IdLists& ids, int64_t N, uint8_t* flags, hipStream_t s) {
  const int64_t n = list_size(ids);
  if (n <= 0) return hipSuccess;
  ProfileScope prof(kKMinibatch, s);
  hipLaunchKernelGGL(mark_kernel, grid_for(n), dim3(256), 0, s, ids, n, N, flags);
  return hipGetLastError();
}

int64_t scan_tiles(int64_t N) { return (N + kScanTile - 1) / kScanTile; }

hipError_t launch_flag_scan(uint8_t* flags, int64_t N, int32_t* tile_sums, int32_t* pos,
                            int32_t* set, int64_t cap, int64_t bound, long long* counts,
                            hipStream_t s) {
  const int64_t tiles = scan_tiles(N);
  if (tiles <= 0 || tiles > 0x7FFFFFFF) return hipErrorInvalidValue;
  ProfileScope prof(kKMinibatch, s);
  hipLaunchKernelGGL(scan_tile_sums_kernel, dim3((unsigned)tiles), dim3(kScanThreads), 0, s,
                     flags, N, tile_sums);
  hipLaunchKernelGGL(scan_tile_offsets_kernel, dim3(1), dim3(1024), 0, s, tile_sums, tiles, counts,
                     bound >= N);
  hipLaunchKernelGGL(scan_tile_finish_kernel, dim3((unsigned)tiles), dim3(kScanThreads), 0, s,
                     flags, N, tile_sums, pos, set, cap, bound, counts);
  return hipGetLastError();
}

hipError_t launch_remap(const IdLists& in, int64_t N, const int32_t* pos, int32_t* out,
                        hipStream_t s) {
  const int64_t n = list_size(in);
  if (n <= 0) return hipSuccess;
  ProfileScope prof(kKMinibatch, s);
  hipLaunchKernelGGL(remap_kernel, grid_for(n), dim3(256), 0, s, in, n, N, pos, out);
  return hipGetLastError();
}

hipError_t launch_gather_rows(const void* table, const int32_t* rows, int64_t n, int64_t row_bytes,
                              void* out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (row_bytes % 16) return hipErrorInvalidValue;
  const int vpr = (int)(row_bytes / 16);
  hipLaunchKernelGGL(gather_rows_kernel, grid_for(n * vpr), dim3(256), 0, s,
                     static_cast<const uint4*>(table), rows, n, vpr, static_cast<uint4*>(out));
  return hipGetLastError();
}

template <bool BF16, bool VEC>
void launch_loss_typed(const LossLaunch& a, hipStream_t s) {
  const dim3 grid((unsigned)((a.B + 15) / 16)), block(512);
  // The queries' operands in LDS: up to 32 KB (bf16) or 96 KB (fp32, d = 1024).
  if (a.d <= 256) hipLaunchKernelGGL((loss_pairs_kernel<BF16, VEC, 8>), grid, block, 0, s, a);
  else if (a.d <= 512) hipLaunchKernelGGL((loss_pairs_kernel<BF16, VEC, 16>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((loss_pairs_kernel<BF16, VEC, 32>), grid, block, 0, s, a);
}

hipError_t launch_loss(const LossLaunch& a, hipStream_t s) {
  if (a.B <= 0) return hipSuccess;
  if (a.d < 1 || a.d > 1024 || a.B >= (1ll << 32)) return hipErrorInvalidValue;
  ProfileScope prof(kKLoss, s);
  // Whole-vector rows: operands load as 16 bytes per lane, else by element.
  const bool vec = a.d % (a.bf16 ? 8 : 4) == 0;
  if (a.bf16) vec ? launch_loss_typed<true, true>(a, s) : launch_loss_typed<true, false>(a, s);
  else vec ? launch_loss_typed<false, true>(a, s) : launch_loss_typed<false, false>(a, s);
  hipLaunchKernelGGL(loss_mean_kernel, dim3(1), dim3(256), 0, s, a.per_pair, a.B, a.loss);
  return hipGetLastError();
}

}  // namespace pinsage
