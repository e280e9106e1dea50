// Dense layers of CONVOLVE on gfx950 matrix cores (Algorithm 1):
//   line 1 over every pin once (Sec. 3.4):  P = ReLU(H Q^T + q)
//   lines 2-3:  h' = normalize(ReLU([h_self | n] W^T + w))
// as one templated MFMA GEMM  C = epi(A B^T + bias), A [M x K] assembled from
// two row sources (self rows through an optional row map, then the pooled
// rows), B [N x K] with a row stride (the PyTorch Linear layout of Q and W,
// or a column block of W).
//
// Work split: a block of WAVES_M x WAVES_N waves owns a BM x BN output tile;
// each wave owns (BM/WAVES_M) x (BN/WAVES_N), i.e. TM x TN blocks of 32 x 32.
//
// K pipeline: K runs in chunks of 64 bytes per row (32 bf16 / 16 fp32
// columns). Chunks travel global -> LDS by DMA (global_load_lds_dwordx4, no
// register staging) into a ring of STAGES LDS stages, STAGES - 1 chunks ahead
// of the MFMAs; one barrier per chunk. A stage packs rows in groups of 16; one
// DMA instruction of a wave fills one group (1 KB, row r of the group at
// 64 r): lanes 4r .. 4r+3 carry the four 16-byte vectors of row r, so a quad
// of lanes reads one contiguous 64-byte piece of a row. Inside a row, vector v
// sits in slot v ^ f(r), f(r) = ((r >> 1) ^ (r >> 3)) & 3, which spreads the
// 16 (resp. 8) rows of one LDS fragment read over distinct banks. Missing rows
// and the K tail read a static zero row, so loads never branch.
//
// bf16 storage: v_mfma_f32_32x32x16_bf16 (gfx950); k-step ks of a chunk takes
// vector 2ks + h in half-wave h. fp32 accumulation. The weight fragment is the
// MFMA's first operand, so the accumulators hold C^T blocks: a lane owns one
// output row and runs of 4 adjacent output columns, stored as one 8-byte (bf16)
// or 16-byte (fp32) vector.
//
// fp32 storage: the matrix cores run bf16 16 times as fast as fp32, so every
// operand is split exactly into three bf16 parts (split3) and the eight products
// of parts that reach fp32's last bits run as bf16 MFMAs, the leading one and
// the seven small ones in accumulators of their own. That is no less precise
// than the fp32 MFMA it replaces: relative error (2-norm, against 64 bits) of a
// K = 256 product 0.9e-7 against 2.8e-7, K = 512 1.3e-7 against 4.0e-7, K = 768
// with the row norm 1.0e-7 against 2.9e-7 (each MFMA rounds the running sum
// once per 16 columns instead of once per 2; with all in one accumulator it
// is 2.4e-7), and a lone product is within 1.01 half units in the last place. With
// six products (12% less time) the 2-norms are the same, but a lone product was up
// to 1.7 half units off, where fp32 rounds it once.
// Operands beyond the parts' range (split_covers) and sums that are not finite send
// their tile through fp32 MFMAs as well, which take the elements concerned.
// What bounds it: the MFMAs and the power they draw (64% busy at K = 256, at about
// 1.7 of 2.4 GHz) beside the VALU work of the splits, 56 instructions per 8 x 64
// values; a wave therefore covers
// 64 x 64 (64 accumulators of each kind, two waves per SIMD), the next chunk is
// split among the current one's MFMAs, and products of many rows read weights
// that one small kernel split beforehand (split_b_kernel, PRE). 1M rows, 256 ->
// 512: 2.34 ms (112 TFLOP/s) with fp32 MFMAs, 1.93 (136) so; 512 -> 256: 2.20,
// 1.75; 1.2M rows of the W layer (768 -> 256, norm): 4.12, 3.09 (153 TFLOP/s). Looking
// for the least magnitudes is 1-6% of that.
// (The row-norm tiles of 256 and 512 columns keep up to 56 bytes a lane in scratch.)
// (The remainders as two-element bf16 dot products are fewer instructions, but
// those run on the matrix pipe: 9% slower.)
//
// Epilogue: + bias, + an optional addend matrix (the pooled neighbour term
// when W is split, see run_layer), ReLU (optional without L2), store in the
// storage dtype; with L2 the block spans
// all N columns, and a row's sum of squares is added over a lane's own columns, its
// partner half-wave and then the groups of 64 (bf16 512 outputs: 128) columns in
// order, through LDS; every row is scaled by 1/||z|| (zero rows stay zero).
//
// Tile order is XCD-aware: hardware hands block b to XCD b % 8; blocks are
// renumbered so that each XCD gets a contiguous run of tiles, keeping the
// column tiles of one row block on one XCD's L2.
#include <type_traits>

#include "device_util.h"
#include "kernels.h"
#include "split_device.h"

namespace pinsage {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

// A row of zeros as long as the widest A row (d_in + m <= 16384 fp32): rows
// that do not exist and the K tail read from here. Never written.
constexpr int kMaxGemmK = 16384;
__device__ __attribute__((aligned(16))) float g_zero_row[kMaxGemmK];

constexpr int kChunkRowBytes = 64;   // bytes of one row per K chunk
constexpr int kGroupBytes = 1024;    // 16 rows x 64 bytes: one DMA instruction

// Slot of 16-byte vector v of row r (r mod 16) inside the row's 64 bytes.
__device__ __forceinline__ int vec_slot(int r, int v) { return v ^ (((r >> 1) ^ (r >> 3)) & 3); }

template <bool BF16, int BM_, int BN_, int WAVES_M_, int WAVES_N_, bool L2_, int STAGES_,
          int WPE_ = 1, bool PRE_ = false, bool ROT_ = false>
struct Cfg {
  static constexpr bool ROT = ROT_;  // bf16: the K sweep starts where the product's large tile does
  static constexpr bool PRE = PRE_;  // fp32: B arrives split (launch_split_b)
  static constexpr int WPE = WPE_;  // waves per SIMD the register budget must allow
  static constexpr bool kBf16 = BF16;
  static constexpr bool kTwoSources = L2_;  // the W layer reads [h_self | n]
  static constexpr bool L2 = L2_;
  static constexpr int BM = BM_, BN = BN_;
  static constexpr int WAVES_M = WAVES_M_, WAVES_N = WAVES_N_;
  static constexpr int NWAVES = WAVES_M * WAVES_N;
  static constexpr int THREADS = 64 * NWAVES;
  static constexpr int STAGES = STAGES_;
  static constexpr int ESZ = BF16 ? 2 : 4;       // bytes per element
  static constexpr int VEC = 16 / ESZ;            // elements per 16-byte vector
  static constexpr int BK = kChunkRowBytes / ESZ; // K columns per chunk
  static constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
  static constexpr int TM = WM / 32, TN = WN / 32;
  // A stage: A_GROUPS groups of 16 A rows, then B's groups (of 16 rows, or the
  // 32-row block parts of split B). Each wave issues the same number of DMAs;
  // the groups that a rounded-up split adds take the zero row. With split B, a
  // wave's first A_DPW DMAs are A's and the rest B's.
  static constexpr int B_GROUPS = PRE ? BN / 32 * 3 : BN / 16;
  static constexpr int A_GROUPS = PRE ? (BM / 16 + NWAVES - 1) / NWAVES * NWAVES : BM / 16;
  static constexpr int GROUPS = (A_GROUPS + B_GROUPS + NWAVES - 1) / NWAVES * NWAVES;
  static constexpr int DPW = GROUPS / NWAVES;     // DMA instructions per wave per chunk
  static constexpr int ROW_DPW = PRE ? A_GROUPS / NWAVES : DPW;  // of them, row groups
  static constexpr int PENDING = (STAGES - 2) * DPW;
  static constexpr int STAGE_BYTES = GROUPS * kGroupBytes;
  // Sums of squares of a row: per group of 32-column blocks (a wave's of the large
  // shapes), or per block and half-wave where a wave holds less than a group.
  static constexpr int NORM_GROUP = BF16 && BN > 256 ? 4 : 2;
  static constexpr bool NORM_WHOLE = TN == NORM_GROUP;
  static constexpr int NORM_SUMS = NORM_WHOLE ? WAVES_N : BN / 16;
  static_assert(!L2_ || NORM_GROUP % TN == 0, "a wave holds a group or a part of one");
  static constexpr int RED_BYTES = L2 ? NORM_SUMS * BM * 4 : 0;
  static constexpr int BIAS_BYTES = BN * 4;
  static constexpr int FLAG_BYTES = BF16 ? 0 : 16;  // fp32: some wave's results need a redo
  static constexpr int LDS_BYTES = STAGES * STAGE_BYTES + RED_BYTES + BIAS_BYTES + FLAG_BYTES;
  // The redo's stages: A and B rows as they are, RAW_DPW row groups per wave.
  static constexpr int RAW_DPW = ((BM + BN) / 16 + NWAVES - 1) / NWAVES;
  static_assert(RAW_DPW * NWAVES <= GROUPS, "a raw stage fits the ring's");
  static_assert(WM % 32 == 0 && WN % 32 == 0, "wave tile is a multiple of 32x32");
  static_assert(STAGES >= 2 && PENDING <= 63, "vmcnt range");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS budget of one workgroup");
};

__device__ __forceinline__ int xcd_tile(int b, int nt) {
  const int per = nt / 8, rem = nt % 8;
  const int xcd = b % 8, slot = b / 8;
  return xcd < rem ? xcd * (per + 1) + slot : rem * (per + 1) + (xcd - rem) * per + slot;
}

// One 16-byte-per-lane DMA from global memory into LDS: lane l's vector lands
// at byte lds_base + 16 l (lds_base wave-uniform, via M0).
__device__ __forceinline__ void dma16(const void* g, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
               :
               : "s"(lds_base), "v"(g)
               : "memory");
}

// The same with a wave-uniform base and a 32-bit byte offset per lane.
__device__ __forceinline__ void dma16_base(const void* base, uint32_t off, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(lds_base), "v"(off), "s"(base)
               : "memory");
}

// Waits until at most N vector-memory operations of this wave are in flight.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

// Workgroup barrier after this wave's LDS operations have completed.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory");
}

__device__ __forceinline__ f32x16 mfma_split(const Split3& b, const Split3& a, int t,
                                             const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, b.p[split_b(t)]),
                                                 __builtin_bit_cast(bf16x8, a.p[split_a(t)]), c, 0,
                                                 0, 0);
}

template <typename C>
__global__ __launch_bounds__(C::THREADS, C::WPE) void gemm_kernel(GemmLaunch a) {
  constexpr int BM = C::BM, BN = C::BN, BK = C::BK, VEC = C::VEC;
  constexpr int TM = C::TM, TN = C::TN, THREADS = C::THREADS, ESZ = C::ESZ;
  constexpr int DPW = C::DPW, ROW_DPW = C::ROW_DPW, STAGES = C::STAGES;
  // LDS: the stage ring, then the cross-wave row-norm partials and the
  // block's bias slice.
  __shared__ __attribute__((aligned(1024))) unsigned char smem[C::LDS_BYTES];
  float* red = reinterpret_cast<float*>(smem + STAGES * C::STAGE_BYTES);
  float* bias_s = reinterpret_cast<float*>(smem + STAGES * C::STAGE_BYTES + C::RED_BYTES);
  const uint32_t smem_base =
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / C::WAVES_N, wn = wave % C::WAVES_N;

  const int tiles_n = (a.N + BN - 1) / BN;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int64_t m0 = (int64_t)(tile / tiles_n) * BM;
  const int n0 = (tile % tiles_n) * BN;
  const int K = a.K0 + a.K1;
  // Bias slice of the block (zero past N).
  for (int c = tid; c < BN; c += THREADS)
    bias_s[c] = (a.bias && n0 + c < a.N) ? a.bias[n0 + c] : 0.0f;
  const int64_t ldb = a.ldb ? a.ldb : K;
  int* const redo_s = reinterpret_cast<int*>(smem + C::LDS_BYTES - C::FLAG_BYTES);
  if constexpr (!C::kBf16)
    if (tid == 0) *redo_s = 0;

  // ---- DMA slots (fixed across the K loop) --------------------------------
  // Slot d of this wave fills group wave*DPW + d of every stage: A groups
  // first, then B groups. Lane l serves row 16 * group + (l >> 2) and LDS
  // slot l & 3 of it, i.e. column vector vec_slot(l >> 2, l & 3). Source-1
  // pointers are biased by -K0 columns so both sources take the column kk;
  // rows that do not exist point at the zero row.
  const unsigned char* const zrow = reinterpret_cast<const unsigned char*>(g_zero_row);
  const int64_t k0b = (int64_t)a.K0 * ESZ;
  const int nb32 = (a.N + 31) / 32;  // 32-row blocks of split B
  // This lane's row of a group, A groups [0, a_groups) first.
  auto row_of_group = [&](int grp, int a_groups, const unsigned char*& q0,
                          const unsigned char*& q1) __attribute__((always_inline)) {
    const int rr = lane >> 2;
    if (grp < a_groups) {
      const int64_t gr = m0 + grp * 16 + rr;
      const bool in_m = gr < a.M && grp < BM / 16;
      const int64_t src = !in_m ? -1 : (a.rowmap ? (int64_t)a.rowmap[gr] : gr);
      q0 = (src >= 0 && src < a.rows_a0)
               ? static_cast<const unsigned char*>(a.A0) + src * a.lda0 * ESZ
               : zrow;
      if constexpr (C::kTwoSources) {
        const unsigned char* q = (in_m && a.A1)
                                     ? static_cast<const unsigned char*>(a.A1) + gr * a.lda1 * ESZ
                                     : zrow;
        q1 = reinterpret_cast<const unsigned char*>(reinterpret_cast<uintptr_t>(q) - k0b);
      }
    } else {
      const int r = n0 + (grp - a_groups) * 16 + rr;
      q0 = r < a.N ? static_cast<const unsigned char*>(a.B) + (int64_t)r * ldb * ESZ : zrow;
      if constexpr (C::kTwoSources) q1 = q0;
    }
  };
  const unsigned char* p0[ROW_DPW];
  const unsigned char* p1[C::kTwoSources ? ROW_DPW : 1];
#pragma unroll
  for (int d = 0; d < ROW_DPW; ++d)
    row_of_group(wave * ROW_DPW + d, C::A_GROUPS, p0[d], p1[C::kTwoSources ? d : 0]);
  const int kvec = vec_slot(lane >> 2, lane & 3) * VEC;
  const int nchunks = (K + BK - 1) / BK;
  // The large bf16 tiles start their K sweep at different chunks (rotation by
  // the tile's index in the whole product): rows of A and B sit at power-of-two
  // strides, and blocks that all read the same K columns at once would pile onto
  // a few L2 channels. Smaller tiles of the same product (few rows) rotate as the
  // large tile around them would, so that a row's bits do not depend on the tile
  // shape its launch takes; products whose large tiles are fp32, or narrow, or
  // gemm_rs_kernel's sum K in order (where it measured neutral).
  int kshift = 0;
  if constexpr (C::ROT) {  // large tiles: 128 rows by all columns (row norm), 256 x 256
    const uint32_t tm = (uint32_t)((a.row_base + m0) >> (C::L2 ? 7 : 8));
    kshift = (int)((C::L2 ? tm : tm * (uint32_t)((a.N + 255) >> 8) + (n0 >> 8)) % (uint32_t)nchunks);
  }
  // Issues the DMAs of the chunk-th chunk of this tile's sweep into its
  // stage. Sweep positions past the end read the zero row, which keeps the
  // in-flight count uniform for wait_vmcnt.
  auto issue = [&](int chunk) __attribute__((always_inline)) {
    int kc = chunk + kshift;
    kc = chunk >= nchunks ? nchunks : (kc >= nchunks ? kc - nchunks : kc);
    const int kk = kc * BK + kvec;
    const bool kin = kk < K;
    const int64_t off = (int64_t)kk * ESZ;
    const uint32_t dst = smem_base + (uint32_t)((chunk % STAGES) * C::STAGE_BYTES);
    const uint32_t dst_rows = dst + (uint32_t)(wave * ROW_DPW * kGroupBytes);
#pragma unroll
    for (int d = 0; d < ROW_DPW; ++d) {
      const unsigned char* p;
      if constexpr (C::kTwoSources) p = (kk < a.K0 ? p0[d] : p1[d]) + off;
      else p = p0[d] + off;
      dma16(kin ? p : zrow, __builtin_amdgcn_readfirstlane(dst_rows + d * kGroupBytes));
    }
    if constexpr (C::PRE) {
      // 1 KB each of split B's chunk: 32-row block n0 / 32 + gb / 3, part gb % 3.
      const unsigned char* const chunk_b =
          static_cast<const unsigned char*>(a.Bs) + (int64_t)kc * nb32 * 3072;
#pragma unroll
      for (int d = 0; d < DPW - ROW_DPW; ++d) {
        const int gb = wave * (DPW - ROW_DPW) + d;
        const int blk = n0 / 32 * 3 + gb;
        const bool in = chunk < nchunks && gb < C::B_GROUPS && blk < 3 * nb32;
        dma16_base(in ? chunk_b + blk * 1024 : zrow, 16u * (uint32_t)lane,
                   __builtin_amdgcn_readfirstlane(dst + (C::A_GROUPS + gb) * kGroupBytes));
      }
    }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  const int row_in_blk = lane & 31;
  const int half = lane >> 5;
  const int a_base_row = wm * C::WM;
  const int b_base_row = wn * C::WN;
  // Byte offset of a lane's fragment row (block-relative row r of A, resp.
  // B) in a stage. Fragment rows start at multiples of 32, so the row's place
  // in its group (lane & 15) and hence its vector slots depend on the lane.
  auto frag_off = [&](int r) __attribute__((always_inline)) {
    return (r >> 4) * kGroupBytes + (r & 15) * kChunkRowBytes;
  };
  const int fa_off = frag_off(a_base_row + row_in_blk);
  const int fb_off = C::A_GROUPS * kGroupBytes + frag_off(b_base_row + row_in_blk);
  // Byte offset of the vector a lane reads in half-step hs (bf16), or of the
  // hs-th vector of its eight columns (fp32).
  auto vec_off = [&](int hs) __attribute__((always_inline)) {
    const int v = C::kBf16 ? 2 * hs + half : 2 * half + hs;
    return vec_slot(lane & 15, v) * 16;
  };
  const int voff0 = vec_off(0), voff1 = vec_off(1);

  constexpr int FW = 4;  // 32-bit words per 16-byte vector
  typedef uint32_t frag_t __attribute__((ext_vector_type(FW)));
  auto stage_of = [&](int chunk) __attribute__((always_inline)) {
    return smem + (chunk % STAGES) * C::STAGE_BYTES;
  };

  if constexpr (C::kBf16) {
    // A chunk is multiplied in two half-steps hs = 0, 1 (the MFMA k-steps);
    // half-wave h reads column vector 2hs + h.
    struct Frags {
      frag_t a[TM], b[TN];
    };
    auto read_frags = [&](const unsigned char* stage, int hs, Frags& f)
        __attribute__((always_inline)) {
      const int v = hs ? voff1 : voff0;
#pragma unroll
      for (int i = 0; i < TM; ++i)
        f.a[i] = *reinterpret_cast<const frag_t*>(stage + fa_off + i * 2 * kGroupBytes + v);
#pragma unroll
      for (int j = 0; j < TN; ++j)
        f.b[j] = *reinterpret_cast<const frag_t*>(stage + fb_off + j * 2 * kGroupBytes + v);
    };
    auto mfma_half = [&](const Frags& f) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              __builtin_bit_cast(bf16x8, f.b[j]), __builtin_bit_cast(bf16x8, f.a[i]), acc[i][j],
              0, 0, 0);
    };

    // Ring protocol: chunks 0..STAGES-2 are in flight before the loop. Before
    // the fragments of chunk c+1 are read, each wave waits for its DMAs of that
    // chunk (STAGES - 2 younger chunks may stay in flight) and for its own LDS
    // reads of chunk c, then a barrier makes all DMAs visible and frees chunk
    // c's stage, which receives chunk c + STAGES. The half-step MFMAs issued
    // just before the barrier keep the matrix pipe busy across it.
#pragma unroll
    for (int c = 0; c < STAGES - 1; ++c) issue(c);
    wait_vmcnt<C::PENDING>();
    lds_barrier();
    issue(STAGES - 1);
    Frags f0, f1;
    read_frags(stage_of(0), 0, f0);
    // The last chunk is peeled off so the loop body has no branch: every
    // half-step's fragment reads then have a known count of younger reads.
    // Scheduling barriers pin the order: fragment reads go out right before a
    // half-step's 16 MFMAs that hide their latency.
    for (int c = 0; c + 1 < nchunks; ++c) {
      read_frags(stage_of(c), 1, f1);
      __builtin_amdgcn_sched_barrier(0);
      mfma_half(f0);
      __builtin_amdgcn_sched_barrier(0);
      wait_vmcnt<C::PENDING>();
      lds_barrier();
      read_frags(stage_of(c + 1), 0, f0);
      __builtin_amdgcn_sched_barrier(0);
      issue(c + STAGES);
      __builtin_amdgcn_sched_barrier(0);
      mfma_half(f1);
      __builtin_amdgcn_sched_barrier(0);
    }
    read_frags(stage_of(nchunks - 1), 1, f1);
    mfma_half(f0);
    mfma_half(f1);
  } else {
    // fp32 storage: one k-step of 16 columns per chunk; half-wave h takes
    // columns 8h .. 8h+7 (vectors 2h, 2h+1) and splits them into bf16 triples.
    f32x16 small[TM][TN];  // the products below the leading one
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) small[i][j][e] = 0.0f;
    struct Parts {
      Split3 a[TM], b[TN];
    };
    struct Raw {
      frag_t a[TM][2], b[C::PRE ? 1 : TN][2];
    };
    auto read_raw = [&](const unsigned char* st, Raw& r) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        r.a[i][0] = *reinterpret_cast<const frag_t*>(st + fa_off + i * 2 * kGroupBytes + voff0);
        r.a[i][1] = *reinterpret_cast<const frag_t*>(st + fa_off + i * 2 * kGroupBytes + voff1);
      }
      if constexpr (!C::PRE)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        r.b[j][0] = *reinterpret_cast<const frag_t*>(st + fb_off + j * 2 * kGroupBytes + voff0);
        r.b[j][1] = *reinterpret_cast<const frag_t*>(st + fb_off + j * 2 * kGroupBytes + voff1);
      }
    };
    auto read_parts = [&](const unsigned char* st, Parts& s) __attribute__((always_inline)) {
      if constexpr (C::PRE)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int t = 0; t < 3; ++t)
            s.b[j].p[t] = *reinterpret_cast<const u32x4*>(
                st + C::A_GROUPS * kGroupBytes + ((wn * TN + j) * 3 + t) * 1024 + 16 * lane);
    };
    // Least magnitudes of the values this lane has split (split_b_kernel's for split B).
    uint32_t key_a = ~0u, key_b = ~0u;
    auto split_raw = [&](const Raw& r, Parts& s) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < TM; ++i) s.a[i] = split3(r.a[i][0], r.a[i][1], key_a);
      if constexpr (!C::PRE)
#pragma unroll
        for (int j = 0; j < TN; ++j) s.b[j] = split3(r.b[j][0], r.b[j][1], key_b);
    };
    auto multiply = [&](const Parts& s) __attribute__((always_inline)) {
#pragma unroll
      for (int t = 0; t < kSplitProducts; ++t)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            if (t < kSplitProducts - 1) small[i][j] = mfma_split(s.b[j], s.a[i], t, small[i][j]);
            else acc[i][j] = mfma_split(s.b[j], s.a[i], t, acc[i][j]);
          }
    };
    // Ring protocol: chunks 0..STAGES-1 are in flight before the loop. Step c
    // waits for this wave's DMAs of chunk c + 1 (STAGES - 2 younger chunks stay
    // in flight); the barrier makes everybody's visible and frees chunk c's
    // stage (read and split in the step before) for chunk c + STAGES. Chunk
    // c + 1 is read and split among the MFMAs of chunk c.
    auto step = [&](int c, const Parts& cur, Parts& nxt) __attribute__((always_inline)) {
      wait_vmcnt<C::PENDING>();
      lds_barrier();
      issue(c + STAGES);
      Raw r;
      read_raw(stage_of(c + 1), r);
      read_parts(stage_of(c + 1), nxt);
      __builtin_amdgcn_sched_barrier(0);
      split_raw(r, nxt);
      multiply(cur);
      constexpr int kMfma = kSplitProducts * TM * TN;
      constexpr int kValu = 56 * (TM + (C::PRE ? 0 : TN));
#pragma unroll
      for (int q = 0; q < kMfma; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                            // MFMA
        __builtin_amdgcn_sched_group_barrier(0x002, (kValu + kMfma - 1) / kMfma, 0);  // VALU
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    Parts s0, s1;
#pragma unroll
    for (int c = 0; c < STAGES; ++c) issue(c);
    wait_vmcnt<C::PENDING + DPW>();
    lds_barrier();
    {
      Raw r;
      read_raw(stage_of(0), r);
      read_parts(stage_of(0), s0);
      split_raw(r, s0);
    }
    // An odd chunk count multiplies one more chunk, all zeros.
    for (int c = 0; c < nchunks; c += 2) {
      step(c, s0, s1);
      step(c + 1, s1, s0);
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] += small[i][j];
    // What the split does not cover shows in the operands' least magnitudes, or, for
    // infinities, NaN and values or sums that round to an infinity, in the results.
    // Such elements are taken from the same product in fp32 MFMAs.
    if constexpr (C::PRE) {
      const uint32_t* const keys = reinterpret_cast<const uint32_t*>(
          static_cast<const unsigned char*>(a.Bs) + (int64_t)nchunks * nb32 * 3072);
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int blk = (n0 + b_base_row) / 32 + j;
        if (blk < nb32) key_b = umin(key_b, keys[blk]);
      }
    }
    float probe = 0.0f;  // NaN unless all results are finite
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) probe = fmaf(acc[i][j][e], 0.0f, probe);
    const bool covered = split_covers(wave_min_key(key_a), wave_min_key(key_b)) &&
                         __ballot(probe != 0.0f) == 0ull;
    if (!covered && lane == 0) *redo_s = 1;
  }
  wait_vmcnt<0>();  // drain the zero-row DMAs issued past the end
  __syncthreads();  // bias slice (and, below, row partials) visible

  if constexpr (!C::kBf16) {
    if (*redo_s) {
      // The tile again with fp32 MFMAs (st of a chunk pairs half-wave h with its
      // column 8h + st), two raw stages in the ring. Each element then follows from
      // its own row and column alone: split where those are covered and the sum is
      // finite, else fp32, so that it does not depend on the tile it lies in. About
      // the time of the fp32 MFMA product on top, in the tiles that need it.
      constexpr int RAW_DPW = C::RAW_DPW, RAW_A = BM / 16;
      const unsigned char* q0[RAW_DPW];
      const unsigned char* q1[C::kTwoSources ? RAW_DPW : 1];
#pragma unroll
      for (int d = 0; d < RAW_DPW; ++d)
        row_of_group(wave * RAW_DPW + d, RAW_A, q0[d], q1[C::kTwoSources ? d : 0]);
      auto issue_raw = [&](int c) __attribute__((always_inline)) {
        const int kk = c * BK + kvec;
        const uint32_t dst = smem_base + (uint32_t)((c & 1) * C::STAGE_BYTES) +
                             (uint32_t)(wave * RAW_DPW * kGroupBytes);
#pragma unroll
        for (int d = 0; d < RAW_DPW; ++d) {
          const unsigned char* p = q0[d];
          if constexpr (C::kTwoSources) p = kk < a.K0 ? q0[d] : q1[d];
          dma16(kk < K ? p + (int64_t)kk * ESZ : zrow,
                __builtin_amdgcn_readfirstlane(dst + d * kGroupBytes));
        }
      };
      f32x16 full[TM][TN];
      uint32_t key_a[TM], key_b[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) key_a[i] = ~0u;
#pragma unroll
      for (int j = 0; j < TN; ++j) key_b[j] = ~0u;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e) full[i][j][e] = 0.0f;
      const int rb_off = RAW_A * kGroupBytes + frag_off(b_base_row + row_in_blk);
      issue_raw(0);
#pragma unroll 1
      for (int c = 0; c < nchunks; ++c) {
        wait_vmcnt<0>();
        lds_barrier();  // chunk c is here; everybody is done with chunk c - 1
        if (c + 1 < nchunks) issue_raw(c + 1);
        const unsigned char* const st = smem + (c & 1) * C::STAGE_BYTES;
        frag_t fa[TM][2], fb[TN][2];
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          fa[i][0] = *reinterpret_cast<const frag_t*>(st + fa_off + i * 2 * kGroupBytes + voff0);
          fa[i][1] = *reinterpret_cast<const frag_t*>(st + fa_off + i * 2 * kGroupBytes + voff1);
          key_a[i] = least_key(fa[i][0], fa[i][1], key_a[i]);
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          fb[j][0] = *reinterpret_cast<const frag_t*>(st + rb_off + j * 2 * kGroupBytes + voff0);
          fb[j][1] = *reinterpret_cast<const frag_t*>(st + rb_off + j * 2 * kGroupBytes + voff1);
          key_b[j] = least_key(fb[j][0], fb[j][1], key_b[j]);
        }
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
              full[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                  __uint_as_float(fb[j][q >> 2][q & 3]), __uint_as_float(fa[i][q >> 2][q & 3]),
                  full[i][j], 0, 0, 0);
      }
      // A lane's row of block i; the column of its element e of block j is lane
      // 8 (e / 4) + 4 half + e % 4's.
#pragma unroll
      for (int i = 0; i < TM; ++i)
        key_a[i] = umin(key_a[i], (uint32_t)__shfl_xor((int)key_a[i], 32));
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        key_b[j] = umin(key_b[j], (uint32_t)__shfl_xor((int)key_b[j], 32));
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const uint32_t kb = (uint32_t)__shfl((int)key_b[j], 8 * (e >> 2) + 4 * half + (e & 3));
#pragma unroll
          for (int i = 0; i < TM; ++i) {
            const float x = acc[i][j][e];
            const bool keep = split_covers(key_a[i], kb) && fabsf(x) < INFINITY;
            acc[i][j][e] = keep ? x : full[i][j][e];
          }
        }
      }
      __syncthreads();  // the ring is free for the epilogue
    }
  }

  // ---- epilogue -----------------------------------------------------------
  // Lane l: output row m0 + a_base_row + 32i + l%32; for group g of tile j,
  // output columns c0(j, g) + 0..3 with c0 = b_base_row + 32j + 8g + 4(l/32)
  // inside the block. N is a multiple of 16, so a group is all in or all out;
  // columns past N have zero weights and zero bias, so they stay zero.
  // Row bands are finished one at a time to keep few accumulators live.
  auto c0 = [&](int j, int g) __attribute__((always_inline)) { return b_base_row + j * 32 + 8 * g + 4 * half; };
  // The output leaves through the (now free) stage ring as whole rows, 16 bytes
  // per lane, rows padded by 16 bytes, instead of as each lane's 4-column pieces
  // of 32 rows per store instruction (measured neutral at 1M x 256 -> 512, and
  // the addend's reads become whole rows too). bf16 tiles that fit are staged
  // whole. (Loading the addend tile the same way, in
  // front of the epilogue, measured slower: its latency is then exposed.)
  constexpr int TROW = BN * ESZ + 16;
  constexpr int NORM_SUMS = C::NORM_SUMS;  // per row, side by side
  constexpr bool kStaged = C::kBf16 && BM * TROW <= STAGES * C::STAGE_BYTES;
  constexpr int PER_ROW = BN / VEC;  // 16-byte pieces per tile row
  // + bias (+ addend), then ReLU unless disabled; the L2 epilogue always
  // follows a ReLU.
  const bool relu = a.relu || C::L2;
  // A lane's four columns at byte `at` of a staged row.
  auto put4 = [&](unsigned char* at, float v0, float v1, float v2, float v3)
      __attribute__((always_inline)) {
    if constexpr (C::kBf16)
      *reinterpret_cast<uint2*>(at) = make_uint2(pack_bf16x2(v0, v1), pack_bf16x2(v2, v3));
    else
      *reinterpret_cast<float4*>(at) = make_float4(v0, v1, v2, v3);
  };
  auto add4 = [&](const unsigned char* at, float (&x)[4]) __attribute__((always_inline)) {
    if constexpr (C::kBf16) {
      const uint2 v = *reinterpret_cast<const uint2*>(at);
      x[0] += __uint_as_float(v.x << 16);
      x[1] += __uint_as_float(v.x & 0xFFFF0000u);
      x[2] += __uint_as_float(v.y << 16);
      x[3] += __uint_as_float(v.y & 0xFFFF0000u);
    } else {
      const float4 v = *reinterpret_cast<const float4*>(at);
      x[0] += v.x;
      x[1] += v.y;
      x[2] += v.z;
      x[3] += v.w;
    }
  };
  // acc[i] = its band + bias + addend (lane_row: the addend's row of this
  // lane, shifted to column 0 of the tile; null = none), ReLU. For the row norm also the
  // sums of squares into LDS: each block's columns of this lane, blocks in order, then the
  // partner half-wave's (lane ^ 32); a wave with less than a group leaves all apart.
  auto finish_band = [&](int i, const unsigned char* lane_row) __attribute__((always_inline)) {
    float sum[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      float s = 0.0f;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 bv = *reinterpret_cast<const float4*>(bias_s + c0(j, g));
        float x[4] = {acc[i][j][4 * g + 0] + bv.x, acc[i][j][4 * g + 1] + bv.y,
                      acc[i][j][4 * g + 2] + bv.z, acc[i][j][4 * g + 3] + bv.w};
        if (lane_row && n0 + c0(j, g) < a.N) add4(lane_row + c0(j, g) * ESZ, x);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float y = relu ? fmaxf(x[e], 0.0f) : x[e];
          acc[i][j][4 * g + e] = y;
          s = fmaf(y, y, s);
        }
      }
      sum[j] = s;
    }
    if constexpr (C::L2) {
      float* const row_sums = red + (a_base_row + i * 32 + row_in_blk) * NORM_SUMS;
      if constexpr (!C::NORM_WHOLE) {
#pragma unroll
        for (int j = 0; j < TN; ++j) row_sums[2 * (wn * TN + j) + half] = sum[j];
      } else {
#pragma unroll
        for (int j = 1; j < TN; ++j) sum[0] += sum[j];
        sum[0] += __shfl_xor(sum[0], 32);
        if (half == 0) row_sums[wn] = sum[0];
      }
    }
  };
  auto stage_band = [&](int i, unsigned char* lane_row, float scale)
      __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        put4(lane_row + c0(j, g) * ESZ, acc[i][j][4 * g] * scale, acc[i][j][4 * g + 1] * scale,
             acc[i][j][4 * g + 2] * scale, acc[i][j][4 * g + 3] * scale);
  };
  // `rows` staged rows -> global, BN / VEC lanes per row; row_of: their tile rows.
  auto flush_rows = [&](int rows, auto row_of) __attribute__((always_inline)) {
#pragma unroll 4
    for (int e = tid; e < rows * PER_ROW; e += THREADS) {
      const int b = e / PER_ROW, ck = e % PER_ROW;
      const int64_t r = m0 + row_of(b);
      const int c = n0 + VEC * ck;
      if (r < a.M && c < a.N)
        *reinterpret_cast<uint4*>(static_cast<unsigned char*>(a.C) + (r * a.N + c) * ESZ) =
            *reinterpret_cast<const uint4*>(smem + b * TROW + 16 * ck);
    }
  };
  // The addend's row of this lane for band i, in memory.
  auto addend_row = [&](int i) __attribute__((always_inline)) {
    const int64_t r = m0 + a_base_row + i * 32 + row_in_blk;
    return a.addend && r < a.M
               ? static_cast<const unsigned char*>(a.addend) + (r * a.N + n0) * ESZ
               : nullptr;
  };
  // Row norm: the groups' sums of the row in order, the same whatever the tile shape.
  auto row_scale = [&](int i) __attribute__((always_inline)) {
    const int r = a_base_row + i * 32 + row_in_blk;
    float ss = 0.0f;
#pragma unroll
    for (int w = 0; w < BN / 32 / C::NORM_GROUP; ++w) {
      if constexpr (!C::NORM_WHOLE) {
        const float* const g = red + r * NORM_SUMS + w * 2 * C::NORM_GROUP;
        float lo = g[0], hi = g[1];
#pragma unroll
        for (int j = 1; j < C::NORM_GROUP; ++j) {
          lo += g[2 * j];
          hi += g[2 * j + 1];
        }
        ss += lo + hi;
      } else {
        ss += red[r * NORM_SUMS + w];
      }
    }
    return ss > 0.0f ? 1.0f / sqrtf(ss) : 0.0f;
  };

  if constexpr (kStaged) {
#pragma unroll
    for (int i = 0; i < TM; ++i) finish_band(i, addend_row(i));
    if constexpr (C::L2) __syncthreads();
#pragma unroll
    for (int i = 0; i < TM; ++i)
      stage_band(i, smem + (a_base_row + i * 32 + row_in_blk) * TROW,
                 C::L2 ? row_scale(i) : 1.0f);
    __syncthreads();
    flush_rows(BM, [](int b) { return b; });
  } else {
    // One row band at a time. Band i is row band i of every wave: tile rows
    // WM wm' + 32 i + (0..31) for each wm'; band row b <-> tile row
    // WM (b / 32) + 32 i + b % 32. The addend of an L2 tile arrives the same
    // way, as whole row pieces.
    constexpr int BROWS = 32 * C::WAVES_M;
    static_assert(BROWS * TROW <= STAGES * C::STAGE_BYTES, "a band fits the ring");
    unsigned char* const lane_row = smem + (wm * 32 + row_in_blk) * TROW;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      auto band_row = [&](int b) __attribute__((always_inline)) {
        return (b >> 5) * C::WM + 32 * i + (b & 31);
      };
      if constexpr (C::L2) {
        if (a.addend) {
#pragma unroll 4
          for (int e = tid; e < BROWS * PER_ROW; e += THREADS) {
            const int b = e / PER_ROW, ck = e % PER_ROW;
            const int64_t r = m0 + band_row(b);
            const int c = n0 + VEC * ck;
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (r < a.M && c < a.N)
              v = *reinterpret_cast<const uint4*>(static_cast<const unsigned char*>(a.addend) +
                                                  (r * a.N + c) * ESZ);
            *reinterpret_cast<uint4*>(smem + b * TROW + 16 * ck) = v;
          }
          __syncthreads();
        }
        finish_band(i, a.addend ? lane_row : nullptr);
        __syncthreads();  // partial sums visible; every addend read of the band done
        stage_band(i, lane_row, row_scale(i));
      } else {
        finish_band(i, addend_row(i));
        stage_band(i, lane_row, 1.0f);
      }
      __syncthreads();
      flush_rows(BROWS, band_row);
      __syncthreads();  // the staged band is read before the next one lands
    }
  }
}

// ---------------------------------------------------------------------------
// bf16 GEMM with register-staged loads, for one A source without a row map
// and without the L2 epilogue (the Q transform and the neighbour half of W).
//
// A 256 x 256 tile per block of 4 waves (2 x 2, 128 x 128 each). K runs in
// chunks of 64 columns, i.e. 128 bytes per row: each load instruction of a
// wave reads 8 whole rows of a chunk (8 lanes x 16 B per row), so every
// request is a full 128-byte line. Chunks travel global -> VGPR -> LDS: two
// register buffers keep chunks c + 2 and c + 3 in flight while chunk c is
// multiplied from one LDS stage and chunk c + 1 waits in the other. In a row
// of a stage, 16-byte vector v sits in slot v ^ ((row >> 1) & 7): a 16-byte
// access is served 16 lanes at a time from 64 banks (two 128-byte rows), so
// the 16 lanes that write two rows, and the 16 rows read by a fragment
// instruction's lane group, fall on distinct banks. Missing rows and the K
// tail read zeros through the buffer descriptors' range checks.
// ---------------------------------------------------------------------------
template <int WAVES_M_, int WAVES_N_>
struct RsCfg {
  static constexpr int BM = 256, BN = 256, BK = 64;
  static constexpr int WAVES_M = WAVES_M_, WAVES_N = WAVES_N_, NW = WAVES_M * WAVES_N;
  static constexpr int THREADS = 64 * NW;
  static constexpr int ROWS = BM + BN;                 // rows of a stage (A rows, then B rows)
  static constexpr int ROW_BYTES = BK * 2;             // 128
  static constexpr int STAGE_BYTES = ROWS * ROW_BYTES; // 64 KB
  static constexpr int RSTEP = THREADS / 8;            // stage rows per block load instruction
  static constexpr int LOADS = ROWS / RSTEP;           // 16-byte vectors per thread per chunk
  static constexpr int SLICE = LOADS / 4;              // loads (and stores) per k-step
  static constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
  static constexpr int TM = WM / 32, TN = WN / 32;     // 32 x 32 blocks per wave
  static_assert(LOADS % 4 == 0 && TM * TN >= TM + TN + 2, "k-step interleave pattern");
};

template <typename C>
__global__ __launch_bounds__(C::THREADS) void gemm_rs_kernel(GemmLaunch a) {
  constexpr int BM = C::BM, BN = C::BN, BK = C::BK, THREADS = C::THREADS;
  constexpr int ROW_BYTES = C::ROW_BYTES, STAGE_BYTES = C::STAGE_BYTES, RSTEP = C::RSTEP;
  constexpr int LOADS = C::LOADS, SLICE = C::SLICE, TM = C::TM, TN = C::TN;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * STAGE_BYTES + BN * 4];
  float* bias_s = reinterpret_cast<float*>(smem + 2 * STAGE_BYTES);
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / C::WAVES_N, wn = wave % C::WAVES_N;

  // Tile coordinates are wave-uniform; readfirstlane keeps them (and the
  // buffer descriptors built from them) in scalar registers.
  const int tiles_n = (a.N + BN - 1) / BN;
  const int tile = __builtin_amdgcn_readfirstlane(xcd_tile(blockIdx.x, gridDim.x));
  const int tm = __builtin_amdgcn_readfirstlane(tile / tiles_n);
  const int n0 = __builtin_amdgcn_readfirstlane((tile - tm * tiles_n) * BN);
  const int64_t m0 = (int64_t)tm * BM;
  const int K = a.K0;
  for (int c = tid; c < BN; c += THREADS)
    bias_s[c] = (a.bias && n0 + c < a.N) ? a.bias[n0 + c] : 0.0f;

  // Load slot i of this thread: stage row (tid >> 3) + RSTEP i (A rows for
  // i < LOADS / 2, B rows after), 16-byte vector tid & 7 of the row's chunk.
  // Loads go
  // through buffer descriptors spanning the rows of this tile that exist, so
  // missing rows read zeros; the K tail takes an offset past every
  // descriptor's range (also zeros). No load is behind a branch.
  const int r0 = tid >> 3, v = tid & 7;
  const int64_t a_rows = a.M < a.rows_a0 ? a.M : a.rows_a0;  // rows of A that exist
  const int64_t a_have = a_rows - m0 < 0 ? 0 : (a_rows - m0 > BM ? BM : a_rows - m0);
  const int64_t b_have = a.N - n0 < 0 ? 0 : (a.N - n0 > BN ? BN : a.N - n0);
  const int a_bytes = __builtin_amdgcn_readfirstlane((int)(a_have * a.lda0 * 2));
  const int b_bytes = __builtin_amdgcn_readfirstlane((int)(b_have * a.ldb * 2));
  const __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<unsigned char*>(static_cast<const unsigned char*>(a.A0)) + m0 * a.lda0 * 2,
      (short)0, a_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t b_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<unsigned char*>(static_cast<const unsigned char*>(a.B)) + (int64_t)n0 * a.ldb * 2,
      (short)0, b_bytes, 0x00020000);
  const int a_off0 = r0 * (int)a.lda0 * 2 + v * 16, a_step = RSTEP * (int)a.lda0 * 2;
  const int b_off0 = r0 * (int)a.ldb * 2 + v * 16, b_step = RSTEP * (int)a.ldb * 2;
  const int nchunks = (K + BK - 1) / BK;

  u32x4 stage_regs[2][LOADS];
  auto load_chunk = [&](int chunk, u32x4 (&r)[LOADS]) __attribute__((always_inline)) {
    // Bit 31 set (arithmetically, not by a select) sends the K tail past the
    // descriptors' ranges.
    const int oob = (int)((uint32_t)(K - 1 - (chunk * BK + v * 8)) & 0x80000000u);
    const int koff = chunk * ROW_BYTES;
#pragma unroll
    for (int i = 0; i < LOADS / 2; ++i)
      r[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                           a_rsrc, (a_off0 + i * a_step + koff) | oob, 0, 0));
#pragma unroll
    for (int i = 0; i < LOADS / 2; ++i)
      r[LOADS / 2 + i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                       b_rsrc, (b_off0 + i * b_step + koff) | oob,
                                                       0, 0));
  };
  // Quarter q of a chunk: load slots SLICE q .. SLICE (q + 1) - 1 (A rows for q < 2).
  auto load_slice = [&](int chunk, u32x4 (&r)[LOADS], int q) __attribute__((always_inline)) {
    const int oob = (int)((uint32_t)(K - 1 - (chunk * BK + v * 8)) & 0x80000000u);
    const int koff = chunk * ROW_BYTES;
#pragma unroll
    for (int u = 0; u < SLICE; ++u) {
      const int i = SLICE * q + u;
      if (i < LOADS / 2)
        r[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                             a_rsrc, (a_off0 + i * a_step + koff) | oob, 0, 0));
      else
        r[i] = __builtin_bit_cast(
            u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                       b_rsrc, (b_off0 + (i - LOADS / 2) * b_step + koff) | oob, 0, 0));
    }
  };
  // ((r0 + RSTEP i) >> 1) & 7 == (r0 >> 1) & 7: one slot for all of this
  // thread's rows.
  const int wslot = (v ^ ((r0 >> 1) & 7)) * 16;
  auto store_chunk = [&](int stage, const u32x4 (&r)[LOADS]) __attribute__((always_inline)) {
    unsigned char* base = smem + stage * STAGE_BYTES + r0 * ROW_BYTES + wslot;
#pragma unroll
    for (int i = 0; i < LOADS; ++i)
      *reinterpret_cast<u32x4*>(base + i * RSTEP * ROW_BYTES) = r[i];
  };
  auto store_slice = [&](int stage, const u32x4 (&r)[LOADS], int q) __attribute__((always_inline)) {
    unsigned char* base = smem + stage * STAGE_BYTES + r0 * ROW_BYTES + wslot;
#pragma unroll
    for (int u = 0; u < SLICE; ++u)
      *reinterpret_cast<u32x4*>(base + (SLICE * q + u) * RSTEP * ROW_BYTES) = r[SLICE * q + u];
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  // Fragment reads: lane l takes row (l & 31) of a 32-row block and vector
  // 2 ks + (l >> 5) of k-step ks; rows of a block start at multiples of 8.
  const int frow = lane & 31, half = lane >> 5;
  const int fa = (wm * C::WM + frow) * ROW_BYTES;
  const int fb = (BM + wn * C::WN + frow) * ROW_BYTES;
  struct Frags {
    u32x4 a[TM], b[TN];
  };
  auto read_frags = [&](int stage, int ks, Frags& f) __attribute__((always_inline)) {
    const unsigned char* st = smem + stage * STAGE_BYTES;
    const int slot = ((2 * ks + half) ^ ((frow >> 1) & 7)) * 16;
#pragma unroll
    for (int i = 0; i < TM; ++i)
      f.a[i] = *reinterpret_cast<const u32x4*>(st + fa + i * 32 * ROW_BYTES + slot);
#pragma unroll
    for (int j = 0; j < TN; ++j)
      f.b[j] = *reinterpret_cast<const u32x4*>(st + fb + j * 32 * ROW_BYTES + slot);
  };
  auto mfma = [&](const Frags& f) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            __builtin_bit_cast(bf16x8, f.b[j]), __builtin_bit_cast(bf16x8, f.a[i]), acc[i][j],
            0, 0, 0);
  };

  // Prologue: chunk 0 into stage 0; chunks 1 and 2 in flight. (The compiler
  // places the vmcnt waits before each store from the loaded registers.)
  load_chunk(0, stage_regs[0]);
  load_chunk(1, stage_regs[1]);
  store_chunk(0, stage_regs[0]);
  load_chunk(2, stage_regs[0]);
  lds_barrier();

  // One chunk: chunk c + 1 (the oldest loads in flight) goes into the other
  // stage, whose last readers passed the barrier that ended the previous
  // step; its registers then take chunk c + 3; chunk c is multiplied. The
  // stage and register-buffer indices are compile-time (two steps per loop
  // trip), so the buffers stay in registers.
  auto step = [&](int c, auto CUR) __attribute__((always_inline)) {
    constexpr int cur = decltype(CUR)::value, nxt = cur ^ 1;
    Frags f[2];
    read_frags(cur, 0, f[0]);
    // Scheduling fences at the k-step boundaries keep each step's fragment
    // reads inside the previous step, so the MFMAs wait only on reads issued
    // a whole k-step earlier (left to itself the scheduler pulled the current
    // step's B reads in between its own MFMAs, exposing their latency).
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      // A quarter of chunk c + 1's LDS writes and of chunk c + 3's loads per
      // k-step, the next k-step's fragment reads, and the 16 MFMAs of this
      // k-step, interleaved one for one so that LDS and memory traffic run
      // under the matrix work.
      if (ks < 3) read_frags(cur, ks + 1, f[(ks + 1) & 1]);
      store_slice(nxt, stage_regs[nxt], ks);
      load_slice(c + 3, stage_regs[nxt], ks);
      mfma(f[ks & 1]);
      constexpr int NR = TM + TN;              // fragment reads of a k-step
      if (ks < 3) {
#pragma unroll
        for (int i = 0; i < NR; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // DS read
        }
      } else {
        __builtin_amdgcn_sched_group_barrier(0x008, NR, 0);
      }
      constexpr int REST = TM * TN - NR;       // MFMAs left for the writes and loads
      constexpr int PER = SLICE < REST / 2 ? 1 : (SLICE + REST / 2 - 1) / (REST / 2);
#pragma unroll
      for (int i = 0; i < SLICE; i += PER) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);    // MFMA
        __builtin_amdgcn_sched_group_barrier(0x200, PER, 0);  // DS write
      }
#pragma unroll
      for (int i = 0; i < SLICE; i += PER) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);    // MFMA
        __builtin_amdgcn_sched_group_barrier(0x020, PER, 0);  // VMEM read
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    lds_barrier();
  };
  // An odd chunk count runs one more chunk, read entirely out of range (all
  // zeros), so the loop body has no exit in the middle.
  for (int c = 0; c < nchunks; c += 2) {
    step(c, std::integral_constant<int, 0>{});
    step(c + 1, std::integral_constant<int, 1>{});
  }

  // ---- epilogue: bias (+ ReLU) into a bf16 C tile in LDS, then row stores ---
  // After the last chunk's barrier both stages are free; they hold the
  // 256 x 256 tile, row r at byte 512 r with its 16-byte slot s (8 columns)
  // at position s ^ (r & 31), so the lanes' 4-column pieces (16 rows per LDS
  // pass) and the row runs read back (16 slots of one row per pass) fall on
  // distinct banks. Each row then leaves as 32 x 16 B contiguous stores.
  // Lane l holds output row WM wm + 32 i + (l & 31) of the tile and, for group
  // g of block j, columns WN wn + 32 j + 8 g + 4 (l >> 5) + 0..3.
  static_assert(2 * STAGE_BYTES >= BM * BN * 2 && BN == 256, "C tile fits the two stages");
  constexpr int ROWB = BN * 2;  // bytes per C tile row
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int rt = wm * C::WM + i * 32 + frow;
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int cb = wn * C::WN + j * 32 + 8 * g + 4 * half;
        const float4 bv = *reinterpret_cast<const float4*>(bias_s + cb);
        float x0 = acc[i][j][4 * g] + bv.x, x1 = acc[i][j][4 * g + 1] + bv.y;
        float x2 = acc[i][j][4 * g + 2] + bv.z, x3 = acc[i][j][4 * g + 3] + bv.w;
        if (a.relu) {
          x0 = fmaxf(x0, 0.0f);
          x1 = fmaxf(x1, 0.0f);
          x2 = fmaxf(x2, 0.0f);
          x3 = fmaxf(x3, 0.0f);
        }
        const int slot = (cb >> 3) ^ (rt & 31);
        *reinterpret_cast<uint2*>(smem + rt * ROWB + slot * 16 + half * 8) =
            make_uint2(pack_bf16x2(x0, x1), pack_bf16x2(x2, x3));
      }
  }
  __syncthreads();
#pragma unroll 4
  for (int k = 0; k < BM * (BN / 8) / THREADS; ++k) {
    const int e = k * THREADS + tid;
    const int rt = e >> 5, sl = e & 31;
    const int64_t r = m0 + rt;
    const int c = n0 + sl * 8;
    if (r < a.M && c < a.N) {
      // Streaming stores: the output is not read again by this kernel, so it
      // should not push the reused B rows out of L2.
      const uint4 v = *reinterpret_cast<const uint4*>(smem + rt * ROWB + ((sl ^ (rt & 31)) * 16));
      typedef uint32_t u32x4s __attribute__((ext_vector_type(4)));
      __builtin_nontemporal_store(
          __builtin_bit_cast(u32x4s, v),
          reinterpret_cast<u32x4s*>(static_cast<uint16_t*>(a.C) + r * a.N + c));
    }
  }
}

// Bs: B [N][K] (row stride ldb) as bf16 triples in the order the fp32 kernel's
// MFMAs read them: [k-step of 16][32-row block][part][lane] x 16 bytes, lane l
// holding columns 8 (l / 32) .. + 7 of row l % 32 (rows past N are zero), then each
// 32-row block's least magnitude key. One workgroup per block of rows.
constexpr int kSplitWaves = 16;
__global__ __launch_bounds__(64 * kSplitWaves) void split_b_kernel(const float* __restrict__ B,
                                                                   int64_t ldb, int N, int K,
                                                                   u32x4* __restrict__ Bs) {
  __shared__ uint32_t least[kSplitWaves];
  const int nb32 = (N + 31) / 32, ksteps = K / 16;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = 32 * (int)blockIdx.x + (lane & 31);
  uint32_t key = ~0u;
  for (int ks = wave; ks < ksteps; ks += kSplitWaves) {
    u32x4 u = {0u, 0u, 0u, 0u}, v = u;
    if (row < N) {
      const u32x4* src =
          reinterpret_cast<const u32x4*>(B + row * ldb + 16 * ks + 8 * (lane >> 5));
      u = src[0];
      v = src[1];
    }
    const Split3 s = split3(u, v, key);
    const int64_t blk = (int64_t)ks * nb32 + blockIdx.x;
#pragma unroll
    for (int t = 0; t < 3; ++t) Bs[(blk * 3 + t) * 64 + lane] = s.p[t];
  }
  key = wave_min_key(key);
  if (lane == 0) least[wave] = key;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kSplitWaves; ++w) key = umin(key, least[w]);
    reinterpret_cast<uint32_t*>(Bs + (int64_t)ksteps * nb32 * 192)[blockIdx.x] = key;
  }
}

// The register-staged kernel covers bf16 launches with one A source, no row
// map, no addend and no L2 epilogue, and rows whose byte strides keep 16-byte
// vectors aligned.
bool use_rs(const GemmLaunch& a) {
  const int64_t ldb = a.ldb ? a.ldb : a.K0;
  // Buffer offsets are 32-bit: a tile's 256 rows must span < 2^31 bytes.
  // The epilogue writes rows in 8-column (16-byte) pieces: N % 8 == 0.
  return a.bf16 && !a.l2norm && a.K1 == 0 && !a.rowmap && !a.addend && a.K0 % 8 == 0 &&
         a.N % 8 == 0 && a.lda0 % 8 == 0 && ldb % 8 == 0 && a.lda0 <= (1 << 20) &&
         ldb <= (1 << 20) && reinterpret_cast<uintptr_t>(a.A0) % 16 == 0 &&
         reinterpret_cast<uintptr_t>(a.B) % 16 == 0 && reinterpret_cast<uintptr_t>(a.C) % 16 == 0;
}

#ifndef PINSAGE_RS_CFG
#define PINSAGE_RS_CFG RsCfg<2, 2>
#endif
hipError_t launch_rs(GemmLaunch a, hipStream_t s) {
  using C = PINSAGE_RS_CFG;
  if (!a.ldb) a.ldb = a.K0;
  const int64_t tiles = ((a.M + C::BM - 1) / C::BM) * (int64_t)((a.N + C::BN - 1) / C::BN);
  if (tiles <= 0) return hipSuccess;
  if (tiles > 0x7FFFFFFFll) return hipErrorInvalidValue;
  hipLaunchKernelGGL(gemm_rs_kernel<C>, dim3((unsigned)tiles), dim3(C::THREADS), 0, s, a);
  return hipGetLastError();
}

template <typename C>
hipError_t launch_cfg(const GemmLaunch& a, hipStream_t s) {
  const int64_t tiles = ((a.M + C::BM - 1) / C::BM) * (int64_t)((a.N + C::BN - 1) / C::BN);
  if (tiles <= 0) return hipSuccess;
  if (tiles > 0x7FFFFFFFll) return hipErrorInvalidValue;
  hipLaunchKernelGGL(gemm_kernel<C>, dim3((unsigned)tiles), dim3(C::THREADS), 0, s, a);
  return hipGetLastError();
}

#ifndef PINSAGE_CFG_Q_BF16
#define PINSAGE_CFG_Q_BF16 Cfg<true, 256, 256, 2, 2, false, 4, 1, false, true>
#endif
#ifndef PINSAGE_CFG_Q_F32
#define PINSAGE_CFG_Q_F32 Cfg<false, 128, 128, 2, 2, false, PRE ? 3 : 4, 2, PRE>
#endif
#ifndef PINSAGE_CFG_W256_BF16
#define PINSAGE_CFG_W256_BF16 Cfg<true, 128, 256, 2, 4, true, 3, 1, false, true>
#endif
#ifndef PINSAGE_CFG_W256_F32
#define PINSAGE_CFG_W256_F32 Cfg<false, PRE ? 128 : 64, 256, PRE ? 2 : 1, 4, true, 3, 2, PRE>
#endif
#ifndef PINSAGE_CFG_W512_BF16
#define PINSAGE_CFG_W512_BF16 Cfg<true, 128, 512, 2, 4, true, 3, 1, false, true>
#endif

// Tile shapes by dtype, epilogue, output width and how many tiles there are. Where
// the large tiles leave CUs idle, smaller ones are faster for as long as they all run
// at once (a second round costs as much as the first, and the large tiles take the
// same time up to one per CU). Measured, us, small / large:
//  - row norm, 32 rows against 128 (fp32 64): up to 8,192 rows, one tile per CU. 256
//    outputs, K = 768: bf16 14.8 / 20.0 at 8,192 rows, 20.8 / 20.2 at 10,000, 39.5 /
//    23.4 at 26,000; fp32 40.4 / 47.8, 63.8 / 49.2; 512 outputs, K = 1,024, bf16
//    25.6 / 40.5, 42.8 / 41.6. Up to 128 outputs, K = 384, twice the rows: bf16 10.6 /
//    11.7 at 16,384 rows, 12.9 / 12.0 at 20,000; fp32 24.6 / 28.5, 31.0 / 29.2.
//  - 64 x 64 against 128 x 128: bf16 K = 256, 256 outputs 10.3 / 10.6 at 200 tiles of
//    128 x 128, 12.9 / 12.7 at 314; K = 2,048, 512 outputs 16.3 / 25.0 at 96, 26.9 / 26.1
//    at 160, 33.6 / 26.8 at 204; fp32 K = 256, 256 outputs 18.2 / 21.6 at 128, 22.8 / 22.4
//    at 158, 27.5 / 23.4 at 200.
//  - bf16 128 x 128 against 256 x 256: K = 2,048, 512 outputs 40.8 / 51.2 at 100 tiles of
//    256 x 256, 46.4 / 51.5 at 128, 62.2 / 53.3 at 158; K = 512, 256 outputs 25.8 / 25.6
//    at 129, 25.9 / 27.2 at 176, 32.1 / 29.7 at 235; K = 256 20.1 / 20.8 at 176, 23.8 / 23.1
//    at 235; up to 128 outputs, which leave half of a large tile empty, 15.4 / 20.4 at 235.
inline int64_t few_norm_rows(const GemmLaunch& a) { return a.N > 128 ? 8192 : 16384; }
inline int64_t few_tiles(const GemmLaunch& a) { return !a.bf16 || a.K0 > 512 ? 128 : 256; }
inline int64_t mid_tiles(const GemmLaunch& a) {
  return a.N <= 128 ? 256 : (a.K0 > 512 ? 128 : 192);
}
inline int64_t tiles_of(const GemmLaunch& a, int bm, int bn) {
  return ((a.M + bm - 1) / bm) * (int64_t)((a.N + bn - 1) / bn);
}

// Row-norm tiles span every output column.
template <bool BF16>
hipError_t launch_small_norm(const GemmLaunch& a, hipStream_t s) {
  if (a.N <= 64) return launch_cfg<Cfg<BF16, 32, 64, 1, 2, true, 4>>(a, s);
  if (a.N <= 128) return launch_cfg<Cfg<BF16, 32, 128, 1, 4, true, 4>>(a, s);
  if (a.N <= 256) return launch_cfg<Cfg<BF16, 32, 256, 1, 8, true, 3, 1, false, BF16>>(a, s);
  return launch_cfg<Cfg<BF16, 32, 512, 1, 8, true, 3, 1, false, BF16>>(a, s);
}

template <bool PRE>
hipError_t launch_f32(const GemmLaunch& a, hipStream_t s) {
  if (!a.l2norm) {
    // 128 x 64 where it leaves no empty half tile.
    if (a.N <= 192 && (a.N + 63) / 64 % 2) return launch_cfg<Cfg<false, 128, 64, 4, 1, false, 4, 2, PRE>>(a, s);
    return launch_cfg<PINSAGE_CFG_Q_F32>(a, s);
  }
  if (a.N <= 64) return launch_cfg<Cfg<false, 128, 64, 4, 1, true, 4, 2, PRE>>(a, s);
  if (a.N <= 128) return launch_cfg<Cfg<false, 128, 128, 2, 2, true, PRE ? 3 : 4, 2, PRE>>(a, s);
  if (a.N <= 256) return launch_cfg<PINSAGE_CFG_W256_F32>(a, s);
  return launch_cfg<Cfg<false, 64, 512, 1, 8, true, PRE ? 2 : 3, 2, PRE>>(a, s);
}

hipError_t launch_bf16(const GemmLaunch& a, hipStream_t s) {
  // Q transform and the neighbour half of W share the tiles.
  if (!a.l2norm) return launch_cfg<PINSAGE_CFG_Q_BF16>(a, s);
  if (a.N <= 64) return launch_cfg<Cfg<true, 128, 64, 4, 1, true, 4>>(a, s);
  if (a.N <= 128) return launch_cfg<Cfg<true, 128, 128, 2, 2, true, 4>>(a, s);
  if (a.N <= 256) return launch_cfg<PINSAGE_CFG_W256_BF16>(a, s);
  return launch_cfg<PINSAGE_CFG_W512_BF16>(a, s);
}

// Few tiles of the large shapes; false when there are enough.
bool launch_few(const GemmLaunch& a, hipStream_t s, hipError_t* e) {
  if (a.l2norm) {
    if (a.M > few_norm_rows(a)) return false;
    *e = a.bf16 ? launch_small_norm<true>(a, s) : launch_small_norm<false>(a, s);
    return true;
  }
  // In bf16, with the K order of the large kernel (gemm_rs_kernel does not rotate).
  const bool rotate = a.bf16 && !use_rs(a);
  if (tiles_of(a, 128, 128) < few_tiles(a)) {
    if (!a.bf16) *e = launch_cfg<Cfg<false, 64, 64, 2, 2, false, 4>>(a, s);
    else if (rotate) *e = launch_cfg<Cfg<true, 64, 64, 2, 2, false, 4, 1, false, true>>(a, s);
    else *e = launch_cfg<Cfg<true, 64, 64, 2, 2, false, 4>>(a, s);
    return true;
  }
  if (a.bf16 && tiles_of(a, 256, 256) < mid_tiles(a)) {
    if (rotate) *e = launch_cfg<Cfg<true, 128, 128, 2, 2, false, 4, 1, false, true>>(a, s);
    else *e = launch_cfg<Cfg<true, 128, 128, 2, 2, false, 4>>(a, s);
    return true;
  }
  return false;
}

}  // namespace

size_t split_b_bytes(int N, int K) {
  const size_t blocks = (N + 31) / 32;
  return (size_t)(K / 16) * blocks * 3072 + blocks * 4;
}

hipError_t launch_gemm(const GemmLaunch& a, hipStream_t s) {
  if (a.M <= 0) return hipSuccess;
  ProfileScope prof(a.prof_class >= 0 ? a.prof_class : (a.l2norm ? kKGemmW : (a.relu ? kKGemmQ : kKGemmR)), s);
  if (a.l2norm && a.N > 512) return hipErrorInvalidValue;
  hipError_t few = hipSuccess;
  if (launch_few(a, s, &few)) return few;
  if (use_rs(a)) return launch_rs(a, s);
  if (a.bf16) return launch_bf16(a, s);
  if (!a.Bs) return launch_f32<false>(a, s);
  hipLaunchKernelGGL(split_b_kernel, dim3((unsigned)((a.N + 31) / 32)), dim3(64 * kSplitWaves), 0, s,
                     static_cast<const float*>(a.B), a.ldb ? a.ldb : (int64_t)a.K0 + a.K1, a.N,
                     a.K0 + a.K1, static_cast<u32x4*>(a.Bs));
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : launch_f32<true>(a, s);
}

}  // namespace pinsage
