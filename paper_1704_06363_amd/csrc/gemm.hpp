// gemm.hpp -- the MFMA tile engines shared by every dense contraction of the hot path: the
// register-staged engine described first (Cfg: the fp32 MoE products, the PCA fit's, the bf16
// assignment to 65 .. 128 centres and rows too wide for the pipelined engine), the direct-to-LDS ring
// (CfgD: assignments to up to 64 centres, projections to up to 64 components) and the pipelined engine
// (CfgP: the bf16 MoE products, the larger assignments and projections).
//
// C[m, n] = sum_k A(m, k) * B(n, k) over one BM x BN output tile per workgroup, split into
// (BM/WM) x (BN/WN) wavefronts of WM x WN.  Operands are staged through LDS in a row-major,
// K-contiguous layout whatever their layout in HBM:
//   K-contiguous operand (stored [rows][K]): 16-byte vector loads go straight to LDS;
//   K-strided operand    (stored [K][rows]): each thread loads a block of K-rows x 4 rows --
//                        8 x 4 for bf16, 4 x 4 for fp32 -- and transposes it in registers, so
//                        the LDS store is again one 16-byte vector (one chunk) per row.
// One stage covers 128 bytes of K per row (64 bf16 or 32 fp32), i.e. 8 chunks of 16 bytes.
// LDS rows are not padded; chunk c of row r lives at chunk c ^ ((r ^ (r >> 2)) & 7).  That
// XOR pattern was chosen by measuring the LDS bank-conflict counter on gfx950 for the three
// access patterns used here -- MFMA operand reads (16 consecutive rows, one chunk per 16
// lanes), direct stores (one row, 8 chunks per 8 lanes) and transposed stores (rows four
// apart) -- and is conflict-free for all of them (r ^ (r >> 3), for instance, is 2-way
// conflicted on the operand reads).
// bf16 uses v_mfma_f32_16x16x32_bf16 (8 consecutive k per lane); fp32 uses
// v_mfma_f32_16x16x4_f32 fed from the same 16-byte LDS reads (4 consecutive k per lane,
// consumed by 4 MFMAs).  Accumulation is fp32.  The K loop is double-buffered: the next
// stage's global loads are in flight while the current stage feeds the MFMAs.
//
// Accumulator ownership (verified layout of the 16x16 MFMA outputs): lane l of wave w holds,
// for sub-tile (i, j) and r = 0..3,
//   row = wm * WM + 16 i + 4 (l / 16) + r,     col = wn * WN + 16 j + (l % 16),
// with wm = w / (BN / WN), wn = w % (BN / WN).
#pragma once
#include "common.hpp"

namespace hmoe {

constexpr int kStageRowBytes = 128;  // K extent of one stage, in bytes

template <typename T, int BM_, int BN_, int WM_, int WN_>
struct Cfg {
  using type = T;
  static constexpr bool DMA = false, PIPE = false, SPLIT = false;  // register-staged engine
  static constexpr bool TRANS = false;  // accumulator element (i, j, r) at row 16 i + 4 (l / 16) + r, col 16 j + l % 16
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_;
  static constexpr int WAVES_N = BN / WN, WAVES_M = BM / WM;
  static constexpr int WAVES = WAVES_M * WAVES_N;
  static constexpr int THREADS = 64 * WAVES;
  static constexpr int MI = WM / 16, NJ = WN / 16;
  static constexpr int EPV = 16 / sizeof(T);             // elements per 16-byte vector
  static constexpr int BK = kStageRowBytes / sizeof(T);  // K per stage
  static constexpr int A_BYTES = BM * kStageRowBytes, B_BYTES = BN * kStageRowBytes;
  static constexpr int LDS = 2 * (A_BYTES + B_BYTES);
};

// fp32 GEMMs and narrow problems: 128 x 128 tiles, four waves of 64 x 64.
template <typename T>
using CfgSmall = Cfg<T, 128, 128, 64, 64>;
// Problems of few tiles: a quarter of the tile, four waves of 32 x 32 (two of 32 x 64 leave half of
// a CU's matrix cores idle).
template <typename T>
using CfgQuarter = Cfg<T, 64, 64, 32, 32>;
__device__ __forceinline__ int swz(int row, int chunk) {
  return row * kStageRowBytes + ((chunk ^ ((row ^ (row >> 2)) & 7)) << 4);
}

// ------------------------------------------------------------------ operand staging

// One ROWS-row operand tile of one K stage, held in registers between the global loads and
// the LDS store.  Rows >= rows_valid and K positions >= k_valid read as zero.
template <typename T, int ROWS, int THREADS, bool KCONTIG>
struct Stager {
  static constexpr int EPV = 16 / sizeof(T);
  static constexpr bool BF = sizeof(T) == 2;
  // K-contiguous: ROWS * 8 vectors of 16 bytes.
  // K-strided bf16: ROWS / 4 * 8 pieces of 8 K-rows x 4 rows, loaded as 8-byte rows.
  // K-strided fp32: ROWS / 4 * 8 blocks of 4 K-rows x 4 rows, loaded as 16-byte rows.
  static constexpr int PIECES = (ROWS / 4) * 8;
  static constexpr bool SPARE = PIECES < THREADS;  // the last threads have none
  static constexpr int NPIECE = KCONTIG ? 0 : (SPARE ? 1 : PIECES / THREADS);
  static constexpr int NV = KCONTIG ? ROWS * 8 / THREADS : (BF ? NPIECE * 4 : NPIECE * 4);
  static_assert(KCONTIG ? (ROWS * 8) % THREADS == 0 : SPARE || PIECES % THREADS == 0, "tile/threads");
  i32x4 v[NV];

  // K-contiguous: element (r, k) at base + r * ld + k (k_valid a multiple of EPV).
  // K-strided:    element (r, k) at base + k * ld + r (rows_valid a multiple of 4).
  __device__ __forceinline__ void load(const T* __restrict__ base, int64_t ld, int rows_valid, int k0,
                                       int k_valid) {
    const int t = threadIdx.x;
    if constexpr (KCONTIG) {
#pragma unroll
      for (int q = 0; q < NV; ++q) {
        const int vi = t + THREADS * q;
        const int r = vi >> 3;
        const int k = k0 + (vi & 7) * EPV;
        if (r < rows_valid && k < k_valid)
          v[q] = *reinterpret_cast<const i32x4*>(base + (int64_t)r * ld + k);
        else
          v[q] = i32x4{0, 0, 0, 0};
      }
    } else {
      constexpr int RQ = ROWS / 4;  // groups of 4 rows
#pragma unroll
      for (int q = 0; q < NPIECE; ++q) {
        const int pc = t + THREADS * q;
        if (SPARE && pc >= PIECES) continue;
        const int r = (pc % RQ) * 4;
        const int kb = pc / RQ;  // which 16-byte chunk of the stage
        if constexpr (BF) {
          // 8 K-rows x 4 bf16: two K-rows per i32x4 (low pair from even, high pair from odd)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int k = k0 + kb * 8 + 2 * i;
            uint2 e = make_uint2(0u, 0u), o = make_uint2(0u, 0u);
            if (r < rows_valid && k < k_valid) e = *reinterpret_cast<const uint2*>(base + (int64_t)k * ld + r);
            if (r < rows_valid && k + 1 < k_valid) o = *reinterpret_cast<const uint2*>(base + (int64_t)(k + 1) * ld + r);
            v[q * 4 + i] = i32x4{(int)e.x, (int)e.y, (int)o.x, (int)o.y};
          }
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int k = k0 + kb * 4 + i;
            if (r < rows_valid && k < k_valid)
              v[q * 4 + i] = *reinterpret_cast<const i32x4*>(base + (int64_t)k * ld + r);
            else
              v[q * 4 + i] = i32x4{0, 0, 0, 0};
          }
        }
      }
    }
  }

  __device__ __forceinline__ void store(lds<char>* dst) const {
    const int t = threadIdx.x;
    if constexpr (KCONTIG) {
#pragma unroll
      for (int q = 0; q < NV; ++q) {
        const int vi = t + THREADS * q;
        *reinterpret_cast<lds<i32x4>*>(dst + swz(vi >> 3, vi & 7)) = v[q];
      }
    } else {
      constexpr int RQ = ROWS / 4;
#pragma unroll
      for (int q = 0; q < NPIECE; ++q) {
        const int pc = t + THREADS * q;
        if (SPARE && pc >= PIECES) continue;
        const int r0 = (pc % RQ) * 4;
        const int kb = pc / RQ;
        if constexpr (BF) {
          // v[q*4+i] = (K-row 2i: rows r0..r0+3 as 2 words, K-row 2i+1: 2 words).
          // Output row j = 8 consecutive K values: word p = (K-row 2p, K-row 2p+1) of row j.
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int word = j >> 1;
            const uint32_t sel = (j & 1) ? 0x07060302u : 0x05040100u;
            uint32_t o[4];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
              const uint32_t a = (uint32_t)v[q * 4 + p][word];      // K-row 2p
              const uint32_t c = (uint32_t)v[q * 4 + p][2 + word];  // K-row 2p+1
              o[p] = __builtin_amdgcn_perm(c, a, sel);
            }
            *reinterpret_cast<lds<i32x4>*>(dst + swz(r0 + j, kb)) = i32x4{(int)o[0], (int)o[1], (int)o[2], (int)o[3]};
          }
        } else {
          const i32x4 s0 = v[q * 4 + 0], s1 = v[q * 4 + 1], s2 = v[q * 4 + 2], s3 = v[q * 4 + 3];
          *reinterpret_cast<lds<i32x4>*>(dst + swz(r0 + 0, kb)) = i32x4{s0[0], s1[0], s2[0], s3[0]};
          *reinterpret_cast<lds<i32x4>*>(dst + swz(r0 + 1, kb)) = i32x4{s0[1], s1[1], s2[1], s3[1]};
          *reinterpret_cast<lds<i32x4>*>(dst + swz(r0 + 2, kb)) = i32x4{s0[2], s1[2], s2[2], s3[2]};
          *reinterpret_cast<lds<i32x4>*>(dst + swz(r0 + 3, kb)) = i32x4{s0[3], s1[3], s2[3], s3[3]};
        }
      }
    }
  }

  // Squared norms of the K-contiguous rows this thread staged: xs[q] gets row
  // (threadIdx.x + THREADS * q) >> 3; the 8 lanes sharing a row together hold its full norm.
  __device__ __forceinline__ void add_sq(float* xs) const {
    static_assert(KCONTIG, "row norms need a K-contiguous operand");
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      const T* e = reinterpret_cast<const T*>(&v[q]);
#pragma unroll
      for (int z = 0; z < EPV; ++z) {
        const float f = to_f32(e[z]);
        xs[q] += f * f;
      }
    }
  }
};

// ------------------------------------------------------------------ MFMA stage

template <class C>
__device__ __forceinline__ void mfma_stage(const lds<char>* ldsA, const lds<char>* ldsB,
                                           floatx4 (&acc)[C::MI][C::NJ]) {
  const int l = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  const int wm = w / C::WAVES_N, wn = w % C::WAVES_N;
  const int lr = l & 15, lg = l >> 4;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int chunk = 4 * s + lg;
    i32x4 a[C::MI], b[C::NJ];
#pragma unroll
    for (int i = 0; i < C::MI; ++i)
      a[i] = *reinterpret_cast<const lds<i32x4>*>(ldsA + swz(wm * C::WM + 16 * i + lr, chunk));
#pragma unroll
    for (int j = 0; j < C::NJ; ++j)
      b[j] = *reinterpret_cast<const lds<i32x4>*>(ldsB + swz(wn * C::WN + 16 * j + lr, chunk));
#pragma unroll
    for (int i = 0; i < C::MI; ++i) {
#pragma unroll
      for (int j = 0; j < C::NJ; ++j) {
        if constexpr (sizeof(typename C::type) == 2) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              __builtin_bit_cast(bf16x8, a[i]), __builtin_bit_cast(bf16x8, b[j]), acc[i][j], 0, 0, 0);
        } else {
          const floatx4 af = __builtin_bit_cast(floatx4, a[i]);
          const floatx4 bf = __builtin_bit_cast(floatx4, b[j]);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[e], bf[e], acc[i][j], 0, 0, 0);
        }
      }
    }
  }
}

// Full K loop for one tile.  A rows [0, a_rows), B rows [0, b_rows), K positions [0, k_len).
// With ROWNORM (K-contiguous A only) xs[] collects squared row norms of A (see add_sq).
template <class C, bool A_KC, bool B_KC, bool ROWNORM = false>
__device__ __forceinline__ void gemm_tile_reg(const typename C::type* __restrict__ A, int64_t lda, int a_rows,
                                          const typename C::type* __restrict__ B, int64_t ldb, int b_rows,
                                          int k_len, lds<char>* smem, floatx4 (&acc)[C::MI][C::NJ],
                                          float* xs = nullptr) {
  using T = typename C::type;
  using SA = Stager<T, C::BM, C::THREADS, A_KC>;
  static_assert(!C::DMA, "register-staged engine");
  using SB = Stager<T, C::BN, C::THREADS, B_KC>;
#pragma unroll
  for (int i = 0; i < C::MI; ++i)
#pragma unroll
    for (int j = 0; j < C::NJ; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  if constexpr (ROWNORM) {
#pragma unroll
    for (int q = 0; q < SA::NV; ++q) xs[q] = 0.f;
  }
  const int nk = (int)cdiv(k_len, C::BK);
  if (nk == 0) return;
  if constexpr (C::BM * C::BN <= 64 * 64) {
    // small tiles: a stage's MFMAs take less than the trip to memory, so loads run two stages ahead
    static_assert(!ROWNORM, "row norms: larger tiles");
    SA sa[2];
    SB sb[2];
    const auto load = [&](int s, int p) {
      sa[p].load(A, lda, a_rows, s * C::BK, k_len);
      sb[p].load(B, ldb, b_rows, s * C::BK, k_len);
    };
    const auto store = [&](int p) {
      sa[p].store(smem + p * C::A_BYTES);
      sb[p].store(smem + 2 * C::A_BYTES + p * C::B_BYTES);
    };
    load(0, 0);
    if (nk > 1) load(1, 1);
    store(0);
    __syncthreads();
    for (int kt = 0; kt < nk; kt += 2) {
#pragma unroll
      for (int p = 0; p < 2; ++p) {  // stage kt + p in buffer p; registers p are free, 1 - p hold the next
        if (kt + p >= nk) break;
        if (kt + p + 2 < nk) load(kt + p + 2, p);
        mfma_stage<C>(smem + p * C::A_BYTES, smem + 2 * C::A_BYTES + p * C::B_BYTES, acc);
        if (kt + p + 1 < nk) store(1 - p);
        __syncthreads();
      }
    }
    return;
  }
  SA sa;
  SB sb;
  lds<char>* const bufA0 = smem;
  lds<char>* const bufB0 = smem + 2 * C::A_BYTES;
  sa.load(A, lda, a_rows, 0, k_len);
  sb.load(B, ldb, b_rows, 0, k_len);
  if constexpr (ROWNORM) sa.add_sq(xs);
  sa.store(bufA0);
  sb.store(bufB0);
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const int cur = kt & 1;
    const bool more = kt + 1 < nk;
    if (more) {
      sa.load(A, lda, a_rows, (kt + 1) * C::BK, k_len);
      sb.load(B, ldb, b_rows, (kt + 1) * C::BK, k_len);
    }
    mfma_stage<C>(bufA0 + cur * C::A_BYTES, bufB0 + cur * C::B_BYTES, acc);
    if (more) {
      if constexpr (ROWNORM) sa.add_sq(xs);
      sa.store(bufA0 + (cur ^ 1) * C::A_BYTES);
      sb.store(bufB0 + (cur ^ 1) * C::B_BYTES);
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ direct-to-LDS ring
//
// NT products with few columns (the gater's assignment to up to 64 centres, the PCA's projection to up
// to 64 components).  Operands travel from HBM to LDS without passing through registers:
// global_load_lds_dwordx4 writes lane l's 16 bytes to LDS at (wave-uniform base) + 16 l, so the LDS
// layout -- including its bank swizzle -- is chosen by the global address each lane loads.  A stage
// covers 32 K (64 bytes per row); NS stages form a ring and the loads for stage kt + NS - 1 are
// issued while stage kt feeds the MFMAs, each wave waiting
// (vmcnt) only for its own loads of the stage it is about to read.  LDS holds [rows][32 K] (64-byte
// rows, chunk c of row r at c ^ ((r >> 1) & 3)); MFMA operands come from one ds_read_b128 per 16 x 32
// fragment, conflict-free (checked with the LDS bank-conflict counter).  Rows past the valid range
// load a clamped (valid) address -- they only feed output rows / columns that are never stored -- and
// a last partial K stage is staged through registers with zero fill.  Needs every row width (ld) to be
// a multiple of 8 elements.

// fp32 operands (F32) take the same path: the engine stages 16-bit units (a float is two, every ld and K doubled), so a 64-byte row still
// holds one stage, and each 16-byte fragment -- four consecutive K of one row -- feeds four
// v_mfma_f32_16x16x4_f32, the lane group g supplying K = 4 g + q to the q-th of them.
template <typename T, int BM_, int BN_, int WM_, int WN_, int NS_>
struct CfgD {
  using type = T;
  static constexpr bool F32 = sizeof(T) == 4;
  static constexpr bool DMA = true, PIPE = false, SPLIT = false;
  static constexpr bool TRANS = true;  // accumulator element (i, j, r) at row 16 i + l % 16, col 16 j + 4 (l / 16) + r
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_;
  static constexpr int WAVES_N = BN / WN, WAVES_M = BM / WM;
  static constexpr int WAVES = WAVES_M * WAVES_N;
  static constexpr int THREADS = 64 * WAVES;
  static constexpr int MI = WM / 16, NJ = WN / 16;
  static constexpr int BK = 32, NS = NS_;  // BK in 16-bit units (64-byte rows)
  static constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2;
  static constexpr int STAGE = A_BYTES + B_BYTES;
  static constexpr int LDS = NS * STAGE;
  static_assert(sizeof(T) == 2 || sizeof(T) == 4, "bf16 or fp32 operands");
};

// At most 64 columns: 128 x 64 tiles of four waves
// and a 3-stage ring (36 KB), four workgroups per CU -- on fp32 rows against 256 x 64 (4 stages:
// 11% slower; 3 stages: 15%), 128 x 64 with 2 or 4 stages (10%, 8%) and 64 x 64 (17%)
typedef CfgD<float, 128, 64, 32, 64, 3> CfgDmaF32Narrow;
typedef CfgD<bf16, 128, 64, 32, 64, 3> CfgDmaNarrow;
// The same with fewer such tiles than CUs, where a tile's chain of stages is all there is: half the
// rows, so twice the workgroups, and four stages in flight instead of two (512 x 2048 bf16, K = 16:
// 30 us, 25)
typedef CfgD<float, 64, 64, 32, 32, 5> CfgDmaF32NarrowFew;
typedef CfgD<bf16, 64, 64, 32, 32, 5> CfgDmaNarrowFew;

// 16-byte chunk swizzle of the 64-byte K-contiguous rows (used by the DMA slot mapping and the
// operand reads alike).  Measured with the LDS bank-conflict counter on gfx950 for the MFMA
// operand read (16 rows x 4 chunks per ds_read_b128): (r >> 1) & 3 is conflict-free, while no
// swizzle, r & 3, (r >> 2) & 3, (r ^ (r >> 2)) & 3 and (r >> 3) & 3 are all 2-way conflicted.
__device__ __forceinline__ int kc_swz(int row) { return (row >> 1) & 3; }
__device__ __forceinline__ int kc_off(int row, int chunk) { return row * 64 + ((chunk ^ kc_swz(row)) << 4); }
// K-strided operands (pipelined engine): LDS [K][R rows] as in HBM (rows contiguous, 16-byte chunk c of
// K-row k at c ^ 2 ((k & 3) | ((k >> 1) & 4))); MFMA operands come from two ds_read_b64_tr_b16 per
// fragment, conflict-free.  Within each 16-lane group that read returns to lane i, slot s, element i % 4
// of the 8 bytes addressed by lane 4 s + i / 4 (verified on gfx950), so lane j addressing K-row
// 8 (l / 16) + 4 h + j / 4, rows 4 (j % 4) .. + 3 gives every lane the 4 consecutive K of its own row
// that the MFMA layout expects.
template <int R>
__device__ __forceinline__ int ks_off(int k, int byte) {
  const int sw = ((k & 3) | ((k >> 1) & 4)) << 1;
  return k * (R * 2) + ((((byte >> 4) ^ sw)) << 4) + (byte & 15);
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wg_barrier() { asm volatile("s_barrier" ::: "memory"); }
__device__ __forceinline__ void wg_barrier_lds() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// One operand of R rows: per-thread slot offsets and the per-stage DMA / tail staging.
template <int R, int THREADS>
struct DmaOperand {
  static constexpr int SLOTS = R * 4;  // 16-byte slots per stage
  static constexpr int NQ = SLOTS / THREADS;
  static_assert(SLOTS % THREADS == 0, "slots/threads");
  int64_t off[NQ];  // element offset of the slot's source for k0 = 0
  int kk[NQ];       // K offset of the chunk (0..31)

  // element (r, k) at base + r * ld + k
  __device__ __forceinline__ void init(int64_t ld, int rows_valid) {
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int slot = (q * (THREADS / 64) + w) * 64 + l;
      const int r = slot >> 2, p = slot & 3;
      const int c = p ^ kc_swz(r);
      const int gr = r < rows_valid ? r : rows_valid - 1;
      off[q] = (int64_t)gr * ld + c * 8;
      kk[q] = c * 8;
    }
  }

  __device__ __forceinline__ void issue(const bf16* __restrict__ base, int k0, lds<char>* buf) const {
    const int w = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      lds<char>* dst = buf + (q * (THREADS / 64) + w) * 1024;
      __builtin_amdgcn_global_load_lds((const void*)(base + off[q] + k0), (lds<void>*)dst, 16, 0, 0);
    }
  }

  // Last partial stage [k0, k_len): through registers, zero outside the valid range.
  __device__ __forceinline__ void tail(const bf16* __restrict__ base, int k0, int k_len, lds<char>* buf) const {
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int slot = (q * (THREADS / 64) + w) * 64 + l;
      i32x4 v = i32x4{0, 0, 0, 0};
      if (k0 + kk[q] < k_len) v = *reinterpret_cast<const i32x4*>(base + off[q] + k0);
      *reinterpret_cast<lds<i32x4>*>(buf + slot * 16) = v;
    }
  }
};

// A stage's MFMA operands for this wave: fragments of its WM rows of A and WN rows of B.
template <class C>
__device__ __forceinline__ void dma_read_frags(const lds<char>* bA, const lds<char>* bB, bf16x8 (&a)[C::MI],
                                               bf16x8 (&b)[C::NJ]) {
  const int l = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  const int wm = w / C::WAVES_N, wn = w % C::WAVES_N;
  const int lr = l & 15, lg = l >> 4;
#pragma unroll
  for (int i = 0; i < C::MI; ++i)
    a[i] = *reinterpret_cast<const lds<bf16x8>*>(bA + kc_off(wm * C::WM + 16 * i + lr, lg));
#pragma unroll
  for (int j = 0; j < C::NJ; ++j)
    b[j] = *reinterpret_cast<const lds<bf16x8>*>(bB + kc_off(wn * C::WN + 16 * j + lr, lg));
}

// The stage's MFMAs.  B is the MFMA's first operand: the 16 x 16 result is the transposed
// sub-tile, so each lane ends up with four consecutive output columns of one row (see TRANS).
// ROWNORM: xs[i / WAVES_N] += squares of this lane's 8 elements of A fragment i, for the fragments
// i = wn (mod WAVES_N) that this wave is responsible for (the work is spread over the waves
// that share the rows; each row's sum stays within one wave), as four packed bf16 dot products
// (the squares of bf16 values are exact in fp32).
template <class C, bool ROWNORM>
__device__ __forceinline__ void dma_mfmas(const bf16x8 (&a)[C::MI], const bf16x8 (&b)[C::NJ],
                                          floatx4 (&acc)[C::MI][C::NJ], float* xs) {
  if constexpr (C::F32) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < C::MI; ++i)
#pragma unroll
        for (int j = 0; j < C::NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(floatx4, b[j])[q],
                                                           __builtin_bit_cast(floatx4, a[i])[q], acc[i][j], 0, 0, 0);
    if constexpr (ROWNORM) {
      const int wn = (threadIdx.x >> 6) % C::WAVES_N;
#pragma unroll
      for (int i = 0; i < C::MI; ++i)
        if ((i % C::WAVES_N) == wn) {
          const floatx4 v = __builtin_bit_cast(floatx4, a[i]);
#pragma unroll
          for (int e = 0; e < 4; ++e) xs[i / C::WAVES_N] = fmaf(v[e], v[e], xs[i / C::WAVES_N]);
        }
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < C::MI; ++i)
#pragma unroll
    for (int j = 0; j < C::NJ; ++j)
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
  if constexpr (ROWNORM) {
    const int wn = (threadIdx.x >> 6) % C::WAVES_N;
#pragma unroll
    for (int i = 0; i < C::MI; ++i)
      if ((i % C::WAVES_N) == wn) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bf16x2 v = {a[i][2 * e], a[i][2 * e + 1]};
          xs[i / C::WAVES_N] = __builtin_amdgcn_fdot2_f32_bf16(v, v, xs[i / C::WAVES_N], false);
        }
      }
  }
}

// Waits for this wave's loads of the stage that has `pending_stages` later stages in flight
// behind it (vmcnt counts in issue order).
template <class C, int LOADS>
__device__ __forceinline__ void wait_stage(int pending_stages) {
  static_assert(C::NS <= 5 && LOADS * (C::NS - 2) <= 63, "vmcnt range");
  switch (pending_stages) {
    case 0: wait_vmcnt<0>(); break;
    case 1: wait_vmcnt<LOADS>(); break;
    case 2: wait_vmcnt<2 * LOADS>(); break;
    default: wait_vmcnt<3 * LOADS>(); break;
  }
}

// The K loop of one tile: prime() issues stages 0 .. NS-2 into the LDS ring, run() is the main loop
// and a partial last stage; it ends with a barrier after which the ring is free again.
template <class C>
struct DmaTile {
  using OA = DmaOperand<C::BM, C::THREADS>;
  using OB = DmaOperand<C::BN, C::THREADS>;
  static constexpr int LOADS = OA::NQ + OB::NQ;
  OA oa;
  OB ob;
  const bf16* A;
  const bf16* B;
  int k_len;

  __device__ __forceinline__ static lds<char>* bufA(lds<char>* smem, int s) { return smem + s * C::STAGE; }
  __device__ __forceinline__ static lds<char>* bufB(lds<char>* smem, int s) {
    return smem + s * C::STAGE + C::A_BYTES;
  }

  __device__ __forceinline__ void prime(const bf16* __restrict__ A_, int64_t lda, int a_rows,
                                        const bf16* __restrict__ B_, int64_t ldb, int b_rows, int k_len_,
                                        lds<char>* smem) {
    A = A_;
    B = B_;
    k_len = k_len_;
    oa.init(lda, a_rows);
    ob.init(ldb, b_rows);
    const int nfull = k_len / C::BK;
#pragma unroll
    for (int s = 0; s < C::NS - 1; ++s)
      if (s < nfull) {
        oa.issue(A, s * C::BK, bufA(smem, s));
        ob.issue(B, s * C::BK, bufB(smem, s));
      }
  }

  template <bool ROWNORM = false>
  __device__ __forceinline__ void run(lds<char>* smem, floatx4 (&acc)[C::MI][C::NJ], float* xs = nullptr) {
    if constexpr (ROWNORM) {
#pragma unroll
      for (int i = 0; i < (C::MI + C::WAVES_N - 1) / C::WAVES_N; ++i) xs[i] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < C::MI; ++i)
#pragma unroll
      for (int j = 0; j < C::NJ; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int nfull = k_len / C::BK;
    auto wait_own = [&](int k) {  // this wave's loads of stage k
      const int ahead = nfull - 1 - k;
      wait_stage<C, LOADS>(ahead < C::NS - 2 ? ahead : C::NS - 2);
    };
    // Two wave groups (waves 0 .. WAVES/2-1 and the rest) run the same stage sequence  [barrier]
    // read fragments + issue loads [barrier] MFMAs  with group 1 one phase behind group 0, so that
    // while one group reads, the other feeds the matrix units.  The offset comes from one extra
    // barrier, taken by group 1 before the loop and by group 0 after it (the group index is
    // wave-uniform, so those are scalar branches and both groups execute the same number of
    // barriers).  Stage kt is read first by group 0, after barrier 2 kt + 1, which for group 1 is the
    // second barrier of its stage kt - 1 (or the extra one): each wave waits for its own loads of
    // stage kt before that barrier; the count of its younger loads is the same in both places.  The
    // slot of stage kt - 1 gets new loads only after barrier 2 kt + 1, when both groups'
    // reads of it have completed (lgkmcnt(0) before every second barrier).
    static_assert(C::WAVES % 2 == 0, "two wave groups");
    const bool g1 = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) >= C::WAVES / 2;
    if (nfull > 0 && g1) {
      wait_own(0);
      wg_barrier();
    }
    for (int kt = 0; kt < nfull; ++kt) {
      if (!g1) wait_own(kt);
      wg_barrier();
      __builtin_amdgcn_sched_barrier(0);
      bf16x8 fa[C::MI], fb[C::NJ];
      const int sc = kt % C::NS;
      dma_read_frags<C>(bufA(smem, sc), bufB(smem, sc), fa, fb);
      const int nx = kt + C::NS - 1;
      if (nx < nfull) {
        oa.issue(A, nx * C::BK, bufA(smem, nx % C::NS));
        ob.issue(B, nx * C::BK, bufB(smem, nx % C::NS));
      }
      if (g1 && kt + 1 < nfull) wait_own(kt + 1);
      wg_barrier_lds();
      __builtin_amdgcn_sched_barrier(0);
      dma_mfmas<C, ROWNORM>(fa, fb, acc, xs);
    }
    if (nfull > 0 && !g1) wg_barrier();
    if (nfull * C::BK < k_len) {
      const int sb = nfull % C::NS;
      oa.tail(A, nfull * C::BK, k_len, bufA(smem, sb));
      ob.tail(B, nfull * C::BK, k_len, bufB(smem, sb));
      wg_barrier_lds();
      bf16x8 fa[C::MI], fb[C::NJ];
      dma_read_frags<C>(bufA(smem, sb), bufB(smem, sb), fa, fb);
      __builtin_amdgcn_sched_barrier(0);  // all of the fragment reads go out before the MFMAs
      dma_mfmas<C, ROWNORM>(fa, fb, acc, xs);
    }
    wg_barrier_lds();
  }
};

// ------------------------------------------------------------------ pipelined engine
//
// 256 x 256 tiles of eight waves (128 x 64 each) on a direct-to-LDS pipeline of 64-element
// stages: 128-byte rows, so that every load instruction reads whole 128-byte lines.  (A ring of
// 32-element stages, the same tile and waves, fetched every line twice, half at a time: on NT
// products of 8192^3 / 65536 x 4096 x 2048 / 2^20 x 1024 x 2048 it ran at 1134 / 1075 / 1125
// TFLOP/s against 1513 / 1339 / 1345 here; with a K-strided B, 65536 x 1024 x 50000, 1225
// against 1454; with both K-strided 1174 against 1415.)
//
// A stage holds four half panels, each in a slot of its own, two stages in LDS (128 KB): half h
// of A has rows 64 h .. 64 h + 63 of every 128-row wave strip, half h of B columns 32 h .. + 31
// of every 64-column wave strip (SPLIT: the halves are contiguous, which keeps the lines of a
// K-strided B whole; a wave then owns 32 columns of each half).  A wave computes its tile in
// two phases per stage, 32 MFMAs and 12 fragment reads each:
//   phase 0   reads A0(s), B1(s):     A0 B0, A0 B1        (B0(s) was read one phase earlier)
//   phase 1   reads A1(s), B0(s + 1): A1 B0, A1 B1
// The two wave groups (waves 0-3 and 4-7, one of each per SIMD) run one half phase apart, so
// that one reads while the other feeds the matrix cores: every phase is [reads, loads, barrier,
// MFMAs, barrier], and the offset is one extra barrier, taken by group 1 before the loop and by
// group 0 after it.  Phase q issues the loads of the slots that phase q - 1 has read, three
// phases before they are needed:
//   phase 0 of s:  A1(s + 1), B0(s + 2)        phase 1 of s:  A0(s + 2), B1(s + 2)
// Slot order: group 0's phase q lies between barriers 2q and 2q + 2 and group 1's between 2q + 1
// and 2q + 3, each with its reads done (lgkmcnt) before its middle barrier, so every read of
// phase q - 1 precedes barrier 2q and the loads that overwrite it follow.  Arrival: each wave
// waits for its own loads of phase q before its middle barrier of phase q - 1, and the barrier
// that starts group 0's phase q is no earlier than that; vmcnt counts in issue order, and the
// events behind the one waited for are those of the last two phases.
// Waves at raised priority around the MFMAs measured 1-3% slower.
//
// Offsets from a tile's base are 32-bit (one VGPR per load, the base in SGPRs): row widths must
// be below kPipeMaxLd elements; wider rows take the register-staged engine.
// fp32 operands (F32) run as 16-bit units, as on the ring engine.
constexpr int64_t kPipeMaxLd = int64_t(1) << 23;  // 255 rows x 2 bytes x ld < 2^32

template <typename T, int BM_, int BN_, int WM_, int WN_, bool SPLIT_>
struct CfgP {
  using type = T;
  static constexpr bool F32 = sizeof(T) == 4;
  static constexpr bool DMA = true, PIPE = true;
  static constexpr bool TRANS = true;  // accumulator element (i, j, r) at row 16 i + l % 16, col 16 j + 4 (l / 16) + r
  static constexpr bool SPLIT = SPLIT_;
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_;
  static constexpr int WAVES_N = BN / WN, WAVES_M = BM / WM;
  static constexpr int WAVES = WAVES_M * WAVES_N;
  static constexpr int THREADS = 64 * WAVES;
  static constexpr int MI = WM / 16, NJ = WN / 16;
  static constexpr int BK = 64;  // in 16-bit units (128-byte rows)
  static constexpr int A_HALF = BM / 2 * BK * 2, B_HALF = BN / 2 * BK * 2;
  static constexpr int STAGE = 2 * (A_HALF + B_HALF);
  static constexpr int LDS = 2 * STAGE;
  static_assert(sizeof(T) == 2 || sizeof(T) == 4, "bf16 or fp32 operands");
  static_assert(WM % 64 == 0 && WN % 64 == 0, "half strips of whole swizzle periods");
};
typedef CfgP<bf16, 256, 256, 128, 64, false> CfgPipe;    // B K-contiguous
typedef CfgP<bf16, 256, 256, 128, 64, true> CfgPipeKS;   // B K-strided
typedef CfgP<float, 256, 256, 128, 64, false> CfgPipeF32;  // fp32, K-contiguous operands
// The last row tile of a group with at most 128 rows (the short buckets of skewed routing) runs
// at half height, with half the MFMA work of the padded 256-row tile.
typedef CfgP<bf16, 128, 256, 64, 64, false> CfgPipeShort;
typedef CfgP<bf16, 128, 256, 64, 64, true> CfgPipeShortKS;
template <class C>
struct ShortTile {
  using type = void;
};
template <>
struct ShortTile<CfgPipe> {
  using type = CfgPipeShort;
};
template <>
struct ShortTile<CfgPipeKS> {
  using type = CfgPipeShortKS;
};

// threadIdx.x, computed with anew at each use: a persistent kernel's per-lane address terms are
// otherwise hoisted out of its tile loop, where they crowd the K loop's registers into scratch.
__device__ __forceinline__ int thread_id() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// A wave-uniform pointer as scalar registers (whatever the compiler keeps its inputs in).
__device__ __forceinline__ const char* uniform(const char* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<const char*>(((uint64_t)hi << 32) | lo);
}

static __device__ const i32x4 kZeros = {0, 0, 0, 0};

// Half panels of an operand of R tile rows, W per wave strip.
//   K-contiguous: slot [R / 2 rows][64 K], 16-byte chunk c of slot row r at c ^ ((r ^ (r >> 2)) & 7).
//   K-strided:    slot [64 K][R / 2 rows], chunk swizzle of ks_off<R / 2>.
template <int R, int W, int THREADS, bool KC, bool SPLIT>
struct HalfPanels {
  static constexpr int HR = R / 2;
  static constexpr int NQ = HR * 128 / (THREADS * 16);  // loads per wave and half
  static_assert(NQ * THREADS * 16 == HR * 128, "whole loads");
  uint32_t off[2][NQ];  // byte offset of this lane's 16 bytes from the stage's base

  // tile row of row q of half h
  __device__ __forceinline__ static int tile_row(int h, int q) {
    if constexpr (SPLIT) return h * HR + q;
    constexpr int G = W / 2;
    return (q / G) * W + h * G + q % G;
  }
  // K position (within the stage) of 16-byte slot piece `piece`
  __device__ __forceinline__ static int k_of(int piece) {
    if constexpr (KC) {
      const int r = piece >> 3;
      return ((piece & 7) ^ ((r ^ (r >> 2)) & 7)) * 8;
    } else {
      return piece / (HR / 8);
    }
  }
  // byte offset of piece `piece` of half h; rows past the valid range take a valid row's bytes (they
  // only feed outputs that are not stored)
  __device__ __forceinline__ static uint32_t source(int h, int piece, int64_t ld, int rows_valid) {
    const int k = k_of(piece);
    if constexpr (KC) {
      int tr = tile_row(h, piece >> 3);
      tr = tr < rows_valid ? tr : rows_valid - 1;
      return (uint32_t)((tr * ld + k) * 2);
    } else {
      const int sw = ((k & 3) | ((k >> 1) & 4)) << 1;
      const int col = tile_row(h, ((piece % (HR / 8)) ^ sw) * 8);
      return (uint32_t)((k * ld + (col < rows_valid ? col : 0)) * 2);
    }
  }
  __device__ __forceinline__ void init(int64_t ld, int rows_valid) {
    const int t = thread_id();  // piece q THREADS + t of a half is this thread's
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int q = 0; q < NQ; ++q) off[h][q] = source(h, q * THREADS + t, ld, rows_valid);
  }
  template <int H>
  __device__ __forceinline__ void issue(const char* __restrict__ base, lds<char>* slot) const {
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      uint32_t o = off[H][q];
      asm("" : "+v"(o));  // keeps base + o an SGPR base with a 32-bit offset (volatile: dD 1.5% slower)
      __builtin_amdgcn_global_load_lds((const void*)(base + o), (lds<void>*)(slot + (q * (THREADS / 64) + w) * 1024),
                                       16, 0, 0);
    }
  }
  // The last, partial stage of k_left K positions: the pieces past them come from a piece of zeros.
  template <int H>
  __device__ __forceinline__ void issue_last(const char* __restrict__ base, int k_left, lds<char>* slot) const {
    const int t = thread_id(), w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint64_t b = reinterpret_cast<uint64_t>(base), z = reinterpret_cast<uint64_t>(&kZeros);
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const bool in = k_of(q * THREADS + t) < k_left;
      // 32-bit halves: as 64-bit sums the offsets would be kept in register pairs
      const uint32_t lo = (uint32_t)b + off[H][q], hi = (uint32_t)(b >> 32) + (lo < off[H][q] ? 1u : 0u);
      const uint64_t from = (uint64_t)(in ? hi : (uint32_t)(z >> 32)) << 32 | (in ? lo : (uint32_t)z);
      __builtin_amdgcn_global_load_lds(reinterpret_cast<const void*>(from),
                                       (lds<void>*)(slot + (q * (THREADS / 64) + w) * 1024), 16, 0, 0);
    }
  }
  // The same through registers, after the loop.
  __device__ __forceinline__ static void tail(int h, const char* __restrict__ base, int64_t ld, int rows_valid,
                                              int k_left, lds<char>* slot) {
    const int t = thread_id();
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int piece = q * THREADS + t;
      const uint32_t o = source(h, piece, ld, rows_valid);
      i32x4 v = i32x4{0, 0, 0, 0};
      if (k_of(piece) < k_left)
        v = *reinterpret_cast<const __attribute__((address_space(1))) i32x4*>(
            (const __attribute__((address_space(1))) char*)base + o);
      *reinterpret_cast<lds<i32x4>*>(slot + piece * 16) = v;
    }
  }
};

// A lane's LDS addresses of the MFMA fragments in a half-panel slot: fragment i covers rows
// row0 + 16 i .. + 15 (row0 a multiple of 32) and K 32 ks .. + 31.  `at` is the slot's offset.
template <bool KC, int HR, int N>
struct HalfFrags {
  // KC: two addresses, the swizzle's bit 2 alternating with i and ks; KS: one per fragment row
  static constexpr int NA = KC ? 2 : N;
  int a[NA];
  __device__ __forceinline__ void init(int row0, int lr, int lg) {
    if constexpr (KC) {
      const int f = (lr ^ (lr >> 2)) & 7;
      a[0] = (row0 + lr) * 128 + ((lg ^ f) << 4);
      a[1] = (row0 + lr) * 128 + (((lg + 4) ^ f) << 4);
    } else {
      const int k = 8 * lg + (lr >> 2);
#pragma unroll
      for (int i = 0; i < N; ++i) a[i] = ks_off<HR>(k, (row0 + 16 * i + 4 * (lr & 3)) * 2);
    }
  }
  // moves every address by d bytes, in place: the other stage's addresses would otherwise be
  // kept in registers of their own through the loop
  __device__ __forceinline__ void move(int d) {
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      a[i] += d;
      asm volatile("" : "+v"(a[i]));
    }
  }
  __device__ __forceinline__ bf16x8 read(lds<char>* slot, int i, int ks) const {
    if constexpr (KC) {
      return *reinterpret_cast<const lds<bf16x8>*>(slot + a[(i ^ ks) & 1] + i * 2048);
    } else {
      typedef short s4 __attribute__((ext_vector_type(4)));
      typedef short s8 __attribute__((ext_vector_type(8)));
      // K advances by 4 and by 32 without touching the swizzle (bits 0, 1 and 3 of K)
      lds<char>* p = slot + a[i] + ks * 32 * HR * 2;
      const s4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds<s4>*)p);
      const s4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds<s4>*)(p + 4 * HR * 2));
      const s8 v = s8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      return __builtin_bit_cast(bf16x8, v);
    }
  }
};

// The K loop of one tile, split in two so that a persistent kernel can start the next tile's
// loads before it runs the current tile's epilogue:
//   prime()  issues the first loads of a tile (LDS must be free: after run()'s closing barrier,
//            or at kernel start);
//   run()    the main loop; it ends with a barrier after which LDS is free again.
//            run<.., X>(.., after_prime) is for a caller that issued exactly X further memory
//            operations (per wave) between prime() and run() when after_prime is true: the waits
//            for the primed loads let those X stay in flight.
// A_SW > 0: A is K-contiguous and stored slab-major -- K split into slabs of A_SW columns,
// slab s of every row at A + s a_sstride, lda = A_SW within a slab (A_SW a multiple of BK).
// Set the stride with slab_a() before prime().
// A partial last stage is one more stage of the loop, its pieces past the end loaded from zeros; with
// REG_TAIL it goes through registers after the loop: the row norms leave no registers for the other
// (48 spilled, 200,000 x 2048 bf16 against 256 centres 319 -> 570 us), and the loop of long reductions
// over rows (dD) comes out 2% slower with it.  The experts' weight gradients take the stage: dW1 of few
// long segments loses 3% (58,224 x 112, six experts 927 -> 955 us), of many gains 8% and more (skewed
// step 685 -> 630, 5003 x 1000 and 50 experts 131 -> 119).
template <class C, bool A_KC, bool B_KC, int A_SW = 0, bool REG_TAIL = false>
struct PipeTile {
  using OA = HalfPanels<C::BM, C::WM, C::THREADS, A_KC, false>;
  using OB = HalfPanels<C::BN, C::WN, C::THREADS, B_KC, C::SPLIT>;
  static constexpr int AL = OA::NQ, BL = OB::NQ;
  static constexpr int HI = C::MI / 2, HJ = C::NJ / 2;
  static_assert(A_SW == 0 || (A_KC && A_SW % C::BK == 0), "slab-major A: K-contiguous, whole stages per slab");
  static_assert(!C::F32 || (A_KC && B_KC), "fp32: K-contiguous operands only");
  OA oa;
  OB ob;
  HalfFrags<A_KC, C::BM / 2, HI> fa;
  HalfFrags<B_KC, C::BN / 2, HJ> fb;
  const char* A;
  const char* B;
  int64_t step_a, step_b;  // bytes per stage
  int64_t slab_bytes = 0;
  int nk, k_last;  // stages, and K positions of the last one (REG_TAIL: of the tail)
  int64_t lda, ldb;
  int a_rows, b_rows;

  __device__ __forceinline__ void slab_a(int64_t stride) { slab_bytes = stride * 2; }
  __device__ __forceinline__ const char* a_at(int k) const {  // stage k of A
    const char* p;
    if constexpr (A_SW > 0)
      p = A + (k / (A_SW / C::BK)) * slab_bytes + (k % (A_SW / C::BK)) * (C::BK * 2);
    else
      p = A + k * step_a;
    return uniform(p);
  }
  __device__ __forceinline__ const char* b_at(int k) const { return uniform(B + k * step_b); }
  __device__ __forceinline__ static lds<char>* slot_a(lds<char>* smem, int par, int h) {
    return smem + par * C::STAGE + h * C::A_HALF;
  }
  __device__ __forceinline__ static lds<char>* slot_b(lds<char>* smem, int par, int h) {
    return smem + par * C::STAGE + 2 * C::A_HALF + h * C::B_HALF;
  }

  // Loads of half H of stage k, which may be the last.
  template <int H>
  __device__ __forceinline__ void load_a(int k, lds<char>* slot) const {
    if (!REG_TAIL && k == nk - 1 && k_last < C::BK) oa.template issue_last<H>(a_at(k), k_last, slot);
    else oa.template issue<H>(a_at(k), slot);
  }
  template <int H>
  __device__ __forceinline__ void load_b(int k, lds<char>* slot) const {
    if (!REG_TAIL && k == nk - 1 && k_last < C::BK) ob.template issue_last<H>(b_at(k), k_last, slot);
    else ob.template issue<H>(b_at(k), slot);
  }

  // LONG: the reduction has at least two stages (no branches among the first one's loads)
  template <bool LONG = false>
  __device__ __forceinline__ void prime(const bf16* __restrict__ A_, int64_t lda_, int a_rows_,
                                        const bf16* __restrict__ B_, int64_t ldb_, int b_rows_, int k_len,
                                        lds<char>* smem) {
    A = uniform(reinterpret_cast<const char*>(A_));
    B = uniform(reinterpret_cast<const char*>(B_));
    lda = lda_;
    ldb = ldb_;
    a_rows = a_rows_;
    b_rows = b_rows_;
    k_len = __builtin_amdgcn_readfirstlane(k_len);
    nk = (REG_TAIL ? k_len : k_len + C::BK - 1) / C::BK;
    k_last = k_len - (REG_TAIL ? nk : nk - 1) * C::BK;
    step_a = A_KC ? C::BK * 2 : C::BK * 2 * lda;
    step_b = B_KC ? C::BK * 2 : C::BK * 2 * ldb;
    oa.init(lda, a_rows);
    ob.init(ldb, b_rows);
    if constexpr (LONG) {
      const char *pa = a_at(0), *pb = b_at(0);
      ob.template issue<0>(pb, slot_b(smem, 0, 0));
      oa.template issue<0>(pa, slot_a(smem, 0, 0));
      ob.template issue<1>(pb, slot_b(smem, 0, 1));
      oa.template issue<1>(pa, slot_a(smem, 0, 1));
    } else if (nk > 0) {
      load_b<0>(0, slot_b(smem, 0, 0));
      load_a<0>(0, slot_a(smem, 0, 0));
      load_b<1>(0, slot_b(smem, 0, 1));
      load_a<1>(0, slot_a(smem, 0, 1));
    }
    if (LONG || nk > 1) {
      load_b<0>(1, slot_b(smem, 1, 0));
      load_a<0>(1, slot_a(smem, 1, 0));
      load_b<1>(1, slot_b(smem, 1, 1));
    }
  }

  __device__ __forceinline__ void read_a(bf16x8 (&a)[HI][2], lds<char>* slot) const {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < HI; ++i) a[i][ks] = fa.read(slot, i, ks);
  }
  __device__ __forceinline__ void read_b(bf16x8 (&b)[HJ][2], lds<char>* slot) const {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int j = 0; j < HJ; ++j) b[j][ks] = fb.read(slot, j, ks);
  }

  // Quadrant (QI, QJ) of the wave's tile.  B is the MFMA's first operand: the 16 x 16 result is
  // the transposed sub-tile, so each lane ends up with four consecutive output columns of one row.
  template <int QI, int QJ>
  __device__ __forceinline__ static void mfmas(const bf16x8 (&a)[HI][2], const bf16x8 (&b)[HJ][2],
                                               floatx4 (&acc)[C::MI][C::NJ]) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int q = 0; q < (C::F32 ? 4 : 1); ++q)
#pragma unroll
        for (int i = 0; i < HI; ++i)
#pragma unroll
          for (int j = 0; j < HJ; ++j) {
            floatx4& c = acc[QI * HI + i][QJ * HJ + j];
            if constexpr (C::F32)
              c = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(floatx4, b[j][ks])[q],
                                                       __builtin_bit_cast(floatx4, a[i][ks])[q], c, 0, 0, 0);
            else
              c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j][ks], a[i][ks], c, 0, 0, 0);
          }
  }
  // xs[i / WAVES_N] += squares of this lane's elements of A fragment i, for the fragments i = wn
  // (mod WAVES_N) this wave is responsible for (each row's sum stays within one wave); bf16 as
  // packed dot products (the squares of bf16 values are exact in fp32).
  template <int QI>
  __device__ __forceinline__ static void row_squares(const bf16x8 (&a)[HI][2], int wn, float* xs) {
#pragma unroll
    for (int i = 0; i < HI; ++i)
      if (((QI * HI + i) % C::WAVES_N) == wn) {
        float& x = xs[(QI * HI + i) / C::WAVES_N];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          if constexpr (C::F32) {
            const floatx4 v = __builtin_bit_cast(floatx4, a[i][ks]);
#pragma unroll
            for (int e = 0; e < 4; ++e) x = fmaf(v[e], v[e], x);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const bf16x2 v = {a[i][ks][2 * e], a[i][ks][2 * e + 1]};
              x = __builtin_amdgcn_fdot2_f32_bf16(v, v, x, false);
            }
          }
        }
      }
  }
  __device__ __forceinline__ static void mid_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    wg_barrier_lds();
    __builtin_amdgcn_sched_barrier(0);
  }
  __device__ __forceinline__ static void end_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    wg_barrier();
    __builtin_amdgcn_sched_barrier(0);
  }

  // Stage s in parity PAR, `left` stages before the last (STEADY: at least two); b0 = B0(s) in
  // registers, b0n receives B0(s + 1).  extra: the caller's X operations may still be in flight.
  template <int PAR, bool STEADY, bool ROWNORM, int X>
  __device__ __forceinline__ void stage(lds<char>* smem, floatx4 (&acc)[C::MI][C::NJ], bf16x8 (&b0)[HJ][2],
                                        bf16x8 (&b0n)[HJ][2], int s, int left, int wn, float* xs, bool extra) {
    constexpr int kFlip = PAR == 0 ? C::STAGE : -C::STAGE;
    bf16x8 a[HI][2], b1[HJ][2];
    read_a(a, slot_a(smem, 0, 0));  // fa and fb carry the stage's parity
    read_b(b1, slot_b(smem, 0, 1));
    if constexpr (STEADY) {
      oa.template issue<1>(a_at(s + 1), slot_a(smem, PAR ^ 1, 1));
      ob.template issue<0>(b_at(s + 2), slot_b(smem, PAR, 0));
    } else {
      if (left >= 1) load_a<1>(s + 1, slot_a(smem, PAR ^ 1, 1));
      if (left >= 2) load_b<0>(s + 2, slot_b(smem, PAR, 0));
    }
    if (X > 0 && extra) {
      if (STEADY || left >= 2) wait_vmcnt<2 * AL + 2 * BL + X>();
      else if (left == 1) wait_vmcnt<2 * AL + BL + X>();
      else wait_vmcnt<X>();
    } else {
      if (STEADY || left >= 2) wait_vmcnt<2 * AL + 2 * BL>();
      else if (left == 1) wait_vmcnt<2 * AL + BL>();
      else wait_vmcnt<0>();
    }
    mid_barrier();
    mfmas<0, 0>(a, b0, acc);
    mfmas<0, 1>(a, b1, acc);
    if constexpr (ROWNORM) row_squares<0>(a, wn, xs);
    end_barrier();
    read_a(a, slot_a(smem, 0, 1));
    fa.move(kFlip);
    fb.move(kFlip);
    if (STEADY || left >= 1) read_b(b0n, slot_b(smem, 0, 0));
    if constexpr (STEADY) {
      oa.template issue<0>(a_at(s + 2), slot_a(smem, PAR, 0));
      ob.template issue<1>(b_at(s + 2), slot_b(smem, PAR, 1));
    } else if (left >= 2) {
      load_a<0>(s + 2, slot_a(smem, PAR, 0));
      load_b<1>(s + 2, slot_b(smem, PAR, 1));
    }
    if (X > 0 && extra) {
      if (STEADY || left >= 2) wait_vmcnt<2 * AL + 2 * BL + X>();
      else if (left == 1) wait_vmcnt<AL + X>();
    } else {
      if (STEADY || left >= 2) wait_vmcnt<2 * AL + 2 * BL>();
      else if (left == 1) wait_vmcnt<AL>();
    }
    mid_barrier();
    mfmas<1, 0>(a, b0, acc);
    mfmas<1, 1>(a, b1, acc);
    if constexpr (ROWNORM) row_squares<1>(a, wn, xs);
    end_barrier();
  }

  // ZERO: the sums start at zero, otherwise at what acc holds
  template <bool ROWNORM = false, int X = 0, bool ZERO = true>
  __device__ __forceinline__ void run(lds<char>* smem, floatx4 (&acc)[C::MI][C::NJ], float* xs = nullptr,
                                      bool after_prime = false) {
    static_assert(!ROWNORM || A_KC, "row norms need a K-contiguous A");
    static_assert(2 * AL + 2 * BL + X <= 63, "vmcnt range");
    if constexpr (ROWNORM) {
#pragma unroll
      for (int i = 0; i < (C::MI + C::WAVES_N - 1) / C::WAVES_N; ++i) xs[i] = 0.f;
    }
    if constexpr (ZERO) {
#pragma unroll
      for (int i = 0; i < C::MI; ++i)
#pragma unroll
        for (int j = 0; j < C::NJ; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    const int l = thread_id() & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wm = w / C::WAVES_N, wn = w % C::WAVES_N;
    fa.init(wm * (C::WM / 2), l & 15, l >> 4);
    fb.init(wn * (C::WN / 2), l & 15, l >> 4);
    const bool g1 = w >= C::WAVES / 2;
    bf16x8 be[HJ][2], bo[HJ][2];  // B0 of even and odd stages
    if (nk > 0) {
      if (X > 0 && after_prime) {
        if (nk > 1) wait_vmcnt<2 * AL + 2 * BL + X>(); else wait_vmcnt<AL + X>();
      } else {
        if (nk > 1) wait_vmcnt<2 * AL + 2 * BL>(); else wait_vmcnt<AL>();
      }
      wg_barrier();
      read_b(be, slot_b(smem, 0, 0));
      wg_barrier_lds();  // B0's slot of stage 0 is loaded again from phase 0 on
      if (g1) wg_barrier();
    }
    int s = 0;
    // a first stage with the caller's operations in flight; the compiler may not see that it is
    // the first (it would make a copy of the loop body for it)
    auto extra = [&]() {
      int first = s;
      asm volatile("" : "+s"(first));
      return X > 0 && after_prime && first == 0;
    };
    const int whole = !REG_TAIL && k_last < C::BK ? nk - 1 : nk;  // stages that may be loaded without a look at their end
    for (; s + 3 < whole; s += 2) {  // loads up to stage s + 3
      stage<0, true, ROWNORM, X>(smem, acc, be, bo, s, 0, wn, xs, extra());
      stage<1, true, ROWNORM, 0>(smem, acc, bo, be, s + 1, 0, wn, xs, false);
    }
    for (; s < nk; s += 2) {
      stage<0, false, ROWNORM, X>(smem, acc, be, bo, s, nk - 1 - s, wn, xs, extra());
      if (s + 1 < nk) stage<1, false, ROWNORM, 0>(smem, acc, bo, be, s + 1, nk - 2 - s, wn, xs, false);
    }
    if (nk > 0 && !g1) wg_barrier();
    if (REG_TAIL && k_last > 0) {
      bf16x8 a[HI][2];
      const char *pa = a_at(nk), *pb = b_at(nk);
      fa.init(wm * (C::WM / 2), l & 15, l >> 4);
      fb.init(wn * (C::WN / 2), l & 15, l >> 4);
      wg_barrier_lds();
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        OA::tail(h, pa, lda, a_rows, k_last, slot_a(smem, 0, h));
        OB::tail(h, pb, ldb, b_rows, k_last, slot_b(smem, 0, h));
      }
      wg_barrier_lds();
      read_b(be, slot_b(smem, 0, 0));
      read_b(bo, slot_b(smem, 0, 1));
      read_a(a, slot_a(smem, 0, 0));
      mfmas<0, 0>(a, be, acc);
      mfmas<0, 1>(a, bo, acc);
      if constexpr (ROWNORM) row_squares<0>(a, wn, xs);
      read_a(a, slot_a(smem, 0, 1));
      mfmas<1, 0>(a, be, acc);
      mfmas<1, 1>(a, bo, acc);
      if constexpr (ROWNORM) row_squares<1>(a, wn, xs);
    }
    wg_barrier_lds();
  }
};

// The tile loop of a direct-to-LDS configuration.
template <class C, bool A_KC, bool B_KC, bool REG_TAIL = false, bool PIPE = C::PIPE>
struct TileLoop {
  using type = PipeTile<C, A_KC, B_KC, 0, REG_TAIL>;
};
template <class C, bool REG_TAIL>
struct TileLoop<C, true, true, REG_TAIL, false> {
  using type = DmaTile<C>;
};

template <class C, bool A_KC, bool B_KC, bool ROWNORM = false, bool REG_TAIL = false>
__device__ __forceinline__ void gemm_tile_dma(const bf16* __restrict__ A, int64_t lda, int a_rows,
                                              const bf16* __restrict__ B, int64_t ldb, int b_rows, int k_len,
                                              lds<char>* smem, floatx4 (&acc)[C::MI][C::NJ],
                                              float* xs = nullptr) {
  typename TileLoop<C, A_KC, B_KC, REG_TAIL>::type t;
  t.prime(A, lda, a_rows, B, ldb, b_rows, k_len, smem);
  t.template run<ROWNORM>(smem, acc, xs);
}

// Whether C is a direct-to-LDS configuration with fp32 operands.
template <class C>
__device__ __host__ constexpr bool dma_f32() {
  if constexpr (C::DMA)
    return C::F32;
  else
    return false;
}

// Full K loop for one tile on whichever engine the configuration names.
template <class C, bool A_KC, bool B_KC, bool ROWNORM = false, bool REG_TAIL = false>
__device__ __forceinline__ void gemm_tile(const typename C::type* __restrict__ A, int64_t lda, int a_rows,
                                          const typename C::type* __restrict__ B, int64_t ldb, int b_rows,
                                          int k_len, lds<char>* smem, floatx4 (&acc)[C::MI][C::NJ],
                                          float* xs = nullptr) {
  if constexpr (dma_f32<C>()) {
    static_assert(A_KC && B_KC, "fp32 on the direct-to-LDS engine: K-contiguous operands only");
    gemm_tile_dma<C, A_KC, B_KC, ROWNORM, REG_TAIL>(reinterpret_cast<const bf16*>(A), 2 * lda, a_rows,
                                          reinterpret_cast<const bf16*>(B), 2 * ldb, b_rows, 2 * k_len, smem, acc, xs);
  } else if constexpr (C::DMA) {
    gemm_tile_dma<C, A_KC, B_KC, ROWNORM, REG_TAIL>(A, lda, a_rows, B, ldb, b_rows, k_len, smem, acc, xs);
  } else {
    gemm_tile_reg<C, A_KC, B_KC, ROWNORM>(A, lda, a_rows, B, ldb, b_rows, k_len, smem, acc, xs);
  }
}

// ------------------------------------------------------------------ tile scheduling

// Which output tile a workgroup owns.
struct TileCoord {
  int group;      // expert id (0 for ungrouped problems)
  int64_t m0;     // first output row (global, in the row space of A / C)
  int m_rows;     // valid rows in this tile
  int n0;         // first output column
  int n_cols;     // valid columns
  int64_t k0;     // first reduction index (grouped-K problems)
  int k_len;      // reduction length
  int valid;      // not bool: whole registers, so that copies of a tile stay out of memory
};

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uniform(int64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}
// The tile in scalar registers: its coordinates come out of 64-bit divisions, which leave them in
// vector registers that a persistent kernel would hold (and spill for) through its K loop.
__device__ __forceinline__ TileCoord uniform(const TileCoord& t) {
  return TileCoord{uniform(t.group), uniform(t.m0), uniform(t.m_rows), uniform(t.n0),
                   uniform(t.n_cols), uniform(t.k0), uniform(t.k_len), uniform(t.valid)};
}

// Plain problem: M x N tiles, bands of `band` m-tiles walked m-fastest so that concurrently
// running workgroups share both operand tiles in the caches.
template <class C>
__device__ __forceinline__ TileCoord tile_plain_at(int64_t M, int N, int K, int64_t b) {
  TileCoord tc;
  const int64_t mt = cdiv(M, C::BM);
  const int nt = (int)cdiv(N, C::BN);
  constexpr int band = 16;
  const int64_t band_tiles = (int64_t)band * nt;
  const int64_t g = b / band_tiles;
  const int64_t in = b - g * band_tiles;
  const int64_t m_first = g * band;
  const int64_t bm = (mt - m_first < band) ? (mt - m_first) : band;
  const int64_t mi = m_first + in % bm;
  const int ni = (int)(in / bm);
  tc.group = 0;
  tc.m0 = mi * C::BM;
  tc.n0 = ni * C::BN;
  tc.valid = (mi < mt) && (ni < nt);
  tc.m_rows = (int)((M - tc.m0) < C::BM ? (M - tc.m0) : C::BM);
  tc.n_cols = (N - tc.n0) < C::BN ? (N - tc.n0) : C::BN;
  tc.k0 = 0;
  tc.k_len = K;
  return tc;
}
template <class C>
__device__ __forceinline__ TileCoord tile_plain(int64_t M, int N, int K) {
  return tile_plain_at<C>(M, N, K, blockIdx.x);
}

// Row-grouped problem (experts' forward / input-gradient GEMMs): group e owns rows
// [seg[e], seg[e+1]) of A and C.  tile_start[e] = number of BM-row tiles of groups < e
// (prefix, tile_start[G] = total).  Launched over an upper bound of m-tiles x n-tiles; the
// excess workgroups find no tile and exit.
// XCD: workgroups go to the 8 XCDs round-robin (blockIdx.x % 8), each with its own L2; this
// order gives each XCD a run of 8 consecutive m-tiles with all their n-tiles (of the
// 64 nt workgroups b = 64 nt r + q: XCD x = q % 8 takes m-tile 64 r + 8 x + (q / 8) / nt,
// n-tile (q / 8) % nt), so an XCD fetches each of its A row blocks once and the B tiles of
// few groups.  The grid must then be a multiple of 64 nt (the m-tile bound rounded up to 64).
template <class C, bool XCD = false>
__device__ __forceinline__ TileCoord tile_group_m(const int32_t* __restrict__ seg,
                                                  const int32_t* __restrict__ tile_start, int G, int N,
                                                  int K) {
  TileCoord tc;
  const int nt = (int)cdiv(N, C::BN);
  const int64_t b = blockIdx.x;
  int64_t mtile;
  int ni;
  if constexpr (XCD) {
    const int64_t r = b / (64 * nt), q = b - r * 64 * nt;
    const int slot = (int)(q / 8);
    mtile = r * 64 + (q % 8) * 8 + slot / nt;
    ni = slot % nt;
  } else {
    mtile = b / nt;
    ni = (int)(b - mtile * nt);
  }
  tc.valid = false;
  const int total = tile_start[G];
  if (mtile >= total) return tc;
  int lo = 0, hi = G - 1;  // last e with tile_start[e] <= mtile
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (tile_start[mid] <= mtile) lo = mid; else hi = mid - 1;
  }
  const int e = lo;
  const int64_t local = mtile - tile_start[e];
  const int64_t rows = seg[e + 1] - seg[e];
  tc.group = e;
  tc.m0 = seg[e] + local * C::BM;
  tc.m_rows = (int)((rows - local * C::BM) < C::BM ? (rows - local * C::BM) : C::BM);
  tc.n0 = ni * C::BN;
  tc.n_cols = (N - tc.n0) < C::BN ? (N - tc.n0) : C::BN;
  tc.k0 = 0;
  tc.k_len = K;
  tc.valid = tc.m_rows > 0;
  return tc;
}

// Reduction-grouped problem (experts' weight gradients): group e reduces over the rows
// [seg[e], seg[e+1]) of both operands; output tile (m, n) of group e.  Groups are taken in the
// order `order` gives (longest reduction first), so the deepest tiles start in the first round
// instead of forming the tail of the launch.  Within a group the tiles run in bands of 16
// m-tiles, m fastest (as tile_plain_at): the tiles that share an A panel are 16 workgroups
// apart, which the round-robin placement of workgroups puts on one XCD (one L2).
template <class C>
__device__ __forceinline__ TileCoord tile_group_k(const int32_t* __restrict__ seg,
                                                  const int32_t* __restrict__ order, int G, int M, int N) {
  TileCoord tc;
  const int mt = (int)cdiv(M, C::BM), nt = (int)cdiv(N, C::BN);
  const int64_t b = blockIdx.x;
  const int per = mt * nt;
  const int slot = (int)(b / per);
  const int in = (int)(b - (int64_t)slot * per);
  constexpr int band = 16;
  const int g = in / (band * nt);
  const int inb = in - g * band * nt;
  const int m_first = g * band;
  const int bm = (mt - m_first < band) ? (mt - m_first) : band;
  const int mi = m_first + inb % bm, ni = inb / bm;
  tc.valid = slot < G;
  const int e = tc.valid ? order[slot] : 0;
  tc.group = e;
  tc.m0 = (int64_t)mi * C::BM;
  tc.m_rows = (M - mi * C::BM) < C::BM ? (M - mi * C::BM) : C::BM;
  tc.n0 = ni * C::BN;
  tc.n_cols = (N - tc.n0) < C::BN ? (N - tc.n0) : C::BN;
  if (tc.valid) {
    tc.k0 = seg[e];
    tc.k_len = seg[e + 1] - seg[e];
  } else {
    tc.k0 = 0;
    tc.k_len = 0;
  }
  return tc;
}

// ------------------------------------------------------------------ epilogue helpers

// Where accumulator element (i, j, r) of this lane sits in the tile, for either orientation.
// A lane holds MI rows x NCOL columns (TRANS: one row per i and four consecutive columns per j;
// otherwise four rows per i and one column per j); qidx(j, r) numbers the lane's columns.
template <class C>
struct Frag {
  static constexpr bool T = C::TRANS;
  static constexpr int NCOL = T ? C::NJ * 4 : C::NJ;
  int wm, wn, lr, lg;
  __device__ __forceinline__ Frag() {
    const int l = thread_id() & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    wm = w / C::WAVES_N;
    wn = w % C::WAVES_N;
    lr = l & 15;
    lg = l >> 4;
  }
  __device__ __forceinline__ int row(int i, int r) const { return wm * C::WM + 16 * i + (T ? lr : 4 * lg + r); }
  // first column of the wave's 16-column block j
  __device__ __forceinline__ int block(int j) const {
    if constexpr (C::SPLIT)
      return (j / (C::NJ / 2)) * (C::BN / 2) + wn * (C::WN / 2) + 16 * (j % (C::NJ / 2));
    else
      return wn * C::WN + 16 * j;
  }
  __device__ __forceinline__ int col(int j, int r) const { return block(j) + (T ? 4 * lg + r : lr); }
  __device__ __forceinline__ static constexpr int qidx(int j, int r) { return T ? 4 * j + r : j; }
  __device__ __forceinline__ int colq(int q) const { return T ? col(q >> 2, q & 3) : col(q, 0); }
};

// Four consecutive output values of one type, as stored by store_direct.
template <typename O>
using vec4 = O __attribute__((ext_vector_type(4)));

// Epilogue store through LDS: the tile is written to LDS row-major (padded rows, conflict-free
// for the accumulator layout) in bands of rows, then copied out so that every lane stores whole
// 16-byte row segments.  Must be entered by the whole workgroup after the main loop.
//   elem(i, j, r, v)            value to store for accumulator element (i, j, r) holding v
//   rowmap(local_row)           destination row index (local_row < m_rows)
//   vec(dst_row, local_row, col, raw)  last transform of a 16-byte vector (e.g. a mask)
// n_cols must be a multiple of 16 / sizeof(O).
struct NoVec {
  template <typename V>
  __device__ __forceinline__ V operator()(int64_t, int, int, V v) const { return v; }
};

template <class C, typename O, class Elem, class RowMap, class Vec>
__device__ __forceinline__ void store_tile(const TileCoord& tc, const floatx4 (&acc)[C::MI][C::NJ],
                                           lds<char>* smem, O* __restrict__ out, int64_t ldo, Elem elem,
                                           RowMap rowmap, Vec vec) {
  constexpr int ROWB = C::BN * (int)sizeof(O) + 16;
  constexpr int FIT = C::LDS / ROWB;
  constexpr int BAND = FIT >= 256 ? 256 : (FIT >= 128 ? 128 : (FIT >= 64 ? 64 : 32));
  constexpr int VPR = C::BN * (int)sizeof(O) / 16;
  constexpr int EPV = 16 / (int)sizeof(O);
  const Frag<C> f;
#pragma unroll
  for (int b = 0; b < (C::BM + BAND - 1) / BAND; ++b) {
    if (b * BAND >= tc.m_rows) break;
#pragma unroll
    for (int i = 0; i < C::MI; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = f.row(i, r) - b * BAND;
        if (row < 0 || row >= BAND) continue;
#pragma unroll
        for (int j = 0; j < C::NJ; ++j)
          *reinterpret_cast<lds<O>*>(smem + row * ROWB + f.col(j, r) * (int)sizeof(O)) =
              from_f32<O>(elem(i, j, r, acc[i][j][r]));
      }
    __syncthreads();
    for (int q = threadIdx.x; q < BAND * VPR; q += C::THREADS) {
      const int lrow = q / VPR, v = q - lrow * VPR;
      const int row = b * BAND + lrow, col = v * EPV;
      if (row < tc.m_rows && col < tc.n_cols) {
        const int64_t dr = rowmap(row);
        i32x4 raw = *reinterpret_cast<const lds<i32x4>*>(smem + lrow * ROWB + v * 16);
        raw = vec(dr, row, col, raw);
        *reinterpret_cast<i32x4*>(out + dr * ldo + tc.n0 + col) = raw;
      }
    }
    __syncthreads();
  }
}

// Epilogue store straight from registers (TRANS orientation): no LDS, no barrier.  Same
// functors as store_tile, with vec applied to the stored vector.
//   2-byte outputs: lanes lg and lg ^ 1 (16 apart, same row) trade halves of their column
//   blocks 2p and 2p + 1 with one v_permlane16_swap per dword, after which every lane holds
//   8 consecutive columns (at 32 p + 16 (lg & 1) + 8 (lg >> 1) of the wave's columns) and
//   stores them as one 16-byte vector: each store instruction covers 64 contiguous bytes of 16
//   rows.
//   4-byte outputs: every lane stores its four consecutive columns as one 16-byte vector.
// direct_stores<C, O>() is the number of store instructions a wave issues for a full tile.
template <class C, typename O>
__device__ __forceinline__ constexpr bool direct_pairs() {
  return sizeof(O) == 2 && (C::SPLIT ? C::NJ % 4 == 0 : C::NJ % 2 == 0);
}
template <class C, typename O>
__device__ __forceinline__ constexpr int direct_stores() {
  return direct_pairs<C, O>() ? C::MI * C::NJ / 2 : C::MI * C::NJ;
}
// FULL: every row and column of the tile is valid, and no store sits behind a branch.  The
// destination rows are all fetched before the first store: fetched one by one between the
// stores, a row map costs a memory latency per 16 rows.
template <class C, typename O, bool FULL, class Elem, class RowMap, class Vec>
__device__ __forceinline__ void store_direct_rows(const TileCoord& tc, const floatx4 (&acc)[C::MI][C::NJ],
                                                  O* __restrict__ out, int64_t ldo, Elem elem, RowMap rowmap,
                                                  Vec vec) {
  static_assert(C::TRANS, "direct stores need the transposed accumulator layout");
  const Frag<C> f;
  int64_t dst[C::MI];
#pragma unroll
  for (int i = 0; i < C::MI; ++i) {
    const int row = f.row(i, 0);
    dst[i] = rowmap(FULL || row < tc.m_rows ? row : tc.m_rows - 1);
  }
  if constexpr (direct_pairs<C, O>()) {
    typedef unsigned int u2v __attribute__((ext_vector_type(2)));
    typedef unsigned int u4v __attribute__((ext_vector_type(4)));
    typedef O v8 __attribute__((ext_vector_type(8)));
    const int cpos = 16 * (f.lg & 1) + 8 * (f.lg >> 1);
#pragma unroll
    for (int i = 0; i < C::MI; ++i) {
      const int row = f.row(i, 0);
      const bool row_ok = FULL || row < tc.m_rows;  // the same for the two lanes of a swap
#pragma unroll
      for (int p = 0; p < C::NJ / 2; ++p) {
        vec4<O> va, vb;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          va[r] = from_f32<O>(elem(i, 2 * p, r, acc[i][2 * p][r]));
          vb[r] = from_f32<O>(elem(i, 2 * p + 1, r, acc[i][2 * p + 1][r]));
        }
        const u2v a = __builtin_bit_cast(u2v, va), b = __builtin_bit_cast(u2v, vb);
        // odd 16-lane rows of the first operand trade with even rows of the second
        const u2v s0 = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
        const u2v s1 = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
        const u4v w = u4v{s0[0], s1[0], s0[1], s1[1]};
        const int col = f.block(2 * p) + cpos;
        if (row_ok && (FULL || col < tc.n_cols))
          *reinterpret_cast<v8*>(out + dst[i] * ldo + tc.n0 + col) = vec(dst[i], row, col, __builtin_bit_cast(v8, w));
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < C::MI; ++i) {
      const int row = f.row(i, 0);
      if (!FULL && row >= tc.m_rows) continue;
      O* orow = out + dst[i] * ldo + tc.n0;
#pragma unroll
      for (int j = 0; j < C::NJ; ++j) {
        const int col = f.col(j, 0);
        if (!FULL && col >= tc.n_cols) continue;
        vec4<O> v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = from_f32<O>(elem(i, j, r, acc[i][j][r]));
        *reinterpret_cast<vec4<O>*>(orow + col) = vec(dst[i], row, col, v);
      }
    }
  }
}
template <class C, typename O, class Elem, class RowMap, class Vec>
__device__ __forceinline__ void store_direct(const TileCoord& tc, const floatx4 (&acc)[C::MI][C::NJ],
                                             O* __restrict__ out, int64_t ldo, Elem elem, RowMap rowmap, Vec vec) {
  if (tc.m_rows == C::BM && tc.n_cols == C::BN)
    store_direct_rows<C, O, true>(tc, acc, out, ldo, elem, rowmap, vec);
  else
    store_direct_rows<C, O, false>(tc, acc, out, ldo, elem, rowmap, vec);
}

// Destination row of a tile row for the plain case: m0 + r.
struct RowId {
  int64_t m0;
  __device__ __forceinline__ int64_t operator()(int r) const { return m0 + r; }
};

// Tile configurations per data type, C for a K-contiguous B and CK for a K-strided one: bf16
// runs the 256 x 256 pipelined engine, fp32 -- and bf16 rows too wide for the pipelined engine's
// 32-bit offsets -- the register-staged 128 x 128 one.
template <typename T, bool WIDE_ = false>
struct Pick {
  static constexpr bool WIDE = true;
  using C = CfgSmall<T>;
  using CK = CfgSmall<T>;
};
template <>
struct Pick<bf16, false> {
  static constexpr bool WIDE = false;
  using C = CfgPipe;
  using CK = CfgPipeKS;
};

// The epilogue store for the configuration's orientation.
template <class C, typename O, class Elem, class RowMap, class Vec>
__device__ __forceinline__ void store_out(const TileCoord& tc, const floatx4 (&acc)[C::MI][C::NJ], lds<char>* smem,
                                          O* __restrict__ out, int64_t ldo, Elem elem, RowMap rowmap, Vec vec) {
  if constexpr (C::TRANS)
    store_direct<C, O>(tc, acc, out, ldo, elem, rowmap, vec);
  else
    store_tile<C, O>(tc, acc, smem, out, ldo, elem, rowmap, vec);
}

}  // namespace hmoe
