// metrics.hip -- the inference tail of Section 4.4: t_m, the m largest logits of every row
// (the softmax keeps their order, so these are the m most probable tags), and the counts
// behind p@m (Eq. 4) and q@m (Eq. 5) for every m' <= m.
//
// k_topm (plain logits): one wave per row; each lane keeps its own m largest entries in a
// register list sorted by (value desc, index asc), and the m results are taken in m rounds of
// a wave-wide (value desc, index asc) maximum over the lists' heads, the lane holding the
// winner dropping it.  Lane l reads the row's 16-byte vectors l, l + 64, ... (so it sees its
// entries in increasing index order, and an entry enters only when strictly greater than the
// list's last, which keeps equal values in increasing index order), and only when it is not
// below a wave-wide bound on the row's m-th value (the m-th largest of the lanes' maxima).
// The row is read once: the kernel is bound by HBM.
// k_topm_anchored (logits stored as offsets <= 0 from per-row anchors, one per 64 columns, as
// the forward writes them; an entry is anchor + offset formed in fp32), one wave per row: a
// block's anchor bounds all its entries, so the row's anchors (a few KB) are read and only the
// blocks whose anchor can reach the row's m-th entry -- a few more than m blocks of 64 columns
// when every anchor is its block's maximum.
//
// k_topm_hits: one thread per row (p) and per draw (q); the rank of each matching tag in the
// top-m list adds 1 to every m' above it.  Integer counts, summed through LDS and then with
// one 64-bit atomic per block and m' -- integer sums, so the result does not depend on order.
#include "launch.hpp"
#include "primitives.hpp"

namespace hmoe {

// Carries entry (cv, ci) down the list ordered by (value desc, index asc): it goes before the
// first entry it ranks above, and each entry it displaces is carried on by the same order.
template <int M>
__device__ __forceinline__ void list_carry(float (&lv)[M], int (&li)[M], float cv, int ci) {
#pragma unroll
  for (int k = 0; k < M; ++k) {
    const bool gt = cv > lv[k] || (cv == lv[k] && ci < li[k]);
    const float tv = lv[k];
    const int ti = li[k];
    lv[k] = gt ? cv : tv;
    li[k] = gt ? ci : ti;
    cv = gt ? tv : cv;
    ci = gt ? ti : ci;
  }
}

// The m largest entries of the union of the lanes' lists, in (value desc, index asc) order.
template <int M>
__device__ __forceinline__ void emit_topm(float (&lv)[M], int (&li)[M], int m, int l, int64_t row,
                                          int32_t* __restrict__ idx, float* __restrict__ val) {
  for (int q = 0; q < m; ++q) {
    float bv = lv[0];
    int bi = li[0];
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) {
      const float ov = shfl_xor(bv, s);
      const int oi = shfl_xor(bi, s);
      if (ov > bv || (ov == bv && oi < bi)) {
        bv = ov;
        bi = oi;
      }
    }
    if (li[0] == bi) {  // this lane's head won: drop it
#pragma unroll
      for (int k = 0; k < M - 1; ++k) {
        lv[k] = lv[k + 1];
        li[k] = li[k + 1];
      }
      lv[M - 1] = -INFINITY;
      li[M - 1] = 0x7fffffff;
    }
    if (l == 0) {
      idx[row * (int64_t)m + q] = bi;
      if (val) val[row * (int64_t)m + q] = bv;
    }
  }
}

// The m-th largest over the lanes of x (with multiplicity): a bitonic sort of the 64 lanes in
// registers, each merge starting with the mirrored pair (so that every step keeps the larger
// value in the lower lane).  About 90 instructions; m rounds of a wave maximum take 16 m.
template <int CTRL>
__device__ __forceinline__ float dpp_of(float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float mth_lane_value(float x, int m, int l) {
  typedef unsigned int u2v __attribute__((ext_vector_type(2)));
  const auto step = [&](float y, int bit) { x = (l & bit) ? fminf(x, y) : fmaxf(x, y); };
  const auto xor1 = [&] { step(dpp_of<0xB1>(x), 1); };           // quad_perm [1,0,3,2]
  const auto xor2 = [&] { step(dpp_of<0x4E>(x), 2); };           // quad_perm [2,3,0,1]
  const auto xor4 = [&] { step(dpp_of<0x1B>(dpp_of<0x141>(x)), 4); };  // half mirror, quad mirror
  const auto xor8 = [&] { step(dpp_of<0x128>(x), 8); };          // row_ror:8
  const auto rows16 = [&](float y) {  // y from the lane 16 away
    const u2v a = __builtin_amdgcn_permlane16_swap(__float_as_uint(y), __float_as_uint(y), false, false);
    return __uint_as_float((l & 16) ? a[0] : a[1]);
  };
  const auto rows32 = [&](float y) {  // y from the lane 32 away
    const u2v a = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
    return __uint_as_float((l & 32) ? a[0] : a[1]);
  };
  xor1();
  step(dpp_of<0x1B>(x), 2);  // quad mirror
  xor1();
  step(dpp_of<0x141>(x), 4);  // half mirror
  xor2();
  xor1();
  step(dpp_of<0x140>(x), 8);  // row mirror
  xor4();
  xor2();
  xor1();
  step(rows16(dpp_of<0x140>(x)), 16);
  xor8();
  xor4();
  xor2();
  xor1();
  step(rows16(rows32(dpp_of<0x140>(x))), 32);
  step(rows16(x), 16);
  xor8();
  xor4();
  xor2();
  xor1();
  return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), m - 1));
}

// Set bits of `mask` below this lane.
__device__ __forceinline__ int lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}

// Orders a wave's LDS writes before its later reads by other lanes of the same wave.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// One row's t_m by one wave, reading the whole row: r its entries, arow its anchors' four-slot
// tiles (tile t at arow[t n]; NULL: the stored values are the entries).  U vectors in flight.
template <typename T, int M, int U>
__device__ __forceinline__ void topm_row(const T* __restrict__ r, const floatx4* __restrict__ arow, int64_t n, int V,
                                         int m, int l, int64_t row, int32_t* __restrict__ idx,
                                         float* __restrict__ val) {
  constexpr int EPV = 16 / sizeof(T);
  float lv[M];
  int li[M];
#pragma unroll
  for (int k = 0; k < M; ++k) {
    lv[k] = -INFINITY;
    li[k] = 0x7fffffff;
  }
  const int nvec = V / EPV;
  // Wave-wide lower bound on the row's m-th largest value (the m-th largest of the lanes'
  // maxima: m entries are at least that large), so an entry below thr is not in t_m (entries
  // equal to it may be, and stay).  It closes in on the m-th value within a few steps, which
  // keeps the insertion branch -- taken by the wave when any lane takes it -- rare.
  float thr = -INFINITY;
  // the trip count is the same for every lane (the bound is a wave-wide shuffle reduction)
  int step = 0;
  for (int b0 = 0; b0 < nvec; b0 += 64 * U, ++step) {
    i32x4 raw[U];
    float an[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int v = b0 + 64 * u + l;
      an[u] = 0.f;
      if (v < nvec) {
        raw[u] = *reinterpret_cast<const i32x4*>(r + (int64_t)v * EPV);
        if (arow) {
          const int c = v * EPV;
          an[u] = reinterpret_cast<const float*>(arow + (int64_t)(c / kAnchorTile) * n)[(c % kAnchorTile) / kAnchorCols];
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int v = b0 + 64 * u + l;
      if (v >= nvec) break;
      const T* e = reinterpret_cast<const T*>(&raw[u]);
      float f[EPV];
      float vmax = -INFINITY;
#pragma unroll
      for (int z = 0; z < EPV; ++z) {
        f[z] = arow ? an[u] + to_f32(e[z]) : to_f32(e[z]);
        vmax = fmaxf(vmax, f[z]);
      }
      // the common case: nothing here enters (an unfilled slot also takes a -inf entry of
      // anchored logits, whose rows may have fewer than m finite ones)
      const bool open = arow && li[M - 1] == 0x7fffffff;
      if (!(vmax >= thr && (vmax > lv[M - 1] || open))) continue;
#pragma unroll
      for (int z = 0; z < EPV; ++z)
        if (f[z] >= thr && (f[z] > lv[M - 1] || (arow && f[z] == lv[M - 1] && li[M - 1] == 0x7fffffff)))
          list_carry(lv, li, f[z], v * EPV + z);
    }
    // the m-th largest of the lanes' maxima: m lanes each hold an entry at least that large
    // (refreshed on the first steps, then every 4th: it settles quickly, and any value it
    // took is a valid bound)
    if (step >= 4 && (step & 3) != 0) continue;
    thr = mth_lane_value(lv[0], m, l);
  }
  emit_topm(lv, li, m, l, row, idx, val);
}

template <typename T, int M>
__global__ void __launch_bounds__(256) k_topm(const T* __restrict__ L, int64_t n, int V, int m,
                                              int32_t* __restrict__ idx, float* __restrict__ val) {
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n) return;
  topm_row<T, M, 4>(L + row * (int64_t)V, nullptr, n, V, m, threadIdx.x & 63, row, idx, val);
}

// Anchored logits, one wave per row and eight adjacent rows per workgroup.  Block b (columns
// [64 b, 64 b + 64)) of row i has its anchor at anc[((b / 4) n + i) 4 + b % 4], and every entry
// of it is at most that anchor; the four anchors of a 256-column tile are one 16-byte vector, and
// the eight rows' vectors one 128-byte line, which the workgroup's waves read at about the same
// time.
//   1. Lane l reads the tiles l, l + 64, ... of its row.  t0 = the m-th largest of the lanes'
//      largest anchors: at least m blocks have an anchor >= t0.  Those blocks are listed in LDS
//      (a few more than m: a lane that holds two of the largest lowers t0 a little).
//   2. The listed blocks are read, a 16-byte vector per lane, several blocks at once.  t1 = the
//      m-th largest of the lanes' largest entries; the entries >= t1 (m and a few more) are
//      collected in LDS, one per lane, and ranked by (value desc, index asc).
//   3. Every entry outside the listed blocks is below t0, so t_m is among the listed ones when
//      the m-th of them is >= t0.  With the forward's anchors (each its block's maximum, so each
//      listed block holds an entry equal to its anchor) this is always the case.  Otherwise, and
//      when the lists overflow (many equal anchors or entries), the wave reads the whole row.
// The work per row is under a thousand vector instructions and two trips to memory (290 MB at
// 65,536 x 50,000 bf16 logits and m = 10): 0.36 -> 0.11 ms there against a lane per row with
// sorted lists of anchors, whose insertions every lane of a wave waits for, and 0.19 -> 0.01 ms
// for 512 rows, which gave that kernel 8 workgroups.  Six waves per SIMD: four (no bound) take
// 0.14 ms, eight 0.11 ms but spill the lists of the whole-row pass, which then takes 295 ms
// instead of 2.5 on anchors above their blocks' entries (6.0 ms with sorted lists per lane).
constexpr int kTopmWaves = 8;    // rows per workgroup
constexpr int kTopmBlocks = 32;  // listed blocks at most
constexpr int kTopmRegTiles = 4;  // anchor tiles a lane keeps between its two looks at them

template <typename T>
__global__ void __launch_bounds__(64 * kTopmWaves, 6)
    k_topm_anchored(const T* __restrict__ L, const float* __restrict__ anc, int64_t n, int V, int m,
                    int32_t* __restrict__ idx, float* __restrict__ val) {
  constexpr int EPV = 16 / sizeof(T);
  constexpr int VPB = kAnchorCols / EPV;           // vectors per block
  constexpr int BPR = 64 / VPB;                    // blocks a wave reads at once
  constexpr int ROUNDS = kTopmBlocks / BPR;
  static_assert(kAnchorSlots == 4, "one 16-byte anchor vector per tile");
  __shared__ int32_t s_blk[kTopmWaves][kTopmBlocks];
  __shared__ float s_anc[kTopmWaves][kTopmBlocks];
  __shared__ float s_val[kTopmWaves][64];
  __shared__ int32_t s_idx[kTopmWaves][64];
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t row = (int64_t)blockIdx.x * kTopmWaves + w;
  if (row >= n) return;
  const int nb = (int)cdiv(V, kAnchorCols);
  const int nt = (int)cdiv(V, kAnchorTile);
  const floatx4* arow = reinterpret_cast<const floatx4*>(anc) + row;  // tile t at arow[t n]
  const T* r = L + row * (int64_t)V;
  // a tile's anchors, absent blocks as -inf
  auto tile = [&](int t) {
    floatx4 q = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    if (t < nt) {
      q = arow[(int64_t)t * n];
#pragma unroll
      for (int sl = 0; sl < 4; ++sl)
        if (4 * t + sl >= nb) q[sl] = -INFINITY;
    }
    return q;
  };
  floatx4 q[kTopmRegTiles];
#pragma unroll
  for (int u = 0; u < kTopmRegTiles; ++u) q[u] = tile(l + 64 * u);
  float top = -INFINITY;
#pragma unroll
  for (int u = 0; u < kTopmRegTiles; ++u) top = fmaxf(fmaxf(fmaxf(top, q[u][0]), fmaxf(q[u][1], q[u][2])), q[u][3]);
  for (int t = 64 * kTopmRegTiles; t < nt; t += 64) {
    const floatx4 x = tile(t + l);
    top = fmaxf(fmaxf(fmaxf(top, x[0]), fmaxf(x[1], x[2])), x[3]);
  }
  const float t0 = mth_lane_value(top, m, l);
  int listed = 0;  // wave-uniform
  auto list = [&](const floatx4& x, int t) {
#pragma unroll
    for (int sl = 0; sl < 4; ++sl) {
      const uint64_t hit = __ballot(4 * t + sl < nb && x[sl] >= t0);
      if (hit == 0) continue;
      const int at = listed + lanes_below(hit);
      if (((hit >> l) & 1) && at < kTopmBlocks) {
        s_blk[w][at] = 4 * t + sl;
        s_anc[w][at] = x[sl];
      }
      listed += __popcll(hit);
    }
  };
#pragma unroll
  for (int u = 0; u < kTopmRegTiles; ++u) list(q[u], l + 64 * u);
  for (int t = 64 * kTopmRegTiles; t < nt; t += 64) list(tile(t + l), t + l);
  bool found = false;
  if (listed <= kTopmBlocks) {
    wave_lds_fence();
    // the listed blocks, BPR at a time: lane l takes vector l % VPB of block l / VPB
    float f[ROUNDS][EPV];
    int c0[ROUNDS];
    i32x4 raw[ROUNDS];
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u) {
      const int k = u * BPR + l / VPB;
      c0[u] = V;
      if (u * BPR < listed && k < listed) {
        c0[u] = s_blk[w][k] * kAnchorCols + (l % VPB) * EPV;
        if (c0[u] < V) raw[u] = *reinterpret_cast<const i32x4*>(r + c0[u]);
      }
    }
    float best = -INFINITY;
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u) {
      if (u * BPR >= listed) break;
      const int k = u * BPR + l / VPB;
      const float a = k < listed ? s_anc[w][k] : 0.f;
      const T* e = reinterpret_cast<const T*>(&raw[u]);
#pragma unroll
      for (int z = 0; z < EPV; ++z) {
        f[u][z] = c0[u] < V ? a + to_f32(e[z]) : -INFINITY;
        best = fmaxf(best, f[u][z]);
      }
    }
    const float t1 = mth_lane_value(best, m, l);
    int kept = 0;  // wave-uniform
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u) {
      if (u * BPR >= listed) break;
#pragma unroll
      for (int z = 0; z < EPV; ++z) {
        const uint64_t hit = __ballot(c0[u] < V && f[u][z] >= t1);
        if (hit == 0) continue;
        const int at = kept + lanes_below(hit);
        if (((hit >> l) & 1) && at < 64) {
          s_val[w][at] = f[u][z];
          s_idx[w][at] = c0[u] + z;
        }
        kept += __popcll(hit);
      }
    }
    if (kept >= m && kept <= 64) {
      wave_lds_fence();
      const float v = l < kept ? s_val[w][l] : -INFINITY;
      const int i = l < kept ? s_idx[w][l] : 0x7fffffff;
      int rank = 0;
      for (int k = 0; k < kept; ++k) {
        const float ov = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), k));
        const int oi = __builtin_amdgcn_readlane(i, k);
        rank += (ov > v || (ov == v && oi < i)) ? 1 : 0;
      }
      // the m-th found entry settles whether anything outside the listed blocks could rank
      const uint64_t last = __ballot(l < kept && rank == m - 1 && v >= t0);
      found = last != 0;
      if (found && l < kept && rank < m) {
        idx[row * (int64_t)m + rank] = i;
        if (val) val[row * (int64_t)m + rank] = v;
      }
    }
  }
  if (!found) topm_row<T, 16, 1>(r, arow, n, V, m, l, row, idx, val);
}

// hits[0 .. m) for p, hits[m .. 2m) for q; must start at zero.
__global__ void __launch_bounds__(256) k_topm_hits(const int32_t* __restrict__ idx, int64_t n, int m,
                                                   const int32_t* __restrict__ row_ptr,
                                                   const int32_t* __restrict__ tag,
                                                   const int32_t* __restrict__ q_sample,
                                                   const int32_t* __restrict__ q_tag, int64_t S,
                                                   unsigned long long* __restrict__ hits) {
  __shared__ unsigned int cnt[2 * 16];
  if (threadIdx.x < 2 * 16) cnt[threadIdx.x] = 0u;
  __syncthreads();
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t < n) {
    const int32_t* top = idx + t * (int64_t)m;
    for (int32_t q = row_ptr[t]; q < row_ptr[t + 1]; ++q) {
      const int32_t tg = tag[q];
      for (int k = 0; k < m; ++k)
        if (top[k] == tg) {
          atomicAdd(&cnt[k], 1u);  // counted for every m' > k below
          break;
        }
    }
  } else if (t - n < S) {
    const int64_t s = t - n;
    const int32_t i = q_sample[s];
    if (i >= 0 && i < n) {  // a draw naming no sample counts as a miss
      const int32_t* top = idx + (int64_t)i * m;
      const int32_t tg = q_tag[s];
      for (int k = 0; k < m; ++k)
        if (top[k] == tg) {
          atomicAdd(&cnt[16 + k], 1u);
          break;
        }
    }
  }
  __syncthreads();
  if (threadIdx.x < m) {
    // the entry at rank k is in t_m' for every m' > k: prefix over the ranks
    unsigned long long p = 0, qh = 0;
    for (int k = 0; k <= (int)threadIdx.x; ++k) {
      p += cnt[k];
      qh += cnt[16 + k];
    }
    if (p) atomicAdd(&hits[threadIdx.x], p);
    if (qh) atomicAdd(&hits[m + threadIdx.x], qh);
  }
}

template <typename T, int M>
static int topm_launch(const T* L, int64_t n, int V, int m, int32_t* idx, float* val, hipStream_t st) {
  HMOE_LAUNCH("top-m", (k_topm<T, M>), dim3((unsigned)cdiv(n, 4)), dim3(256), 0, st, L, n, V, m, idx, val);
  return HMOE_OK;
}

// The plain kernel's register lists hold exactly m entries (the insertion and the registers
// scale with the list length: a 16-entry list for m = 10 ran 25% slower than a 12-entry one).
template <typename T>
static int topm_t(const T* L, const float* anc, int64_t n, int V, int m, int32_t* idx, float* val, hipStream_t st) {
  if (anc) {
    HMOE_LAUNCH("top-m", k_topm_anchored<T>, dim3((unsigned)cdiv(n, kTopmWaves)), dim3(64 * kTopmWaves), 0, st, L, anc,
                n, V, m, idx, val);
    return HMOE_OK;
  }
  switch (m) {
    case 1: return topm_launch<T, 1>(L, n, V, m, idx, val, st);
    case 2: return topm_launch<T, 2>(L, n, V, m, idx, val, st);
    case 3: return topm_launch<T, 3>(L, n, V, m, idx, val, st);
    case 4: return topm_launch<T, 4>(L, n, V, m, idx, val, st);
    case 5: return topm_launch<T, 5>(L, n, V, m, idx, val, st);
    case 6: return topm_launch<T, 6>(L, n, V, m, idx, val, st);
    case 7: return topm_launch<T, 7>(L, n, V, m, idx, val, st);
    case 8: return topm_launch<T, 8>(L, n, V, m, idx, val, st);
    case 9: return topm_launch<T, 9>(L, n, V, m, idx, val, st);
    case 10: return topm_launch<T, 10>(L, n, V, m, idx, val, st);
    case 11: return topm_launch<T, 11>(L, n, V, m, idx, val, st);
    case 12: return topm_launch<T, 12>(L, n, V, m, idx, val, st);
    case 13: return topm_launch<T, 13>(L, n, V, m, idx, val, st);
    case 14: return topm_launch<T, 14>(L, n, V, m, idx, val, st);
    case 15: return topm_launch<T, 15>(L, n, V, m, idx, val, st);
    default: return topm_launch<T, 16>(L, n, V, m, idx, val, st);
  }
}

int launch_topm(const void* L, const float* anc, hmoe_dtype_t dt, int64_t n, int V, int m, int32_t* idx, float* val,
                hipStream_t st) {
  if (dt == HMOE_BF16) return topm_t<bf16>((const bf16*)L, anc, n, V, m, idx, val, st);
  return topm_t<float>((const float*)L, anc, n, V, m, idx, val, st);
}

int launch_topm_hits(const int32_t* idx, int64_t n, int m, const hmoe_labels_t* y, const int32_t* q_sample,
                     const int32_t* q_tag, int64_t S, int64_t* hits, hipStream_t st) {
  HMOE_TRY(launch_zero_f32((float*)hits, 4 * (int64_t)m, st));  // 2m int64 = 4m zero words
  if (n + S == 0) return HMOE_OK;
  HMOE_LAUNCH("top-m hits", k_topm_hits, dim3((unsigned)cdiv(n + S, 256)), dim3(256), 0, st, idx, n, m, y->row_ptr,
              y->tag, q_sample, q_tag, S, (unsigned long long*)hits);
  return HMOE_OK;
}

}  // namespace hmoe
