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

// The m-th largest over the lanes of x (with multiplicity), m <= 16: each row of 16 lanes is sorted
// (bitonic, each merge starting with the mirrored pair, so that every step keeps the larger value
// in the lower lane), then the 16 largest of two rows are the larger ones of one row and the other
// reversed, sorted again.  A step is a lane move and a median with +inf or -inf: about 50
// instructions (130 in a full sort by selects of minima and maxima).
__device__ __forceinline__ float max_of(float a, float b) {  // one instruction, any NaN passed over
  return __builtin_amdgcn_fmed3f(a, b, INFINITY);
}
__device__ __forceinline__ float mth_lane_value(float x, int m, int l) {
  const auto step = [&](float y, int bit) {
    x = __builtin_amdgcn_fmed3f(x, y, (l & bit) ? -INFINITY : INFINITY);  // the smaller : the larger
  };
  const auto xor1 = [&] { step(dpp<0xB1>(x), 1); };           // quad_perm [1,0,3,2]
  const auto xor2 = [&] { step(dpp<0x4E>(x), 2); };           // quad_perm [2,3,0,1]
  const auto xor4 = [&] { step(dpp<0x1B>(dpp<0x141>(x)), 4); };  // half mirror, quad mirror
  const auto xor8 = [&] { step(dpp<0x128>(x), 8); };          // row_ror:8
  xor1();
  step(dpp<0x1B>(x), 2);  // quad mirror
  xor1();
  step(dpp<0x141>(x), 4);  // half mirror
  xor2();
  xor1();
  step(dpp<0x140>(x), 8);  // row mirror
  xor4();
  xor2();
  xor1();
  // rows 0 and 2 take the best of rows 0, 1 and 2, 3
  unsigned y = __float_as_uint(dpp<0x140>(x));
  x = max_of(x, __uint_as_float(__builtin_amdgcn_permlane16_swap(y, y, false, false)[1]));
  xor8();
  xor4();
  xor2();
  xor1();
  // row 0 the best of all
  y = __float_as_uint(dpp<0x140>(x));
  x = max_of(x, __uint_as_float(__builtin_amdgcn_permlane32_swap(y, y, false, false)[1]));
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

template <typename T, int M>
__global__ void __launch_bounds__(256) k_topm(const T* __restrict__ L, int64_t n, int V, int m,
                                              int32_t* __restrict__ idx, float* __restrict__ val) {
  constexpr int EPV = 16 / sizeof(T);
  constexpr int U = 4;  // vectors in flight
  const int l = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n) return;
  const T* r = L + row * (int64_t)V;
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
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int v = b0 + 64 * u + l;
      if (v < nvec) raw[u] = *reinterpret_cast<const i32x4*>(r + (int64_t)v * EPV);
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
        f[z] = to_f32(e[z]);
        vmax = fmaxf(vmax, f[z]);
      }
      if (!(vmax >= thr && vmax > lv[M - 1])) continue;  // the common case: nothing here enters
#pragma unroll
      for (int z = 0; z < EPV; ++z)
        if (f[z] >= thr && f[z] > lv[M - 1]) list_carry(lv, li, f[z], v * EPV + z);
    }
    // the m-th largest of the lanes' maxima: m lanes each hold an entry at least that large
    // (refreshed on the first steps, then every 4th: it settles quickly, and any value it
    // took is a valid bound)
    if (step >= 4 && (step & 3) != 0) continue;
    thr = mth_lane_value(lv[0], m, l);
  }
  emit_topm(lv, li, m, l, row, idx, val);
}

// Anchored logits, one wave per row and eight adjacent rows per workgroup.  Block b (columns
// [64 b, 64 b + 64)) of row i has its anchor at anc[((b / 4) n + i) 4 + b % 4], and every entry
// of it is at most that anchor; the four anchors of a 256-column tile are one 16-byte vector, and
// the eight rows' vectors one 128-byte line, which the workgroup's waves read at about the same
// time.
//   1. The workgroup stages the rows' anchors in LDS, whole lines, and lane l takes the tiles l, l + 64,
//      ... of its wave's row.  The m-th largest of the lanes' largest anchors is a bound t0 that at
//      least m blocks reach, and those are listed.  Neighbouring blocks are in one lane, so a
//      vocabulary in order of frequency lists up to 4 m: with more than whole reads of m blocks need,
//      t0 becomes the m-th largest of the listed anchors, and the blocks below it are dropped.
//   2. The blocks are read, a 16-byte vector per lane, several blocks at once.  t1 = the
//      m-th largest of the lanes' largest entries; the entries >= t1 (m and a few more) are
//      collected in LDS, one per lane, and ranked by (value desc, index asc).
//   3. Every entry outside those blocks is below t0, so t_m is among theirs when the m-th of them is
//      >= t0.  With the forward's anchors (each its block's maximum, so each block holds an entry
//      equal to its anchor) this is always the case.
//   4. Otherwise, and where a list overflows (equal anchors or entries, best entries in few blocks),
//      the wave goes through the blocks in order, reads those whose anchor ranks before the
//      m-th best entry so far, and keeps the entries that do (k_topm_anchored's `stream`).
// The work per row is under a thousand vector instructions and two trips to memory (290 MB at
// 65,536 x 50,000 bf16 logits and m = 10).
//   At 65,536 x 50,000 bf16, in us (a lane per row with sorted lists of anchors / a wave per row that
//   reads its own anchors, a lane's 16 bytes a line apart / this): m = 10 on i.i.d. logits
//   375 / 141 / 111, m = 1 69 / 84 / 54; logits -1.1 ln(rank) + 0.5 N(0, 1) m = 10 400 / 1540 / 124,
//   and 1.0 N(0, 1) m = 16 659 / 2046 / 157 (whole rows where the candidates outnumbered a list of
//   32); logits in steps of 4 (many equal anchors) 1431 / 3662 / 438; 512 rows 194 / 17 / 14.
constexpr int kTopmWaves = 8;    // rows per workgroup
constexpr int kTopmBlocks = 32;  // blocks read at once at most
constexpr int kTopmRegTiles = 4;  // anchor tiles of a lane in registers
constexpr int kTopmLd = 64 * kTopmRegTiles + 2;  // 16 lanes' stores (8 rows of 2 tiles) in 16 bank groups

template <typename T>
__global__ void __launch_bounds__(64 * kTopmWaves, 6)
    k_topm_anchored(const T* __restrict__ L, const float* __restrict__ anc, int64_t n, int V, int m,
                    int32_t* __restrict__ idx, float* __restrict__ val) {
  constexpr int EPV = 16 / sizeof(T);
  constexpr int VPB = kAnchorCols / EPV;           // vectors per block
  constexpr int BPR = 64 / VPB;                    // blocks a wave reads at once
  constexpr int ROUNDS = kTopmBlocks / BPR;
  static_assert(kAnchorSlots == 4, "one 16-byte anchor vector per tile");
  __shared__ floatx4 s_tile[kTopmWaves][kTopmLd];
  const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t row0 = (int64_t)blockIdx.x * kTopmWaves, row = row0 + w;
  const int nb = (int)cdiv(V, kAnchorCols);
  const int nt = (int)cdiv(V, kAnchorTile);
  const floatx4* arow = reinterpret_cast<const floatx4*>(anc) + row;  // tile t at arow[t n]
  {
    const int sr = threadIdx.x % kTopmWaves, st = threadIdx.x / kTopmWaves;
    const floatx4* from = reinterpret_cast<const floatx4*>(anc) + row0 + (row0 + sr < n ? sr : 0) + (int64_t)st * n;
    floatx4 x[kTopmRegTiles];
#pragma unroll
    for (int u = 0; u < kTopmRegTiles; ++u)
      if (st + 64 * u < nt) x[u] = from[(int64_t)(64 * u) * n];
#pragma unroll
    for (int u = 0; u < kTopmRegTiles; ++u)
      if (st + 64 * u < nt) s_tile[sr][st + 64 * u] = x[u];
  }
  __syncthreads();
  if (row >= n) return;
  const T* r = L + row * (int64_t)V;
  const auto present = [&](floatx4 x, int t) {
#pragma unroll
    for (int sl = 1; sl < 4; ++sl) x[sl] = 4 * t + sl < nb ? x[sl] : NAN;
    return x;
  };
  const auto tile = [&](int t) { return present(t < nt ? arow[(int64_t)t * n] : floatx4{NAN, NAN, NAN, NAN}, t); };
  const auto top_of = [](float x, const floatx4& q) {
    return max_of(max_of(max_of(max_of(x, q[0]), q[1]), q[2]), q[3]);
  };
  floatx4 q[kTopmRegTiles];
#pragma unroll
  for (int u = 0; u < kTopmRegTiles; ++u) {
    q[u] = s_tile[w][l + 64 * u];
    q[u][0] = l + 64 * u < nt ? q[u][0] : NAN;
    q[u] = present(q[u], l + 64 * u);
  }
  wave_lds_fence();
  // the row's tiles are in registers: their place holds the lists
  int32_t* s_blk = reinterpret_cast<int32_t*>(s_tile[w]);  // blocks: 64, in `stream` 256
  float* s_anc = reinterpret_cast<float*>(s_blk + 256);
  float* s_val = s_anc + 256;  // entries
  int32_t* s_idx = reinterpret_cast<int32_t*>(s_val + 64);
  float top = -INFINITY;
#pragma unroll
  for (int u = 0; u < kTopmRegTiles; ++u) top = top_of(top, q[u]);
  for (int t = 64 * kTopmRegTiles; t < nt; t += 64) top = top_of(top, tile(t + l));
  float t0 = mth_lane_value(top, m, l);
  int listed = 0;  // wave-uniform
  auto list = [&](const floatx4& x, int t) {
#pragma unroll
    for (int sl = 0; sl < 4; ++sl) {
      const uint64_t hit = __ballot(x[sl] >= t0);
      if (hit == 0) continue;
      const int at = listed + lanes_below(hit);
      if (((hit >> l) & 1) && at < 64) {
        s_blk[at] = 4 * t + sl;
        s_anc[at] = x[sl];
      }
      listed += __popcll(hit);
    }
  };
#pragma unroll
  for (int u = 0; u < kTopmRegTiles; ++u) list(q[u], l + 64 * u);
  for (int t = 64 * kTopmRegTiles; t < nt; t += 64) list(tile(t + l), t + l);
  wave_lds_fence();
  if (listed > (m + BPR - 1) / BPR * BPR && listed <= 64) {
    const float a = l < listed ? s_anc[l] : -INFINITY;
    const int32_t b = l < listed ? s_blk[l] : 0;
    t0 = mth_lane_value(a, m, l);
    const uint64_t keep = __ballot(l < listed && a >= t0);
    wave_lds_fence();
    if ((keep >> l) & 1) {
      s_blk[lanes_below(keep)] = b;
      s_anc[lanes_below(keep)] = a;
    }
    listed = __popcll(keep);
    wave_lds_fence();
  }
  // The m-th of the `count` <= 64 entries listed, ranked by (value desc, index asc), as (vb, ib); `rank`
  // of this lane's entry (v, i).
  float vb = t0, v = 0.f;
  int ib = INT32_MAX, i = 0, rank = 0;
  const auto rank_entries = [&](int count) {
    wave_lds_fence();
    v = l < count ? s_val[l] : -INFINITY;
    i = l < count ? s_idx[l] : INT32_MAX;
    rank = 0;
    for (int k = 0; k < count; ++k) {
      const float ov = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), k));
      const int oi = __builtin_amdgcn_readlane(i, k);
      rank += (ov > v || (ov == v && oi < i)) ? 1 : 0;
    }
    const uint64_t last = __ballot(l < count && rank == m - 1);
    if (last == 0) return false;
    const int at = 63 - __builtin_clzll(last);
    vb = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), at));
    ib = __builtin_amdgcn_readlane(i, at);
    return true;
  };
  const auto emit = [&](int count) {
    const int at = l < count ? rank : l;  // past the entries (a row with NaN): no index
    if (at < m) {
      idx[row * (int64_t)m + at] = i;
      if (val) val[row * (int64_t)m + at] = v;
    }
  };
  bool bounded = false;  // m entries rank at or before (vb, ib)
  if (listed <= kTopmBlocks) {
    // the blocks, BPR at a time: lane l takes vector l % VPB of block l / VPB
    float f[ROUNDS][EPV];
    int c0[ROUNDS];
    i32x4 raw[ROUNDS];
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u) {
      const int k = u * BPR + l / VPB;
      c0[u] = V;
      if (u * BPR < listed && k < listed) {
        c0[u] = s_blk[k] * kAnchorCols + (l % VPB) * EPV;
        if (c0[u] < V) raw[u] = *reinterpret_cast<const i32x4*>(r + c0[u]);
      }
    }
    float best = -INFINITY;
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u) {
      if (u * BPR >= listed) break;
      const int k = u * BPR + l / VPB;
      const float a = k < listed ? s_anc[k] : 0.f;
      const T* e = reinterpret_cast<const T*>(&raw[u]);
#pragma unroll
      for (int z = 0; z < EPV; ++z) {
        f[u][z] = c0[u] < V ? a + to_f32(e[z]) : NAN;  // absent: never listed
        best = max_of(best, f[u][z]);
      }
    }
    const float t1 = mth_lane_value(best, m, l);
    int kept = 0;  // wave-uniform
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u) {
      if (u * BPR >= listed) break;
#pragma unroll
      for (int z = 0; z < EPV; ++z) {
        const uint64_t hit = __ballot(f[u][z] >= t1);
        if (hit == 0) continue;
        const int at = kept + lanes_below(hit);
        if (((hit >> l) & 1) && at < 64) {
          s_val[at] = f[u][z];
          s_idx[at] = c0[u] + z;
        }
        kept += __popcll(hit);
      }
    }
    if (kept <= 64) {
      bounded = rank_entries(kept);
      if (bounded && vb >= t0) {
        emit(kept);
        return;
      }
    } else {
      vb = t1;
      bounded = true;
    }
  }
  // Goes through the blocks in order and lists the entries that rank before (vb, ib), which the m-th best
  // one becomes whenever the list is full.  False when there are fewer than m (written if `last`).
  const auto stream = [&](bool last) {
    int count = 0;
    const auto before = [&](float x, int j) { return x > vb || (x == vb && j < ib); };
    for (int t = 0; t < nt; t += 64) {
      const floatx4 x = tile(t + l);
      uint64_t hit[4];
      int total = 0, at = 0;
#pragma unroll
      for (int sl = 0; sl < 4; ++sl) {
        hit[sl] = __ballot(before(x[sl], (4 * (t + l) + sl) * kAnchorCols));
        at += lanes_below(hit[sl]);
        total += __popcll(hit[sl]);
      }
      wave_lds_fence();
#pragma unroll
      for (int sl = 0; sl < 4; ++sl)
        if ((hit[sl] >> l) & 1) {
          s_blk[at] = 4 * (t + l) + sl;
          s_anc[at++] = x[sl];
        }
      wave_lds_fence();
      for (int k0 = 0; k0 < total; k0 += BPR) {
        const int k = k0 + l / VPB;
        const int b = k < total ? s_blk[k] : 0;
        const float a = k < total ? s_anc[k] : NAN;
        const int c = b * kAnchorCols + (l % VPB) * EPV;
        const bool in = before(a, b * kAnchorCols) && c < V;
        if (__ballot(in) == 0) continue;
        i32x4 raw = {0, 0, 0, 0};
        if (in) raw = *reinterpret_cast<const i32x4*>(r + c);
        for (int z = 0; z < EPV; ++z) {
          const int q = z * (int)sizeof(T) / 4;
          const uint32_t word = (uint32_t)(q < 2 ? (q == 0 ? raw[0] : raw[1]) : (q == 2 ? raw[2] : raw[3]));
          const uint32_t bits = sizeof(T) == 4 ? word : ((z & 1) ? word & 0xffff0000u : word << 16);
          float f = in ? a + __uint_as_float(bits) : NAN;
          for (;;) {
            const uint64_t enter = __ballot(before(f, c + z));
            const int at = count + lanes_below(enter), full = count + __popcll(enter);
            if (((enter >> l) & 1) && at < 64) {
              s_val[at] = f;
              s_idx[at] = c + z;
              f = NAN;
            }
            count = full < 64 ? full : 64;
            if (full <= 64) break;
            rank_entries(count);
            wave_lds_fence();
            if (rank < m) {
              s_val[rank] = v;
              s_idx[rank] = i;
            }
            count = m;
          }
        }
      }
    }
    const bool found = rank_entries(count);
    if (found || last) emit(count);
    return found;
  };
  // entries equal to the bound count, but those of it that are behind the m-th one known
  if (bounded && ib < INT32_MAX) ++ib;
  if (stream(bounded) || bounded) return;
  // t0 bounds anchors that are their blocks' maxima: here they are not
  vb = -INFINITY;
  ib = INT32_MAX;
  stream(true);
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
