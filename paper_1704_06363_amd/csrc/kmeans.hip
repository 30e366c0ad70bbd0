// kmeans.hip -- the K-means gater of Section 2: nearest-centroid assignment (Eq. 2) as a fused
// distance GEMM + argmin on MFMA, k-means++ seeding, and the Lloyd centre update as a
// deterministic segmented reduction with farthest-point reseeding of empty clusters.
#include <float.h>
#include <limits.h>

#include "gemm.hpp"
#include "launch.hpp"
#include "primitives.hpp"

namespace hmoe {

// ------------------------------------------------------------------ centre norms

// cn[k] = |c_k|^2, one wave per centre; lane l adds elements l, l + 64, ... in that order, eight
// loads in flight (one at a time a row of 2048 was 32 dependent trips to memory: 16 us, 5 us now).
// The order stays: a row between two centres goes to either with the last bit of a norm, and over
// Lloyd iterations whole clusters go with it.
// k_finalize_norm forms the same sum while it writes the centres.
template <typename T>
__global__ void __launch_bounds__(256) k_cnorm(const T* __restrict__ C, int K, int d, float* __restrict__ cn) {
  const int k = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int l = threadIdx.x & 63;
  if (k >= K) return;
  const T* row = C + (int64_t)k * d;
  float s = 0.f;
  int j = l;
  for (; j + 7 * 64 < d; j += 8 * 64) {
    T e[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) e[u] = row[j + 64 * u];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float c = to_f32(e[u]);
      s += c * c;
    }
  }
  for (; j < d; j += 64) {
    const float c = to_f32(row[j]);
    s += c * c;
  }
  s = wave_sum(s);
  if (l == 0) cn[k] = s;
}

// ------------------------------------------------------------------ distance GEMM + argmin

// One BM-row x BN-centre tile: dist'(i, k) = |c_k|^2 - 2 x_i . c_k (the |x_i|^2 term is
// common to the row); the tile's minimum per row (lowest k on ties) goes either straight to
// assign / min_dist (all centres in one tile) or to per-tile partials merged afterwards.
template <class C>
__global__ void __launch_bounds__(C::THREADS)
    k_assign(const typename C::type* __restrict__ X, int64_t n, int d, const typename C::type* __restrict__ Cn, int K,
             const float* __restrict__ cn, int32_t* __restrict__ assign, float* __restrict__ min_dist,
             float* __restrict__ part_v, int32_t* __restrict__ part_i, float* __restrict__ xnorm) {
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  lds<char>* smem = (lds<char>*)smem_raw;
  constexpr int NV = C::BM * 8 / C::THREADS;  // staged A vectors per thread
  const TileCoord tc = tile_plain<C>(n, K, d);
  if (!tc.valid) return;
  floatx4 acc[C::MI][C::NJ];
  float xs[NV];
  gemm_tile<C, true, true, true>(X + tc.m0 * d, d, tc.m_rows, Cn + (int64_t)tc.n0 * d, d, tc.n_cols, d, smem, acc,
                                 xs);
  lds<float>* xn = reinterpret_cast<lds<float>*>(smem);  // [BM]
  lds<float>* rv = xn + C::BM;                       // [WAVES_N][BM]
  lds<int32_t>* ri = reinterpret_cast<lds<int32_t>*>(rv + C::WAVES_N * C::BM);
  const int t = threadIdx.x;
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    float s = xs[q];
    s += shfl_xor(s, 1);
    s += shfl_xor(s, 2);
    s += shfl_xor(s, 4);
    if ((t & 7) == 0) xn[(t + C::THREADS * q) >> 3] = s;
  }
  const Frag<C> f;
#pragma unroll
  for (int i = 0; i < C::MI; ++i) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float best = FLT_MAX;
      int bi = INT_MAX;
#pragma unroll
      for (int j = 0; j < C::NJ; ++j) {
        const int col = f.col(j, 0);
        if (col < tc.n_cols) argmin_merge(best, bi, cn[tc.n0 + col] - 2.f * acc[i][j][r], tc.n0 + col);
      }
#pragma unroll
      for (int m = 1; m < 16; m <<= 1) {
        const float v2 = shfl_xor(best, m);
        const int i2 = shfl_xor(bi, m);
        argmin_merge(best, bi, v2, i2);
      }
      if (f.lr == 0) {
        rv[f.wn * C::BM + f.row(i, r)] = best;
        ri[f.wn * C::BM + f.row(i, r)] = bi;
      }
    }
  }
  __syncthreads();
  const int nt = (int)cdiv(K, C::BN);
  for (int q = t; q < tc.m_rows; q += C::THREADS) {
    float v = rv[q];
    int bi = ri[q];
#pragma unroll
    for (int w = 1; w < C::WAVES_N; ++w) argmin_merge(v, bi, rv[w * C::BM + q], ri[w * C::BM + q]);
    const int64_t row = tc.m0 + q;
    if (nt == 1) {
      assign[row] = bi;
      if (min_dist) min_dist[row] = fmaxf(v + xn[q], 0.f);
    } else {
      const int ti = tc.n0 / C::BN;
      part_v[(int64_t)ti * n + row] = v;
      part_i[(int64_t)ti * n + row] = bi;
      if (ti == 0) xnorm[row] = xn[q];
    }
  }
}

// (value, index) maximum with ties to the lower index over the four lanes 16 apart.
__device__ __forceinline__ void rows16_argmax(float& v, int& i) {
  typedef unsigned int u2v __attribute__((ext_vector_type(2)));
  const auto merge = [&](u2v a, u2v b) {
    const float v0 = __uint_as_float(a[0]), v1 = __uint_as_float(a[1]);
    const int i0 = (int)b[0], i1 = (int)b[1];
    const bool second = v1 > v0 || (v1 == v0 && i1 < i0);
    v = second ? v1 : v0;
    i = second ? i1 : i0;
  };
  merge(__builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false),
        __builtin_amdgcn_permlane16_swap((unsigned)i, (unsigned)i, false, false));
  merge(__builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false),
        __builtin_amdgcn_permlane32_swap((unsigned)i, (unsigned)i, false, false));
}

// The same tile on the direct-to-LDS engines (bf16 with many centres, and fp32).  A row's nearest
// centre is the maximum of x . c_k - |c_k|^2 / 2 = -dist' / 2 (the factor is exact): the epilogue
// is a subtraction, a compare and two selects per element, in increasing centre order, where a
// guarded (value, index) merge per element took 1.2 of 4.5 ms at 2^20 x 2048 rows and 1024
// centres.  The tile's |c_k|^2 / 2 wait in LDS past the operands, +inf for absent centres.  Each
// lane holds four consecutive centres of one row per fragment; the row norms come from the A
// fragments the engine already reads (fragment i summed by wave i mod WAVES_N).  fp32 rows are
// staged as 16-bit units (U per element).
template <class C>
constexpr int assign_lds() {
  return C::LDS + C::BN * (int)sizeof(float);
}
template <class C>
__global__ void __launch_bounds__(C::THREADS)
    k_assign_dma(const typename C::type* __restrict__ X, int64_t n, int d, const typename C::type* __restrict__ Cn,
                 int K,
                 const float* __restrict__ cn, int32_t* __restrict__ assign, float* __restrict__ min_dist,
                 float* __restrict__ part_v, int32_t* __restrict__ part_i, float* __restrict__ xnorm) {
  static_assert(C::DMA && C::TRANS, "direct-to-LDS configuration expected");
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  lds<char>* smem = (lds<char>*)smem_raw;
  const TileCoord tc = tile_plain<C>(n, K, d);
  if (!tc.valid) return;
  floatx4 acc[C::MI][C::NJ];
  float xs[(C::MI + C::WAVES_N - 1) / C::WAVES_N];
  using F = Frag<C>;
  // only the first centre tile of a row block needs the row norms (min_dist = min + |x|^2)
  constexpr int U = C::F32 ? 2 : 1;
  const bf16* Xu = reinterpret_cast<const bf16*>(X);
  const bf16* Cu = reinterpret_cast<const bf16*>(Cn);
  typename TileLoop<C, true, true, true>::type pipe;
  lds<float>* hn = reinterpret_cast<lds<float>*>(smem + C::LDS);  // [BN]
  static_assert(C::BN <= C::THREADS, "one thread per centre");
  float h = INFINITY;
  if ((int)threadIdx.x < tc.n_cols) h = 0.5f * cn[tc.n0 + threadIdx.x];
  pipe.prime(Xu + tc.m0 * d * U, (int64_t)d * U, tc.m_rows, Cu + (int64_t)tc.n0 * d * U, (int64_t)d * U, tc.n_cols,
             d * U, smem);
  if ((int)threadIdx.x < C::BN) hn[threadIdx.x] = h;  // read after the K loop's barriers
  if (tc.n0 == 0)
    pipe.template run<true>(smem, acc, xs);
  else
    pipe.template run<false>(smem, acc);
  const F f;
  lds<float>* xn = reinterpret_cast<lds<float>*>(smem);  // [BM]
  lds<float>* rv = xn + C::BM;                           // [WAVES_N][BM]
  lds<int32_t>* ri = reinterpret_cast<lds<int32_t>*>(rv + C::WAVES_N * C::BM);
#pragma unroll
  for (int i = 0; i < C::MI; ++i)
    if (tc.n0 == 0 && (i % C::WAVES_N) == f.wn) {
      const float s = rows16_reduce(xs[i / C::WAVES_N], [](float a, float b) { return a + b; });
      if (f.lg == 0) xn[f.row(i, 0)] = s;
    }
  floatx4 hv[C::NJ];
#pragma unroll
  for (int j = 0; j < C::NJ; ++j) hv[j] = *reinterpret_cast<const lds<floatx4>*>(hn + f.col(j, 0));
  float best[C::MI];
  int bi[C::MI];
#pragma unroll
  for (int i = 0; i < C::MI; ++i) {
    best[i] = -0.5f * FLT_MAX;  // dist' below FLT_MAX
    int o = -1;                 // 16 j + r of this lane's best
#pragma unroll
    for (int j = 0; j < C::NJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float v = acc[i][j][r] - hv[j][r];
        const bool gt = v > best[i];
        best[i] = gt ? v : best[i];
        o = gt ? f.col(j, r) - f.col(0, 0) : o;
      }
    bi[i] = o < 0 ? INT_MAX : tc.n0 + f.col(0, 0) + o;
  }
#pragma unroll
  for (int i = 0; i < C::MI; ++i) rows16_argmax(best[i], bi[i]);
  if (f.lg == 0) {
#pragma unroll
    for (int i = 0; i < C::MI; ++i) {
      rv[f.wn * C::BM + f.row(i, 0)] = -2.f * best[i];
      ri[f.wn * C::BM + f.row(i, 0)] = bi[i];
    }
  }
  __syncthreads();
  const int nt = (int)cdiv(K, C::BN);
  for (int q = threadIdx.x; q < tc.m_rows; q += C::THREADS) {
    float v = rv[q];
    int b = ri[q];
#pragma unroll
    for (int w = 1; w < C::WAVES_N; ++w) argmin_merge(v, b, rv[w * C::BM + q], ri[w * C::BM + q]);
    const int64_t row = tc.m0 + q;
    if (nt == 1) {
      assign[row] = b;
      if (min_dist) min_dist[row] = fmaxf(v + xn[q], 0.f);
    } else {
      const int ti = tc.n0 / C::BN;
      part_v[(int64_t)ti * n + row] = v;
      part_i[(int64_t)ti * n + row] = b;
      if (ti == 0) xnorm[row] = xn[q];
    }
  }
}

__global__ void __launch_bounds__(256) k_assign_merge(const float* __restrict__ part_v,
                                                      const int32_t* __restrict__ part_i,
                                                      const float* __restrict__ xnorm, int64_t n, int nt,
                                                      int32_t* __restrict__ assign, float* __restrict__ min_dist) {
  const int64_t row = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (row >= n) return;
  float v = FLT_MAX;
  int bi = INT_MAX;
  for (int t = 0; t < nt; ++t) argmin_merge(v, bi, part_v[(int64_t)t * n + row], part_i[(int64_t)t * n + row]);
  assign[row] = bi;
  if (min_dist) min_dist[row] = fmaxf(v + xnorm[row], 0.f);
}

// Centre-tile width of the assignment: up to 64 centres run the narrow 128 x 64 tiles of the
// ring engine, fp32 above that and bf16 above 128 centres the 256 x 256 tiles of the pipelined
// engine, bf16 with 65 .. 128 centres the register-staged 128 x 128 tiles -- and so do rows too
// wide for the pipelined engine.
static bool assign_pipe(int64_t d, hmoe_dtype_t dt, int32_t K) {
  return dt == HMOE_BF16 ? K > 128 && d < kPipeMaxLd : K > 64 && 2 * d < kPipeMaxLd;
}

static int assign_bn(int64_t d, hmoe_dtype_t dt, int32_t K) {
  if (K <= 64) return 64;
  return assign_pipe(d, dt, K) ? CfgPipe::BN : 128;
}

static size_t assign_ws_bytes(int64_t n, int32_t d, int32_t K, hmoe_dtype_t dt) {
  Workspace ws(nullptr, 0);
  const int nt = (int)cdiv(K, assign_bn(d, dt, K));
  ws.take<float>(K);
  if (nt > 1) {
    ws.take<float>((size_t)nt * n);
    ws.take<int32_t>((size_t)nt * n);
    ws.take<float>(n);
  }
  return ws.off;
}

template <class C>
static int assign_t(const typename C::type* X, int64_t n, int32_t d, const typename C::type* Cn, int32_t K,
                    int32_t* assign, float* min_dist, Workspace& ws, hipStream_t st, float* norms, bool normed) {
  using T = typename C::type;
  const int nt = (int)cdiv(K, C::BN);
  float* cn = norms ? norms : ws.take<float>(K);
  float *pv = nullptr, *xn = nullptr;
  int32_t* pi = nullptr;
  if (nt > 1) {
    pv = ws.take<float>((size_t)nt * n);
    pi = ws.take<int32_t>((size_t)nt * n);
    xn = ws.take<float>(n);
  }
  if (!ws.fits()) return HMOE_EWORKSPACE;
  if (!normed)
    HMOE_LAUNCH("centre norms", k_cnorm<T>, dim3((unsigned)cdiv(K, 4)), dim3(256), 0, st, Cn, K, d, cn);
  if (n == 0) return HMOE_OK;
  const int64_t tiles = cdiv(n, C::BM) * nt;
  if constexpr (C::DMA)
    HMOE_LAUNCH("assign", k_assign_dma<C>, dim3((unsigned)tiles), dim3(C::THREADS), assign_lds<C>(), st, X, n, d, Cn, K, cn,
                assign, min_dist, pv, pi, xn);
  else
    HMOE_LAUNCH("assign", k_assign<C>, dim3((unsigned)tiles), dim3(C::THREADS), C::LDS, st, X, n, d, Cn, K, cn,
                assign, min_dist, pv, pi, xn);
  if (nt > 1)
    HMOE_LAUNCH("assign merge", k_assign_merge, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, st, pv, pi, xn, n, nt,
                assign, min_dist);
  return HMOE_OK;
}

int launch_assign(const void* X, hmoe_dtype_t dt, int64_t n, int32_t d, const void* C, int32_t K, int32_t* assign,
                  float* min_dist, Workspace& ws, hipStream_t st, float* norms, bool normed) {
  const bool pipe = assign_pipe(d, dt, K);
  const bool few = cdiv(n, CfgDmaNarrow::BM) < device_cus();
  if (dt == HMOE_BF16) {
    const bf16 *x = (const bf16*)X, *c = (const bf16*)C;
    if (K <= 64 && few) return assign_t<CfgDmaNarrowFew>(x, n, d, c, K, assign, min_dist, ws, st, norms, normed);
    if (K <= 64) return assign_t<CfgDmaNarrow>(x, n, d, c, K, assign, min_dist, ws, st, norms, normed);
    if (pipe) return assign_t<CfgPipe>(x, n, d, c, K, assign, min_dist, ws, st, norms, normed);
    return assign_t<CfgSmall<bf16>>(x, n, d, c, K, assign, min_dist, ws, st, norms, normed);
  }
  const float *x = (const float*)X, *c = (const float*)C;
  if (K <= 64 && few) return assign_t<CfgDmaF32NarrowFew>(x, n, d, c, K, assign, min_dist, ws, st, norms, normed);
  if (K <= 64) return assign_t<CfgDmaF32Narrow>(x, n, d, c, K, assign, min_dist, ws, st, norms, normed);
  if (pipe) return assign_t<CfgPipeF32>(x, n, d, c, K, assign, min_dist, ws, st, norms, normed);
  return assign_t<CfgSmall<float>>(x, n, d, c, K, assign, min_dist, ws, st, norms, normed);
}

// ------------------------------------------------------------------ k-means++ seeding

constexpr int kKppRows = 256;  // rows per block of the D^2 pass

__global__ void k_kpp_first(const double* __restrict__ u, int64_t n, int32_t* __restrict__ idx) {
  if (threadIdx.x == 0) {
    int64_t f = (int64_t)floor(u[0] * (double)n);
    idx[0] = (int32_t)(f > n - 1 ? n - 1 : f);
  }
}

// |x - c|^2 in fp64 from direct differences, by the 16 lanes of a row group (16-byte loads, the
// partial sums combined in a fixed order); in every lane.
template <typename T>
__device__ __forceinline__ double kpp_dist(const T* __restrict__ x, const T* __restrict__ c, int d, int lane) {
  constexpr int EPV = 16 / sizeof(T);
  const int vpr = d / EPV;
  double s = 0.0;
  for (int v = lane; v < vpr; v += 16) {
    const i32x4 xr = *reinterpret_cast<const i32x4*>(x + v * EPV);
    const i32x4 cr = *reinterpret_cast<const i32x4*>(c + v * EPV);
    const T* xe = reinterpret_cast<const T*>(&xr);
    const T* ce = reinterpret_cast<const T*>(&cr);
#pragma unroll
    for (int z = 0; z < EPV; ++z) {
      const double df = (double)to_f32(xe[z]) - (double)to_f32(ce[z]);
      s += df * df;
    }
  }
  return row_sum_up(s);
}

// bsum[block] = sum of the block's D2 in row order, split over the first wave: lane l adds rows
// 4l..4l+3, then the lanes are combined by the wave's fixed butterfly.
__device__ __forceinline__ void kpp_block_sum(const double* rowv, double* __restrict__ bsum) {
  if (threadIdx.x < 64) {
    double s = ((rowv[4 * threadIdx.x] + rowv[4 * threadIdx.x + 1]) + rowv[4 * threadIdx.x + 2]) +
               rowv[4 * threadIdx.x + 3];
    s = wave_sum(s);
    if (threadIdx.x == 0) bsum[blockIdx.x] = s;
  }
}

// The D^2 pass over an 8-bit copy of the rows.  A pass over X for each centre is bound by reading X
// (2^20 x 512 fp32 rows: 366 us at 5.9 TB/s), yet a new centre changes the D^2 of few rows.  So
// the first pass also writes each row as x = s q + r with integers |q| <= 127 and e >= |r|, and a
// later pass reads q instead of x: |x - c| >= |s q - s' q'| - e - e' (the triangle inequality; q . q'
// is exact in integers), and a row whose bound lies above its D^2 keeps it.  Only the other rows
// are read in full and measured as k_kpp_update does, so every D^2, and with it every pick, is the
// same to the last bit: the margins below cover the rounding of the bound and of the distance.
// Rows with entries that are not finite, or too large or small to square, have e = inf: they are
// always measured.
// 2^20 x 512 fp32, 64 centres: 23.4 ms -> 8.5 (118 us a pass, 1.06 ms for the first, which also writes
// the copy).
// Rows with a few entries far above the rest keep little of the others in 8 bits: e is of the order of the
// distances, the bounds rule out nothing, and a pass that reads the copy and then X took 30% longer than
// X alone (the same rows with one column at 300: 33.1 ms, 25.5 without a copy).  So a block of rows
// is sifted only while that pays: it makes no copy (all e = inf but the first centre's) when most of its
// first 16 rows have e > |x - c| / 8 against the first centre c, and after two passes in a row (the
// third and later) in which the copy left too many of its rows, it skips 2, 4, ... 32 before it tries again.
// (33.1 -> 24.1 ms there; mixtures and i.i.d. rows take the same as with the copy throughout.)
struct KppMeta {
  float s, e;    // scale; upper bound of |x - s q|
  int32_t qq;    // |q|^2
  int32_t wait;  // of a block's first row: 8 (first pass that is sifted) + passes in vain before it, up to 6
};
constexpr int32_t kKppNever = INT32_MAX;
static_assert(sizeof(KppMeta) == 16, "one 16-byte load");

__host__ __device__ __forceinline__ int64_t kpp_row_bytes(int d) { return (int64_t)((d + 15) & ~15); }

// Sum over the 16 lanes of a row group, in every lane of it.
__device__ __forceinline__ int row16_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x128, 0xf, 0xf, true);  // row_ror:8, 4, 2, 1
  v += __builtin_amdgcn_update_dpp(0, v, 0x124, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x122, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x121, 0xf, 0xf, true);
  return v;
}

// Row i's 8-bit copy; 16 lanes of a wave share the row, lane taking vectors lane, lane + 16, ...
// of 16 entries (absent ones 0, up to the padded row).  Returns e.
template <typename T>
__device__ __forceinline__ float kpp_quantise(const T* __restrict__ x, int64_t i, int d, int lane,
                                             int8_t* __restrict__ Xq, KppMeta* __restrict__ meta) {
  constexpr int EPV = 16 / sizeof(T);
  constexpr int PER = 16 / EPV;  // source vectors per destination vector
  const int vpr = d / EPV;
  float amax = 0.f;
  bool finite = true;
  for (int v = lane; v < vpr; v += 16) {
    const i32x4 raw = *reinterpret_cast<const i32x4*>(x + v * EPV);
    const T* e = reinterpret_cast<const T*>(&raw);
#pragma unroll
    for (int z = 0; z < EPV; ++z) {
      const float a = fabsf(to_f32(e[z]));
      finite = finite && a <= 1e15f;  // false for NaN
      amax = fmaxf(amax, a);
    }
  }
#pragma unroll
  for (int m = 1; m < 16; m <<= 1) amax = fmaxf(amax, shfl_xor(amax, m));
  const uint64_t bad = __ballot(!finite) >> (threadIdx.x & 48) & 0xffff;
  const bool ok = bad == 0 && (amax >= 1e-15f || amax == 0.f);
  const float s = ok ? amax * (1.f / 127.f) : 0.f;
  const float inv = ok && amax > 0.f ? 127.f / amax : 0.f;
  const int qv = (int)(kpp_row_bytes(d) / 16);
  int qq = 0;
  double r2 = 0.0;
  for (int v = lane; v < qv; v += 16) {
    i32x4 out = i32x4{0, 0, 0, 0};
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      if (!ok || v * PER + p >= vpr) continue;
      const i32x4 raw = *reinterpret_cast<const i32x4*>(x + (v * PER + p) * EPV);
      const T* e = reinterpret_cast<const T*>(&raw);
#pragma unroll
      for (int z = 0; z < EPV; ++z) {
        const float f = to_f32(e[z]);
        int q = (int)rintf(f * inv);
        q = q > 127 ? 127 : (q < -127 ? -127 : q);
        qq += q * q;
        const double r = (double)f - (double)s * (double)q;
        r2 += r * r;
        const int at = p * EPV + z;
        out[at / 4] |= (q & 255) << (8 * (at % 4));
      }
    }
    *reinterpret_cast<i32x4*>(Xq + i * kpp_row_bytes(d) + v * 16) = out;
  }
#pragma unroll
  for (int m = 1; m < 16; m <<= 1) r2 += shfl_xor(r2, m);
  qq = row16_sum(qq);
  const float e = ok ? (float)(sqrt(r2) * (1.0 + 1e-6)) : INFINITY;
  if (lane == 0) meta[i] = KppMeta{s, e, qq, 0};
  return e;
}

// A lower bound of the distance of two rows by their copies, P = q . q'; negative, infinite or NaN
// where there is none.
__device__ __forceinline__ double kpp_bound(const KppMeta& x, const KppMeta& c, int P) {
  const double sx = x.s, sc = c.s;
  const double xx = sx * sx * (double)x.qq, cc = sc * sc * (double)c.qq;
  const double d2 = xx + cc - 2.0 * (sx * sc * (double)P) - 1e-12 * (xx + cc);
  return (double)sqrtf((float)fmax(d2, 0.0)) * (1.0 - 1e-6) - (double)x.e - (double)c.e;
}
// Whether a distance of at least lb has a square above D2 (false for a bound that is none).
__device__ __forceinline__ bool kpp_far(double lb, double D2) { return lb > 1e-12 && lb * lb * (1.0 - 1e-6) > D2; }

// D2[i] = min(D2[i], |x_i - X[idx[t]]|^2) (fp64 direct differences; t == 0 initialises) and
// bsum[b] = sum of D2 over the block's kKppRows rows, in a fixed order.  16 lanes share a row, so
// each wave streams 4 rows at once.  QUANT: also writes the rows' 8-bit copies.  THREADS: 256, or
// 1024 where there are fewer blocks than CUs and a block's rows are a chain of memory latencies
// (4096 x 64: 11 us, 4).
template <typename T, bool QUANT, int THREADS>
__global__ void __launch_bounds__(THREADS) k_kpp_update(const T* __restrict__ X, int64_t n, int d,
                                                    const int32_t* __restrict__ idx, int t,
                                                    double* __restrict__ D2, double* __restrict__ bsum,
                                                    int8_t* __restrict__ Xq, KppMeta* __restrict__ meta,
                                                    int32_t* __restrict__ near) {
  __shared__ double rowv[kKppRows];
  __shared__ int poor;  // rows among the first 16 whose copy is of no use
  const int lane = threadIdx.x & 15;        // position inside the row group
  const int grp = threadIdx.x >> 4;         // row groups per block
  const T* c = X + (int64_t)idx[t] * d;
  const int64_t r0 = (int64_t)blockIdx.x * kKppRows;
  bool copies = true;
  if constexpr (QUANT) {
    if (threadIdx.x == 0) poor = 0;
    __syncthreads();
  }
#pragma unroll(QUANT ? 1 : 2)
  for (int q = 0; q < kKppRows / (THREADS / 16); ++q) {
    const int lr = q * (THREADS / 16) + grp;
    const int64_t i = r0 + lr;
    double s = 0.0;
    if (i < n) {
      s = kpp_dist(X + i * d, c, d, lane);
      if constexpr (QUANT) {
        if (copies || i == idx[t]) {
          const float e = kpp_quantise(X + i * d, i, d, lane, Xq, meta);
          if (q == 0 && lane == 0 && !(64.0 * (double)e * (double)e <= s)) atomicAdd(&poor, 1);
        } else if (lane == 0) {
          meta[i] = KppMeta{0.f, INFINITY, 0, 0};
        }
      }
    }
    if constexpr (QUANT) {
      if (q == 0) {
        __syncthreads();
        const int rows = n - r0 < THREADS / 16 ? (int)(n - r0) : THREADS / 16;
        copies = 4 * poor < 3 * rows;
      }
    }
    if (lane == 0) {
      double v = 0.0;
      if (i < n) {
        v = s;
        if (t > 0) {
          const double old = D2[i];
          v = old < s ? old : s;
        }
        D2[i] = v;
        if constexpr (QUANT) near[i] = 0;
      }
      rowv[lr] = v;
    }
  }
  if constexpr (QUANT) {
    if (threadIdx.x == 0 && !copies) meta[r0].wait = kKppNever;  // the thread that wrote meta[r0]
  }
  __syncthreads();
  kpp_block_sum(rowv, bsum);
}

// cc[s] = lower bound of the distance of centres t and s < t, by 64 groups of 16 lanes.
__device__ __forceinline__ void kpp_centre_bounds(const int8_t* __restrict__ Xq, const KppMeta* __restrict__ meta,
                                                  const int32_t* __restrict__ idx, int64_t ct, int t, int d,
                                                  float* __restrict__ cc) {
  const int lane = threadIdx.x & 15;
  const int64_t rb = kpp_row_bytes(d);
  for (int s = threadIdx.x >> 4; s < t; s += 64) {
    const int64_t c = idx[s];
    int P = 0;
    for (int v = lane; v < rb / 16; v += 16) {
      const i32x4 x = *reinterpret_cast<const i32x4*>(Xq + c * rb + v * 16);
      const i32x4 y = *reinterpret_cast<const i32x4*>(Xq + ct * rb + v * 16);
#pragma unroll
      for (int z = 0; z < 4; ++z) P = __builtin_amdgcn_sdot4(x[z], y[z], P, false);
    }
    P = row16_sum(P);
    if (lane == 0) cc[s] = (float)(kpp_bound(meta[c], meta[ct], P) * (1.0 - 1e-6));
  }
}

// Pass t > 0 over the copy.  A row whose nearest centre so far (near) is at least twice as far from
// the new one as from the row keeps its D^2 without a look at it; the block's other rows are
// sifted by the copy, four at a time by each group of 16 lanes, unless the block waits or the centre
// has no copy, and those that remain are measured by all groups.  The copy has paid when it left at most
// the share of the rows read whose bytes it saved: 3/4 of fp32 rows, 1/2 of bf16 rows.
template <typename T>
__global__ void __launch_bounds__(256) k_kpp_sift(const T* __restrict__ X, const int8_t* __restrict__ Xq,
                                                  KppMeta* __restrict__ meta, const float* __restrict__ cc,
                                                  int64_t n, int d, const int32_t* __restrict__ idx, int t,
                                                  double* __restrict__ D2, int32_t* __restrict__ near,
                                                  double* __restrict__ bsum) {
  constexpr int U = 4;
  __shared__ double rowv[kKppRows];
  __shared__ int32_t list[2][kKppRows];
  __shared__ int32_t left[2];
  if (threadIdx.x < 2) left[threadIdx.x] = 0;
  __syncthreads();
  const int lane = threadIdx.x & 15, grp = threadIdx.x >> 4;
  const int64_t r0 = (int64_t)blockIdx.x * kKppRows;
  const int64_t ci = idx[t];
  static_assert(kKppRows == 256, "a thread per row");
  double old = 0.0;  // past the last row
  if (r0 + threadIdx.x < n) {
    old = D2[r0 + threadIdx.x];
    if (!kpp_far(cc[near[r0 + threadIdx.x]], 4.0 * old)) list[0][atomicAdd(&left[0], 1)] = threadIdx.x;
  }
  rowv[threadIdx.x] = old;
  __syncthreads();
  const int todo = left[0];
  const KppMeta cm = meta[ci];
  const int32_t wait = meta[r0].wait;
  const bool sift = t >= wait / 8 && cm.e < INFINITY;
  const int64_t rb = kpp_row_bytes(d);
  const int qv = (int)(rb / 16);
  const int8_t* cq = Xq + ci * rb;
  for (int q = 0; sift && q < todo; q += 16 * U) {
    const int own = q + (lane & (U - 1)) * 16 + grp;  // the entry this lane decides on
    const int mine = list[0][own < todo ? own : 0];
    const KppMeta xm = meta[r0 + mine];
    int acc[U] = {0, 0, 0, 0};
    const int8_t* x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int at = q + u * 16 + grp;
      x[u] = Xq + (r0 + list[0][at < todo ? at : 0]) * rb;
    }
    for (int v = lane; v < qv; v += 16) {
      const i32x4 c = *reinterpret_cast<const i32x4*>(cq + v * 16);
      i32x4 xv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) xv[u] = *reinterpret_cast<const i32x4*>(x[u] + v * 16);
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int z = 0; z < 4; ++z) acc[u] = __builtin_amdgcn_sdot4(xv[u][z], c[z], acc[u], false);
    }
    int P = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int a = row16_sum(acc[u]);
      P = (lane & (U - 1)) == u ? a : P;
    }
    if (lane < U && own < todo && !kpp_far(kpp_bound(xm, cm, P), rowv[mine])) list[1][atomicAdd(&left[1], 1)] = mine;
  }
  __syncthreads();
  const int cnt = sift ? left[1] : todo;
  const int32_t* rows = list[sift ? 1 : 0];
  if (threadIdx.x == 0 && sift && todo >= 64) {
    const bool vain = t > 2 && cnt * (int)sizeof(T) > todo * ((int)sizeof(T) - 1);
    const int32_t tries = !vain ? 0 : (wait % 8 < 6 ? wait % 8 + 1 : 6);
    const int32_t next = (t + (tries < 2 ? 1 : 1 + (1 << (tries - 1)))) * 8 + tries;
    if (vain || wait % 8 != 0) meta[r0].wait = next;
  }
  const T* c = X + ci * d;
  for (int q = grp; q < cnt; q += 16) {
    const int lr = rows[q];
    const double s = kpp_dist(X + (r0 + lr) * d, c, d, lane);
    if (lane == 0) {
      const double v = rowv[lr];
      if (!(v < s)) {  // as min(): a NaN takes its place, too
        D2[r0 + lr] = s;
        near[r0 + lr] = t;
        rowv[lr] = s;
      }
    }
  }
  __syncthreads();
  kpp_block_sum(rowv, bsum);
}

// Picks centre t: the first row whose running D^2 sum exceeds u[t] * total (lowest unchosen row
// if the total is zero).  With the 8-bit copy, also bounds the centre's distances to the earlier ones
// (cc).  One block of 1024 threads.
__global__ void __launch_bounds__(1024) k_kpp_select(const double* __restrict__ D2, int64_t n,
                                                     const double* __restrict__ bsum, int nb,
                                                     const double* __restrict__ u, int t,
                                                     int32_t* __restrict__ idx, const int8_t* __restrict__ Xq,
                                                     const KppMeta* __restrict__ meta, int d,
                                                     float* __restrict__ cc) {
  __shared__ double sh[17], rowd[kKppRows], before;
  __shared__ int32_t pick;
  __shared__ int who, block;
  const int per = (nb + 1023) / 1024;
  const int b0 = threadIdx.x * per;
  double s = 0.0;
  for (int q = 0; q < per; ++q)
    if (b0 + q < nb) s += bsum[b0 + q];
  double S;
  const double ex = block_excl_scan<double>(s, sh, &S);
  if (threadIdx.x == 0) pick = -1;
  __syncthreads();
  if (S > 0.0) {
    const double target = u[t] * S;
    // the first thread whose run of blocks crosses the target finds the block, all threads fetch
    // its rows, and one walks them in order (a trip to memory for each row took 20 us, now 7)
    if (threadIdx.x == 0) who = INT_MAX;
    __syncthreads();
    if (ex <= target && target < ex + s) atomicMin(&who, (int)threadIdx.x);
    __syncthreads();
    if ((int)threadIdx.x == who) {
      double P = ex;
      int b = b0;
      while (b + 1 < nb && b + 1 < b0 + per && P + bsum[b] <= target) P += bsum[b++];
      block = b;
      before = P;
    }
    __syncthreads();
    if (who != INT_MAX) {
      const int64_t first = (int64_t)block * kKppRows;
      if (threadIdx.x < kKppRows) rowd[threadIdx.x] = first + threadIdx.x < n ? D2[first + threadIdx.x] : 0.0;
      __syncthreads();
      if (threadIdx.x == 0) {
        double P = before;
        int found = -1;
        for (int i = 0; i < kKppRows && found < 0; i += 8) {
          double v[8];
#pragma unroll
          for (int z = 0; z < 8; ++z) v[z] = rowd[i + z];
#pragma unroll
          for (int z = 0; z < 8; ++z) {
            P += v[z];
            if (found < 0 && P > target) found = i + z;
          }
        }
        // rounding left the crossing just past this block: take its last row with D2 > 0
        for (int i = kKppRows - 1; i >= 0 && found < 0; --i)
          if (rowd[i] > 0.0) found = i;
        if (found >= 0) pick = (int32_t)(first + found);
      }
    }
    __syncthreads();
    if (threadIdx.x == 0 && pick < 0) {  // target beyond the rounded total: last row with D2 > 0
      for (int64_t i = n - 1; i >= 0; --i)
        if (D2[i] > 0.0) { pick = (int32_t)i; break; }
    }
    __syncthreads();
  }
  if (pick < 0) {
    // every D^2 is zero: the lowest row not chosen yet (one of 0..t)
    __shared__ int32_t low;
    if (threadIdx.x == 0) low = INT_MAX;
    __syncthreads();
    for (int i = threadIdx.x; i <= t; i += 1024) {
      bool used = false;
      for (int q = 0; q < t; ++q) used |= (idx[q] == i);
      if (!used) atomicMin(&low, i);
    }
    __syncthreads();
    if (threadIdx.x == 0) pick = low;
    __syncthreads();
  }
  if (threadIdx.x == 0) idx[t] = pick;
  if (Xq) kpp_centre_bounds(Xq, meta, idx, pick, t, d, cc);
}

// C[k][:] = X[idx[k]][:] as fp32, and Cd (the data-precision copy) when given.
template <typename T>
__global__ void __launch_bounds__(256) k_gather_centres(const T* __restrict__ X, int d,
                                                        const int32_t* __restrict__ idx, int K,
                                                        float* __restrict__ C, T* __restrict__ Cd) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= (int64_t)K * d) return;
  const int k = (int)(q / d), j = (int)(q % d);
  const T v = X[(int64_t)idx[k] * d + j];
  C[q] = to_f32(v);
  if (Cd) Cd[q] = v;
}

// ------------------------------------------------------------------ Lloyd update

// The farthest-row search of the first reseed, spread over the grid: block b takes rows
// [b chunk, (b + 1) chunk) and writes its largest min_dist among rows whose cluster has more
// than one member (lowest index on ties; -1 / INT64_MAX when it has none) to pv[b], pi[b].
// Every block returns at once when no cluster is empty.
constexpr int kReseedBlocks = 512;

__global__ void __launch_bounds__(1024) k_reseed_scan(const int32_t* __restrict__ assign,
                                                      const float* __restrict__ d1, int64_t n, int K,
                                                      const int32_t* __restrict__ counts32, float* __restrict__ pv,
                                                      int64_t* __restrict__ pi) {
  __shared__ int any_empty;
  __shared__ float bv[16];
  __shared__ int64_t bix[16];
  if (threadIdx.x == 0) any_empty = 0;
  __syncthreads();
  for (int k = threadIdx.x; k < K; k += 1024)
    if (counts32[k] == 0) any_empty = 1;
  __syncthreads();
  if (!any_empty) return;
  const int64_t chunk = cdiv(n, (int64_t)gridDim.x);
  const int64_t i0 = (int64_t)blockIdx.x * chunk;
  const int64_t i1 = i0 + chunk < n ? i0 + chunk : n;
  float best = -1.f;
  int64_t bi = INT64_MAX;
  for (int64_t i = i0 + threadIdx.x; i < i1; i += 1024) {
    const int32_t a = assign[i];
    if ((unsigned)a >= (unsigned)K || counts32[a] <= 1) continue;  // out-of-range ids are never donors
    const float v = d1[i];
    if (v > best || (v == best && i < bi)) {
      best = v;
      bi = i;
    }
  }
  for (int m = 1; m < 64; m <<= 1) {
    const float v2 = __shfl_xor(best, m, 64);
    const int64_t i2 = __shfl_xor(bi, m, 64);
    if (v2 > best || (v2 == best && i2 < bi)) {
      best = v2;
      bi = i2;
    }
  }
  if ((threadIdx.x & 63) == 0) {
    bv[threadIdx.x >> 6] = best;
    bix[threadIdx.x >> 6] = bi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 16; ++w)
      if (bv[w] > best || (bv[w] == best && bix[w] < bi)) {
        best = bv[w];
        bi = bix[w];
      }
    pv[blockIdx.x] = best;
    pi[blockIdx.x] = bi;
  }
}

// Loads counts into shared memory, reseeds empty clusters (ascending ids; each takes the
// farthest row -- largest min_dist, lowest index on ties -- whose cluster has more than one
// member, moves it and its vector between the fp64 sums), then writes counts back.  The first
// reseed takes its row from the np partials of k_reseed_scan (the same counts and assignment,
// so the same row); later ones scan the rows here.  One block of 1024 threads; K <= 4096.
template <typename T>
__global__ void __launch_bounds__(1024) k_reseed(const T* __restrict__ X, int64_t n, int d, int K,
                                                 int32_t* __restrict__ assign, const float* __restrict__ d1,
                                                 int32_t* __restrict__ counts32, int64_t* __restrict__ counts64,
                                                 double* __restrict__ sums, int reseed, const float* __restrict__ pv,
                                                 const int64_t* __restrict__ pi, int np) {
  __shared__ int32_t cnt[4096];
  __shared__ float bv[16];
  __shared__ int64_t bix[16];
  __shared__ int64_t chosen;
  for (int k = threadIdx.x; k < K; k += 1024) cnt[k] = counts32[k];
  __syncthreads();
  if (reseed && n > 0) {
    bool first = true;
    for (int k = 0; k < K; ++k) {
      if (cnt[k] != 0) continue;
      float best = -1.f;
      int64_t bi = INT64_MAX;
      if (first && np > 0) {
        for (int q = threadIdx.x; q < np; q += 1024) {
          const float v = pv[q];
          const int64_t i = pi[q];
          if (v > best || (v == best && i < bi)) {
            best = v;
            bi = i;
          }
        }
      } else {
        for (int64_t i = threadIdx.x; i < n; i += 1024) {
          const int32_t a = __hip_atomic_load(assign + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if ((unsigned)a >= (unsigned)K || cnt[a] <= 1) continue;
          const float v = d1[i];
          if (v > best || (v == best && i < bi)) {
            best = v;
            bi = i;
          }
        }
      }
      first = false;
      for (int m = 1; m < 64; m <<= 1) {
        const float v2 = __shfl_xor(best, m, 64);
        const int64_t i2 = __shfl_xor(bi, m, 64);
        if (v2 > best || (v2 == best && i2 < bi)) {
          best = v2;
          bi = i2;
        }
      }
      if ((threadIdx.x & 63) == 0) {
        bv[threadIdx.x >> 6] = best;
        bix[threadIdx.x >> 6] = bi;
      }
      __syncthreads();
      if (threadIdx.x == 0) {
        float b = bv[0];
        int64_t c = bix[0];
        for (int w = 1; w < 16; ++w)
          if (bv[w] > b || (bv[w] == b && bix[w] < c)) {
            b = bv[w];
            c = bix[w];
          }
        chosen = (c == INT64_MAX) ? -1 : c;
      }
      __syncthreads();
      const int64_t i = chosen;
      if (i < 0) break;  // no donor left; eligibility only shrinks, so later empties stay empty
      const int32_t donor = __hip_atomic_load(assign + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      for (int j = threadIdx.x; j < d; j += 1024) {
        const double x = (double)to_f32(X[i * d + j]);
        sums[(int64_t)donor * d + j] -= x;
        sums[(int64_t)k * d + j] = x;
      }
      __syncthreads();
      if (threadIdx.x == 0) {
        cnt[donor] -= 1;
        cnt[k] = 1;
        __hip_atomic_store(assign + i, k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      __syncthreads();
    }
  }
  for (int k = threadIdx.x; k < K; k += 1024) {
    counts32[k] = cnt[k];
    if (counts64) counts64[k] = cnt[k];
  }
}

__global__ void __launch_bounds__(256) k_add_counts(const int32_t* __restrict__ c32, int K, int64_t* __restrict__ c64) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k < K) c64[k] += c32[k];
}

// Cd = C rounded to the data precision.
template <typename T>
__global__ void __launch_bounds__(256) k_convert_centres(const float* __restrict__ C, int64_t count,
                                                         T* __restrict__ Cd) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q < count) Cd[q] = from_f32<T>(C[q]);
}

// C = sums / counts for non-empty clusters (others keep C); Cd = data-precision copy of C.
template <typename T, typename CNT>
__global__ void __launch_bounds__(256) k_finalize(const double* __restrict__ sums, const CNT* __restrict__ counts,
                                                  int K, int d, float* __restrict__ C, T* __restrict__ Cd) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= (int64_t)K * d) return;
  const int k = (int)(q / d);
  float c = C[q];
  if (counts[k] > 0) c = (float)(sums[q] / (double)counts[k]);
  C[q] = c;
  if (Cd) Cd[q] = from_f32<T>(c);
}

// The same for a fit's next assignment, with the centres' norms (of the data-precision copy, in
// k_cnorm's order): one wave per centre.
template <typename T>
__global__ void __launch_bounds__(256) k_finalize_norm(const double* __restrict__ sums,
                                                       const int64_t* __restrict__ counts, int K, int d,
                                                       float* __restrict__ C, T* __restrict__ Cd,
                                                       float* __restrict__ cn) {
  const int k = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int l = threadIdx.x & 63;
  if (k >= K) return;
  const int64_t cnt = counts[k];
  float s = 0.f;
#pragma unroll 4
  for (int j = l; j < d; j += 64) {
    const int64_t q = (int64_t)k * d + j;
    float c = C[q];
    if (cnt > 0) c = (float)(sums[q] / (double)cnt);
    C[q] = c;
    const T lo = from_f32<T>(c);
    if (Cd) Cd[q] = lo;
    const float f = to_f32(lo);
    s += f * f;
  }
  s = wave_sum(s);
  if (l == 0) cn[k] = s;
}

// ------------------------------------------------------------------ fit / update drivers

struct UpdateBufs {
  int32_t *counts32, *offsets, *perm, *inv, *pieces;
};

// Rows above which the reseeding's first search runs over the grid: one workgroup looks through
// fewer in less than that launch takes, and only when a cluster is empty.
constexpr int64_t kReseedGrid = 16384;

template <typename T>
static int update_core(const T* X, int64_t n, int32_t d, int32_t K, int32_t* assign, const float* d1,
                       double* sums, int64_t* counts64, int accumulate, int reseed, const UpdateBufs& b,
                       Workspace& ws, hipStream_t st) {
  HMOE_TRY(launch_dispatch(assign, n, K, b.counts32, b.offsets, b.perm, b.inv, ws, st, b.pieces));
  HMOE_TRY(launch_segsum<T, double>(X, d, b.perm, b.offsets, K, d, n, sums, accumulate, ws, st, b.pieces));
  if (accumulate) {
    HMOE_LAUNCH("add counts", k_add_counts, dim3((unsigned)cdiv(K, 256)), dim3(256), 0, st, b.counts32, K, counts64);
    return HMOE_OK;
  }
  float* pv = nullptr;
  int64_t* pi = nullptr;
  int np = 0;
  if (reseed && n > kReseedGrid) {
    np = (int)(cdiv(n, (int64_t)4096) < kReseedBlocks ? cdiv(n, (int64_t)4096) : kReseedBlocks);
    pv = ws.take<float>(np);
    pi = ws.take<int64_t>(np);
    if (!ws.fits()) return HMOE_EWORKSPACE;
    HMOE_LAUNCH("reseed scan", k_reseed_scan, dim3((unsigned)np), dim3(1024), 0, st, (const int32_t*)assign, d1, n, K,
                (const int32_t*)b.counts32, pv, pi);
  }
  HMOE_LAUNCH("reseed", k_reseed<T>, dim3(1), dim3(1024), 0, st, X, n, d, K, assign, d1, b.counts32, counts64, sums,
                     reseed, (const float*)pv, (const int64_t*)pi, np);
  return HMOE_OK;
}

static size_t update_scratch(int64_t n, int32_t d, int32_t K) {
  Workspace ws(nullptr, 0);
  ws.take<int32_t>(K);
  ws.take<int32_t>(K + 1);
  ws.take<int32_t>(n);
  ws.take<int32_t>(n);
  // the pieces' table, which the sort leaves, is the one that the segmented sums have room for
  size_t s = ws.off + dispatch_ws(n, K) + segsum_ws(n, K, d) +
             (size_t)kReseedBlocks * (sizeof(float) + sizeof(int64_t)) + 4096;
  return s;
}

template <typename T>
static int update_t(const T* X, int64_t n, int32_t d, int32_t K, int32_t* assign, const float* d1, double* sums,
                    int64_t* counts64, float* C, int32_t mode, int32_t reseed, Workspace& ws, hipStream_t st) {
  UpdateBufs b;
  b.counts32 = ws.take<int32_t>(K);
  b.offsets = ws.take<int32_t>(K + 1);
  b.pieces = ws.take<int32_t>(K + 1);
  b.perm = ws.take<int32_t>(n);
  b.inv = ws.take<int32_t>(n);
  if (!ws.fits()) return HMOE_EWORKSPACE;
  if (mode != HMOE_UPDATE_FINALIZE) {
    HMOE_TRY(update_core<T>(X, n, d, K, assign, d1, sums, counts64, mode == HMOE_UPDATE_ACCUMULATE,
                            mode == HMOE_UPDATE_FULL ? reseed : 0, b, ws, st));
  }
  if (mode != HMOE_UPDATE_ACCUMULATE) {
    HMOE_LAUNCH("finalize centres", (k_finalize<T, int64_t>), dim3((unsigned)cdiv((int64_t)K * d, 256)), dim3(256), 0, st, sums,
                       counts64, K, d, C, (T*)nullptr);
  }
  return HMOE_OK;
}

int launch_update(const void* X, hmoe_dtype_t dt, int64_t n, int32_t d, int32_t K, int32_t* assign,
                  const float* min_dist, double* sums, int64_t* counts, float* C, int32_t mode, int32_t reseed,
                  Workspace& ws, hipStream_t st) {
  if (dt == HMOE_BF16)
    return update_t<bf16>((const bf16*)X, n, d, K, assign, min_dist, sums, counts, C, mode, reseed, ws, st);
  return update_t<float>((const float*)X, n, d, K, assign, min_dist, sums, counts, C, mode, reseed, ws, st);
}

size_t update_ws_bytes(int64_t n, int32_t d, int32_t K) { return update_scratch(n, d, K); }

// The seeding's 8-bit copy pays where a pass over X is a trip to memory, and over enough passes to earn
// its first one.  Seeding with the copy and without: 32 MB (90,000 x 96 fp32) 16 centres 347 / 450 us,
// 16 MB 301 / 230, 8 MB 299 / 231; 2 GB (2^20 x 512) 64 centres 9.9 / 24.7 ms, 16 centres 5.0 / 6.7,
// 8 centres 3.8 / 3.6.  Wider rows than kKppMaxWidth would overflow the integer sums.
constexpr int32_t kKppMaxWidth = INT32_MAX / (127 * 127);  // 133,144
static bool kpp_copies(int64_t n, int32_t d, int32_t K, hmoe_dtype_t dt) {
  return K >= 16 && d <= kKppMaxWidth && n * d * (int64_t)dtype_size(dt) >= (int64_t(32) << 20);
}

// What a fit needs, and the 8-bit copy on top of it (a fit in a smaller workspace goes without).
size_t fit_ws_copy_bytes(int64_t n, int32_t d, int32_t K, hmoe_dtype_t dt) {
  return kpp_copies(n, d, K, dt) ? (size_t)n * (kpp_row_bytes(d) + sizeof(KppMeta) + 4) + 4 * (size_t)K + 1024 : 0;
}

size_t fit_ws_bytes(int64_t n, int32_t d, int32_t K, hmoe_dtype_t dt) {
  Workspace ws(nullptr, 0);
  ws.take<double>((size_t)K * d);           // sums
  ws.take<int64_t>(K);                      // counts64
  ws.take<char>((size_t)K * d * dtype_size(dt));  // data-precision centres
  ws.take<float>(n);                        // min distances when the caller passes none
  ws.take<double>(n);                       // D^2 for k-means++
  ws.take<double>(cdiv(n, kKppRows));       // block sums
  ws.take<int32_t>(K);                      // picks when the caller passes none
  size_t s = ws.off + update_scratch(n, d, K) + assign_ws_bytes(n, d, K, dt) + 4096;  // centre norms: the assignment's
  return s;
}

size_t assign_ws(int64_t n, int32_t d, int32_t K, hmoe_dtype_t dt) { return assign_ws_bytes(n, d, K, dt) + 256; }

template <typename T>
static int fit_t(const T* X, int64_t n, int32_t d, int32_t K, int32_t n_iter, const double* u, int32_t reseed,
                 float* C, int32_t* assign, float* min_dist, int32_t* counts, double* objective, int32_t* init_idx,
                 Workspace& ws, hipStream_t st) {
  double* sums = ws.take<double>((size_t)K * d);
  int64_t* c64 = ws.take<int64_t>(K);
  T* Cd = reinterpret_cast<T*>(ws.take<char>((size_t)K * d * sizeof(T)));
  float* d1 = min_dist ? min_dist : ws.take<float>(n);
  double* D2 = ws.take<double>(n);
  const int nb = (int)cdiv(n, kKppRows);
  double* bsum = ws.take<double>(nb);
  int32_t* idx = init_idx ? init_idx : ws.take<int32_t>(K);
  if (!ws.fits()) return HMOE_EWORKSPACE;
  const int64_t Kd = (int64_t)K * d;
  const bool same = sizeof(T) == sizeof(float);  // fp32 data assigns against C itself
  const T* Cuse = same ? reinterpret_cast<const T*>(C) : Cd;
  if (u) {
    // the copy lies past everything else in the workspace
    int8_t* Xq = nullptr;
    KppMeta* meta = nullptr;
    int32_t* near = nullptr;
    float* cc = nullptr;
    if (fit_ws_copy_bytes(n, d, K, DT<T>::id) > 0) {
      Workspace w(ws.base, ws.cap);
      w.off = fit_ws_bytes(n, d, K, DT<T>::id);
      Xq = w.take<int8_t>((size_t)n * kpp_row_bytes(d));
      meta = w.take<KppMeta>(n);
      near = w.take<int32_t>(n);
      cc = w.take<float>(K);
      if (!w.fits()) Xq = nullptr;
    }
    HMOE_LAUNCH("kmeans++ first", k_kpp_first, dim3(1), dim3(64), 0, st, u, n, idx);
    for (int t = 0; t < K; ++t) {
      if (Xq && t == 0)
        HMOE_LAUNCH("kmeans++ D2", (k_kpp_update<T, true, 256>), dim3((unsigned)nb), dim3(256), 0, st, X, n, d, idx, t, D2,
                    bsum, Xq, meta, near);
      else if (Xq)
        HMOE_LAUNCH("kmeans++ D2", k_kpp_sift<T>, dim3((unsigned)nb), dim3(256), 0, st, X, (const int8_t*)Xq,
                    meta, (const float*)cc, n, d, idx, t, D2, near, bsum);
      else {
        const bool few = nb < device_cus();
        const auto update = few ? k_kpp_update<T, false, 1024> : k_kpp_update<T, false, 256>;
        HMOE_LAUNCH("kmeans++ D2", update, dim3((unsigned)nb), dim3(few ? 1024 : 256), 0, st, X, n, d, idx, t, D2, bsum,
                    (int8_t*)nullptr, (KppMeta*)nullptr, (int32_t*)nullptr);
      }
      if (t + 1 < K) {
        HMOE_LAUNCH("kmeans++ select", k_kpp_select, dim3(1), dim3(1024), 0, st, D2, n, bsum, nb, u, t + 1, idx,
                    (const int8_t*)Xq, (const KppMeta*)meta, d, cc);
      }
    }
    HMOE_LAUNCH("gather centres", k_gather_centres<T>, dim3((unsigned)cdiv(Kd, 256)), dim3(256), 0, st, X, d, idx, K, C,
                       same ? (T*)nullptr : Cd);
  }
  if (!u && !same) {
    // data-precision copy of the given centres
    HMOE_LAUNCH("convert centres", (k_convert_centres<T>), dim3((unsigned)cdiv(Kd, 256)), dim3(256), 0, st, C, Kd, Cd);
  }
  UpdateBufs b;
  Workspace* wsp = &ws;
  b.counts32 = wsp->take<int32_t>(K);
  b.offsets = wsp->take<int32_t>(K + 1);
  b.pieces = wsp->take<int32_t>(K + 1);
  b.perm = wsp->take<int32_t>(n);
  b.inv = wsp->take<int32_t>(n);
  if (!ws.fits()) return HMOE_EWORKSPACE;
  float* norms = ws.take<float>(K);
  const size_t mark = ws.off;
  for (int t = 0; t <= n_iter; ++t) {
    ws.off = mark;
    HMOE_TRY(launch_assign(X, DT<T>::id, n, d, Cuse, K, assign, d1, ws, st, norms, t > 0));
    if (objective) HMOE_TRY(launch_sum_f32(d1, n, 1.0, objective + t, nullptr, ws, st));
    if (t == n_iter) break;
    HMOE_TRY(update_core<T>(X, n, d, K, assign, d1, sums, c64, 0, reseed, b, ws, st));
    HMOE_LAUNCH("finalize centres", k_finalize_norm<T>, dim3((unsigned)cdiv(K, 4)), dim3(256), 0, st,
                (const double*)sums, (const int64_t*)c64, K, d, C, same ? (T*)nullptr : Cd, norms);
  }
  if (counts) {
    ws.off = mark;
    HMOE_TRY(launch_dispatch(assign, n, K, counts, b.offsets, b.perm, b.inv, ws, st));
  }
  return HMOE_OK;
}

int launch_fit(const void* X, hmoe_dtype_t dt, int64_t n, int32_t d, int32_t K, int32_t n_iter, const double* u,
               int32_t reseed, float* C, int32_t* assign, float* min_dist, int32_t* counts, double* objective,
               int32_t* init_idx, Workspace& ws, hipStream_t st) {
  if (dt == HMOE_BF16)
    return fit_t<bf16>((const bf16*)X, n, d, K, n_iter, u, reseed, C, assign, min_dist, counts, objective, init_idx,
                       ws, st);
  return fit_t<float>((const float*)X, n, d, K, n_iter, u, reseed, C, assign, min_dist, counts, objective, init_idx,
                      ws, st);
}

}  // namespace hmoe
