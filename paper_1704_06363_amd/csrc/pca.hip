// pca.hip -- the projection before the K-means (Section 4.2: the trunk's features are projected
// to their first 256 principal directions before the clustering).
//
// Fit: the sample mean (fp64 column sums), the covariance C = (X^T X - n m m^T) / (n - 1) with
// the lower triangle of X^T X on the tile engines (fp32 accumulation, the correction in fp64), and
// the r leading eigenpairs of C by subspace iteration: Q <- orth(C Q), n_iter times from a seeded
// start, then Rayleigh-Ritz (the eigenpairs of Q^T C Q, rotated back by Q).  The r x r steps -- the
// Cholesky factor behind each orthonormalisation (CholeskyQR) and the final symmetric eigensolve
// (Householder tridiagonalisation and implicit QR steps) -- are in fp64: for r <= kSmallN on the GPU
// but for the QR steps' scalars, for larger r, and where the block loses rank, on the host.  A fit
// synchronises its stream.
// Projection: Z = (X - m) U^T on the tile engine, the mean folded into an fp32 column bias.
#include <math.h>

#include <algorithm>
#include <vector>

#include "gemm.hpp"
#include "host_linalg.hpp"
#include "launch.hpp"
#include "primitives.hpp"
#include "small_linalg.hpp"

namespace hmoe {

static __global__ void k_pca_seg(int32_t* __restrict__ seg, int64_t rows) {
  if (threadIdx.x == 0) {
    seg[0] = 0;
    seg[1] = (int32_t)rows;
  }
}

// C = (C - s s^T / n) / (n - 1) in place (C holds X^T X on and below the diagonal, s the fp64 column
// sums), both triangles; mean = s / n.
static __global__ void __launch_bounds__(256) k_cov_finalize(float* __restrict__ C, const double* __restrict__ s,
                                                             int64_t n, int d, float* __restrict__ mean) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q < d) mean[q] = (float)(s[q] / (double)n);
  if (q >= (int64_t)d * d) return;
  const int i = (int)(q / d), j = (int)(q % d);
  if (j > i) return;
  const float c = (float)(((double)C[q] - s[i] * s[j] / (double)n) / (double)(n - 1));
  C[q] = c;
  C[(int64_t)j * d + i] = c;
}

// A seeded start for the subspace iteration: uniform in [-1, 1) from SplitMix64 of seed + index.
static __global__ void __launch_bounds__(256) k_pca_start(float* __restrict__ Q, int64_t count, uint64_t seed) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= count) return;
  uint64_t z = seed + (uint64_t)q + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  Q[q] = (float)((double)(z >> 11) * (1.0 / 9007199254740992.0) * 2.0 - 1.0);
}

// Fresh directions for the columns of Z [d][r] that flags[] marks (rank lost): uniform in
// [-1, 1) from SplitMix64 of seed + index, as k_pca_start.
static __global__ void __launch_bounds__(256) k_pca_refill(float* __restrict__ Z, int d, int r,
                                                           const int32_t* __restrict__ flags, uint64_t seed) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= (int64_t)d * r || !flags[q % r]) return;
  uint64_t z = seed + (uint64_t)q + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  Z[q] = (float)((double)(z >> 11) * (1.0 / 9007199254740992.0) * 2.0 - 1.0);
}

// comps[j][:] = sign_j U[:, j], sign_j making the largest-magnitude entry of the column positive
// (lowest index on ties).  One block per column.
static __global__ void __launch_bounds__(256) k_pca_comps(const float* __restrict__ U, int d, int r,
                                                          float* __restrict__ comps) {
  __shared__ float sv[256];
  __shared__ int si[256];
  const int j = blockIdx.x;
  float bv = -1.f;
  int bi = 0x7fffffff;
  for (int i = threadIdx.x; i < d; i += 256) {
    const float a = fabsf(U[(int64_t)i * r + j]);
    if (a > bv) {  // i increases: ties keep the lower index
      bv = a;
      bi = i;
    }
  }
  sv[threadIdx.x] = bv;
  si[threadIdx.x] = bi;
  __syncthreads();
  for (int w = 128; w >= 1; w >>= 1) {
    if (threadIdx.x < w) {
      const float ov = sv[threadIdx.x + w];
      const int oi = si[threadIdx.x + w];
      if (ov > sv[threadIdx.x] || (ov == sv[threadIdx.x] && oi < si[threadIdx.x])) {
        sv[threadIdx.x] = ov;
        si[threadIdx.x] = oi;
      }
    }
    __syncthreads();
  }
  const float sign = U[(int64_t)si[0] * r + j] < 0.f ? -1.f : 1.f;
  for (int i = threadIdx.x; i < d; i += 256) comps[(int64_t)j * d + i] = sign * U[(int64_t)i * r + j];
}

// b[j] = mean . comps[j] (fp32, fixed-order block sum) and the components in the data dtype.
template <typename T>
__global__ void __launch_bounds__(256) k_pca_bias(const float* __restrict__ mean, const float* __restrict__ comps,
                                                  int d, float* __restrict__ b, T* __restrict__ comps_lo) {
  __shared__ double sh[256];
  const int j = blockIdx.x;
  double s = 0.0;
  for (int i = threadIdx.x; i < d; i += 256) {
    const float c = comps[(int64_t)j * d + i];
    s += (double)mean[i] * (double)c;
    comps_lo[(int64_t)j * d + i] = from_f32<T>(c);
  }
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w >= 1; w >>= 1) {
    if (threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) b[j] = (float)sh[0];
}

// Z [n][r] = X comps_lo^T - b (the centred projection), in the data dtype.
template <class C>
__global__ void __launch_bounds__(C::THREADS)
    k_pca_project(const typename C::type* __restrict__ X, const typename C::type* __restrict__ W,
                  const float* __restrict__ b, int64_t n, int d, int r, typename C::type* __restrict__ Z) {
  using T = typename C::type;
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  lds<char>* smem = (lds<char>*)smem_raw;
  const TileCoord tc = tile_plain<C>(n, r, d);
  if (!tc.valid) return;
  floatx4 acc[C::MI][C::NJ];
  gemm_tile<C, true, true>(X + tc.m0 * d, d, tc.m_rows, W + (int64_t)tc.n0 * d, d, tc.n_cols, d, smem, acc);
  using F = Frag<C>;
  const F f;
  float bb[F::NCOL];
#pragma unroll
  for (int q = 0; q < F::NCOL; ++q) {
    const int col = f.colq(q);
    bb[q] = col < tc.n_cols ? b[tc.n0 + col] : 0.f;
  }
  store_out<C, T>(tc, acc, smem, Z, r, [&](int, int j, int rr, float v) { return v - bb[F::qidx(j, rr)]; },
                  RowId{tc.m0}, NoVec{});
}

// ------------------------------------------------------------------ host side of the fit (the r x r steps: host_linalg.hpp)

static int d2h(void* dst, const void* src, size_t bytes, hipStream_t st) {
  HMOE_TRY(hip_check(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, st), "pca: copy to host"));
  return hip_check(hipStreamSynchronize(st), "pca: synchronise");
}
static int h2d(void* dst, const void* src, size_t bytes, hipStream_t st) {
  HMOE_TRY(hip_check(hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, st), "pca: copy to device"));
  return hip_check(hipStreamSynchronize(st), "pca: synchronise");
}

// Q <- Q R^{-1} with Q^T Q = R^T R (CholeskyQR), `passes` times (the second pass restores the
// orthonormality the fp32 Gram matrix loses on an ill-conditioned Q); Z is scratch of Q's size.
// Rank-revealing: when a pivot falls below 1e-9 of the largest diagonal of Q^T Q (the fp32
// Gram matrix's noise; a covariance of rank below r does this), Q is rebuilt from the
// eigenpairs (w_j, v_j) of Q^T Q -- column j = Q v_j / sqrt(w_j) where w_j stays above that
// level, a fresh seeded random column where it does not -- and the passes start again.  The
// kept columns span what Q determined; the fresh ones lie outside it with probability 1.
constexpr double kRank = 1e-9;
static int orthonormalise(float*& Q, float*& Z, int d, int r, float* S, float* Rinv, int passes, uint64_t seed,
                          Workspace& ws, hipStream_t st) {
  std::vector<float> hs((size_t)r * r);
  std::vector<double> Sd((size_t)r * r), Ri;
  int refills = 0;
  for (int pass = 0; pass < passes; ++pass) {
    const size_t mark = ws.off;
    HMOE_TRY(launch_gemm_tn<float>(Q, Q, d, r, r, S, ws, st));
    HMOE_TRY(d2h(hs.data(), S, hs.size() * sizeof(float), st));
    for (size_t i = 0; i < hs.size(); ++i) Sd[i] = hs[i];
    if (!chol_inverse(Sd, r, Ri, kRank)) {
      if (++refills > 4) {
        set_error("pca: could not complete an orthonormal basis of %d columns", r);
        return HMOE_EINVAL;
      }
      std::vector<double> A = Sd, w, VT;
      if (!sym_eigen(A, r, w, VT)) {
        set_error("pca: the eigensolve of the %d x %d Gram matrix did not converge", r, r);
        return HMOE_ENUMERIC;
      }
      double wmax = 0.0;
      for (double x : w) wmax = x > wmax ? x : wmax;
      std::vector<int32_t> flags(r, 0);
      for (int j = 0; j < r; ++j) {
        const bool keep = wmax > 0.0 && w[j] > kRank * wmax;
        const double sc = keep ? 1.0 / sqrt(w[j]) : 0.0;
        for (int i = 0; i < r; ++i) hs[(size_t)i * r + j] = (float)(VT[(size_t)j * r + i] * sc);
        flags[j] = keep ? 0 : 1;
      }
      HMOE_TRY(h2d(Rinv, hs.data(), hs.size() * sizeof(float), st));
      HMOE_TRY(launch_gemm_nn<float>(Q, Rinv, d, r, r, Z, st));
      ws.off = mark;
      HMOE_TRY(h2d(S, flags.data(), flags.size() * sizeof(int32_t), st));  // S is free until the next pass
      HMOE_LAUNCH("pca refill", k_pca_refill, dim3((unsigned)cdiv((int64_t)d * r, 256)), dim3(256), 0, st, Z, d, r,
                  (const int32_t*)S, seed + 0x5851F42D4C957F2Dull * (uint64_t)refills);
      std::swap(Q, Z);
      pass = -1;  // orthonormalise the rebuilt block from scratch
      continue;
    }
    for (size_t i = 0; i < hs.size(); ++i) hs[i] = (float)Ri[i];
    HMOE_TRY(h2d(Rinv, hs.data(), hs.size() * sizeof(float), st));
    HMOE_TRY(launch_gemm_nn<float>(Q, Rinv, d, r, r, Z, st));
    ws.off = mark;
    std::swap(Q, Z);
  }
  return HMOE_OK;
}

// The fp64 scratch of the r x r steps on the GPU, over the products' partial sums: free whenever one
// of them runs (gemm_tn_ws() of either type holds it).
struct SmallBufs {
  double *U, *dinv, *W, *de;  // kSmallN^2, kSmallN, kSmallN^2, 2 kSmallN
  SmallRot* rot;              // kRotGroups groups
  int32_t *k0, *order;
  static constexpr int kRotGroups = 8192;
  explicit SmallBufs(Workspace ws)
      : U(ws.take<double>(kSmallN * kSmallN)), dinv(ws.take<double>(kSmallN)), W(ws.take<double>(kSmallN * kSmallN)),
        de(ws.take<double>(2 * kSmallN)), rot(ws.take<SmallRot>((size_t)kRotGroups * kRotGroup)),
        k0(ws.take<int32_t>(kRotGroups)), order(ws.take<int32_t>(kSmallN)), fits(ws.fits()) {}
  bool fits;
};

// orthonormalise() without a trip to the host, r <= kSmallN: a block that loses rank sets *flag
// (and leaves Q undefined).  r = 256, d = 512: 0.26 ms a pass (1.0 with the factor and the inverse on the host).
static int orthonormalise_gpu(float*& Q, float*& Z, int d, int r, float* S, float* Rinv, int passes, int32_t* flag,
                              Workspace& ws, hipStream_t st) {
  const SmallBufs b(ws);
  if (!b.fits) return HMOE_EWORKSPACE;
  for (int pass = 0; pass < passes; ++pass) {
    const size_t mark = ws.off;
    HMOE_TRY(launch_gemm_tn<float>(Q, Q, d, r, r, S, ws, st));
    ws.off = mark;
    HMOE_LAUNCH("pca cholesky", k_small_chol, dim3(1), dim3(1024), 0, st, (const float*)S, r, kRank, b.U, b.dinv, flag);
    HMOE_LAUNCH("pca triangular inverse", k_small_tri_inverse, dim3((unsigned)cdiv(r, 4)), dim3(256), 0, st,
                (const double*)b.U, (const double*)b.dinv, r, Rinv);
    HMOE_TRY(launch_gemm_nn<float>(Q, Rinv, d, r, r, Z, st));
    std::swap(Q, Z);
  }
  return HMOE_OK;
}

// Up to this r the final eigensolve runs on the host: its r^3 steps take less there than the GPU's chain
// of launches and copies.  A fit of 2000 x 256 without iterations, GPU / host: r = 32 0.56 / 0.35 ms, 64
// 0.94 / 0.70, 96 1.37 / 1.32, 128 1.93 / 2.47.
constexpr int kRitzHost = 96;

// The eigenvectors of (S + S^T) / 2, r <= kSmallN, as the columns of V (fp32, r x r) in decreasing
// order of their eigenvalues, which go to eigvals.  r = 256: 2.9 ms (16 on the host).
static int ritz_gpu(const float* S, int r, float* V, float* eigvals, Workspace& ws, hipStream_t st) {
  const SmallBufs b(ws);
  if (!b.fits) return HMOE_EWORKSPACE;
  HMOE_LAUNCH("pca tridiagonal", k_small_tridiag, dim3(1), dim3(1024), 0, st, S, r, b.U, b.de);
  std::vector<double> de(2 * kSmallN);
  HMOE_TRY(d2h(de.data(), b.de, de.size() * sizeof(double), st));
  std::vector<double> d(de.begin(), de.begin() + r), e(r, 0.0);
  for (int i = 0; i + 1 < r; ++i) e[i] = de[kSmallN + i];
  // the rotations go out in pieces while the next ones are formed; the host's copies of them stay
  // until the device has read them (the vectors never grow past their room)
  constexpr int kPiece = 1024;
  constexpr int kRotLds = (kSmallN + kRotGroup) * 64 * (int)sizeof(double);
  std::vector<SmallRot> rot;
  std::vector<int32_t> k0;
  rot.reserve((size_t)SmallBufs::kRotGroups * kRotGroup);
  k0.reserve(SmallBufs::kRotGroups);
  size_t sent = 0;
  bool first = true;
  const auto close = [&] { rot.resize(k0.size() * kRotGroup, SmallRot{1.0, 0.0}); };
  const auto send = [&]() -> int {
    const int m = (int)(k0.size() - sent);
    if (m > 0) {
      HMOE_TRY(hip_check(hipMemcpyAsync(b.rot + sent * kRotGroup, rot.data() + sent * kRotGroup,
                                        (size_t)m * kRotGroup * sizeof(SmallRot), hipMemcpyHostToDevice, st),
                         "pca: copy to device"));
      HMOE_TRY(hip_check(hipMemcpyAsync(b.k0 + sent, k0.data() + sent, (size_t)m * sizeof(int32_t),
                                        hipMemcpyHostToDevice, st),
                         "pca: copy to device"));
    }
    HMOE_LAUNCH("pca rotations", k_small_rotate, dim3(kSmallN / 64), dim3(64), kRotLds, st,
                (const SmallRot*)(b.rot + sent * kRotGroup), (const int32_t*)(b.k0 + sent), m, r, (int)first, b.W);
    first = false;
    sent = k0.size();
    return HMOE_OK;
  };
  int rc = HMOE_OK;
  const bool ok = tridiag_eigen(
      d, e, r,
      [&](int lo, int hi) {
        close();
        if (rc == HMOE_OK && k0.size() - sent >= kPiece) rc = send();
        if (k0.size() + (hi - lo + kRotGroup - 1) / kRotGroup > SmallBufs::kRotGroups) {  // no room for this step
          if (rc == HMOE_OK) rc = send();
          if (rc == HMOE_OK) rc = hip_check(hipStreamSynchronize(st), "pca: synchronise");
          rot.clear();
          k0.clear();
          sent = 0;
        }
      },
      [&](int k, double c, double s) {
        if (rot.size() == k0.size() * kRotGroup) k0.push_back(k);
        rot.push_back(SmallRot{c, s});
      });
  close();
  if (rc == HMOE_OK) rc = send();
  if (rc != HMOE_OK || !ok) {
    const int drained = hip_check(hipStreamSynchronize(st), "pca: synchronise");  // before the copies go
    if (rc != HMOE_OK || drained != HMOE_OK) return rc != HMOE_OK ? rc : drained;
    set_error("pca: the eigensolve of the %d x %d Rayleigh-Ritz matrix did not converge", r, r);
    return HMOE_ENUMERIC;
  }
  std::vector<int32_t> ord(r);
  for (int i = 0; i < r; ++i) ord[i] = i;
  std::stable_sort(ord.begin(), ord.end(), [&](int x, int y) { return d[x] > d[y]; });
  std::vector<float> hw(r);
  for (int j = 0; j < r; ++j) hw[j] = (float)d[ord[j]];
  HMOE_TRY(h2d(b.order, ord.data(), (size_t)r * sizeof(int32_t), st));
  HMOE_TRY(h2d(eigvals, hw.data(), hw.size() * sizeof(float), st));
  HMOE_LAUNCH("pca eigenvectors", k_small_back, dim3((unsigned)cdiv(r, 4)), dim3(256), 0, st, (const double*)b.W,
              (const double*)b.U, (const int32_t*)b.order, r, V);
  return HMOE_OK;
}

size_t pca_fit_ws(int64_t n, int d, int r, hmoe_dtype_t dt) {
  Workspace ws(nullptr, 0);
  ws.take<double>(d);
  ws.take<int32_t>(2);
  ws.take<float>((size_t)d * d);
  ws.take<float>((size_t)d * r);
  ws.take<float>((size_t)d * r);
  ws.take<float>((size_t)r * r);
  ws.take<float>((size_t)r * r);
  const size_t g = dt == HMOE_BF16 ? gemm_tn_ws<bf16>() : gemm_tn_ws<float>();
  const size_t sg = segsum_ws(n, 1, d);
  return ws.off + (g > sg ? g : sg) + 4096;
}

template <typename T>
static int pca_fit_t(const T* X, int64_t n, int d, int r, int n_iter, uint64_t seed, float* mean, float* comps,
                     float* eigvals, Workspace& ws, hipStream_t st) {
  double* msum = ws.take<double>(d);
  int32_t* seg = ws.take<int32_t>(2);
  float* Cv = ws.take<float>((size_t)d * d);
  float* Q = ws.take<float>((size_t)d * r);
  float* Z = ws.take<float>((size_t)d * r);
  float* S = ws.take<float>((size_t)r * r);
  float* Rinv = ws.take<float>((size_t)r * r);
  if (!ws.fits()) return HMOE_EWORKSPACE;
  const size_t mark = ws.off;
  HMOE_LAUNCH("pca segment", k_pca_seg, dim3(1), dim3(64), 0, st, seg, n);
  HMOE_TRY(launch_segsum<T, double>(X, d, nullptr, seg, 1, d, n, msum, 0, ws, st));
  ws.off = mark;
  HMOE_TRY(launch_gram<T>(X, n, d, Cv, ws, st, "pca X^T X"));
  ws.off = mark;
  HMOE_LAUNCH("pca covariance", k_cov_finalize, dim3((unsigned)cdiv((int64_t)d * d, 256)), dim3(256), 0, st, Cv, msum,
              n, d, mean);
  // one CholeskyQR pass per iteration keeps the subspace; the basis that enters Rayleigh-Ritz
  // gets two
  const auto iterate = [&](bool gpu, bool& lost) -> int {
    HMOE_LAUNCH("pca start", k_pca_start, dim3((unsigned)cdiv((int64_t)d * r, 256)), dim3(256), 0, st, Q,
                (int64_t)d * r, seed);
    const auto orth = [&](int passes, uint64_t s) {
      return gpu ? orthonormalise_gpu(Q, Z, d, r, S, Rinv, passes, seg, ws, st)
                 : orthonormalise(Q, Z, d, r, S, Rinv, passes, s, ws, st);
    };
    HMOE_TRY(orth(n_iter == 0 ? 2 : 1, seed ^ 0xA5A5A5A5u));
    for (int it = 0; it < n_iter; ++it) {
      HMOE_TRY(launch_gemm_nn<float>(Cv, Q, d, d, r, Z, st));
      std::swap(Q, Z);
      HMOE_TRY(orth(it == n_iter - 1 ? 2 : 1, seed + 0x9E3779B9u * (uint64_t)(it + 1)));
      // a covariance of rank below r shows in the first product
      if (gpu && (it == 0 || it == n_iter - 1)) {
        int32_t flag = 0;
        HMOE_TRY(d2h(&flag, seg, sizeof flag, st));
        if ((lost = flag != 0)) return HMOE_OK;
      }
    }
    if (gpu && n_iter == 0) {
      int32_t flag = 0;
      HMOE_TRY(d2h(&flag, seg, sizeof flag, st));
      lost = flag != 0;
    }
    return HMOE_OK;
  };
  bool lost = false;
  const bool small = r <= kSmallN;
  if (small) {
    HMOE_LAUNCH("pca segment", k_pca_seg, dim3(1), dim3(64), 0, st, seg, (int64_t)0);  // seg[0] = 0: the flag
    HMOE_TRY(iterate(true, lost));
  }
  if (!small || lost) HMOE_TRY(iterate(false, lost));
  // Rayleigh-Ritz: the eigenpairs of Q^T C Q, sorted by decreasing eigenvalue
  HMOE_TRY(launch_gemm_nn<float>(Cv, Q, d, d, r, Z, st));
  HMOE_TRY(launch_gemm_tn<float>(Q, Z, d, r, r, S, ws, st));
  ws.off = mark;
  if (small && r > kRitzHost) {
    HMOE_TRY(ritz_gpu(S, r, Rinv, eigvals, ws, st));
    HMOE_TRY(launch_gemm_nn<float>(Q, Rinv, d, r, r, Z, st));
    HMOE_LAUNCH("pca components", k_pca_comps, dim3((unsigned)r), dim3(256), 0, st, (const float*)Z, d, r, comps);
    return HMOE_OK;
  }
  std::vector<float> hs((size_t)r * r);
  HMOE_TRY(d2h(hs.data(), S, hs.size() * sizeof(float), st));
  std::vector<double> Tm((size_t)r * r), w, VT;
  for (int i = 0; i < r; ++i)
    for (int j = 0; j < r; ++j) Tm[(size_t)i * r + j] = 0.5 * ((double)hs[(size_t)i * r + j] + hs[(size_t)j * r + i]);
  if (!sym_eigen(Tm, r, w, VT)) {
    set_error("pca: the eigensolve of the %d x %d Rayleigh-Ritz matrix did not converge", r, r);
    return HMOE_ENUMERIC;
  }
  std::vector<int> ord(r);
  for (int i = 0; i < r; ++i) ord[i] = i;
  std::stable_sort(ord.begin(), ord.end(), [&](int a, int b) { return w[a] > w[b]; });
  std::vector<float> hw(r);
  for (int i = 0; i < r; ++i)
    for (int j = 0; j < r; ++j) hs[(size_t)i * r + j] = (float)VT[(size_t)ord[j] * r + i];
  for (int j = 0; j < r; ++j) hw[j] = (float)w[ord[j]];
  HMOE_TRY(h2d(Rinv, hs.data(), hs.size() * sizeof(float), st));
  HMOE_TRY(h2d(eigvals, hw.data(), hw.size() * sizeof(float), st));
  HMOE_TRY(launch_gemm_nn<float>(Q, Rinv, d, r, r, Z, st));
  HMOE_LAUNCH("pca components", k_pca_comps, dim3((unsigned)r), dim3(256), 0, st, (const float*)Z, d, r, comps);
  return HMOE_OK;
}

int launch_pca_fit(const void* X, hmoe_dtype_t dt, int64_t n, int d, int r, int n_iter, uint64_t seed, float* mean,
                   float* comps, float* eigvals, Workspace& ws, hipStream_t st) {
  if (dt == HMOE_BF16) return pca_fit_t<bf16>((const bf16*)X, n, d, r, n_iter, seed, mean, comps, eigvals, ws, st);
  return pca_fit_t<float>((const float*)X, n, d, r, n_iter, seed, mean, comps, eigvals, ws, st);
}

size_t pca_project_ws(int d, int r, hmoe_dtype_t dt) {
  Workspace ws(nullptr, 0);
  ws.take<float>(r);
  ws.take<char>((size_t)r * d * (dt == HMOE_BF16 ? 2 : 4));
  return ws.off;
}

// Up to 64 components run the narrow tiles of the ring engine (a 256 x 256 tile would be padding, and a
// reduction of one short stage nothing but its latency: 300,000 x 16 fp32 to 8 components 64 us, 20
// on these; x 512 to 64 645 and 252), half as high where there are fewer of those than CUs.
template <typename T, class C>
static int pca_project_t(const T* X, int64_t n, int d, const float* mean, const float* comps, int r, T* Zo,
                         Workspace& ws, hipStream_t st) {
  float* b = ws.take<float>(r);
  T* W = ws.take<T>((size_t)r * d);
  if (!ws.fits()) return HMOE_EWORKSPACE;
  HMOE_LAUNCH("pca bias", k_pca_bias<T>, dim3((unsigned)r), dim3(256), 0, st, mean, comps, d, b, W);
  HMOE_LAUNCH("pca project", k_pca_project<C>, dim3((unsigned)(cdiv(n, C::BM) * cdiv(r, C::BN))), dim3(C::THREADS),
              C::LDS, st, X, (const T*)W, (const float*)b, n, d, r, Zo);
  return HMOE_OK;
}

int launch_pca_project(const void* X, hmoe_dtype_t dt, int64_t n, int d, const float* mean, const float* comps,
                       int r, void* Z, Workspace& ws, hipStream_t st) {
  // both operands K-contiguous: the direct-to-LDS engines in either dtype (the workspace has room for
  // d^2 floats, so d is far below kPipeMaxLd / 2)
  const bool few = cdiv(n, CfgDmaNarrow::BM) < device_cus();
  if (dt == HMOE_BF16) {
    const auto run = r > 64 ? pca_project_t<bf16, CfgPipe>
                            : (few ? pca_project_t<bf16, CfgDmaNarrowFew> : pca_project_t<bf16, CfgDmaNarrow>);
    return run((const bf16*)X, n, d, mean, comps, r, (bf16*)Z, ws, st);
  }
  const auto run = r > 64 ? pca_project_t<float, CfgPipeF32>
                          : (few ? pca_project_t<float, CfgDmaF32NarrowFew> : pca_project_t<float, CfgDmaF32Narrow>);
  return run((const float*)X, n, d, mean, comps, r, (float*)Z, ws, st);
}

}  // namespace hmoe
