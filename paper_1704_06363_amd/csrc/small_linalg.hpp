// small_linalg.hpp -- the r x r steps of the PCA fit on the GPU, in fp64, for r <= 256: the Cholesky
// factor of a Gram matrix with the inverse behind CholeskyQR, and the symmetric eigensolve's
// tridiagonalisation and eigenvectors (its scalar QR steps run on the host, host_linalg.hpp).
// The serial chains of both sit in one workgroup that holds the matrix in registers: thread
// (ty, tx) of 32 x 32 has the elements (ty + 32 a, tx + 32 b), b <= a, of the lower triangle in
// 32 x 32 blocks (the diagonal blocks whole), 72 of its 128 registers.
#pragma once
#include "common.hpp"

namespace hmoe {

constexpr int kSmallN = 256;  // largest r, and the leading dimension of the fp64 scratch matrices
constexpr int kSmallB = kSmallN / 32;

__device__ __forceinline__ double small_lane(double v, int lane) {  // `lane` wave-uniform
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), lane);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// 1 / sqrt(x) to fp64's last bits: the hardware's estimate and two Newton steps.
__device__ __forceinline__ double small_rsqrt(double x) {
  double y = __builtin_amdgcn_rsq(x);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const double e = fma(-x * y, y, 1.0);
    y = fma(0.5 * y, e, y);
  }
  return y;
}

struct CholLds {
  double col[2][kSmallN], rroot[2];
};

// The columns of block kb (a constant, so that A stays in registers) and of those after it.
template <int kb>
__device__ __forceinline__ void chol_block(double (&A)[kSmallB][kSmallB], int r, double least, double* __restrict__ U,
                                           double* __restrict__ dinv, int32_t* __restrict__ flag, CholLds& m) {
  const int t = threadIdx.x, tx = t & 31, ty = t >> 5;
  for (int kr = 0; kr < 32; ++kr) {
    const int k = 32 * kb + kr;
    if (k >= r) return;
    double* c = m.col[k & 1];
    if (tx == kr) {
#pragma unroll
      for (int a = kb; a < kSmallB; ++a) c[ty + 32 * a] = A[a][kb];
      if (ty == kr) m.rroot[k & 1] = small_rsqrt(A[kb][kb]);
    }
    __syncthreads();  // the other buffer's readers are one barrier behind at most
    const double piv = c[k];
    if (!(piv > 0.0) || !(piv > least)) {
      if (t == 0) *flag = 1;
      return;
    }
    const double rs = m.rroot[k & 1];  // by one thread: with root and divisions in all of them 216 us
    if (t < kSmallN) U[(int64_t)k * kSmallN + t] = t > k ? c[t] * rs : 0.0;
    if (t == 0) dinv[k] = rs;
    const double w = -rs * rs;
    double cj[kSmallB];
#pragma unroll
    for (int b = kb; b < kSmallB; ++b) cj[b] = c[tx + 32 * b];
#pragma unroll
    for (int a = kb; a < kSmallB; ++a) {
      const double ci = c[ty + 32 * a] * w;
#pragma unroll
      for (int b = kb; b <= a; ++b) A[a][b] = fma(ci, cj[b], A[a][b]);
    }
  }
  if constexpr (kb + 1 < kSmallB) chol_block<kb + 1>(A, r, least, U, dinv, flag, m);
}

// S (r x r, fp32) + shift I = L L^T, the shift 1e-12 of the mean diagonal: U[k][i] = L[i][k] (fp64,
// ld kSmallN, 0 for i <= k and past r), dinv[k] = 1 / L[k][k].  A pivot (before its square root)
// that is not above min_rel_pivot of the largest diagonal entry ends the factorisation and sets
// *flag.  One workgroup, right-looking, a barrier per column; bound by the LDS
// reads of the column (publishing the next column before the other updates changes nothing;
// two entries to a read needs registers that are not there: 251 us).  r = 256: 190 us.
static __global__ void __launch_bounds__(1024) k_small_chol(const float* __restrict__ S, int r, double min_rel_pivot,
                                                            double* __restrict__ U, double* __restrict__ dinv,
                                                            int32_t* __restrict__ flag) {
  __shared__ CholLds m;
  __shared__ double s_tr, s_max;
  const int t = threadIdx.x, tx = t & 31, ty = t >> 5;
  if (t < 64) {
    double tr = 0.0, mx = 0.0;
    for (int i = t; i < r; i += 64) {
      const double v = (double)S[(int64_t)i * r + i];
      tr += v;
      mx = fmax(mx, v);
    }
    tr = wave_sum(tr);
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) mx = fmax(mx, shfl_xor(mx, m));
    if (t == 0) {
      s_tr = tr;
      s_max = mx;
    }
  }
  __syncthreads();
  const double shift = 1e-12 * s_tr / r, least = min_rel_pivot * s_max;
  double A[kSmallB][kSmallB];
#pragma unroll
  for (int a = 0; a < kSmallB; ++a)
#pragma unroll
    for (int b = 0; b <= a; ++b) {
      const int i = ty + 32 * a, j = tx + 32 * b;
      double v = 0.0;
      if (i < r && j < r) v = (double)S[(int64_t)(i > j ? i : j) * r + (i > j ? j : i)];
      A[a][b] = i == j ? v + shift : v;
    }
  chol_block<0>(A, r, least, U, dinv, flag, m);
}

// Rinv (fp32, r x r) = R^-1 for R = L^T: its row j is column j of L^-1, by a wave each, lane l
// holding entries l, l + 64, ... of the forward solve, a column of L at a time.
static __global__ void __launch_bounds__(256) k_small_tri_inverse(const double* __restrict__ U,
                                                                  const double* __restrict__ dinv, int r,
                                                                  float* __restrict__ Rinv) {
  const int j = blockIdx.x * 4 + (threadIdx.x >> 6), l = threadIdx.x & 63;
  if (j >= r) return;
  constexpr int P = 8;  // columns of L fetched ahead of their use (one by one: 72 us)
  double x[4], dv[4], u[P][4], un[P][4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    x[q] = l + 64 * q == j ? 1.0 : 0.0;
    dv[q] = l + 64 * q < r ? dinv[l + 64 * q] : 0.0;
  }
  const auto fetch = [&](double (&to)[P][4], int k0, int q0) {  // rows past r are not used
#pragma unroll
    for (int z = 0; z < P; ++z)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (q >= q0) to[z][q] = U[(int64_t)(k0 + z < r ? k0 + z : r - 1) * kSmallN + l + 64 * q];
  };
  fetch(u, 0, 0);
#pragma unroll
  for (int kq = 0; kq < 4; ++kq)
    for (int k0 = 0; k0 < 64; k0 += P) {
      if (64 * kq + k0 >= r) break;
      fetch(un, 64 * kq + k0 + P, kq);
#pragma unroll
      for (int z = 0; z < P; ++z) {
        const int kl = k0 + z;
        const double xk = small_lane(x[kq], kl) * small_lane(dv[kq], kl);  // 0 until k = j, and past r
#pragma unroll
        for (int q = kq; q < 4; ++q) x[q] = fma(-u[z][q], xk, x[q]);
        if (l == kl) x[kq] = xk;
      }
#pragma unroll
      for (int z = 0; z < P; ++z)
#pragma unroll
        for (int q = kq; q < 4; ++q) u[z][q] = un[z][q];
    }
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (l + 64 * q < r) Rinv[(int64_t)j * r + l + 64 * q] = (float)x[q];
}

// Householder reduction of A = (S + S^T) / 2 (r x r, fp32 in) to tridiagonal form, as sym_eigen in
// host_linalg.hpp: the reflection of step k is I - u u^T with u in refl[k][k + 1 ..] (zeros before
// and past r; all zeros where nothing is to be done), the diagonal and off-diagonal in de[0 .. r)
// and de[kSmallN ..].  One workgroup; a step multiplies the trailing block by u from the lower
// triangle (row sums over the 32 lanes, column sums over the 16 waves) and updates it.
// r = 256: 787 us.
struct TridiagLds {
  double u[kSmallN], q[kSmallN], row[kSmallN], col[16][kSmallN], half;
};

// The steps whose column lies in block KB (a constant, so that A stays in registers).
template <int kb>
__device__ __forceinline__ void tridiag_block(double (&A)[kSmallB][kSmallB], int r, double* __restrict__ refl,
                                              double* __restrict__ de, TridiagLds& m) {
  const int t = threadIdx.x, tx = t & 31, ty = t >> 5, w = t >> 6, l = t & 63;
  for (int kr = 0; kr < 32; ++kr) {
    const int k = 32 * kb + kr;
    if (k >= r) return;
    // column k from the diagonal down
    if (tx == kr) {
#pragma unroll
      for (int a = kb; a < kSmallB; ++a) m.u[ty + 32 * a] = A[a][kb];
    }
    __syncthreads();
    if (t == 0) de[k] = m.u[k];
    if (k + 1 >= r) continue;
    // u by the first wave: lane l has entries l, l + 64, ...
    if (w == 0) {
      double x[4], s = 0.0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = l + 64 * q;
        x[q] = i > k && i < r ? m.u[i] : 0.0;
        s += x[q] * x[q];
      }
      const double x0 = m.u[k + 1];
      const double xn = sqrt(wave_sum(s));
      if (k + 2 >= r) {  // the last off-diagonal entry as it is
        if (l == 0) de[kSmallN + k] = x0;
      } else {
        const double alpha = x0 > 0.0 ? -xn : xn;
        s = 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (l + 64 * q == k + 1) x[q] -= alpha;
          s += x[q] * x[q];
        }
        s = wave_sum(s);
        const double sc = xn == 0.0 ? 0.0 : sqrt(2.0 / s);
        if (l == 0) de[kSmallN + k] = xn == 0.0 ? 0.0 : alpha;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int i = l + 64 * q;
          const double u = xn == 0.0 ? 0.0 : x[q] * sc;
          m.u[i] = u;
          refl[(int64_t)k * kSmallN + i] = u;
        }
      }
    }
    __syncthreads();
    if (k + 2 >= r) continue;
    // p = A u: row sums of the stored blocks, column sums of those below the diagonal
    double uj[kSmallB], cs[kSmallB];
#pragma unroll
    for (int b = kb; b < kSmallB; ++b) {
      uj[b] = m.u[tx + 32 * b];
      cs[b] = 0.0;
    }
#pragma unroll
    for (int a = kb; a < kSmallB; ++a) {
      const double ui = m.u[ty + 32 * a];
      double rs = 0.0;
#pragma unroll
      for (int b = kb; b <= a; ++b) {
        rs = fma(A[a][b], uj[b], rs);
        if (b < a) cs[b] = fma(A[a][b], ui, cs[b]);
      }
      rs = swap_add<false>(row_sum(rs));
      if (tx == 0) m.row[ty + 32 * a] = rs;
    }
#pragma unroll
    for (int b = kb; b < kSmallB; ++b) {
      cs[b] = swap_add<true>(cs[b]);  // the wave's two rows ty
      if (l < 32) m.col[w][tx + 32 * b] = cs[b];
    }
    __syncthreads();
    // q = p - (u . p / 2) u by the first four waves
    if (t < kSmallN && t >= 32 * kb) {
      double p = m.row[t];
#pragma unroll
      for (int v = 0; v < 16; ++v) p += m.col[v][t];
      m.q[t] = p;
    }
    __syncthreads();
    if (w == 0) {
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (l + 64 * q >= 32 * kb) s = fma(m.u[l + 64 * q], m.q[l + 64 * q], s);
      s = wave_sum(s);
      if (l == 0) m.half = 0.5 * s;
    }
    __syncthreads();
    const double half = m.half;
    double qj[kSmallB];
#pragma unroll
    for (int b = kb; b < kSmallB; ++b) {
      uj[b] = m.u[tx + 32 * b];
      qj[b] = fma(-half, uj[b], m.q[tx + 32 * b]);
    }
#pragma unroll
    for (int a = kb; a < kSmallB; ++a) {
      const double ui = m.u[ty + 32 * a];
      const double qi = fma(-half, ui, m.q[ty + 32 * a]);
#pragma unroll
      for (int b = kb; b <= a; ++b) A[a][b] = A[a][b] - fma(ui, qj[b], qi * uj[b]);
    }
    __syncthreads();  // m.u is rewritten by the next step
  }
  if constexpr (kb + 1 < kSmallB) tridiag_block<kb + 1>(A, r, refl, de, m);
}

static __global__ void __launch_bounds__(1024) k_small_tridiag(const float* __restrict__ S, int r,
                                                               double* __restrict__ refl, double* __restrict__ de) {
  __shared__ TridiagLds m;
  const int t = threadIdx.x, tx = t & 31, ty = t >> 5;
  double A[kSmallB][kSmallB];
#pragma unroll
  for (int a = 0; a < kSmallB; ++a)
#pragma unroll
    for (int b = 0; b <= a; ++b) {
      const int i = ty + 32 * a, j = tx + 32 * b;
      A[a][b] = i < r && j < r ? 0.5 * ((double)S[(int64_t)i * r + j] + (double)S[(int64_t)j * r + i]) : 0.0;
    }
  tridiag_block<0>(A, r, refl, de, m);
}

// A rotation of rows (k, k + 1): row k <- c row k - s row k+1, row k+1 <- s row k + c row k+1.
struct SmallRot {
  double c, s;
};
constexpr int kRotGroup = 16;  // rotations come in groups of consecutive k, the first k of each in k0

// Applies `groups` groups of rotations to the rows of V ([r][kSmallN], row k of column j at lane
// j); `first` starts from the identity.  A wave per 64 columns, which sit in LDS; the rows past
// r absorb the identity rotations that fill a group.  Bound by the one wave's instructions: a lane
// fetches one of four groups' rotations, the next four while these run, and each is handed to all
// lanes through scalar registers (a load of its own for each rotation, the same in every lane, took
// longer than the rotation); where a group follows on from the one before, its rows are read ahead.
// r = 256: 1.7 ms.
static __global__ void __launch_bounds__(64) k_small_rotate(const SmallRot* __restrict__ rot,
                                                            const int32_t* __restrict__ k0, int groups, int r,
                                                            int first, double* __restrict__ V) {
  extern __shared__ __attribute__((aligned(16))) char small_smem[];
  double* v = reinterpret_cast<double*>(small_smem);  // [kSmallN + kRotGroup][64]
  const int l = threadIdx.x, j = blockIdx.x * 64 + l;
  for (int k = 0; k < kSmallN + kRotGroup; ++k)
    v[k * 64 + l] = first ? (k == j ? 1.0 : 0.0) : (k < r ? V[(int64_t)k * kSmallN + j] : 0.0);
  constexpr int GS = 64 / kRotGroup;  // groups per fetch
  const auto fetch = [&](int g, SmallRot& q, int& k) {  // past the end: the last group again
    g += l / kRotGroup;
    g = g < groups ? g : groups - 1;
    q = rot[(int64_t)g * kRotGroup + l % kRotGroup];
    k = k0[g];
  };
  double x[kRotGroup + 1];
  if (groups > 0) {
    SmallRot q, nq;
    int k, nk;
    fetch(0, q, k);
    const int f = __builtin_amdgcn_readlane(k, 0);
#pragma unroll
    for (int z = 0; z <= kRotGroup; ++z) x[z] = v[(f + z) * 64 + l];
    for (int g = 0; g < groups; g += GS) {
      fetch(g + GS, nq, nk);
#pragma unroll
      for (int i = 0; i < GS; ++i) {
        if (g + i >= groups) break;
        const int kc = __builtin_amdgcn_readlane(k, i * kRotGroup);
        const int kn = i + 1 < GS ? __builtin_amdgcn_readlane(k, (i + 1) % GS * kRotGroup) : __builtin_amdgcn_readlane(nk, 0);
        const bool on = kn - kc == kRotGroup;
        double* row = v + kc * 64 + l;
        const double* nrow = v + kn * 64 + l;
        double y[kRotGroup + 1];
        if (on) {
#pragma unroll
          for (int z = 1; z <= kRotGroup; ++z) y[z] = nrow[z * 64];
        }
#pragma unroll
        for (int z = 0; z < kRotGroup; ++z) {
          const double c = small_lane(q.c, i * kRotGroup + z), s = small_lane(q.s, i * kRotGroup + z);
          const double a = x[z], b = x[z + 1];
          row[z * 64] = c * a - s * b;
          x[z + 1] = s * a + c * b;
        }
        if (on) {
          y[0] = x[kRotGroup];
        } else {
          row[kRotGroup * 64] = x[kRotGroup];
#pragma unroll
          for (int z = 0; z <= kRotGroup; ++z) y[z] = nrow[z * 64];
        }
#pragma unroll
        for (int z = 0; z <= kRotGroup; ++z) x[z] = y[z];
      }
      q = nq;
      k = nk;
    }
  }
  for (int k = 0; k < r; ++k) V[(int64_t)k * kSmallN + j] = v[k * 64 + l];
}

// Column order[j] of the eigenvector matrix: H_0 (H_1 ( ... W[:, order[j]])) with the reflections
// of k_small_tridiag, as column j of out (fp32, r x r).  W [r][kSmallN] holds the tridiagonal
// matrix's eigenvectors as rows.  A wave per column.
static __global__ void __launch_bounds__(256) k_small_back(const double* __restrict__ W,
                                                           const double* __restrict__ refl,
                                                           const int32_t* __restrict__ order, int r,
                                                           float* __restrict__ out) {
  const int j = blockIdx.x * 4 + (threadIdx.x >> 6), l = threadIdx.x & 63;
  if (j >= r) return;
  double x[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) x[q] = l + 64 * q < r ? W[(int64_t)order[j] * kSmallN + l + 64 * q] : 0.0;
#pragma unroll 4
  for (int k = r - 3; k >= 0; --k) {
    double u[4], s = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      u[q] = refl[(int64_t)k * kSmallN + l + 64 * q];
      s = fma(u[q], x[q], s);
    }
    s = wave_sum(s);
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = fma(-u[q], s, x[q]);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (l + 64 * q < r) out[(int64_t)(l + 64 * q) * r + j] = (float)x[q];
}

}  // namespace hmoe
