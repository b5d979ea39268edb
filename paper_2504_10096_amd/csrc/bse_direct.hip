// Kernels of the direct structure-preserving solve (paper Sec. 2.1): the
// dense matrices it factors are formed from the block storage of the stored
// triangles; M_r = L L^T is factored by a blocked Cholesky (diagonal blocks in
// LDS, panel solves, trailing updates on FP64 MFMA); W = L^T J L is one MFMA
// product; the real skew-symmetric W is reduced to tridiagonal form by
// Householder reflections, a panel of columns at a time, with the skew rank-2
// updates of a panel applied to the trailing matrix as MFMA products; the
// eigenvectors are carried back through the reflections and L^-T.  (The TDA
// dense solve hands A to rocSOLVER's Hermitian eigensolver.)
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bse_internal.h"
#include "bse_wave.h"

namespace bse {
namespace {

constexpr int kT = 256;

// FP64 value of stored element d of a triangle (complex128, or hi + lo).
__device__ inline double2 entry(const void* t, const void* tlo, int hilo, size_t d) {
  if (hilo) {
    const float2 h = static_cast<const float2*>(t)[d];
    const float2 l = static_cast<const float2*>(tlo)[d];
    return make_double2((double)h.x + (double)l.x, (double)h.y + (double)l.y);
  }
  return static_cast<const double2*>(t)[d];
}

// One workgroup per stored R x R block (P, Q), P <= Q; every stored (i <= j)
// entry is written to both of its places.  Diagonal blocks hold the diagonal
// halved and zeros below it: the diagonal is doubled, entries below skipped.
// TDA (b == nullptr): the Hermitian A, complex, column-major, leading
// dimension ld.  PH: M_r of Eq. (5), real 2N x 2N, leading dimension ld:
//   [ Re(A + B)   Im(A - B) ]
//   [ -Im(A + B)  Re(A - B) ]
// written in full (it is symmetric: A Hermitian, B symmetric).
__global__ void __launch_bounds__(kT)
    dense_kernel(const int2* __restrict__ blkmap, int R, int64_t n, int hilo, const void* __restrict__ a,
                 const void* __restrict__ alo, const void* __restrict__ b, const void* __restrict__ blo,
                 double2* __restrict__ ad, double* __restrict__ mr, int64_t ld) {
  const int64_t blk = blockIdx.x;
  const int2 pq = blkmap[blk];
  const size_t base = (size_t)blk * R * R;
  for (int e = threadIdx.x; e < R * R; e += kT) {
    const int c = e / R, r = e % R;
    const int64_t i = (int64_t)pq.x * R + r, j = (int64_t)pq.y * R + c;
    if (i >= n || j >= n || i > j) continue;
    double2 va = entry(a, alo, hilo, base + e);
    double2 vb = b ? entry(b, blo, hilo, base + e) : make_double2(0.0, 0.0);
    if (i == j) {
      va = make_double2(2.0 * va.x, 0.0);
      vb = make_double2(2.0 * vb.x, 2.0 * vb.y);
    }
    if (!b) {
      ad[(size_t)j * ld + i] = va;
      ad[(size_t)i * ld + j] = make_double2(va.x, -va.y);
      continue;
    }
    // (i, j) and (j, i) of each quadrant; A_ji = conj(A_ij), B_ji = B_ij
    const double rp = va.x + vb.x, rm = va.x - vb.x;  // Re(A + B), Re(A - B): same at (j, i)
    const double ip = va.y + vb.y, im = va.y - vb.y;  // Im(A + B), Im(A - B) at (i, j)
    const double ipt = -va.y + vb.y, imt = -va.y - vb.y;  // the same at (j, i)
    const size_t n_ = (size_t)n;
    mr[(size_t)j * ld + i] = rp;
    mr[(size_t)i * ld + j] = rp;
    mr[(size_t)(n_ + j) * ld + i] = im;
    mr[(size_t)(n_ + i) * ld + j] = imt;
    mr[(size_t)j * ld + n_ + i] = -ip;
    mr[(size_t)i * ld + n_ + j] = -ipt;
    mr[(size_t)(n_ + j) * ld + n_ + i] = rm;
    mr[(size_t)(n_ + i) * ld + n_ + j] = rm;
  }
}

// L: the lower triangle of a 2N x 2N Cholesky factor (upper part set to
// zero here).  G = J L with J = [0 I; -I 0]: rows N.. of L, then minus rows 0..N-1.
__global__ void __launch_bounds__(kT)
    jl_kernel(double* __restrict__ l, int64_t ld, int64_t n, double* __restrict__ g) {
  const int64_t n2 = 2 * n;
  const int64_t col = blockIdx.y;
  for (int64_t row = (int64_t)blockIdx.x * kT + threadIdx.x; row < n2; row += (int64_t)gridDim.x * kT) {
    const int64_t src = row < n ? row + n : row - n;
    const double sg = row < n ? 1.0 : -1.0;
    g[(size_t)col * ld + row] = col <= src ? sg * l[(size_t)col * ld + src] : 0.0;
  }
  __syncthreads();
  // zero the strict upper triangle of L (read above only where col <= src)
  for (int64_t row = (int64_t)blockIdx.x * kT + threadIdx.x; row < n2; row += (int64_t)gridDim.x * kT)
    if (row < col) l[(size_t)col * ld + row] = 0.0;
}

// Z = -i W (W real skew-symmetric: -i W is Hermitian), column-major.
__global__ void __launch_bounds__(kT)
    negi_kernel(const double* __restrict__ w, int64_t ld, int64_t n2, double2* __restrict__ z, int64_t ldz) {
  const int64_t col = blockIdx.y;
  for (int64_t row = (int64_t)blockIdx.x * kT + threadIdx.x; row < n2; row += (int64_t)gridDim.x * kT)
    z[(size_t)col * ldz + row] = make_double2(0.0, -w[(size_t)col * ld + row]);
}

// Columns c0 .. c0 + k - 1 of the complex eigenvectors -> a real 2N x 2k
// matrix: real parts in columns 0..k-1, imaginary parts in k..2k-1.
__global__ void __launch_bounds__(kT)
    split_kernel(const double2* __restrict__ z, int64_t ldz, int64_t n2, int c0, int k, double* __restrict__ rm,
                 int64_t ldr) {
  const int c = blockIdx.y;
  for (int64_t row = (int64_t)blockIdx.x * kT + threadIdx.x; row < n2; row += (int64_t)gridDim.x * kT) {
    const double2 v = z[(size_t)(c0 + c) * ldz + row];
    rm[(size_t)c * ldr + row] = v.x;
    rm[(size_t)(k + c) * ldr + row] = v.y;
  }
}

// x = (real part, imaginary part) of L^{-T} z, halves x1 = x[0, N), x2 = x[N, 2N);
// v = Q x with Q of Eq. (4): X = (x1 - i x2) / sqrt(2), Y = (x1 + i x2) / sqrt(2).
__global__ void __launch_bounds__(kT)
    back_kernel(const double* __restrict__ rm, int64_t ldr, int64_t n, int k, double2* __restrict__ x,
                double2* __restrict__ y, int64_t ldo) {
  const int c = blockIdx.y;
  const double s = 0.70710678118654752440;
  for (int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kT) {
    const double a = rm[(size_t)c * ldr + i], b = rm[(size_t)(k + c) * ldr + i];          // x1
    const double cc = rm[(size_t)c * ldr + n + i], d = rm[(size_t)(k + c) * ldr + n + i];  // x2
    x[(size_t)c * ldo + i] = make_double2(s * (a + d), s * (b - cc));
    y[(size_t)c * ldo + i] = make_double2(s * (a - d), s * (b + cc));
  }
}

// Scale column c of X (and Y) by f[c].
__global__ void __launch_bounds__(kT)
    scale_kernel(double2* __restrict__ x, double2* __restrict__ y, int64_t ld, int64_t n,
                 const double* __restrict__ f) {
  const int c = blockIdx.y;
  const double s = f[c];
  for (int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kT) {
    double2 v = x[(size_t)c * ld + i];
    x[(size_t)c * ld + i] = make_double2(s * v.x, s * v.y);
    if (y) {
      v = y[(size_t)c * ld + i];
      y[(size_t)c * ld + i] = make_double2(s * v.x, s * v.y);
    }
  }
}


// ---------------------------------------------------------------------
// Dense FP64 building blocks of the pseudo-Hermitian direct solve.
// ---------------------------------------------------------------------
typedef double dbl4 __attribute__((ext_vector_type(4)));

// C (M x N) = alpha op(A) op(B) + beta C, column-major, FP64 MFMA 16x16x4.
// op(A) is M x K: A stored M x K (TA = 0) or K x M (TA = 1, op = transpose);
// op(B) is K x N: B stored K x N (TB = 0) or N x K (TB = 1).  A 64 x 64 tile
// of C per workgroup (each of the four waves a 32 x 32 quarter), k-chunks of
// 16 staged through LDS with loads along each operand's contiguous
// dimension.  lower != 0: only entries on or below the diagonal are written
// (tiles entirely above it are skipped).  Operand layout of the instruction:
// A[i][k] in lane i + 16 k, B[k][j] in lane j + 16 k, D[i][j] in lane
// j + 16 (i % 4), register i / 4.
template <int TA, int TB>
__global__ void __launch_bounds__(256)
    gemm_kernel(int64_t M, int64_t N, int64_t K, double alpha, const double* __restrict__ A, int64_t lda,
                const double* __restrict__ B, int64_t ldb, double beta, double* __restrict__ C, int64_t ldc,
                int lower) {
  const int64_t tm = blockIdx.x, tn = blockIdx.y;
  if (lower && tm < tn) return;
  __shared__ double As[16][65];
  __shared__ double Bs[16][65];
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  const int li = lane & 15, lk = lane >> 4;
  const int wm = (wave & 1) * 32, wn = (wave >> 1) * 32;
  dbl4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = dbl4{0.0, 0.0, 0.0, 0.0};
  for (int64_t k0 = 0; k0 < K; k0 += 16) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int idx = t + 256 * r;
      const int i = TA == 0 ? (idx & 63) : (idx >> 4);
      const int k = TA == 0 ? (idx >> 6) : (idx & 15);
      const int64_t gi = tm * 64 + i, gk = k0 + k;
      double v = 0.0;
      if (gi < M && gk < K) v = TA == 0 ? A[(size_t)gk * lda + gi] : A[(size_t)gi * lda + gk];
      As[k][i] = v;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int idx = t + 256 * r;
      const int j = TB == 0 ? (idx >> 4) : (idx & 63);
      const int k = TB == 0 ? (idx & 15) : (idx >> 6);
      const int64_t gj = tn * 64 + j, gk = k0 + k;
      double v = 0.0;
      if (gj < N && gk < K) v = TB == 0 ? B[(size_t)gj * ldb + gk] : B[(size_t)gk * ldb + gj];
      Bs[k][j] = v;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; kk += 4) {
      double av[2], bv[2];
#pragma unroll
      for (int a = 0; a < 2; ++a) av[a] = As[kk + lk][wm + a * 16 + li];
#pragma unroll
      for (int b = 0; b < 2; ++b) bv[b] = Bs[kk + lk][wn + b * 16 + li];
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], acc[a][b], 0, 0, 0);
    }
    __syncthreads();
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int64_t gj = tn * 64 + wn + b * 16 + li;
      if (gj >= N) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t gi = tm * 64 + wm + a * 16 + 4 * r + lk;
        if (gi >= M || (lower && gi < gj)) continue;
        const size_t o = (size_t)gj * ldc + gi;
        C[o] = beta == 0.0 ? alpha * acc[a][b][r] : fma(alpha, acc[a][b][r], beta * C[o]);
      }
    }
}

// Cholesky of the diagonal block A11 (nb <= 64 columns from j0), lower triangle; a
// pivot that is not positive (or NaN) sets *flag.  A chain of 64 columns, bound by the
// latency of a pivot's root and quotients and of one barrier per column: lane r holds row r,
// wave w the columns w, w + 4, ... in registers (a block of fewer columns is
// filled up with the identity), and a finished column goes to the other waves
// through LDS.  The block in LDS with three barriers per column and an index
// division per entry took 83 us, 22 us here.
__global__ void __launch_bounds__(256)
    potrf_diag_kernel(double* __restrict__ A, int64_t ld, int64_t j0, int nb, int* __restrict__ flag) {
  __shared__ double L[2][64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r = threadIdx.x & 63;
  double a[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int c = 4 * k + wave;
    a[k] = r >= nb || c >= nb || r < c ? (r == c ? 1.0 : 0.0) : A[(size_t)(j0 + c) * ld + j0 + r];
  }
#pragma unroll
  for (int c = 0; c < 64; ++c) {
    const int k0 = c >> 2;
    if (wave == (c & 3)) {
      const double piv = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(a[k0]), c),
                                          __builtin_amdgcn_readlane(__double2loint(a[k0]), c));
      if (r == 0 && !(piv > 0.0)) atomicExch(flag, 1);
      const double d = sqrt(piv);
      a[k0] = r > c ? a[k0] / d : d;  // rows above the diagonal are never read
      L[c & 1][r] = a[k0];
    }
    __syncthreads();
    const double lr = L[c & 1][r];
#pragma unroll
    for (int k = k0; k < 16; ++k)
      if (k > k0 || wave > (c & 3)) a[k] = fma(-lr, L[c & 1][4 * k + wave], a[k]);
  }
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int c = 4 * k + wave;
    if (r < nb && r >= c) A[(size_t)(j0 + c) * ld + j0 + r] = a[k];
  }
}

// Panel solve of the blocked Cholesky: rows i >= j0 + nb of columns
// [j0, j0 + nb) become L21 = A21 L11^{-T} (each row a forward substitution
// with the factored diagonal block, held in LDS).
__global__ void __launch_bounds__(256)
    trsm_panel_kernel(double* __restrict__ A, int64_t ld, int64_t j0, int nb, int64_t m) {
  __shared__ double Ls[64][65];  // Ls[r][c] = L11(r, c)
  const int t = threadIdx.x;
  for (int e = t; e < nb * nb; e += 256) {
    const int c = e / nb, r = e % nb;
    Ls[r][c] = r >= c ? A[(size_t)(j0 + c) * ld + j0 + r] : 0.0;
  }
  __syncthreads();
  const int64_t i = j0 + nb + (int64_t)blockIdx.x * 256 + t;
  if (i >= m) return;
  double x[64];
#pragma unroll
  for (int c = 0; c < 64; ++c) x[c] = c < nb ? A[(size_t)(j0 + c) * ld + i] : 0.0;
#pragma unroll
  for (int c = 0; c < 64; ++c) {
    if (c < nb) {
      double s = x[c];
#pragma unroll
      for (int r = 0; r < c; ++r) s = fma(-x[r], Ls[c][r], s);
      x[c] = s / Ls[c][c];
    }
  }
#pragma unroll
  for (int c = 0; c < 64; ++c)
    if (c < nb) A[(size_t)(j0 + c) * ld + i] = x[c];
}

// Sum over a wavefront into every lane, fixed order.
__device__ inline double wave_sum64(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Skew-symmetric Householder reduction while more than kSkewOne rows are left: two
// launches per column j (local panel column t), bound by their latency, not by the
// reads (the trailing matrix is 33 MB at order 2048).  A launch for each of the reflector, the product, the
// corrections, p and the panel update, one row per thread with 256 columns in
// sequence in the product, took 29 us per column at order 2048; 11.3 us now.
//
// 16 waves per workgroup, so that a wave's share of the columns (16 of 256), of the
// panel's pairs and of its remaining columns is one batch of loads (four waves:
// 13.3 us per column for both).
constexpr int kSW = 16;

// The reflector of a column a, (I - tau v v^T) a = beta e_1, v_0 = 1, v_i = a_i sc,
// from alpha = a_0 and the sum sig2 of the squares of the others.
__device__ inline void reflector(double sig2, double alpha, double& beta, double& tau, double& sc) {
  if (sig2 == 0.0) {
    beta = alpha;
    tau = 0.0;
    sc = 0.0;
  } else {
    beta = -copysign(sqrt(fma(alpha, alpha, sig2)), alpha);
    tau = (beta - alpha) / beta;
    sc = 1.0 / (alpha - beta);
  }
}
// The same with sig2 as npn partial sums, by a wave.
__device__ inline void reflector(const double* __restrict__ pn, int npn, double alpha, int lane, double& beta,
                                 double& tau, double& sc) {
  double s = 0.0;
  for (int q = lane; q < npn; q += 64) s += pn[q];
  reflector(wave_sum64(s), alpha, beta, tau, sc);
}

// pn[b] = sum of W[i, j]^2 over the block's rows i >= j + 2 (a panel's first column).
__global__ void __launch_bounds__(256)
    skew_norm_kernel(const double* __restrict__ W, int64_t ld, int64_t m, int64_t j, double* __restrict__ pn) {
  __shared__ double red[4];
  const int64_t i = j + 2 + (int64_t)blockIdx.x * 256 + threadIdx.x;
  const double a = i < m ? W[(size_t)j * ld + i] : 0.0;
  const double s = wave_sum64(a * a);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) pn[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

// First launch of column j.  Workgroups b < nrow nchunk: partial products of
// the stored trailing matrix with v, 64 rows by 256 columns (each wave an equal
// share): part[y m + i] = sum over columns c of chunk y (from j + 1) of W[i, c]
// v_c.  The others, 2 t of them: dots[s] = Vp[:, s] . v and dots[t + s] =
// Zp[:, s] . v over the rows from r0 on (s = t - 1: from j + 1 on), the part of
// the panel's updates not yet stored in W (see skew_update_kernel).  Workgroup
// 0 records e[j] = beta, tau[j] and *scp = sc.
__global__ void __launch_bounds__(64 * kSW)
    skew_mv_kernel(const double* __restrict__ W, int64_t ld, int64_t m, int64_t j, int64_t r0, int t, int nrow,
                   int nchunk, const double* __restrict__ pn, int npn, const double* __restrict__ Vp,
                   const double* __restrict__ Zp, int64_t ldp, double* __restrict__ part, double* __restrict__ dots,
                   double* __restrict__ tau, double* __restrict__ e, double* __restrict__ scp) {
  constexpr int CW = 256 / kSW;  // columns of a wave
  __shared__ double vs[256];
  __shared__ double red[kSW][64];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const double* a = W + (size_t)j * ld;
  double beta, tj, sc;
  reflector(pn, npn, a[j + 1], lane, beta, tj, sc);
  const int b = blockIdx.x;
  if (b == 0 && tid == 0) {
    e[j] = beta;
    tau[j] = tj;
    *scp = sc;
  }
  if (b >= nrow * nchunk) {
    const int d = b - nrow * nchunk, s_ = d < t ? d : d - t;
    const double* q = (d < t ? Vp : Zp) + (size_t)s_ * ldp;
    double acc = 0.0;
    for (int64_t i = (s_ == t - 1 ? j + 1 : r0) + tid; i < m; i += 64 * kSW)
      acc = fma(q[i], i == j + 1 ? 1.0 : a[i] * sc, acc);
    acc = wave_sum64(acc);
    if (lane == 0) red[0][wave] = acc;
    __syncthreads();
    if (tid == 0) {
      double t = red[0][0];
      for (int w = 1; w < kSW; ++w) t += red[0][w];
      dots[d] = t;
    }
    return;
  }
  const int y = b / nrow;
  const int64_t i = j + 1 + (int64_t)(b % nrow) * 64 + lane;
  const int64_t cy = j + 1 + (int64_t)y * 256, c0 = cy + wave * CW;
  if (tid < 256) vs[tid] = cy + tid < m ? (cy + tid == j + 1 ? 1.0 : a[cy + tid] * sc) : 0.0;
  double w[CW];
  const double* wr = W + (size_t)c0 * ld + i;
#pragma unroll
  for (int u = 0; u < CW; ++u) w[u] = i < m && c0 + u < m ? wr[(size_t)u * ld] : 0.0;
  __syncthreads();
  double s0 = 0.0, s1 = 0.0;
#pragma unroll
  for (int u = 0; u < CW; u += 2) {
    s0 = fma(w[u], vs[wave * CW + u], s0);
    s1 = fma(w[u + 1], vs[wave * CW + u + 1], s1);
  }
  red[wave][lane] = s0 + s1;
  __syncthreads();
  if (wave == 0 && i < m) {
    double t = red[0][lane];
#pragma unroll
    for (int u = 1; u < kSW; ++u) t += red[u][lane];
    part[(size_t)y * m + i] = t;
  }
}

// Second launch of column j, 64 rows i > j per workgroup: the reflector goes to
// W[j+1:, j] and Vp[:, t]; z = tau p with p = (the skew matrix as updated by the
// panel so far) v = part + Vp (Zp^T v) - Zp (Vp^T v) goes to Zp[:, t].  The
// reflection pair (v, z) of a column changes the panel's remaining columns c by
// W[i, c] += v_i z_c - z_i v_c; z_c of other workgroups' rows is not known
// here, so the pair is applied one launch later (the pair of column j - 1 to
// the columns c > j), except to the next column j + 1, whose z every workgroup
// forms for itself.  With the next column complete its norm partials pn are
// left for the next reflector.
__global__ void __launch_bounds__(64 * kSW)
    skew_update_kernel(double* __restrict__ W, int64_t ld, int64_t m, int64_t j, int64_t r0, int t, int nchunk,
                       const double* __restrict__ part, const double* __restrict__ dots,
                       const double* __restrict__ tau, const double* __restrict__ scp, double* __restrict__ Vp,
                       double* __restrict__ Zp, int64_t ldp, double* __restrict__ pn) {
  __shared__ double red[kSW][64];
  __shared__ double znext;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int64_t i = j + 1 + (int64_t)blockIdx.x * 64 + lane;
  const bool in = i < m;
  const double tj = tau[j], sc = *scp;
  double p = 0.0;
  if (in) {
    for (int y = wave; y < nchunk; y += kSW) p += part[(size_t)y * m + i];
#pragma unroll 4
    for (int s_ = wave; s_ < t; s_ += kSW)
      p = fma(Vp[(size_t)s_ * ldp + i], dots[t + s_], fma(-Zp[(size_t)s_ * ldp + i], dots[s_], p));
  }
  red[wave][lane] = p;
  const bool more = j + 1 < r0;  // panel columns remain
  if (wave == kSW - 1 && more) {
    double q = 0.0;
    for (int y = lane; y < nchunk; y += 64) q += part[(size_t)y * m + j + 1];
    if (lane < t) q = fma(Vp[(size_t)lane * ldp + j + 1], dots[t + lane], fma(-Zp[(size_t)lane * ldp + j + 1], dots[lane], q));
    q = wave_sum64(q);
    if (lane == 0) znext = tj * q;
  }
  __syncthreads();
  double z = red[0][lane];
#pragma unroll
  for (int w = 1; w < kSW; ++w) z += red[w][lane];
  z *= tj;
  // (every wave reads its rows of column j before wave 0 writes them below)
  const double v = !in ? 0.0 : i == j + 1 ? 1.0 : W[(size_t)j * ld + i] * sc;
  const double vo = in && t > 0 ? Vp[(size_t)(t - 1) * ldp + i] : 0.0;
  const double zo = in && t > 0 ? Zp[(size_t)(t - 1) * ldp + i] : 0.0;
  double nrm = 0.0;
  if (in) {
#pragma unroll 4
    for (int64_t c = j + 1 + wave; c < r0; c += kSW) {
      double w = W[(size_t)c * ld + i];
      if (t > 0) w = fma(vo, Zp[(size_t)(t - 1) * ldp + c], fma(-zo, Vp[(size_t)(t - 1) * ldp + c], w));
      if (c == j + 1) {
        w = fma(v, znext, w - z);  // v_c = 1
        if (i >= j + 3) nrm = w * w;
      }
      W[(size_t)c * ld + i] = w;
    }
  }
  __syncthreads();
  if (wave == 0) {
    if (in) {
      W[(size_t)j * ld + i] = v;
      Vp[(size_t)t * ldp + i] = v;
      Zp[(size_t)t * ldp + i] = z;
    }
    if (more) {
      nrm = wave_sum64(nrm);
      if (lane == 0) pn[blockIdx.x] = nrm;
    }
  }
}

// Reduction of the last kSkewOne rows, one launch per column j.  The launch takes
// the reflection pair (v, z = tau p) of column j - 1 (vo, po) to the rest of the
// matrix, W += v z^T - z v^T, and forms p = W v of column j from the updated
// entries while it has them: the matrix is read and written once per column and
// nothing waits for a second launch.  Every workgroup applies the pair to column j
// and forms the reflector of it for itself (column j is not written in this launch;
// its v goes there in the next one).
//
// Bound by latency below some 1000 rows (4 us per column at order 512) and by the
// traffic of reading and writing the matrix in the caches above: order 2048 14.9 ms
// (7.3 us per column) against 23 ms in two launches with the updates blocked by 64
// columns.  Those read the matrix and write it 64 times less often, which wins
// above: order 3584 with the last 1536 / 2048 / 2560 / 3072 rows in this form 51.1 /
// 49.7 / 51.2 / 53.9 ms.  Whole columns go to a wave, or shares of one, so that
// loads are contiguous and the products end in one sum per column; few columns
// per wave and small workgroups are the better the shorter the columns (order
// 2048: 8 waves with 4 columns 14.9, 16 with 8 14.9, four columns per wave 15.5, 2
// columns per workgroup 18 to 19 ms).
constexpr int kSkewOne = 2048;
constexpr int kCW = 8;  // waves of a workgroup
constexpr int kSC = 4;  // columns of a workgroup
constexpr int kSN = 2;  // columns of a wave, so that v and z are read from LDS once for both
constexpr int kSB = 8;  // rows of a lane in flight

// x + v_i z_c - z_i v_c with both products rounded: W stays exactly skew
__device__ inline double skew_pair(double x, double vi, double zi, double vc, double zc) {
#pragma clang fp contract(off)
  const double a = vi * zc, b = zi * vc;
  return x + (a - b);
}

__global__ void __launch_bounds__(64 * kCW)
    skew_column_kernel(double* __restrict__ W, int64_t ld, int m, int j, const double* __restrict__ vo,
                       const double* __restrict__ po, double* __restrict__ vn, double* __restrict__ pn,
                       double* __restrict__ tau, double* __restrict__ e) {
  constexpr int HW = kCW * kSN / kSC;  // waves that share a column
  __shared__ double vs[kSkewOne], zs[kSkewOne], xs[kSkewOne];
  __shared__ double red[kCW], dot[kSN][kCW];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int L = m - j;  // rows and columns from j on; r, c below count from j
  const int c0 = 1 + blockIdx.x * kSC + wave / HW * kSN, r1 = 1 + wave % HW * 64;
  double* const col = W + (size_t)(j + c0) * ld + j;
  double w[kSB][kSN];
  auto load = [&](int rb) {
#pragma unroll
    for (int u = 0; u < kSB; ++u)
#pragma unroll
      for (int q = 0; q < kSN; ++q) {
        const int r = rb + u * 64 * HW + lane;
        w[u][q] = r < L && c0 + q < L ? col[(size_t)q * ld + r] : 0.0;
      }
  };
  load(r1);  // in flight while the reflector is formed
  const double* cj = W + (size_t)j * ld + j;
  const double tp = j > 0 ? tau[j - 1] : 0.0, zj = j > 0 ? tp * po[j] : 0.0;
  double acc = 0.0;
  for (int r = tid; r < L; r += 64 * kCW) {
    double x = cj[r];
    if (j > 0) {
      const double v = vo[j + r], z = tp * po[j + r];
      vs[r] = v;
      zs[r] = z;
      x = skew_pair(x, v, z, 1.0, zj);
    }
    xs[r] = x;
    if (r >= 2) acc = fma(x, x, acc);
  }
  acc = wave_sum_dpp(acc);
  if (lane == 0) red[wave] = acc;
  __syncthreads();
  double sig2 = red[0];
#pragma unroll
  for (int q = 1; q < kCW; ++q) sig2 += red[q];
  double beta, tj, sc;
  reflector(sig2, L > 1 ? xs[1] : 0.0, beta, tj, sc);
  if (blockIdx.x == 0) {
    if (j > 0)
      for (int r = tid; r < L; r += 64 * kCW) W[(size_t)(j - 1) * ld + j + r] = vs[r];
    for (int r = 1 + tid; r < L; r += 64 * kCW) vn[j + r] = r == 1 ? 1.0 : xs[r] * sc;
    if (tid == 0 && L > 1) {
      e[j] = beta;
      tau[j] = tj;
    }
  }
  double vc[kSN], zc[kSN], s[kSN];
#pragma unroll
  for (int q = 0; q < kSN; ++q) {
    const bool in = j > 0 && c0 + q < L;
    vc[q] = in ? vs[c0 + q] : 0.0;
    zc[q] = in ? zs[c0 + q] : 0.0;
    s[q] = 0.0;
  }
  // One batch covers the rows (asserted), so this runs at most once; written
  // without the loop and its reload a column took 7.7 us instead of 7.55 at order
  // 2048 (three traces of each)
  static_assert(kSB * 64 * HW >= kSkewOne, "a wave's share of the rows is one batch of loads");
  for (int rb = r1; rb < L; rb += kSB * 64 * HW) {
    if (rb != r1) load(rb);
#pragma unroll
    for (int u = 0; u < kSB; ++u) {
      const int r = rb + u * 64 * HW + lane;
      if (r >= L) continue;
      const double x = r == 1 ? 1.0 : xs[r] * sc;
      const double v = j > 0 ? vs[r] : 0.0, z = j > 0 ? zs[r] : 0.0;
#pragma unroll
      for (int q = 0; q < kSN; ++q) {
        if (c0 + q >= L) continue;
        double t = w[u][q];
        if (j > 0) {
          t = skew_pair(t, v, z, vc[q], zc[q]);
          col[(size_t)q * ld + r] = t;
        }
        s[q] = fma(t, x, s[q]);
      }
    }
  }
#pragma unroll
  for (int q = 0; q < kSN; ++q) {
    s[q] = wave_sum_dpp(s[q]);
    if (lane == 0) dot[q][wave] = s[q];
  }
  __syncthreads();
  if (tid < kSC) {  // column c of the workgroup: p_c = -(column c) . v
    const int c = 1 + blockIdx.x * kSC + tid;
    double t = 0.0;
    for (int q = 0; q < HW; ++q) t += dot[tid % kSN][tid / kSN * HW + q];
    if (c < L) pn[j + c] = -t;
  }
}

// Back-transformation of the eigenvectors, one workgroup per real column x
// of R (m rows): x <- H_0 H_1 ... H_{m-2} x with H_j = I - tau_j v_j v_j^T
// (v_j in W[j+1:, j]), then x <- L^{-T} x (L lower, in l).  Both are chains of m
// reductions over the workgroup and bound by their latency, so they go eight at
// a time: one reduction gives the eight products v_q . x and the 28 products v_q .
// v_r of a block of reflectors, from which every thread forms the eight steps
// y_q = tau_q (v_q . x - sum over the reflectors r applied before of y_r v_q . v_r);
// the solve takes the eight dot products of a block of rows with the solved part
// together and finishes the 8 x 8 triangle in one thread.  One reflector and
// one row at a time took 6.0 ms at order 2048, 2.0 ms here.
__global__ void __launch_bounds__(1024)
    skew_back_kernel(const double* __restrict__ W, int64_t ld, const double* __restrict__ tau,
                     const double* __restrict__ l, int64_t ldl, int64_t m, double* __restrict__ R, int64_t ldr) {
  constexpr int NB = 8, NG = NB * (NB - 1) / 2, NV = 48;  // 8 + 28 values, padded to three groups of 16
  __shared__ double red[16][NV];
  __shared__ double tot[NV];
  __shared__ double tri[NB][NB];
  double* x = R + (size_t)blockIdx.x * ldr;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  // pair (q, r), r > q -> 8 + gi(q, r)
  auto gi = [](int q, int r) { return NB + q * (2 * NB - q - 1) / 2 + (r - q - 1); };
  for (int64_t jb = (m - 2) / NB * NB; jb >= 0; jb -= NB) {  // reflectors jb .. jb + 7 (those below m - 1)
    double val[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) val[q] = 0.0;
    for (int64_t i = jb + 1 + tid; i < m; i += 1024) {
      double v[NB];
#pragma unroll
      for (int q = 0; q < NB; ++q) v[q] = jb + q < i ? W[(size_t)(jb + q) * ld + i] : 0.0;  // i < m: jb + q < m - 1
      const double xi = x[i];
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        val[q] = fma(v[q], xi, val[q]);
#pragma unroll
        for (int r = q + 1; r < NB; ++r) val[gi(q, r)] = fma(v[q], v[r], val[gi(q, r)]);
      }
    }
#pragma unroll
    for (int g = 0; g < NV / 16; ++g) {
      double t[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) t[q] = val[16 * g + q];
      red[wave][16 * g + wave_sum_index<16>(lane)] = wave_sum_n<16>(t);
    }
    __syncthreads();
    if (tid < NB + NG) {
      double t = 0.0;
#pragma unroll
      for (int w = 0; w < 16; ++w) t += red[w][tid];
      tot[tid] = t;
    }
    __syncthreads();
    double y[NB];
#pragma unroll
    for (int q = NB - 1; q >= 0; --q) {  // H_{jb+7} is applied first
      double d = tot[q];
#pragma unroll
      for (int r = q + 1; r < NB; ++r) d = fma(-y[r], tot[gi(q, r)], d);
      y[q] = (jb + q < m - 1 ? tau[jb + q] : 0.0) * d;
    }
    for (int64_t i = jb + 1 + tid; i < m; i += 1024) {
      double xi = x[i];
#pragma unroll
      for (int q = NB - 1; q >= 0; --q) xi = fma(-y[q], jb + q < i ? W[(size_t)(jb + q) * ld + i] : 0.0, xi);
      x[i] = xi;
    }
    __syncthreads();
  }
  // L^T x = b, backward, rows jb .. jb + 7 (those below m): x_j = (b_j - sum_{i > j} L_ij x_i) / L_jj
  for (int64_t jb = (m - 1) / NB * NB; jb >= 0; jb -= NB) {
    double val[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) val[q] = 0.0;
    for (int64_t i = jb + NB + tid; i < m; i += 1024) {
      const double xi = x[i];
#pragma unroll
      for (int q = 0; q < NB; ++q) val[q] = fma(l[(size_t)(jb + q) * ldl + i], xi, val[q]);
    }
    red[wave][wave_sum_index<NB>(lane)] = wave_sum_n<NB>(val);
    if (tid < NB * NB) {  // the block's triangle, identity past the last row
      const int q = tid / NB, r = tid % NB;
      tri[q][r] = jb + r < m && r >= q ? l[(size_t)(jb + q) * ldl + jb + r] : (q == r ? 1.0 : 0.0);
    }
    __syncthreads();
    if (tid == 0) {
      double xs[NB];
#pragma unroll
      for (int q = NB - 1; q >= 0; --q) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < 16; ++w) s += red[w][q];
#pragma unroll
        for (int r = q + 1; r < NB; ++r) s = fma(tri[q][r], xs[r], s);
        xs[q] = jb + q < m ? (x[jb + q] - s) / tri[q][q] : 0.0;
      }
#pragma unroll
      for (int q = 0; q < NB; ++q)
        if (jb + q < m) x[jb + q] = xs[q];
    }
    __syncthreads();
  }
}

unsigned grid_rows(int64_t rows) {
  const int64_t g = (rows + kT - 1) / kT;
  return (unsigned)(g < 1024 ? g : 1024);
}

}  // namespace

hipError_t direct_dense(const Layout& L, bool hilo, const MatPtrs& m, double2* ad, double* mr, int64_t ld,
                        hipStream_t s) {
  hipLaunchKernelGGL(dense_kernel, dim3((unsigned)L.nblk), dim3(kT), 0, s, L.blkmap, L.R, L.n, hilo ? 1 : 0, m.a,
                     m.alo, m.b, m.blo, ad, mr, ld);
  return hipGetLastError();
}

hipError_t direct_jl(double* l, int64_t ld, int64_t n, double* g, hipStream_t s) {
  hipLaunchKernelGGL(jl_kernel, dim3(grid_rows(2 * n), (unsigned)(2 * n)), dim3(kT), 0, s, l, ld, n, g);
  return hipGetLastError();
}

hipError_t direct_negi(const double* w, int64_t ld, int64_t n2, double2* z, int64_t ldz, hipStream_t s) {
  hipLaunchKernelGGL(negi_kernel, dim3(grid_rows(n2), (unsigned)n2), dim3(kT), 0, s, w, ld, n2, z, ldz);
  return hipGetLastError();
}

hipError_t direct_split(const double2* z, int64_t ldz, int64_t n2, int c0, int k, double* rm, int64_t ldr,
                        hipStream_t s) {
  hipLaunchKernelGGL(split_kernel, dim3(grid_rows(n2), (unsigned)k), dim3(kT), 0, s, z, ldz, n2, c0, k, rm, ldr);
  return hipGetLastError();
}

hipError_t direct_back(const double* rm, int64_t ldr, int64_t n, int k, double2* x, double2* y, int64_t ldo,
                       hipStream_t s) {
  hipLaunchKernelGGL(back_kernel, dim3(grid_rows(n), (unsigned)k), dim3(kT), 0, s, rm, ldr, n, k, x, y, ldo);
  return hipGetLastError();
}


hipError_t dense_gemm(int ta, int tb, int64_t M, int64_t N, int64_t K, double alpha, const double* A, int64_t lda,
                      const double* B, int64_t ldb, double beta, double* C, int64_t ldc, int lower, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  const dim3 grid((unsigned)((M + 63) / 64), (unsigned)((N + 63) / 64));
  if (ta == 0 && tb == 0)
    hipLaunchKernelGGL((gemm_kernel<0, 0>), grid, dim3(256), 0, s, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, lower);
  else if (ta == 0)
    hipLaunchKernelGGL((gemm_kernel<0, 1>), grid, dim3(256), 0, s, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, lower);
  else if (tb == 0)
    hipLaunchKernelGGL((gemm_kernel<1, 0>), grid, dim3(256), 0, s, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, lower);
  else
    hipLaunchKernelGGL((gemm_kernel<1, 1>), grid, dim3(256), 0, s, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, lower);
  return hipGetLastError();
}

hipError_t dense_cholesky(double* A, int64_t ld, int64_t m, int* flag, hipStream_t s) {
  for (int64_t j0 = 0; j0 < m; j0 += 64) {
    const int nb = (int)(m - j0 < 64 ? m - j0 : 64);
    hipLaunchKernelGGL(potrf_diag_kernel, dim3(1), dim3(256), 0, s, A, ld, j0, nb, flag);
    const int64_t rest = m - j0 - nb;
    if (rest <= 0) break;
    hipLaunchKernelGGL(trsm_panel_kernel, dim3((unsigned)((rest + 255) / 256)), dim3(256), 0, s, A, ld, j0, nb, m);
    // A22 -= L21 L21^T, lower triangle
    const double* l21 = A + (size_t)j0 * ld + j0 + nb;
    double* a22 = A + (size_t)(j0 + nb) * ld + j0 + nb;
    hipError_t e = dense_gemm(0, 1, rest, rest, nb, -1.0, l21, ld, l21, ld, 1.0, a22, ld, 1, s);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

hipError_t skew_tridiag(double* W, int64_t ld, int64_t m, double* Vp, double* Zp, int64_t ldp, double* part,
                        double* dots, double* tau, double* e, hipStream_t s) {
  constexpr int nb = 64;
  // behind the partial products: sc of the current reflector, the norm partials of the next one
  double* scp = part + (size_t)((m - 1 + 255) / 256) * m;
  double* pn = scp + 1;
  int64_t j0 = 0;
  for (; m - j0 > kSkewOne; j0 += nb) {
    const int64_t r0 = j0 + nb;
    int npn = (int)((m - j0 - 2 + 255) / 256);
    hipLaunchKernelGGL(skew_norm_kernel, dim3((unsigned)npn), dim3(256), 0, s, W, ld, m, j0, pn);
    for (int t = 0; t < nb; ++t) {
      const int64_t j = j0 + t, L = m - j - 1;
      const int nrow = (int)((L + 63) / 64), nchunk = (int)((L + 255) / 256);
      hipLaunchKernelGGL(skew_mv_kernel, dim3((unsigned)(nrow * nchunk + 2 * t)), dim3(64 * kSW), 0, s, W, ld, m, j, r0, t,
                         nrow, nchunk, pn, npn, Vp, Zp, ldp, part, dots, tau, e, scp);
      hipLaunchKernelGGL(skew_update_kernel, dim3((unsigned)nrow), dim3(64 * kSW), 0, s, W, ld, m, j, r0, t, nchunk, part,
                         dots, tau, scp, Vp, Zp, ldp, pn);
      npn = nrow;
    }
    // trailing W += Vp Zp^T - Zp Vp^T (rows and columns >= r0)
    const int64_t rest = m - r0;
    double* c = W + (size_t)r0 * ld + r0;
    hipError_t err = dense_gemm(0, 1, rest, rest, nb, 1.0, Vp + r0, ldp, Zp + r0, ldp, 1.0, c, ld, 0, s);
    if (err == hipSuccess) err = dense_gemm(0, 1, rest, rest, nb, -1.0, Zp + r0, ldp, Vp + r0, ldp, 1.0, c, ld, 0, s);
    if (err != hipSuccess) return err;
  }
  // the matrix that is left, which all pairs so far have been applied to; v and
  // p of the last column and of this one in two columns of Vp and Zp in turn
  double* Wr = W + (size_t)j0 * ld + j0;
  const int mr = (int)(m - j0);
  for (int j = 0; j < mr; ++j) {
    const int L = mr - j - 1;
    double *v0 = Vp + ((j + 1) & 1) * ldp, *p0 = Zp + ((j + 1) & 1) * ldp, *v1 = Vp + (j & 1) * ldp, *p1 = Zp + (j & 1) * ldp;
    hipLaunchKernelGGL(skew_column_kernel, dim3((unsigned)(L > 0 ? (L + kSC - 1) / kSC : 1)), dim3(64 * kCW), 0, s, Wr,
                       ld, mr, j, v0, p0, v1, p1, tau + j0, e + j0);
  }
  return hipGetLastError();
}

hipError_t skew_back(const double* W, int64_t ld, const double* tau, const double* l, int64_t ldl, int64_t m,
                     double* R, int64_t ldr, int ncol, hipStream_t s) {
  if (ncol <= 0) return hipSuccess;
  hipLaunchKernelGGL(skew_back_kernel, dim3((unsigned)ncol), dim3(1024), 0, s, W, ld, tau, l, ldl, m, R, ldr);
  return hipGetLastError();
}

hipError_t scale_cols(double2* x, double2* y, int64_t ld, int64_t n, int k, const double* f, hipStream_t s) {
  hipLaunchKernelGGL(scale_kernel, dim3(grid_rows(n), (unsigned)k), dim3(kT), 0, s, x, y, ld, n, f);
  return hipGetLastError();
}

}  // namespace bse
