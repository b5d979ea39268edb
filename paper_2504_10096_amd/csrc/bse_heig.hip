// Reduction of a dense complex Hermitian matrix to real tridiagonal form on the
// device, for the projected eigenproblems of the solves (orders of a hundred
// to a few hundred: ncv of the full-H iteration, the refinement's pencil).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bse_internal.h"

namespace bse {
namespace {

// A = Q T Q^H, Q = H_0 H_1 ... H_{m-2}, H_j = I - tau_j v_j v_j^H with v_j zero
// above row j + 1 and one there.  The reflector of a = A[j+1:, j] maps it to a
// real multiple of the first unit vector (H_j^H a = beta e_1):
//   beta = -sign(Re a_0) ||a||, tau = (beta - a_0)* / beta taken as
//   ((beta - Re a_0) / beta, -Im a_0 / beta), v = a / (a_0 - beta),
// and with p = A v, g = v^H A v, w = tau p - |tau|^2 g / 2 v the transformed
// trailing matrix is A - v w^H - w v^H.
//
// A chain of m columns with two sums over the whole column each (the norm, g), so
// two launches per column and nothing else: the time is their latency (the
// matrix sits in the caches; order 224: 0.8 MB).  The library's blocked
// reduction takes six launches per column: order 224 4.33 ms, 608 11.1 ms, against
// 2.09 and 7.7 ms here.  A is kept in full, so products and updates read columns only.
constexpr int kW = 16;  // waves per workgroup
constexpr int kRows = 64;

__device__ inline double wsum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ inline double2 cmul(double2 a, double2 b) {
  return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}

// pn[b] = sum of |A[i, 0]|^2 over the block's rows i >= 2.
__global__ void __launch_bounds__(64) heig_norm_kernel(const double2* __restrict__ A, int m, double* __restrict__ pn) {
  const int i = 2 + blockIdx.x * 64 + threadIdx.x;
  const double2 a = i < m ? A[i] : make_double2(0.0, 0.0);
  const double s = wsum(fma(a.x, a.x, a.y * a.y));
  if (threadIdx.x == 0) pn[blockIdx.x] = s;
}

// First launch of column j: 64 rows i > j per workgroup.  The reflector (every
// wave forms it from the npn norm partials), its v in column j of V, p = A v and
// the workgroup's share of g; workgroup 0 records d, e, tau.
__global__ void __launch_bounds__(64 * kW)
    heig_mv_kernel(const double2* __restrict__ A, int m, int j, const double* __restrict__ pn, int npn,
                   double2* __restrict__ V, double2* __restrict__ p, double* __restrict__ gpart,
                   double* __restrict__ d, double* __restrict__ e, double2* __restrict__ tau) {
  extern __shared__ double2 vs[];  // v_c, c = j + 1 .. m - 1, then the waves' sums
  __shared__ double2 red[kW][kRows];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const double2* a = A + (size_t)j * m;
  double s = 0.0;
  for (int q = lane; q < npn; q += 64) s += pn[q];
  const double sig2 = wsum(s);
  const double2 al = a[j + 1];
  double beta = al.x;
  double2 tj = make_double2(0.0, 0.0), sc = tj;
  if (sig2 != 0.0 || al.y != 0.0) {
    beta = -copysign(sqrt(fma(al.x, al.x, fma(al.y, al.y, sig2))), al.x);
    tj = make_double2((beta - al.x) / beta, -al.y / beta);
    const double dr = al.x - beta, den = fma(dr, dr, al.y * al.y);  // 1 / (a_0 - beta)
    sc = make_double2(dr / den, -al.y / den);
  }
  if (blockIdx.x == 0 && tid == 0) {
    d[j] = a[j].x;
    e[j] = beta;
    tau[j] = tj;
  }
  const int L = m - j - 1;
  for (int c = tid; c < L; c += 64 * kW) vs[c] = c == 0 ? make_double2(1.0, 0.0) : cmul(a[j + 1 + c], sc);
  __syncthreads();
  const int r = blockIdx.x * kRows + lane, i = j + 1 + r;
  const bool in = r < L;
  const int c0 = L * wave / kW, c1 = L * (wave + 1) / kW;
  double sx = 0.0, sy = 0.0;
  if (in) {
    const double2* row = A + (size_t)(j + 1) * m + i;
    int c = c0;
    for (; c + 8 <= c1; c += 8) {
      double2 w[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) w[u] = row[(size_t)(c + u) * m];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const double2 v = vs[c + u];
        sx = fma(w[u].x, v.x, fma(-w[u].y, v.y, sx));
        sy = fma(w[u].x, v.y, fma(w[u].y, v.x, sy));
      }
    }
    for (; c < c1; ++c) {
      const double2 w = row[(size_t)c * m], v = vs[c];
      sx = fma(w.x, v.x, fma(-w.y, v.y, sx));
      sy = fma(w.x, v.y, fma(w.y, v.x, sy));
    }
  }
  red[wave][lane] = make_double2(sx, sy);
  __syncthreads();
  if (wave != 0) return;
  double2 t = red[0][lane];
#pragma unroll
  for (int w = 1; w < kW; ++w) {
    t.x += red[w][lane].x;
    t.y += red[w][lane].y;
  }
  double g = 0.0;
  if (in) {
    const double2 v = vs[r];
    V[(size_t)j * m + i] = v;
    p[i] = t;
    g = fma(v.x, t.x, v.y * t.y);  // Re conj(v) p
  }
  g = wsum(g);
  if (lane == 0) gpart[blockIdx.x] = g;
}

// Second launch of column j: A -= v w^H + w v^H on 64 x 64 tiles of the trailing
// matrix (wave w the columns w, w + 16, ...); the tiles of column j + 1 leave its
// norm partials.
__global__ void __launch_bounds__(64 * kW)
    heig_update_kernel(double2* __restrict__ A, int m, int j, int nrow, const double2* __restrict__ V,
                       const double2* __restrict__ p, const double* __restrict__ gpart,
                       const double2* __restrict__ tau, double* __restrict__ pn) {
  __shared__ double2 wc[kRows], vc[kRows];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const double2 tj = tau[j];
  double s = 0.0;
  for (int q = lane; q < nrow; q += 64) s += gpart[q];
  const double h = 0.5 * fma(tj.x, tj.x, tj.y * tj.y) * wsum(s);
  const int L = m - j - 1;
  const double2* v0 = V + (size_t)j * m + j + 1;
  auto pair = [&](int r, double2& v, double2& w) {
    v = w = make_double2(0.0, 0.0);
    if (r < L) {
      v = v0[r];
      w = cmul(tj, p[j + 1 + r]);
      w.x = fma(-h, v.x, w.x);
      w.y = fma(-h, v.y, w.y);
    }
  };
  const int r = blockIdx.x * kRows + lane, cb = blockIdx.y * kRows;
  if (wave == 0) {
    double2 v, w;
    pair(cb + lane, v, w);
    vc[lane] = v;
    wc[lane] = w;
  }
  double2 v, w;
  pair(r, v, w);
  __syncthreads();
  double nrm = 0.0;
  if (r < L) {
#pragma unroll
    for (int u = 0; u < kRows / kW; ++u) {
      const int k = wave + kW * u, c = cb + k;
      if (c >= L) break;
      double2* q = A + (size_t)(j + 1 + c) * m + j + 1 + r;
      const double2 vk = vc[k], wk = wc[k];
      double2 x = *q;
      x.x -= fma(v.x, wk.x, v.y * wk.y) + fma(w.x, vk.x, w.y * vk.y);
      x.y -= fma(v.y, wk.x, -v.x * wk.y) + fma(w.y, vk.x, -w.x * vk.y);
      if (c == r) x.y = 0.0;
      *q = x;
      if (c == 0 && r >= 2) nrm = fma(x.x, x.x, x.y * x.y);
    }
  }
  if (blockIdx.y == 0 && wave == 0) {
    nrm = wsum(nrm);
    if (lane == 0) pn[blockIdx.x] = nrm;
  }
}

__global__ void heig_last_kernel(const double2* __restrict__ A, int m, double* __restrict__ d) {
  d[m - 1] = A[(size_t)m * m - 1].x;
}

}  // namespace

hipError_t herm_tridiag(int m, double2* A, double2* V, double* d, double* e, double2* tau, double2* work,
                        hipStream_t s) {
  if (m < 2 || m > kHermTridiagMax) return hipErrorInvalidValue;
  double2* p = work;
  double* gpart = (double*)(work + m);  // m values, then the norm partials
  double* pn = gpart + m;
  int npn = (m - 2 + 63) / 64;
  if (npn > 0) hipLaunchKernelGGL(heig_norm_kernel, dim3((unsigned)npn), dim3(64), 0, s, A, m, pn);
  for (int j = 0; j + 1 < m; ++j) {
    const int L = m - j - 1, nrow = (L + kRows - 1) / kRows;
    hipLaunchKernelGGL(heig_mv_kernel, dim3((unsigned)nrow), dim3(64 * kW), sizeof(double2) * L, s, A, m, j, pn, npn,
                       V, p, gpart, d, e, tau);
    hipLaunchKernelGGL(heig_update_kernel, dim3((unsigned)nrow, (unsigned)nrow), dim3(64 * kW), 0, s, A, m, j, nrow,
                       V, p, gpart, tau, pn);
    npn = nrow;
  }
  hipLaunchKernelGGL(heig_last_kernel, dim3(1), dim3(1), 0, s, A, m, d);
  return hipGetLastError();
}

}  // namespace bse
