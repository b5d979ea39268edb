// Reduction of a dense complex Hermitian matrix to real tridiagonal form on the
// device, for the projected eigenproblems of the solves (orders of a hundred
// to a few hundred: ncv of the full-H iteration, the refinement's pencil).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bse_internal.h"
#include "bse_wave.h"

namespace bse {
namespace {

// A = Q T Q^H, Q = H_0 H_1 ... H_{m-2}, H_j = I - tau_j v_j v_j^H with v_j zero
// above row j + 1 and one there.  The reflector of a = A[j+1:, j] maps it to a
// real multiple of the first unit vector (H_j^H a = beta e_1):
//   beta = -sign(Re a_0) ||a||, tau = (beta - a_0)* / beta taken as
//   ((beta - Re a_0) / beta, -Im a_0 / beta), v = a / (a_0 - beta)
// (a column whose squares may underflow counts as zero and has v = e_1, tau = 2:
// kEigTiny.  tau is never 0, not even where nothing is to be reduced: the
// library's blocked back-transformation divides by it and returns NaN),
// and with p = A v, g = v^H A v, w = tau p - |tau|^2 g / 2 v the transformed
// trailing matrix is A - v w^H - w v^H.
//
// A chain of m columns with two sums over the whole column each (the norm, g): the
// time is latency (the matrix sits in the caches; order 224: 0.8 MB).  One launch
// per column: it takes the pair (v, w) of column j - 1 to the rest of the matrix
// and forms p = A v of column j from the updated entries while it has them.  Every
// workgroup applies the pair to column j and forms its reflector for itself
// (column j is not written in this launch).  A is kept in full, so that a wave reads
// columns only.  Order 224 takes 1.07 ms, 608 3.5; in two launches per column (product,
// then update) 2.09 and 7.7, by the library's blocked reduction with six 4.33 and
// 11.1.  8 waves with 8 columns: 1.13 and 3.9 ms, two columns per wave 1.21 and 3.8.
constexpr int kW = 8;  // waves of a workgroup
constexpr int kC = 4;  // columns of a workgroup
constexpr int kB = 4;  // rows of a lane in flight

__device__ inline double2 cmul(double2 a, double2 b) {
  return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}

// x - v_i w_c^* - w_i v_c^*
__device__ inline double2 pair_sub(double2 x, double2 vi, double2 wi, double2 vc, double2 wc) {
  x.x -= fma(vi.x, wc.x, vi.y * wc.y) + fma(wi.x, vc.x, wi.y * vc.y);
  x.y -= fma(vi.y, wc.x, -vi.x * wc.y) + fma(wi.y, vc.x, -wi.x * vc.y);
  return x;
}

// Column j: po, go (ngo shares of g) of column j - 1, pn, gn those of column j.
__global__ void __launch_bounds__(64 * kW)
    heig_column_kernel(double2* __restrict__ A, int m, int j, double2* __restrict__ V, const double2* __restrict__ po,
                       double2* __restrict__ pn, const double* __restrict__ go, int ngo, double* __restrict__ gn,
                       double* __restrict__ d, double* __restrict__ e, double2* __restrict__ tau) {
  constexpr int HW = kW / kC;  // waves that share a column
  __shared__ double2 vs[kHermTridiagMax], ws[kHermTridiagMax], xs[kHermTridiagMax];
  __shared__ double red[kW];
  __shared__ double2 dot[kW];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int L = m - j;  // rows and columns from j on; r, c below count from j
  const int c0 = 1 + blockIdx.x * kC + wave / HW, r1 = 1 + wave % HW * 64;
  double2* const col = A + (size_t)(j + c0) * m + j;
  double2 a[kB];
  auto load = [&](int rb) {
#pragma unroll
    for (int u = 0; u < kB; ++u) {
      const int r = rb + u * 64 * HW + lane;
      a[u] = r < L && c0 < L ? col[r] : make_double2(0.0, 0.0);
    }
  };
  load(r1);  // in flight while the reflector is formed
  const double2* cj = A + (size_t)j * m + j;
  double2 tp = make_double2(0.0, 0.0), w0 = tp;
  double h = 0.0;
  if (j > 0) {
    tp = tau[j - 1];
    double s = 0.0;
    for (int q = lane; q < ngo; q += 64) s += go[q];
    h = 0.5 * fma(tp.x, tp.x, tp.y * tp.y) * wave_sum_dpp(s);
    w0 = cmul(tp, po[j]);
    w0.x -= h;  // v_0 = 1
  }
  double acc = 0.0;
  for (int r = tid; r < L; r += 64 * kW) {
    double2 x = cj[r];
    if (j > 0) {
      const double2 v = V[(size_t)(j - 1) * m + j + r];
      double2 w = cmul(tp, po[j + r]);
      w.x = fma(-h, v.x, w.x);
      w.y = fma(-h, v.y, w.y);
      vs[r] = v;
      ws[r] = w;
      x = pair_sub(x, v, w, make_double2(1.0, 0.0), w0);
    }
    xs[r] = x;
    if (r >= 2) acc += fma(x.x, x.x, x.y * x.y);
  }
  acc = wave_sum_dpp(acc);
  if (lane == 0) red[wave] = acc;
  __syncthreads();
  double sig2 = red[0];
#pragma unroll
  for (int q = 1; q < kW; ++q) sig2 += red[q];
  const double2 al = L > 1 ? xs[1] : make_double2(0.0, 0.0);
  double beta = -al.x;
  double2 tj = make_double2(2.0, 0.0), sc = make_double2(0.0, 0.0);
  const double nrm2 = fma(al.x, al.x, fma(al.y, al.y, sig2));
  if (nrm2 >= kEigTiny) {
    beta = -copysign(sqrt(nrm2), al.x);
    tj = make_double2((beta - al.x) / beta, -al.y / beta);
    const double dr = al.x - beta, den = fma(dr, dr, al.y * al.y);  // 1 / (a_0 - beta)
    sc = make_double2(dr / den, -al.y / den);
  }
  auto refl = [&](int r) { return r == 1 ? make_double2(1.0, 0.0) : cmul(xs[r], sc); };
  if (blockIdx.x == 0) {
    for (int r = 1 + tid; r < L; r += 64 * kW) V[(size_t)j * m + j + r] = refl(r);
    if (tid == 0) {
      d[j] = xs[0].x;
      if (L > 1) {
        e[j] = beta;
        tau[j] = tj;
      }
    }
  }
  const bool in = j > 0 && c0 < L;
  const double2 vc = in ? vs[c0] : make_double2(0.0, 0.0), wc = in ? ws[c0] : make_double2(0.0, 0.0);
  double2 s = make_double2(0.0, 0.0);
  for (int rb = r1; rb < L; rb += kB * 64 * HW) {
    if (rb != r1) load(rb);
#pragma unroll
    for (int u = 0; u < kB; ++u) {
      const int r = rb + u * 64 * HW + lane;
      if (r >= L || c0 >= L) continue;
      const double2 x = refl(r);
      double2 t = a[u];
      if (j > 0) {
        t = pair_sub(t, vs[r], ws[r], vc, wc);
        if (r == c0) t.y = 0.0;
        col[r] = t;
      }
      s.x = fma(t.x, x.x, fma(t.y, x.y, s.x));  // t^* x
      s.y = fma(t.x, x.y, fma(-t.y, x.x, s.y));
    }
  }
  s.x = wave_sum_dpp(s.x);
  s.y = wave_sum_dpp(s.y);
  if (lane == 0) dot[wave] = s;
  __syncthreads();
  if (wave != 0) return;
  double g = 0.0;
  const int c = 1 + blockIdx.x * kC + lane;
  if (lane < kC && c < L) {
    double2 t = dot[lane * HW];
#pragma unroll
    for (int q = 1; q < HW; ++q) {
      const double2 u = dot[lane * HW + q];
      t.x += u.x;
      t.y += u.y;
    }
    pn[j + c] = t;
    const double2 v = refl(c);
    g = fma(v.x, t.x, v.y * t.y);  // Re v^* p
  }
  g = wave_sum_dpp(g);
  if (lane == 0) gn[blockIdx.x] = g;
}

}  // namespace

hipError_t herm_tridiag(int m, double2* A, double2* V, double* d, double* e, double2* tau, double2* work,
                        hipStream_t s) {
  if (m < 2 || m > kHermTridiagMax) return hipErrorInvalidValue;
  // p and the shares of g, of the last column and of this one in turn
  double2* p[2] = {work, work + m};
  double* g[2] = {(double*)(work + 2 * (size_t)m), (double*)(work + 2 * (size_t)m) + m};
  int ng = 0;
  for (int j = 0; j < m; ++j) {
    const int L = m - j - 1, nwg = L > 0 ? (L + kC - 1) / kC : 1;
    hipLaunchKernelGGL(heig_column_kernel, dim3((unsigned)nwg), dim3(64 * kW), 0, s, A, m, j, V, p[(j + 1) & 1],
                       p[j & 1], g[(j + 1) & 1], ng, g[j & 1], d, e, tau);
    ng = nwg;
  }
  return hipGetLastError();
}

}  // namespace bse
