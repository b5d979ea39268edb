// HIP kernels of the structured BSE eigensolver, written for gfx950 (CDNA4,
// 64-wide wavefronts).
//
// The pass over the stored triangles (matvec) is the hot spot of the method
// (Sec. 2.2.2 of the paper): it is HBM-bound at 1-2 flop/byte, so the design
// goal is to stream every stored block exactly once with fully coalesced
// loads and keep everything else small next to it.
#include <hip/hip_runtime.h>
#include <type_traits>
#include <math.h>

#include <algorithm>

#include "bse_internal.h"
#include "bse_wave.h"

namespace bse {

namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Block-wide sum (256 threads) in a fixed order: deterministic.
__device__ double block_sum(double v, double* sh) {
  v = wave_sum(v);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  __syncthreads();
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  double t = sh[0] + sh[1] + sh[2] + sh[3];
  __syncthreads();
  return t;
}

// ---------------------------------------------------------------- storage
// Matrix blocks are streamed once per pass: nontemporal loads keep them from
// evicting the (reused) vectors and partials from the caches.
typedef double nd2 __attribute__((ext_vector_type(2)));
typedef float nf2 __attribute__((ext_vector_type(2)));

typedef float nf4 __attribute__((ext_vector_type(4)));

// arithmetic type of a pass
template <int AR>
struct Elem {
  using T = double;
};
template <>
struct Elem<AR_HI> {
  using T = float;
};

// ----------------------------------------------------------------- matvec
//
// One workgroup (4 waves) per stored R x R block (P, Q), R >= 128 (block edge
// 64: tile64_kernel).  In each column a lane owns VW adjacent rows per
// 64 VW-row group (VW = 2 for the complex64 triangles: 16-byte loads), so
// every load instruction reads one contiguous 64 VW-entry segment.  The lane
// adds A_rc x_c into its row accumulators and conj(A_rc) x_r into the column
// sum, which a wavefront reduction completes.  Row sums of the four waves are
// combined through LDS.  Outputs are per-block partial vectors in FP64 (rows:
// rowpart[blk][R]; columns: colpart[blk][slice][R]); mv_reduce_kernel sums
// them in a fixed order, so the result is deterministic and each block is read
// once.
// entries per lane-load: two complex64 (16 bytes) where a slice has >= 128 rows
template <int R, int AR>
struct MvShape {
  static constexpr int RS = R;
  static constexpr int NS = R / RS;
  static constexpr int VW = (AR != AR_C128 && RS >= 128) ? 2 : 1;
  static constexpr int G = RS / (64 * VW);
  static constexpr int RPL = G * VW;
};

// Wavefront sum with DPP row shifts and row broadcasts (no LDS traffic);
// the total is returned to every lane (read from lane 63).
__device__ __forceinline__ double dpp_shift(double v, int ctrl_id) {
  // the DPP control must be a constant: dispatch on the few used here
  const int lo = __double2loint(v), hi = __double2hiint(v);
  int rlo, rhi;
  switch (ctrl_id) {
    case 0:
      rlo = __builtin_amdgcn_update_dpp(0, lo, 0x111, 0xf, 0xf, false);  // row_shr:1
      rhi = __builtin_amdgcn_update_dpp(0, hi, 0x111, 0xf, 0xf, false);
      break;
    case 1:
      rlo = __builtin_amdgcn_update_dpp(0, lo, 0x112, 0xf, 0xf, false);  // row_shr:2
      rhi = __builtin_amdgcn_update_dpp(0, hi, 0x112, 0xf, 0xf, false);
      break;
    case 2:
      rlo = __builtin_amdgcn_update_dpp(0, lo, 0x114, 0xf, 0xf, false);  // row_shr:4
      rhi = __builtin_amdgcn_update_dpp(0, hi, 0x114, 0xf, 0xf, false);
      break;
    case 3:
      rlo = __builtin_amdgcn_update_dpp(0, lo, 0x118, 0xf, 0xf, false);  // row_shr:8
      rhi = __builtin_amdgcn_update_dpp(0, hi, 0x118, 0xf, 0xf, false);
      break;
    case 4:
      rlo = __builtin_amdgcn_update_dpp(0, lo, 0x142, 0xa, 0xf, false);  // row_bcast:15
      rhi = __builtin_amdgcn_update_dpp(0, hi, 0x142, 0xa, 0xf, false);
      break;
    default:
      rlo = __builtin_amdgcn_update_dpp(0, lo, 0x143, 0xc, 0xf, false);  // row_bcast:31
      rhi = __builtin_amdgcn_update_dpp(0, hi, 0x143, 0xc, 0xf, false);
      break;
  }
  return __hiloint2double(rhi, rlo);
}

__device__ __forceinline__ double dpp_wave_sum(double v) {
  v += dpp_shift(v, 0);
  v += dpp_shift(v, 1);
  v += dpp_shift(v, 2);
  v += dpp_shift(v, 3);
  v += dpp_shift(v, 4);
  v += dpp_shift(v, 5);
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
  return __hiloint2double(hi, lo);
}

// Wave-local LDS between lanes of one wavefront: the writes of every lane
// are ordered before the reads that follow (no workgroup barrier).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Column sums of NV per-lane partials (4 <= NV <= 16) over the 64 lanes of
// a wavefront, through LDS instead of NV separate wavefront reductions:
// every lane writes its partials value-major to stage (row stride
// stage_ld(NV) doubles); lane (j, p) = (lane / LPV, lane % LPV), with LPV =
// 64 / NP and NP = NV rounded up to 4, 8 or 16, adds value j of lanes p,
// p + LPV, ..., p + (NP - 1) LPV; a DPP butterfly over the LPV lanes of
// value j (lane xor 1, xor 2, then mirror within 8 and within 16 as LPV
// requires) completes the sum (lds_group_sum returns it in every lane of
// group j; the caller syncs before the stage is written again), which
// lds_colsum stores to colsum[j * 64 + c].  Fixed order: deterministic.
// colsum holds (NV + 1) rows of 64 when NV < NP.
// The stride puts the lanes of each 16-lane read phase on distinct banks
// (72 for two value groups per phase, 68 for four).
__host__ __device__ constexpr int colsum_np(int nv) { return nv <= 4 ? 4 : (nv <= 8 ? 8 : 16); }
__host__ __device__ constexpr int stage_ld(int nv) { return colsum_np(nv) == 16 ? 68 : 72; }
// doubles of LDS per wave for NV values: the stage and the column sums
__host__ __device__ constexpr int colsum_lds(int nv) { return nv * stage_ld(nv) + (nv + 1) * 64; }
template <int NV>
__device__ __forceinline__ double lds_group_sum(const double (&v)[NV], double* stage, int lane) {
  static_assert(NV >= 4 && NV <= 16, "lds_colsum: 4..16 values");
  constexpr int NP = colsum_np(NV);
  constexpr int LPV = 64 / NP;
  constexpr int LD = stage_ld(NV);
#pragma unroll
  for (int j = 0; j < NV; ++j) stage[j * LD + lane] = v[j];
  wave_lds_sync();
  const int j = lane / LPV, p = lane % LPV;
  const int jj = j < NV ? j : 0;
  double t[NP];
#pragma unroll
  for (int m = 0; m < NP; ++m) t[m] = stage[jj * LD + p + LPV * m];
  // pairwise: depth log2 NP instead of a chain of NP - 1 dependent adds
#pragma unroll
  for (int h = NP / 2; h >= 1; h /= 2)
#pragma unroll
    for (int m = 0; m < h; ++m) t[m] += t[m + h];
  double s = t[0];
  s += dpp_f64<0xB1>(s);                     // quad_perm [1,0,3,2]: lane xor 1
  s += dpp_f64<0x4E>(s);                     // quad_perm [2,3,0,1]: lane xor 2
  if (LPV >= 8) s += dpp_f64<0x141>(s);      // row_half_mirror: 8-lane groups
  if (LPV == 16) s += dpp_f64<0x140>(s);     // row_mirror: 16-lane rows
  return s;
}
template <int NV>
__device__ __forceinline__ void lds_colsum(const double (&v)[NV], double* stage, double* colsum, int c,
                                           int lane) {
  constexpr int LPV = 64 / colsum_np(NV);
  const double s = lds_group_sum<NV>(v, stage, lane);
  // every lane of a group stores the same sum (no branch); the padding
  // groups of NV < NP store to row NV, which is never read
  const int j = lane / LPV;
  colsum[(j < NV ? j : NV) * 64 + c] = s;
  wave_lds_sync();
}

// acc += a b with one rounding; the multi-vector kernels accumulate every
// product this way (a separate multiply and add per product, as plain
// expressions compile to, costs half again the VALU work of these
// VALU-heavy loops)
__device__ __forceinline__ void mac(double& acc, double a, double b) { acc = __builtin_fma(a, b, acc); }
__device__ __forceinline__ void mac(float& acc, float a, float b) { acc = __builtin_fmaf(a, b, acc); }

// Raw 16-byte loads of one column segment: complex64 pairs (hi, and lo for
// HILO) or one complex128 entry; converted after the next column's loads
// have been issued.
template <int AR>
struct RawCol;
template <>
struct RawCol<AR_HI> {
  nf4 h;
};
template <>
struct RawCol<AR_HI64> {
  nf4 h;
};
template <>
struct RawCol<AR_HILO> {
  nf4 h, l;
};
template <>
struct RawCol<AR_C128> {
  nd2 h;
};

template <int AR>
__device__ __forceinline__ void raw_load(const void* p, const void* q, size_t i, RawCol<AR>& r) {
  if constexpr (AR == AR_C128) {
    r.h = __builtin_nontemporal_load(static_cast<const nd2*>(p) + i);
  } else {
    r.h = __builtin_nontemporal_load(reinterpret_cast<const nf4*>(static_cast<const nf2*>(p) + i));
    if constexpr (AR == AR_HILO)
      r.l = __builtin_nontemporal_load(reinterpret_cast<const nf4*>(static_cast<const nf2*>(q) + i));
  }
}

template <int AR, typename T>
__device__ __forceinline__ void raw_get(const RawCol<AR>& r, int e, T& re, T& im) {
  if constexpr (AR == AR_C128) {
    re = r.h.x;
    im = r.h.y;
  } else if constexpr (AR == AR_HILO) {
    re = e ? (double)r.h.z + (double)r.l.z : (double)r.h.x + (double)r.l.x;
    im = e ? (double)r.h.w + (double)r.l.w : (double)r.h.y + (double)r.l.y;
  } else {
    re = (T)(e ? r.h.z : r.h.x);
    im = (T)(e ? r.h.w : r.h.y);
  }
}

// One-vector pass, streaming form: the four waves interleave columns (wave w
// takes columns w, w + 4, ...), the loads of a wave's next column are issued
// before its current one is consumed (two columns in flight per wave in
// registers), the column sums use DPP reductions, and they are kept one per
// lane and stored per 64 columns, so the column loop has no branches.
template <int R, int AR, int BM>
__global__ void __launch_bounds__(kThreads)
    mv_stream_kernel(const void* __restrict__ a0, const void* __restrict__ a1,
                     const void* __restrict__ b0, const void* __restrict__ b1,
                     const int2* __restrict__ blkmap, int64_t n, const double2* __restrict__ va,
                     int conja, const double2* __restrict__ vb, int conjb, double sb,
                     double2* __restrict__ rowpart, double2* __restrict__ colpart) {
  using T = typename Elem<AR>::T;
  using Sh = MvShape<R, AR>;
  constexpr int RS = Sh::RS, NS = Sh::NS, VW = Sh::VW, G = Sh::G, RPL = Sh::RPL;
  constexpr int CPW = R / 4;
  constexpr int CH = CPW < 64 ? CPW : 64;
  static_assert(AR == AR_C128 ? VW == 1 : VW == 2, "stream layout (R >= 128)");
  __shared__ double2 sh[4][RS];

  const int blk = blockIdx.x;
  const int slice = blockIdx.y;
  const int2 pq = blkmap[blk];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int64_t row0 = (int64_t)pq.x * R + slice * RS, col0 = (int64_t)pq.y * R;
  const size_t base = (size_t)blk * R * R + (size_t)slice * RS;
  const T ca = conja ? T(-1) : T(1);
  const T cbs = conjb ? T(-1) : T(1);
  const T tsb = (T)sb;

  T xar[RPL], xai[RPL], xbr[RPL], xbi[RPL], rr[RPL], ri[RPL];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int e = 0; e < VW; ++e) {
      const int q = g * VW + e;
      const int64_t i = row0 + g * 64 * VW + lane * VW + e;
      const bool in = i < n;
      const int64_t ii = in ? i : 0;
      double2 v = va[ii], w = make_double2(0.0, 0.0);
      if (BM == BM_EXPLICIT) w = vb[ii];
      xar[q] = in ? (T)v.x : T(0);
      xai[q] = in ? ca * (T)v.y : T(0);
      xbr[q] = (BM == BM_EXPLICIT && in) ? tsb * (T)w.x : T(0);
      xbi[q] = (BM == BM_EXPLICIT && in) ? tsb * cbs * (T)w.y : T(0);
      rr[q] = T(0);
      ri[q] = T(0);
    }

  // the four waves interleave columns (wave w takes columns 4 cc + w), so a
  // workgroup reads 4 adjacent columns, 16 KB of each array, at a time
  const size_t lbase = base + (size_t)wave * R + lane * VW;
  RawCol<AR> ca_[G], cbm[G], na_[G], nbm[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    raw_load<AR>(a0, a1, lbase + g * 64 * VW, ca_[g]);
    if (BM != BM_NONE) raw_load<AR>(b0, b1, lbase + g * 64 * VW, cbm[g]);
  }
  for (int cb = 0; cb < CPW; cb += CH) {
    double2 keep = make_double2(0.0, 0.0);
#pragma unroll 2
    for (int c2 = 0; c2 < CH; ++c2) {
      const int cc = cb + c2;
      // next column's loads first (the last column reloads itself: in bounds)
      const int cn = cc + 1 < CPW ? cc + 1 : cc;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        raw_load<AR>(a0, a1, lbase + (size_t)cn * 4 * R + g * 64 * VW, na_[g]);
        if (BM != BM_NONE) raw_load<AR>(b0, b1, lbase + (size_t)cn * 4 * R + g * 64 * VW, nbm[g]);
      }
      const int c = cc * 4 + wave;
      const int64_t j = col0 + c;
      const bool in = j < n;
      const int64_t jj = in ? j : 0;
      double2 vj = va[jj], wj = make_double2(0.0, 0.0);
      if (BM == BM_EXPLICIT) wj = vb[jj];
      const T xcr = in ? (T)vj.x : T(0), xci = in ? ca * (T)vj.y : T(0);
      T ycr = T(0), yci = T(0);
      if (BM == BM_CONJ) {
        ycr = tsb * xcr;
        yci = -tsb * xci;
      } else if (BM == BM_EXPLICIT) {
        ycr = in ? tsb * (T)wj.x : T(0);
        yci = in ? tsb * cbs * (T)wj.y : T(0);
      }
      T cr = T(0), ci = T(0), dr = T(0), di = T(0);
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < VW; ++e) {
          const int q = g * VW + e;
          T ar, ai;
          raw_get<AR, T>(ca_[g], e, ar, ai);
          mac(rr[q], ar, xcr);
          mac(rr[q], -ai, xci);
          mac(ri[q], ar, xci);
          mac(ri[q], ai, xcr);
          mac(cr, ar, xar[q]);
          mac(cr, ai, xai[q]);
          mac(ci, ar, xai[q]);
          mac(ci, -ai, xar[q]);
          if (BM != BM_NONE) {
            T br, bi;
            raw_get<AR, T>(cbm[g], e, br, bi);
            mac(rr[q], br, ycr);
            mac(rr[q], -bi, yci);
            mac(ri[q], br, yci);
            mac(ri[q], bi, ycr);
            if (BM == BM_CONJ) {
              mac(dr, br, xar[q]);
              mac(dr, bi, xai[q]);
              mac(di, bi, xar[q]);
              mac(di, -br, xai[q]);
            } else {
              mac(dr, br, xbr[q]);
              mac(dr, -bi, xbi[q]);
              mac(di, br, xbi[q]);
              mac(di, bi, xbr[q]);
            }
          }
        }
      if (BM == BM_CONJ) {
        cr += tsb * dr;
        ci += tsb * di;
      } else if (BM == BM_EXPLICIT) {
        cr += dr;
        ci += di;
      }
      const double sr = dpp_wave_sum((double)cr), si = dpp_wave_sum((double)ci);
      keep = lane == c2 ? make_double2(sr, si) : keep;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        ca_[g] = na_[g];
        if (BM != BM_NONE) cbm[g] = nbm[g];
      }
    }
    if (lane < CH) colpart[((size_t)blk * NS + slice) * R + (cb + lane) * 4 + wave] = keep;
  }

#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int e = 0; e < VW; ++e) {
      const int q = g * VW + e;
      sh[wave][g * 64 * VW + lane * VW + e] = make_double2((double)rr[q], (double)ri[q]);
    }
  __syncthreads();
  for (int r = threadIdx.x; r < RS; r += kThreads) {
    double2 t = sh[0][r];
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      t.x += sh[w][r].x;
      t.y += sh[w][r].y;
    }
    rowpart[(size_t)blk * R + slice * RS + r] = t;
  }
}

// Partial sums of one output: row i = P R + r takes the row partials of blocks
// (P, Q >= P) and the column partials of blocks (Q <= P, P), slice by slice,
// nb + 1 terms for NS = 1.  They are cut into W consecutive ranges: lane l of
// wave w sums range w of row blockIdx.x * 64 + l in order, the W range sums
// are added in wave order (fixed order: deterministic).  A workgroup covers
// 64 rows of one panel (R is a multiple of 64), so the loop bounds are uniform
// per wave.
//
// The sums are a latency chain, not a bandwidth problem: one thread per row
// with all its terms left 41 x 2 workgroups of serial loads at N = 10368
// (82 terms; 54 us beside 163 us for the read of the triangles).  Read and sum
// of two full-H vectors there: 219 us before, 178 us with 16 waves per 64 rows.
// W = 16 up to kReduceWide rows, where 64-row workgroups of four waves do not
// fill the chip, if each wave has a term (nb >= 16); W = 4 otherwise (N = 320,
// six terms: 11.5 us per small pass with four waves, 12.8 us with 16).  From 18001 to
// 40000 rows the two differ by less than runs of one do (four full-H vectors on
// hi: 580 to 585 us at 18001, 2831 to 2838 at 40000, with either).
constexpr int64_t kReduceWide = 32768;
inline bool reduce_wide(const Layout& L) { return L.n <= kReduceWide && L.nb >= 16; }
template <int W>
__device__ __forceinline__ void part_range(const double2* __restrict__ rp, const double2* __restrict__ cp, int R,
                                           int NS, int nb, int P, int r, int wave, double& sx, double& sy) {
  const int nrow = nb - P;
  const int len = nrow + (P + 1) * NS;
  const int t0 = (int)((int64_t)len * wave / W), t1 = (int)((int64_t)len * (wave + 1) / W);
  const int64_t pstart = (int64_t)P * nb - (int64_t)P * (P - 1) / 2;
  const int te = t1 < nrow ? t1 : nrow;
#pragma unroll 4
  for (int t = t0; t < te; ++t) {  // row partials, Q = P + t
    const double2 v = rp[(size_t)(pstart + t) * R + r];
    sx += v.x;
    sy += v.y;
  }
#pragma unroll 4
  for (int t = (t0 > nrow ? t0 : nrow); t < t1; ++t) {  // column partials, u = Q NS + slice
    const int u = t - nrow;
    const int Q = NS == 1 ? u : u / NS, sl = u - Q * NS;
    const int64_t qs = (int64_t)Q * nb - (int64_t)Q * (Q - 1) / 2;
    const double2 v = cp[((size_t)(qs + (P - Q)) * NS + sl) * R + r];
    sx += v.x;
    sy += v.y;
  }
}

// Sum over the waves of one value pair per lane, in wave order; the result is
// valid in wave 0.
template <int W>
__device__ __forceinline__ double2 wave_order_sum(double2 (*sh)[64], int wave, int lane, double sx, double sy) {
  __syncthreads();  // the array may still be read for the previous output
  sh[wave][lane] = make_double2(sx, sy);
  __syncthreads();
  double2 t = make_double2(0.0, 0.0);
  if (wave == 0) {
    t = sh[0][lane];
#pragma unroll
    for (int w = 1; w < W; ++w) {
      t.x += sh[w][lane].x;
      t.y += sh[w][lane].y;
    }
  }
  return t;
}

// One-vector pass: out[i] = the sum of row i's partials (+ the diagonal
// correction on the A input).
template <int W>
__global__ void __launch_bounds__(64 * W)
    mv_reduce_kernel(const double2* __restrict__ rowpart, const double2* __restrict__ colpart,
                     int R, int NS, int nb, int64_t n, double2* __restrict__ out, const double* __restrict__ dc,
                     double dsg, const double2* __restrict__ xa, int conja) {
  __shared__ double2 sh[W][64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t i0 = (int64_t)blockIdx.x * 64, i = i0 + lane;
  double sx = 0.0, sy = 0.0;
  // partial rows past n exist (the blocks are padded)
  part_range<W>(rowpart, colpart, R, NS, nb, (int)(i0 / R), (int)(i0 % R) + lane, wave, sx, sy);
  double2 t = wave_order_sum<W>(sh, wave, lane, sx, sy);
  if (wave == 0 && i < n) {
    if (dc) {  // diagonal correction on the A input
      const double f = dsg * dc[i];
      const double2 x = xa[i];
      t.x = fma(f, x.x, t.x);
      t.y = fma(f, conja ? -x.y : x.y, t.y);
    }
    out[i] = t;
  }
}

// ------------------------------------------- small matrices: 64 x 64 blocks
//
// Every product of a pass on block edge 64 (N up to 5632): one workgroup
// per stored block, lane = row, wave w the CPW columns [w CPW, (w + 1) CPW) of
// the block.  MODE: T64_A rows A x, T64_K A x + sb B conj(x) through the real
// 2 x 2 block of the entry pair (as in mk_block_kernel), T64_E A x + B y with
// an explicit y, T64_H the full-H product of NV / 2 vectors [x; y]: output 2p is
// A x + B y, output 2p + 1 the conjugate of the bottom, A conj(y) + B conj(x).
// Both are summed from A and B themselves.  In the sum / difference basis of the
// larger blocks (u = x + conj(y), w = x - conj(y), halves of K1 u +- K2 w) the
// products are half as many, but each half is accurate only to eps (|A| + |B|)
// (|x| + |y|): with y = 0, |A| = 13 and |B| = 0.25 the bottom B conj(x) had an
// error of 3.8e-14 of its largest entry at N = 400, 2.3e-16 this way.
//
// What bounds it: below N = 1500 or so the latency of one block's loads and
// column sums, above it the loads; with the column sums as one six-step
// wavefront sum per value (18 instructions each) it was bound by those sums.
// Here a wave sums 16 values at once: four exchange steps (lanes 32, 16, 8
// and 4 apart) each halve the number of registers instead of summing the same
// value in every lane, so 16 values take 57 instructions.  All loads of a wave's
// columns are issued before the first is used (8 columns ahead where A and B
// take 32 bytes per entry pair, 4 with eight half-vectors, to fit the registers;
// held to two waves per SIMD there with 13 registers spilled, 104 -> 86 us for four
// vectors of H in complex128 at N = 4096).
// Eight waves of 8 columns instead of four of 16 gained 3 % at N <= 1024 and
// lost up to 45 % above.  Times of a pass with its sum, before and after (us):
//   N = 1024 complex128: A x 16.0 -> 6.5, H x four vectors 68 -> 16
//   N = 4096 complex128: K1 64 -> 45 (268 MB), A x four 202 -> 40
//   N = 4096 hi: K1 53 -> 27 (134 MB), H x four vectors 330 -> 77
// (H: 67 in the sum / difference basis; 2001, complex128, three vectors 101 -> 30,
// 28 there).
enum { T64_A = 0, T64_K = 1, T64_E = 2, T64_H = 3 };

template <int AR>
struct Raw1 {
  nf2 h, l;  // complex64 hi, and lo for HILO
};
template <>
struct Raw1<AR_C128> {
  nd2 h;
};
template <int AR>
__device__ __forceinline__ void raw1_load(const void* p, const void* q, size_t i, Raw1<AR>& r) {
  if constexpr (AR == AR_C128) {
    r.h = static_cast<const nd2*>(p)[i];
  } else {
    r.h = static_cast<const nf2*>(p)[i];
    if constexpr (AR == AR_HILO) r.l = static_cast<const nf2*>(q)[i];
  }
}
template <int AR, typename T>
__device__ __forceinline__ void raw1_get(const Raw1<AR>& r, T& re, T& im) {
  if constexpr (AR == AR_HILO) {
    re = (double)r.h.x + (double)r.l.x;
    im = (double)r.h.y + (double)r.l.y;
  } else {
    re = (T)r.h.x;
    im = (T)r.h.y;
  }
}

// Half-vector q of the input at row i (zero past n).
template <int MODE>
__device__ __forceinline__ double2 t64_input(const double2* __restrict__ V, int64_t ldv, int64_t ldh, int64_t n,
                                             int conja, const double2* __restrict__ vb, int conjb, double sb, int q,
                                             int64_t i) {
  if (i >= n) return make_double2(0.0, 0.0);
  if constexpr (MODE == T64_H) {
    return V[(size_t)(q >> 1) * ldv + (q & 1 ? ldh : 0) + i];  // x, y
  } else {
    if (MODE == T64_E && q == 1) {
      const double2 y = vb[i];
      return make_double2(sb * y.x, conjb ? -sb * y.y : sb * y.y);
    }
    const double2 x = V[(size_t)q * ldv + i];
    return make_double2(x.x, conja ? -x.y : x.y);
  }
}

// V: NV half-vectors (T64_H: NV / 2 full-H columns, bottom at ldh), column q at
// q ldv.  Partials as in the streaming kernels: rowpart[o][blk][64],
// colpart[o][blk][64], o = 0 .. NV - 1.
template <int AR, int MODE, int NV>
__global__ void __launch_bounds__(kThreads, NV == 8 ? 2 : 1)
    tile64_kernel(const void* __restrict__ a0, const void* __restrict__ a1, const void* __restrict__ b0,
                  const void* __restrict__ b1, const int2* __restrict__ blkmap, int64_t nblk, int64_t n,
                  const double2* __restrict__ V, int64_t ldv, int64_t ldh, int conja,
                  const double2* __restrict__ vb, int conjb, double sb, double2* __restrict__ rowpart,
                  double2* __restrict__ colpart) {
  using T = typename Elem<AR>::T;
  constexpr int WAVES = 4, CPW = 64 / WAVES;
  constexpr bool HASB = MODE != T64_A;
  constexpr int NI = MODE == T64_E ? 2 : NV;  // input half-vectors
  static_assert(MODE != T64_E || NV == 1, "explicit B input: one vector");
  // values per column (two per output), padded to a power of two; columns per group of 16 values
  constexpr int VP = NV == 1 ? 2 : NV == 2 ? 4 : NV <= 4 ? 8 : 16;
  constexpr int CG = 16 / VP;
  constexpr int DEPTH = (AR == AR_HI || AR == AR_HI64 || !HASB) ? CPW : NV == 8 ? 4 : 8;
  // column entries of the wave, then (all waves done) the row sums
  constexpr int LROW = WAVES * NV * 64, LCOL = 64 * NI;
  __shared__ double2 lds[LROW > LCOL ? LROW : LCOL];
  __shared__ double csum[WAVES][CPW * VP];  // column sums: [column group][value]

  const int blk = blockIdx.x;
  const int2 pq = blkmap[blk];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int64_t row0 = (int64_t)pq.x * 64, col0 = (int64_t)pq.y * 64 + wave * CPW;
  const size_t base = (size_t)blk * 4096 + (size_t)wave * CPW * 64 + lane;

  Raw1<AR> ra[CPW], rb[HASB ? CPW : 1];
#pragma unroll
  for (int c = 0; c < DEPTH; ++c) {
    raw1_load<AR>(a0, a1, base + c * 64, ra[c]);
    if (HASB) raw1_load<AR>(b0, b1, base + c * 64, rb[c]);
  }
  double2* cx = lds + (size_t)wave * CPW * NI;  // [c][input]
#pragma unroll
  for (int e0 = 0; e0 < CPW * NI; e0 += 64) {
    const int e = e0 + lane;
    if (e < CPW * NI) cx[e] = t64_input<MODE>(V, ldv, ldh, n, conja, vb, conjb, sb, e % NI, col0 + e / NI);
  }
  T xr[NI], xi[NI], rr[NV], ri[NV];
#pragma unroll
  for (int q = 0; q < NI; ++q) {
    const double2 x = t64_input<MODE>(V, ldv, ldh, n, conja, vb, conjb, sb, q, row0 + lane);
    xr[q] = (T)x.x;
    xi[q] = (T)x.y;
  }
#pragma unroll
  for (int q = 0; q < NV; ++q) rr[q] = ri[q] = T(0);
  const T tsb = (T)sb;
  // this lane's place among the 16 sums of a column group
  double* cdst = csum[wave] + wave_sum_index<16>(lane);
  wave_lds_sync();

  double vals[16];
#pragma unroll
  for (int c = 0; c < CPW; ++c) {
    if (DEPTH < CPW && c + DEPTH < CPW) {
      raw1_load<AR>(a0, a1, base + (c + DEPTH) * 64, ra[c + DEPTH]);
      if (HASB) raw1_load<AR>(b0, b1, base + (c + DEPTH) * 64, rb[c + DEPTH]);
    }
    T ar, ai, br = T(0), bi = T(0);
    raw1_get<AR, T>(ra[c], ar, ai);
    if (HASB) raw1_get<AR, T>(rb[c], br, bi);
    T xc[NI], yc[NI], sr[NV], si[NV];
#pragma unroll
    for (int q = 0; q < NI; ++q) {
      const double2 x = cx[c * NI + q];
      xc[q] = (T)x.x;
      yc[q] = (T)x.y;
    }
#pragma unroll
    for (int q = 0; q < NV; ++q) sr[q] = si[q] = T(0);
    if constexpr (MODE == T64_H) {
#pragma unroll
      for (int q = 0; q < NV; q += 2) {
        // row r: A_rc x_c + B_rc y_c, A_rc conj(y_c) + B_rc conj(x_c)
        mac(rr[q], ar, xc[q]);
        mac(rr[q], -ai, yc[q]);
        mac(rr[q], br, xc[q + 1]);
        mac(rr[q], -bi, yc[q + 1]);
        mac(ri[q], ar, yc[q]);
        mac(ri[q], ai, xc[q]);
        mac(ri[q], br, yc[q + 1]);
        mac(ri[q], bi, xc[q + 1]);
        mac(rr[q + 1], ar, xc[q + 1]);
        mac(rr[q + 1], ai, yc[q + 1]);
        mac(rr[q + 1], br, xc[q]);
        mac(rr[q + 1], bi, yc[q]);
        mac(ri[q + 1], ai, xc[q + 1]);
        mac(ri[q + 1], -ar, yc[q + 1]);
        mac(ri[q + 1], bi, xc[q]);
        mac(ri[q + 1], -br, yc[q]);
        // column c: conj(A_rc) x_r + B_rc y_r, conj(A_rc) conj(y_r) + B_rc conj(x_r)
        mac(sr[q], ar, xr[q]);
        mac(sr[q], ai, xi[q]);
        mac(sr[q], br, xr[q + 1]);
        mac(sr[q], -bi, xi[q + 1]);
        mac(si[q], ar, xi[q]);
        mac(si[q], -ai, xr[q]);
        mac(si[q], br, xi[q + 1]);
        mac(si[q], bi, xr[q + 1]);
        mac(sr[q + 1], ar, xr[q + 1]);
        mac(sr[q + 1], -ai, xi[q + 1]);
        mac(sr[q + 1], br, xr[q]);
        mac(sr[q + 1], bi, xi[q]);
        mac(si[q + 1], -ar, xi[q + 1]);
        mac(si[q + 1], -ai, xr[q + 1]);
        mac(si[q + 1], bi, xr[q]);
        mac(si[q + 1], -br, xi[q]);
      }
    } else if constexpr (MODE == T64_K) {
      const T bs = tsb * br, bt = tsb * bi;  // sb = 1 or -1
      const T kp = ar + bs, kq = ar - bs, ks = ai + bt, kt = bt - ai;
#pragma unroll
      for (int q = 0; q < NV; ++q) {
        mac(rr[q], kp, xc[q]);
        mac(rr[q], kt, yc[q]);
        mac(ri[q], ks, xc[q]);
        mac(ri[q], kq, yc[q]);
        mac(sr[q], kp, xr[q]);
        mac(sr[q], ks, xi[q]);
        mac(si[q], kt, xr[q]);
        mac(si[q], kq, xi[q]);
      }
    } else {
#pragma unroll
      for (int q = 0; q < NV; ++q) {
        // row r: A_rc x_c; column c: conj(A_rc) x_r
        mac(rr[q], ar, xc[q]);
        mac(rr[q], -ai, yc[q]);
        mac(ri[q], ar, yc[q]);
        mac(ri[q], ai, xc[q]);
        mac(sr[q], ar, xr[q]);
        mac(sr[q], ai, xi[q]);
        mac(si[q], ar, xi[q]);
        mac(si[q], -ai, xr[q]);
      }
      if constexpr (MODE == T64_E) {  // + B_rc y_c, + B_rc y_r
        mac(rr[0], br, xc[1]);
        mac(rr[0], -bi, yc[1]);
        mac(ri[0], br, yc[1]);
        mac(ri[0], bi, xc[1]);
        mac(sr[0], br, xr[1]);
        mac(sr[0], -bi, xi[1]);
        mac(si[0], br, xi[1]);
        mac(si[0], bi, xr[1]);
      }
    }
#pragma unroll
    for (int j = 0; j < VP; ++j) {
      double v = 0.0;
      if (j < 2 * NV) v = (j & 1) ? (double)si[j / 2] : (double)sr[j / 2];
      vals[(c % CG) * VP + j] = v;
    }
    if (c % CG == CG - 1) {
      cdst[(c - (CG - 1)) * VP] = wave_sum_n<16>(vals);  // the four lanes of a group store the same value
    }
    // one column at a time: interleaved, the columns' entries and sums would
    // not fit the registers
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  }
  wave_lds_sync();
#pragma unroll
  for (int e0 = 0; e0 < CPW * NV; e0 += 64) {
    const int e = e0 + lane, q = e / CPW, c = e % CPW;
    if (e < CPW * NV)
      colpart[((size_t)q * nblk + blk) * 64 + wave * CPW + c] =
          make_double2(csum[wave][c * VP + 2 * q], csum[wave][c * VP + 2 * q + 1]);
  }

  __syncthreads();
#pragma unroll
  for (int q = 0; q < NV; ++q) lds[(wave * NV + q) * 64 + lane] = make_double2((double)rr[q], (double)ri[q]);
  __syncthreads();
  for (int e = threadIdx.x; e < NV * 64; e += 64 * WAVES) {
    double2 t = lds[e];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) {
      t.x += lds[w * NV * 64 + e].x;
      t.y += lds[w * NV * 64 + e].y;
    }
    rowpart[((size_t)(e >> 6) * nblk + blk) * 64 + (e & 63)] = t;
  }
}

template <int AR, int MODE, int NV>
void launch_tile64(const Layout& L, const MatPtrs& m, const double2* V, int64_t ldv, int64_t ldh, int conja,
                   const double2* vb, int conjb, double sb, double2* part, hipStream_t s) {
  double2* rowpart = part;
  double2* colpart = part + (size_t)NV * L.nblk * 64;
  hipLaunchKernelGGL((tile64_kernel<AR, MODE, NV>), dim3((unsigned)L.nblk), dim3(kThreads), 0, s, m.a, m.alo, m.b,
                     m.blo, L.blkmap, L.nblk, L.n, V, ldv, ldh, conja, vb, conjb, sb, rowpart, colpart);
}

template <int AR>
hipError_t tile64_mv(BMode bm, const Layout& L, const MatPtrs& m, const double2* va, int conja, const double2* vb,
                     int conjb, double sb, double2* part, hipStream_t s) {
  if (bm == BM_NONE)
    launch_tile64<AR, T64_A, 1>(L, m, va, 0, 0, conja, nullptr, 0, 1.0, part, s);
  else if (bm == BM_CONJ)
    launch_tile64<AR, T64_K, 1>(L, m, va, 0, 0, conja, nullptr, 0, sb, part, s);
  else
    launch_tile64<AR, T64_E, 1>(L, m, va, 0, 0, conja, vb, conjb, sb, part, s);
  return hipGetLastError();
}

template <int AR>
hipError_t tile64_mh(int nh, const Layout& L, const MatPtrs& m, const double2* V, int64_t ldv, int64_t ldh,
                     double2* part, hipStream_t s) {
  switch (nh) {
    case 1:
      launch_tile64<AR, T64_H, 2>(L, m, V, ldv, ldh, 0, nullptr, 0, 1.0, part, s);
      break;
    case 2:
      launch_tile64<AR, T64_H, 4>(L, m, V, ldv, ldh, 0, nullptr, 0, 1.0, part, s);
      break;
    case 3:
      launch_tile64<AR, T64_H, 6>(L, m, V, ldv, ldh, 0, nullptr, 0, 1.0, part, s);
      break;
    default:
      launch_tile64<AR, T64_H, 8>(L, m, V, ldv, ldh, 0, nullptr, 0, 1.0, part, s);
  }
  return hipGetLastError();
}

// rows per workgroup slice of the multi-vector pass: as many as the
// register budget allows (four vectors at 256 rows would leave one wave
// per SIMD)
__host__ __device__ constexpr int mk_rows(int nv) { return nv >= 4 ? 128 : (nv >= 2 ? 256 : 512); }

// Multi-vector pass: out_q = A x_q (BM_NONE) or A x_q + sb B conj(x_q)
// (BM_CONJ: K1 for sb = 1, K2 for sb = -1) for NV vectors in one read of the
// triangles.  Row r gains A_rc x_c (+ sb B_rc conj(x_c)), column c gains
// conj(A_rc) x_r (+ sb B_rc conj(x_r)); with B, both through the real 2 x 2
// block of the entry pair (see the column loop).  Same lane and partial
// layout as mv_stream_kernel, with row slices and NV outputs:
// rowpart[q][blk][R], colpart[q][blk][slice][R].
template <int R, int AR, int NV>
struct MkShape {
  static constexpr int RS = R < mk_rows(NV) ? R : mk_rows(NV);
  static constexpr int NS = R / RS;
  static constexpr int VW = (AR != AR_C128 && RS >= 128) ? 2 : 1;
  static constexpr int G = RS / (64 * VW);
  static constexpr int RPL = G * VW;
};

template <int R, int AR, int BM, int NV>
__global__ void __launch_bounds__(kThreads)
    mk_block_kernel(const void* __restrict__ a0, const void* __restrict__ a1,
                    const void* __restrict__ b0, const void* __restrict__ b1,
                    const int2* __restrict__ blkmap, int64_t nblk, int64_t n,
                    const double2* __restrict__ V, int64_t ldv, double sb,
                    double2* __restrict__ rowpart, double2* __restrict__ colpart) {
  using T = typename Elem<AR>::T;
  using Sh = MkShape<R, AR, NV>;
  constexpr int RS = Sh::RS, NS = Sh::NS, VW = Sh::VW, G = Sh::G, RPL = Sh::RPL;
  constexpr int CPW = R / 4;
  constexpr int CH = CPW < 64 ? CPW : 64;
  // two or more vectors: column sums through LDS (lds_colsum); the same
  // memory combines the row sums after the column loop
  constexpr int NVAL = 2 * NV;
  constexpr bool LCS = NVAL >= 4;
  constexpr int CSW = LCS ? colsum_lds(NVAL) : 0;
  constexpr int LDS2 = (4 * CSW > 8 * RS ? 4 * CSW : 8 * RS) / 2;
  __shared__ double2 lds[LDS2];
  double2(*sh)[RS] = reinterpret_cast<double2(*)[RS]>(lds);

  const int blk = blockIdx.x;
  const int slice = blockIdx.y;
  const int2 pq = blkmap[blk];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int64_t row0 = (int64_t)pq.x * R + slice * RS, col0 = (int64_t)pq.y * R;
  const size_t base = (size_t)blk * R * R + (size_t)slice * RS;
  const T tsb = (T)sb;
  double* stage = reinterpret_cast<double*>(lds) + wave * CSW;
  double* colsum = stage + NVAL * stage_ld(NVAL);

  T xr[NV][RPL], xi[NV][RPL], rr[NV][RPL], ri[NV][RPL];
#pragma unroll
  for (int v = 0; v < NV; ++v)
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int e = 0; e < VW; ++e) {
        const int q = g * VW + e;
        const int64_t i = row0 + g * 64 * VW + lane * VW + e;
        const bool in = i < n;
        const double2 x = V[(size_t)v * ldv + (in ? i : 0)];
        xr[v][q] = in ? (T)x.x : T(0);
        xi[v][q] = in ? (T)x.y : T(0);
        rr[v][q] = T(0);
        ri[v][q] = T(0);
      }

  // the next column's loads are issued before the current column is consumed
  const size_t lbase = base + (size_t)wave * CPW * R + lane * VW;
  RawCol<AR> ca_[G], cbm[G], na_[G], nbm[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    raw_load<AR>(a0, a1, lbase + g * 64 * VW, ca_[g]);
    if (BM == BM_CONJ) raw_load<AR>(b0, b1, lbase + g * 64 * VW, cbm[g]);
  }
  for (int cb = 0; cb < CPW; cb += CH) {
    double2 keep[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) keep[v] = make_double2(0.0, 0.0);
    // unrolled by two: see mh_stream_kernel
#pragma unroll 2
    for (int c2 = 0; c2 < CH; ++c2) {
      const int cc = cb + c2;
      const int cn = cc + 1 < CPW ? cc + 1 : cc;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        raw_load<AR>(a0, a1, lbase + (size_t)cn * R + g * 64 * VW, na_[g]);
        if (BM == BM_CONJ) raw_load<AR>(b0, b1, lbase + (size_t)cn * R + g * 64 * VW, nbm[g]);
      }
      __builtin_amdgcn_sched_barrier(0);  // see mh_stream_kernel
      const int c = wave * CPW + cc;
      const int64_t j = col0 + c;
      const bool in = j < n;
      const int64_t jj = in ? j : 0;
      T cxr[NV], cxi[NV], sr[NV], si[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const double2 x = V[(size_t)v * ldv + jj];
        cxr[v] = in ? (T)x.x : T(0);
        cxi[v] = in ? (T)x.y : T(0);
        sr[v] = T(0);
        si[v] = T(0);
      }
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < VW; ++e) {
          const int q = g * VW + e;
          T ar, ai;
          raw_get<AR, T>(ca_[g], e, ar, ai);
          if constexpr (BM == BM_CONJ) {
            // K = A + sb B conj acts on (Re, Im) of a vector entry as the real
            // block [[ar + sb br, sb bi - ai], [ai + sb bi, ar - sb br]] (its
            // transpose with conj(A) for the column use): 8 FMAs per vector
            // and entry pair instead of 16
            T br, bi;
            raw_get<AR, T>(cbm[g], e, br, bi);
            const T kp = ar + tsb * br, kq = ar - tsb * br, ks = ai + tsb * bi, kt = tsb * bi - ai;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
              mac(rr[v][q], kp, cxr[v]);
              mac(rr[v][q], kt, cxi[v]);
              mac(ri[v][q], ks, cxr[v]);
              mac(ri[v][q], kq, cxi[v]);
              mac(sr[v], kp, xr[v][q]);
              mac(sr[v], ks, xi[v][q]);
              mac(si[v], kt, xr[v][q]);
              mac(si[v], kq, xi[v][q]);
            }
          } else {
#pragma unroll
            for (int v = 0; v < NV; ++v) {
              // row r: A_rc x_c; column c: conj(A_rc) x_r
              mac(rr[v][q], ar, cxr[v]);
              mac(rr[v][q], -ai, cxi[v]);
              mac(ri[v][q], ar, cxi[v]);
              mac(ri[v][q], ai, cxr[v]);
              mac(sr[v], ar, xr[v][q]);
              mac(sr[v], ai, xi[v][q]);
              mac(si[v], ar, xi[v][q]);
              mac(si[v], -ai, xr[v][q]);
            }
          }
        }
      if constexpr (LCS) {
        double vals[LCS ? NVAL : 4];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          vals[2 * v] = (double)sr[v];
          vals[2 * v + 1] = (double)si[v];
        }
        lds_colsum<NVAL>(vals, stage, colsum, c2, lane);
      } else {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const double ur = dpp_wave_sum((double)sr[v]), ui = dpp_wave_sum((double)si[v]);
          keep[v] = lane == c2 ? make_double2(ur, ui) : keep[v];
        }
      }
#pragma unroll
      for (int g = 0; g < G; ++g) {
        ca_[g] = na_[g];
        if (BM == BM_CONJ) cbm[g] = nbm[g];
      }
    }
    if (lane < CH) {
#pragma unroll
      for (int v = 0; v < NV; ++v)
        colpart[(((size_t)v * nblk + blk) * NS + slice) * R + wave * CPW + cb + lane] =
            LCS ? make_double2(colsum[(2 * v) * 64 + lane], colsum[(2 * v + 1) * 64 + lane]) : keep[v];
    }
  }
  __syncthreads();  // the row-sum combine below reuses the column-sum LDS of every wave

#pragma unroll
  for (int v = 0; v < NV; ++v) {
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int e = 0; e < VW; ++e) {
        const int q = g * VW + e;
        sh[wave][g * 64 * VW + lane * VW + e] = make_double2((double)rr[v][q], (double)ri[v][q]);
      }
    __syncthreads();
    for (int r = threadIdx.x; r < RS; r += kThreads) {
      double2 t = sh[0][r];
#pragma unroll
      for (int w = 1; w < 4; ++w) {
        t.x += sh[w][r].x;
        t.y += sh[w][r].y;
      }
      rowpart[((size_t)v * nblk + blk) * R + slice * RS + r] = t;
    }
    __syncthreads();
  }
}

// The sum / difference inputs of mh_stream_kernel: UW[2q][i] = x_q[i] + conj(y_q[i]),
// UW[2q + 1][i] = x_q[i] - conj(y_q[i]) (rot: times -i) for i < pl (zero past n),
// column q of V being [x_q (ldh); y_q].  Grid (ceil(pl / 256), nh).
__global__ void __launch_bounds__(kThreads)
    hsd_stage_kernel(const double2* __restrict__ V, int64_t ldv, int64_t ldh, int64_t n, int64_t pl, int rot,
                     double2* __restrict__ UW) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int q = blockIdx.y;
  if (i >= pl) return;
  double2 u = make_double2(0.0, 0.0), w = u;
  if (i < n) {
    const double2 x = V[(size_t)q * ldv + i], y = V[(size_t)q * ldv + ldh + i];
    u = make_double2(x.x + y.x, x.y - y.y);
    w = make_double2(x.x - y.x, x.y + y.y);
  }
  UW[(size_t)(2 * q) * pl + i] = u;
  UW[(size_t)(2 * q + 1) * pl + i] = rot ? make_double2(w.y, -w.x) : w;
}

// rows per workgroup slice of the streaming full-H kernel: 256 rows spread
// each column's wavefront reductions (four per vector) over four rows per
// lane; 128 rows left the kernel bound by those reductions (37 ms vs 30 ms
// per read for two vectors at N = 1e5)
__host__ __device__ constexpr int mh_rows(int nh) { return nh >= 3 ? 128 : 256; }

// Full-H products in the streaming form (R >= 128), with the layout of
// mk_block_kernel: 16-byte loads of column segments, the next column's loads
// issued before the current one is consumed, column sums kept one per lane
// and stored per 64 columns.  The outputs are taken in the sum / difference
// basis: with u = x + conj(y) and w = x - conj(y),
//   top T = A x + B y and conjugated bottom C = A conj(y) + B conj(x) satisfy
//   T + C = K1 u = A u + B conj(u),  T - C = K2 w = A w - B conj(w),
// and each of K1, K2 acts on (Re, Im) of a vector entry as the real 2 x 2
// block [[ar + br, bi - ai], [ai + bi, ar - br]] (K2: B negated) of the
// stored pair (a, b), the column (transposed) use as its transpose with the
// conjugate of A.  The four sums are formed once per entry pair, so a vector
// costs 16 FMAs per pair instead of the 32 of the four complex products.
// Outputs 2q: K1 u_q, 2q+1: K2 w_q (mh_reduce_kernel, form 2, forms T and C).
// One workgroup per block takes its R / mh_rows(NH) row slices in turn.
// Row partials: rowpart[o][blk][R]; column partials: colpart[o][blk][R].
template <int R, int AR, int NH>
__global__ void __launch_bounds__(kThreads)
    mh_stream_kernel(const void* __restrict__ a0, const void* __restrict__ a1,
                     const void* __restrict__ b0, const void* __restrict__ b1,
                     const int2* __restrict__ blkmap, int64_t nblk, int64_t n,
                     const double2* __restrict__ UW, int64_t pl,
                     double2* __restrict__ rowpart, double2* __restrict__ colpart) {
  constexpr int RS = R < mh_rows(NH) ? R : mh_rows(NH);
  constexpr int NS = R / RS;
  constexpr int VW = AR != AR_C128 ? 2 : 1;
  constexpr int G = RS / (64 * VW);
  constexpr int RPL = G * VW;
  constexpr int CPW = R / 4;
  constexpr int CH = CPW < 64 ? CPW : 64;
  constexpr int NO = 2 * NH;
  static_assert(RS >= 128 && G >= 1, "streaming full-H layout");
  // LDS: per wave the column-sum stage and the 64 column sums of the current
  // chunk; after the column loop the same memory combines the row sums
  constexpr int NVAL = 2 * NO;
  constexpr int CSW = colsum_lds(NVAL);
  constexpr int LDS2 = (4 * CSW > 8 * RS ? 4 * CSW : 8 * RS) / 2;
  __shared__ double2 lds[LDS2];
  double2(*sh)[RS] = reinterpret_cast<double2(*)[RS]>(lds);

  const int blk = blockIdx.x;
  const int2 pq = blkmap[blk];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int64_t col0 = (int64_t)pq.y * R;
  double* stage = reinterpret_cast<double*>(lds) + wave * CSW;
  double* colsum = stage + NVAL * stage_ld(NVAL);

  // the row slices of the block in sequence: each adds its column sums to
  // those of the slices before (the same lane wrote them), so one set of
  // column partials per block leaves the kernel instead of one per slice
  for (int slice = 0; slice < NS; ++slice) {
    const int64_t row0 = (int64_t)pq.x * R + slice * RS;
    const size_t base = (size_t)blk * R * R + (size_t)slice * RS;

    // row entries of u = x + conj(y) and w = x - conj(y) (staged by hsd_stage_kernel over the
    // padded length pl, zero past n: no bounds selects here)
    double ur[NH][RPL], ui[NH][RPL], wr[NH][RPL], wi[NH][RPL], rr[NO][RPL], ri[NO][RPL];
#pragma unroll
    for (int q = 0; q < NH; ++q)
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < VW; ++e) {
          const int t = g * VW + e;
          const int64_t i = row0 + g * 64 * VW + lane * VW + e;
          const double2 u = UW[(size_t)(2 * q) * pl + i];
          const double2 w = UW[(size_t)(2 * q + 1) * pl + i];
          ur[q][t] = u.x;
          ui[q][t] = u.y;
          wr[q][t] = w.x;
          wi[q][t] = w.y;
        }
#pragma unroll
    for (int o = 0; o < NO; ++o)
#pragma unroll
      for (int t = 0; t < RPL; ++t) {
        rr[o][t] = 0.0;
        ri[o][t] = 0.0;
      }

    // hi + lo: the four waves interleave columns (wave w takes columns
    // 4 cc + w; measured 27.4 vs 28.3 ms per read); the lo-only products keep
    // contiguous column ranges per wave (16.5 vs 17.5 ms)
    constexpr bool IL = AR == AR_HILO;
    constexpr int CST = IL ? 4 : 1;  // column stride of a wave
    const size_t lbase = base + (size_t)wave * (IL ? 1 : CPW) * R + lane * VW;
    // column buffers: a wave's loads run NBUF - 1 columns ahead of its
    // arithmetic (three for the complex64 hi triangles, whose columns are 8
    // VGPRs; one for the wider hi + lo and complex128 columns); column cc sits
    // in slot cc % NBUF, and the loop is unrolled by NBUF so the slots are
    // renamed, not copied (a copy would wait for the loads just issued)
    constexpr int NBUF = AR == AR_HI64 && G == 1 ? 4 : 2;
    static_assert(CH % NBUF == 0, "column chunk of whole buffer rounds");
    RawCol<AR> ra[NBUF][G], rb[NBUF][G];
#pragma unroll
    for (int k = 0; k < NBUF - 1; ++k) {
      const int cn = k < CPW ? k : CPW - 1;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        raw_load<AR>(a0, a1, lbase + (size_t)cn * CST * R + g * 64 * VW, ra[k][g]);
        raw_load<AR>(b0, b1, lbase + (size_t)cn * CST * R + g * 64 * VW, rb[k][g]);
      }
    }
    for (int cb = 0; cb < CPW; cb += CH) {
      for (int c4 = 0; c4 < CH; c4 += NBUF) {
        auto step = [&](auto slot) {
          constexpr int S = decltype(slot)::value;
          constexpr int SN = (S + NBUF - 1) % NBUF;  // the slot of column cc + NBUF - 1
          const int c2 = c4 + S;
          const int cc = cb + c2;
          const int cn = cc + NBUF - 1 < CPW ? cc + NBUF - 1 : CPW - 1;
#pragma unroll
          for (int g = 0; g < G; ++g) {
            raw_load<AR>(a0, a1, lbase + (size_t)cn * CST * R + g * 64 * VW, ra[SN][g]);
            raw_load<AR>(b0, b1, lbase + (size_t)cn * CST * R + g * 64 * VW, rb[SN][g]);
          }
          // keep the loads here: under register pressure the scheduler would sink
          // them next to their use in the following column
          __builtin_amdgcn_sched_barrier(0);
          const int c = IL ? cc * 4 + wave : wave * CPW + cc;
          const int64_t j = col0 + c;
          double cur[NH], cui[NH], cwr[NH], cwi[NH], sr[NO], si[NO];
#pragma unroll
          for (int q = 0; q < NH; ++q) {
            const double2 u = UW[(size_t)(2 * q) * pl + j];
            const double2 w = UW[(size_t)(2 * q + 1) * pl + j];
            cur[q] = u.x;
            cui[q] = u.y;
            cwr[q] = w.x;
            cwi[q] = w.y;
          }
#pragma unroll
          for (int o = 0; o < NO; ++o) {
            sr[o] = 0.0;
            si[o] = 0.0;
          }
#pragma unroll
          for (int g = 0; g < G; ++g)
#pragma unroll
            for (int e = 0; e < VW; ++e) {
              const int t = g * VW + e;
              double ar, ai, br, bi;
              raw_get<AR, double>(ra[S][g], e, ar, ai);
              raw_get<AR, double>(rb[S][g], e, br, bi);
              const double sp = ar + br, sq = ar - br, ss = ai + bi, st = bi - ai;
#pragma unroll
              for (int q = 0; q < NH; ++q) {
                // rows: K1 u_c = (sp ur + st ui, ss ur + sq ui); K2 w_c = (sq wr - ss wi, -st wr + sp wi)
                mac(rr[2 * q][t], sp, cur[q]);
                mac(rr[2 * q][t], st, cui[q]);
                mac(ri[2 * q][t], ss, cur[q]);
                mac(ri[2 * q][t], sq, cui[q]);
                mac(rr[2 * q + 1][t], sq, cwr[q]);
                mac(rr[2 * q + 1][t], -ss, cwi[q]);
                mac(ri[2 * q + 1][t], -st, cwr[q]);
                mac(ri[2 * q + 1][t], sp, cwi[q]);
                // columns (conj(A) transposed, B): K1 u_r = (sp ur + ss ui, st ur + sq ui);
                // K2 w_r = (sq wr - st wi, -ss wr + sp wi)
                mac(sr[2 * q], sp, ur[q][t]);
                mac(sr[2 * q], ss, ui[q][t]);
                mac(si[2 * q], st, ur[q][t]);
                mac(si[2 * q], sq, ui[q][t]);
                mac(sr[2 * q + 1], sq, wr[q][t]);
                mac(sr[2 * q + 1], -st, wi[q][t]);
                mac(si[2 * q + 1], -ss, wr[q][t]);
                mac(si[2 * q + 1], sp, wi[q][t]);
              }
            }
          double vals[NVAL];
#pragma unroll
          for (int o = 0; o < NO; ++o) {
            vals[2 * o] = sr[o];
            vals[2 * o + 1] = si[o];
          }
          lds_colsum<NVAL>(vals, stage, colsum, c2, lane);
        };
        step(std::integral_constant<int, 0>());
        step(std::integral_constant<int, 1>());
        if constexpr (NBUF == 4) {
          step(std::integral_constant<int, 2>());
          step(std::integral_constant<int, 3>());
        }
      }
      if (lane < CH) {
#pragma unroll
        for (int o = 0; o < NO; ++o) {
          double2* cp = colpart + ((size_t)o * nblk + blk) * R + (IL ? (cb + lane) * 4 + wave : wave * CPW + cb + lane);
          double2 t = make_double2(colsum[(2 * o) * 64 + lane], colsum[(2 * o + 1) * 64 + lane]);
          if (slice) {
            const double2 p = *cp;
            t.x += p.x;
            t.y += p.y;
          }
          *cp = t;
        }
      }
      wave_lds_sync();  // the flush reads colsum before the next chunk's columns store to it
    }
    __syncthreads();  // the row-sum combine below reuses the column-sum LDS of every wave

#pragma unroll
    for (int o = 0; o < NO; ++o) {
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < VW; ++e)
          sh[wave][g * 64 * VW + lane * VW + e] = make_double2(rr[o][g * VW + e], ri[o][g * VW + e]);
      __syncthreads();
      for (int r = threadIdx.x; r < RS; r += kThreads) {
        double2 t = sh[0][r];
#pragma unroll
        for (int w = 1; w < 4; ++w) {
          t.x += sh[w][r].x;
          t.y += sh[w][r].y;
        }
        rowpart[((size_t)o * nblk + blk) * R + slice * RS + r] = t;
      }
      __syncthreads();
    }
  }
}

// Multi-vector passes on FP64 matrix cores (R >= 128): NV <= 4 NG half-vectors
// (MODE as in tile64_kernel: T64_A, T64_K, or T64_H in the sum / difference basis:
// u = x + conj(y) and -i w = -i (x - conj(y)) of NV / 2 full-H vectors, both
// through K1 since K2 w = i K1 (-i w)).
//
// What bounds it: with FMAs the four-vector full-H read on hi was bound by
// their issue at two waves per SIMD (2.75 ms at N = 32768, where its 8.6 GB take
// 1.4 ms at the rate of a plain read).  v_mfma_f64_4x4x4 sustains 73 TFLOP/s
// against 58 for a pure FMA loop in a quarter of the instructions; its four
// independent 4 x 4 blocks take four vectors on the right, so eight
// half-vectors are two instructions with nothing padded (the 16 x 16 form would
// run half empty).  1.85 to 1.95 ms here, of which the products alone take 0.95 (matrix
// instructions and FP64 vector instructions share one unit: together they ran
// at 72 TFLOP/s, so conversions and sums are worth removing).
//
// Row products: lane l holds entry (row pair l & 15, column l >> 4) of a 16 VW x 4
// subtile, which is the A operand A[i = l & 3][k = l >> 4] of block
// (l >> 2) & 3 with the column as k; the four real coefficients kp, kt, ks, kq
// of the entry pair are four such operands.  Column products contract over
// rows: the same coefficients with lane bits 0-1 and 4-5 exchanged, through
// LDS within the wave (columns 320 bytes apart: the 16 lanes of a read phase on
// distinct banks); exchanging the entries instead and forming the coefficients
// twice took 2.00 ms.  64 entry pairs cost 8 NG matrix instructions and eight
// conversions and sums.
//
// A workgroup takes one R x R block; each wave owns an equal share of its rows for
// all columns, so the row sums stay in its registers to the end; the column
// sums of a step (four columns) are added over the lanes' row blocks and meet
// the other waves' in LDS every 32 columns (fixed order: deterministic).  The
// loads of the next four columns are issued before the current ones are used.
constexpr int kMfmaChunk = 32;  // columns between two combinations of the waves' column sums

__device__ __forceinline__ double mfma4(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// Which products take the matrix cores, from reads with their sums (us, FMA
// kernel / matrix cores; hi unless marked):
//   H of 4 vectors, R = 128: 308 / 225, 256: 764 / 494, 512: 2748 / 1846; hi + lo
//   R = 256: 966 / 869, complex128 1142 / 840, but R = 128 363 / 377 and 362 /
//   365; of 3: R = 128 219 / 218, 256 568 / 475, 512 2181 / 1798; of 2: R = 128
//   179 / 188, 256 459 / 442, hi + lo 789 / 828 (bound by the read).
//   A x four: R = 128 133 / 114, 256 332 / 245, 512 1233 / 921, hi + lo R = 256
//   456 / 437, R = 128 177 / 192, complex128 446 / 424 and 185 / 177; K1 x
//   four: R = 128 178 / 184, 256 466 / 432, 512 1748 / 1632, hi + lo 858 / 810
//   and 322 / 339, complex128 938 / 786 and 341 / 321; three vectors within 5 %
//   either way (K1: R = 128 167 / 175, 256 441 / 421, 512 1570 / 1587, no gain in
//   a Haydock run at N = 12001).
constexpr bool mh_on_mfma(int R, int AR, int nh) { return AR != AR_HI && nh >= 3 && (R >= 256 || AR == AR_HI64); }
constexpr bool mk_on_mfma(int R, int AR, int BM, int nv) {
  if (AR == AR_HI || R < 128 || nv < 4) return false;
  if (R == 128) return AR == AR_C128 || (AR == AR_HI64 && BM == BM_NONE);
  return true;
}

// waves of a workgroup: the row state of 64 rows and eight half-vectors fits
// two waves per SIMD, that of 128 rows (block edge 512 on four waves) spilled
constexpr int mfma_waves(int R) { return R == 512 ? 8 : 4; }

template <int R, int AR, int MODE, int NG>
__global__ void __launch_bounds__(64 * mfma_waves(R), 2)
    mfma_pass_kernel(const void* __restrict__ a0, const void* __restrict__ a1, const void* __restrict__ b0,
                     const void* __restrict__ b1, const int2* __restrict__ blkmap, int64_t nblk, int64_t n,
                     const double2* __restrict__ V, int64_t ldv, int nv, double sb,
                     double2* __restrict__ rowpart, double2* __restrict__ colpart) {
  constexpr int VW = AR == AR_C128 ? 1 : 2;  // rows per lane load
  constexpr int WAVES = mfma_waves(R);
  constexpr int RT = R / WAVES;              // rows of a wave
  constexpr int SUB = RT / (16 * VW);        // 16 VW x 4 subtiles of a step
  constexpr bool HASB = MODE != T64_A;
  constexpr int NM = HASB ? 2 : 1;  // double2 of coefficients per entry pair
  constexpr int STEPS = R / 4, SPC = kMfmaChunk / 4;
  constexpr int TLD = 20;  // double2 per transposed column (16 and padding)
  __shared__ double2 trn[WAVES][2][NM][4 * TLD];                   // [wave][buffer][matrix]
  __shared__ double2 csum[2][WAVES][4 * NG][kMfmaChunk + 4];       // [buffer][wave][output][column]

  const int blk = blockIdx.x;
  const int2 pq = blkmap[blk];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int l0 = lane & 3, lb = (lane >> 2) & 3, l2 = lane >> 4;
  const int64_t row0 = (int64_t)pq.x * R + wave * RT, col0 = (int64_t)pq.y * R;
  // half-vector q at index i; past the ends the last one (past nv the outputs are
  // not written)
  auto input = [&](int q, int64_t i) -> double2 {
    return V[(size_t)(q < nv ? q : nv - 1) * ldv + (i < n ? i : n - 1)];
  };
  // and zero past n: the stored entries there are zero, but zero times an infinite
  // last entry is not.  Selected where it is used, so that the load stays in
  // flight.  (H: staged with zeros over the padded length, nothing is past n)
  auto inside = [&](bool in, double2 v) {
    if constexpr (MODE == T64_H) return v;
    return in ? v : make_double2(0.0, 0.0);
  };
  const int cleft = (int)(n - col0 < R ? n - col0 : R);  // columns of the block below n

  // row-side operands B[k = l2][j = l0] of block lb: row pair lb + 4 l2
  double xr[SUB][VW][NG], xi[SUB][VW][NG], dr[SUB][VW][NG], di[SUB][VW][NG];
#pragma unroll
  for (int s = 0; s < SUB; ++s)
#pragma unroll
    for (int e = 0; e < VW; ++e)
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        const int64_t i = row0 + s * 16 * VW + (lb + 4 * l2) * VW + e;
        const double2 x = inside(i < n, input(4 * g + l0, i));
        xr[s][e][g] = x.x;
        xi[s][e][g] = x.y;
        dr[s][e][g] = 0.0;
        di[s][e][g] = 0.0;
      }

  const size_t lbase = (size_t)blk * R * R + (size_t)l2 * R + wave * RT + (lane & 15) * VW;
  // the loads run AHEAD steps ahead of their use, in slots that the unrolled
  // loop renames (hi: the next step's first exchange needs its entries a step
  // early, 2111 -> 2004 us at N = 32768; the wider entries have no registers
  // for it and lose 4 %)
  constexpr int AHEAD = AR == AR_HI64 ? 2 : 1;
  RawCol<AR> ra[4][SUB], rb[4][HASB ? SUB : 1];
  double2 xc[4][NG];
  auto fetch = [&](int st, auto slot) {
    constexpr int S = decltype(slot)::value;
#pragma unroll
    for (int s = 0; s < SUB; ++s) {
      raw_load<AR>(a0, a1, lbase + (size_t)st * 4 * R + s * 16 * VW, ra[S][s]);
      if constexpr (HASB) raw_load<AR>(b0, b1, lbase + (size_t)st * 4 * R + s * 16 * VW, rb[S][s]);
    }
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const int q = 4 * g + l0, c = st * 4 + l2;
      if constexpr (MODE == T64_H)
        xc[S][g] = input(q, col0 + c);
      else
        xc[S][g] = (V + (size_t)(q < nv ? q : nv - 1) * ldv + col0)[c < cleft ? c : cleft - 1];
    }
  };
  double2* const tw = &trn[wave][0][0][0];
  const int wr = (lane >> 4) * TLD + (lane & 15);  // this lane's place as written
  const int rd = l0 * TLD + lb + 4 * l2;           // and as read: column l0, row pair lb + 4 l2

  // the real 2 x 2 block of an entry pair
  struct Coef {
    double kp, kt, ks, kq;
  };
  auto coef = [&](double ar, double ai, double br, double bi) {
    Coef c;
    if constexpr (MODE == T64_A) {
      c.kp = c.kq = ar;
      c.ks = ai;
      c.kt = -ai;
    } else {
      if constexpr (MODE == T64_K) {  // sb = 1 or -1
        br *= sb;
        bi *= sb;
      }
      c.kp = ar + br;
      c.kq = ar - br;
      c.ks = ai + bi;
      c.kt = bi - ai;
    }
    return c;
  };

  // unit u of a step: rows e = u % VW of subtile u / VW, 64 entry pairs; its
  // coefficients (rc) go through LDS into the transposed lanes (tc)
  constexpr int UN = SUB * VW;
  Coef rc[2], tc[2];
  auto exchange = [&](auto slot, auto unit, auto bufc) {
    constexpr int S = decltype(slot)::value, u = decltype(unit)::value, X = decltype(bufc)::value;
    double ar, ai, br = 0.0, bi = 0.0;
    raw_get<AR, double>(ra[S][u / VW], u % VW, ar, ai);
    if constexpr (HASB) raw_get<AR, double>(rb[S][u / VW], u % VW, br, bi);
    const Coef c = coef(ar, ai, br, bi);
    rc[X] = c;
    double2* w = tw + X * NM * 4 * TLD;
    w[wr] = make_double2(c.kp, c.ks);
    if constexpr (HASB) w[4 * TLD + wr] = make_double2(c.kt, c.kq);
    wave_lds_sync();
    const double2 t = w[rd];
    tc[X].kp = t.x;
    tc[X].ks = t.y;
    if constexpr (HASB) {
      const double2 t2 = w[4 * TLD + rd];
      tc[X].kt = t2.x;
      tc[X].kq = t2.y;
    } else {
      tc[X].kt = -t.y;
      tc[X].kq = t.x;
    }
    wave_lds_sync();
  };
  // column sums of a step over the row blocks lb (lane bits 2-3, the banks of a
  // DPP row): the 2 NG values of a lane are exchanged so that each bank ends up
  // with the sum of one of them (NG = 1: each of two, twice)
  double cr[NG], ci[NG];
  double* const cdst = reinterpret_cast<double*>(&csum[0][wave][NG == 2 ? (lb & 2) * 2 + l0 : l0][l2]) +
                       (NG == 2 ? lb & 1 : lb >> 1);
  auto col_out = [&](int st, const double (&pr)[NG], const double (&pi)[NG]) {
    double v;
    if constexpr (NG == 2) {
      const double p = dpp_swap_add<0x128, 0x3>(pr[0], pr[1]);  // row_ror:8; banks 0, 1: group 0
      const double q = dpp_swap_add<0x128, 0x3>(pi[0], pi[1]);
      v = bank_pair_add(p, q);  // banks 0, 2: real part, 1, 3: imaginary part
    } else {
      const double p = dpp_swap_add<0x128, 0x3>(pr[0], pi[0]);  // banks 0, 1: real part, 2, 3: imaginary part
      v = bank_pair_add(p, p);
    }
    constexpr int BUFD = WAVES * 4 * NG * (kMfmaChunk + 4) * 2;  // doubles of one buffer of csum
    cdst[((st / SPC) & 1) * BUFD + (st % SPC) * 8] = v;
  };
  // the waves' column sums of a chunk
  auto chunk_out = [&](int ch) {
    __syncthreads();  // the other buffer of csum is free once every wave is here again
    for (int v = threadIdx.x; v < 4 * NG * kMfmaChunk; v += 64 * WAVES) {
      const int q = v / kMfmaChunk, c = v % kMfmaChunk;
      double2 t = csum[ch & 1][0][q][c];
#pragma unroll
      for (int w = 1; w < WAVES; ++w) {
        t.x += csum[ch & 1][w][q][c].x;
        t.y += csum[ch & 1][w][q][c].y;
      }
      if (MODE == T64_H && (q & 1)) t = make_double2(-t.y, t.x);  // K2 w = i K1 (-i w)
      if (q < nv) colpart[((size_t)q * nblk + blk) * R + ch * kMfmaChunk + c] = t;
    }
  };

  // One step: the exchanges run one unit ahead of the products (the next
  // step's first unit included), the previous step's column sums are finished
  // under this step's products.
  auto step = [&](int st, auto slot) {
    constexpr int S = decltype(slot)::value;
    fetch(st + AHEAD < STEPS ? st + AHEAD : STEPS - 1, std::integral_constant<int, (S + AHEAD) % 4>());
    __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of their use
    double pr[NG], pi[NG];
    double2 x[NG];  // the column-side operands of the step
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      x[g] = inside(st * 4 + l2 < cleft, xc[S][g]);
      pr[g] = cr[g];
      pi[g] = ci[g];
      cr[g] = ci[g] = 0.0;
    }
    auto unit = [&](auto uc) {
      constexpr int u = decltype(uc)::value;
      constexpr int X = (S * UN + u) & 1;
      if constexpr (u + 1 < UN)
        exchange(slot, std::integral_constant<int, u + 1>(), std::integral_constant<int, 1 - X>());
      else
        exchange(std::integral_constant<int, (S + 1) % 4>(), std::integral_constant<int, 0>(),
                 std::integral_constant<int, 1 - X>());
      constexpr int s = u / VW, e = u % VW;
      const Coef &c = rc[X], &t = tc[X];
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        dr[s][e][g] = mfma4(c.kp, x[g].x, dr[s][e][g]);
        di[s][e][g] = mfma4(c.ks, x[g].x, di[s][e][g]);
        cr[g] = mfma4(t.kp, xr[s][e][g], cr[g]);
        ci[g] = mfma4(t.kt, xr[s][e][g], ci[g]);
      }
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        dr[s][e][g] = mfma4(c.kt, x[g].y, dr[s][e][g]);
        di[s][e][g] = mfma4(c.kq, x[g].y, di[s][e][g]);
        cr[g] = mfma4(t.ks, xi[s][e][g], cr[g]);
        ci[g] = mfma4(t.kq, xi[s][e][g], ci[g]);
      }
      if (u == 0 && st > 0) col_out(st - 1, pr, pi);
    };
    unit(std::integral_constant<int, 0>());
    unit(std::integral_constant<int, 1>());
    if constexpr (UN > 2) {
      unit(std::integral_constant<int, 2>());
      unit(std::integral_constant<int, 3>());
    }
    static_assert(UN == 2 || UN == 4, "units of a step");
    if (st > 0 && st % SPC == 0) chunk_out(st / SPC - 1);
  };
  fetch(0, std::integral_constant<int, 0>());
  if constexpr (AHEAD == 2) fetch(1, std::integral_constant<int, 1>());
  exchange(std::integral_constant<int, 0>(), std::integral_constant<int, 0>(), std::integral_constant<int, 0>());
  for (int st = 0; st < STEPS; st += 4) {
    step(st, std::integral_constant<int, 0>());
    step(st + 1, std::integral_constant<int, 1>());
    step(st + 2, std::integral_constant<int, 2>());
    step(st + 3, std::integral_constant<int, 3>());
  }
  col_out(STEPS - 1, cr, ci);
  chunk_out(STEPS / SPC - 1);
  // D[i = l2][j = l0] of block lb: row pair l2 + 4 lb, half-vector l0
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    const int q = 4 * g + l0;
    if (q >= nv) continue;
    double2* rp = rowpart + ((size_t)q * nblk + blk) * R + wave * RT + (l2 + 4 * lb) * VW;
#pragma unroll
    for (int s = 0; s < SUB; ++s)
#pragma unroll
      for (int e = 0; e < VW; ++e) {
        const double vx = dr[s][e][g], vy = di[s][e][g];
        rp[s * 16 * VW + e] = (MODE == T64_H && (q & 1)) ? make_double2(-vy, vx) : make_double2(vx, vy);
      }
  }
}

// nx: entries of a column of V (its leading dimension ldv)
template <int R, int AR, int MODE>
hipError_t launch_mfma(int nv, const Layout& L, const MatPtrs& m, const double2* V, int64_t ldv, int64_t nx,
                       double sb, double2* part, hipStream_t s) {
  double2* rowpart = part;
  double2* colpart = part + (size_t)nv * L.nblk * R;
  const dim3 grid((unsigned)L.nblk), wg(64 * mfma_waves(R));
  constexpr int NG = MODE == T64_H ? 2 : 1;  // six or eight half-vectors, else four vectors
  hipLaunchKernelGGL((mfma_pass_kernel<R, AR, MODE, NG>), grid, wg, 0, s, m.a, m.alo, m.b, m.blo, L.blkmap, L.nblk,
                     nx, V, ldv, nv, sb, rowpart, colpart);
  return hipGetLastError();
}

// Sum of the partials of a multi-vector pass (form 0: output q to column q of
// MV) or of a full-H product, where the workgroup of vector q sums outputs 2q and
// 2q + 1 and writes the top and the conjugated bottom, the bottom times bsign: 1
// for M v, -1 for H v.  Form 1 (block edge 64): the outputs are the two halves.
// Form 2: they are K1 u_q and K2 w_q, top (K1 u + K2 w) / 2, conjugated bottom
// (K1 u - K2 w) / 2.  Grid (ceil(n / 64), vectors).
template <int W>
__global__ void __launch_bounds__(64 * W)
    mh_reduce_kernel(const double2* __restrict__ rowpart, const double2* __restrict__ colpart, int R, int NS,
                     int nb, int64_t nblk, int64_t n, double2* __restrict__ MV, int64_t ldv, int64_t ldh,
                     double bsign, const double* __restrict__ dc, double dsg,
                     const double2* __restrict__ X, int64_t ldx, int64_t ldhx, int form) {
  __shared__ double2 sh[W][64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t i0 = (int64_t)blockIdx.x * 64, i = i0 + lane;
  const int P = (int)(i0 / R), r = (int)(i0 % R) + lane;
  const size_t rs = (size_t)nblk * R, cs = rs * NS;
  if (form) {
    const int q = blockIdx.y;
    double s1x = 0.0, s1y = 0.0, s2x = 0.0, s2y = 0.0;
    part_range<W>(rowpart + 2 * q * rs, colpart + 2 * q * cs, R, NS, nb, P, r, wave, s1x, s1y);
    part_range<W>(rowpart + (2 * q + 1) * rs, colpart + (2 * q + 1) * cs, R, NS, nb, P, r, wave, s2x, s2y);
    const double2 k1 = wave_order_sum<W>(sh, wave, lane, s1x, s1y);
    const double2 k2 = wave_order_sum<W>(sh, wave, lane, s2x, s2y);
    if (wave != 0 || i >= n) return;
    double tx = k1.x, ty = k1.y;  // top
    double cx = k2.x, cy = k2.y;  // conjugated bottom
    if (form == 2) {
      tx = 0.5 * (k1.x + k2.x);
      ty = 0.5 * (k1.y + k2.y);
      cx = 0.5 * (k1.x - k2.x);
      cy = 0.5 * (k1.y - k2.y);
    }
    if (dc) {
      const double f = dsg * dc[i];
      const double2 x = X[(size_t)q * ldx + i];
      const double2 y = X[(size_t)q * ldx + ldhx + i];
      tx = fma(f, x.x, tx);
      ty = fma(f, x.y, ty);
      cx = fma(f, y.x, cx);
      cy = fma(-f, y.y, cy);
    }
    MV[(size_t)q * ldv + i] = make_double2(tx, ty);
    MV[(size_t)q * ldv + ldh + i] = make_double2(bsign * cx, -bsign * cy);
    return;
  }
  const int o = blockIdx.y;
  double sx = 0.0, sy = 0.0;
  part_range<W>(rowpart + o * rs, colpart + o * cs, R, NS, nb, P, r, wave, sx, sy);
  const double2 t = wave_order_sum<W>(sh, wave, lane, sx, sy);
  if (wave != 0 || i >= n) return;
  double tx = t.x, ty = t.y;
  if (dc) {
    const double f = dsg * dc[i];
    const double2 x = X[(size_t)o * ldx + i];
    tx = fma(f, x.x, tx);
    ty = fma(f, x.y, ty);
  }
  MV[(size_t)o * ldv + i] = make_double2(tx, ty);
}

void launch_mh_reduce(const Layout& L, int ny, int ns, const double2* rowpart, const double2* colpart, double2* MV,
                      int64_t ldv, int64_t ldh, double bsign, const MatPtrs& m, const double2* X,
                      int64_t ldx, int64_t ldhx, int form, hipStream_t s) {
  const dim3 grid((unsigned)((L.n + 63) / 64), (unsigned)ny);
  if (reduce_wide(L))
    hipLaunchKernelGGL(mh_reduce_kernel<16>, grid, dim3(1024), 0, s, rowpart, colpart, L.R, ns, L.nb, L.nblk, L.n,
                       MV, ldv, ldh, bsign, m.dc, m.dsign, X, ldx, ldhx, form);
  else
    hipLaunchKernelGGL(mh_reduce_kernel<4>, grid, dim3(256), 0, s, rowpart, colpart, L.R, ns, L.nb, L.nblk, L.n, MV,
                       ldv, ldh, bsign, m.dc, m.dsign, X, ldx, ldhx, form);
}

template <int R, int AR>
hipError_t launch_mh(int nh, const Layout& L, const MatPtrs& m, const double2* V, int64_t ldv, int64_t ldh,
                     double2* part, hipStream_t s) {
  if constexpr (R == 64) {
    return tile64_mh<AR>(nh, L, m, V, ldv, ldh, part, s);
  } else {
    double2* rowpart = part;
    double2* colpart = part + (size_t)2 * nh * L.nblk * R;
    // u, w of every vector over the padded length, after the partials (mh_part_elems)
    const int64_t pl = (int64_t)L.nb * R;
    double2* uw = colpart + (size_t)2 * nh * L.nblk * R;
    const bool mfma = mh_on_mfma(R, AR, nh);
    hipLaunchKernelGGL(hsd_stage_kernel, dim3((unsigned)((pl + kThreads - 1) / kThreads), (unsigned)nh),
                       dim3(kThreads), 0, s, V, ldv, ldh, L.n, pl, (int)mfma, uw);
    if constexpr (mh_on_mfma(R, AR, 4)) {
      if (mfma) return launch_mfma<R, AR, T64_H>(2 * nh, L, m, uw, pl, pl, 1.0, part, s);
    }
    const dim3 grid((unsigned)L.nblk);
    if (nh == 1)
      hipLaunchKernelGGL((mh_stream_kernel<R, AR, 1>), grid, dim3(kThreads), 0, s, m.a, m.alo, m.b, m.blo,
                         L.blkmap, L.nblk, L.n, uw, pl, rowpart, colpart);
    else if (nh == 2)
      hipLaunchKernelGGL((mh_stream_kernel<R, AR, 2>), grid, dim3(kThreads), 0, s, m.a, m.alo, m.b, m.blo,
                         L.blkmap, L.nblk, L.n, uw, pl, rowpart, colpart);
    if constexpr (!mh_on_mfma(R, AR, 3)) {
      if (nh == 3)
        hipLaunchKernelGGL((mh_stream_kernel<R, AR, 3>), grid, dim3(kThreads), 0, s, m.a, m.alo, m.b, m.blo,
                           L.blkmap, L.nblk, L.n, uw, pl, rowpart, colpart);
      else if (nh == 4)
        hipLaunchKernelGGL((mh_stream_kernel<R, AR, 4>), grid, dim3(kThreads), 0, s, m.a, m.alo, m.b, m.blo,
                           L.blkmap, L.nblk, L.n, uw, pl, rowpart, colpart);
    }
    return hipGetLastError();
  }
}

template <int R>
hipError_t dispatch_mh(Arith ar, int nh, const Layout& L, const MatPtrs& m, const double2* V, int64_t ldv,
                       int64_t ldh, double2* part, hipStream_t s) {
  if (ar == AR_C128) return launch_mh<R, AR_C128>(nh, L, m, V, ldv, ldh, part, s);
  if (ar == AR_HI64) return launch_mh<R, AR_HI64>(nh, L, m, V, ldv, ldh, part, s);
  return launch_mh<R, AR_HILO>(nh, L, m, V, ldv, ldh, part, s);
}

template <int R, int AR, int BM>
hipError_t launch_mv(const Layout& L, const MatPtrs& m, const double2* va, int conja,
                     const double2* vb, int conjb, double sb, double2* part, hipStream_t s) {
  if constexpr (R == 64) {
    return tile64_mv<AR>((BMode)BM, L, m, va, conja, vb, conjb, sb, part, s);
  } else {
    double2* rowpart = part;
    double2* colpart = part + (size_t)L.nblk * L.R;
    hipLaunchKernelGGL((mv_stream_kernel<R, AR, BM>), dim3((unsigned)L.nblk, (unsigned)MvShape<R, AR>::NS),
                       dim3(kThreads), 0, s, m.a, m.alo, m.b, m.blo, L.blkmap, L.n, va, conja, vb, conjb, sb,
                       rowpart, colpart);
    return hipGetLastError();
  }
}

template <int R, int AR>
hipError_t dispatch_bm(BMode bm, const Layout& L, const MatPtrs& m, const double2* va, int conja,
                       const double2* vb, int conjb, double sb, double2* part, hipStream_t s) {
  switch (bm) {
    case BM_NONE:
      return launch_mv<R, AR, BM_NONE>(L, m, va, conja, vb, conjb, sb, part, s);
    case BM_CONJ:
      return launch_mv<R, AR, BM_CONJ>(L, m, va, conja, vb, conjb, sb, part, s);
    default:
      return launch_mv<R, AR, BM_EXPLICIT>(L, m, va, conja, vb, conjb, sb, part, s);
  }
}

template <int R>
hipError_t dispatch_ar(Arith ar, BMode bm, const Layout& L, const MatPtrs& m, const double2* va,
                       int conja, const double2* vb, int conjb, double sb, double2* part,
                       hipStream_t s) {
  switch (ar) {
    case AR_C128:
      return dispatch_bm<R, AR_C128>(bm, L, m, va, conja, vb, conjb, sb, part, s);
    case AR_HI:
      return dispatch_bm<R, AR_HI>(bm, L, m, va, conja, vb, conjb, sb, part, s);
    case AR_HI64:
      return dispatch_bm<R, AR_HI64>(bm, L, m, va, conja, vb, conjb, sb, part, s);
    default:
      return dispatch_bm<R, AR_HILO>(bm, L, m, va, conja, vb, conjb, sb, part, s);
  }
}

// ----------------------------------------------------------------- ingest
// One workgroup per source column j; entry (i, j) of the packed upper
// triangle goes to block (i / R, j / R) at (j % R) * R + (i % R).  Diagonal
// entries are halved (A: real part only).
__global__ void __launch_bounds__(kThreads)
    ingest_kernel(const void* __restrict__ src, int src_c64, int64_t j0, int64_t base, int R,
                  int nb, int is_a, int hilo, void* __restrict__ dst, void* __restrict__ dst_lo) {
  const int64_t j = j0 + blockIdx.x;
  const int64_t off = j * (j + 1) / 2 - base;
  const int Q = (int)(j / R), c = (int)(j % R);
  for (int64_t i = threadIdx.x; i <= j; i += kThreads) {
    double re, im;
    if (src_c64) {
      const float2 v = static_cast<const float2*>(src)[off + i];
      re = v.x;
      im = v.y;
    } else {
      const double2 v = static_cast<const double2*>(src)[off + i];
      re = v.x;
      im = v.y;
    }
    if (i == j) {
      re *= 0.5;
      im = is_a ? 0.0 : 0.5 * im;
    }
    const int P = (int)(i / R), r = (int)(i % R);
    const int64_t blk = (int64_t)P * nb - (int64_t)P * (P - 1) / 2 + (Q - P);
    const size_t d = (size_t)blk * R * R + (size_t)c * R + r;
    if (hilo) {
      const float hr = __double2float_rn(re), hi = __double2float_rn(im);
      static_cast<float2*>(dst)[d] = make_float2(hr, hi);
      static_cast<float2*>(dst_lo)[d] =
          make_float2(__double2float_rn(re - (double)hr), __double2float_rn(im - (double)hi));
    } else {
      static_cast<double2*>(dst)[d] = make_double2(re, im);
    }
  }
}

// ------------------------------------------------------- continued fraction
// One thread per frequency: g = 1 / (s - alpha_{n-1}), then
// g = 1 / (s - alpha_j - beta_j^2 g) down to j = 0; chi = scale g.  The
// coefficients are read by every thread of a wave at the same address.
__global__ void __launch_bounds__(kThreads)
    cfrac_kernel(int ph, int n, const double* __restrict__ alpha, const double* __restrict__ beta,
                 double scale, const double* __restrict__ freq, int nw, double eta, double2* __restrict__ chi) {
  const int f = blockIdx.x * kThreads + threadIdx.x;
  if (f >= nw) return;
  const double zr = freq[f], zi = eta;
  const double sr = ph ? zr * zr - zi * zi : zr, si = ph ? 2.0 * zr * zi : zi;
  double gr = 0.0, gi = 0.0;
  for (int j = n - 1; j >= 0; --j) {
    const double b2 = (j < n - 1) ? beta[j] * beta[j] : 0.0;
    const double dr = sr - alpha[j] - b2 * gr, di = si - b2 * gi;
    const double den = dr * dr + di * di;
    gr = dr / den;
    gi = -di / den;
  }
  chi[f] = make_double2(scale * gr, scale * gi);
}

// -------------------------------------------------- orthogonalization (CGS)
// h[q ncol + c] = sum_i conj(V[i, c]) w_q[i] for the NW vectors w_q = W + q ldw
// (NW = 1: columns of V0, then of V1), in one launch: a workgroup of 16 waves
// takes two columns, wave w rows 64 (w + 16 t) + lane; the waves' sums meet in
// LDS and are added in wave order.  For vectors up to kDotRows rows, where the
// chunk partials of cdot_part_kernel and their sum in a second launch are
// latency only: n = 4096, 64 columns 8.0 us for both launches, 3.3 us here;
// n = 10048 8.1 against 5.2 us; at n = 20736 a wave's 20 row steps take longer
// (8 columns: 5.6 against 8.4 us).  Four columns per workgroup leave half the
// workgroups and took 4.2 us at n = 4096.
constexpr int64_t kDotRows = 12288;
template <int NW>
__global__ void __launch_bounds__(1024)
    cdot_short_kernel(const double2* __restrict__ V0, int n0, const double2* __restrict__ V1, int n1, int64_t ld,
                      const double2* __restrict__ W, int64_t ldw, int64_t n, double2* __restrict__ h) {
  constexpr int CB = 2, NVAL = 2 * CB * NW;
  constexpr int GV = NVAL % 16 == 0 ? 16 : NVAL % 8 == 0 ? 8 : 4;  // values per wavefront sum
  static_assert(NVAL % GV == 0, "whole groups of values");
  __shared__ double red[16][NVAL];
  const int ncol = n0 + n1;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int c0 = blockIdx.x * CB;
  const double2* col[CB];
#pragma unroll
  for (int u = 0; u < CB; ++u) {
    const int c = c0 + u < ncol ? c0 + u : c0;  // past the end: a valid column, result unused
    col[u] = c < n0 ? V0 + (size_t)c * ld : V1 + (size_t)(c - n0) * ld;
  }
  double vals[NVAL];  // value 2 (q CB + u) + component
#pragma unroll
  for (int j = 0; j < NVAL; ++j) vals[j] = 0.0;
#pragma unroll 4
  for (int64_t i = wave * 64 + lane; i < n; i += 1024) {
    double2 v[CB], w[NW];
#pragma unroll
    for (int u = 0; u < CB; ++u) v[u] = col[u][i];
#pragma unroll
    for (int q = 0; q < NW; ++q) w[q] = W[(size_t)q * ldw + i];
#pragma unroll
    for (int q = 0; q < NW; ++q)
#pragma unroll
      for (int u = 0; u < CB; ++u) {
        const int j = 2 * (q * CB + u);
        mac(vals[j], v[u].x, w[q].x);
        mac(vals[j], v[u].y, w[q].y);
        mac(vals[j + 1], v[u].x, w[q].y);
        mac(vals[j + 1], -v[u].y, w[q].x);
      }
  }
#pragma unroll
  for (int g = 0; g < NVAL / GV; ++g) {
    double t[GV];
#pragma unroll
    for (int j = 0; j < GV; ++j) t[j] = vals[g * GV + j];
    red[wave][g * GV + wave_sum_index<GV>(lane)] = wave_sum_n<GV>(t);
  }
  __syncthreads();
  for (int j = threadIdx.x; j < NVAL; j += 1024) {
    double t = red[0][j];
#pragma unroll
    for (int w = 1; w < 16; ++w) t += red[w][j];
    const int q = j / (2 * CB), u = (j / 2) % CB;
    if (c0 + u < ncol) reinterpret_cast<double*>(h)[2 * ((size_t)q * ncol + c0 + u) + (j & 1)] = t;
  }
}

// part[chunk * ncol + c] = sum over the 256-row chunk of conj(V[i, c]) w[i].
// Grid (chunks, ceil(ncol / (4 cpw))); wave w of the group handles cpw columns
// (dot_cpw), four at a time: the 16 loads of four columns are issued together, then the
// eight sums over the wavefront go through LDS (lds_group_sum: eight values
// per lane in, one sum per eight-lane group out); lane l holds rows
// l + 64 s (s < 4) of w in registers.
__global__ void __launch_bounds__(kThreads)
    cdot_part_kernel(const double2* __restrict__ V0, int n0, const double2* __restrict__ V1,
                     int n1, int64_t ld, const double2* __restrict__ w, int64_t n,
                     double2* __restrict__ part, int cpw) {
  __shared__ double stg[4][8 * stage_ld(8)];  // per wave: the column-sum stage
  const int ncol = n0 + n1;
  const int64_t r0 = (int64_t)blockIdx.x * kChunk;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  double wr[4], wi[4];
  bool rin[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int64_t i = r0 + lane + 64 * s;
    rin[s] = i < n;
    const double2 v = rin[s] ? w[i] : make_double2(0.0, 0.0);
    wr[s] = v.x;
    wi[s] = v.y;
  }
  const int cbeg = (blockIdx.y * 4 + wave) * cpw;
  const int cend = min(cbeg + cpw, ncol);
  for (int t0 = cbeg; t0 < cend; t0 += 4) {
    double2 v[4][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = t0 + u < cend ? t0 + u : t0;  // past the end: a valid column, result unused
      const double2* col = (c < n0) ? V0 + (size_t)c * ld : V1 + (size_t)(c - n0) * ld;
#pragma unroll
      for (int s = 0; s < 4; ++s) v[u][s] = rin[s] ? col[r0 + lane + 64 * s] : make_double2(0.0, 0.0);
    }
    double sr[4], si[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      sr[u] = 0.0;
      si[u] = 0.0;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        sr[u] += v[u][s].x * wr[s] + v[u][s].y * wi[s];
        si[u] += v[u][s].x * wi[s] - v[u][s].y * wr[s];
      }
    }
    double vals[8];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      vals[2 * u] = sr[u];
      vals[2 * u + 1] = si[u];
    }
    const double sum = lds_group_sum<8>(vals, stg[wave], lane);
    wave_lds_sync();
    const int j = lane >> 3, u = j >> 1;
    if ((lane & 7) == 0 && t0 + u < cend)
      reinterpret_cast<double*>(part)[2 * ((size_t)blockIdx.x * ncol + t0 + u) + (j & 1)] = sum;
  }
}

// h[c] = sum over chunks of part[chunk * ncol + c], chunks in order.
__global__ void __launch_bounds__(kThreads)
    colsum_kernel(const double2* __restrict__ part, int64_t nch, int ncol, double2* __restrict__ h) {
  // one wavefront per column: lanes stride over the chunks, then a fixed-order
  // wavefront reduction (deterministic)
  const int c = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (c >= ncol) return;
  double sr = 0.0, si = 0.0;
  for (int64_t k = lane; k < nch; k += 64) {
    const double2 v = part[(size_t)k * ncol + c];
    sr += v.x;
    si += v.y;
  }
  sr = wave_sum(sr);
  si = wave_sum(si);
  if (lane == 0) h[c] = make_double2(sr, si);
}

// w[i] -= sum_c V[i, c] h[c];  z[i] -= sum_c P[i, c] h[c] (WithZ).
// real_h 1: h[c] -> Re h[c]; 2: Re h[c] on the first n0 columns and
// i Im h[c] on the others (a real coefficient on each basis vector and on
// each i-multiple of the second basis).
//
// A workgroup takes 256 / CG rows, thread group g of CG the g-th share of the
// columns, whose sums meet in LDS in group order.  One row per thread with all
// its columns, as this kernel was first written, is a serial chain on a few CUs
// for short vectors (n = 4096: 16 workgroups, 19 us for 200 columns of V and P
// against 4.6 us in 16 groups); at HBM-bound lengths the groups cost nothing
// (gemv_groups).  The column loops of the two bases are separate and take
// batches of 8 columns so that several loads are in flight per thread.
template <bool WithZ>
__device__ __forceinline__ void gemv_range(const double2* __restrict__ V, const double2* __restrict__ P, int64_t ld,
                                           const double2* hs, int c, int end, int64_t i, double& ar, double& ai,
                                           double& br, double& bi) {
  // batches of 8 columns: all loads of a batch are issued before the first use
  for (; c + 8 <= end; c += 8) {
    double2 v[8], q[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = V[(size_t)(c + u) * ld + i];
    if (WithZ) {
#pragma unroll
      for (int u = 0; u < 8; ++u) q[u] = P[(size_t)(c + u) * ld + i];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const double2 hc = hs[c + u];
      ar += v[u].x * hc.x - v[u].y * hc.y;
      ai += v[u].x * hc.y + v[u].y * hc.x;
      if (WithZ) {
        br += q[u].x * hc.x - q[u].y * hc.y;
        bi += q[u].x * hc.y + q[u].y * hc.x;
      }
    }
  }
  for (; c < end; ++c) {
    const double2 hc = hs[c];
    const double2 v = V[(size_t)c * ld + i];
    ar += v.x * hc.x - v.y * hc.y;
    ai += v.x * hc.y + v.y * hc.x;
    if (WithZ) {
      const double2 q = P[(size_t)c * ld + i];
      br += q.x * hc.x - q.y * hc.y;
      bi += q.x * hc.y + q.y * hc.x;
    }
  }
}

template <bool WithZ, int CG>
__global__ void __launch_bounds__(kThreads)
    cgemv_sub_kernel(const double2* __restrict__ V0, int n0, const double2* __restrict__ V1, int n1,
                     const double2* __restrict__ P0, const double2* __restrict__ P1, int64_t ld,
                     const double2* __restrict__ h, int real_h, double2* __restrict__ w,
                     double2* __restrict__ z, int64_t n) {
  extern __shared__ double2 hs[];  // the coefficients, then the groups' sums
  constexpr int RW = kThreads / CG;
  const int ncol = n0 + n1;
  for (int c = threadIdx.x; c < ncol; c += kThreads) {
    double2 v = h[c];
    if (real_h == 1 || (real_h == 2 && c < n0))
      v.y = 0.0;
    else if (real_h == 2)
      v.x = 0.0;
    hs[c] = v;
  }
  __syncthreads();
  const int r = threadIdx.x % RW, g = threadIdx.x / RW;
  const int64_t i = (int64_t)blockIdx.x * RW + r;
  double ar = 0.0, ai = 0.0, br = 0.0, bi = 0.0;
  if (i < n) {
    const int c0 = (int)((int64_t)ncol * g / CG), c1 = (int)((int64_t)ncol * (g + 1) / CG);
    if (c0 < n0) gemv_range<WithZ>(V0, P0, ld, hs, c0, min(c1, n0), i, ar, ai, br, bi);
    if (c1 > n0) gemv_range<WithZ>(V1, P1, ld, hs + n0, max(c0 - n0, 0), c1 - n0, i, ar, ai, br, bi);
  }
  __syncthreads();
  hs[threadIdx.x] = make_double2(ar, ai);
  if (WithZ) hs[kThreads + threadIdx.x] = make_double2(br, bi);
  __syncthreads();
  if (g != 0 || i >= n) return;
#pragma unroll
  for (int t = 1; t < CG; ++t) {
    ar += hs[t * RW + r].x;
    ai += hs[t * RW + r].y;
    if (WithZ) {
      br += hs[kThreads + t * RW + r].x;
      bi += hs[kThreads + t * RW + r].y;
    }
  }
  double2 wv = w[i];
  wv.x -= ar;
  wv.y -= ai;
  w[i] = wv;
  if (WithZ) {
    double2 zv = z[i];
    zv.x -= br;
    zv.y -= bi;
    z[i] = zv;
  }
}

// Several vectors against one basis, one read of the basis for all of them
// (the block steps of the full-H iteration).  part[chunk * NW ncol + q ncol +
// c] = sum over the chunk of conj(V[i, c]) w_q[i], w_q = W + q ldw; the same
// layout of waves, columns and loads as cdot_part_kernel, with the NW
// vectors' rows held in registers.
template <int NW>
__global__ void __launch_bounds__(kThreads)
    cdotm_part_kernel(const double2* __restrict__ V, int ncol, int64_t ld, const double2* __restrict__ W,
                      int64_t ldw, int64_t n, double2* __restrict__ part, int cpw) {
  __shared__ double stg[4][8 * stage_ld(8)];  // per wave: the column-sum stage
  const int64_t r0 = (int64_t)blockIdx.x * kChunk;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  double wr[NW][4], wi[NW][4];
  bool rin[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) rin[s] = r0 + lane + 64 * s < n;
#pragma unroll
  for (int q = 0; q < NW; ++q)
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const double2 v = rin[s] ? W[(size_t)q * ldw + r0 + lane + 64 * s] : make_double2(0.0, 0.0);
      wr[q][s] = v.x;
      wi[q][s] = v.y;
    }
  const int cbeg = (blockIdx.y * 4 + wave) * cpw;
  const int cend = min(cbeg + cpw, ncol);
  for (int t0 = cbeg; t0 < cend; t0 += 4) {
    double2 v[4][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = t0 + u < cend ? t0 + u : t0;  // past the end: a valid column, result unused
      const double2* col = V + (size_t)c * ld;
#pragma unroll
      for (int s = 0; s < 4; ++s) v[u][s] = rin[s] ? col[r0 + lane + 64 * s] : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int q = 0; q < NW; ++q) {
      double sr[4], si[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        sr[u] = 0.0;
        si[u] = 0.0;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          sr[u] += v[u][s].x * wr[q][s] + v[u][s].y * wi[q][s];
          si[u] += v[u][s].x * wi[q][s] - v[u][s].y * wr[q][s];
        }
      }
      // the eight sums over the wavefront through LDS: lane group j = lane / 8
      // holds value j (column u = j / 2, real part for even j)
      double vals[8];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        vals[2 * u] = sr[u];
        vals[2 * u + 1] = si[u];
      }
      const double sum = lds_group_sum<8>(vals, stg[wave], lane);
      wave_lds_sync();
      const int j = lane >> 3, u = j >> 1;
      if ((lane & 7) == 0 && t0 + u < cend)
        reinterpret_cast<double*>(part)[2 * ((size_t)blockIdx.x * NW * ncol + (size_t)q * ncol + t0 + u) + (j & 1)] =
            sum;
    }
  }
}

// w_q[i] -= sum_c V[i, c] h[q ldh + c] for q < NW, each basis entry loaded once
// for all NW vectors; rows and column groups as in cgemv_sub_kernel.
template <int NW, int CG>
__global__ void __launch_bounds__(kThreads)
    cgemvm_sub_kernel(const double2* __restrict__ V, int ncol, int64_t ld, const double2* __restrict__ h,
                      int ldh, double2* __restrict__ W, int64_t ldw, int64_t n) {
  extern __shared__ double2 hs[];  // NW * ncol coefficients, then the groups' sums
  constexpr int RW = kThreads / CG;
  for (int t = threadIdx.x; t < NW * ncol; t += kThreads) hs[t] = h[(size_t)(t / ncol) * ldh + t % ncol];
  __syncthreads();
  const int r = threadIdx.x % RW, g = threadIdx.x / RW;
  const int64_t i = (int64_t)blockIdx.x * RW + r;
  double ar[NW], ai[NW];
#pragma unroll
  for (int q = 0; q < NW; ++q) ar[q] = ai[q] = 0.0;
  if (i < n) {
    int c = (int)((int64_t)ncol * g / CG);
    const int end = (int)((int64_t)ncol * (g + 1) / CG);
    for (; c + 8 <= end; c += 8) {
      double2 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = V[(size_t)(c + u) * ld + i];
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int q = 0; q < NW; ++q) {
          const double2 hc = hs[q * ncol + c + u];
          ar[q] += v[u].x * hc.x - v[u].y * hc.y;
          ai[q] += v[u].x * hc.y + v[u].y * hc.x;
        }
    }
    for (; c < end; ++c) {
      const double2 v = V[(size_t)c * ld + i];
#pragma unroll
      for (int q = 0; q < NW; ++q) {
        const double2 hc = hs[q * ncol + c];
        ar[q] += v.x * hc.x - v.y * hc.y;
        ai[q] += v.x * hc.y + v.y * hc.x;
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NW; ++q) hs[q * kThreads + threadIdx.x] = make_double2(ar[q], ai[q]);
  __syncthreads();
  if (g != 0 || i >= n) return;
#pragma unroll
  for (int q = 0; q < NW; ++q)
#pragma unroll
    for (int t = 1; t < CG; ++t) {
      ar[q] += hs[q * kThreads + t * RW + r].x;
      ai[q] += hs[q * kThreads + t * RW + r].y;
    }
#pragma unroll
  for (int q = 0; q < NW; ++q) {
    double2 wv = W[(size_t)q * ldw + i];
    wv.x -= ar[q];
    wv.y -= ai[q];
    W[(size_t)q * ldw + i] = wv;
  }
}

// part[chunk] = Re sum conj(w_i) z_i over the chunk.
__global__ void __launch_bounds__(kThreads)
    rdot_part_kernel(const double2* __restrict__ w, const double2* __restrict__ z, int64_t n,
                     double* __restrict__ part) {
  __shared__ double sh[4];
  const int64_t i = (int64_t)blockIdx.x * kChunk + threadIdx.x;
  double s = 0.0;
  if (i < n) {
    const double2 a = w[i], b = z[i];
    s = a.x * b.x + a.y * b.y;
  }
  s = block_sum(s, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// 1 / beta of beta^2 = b2; the first thread of the grid records alpha, beta.
__device__ __forceinline__ double norm_scale(double b2, const double2* __restrict__ h1, const double2* __restrict__ h2,
                                             int jh, double* __restrict__ alpha, double* __restrict__ beta, int j,
                                             int* __restrict__ flag) {
  // b2 < 0: the K1 metric is indefinite (M not positive definite);
  // b2 == 0: exact breakdown (invariant subspace), the vector stays zero.
  const bool nonfinite = !isfinite(b2);
  const bool indefinite = b2 < 0.0;
  const bool bad = nonfinite || indefinite || !(b2 > 0.0);
  const double bt = bad ? 1.0 : sqrt(b2);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (alpha) alpha[j] = (h1 ? h1[jh].x : 0.0) + (h2 ? h2[jh].x : 0.0);
    if (beta) beta[j] = bad ? 0.0 : bt;
    // the first failure is the one reported (later ones are its consequences)
    if (flag && (nonfinite || indefinite) && flag[0] == 0) flag[0] = nonfinite ? 2 : 1;
  }
  return 1.0 / bt;
}

// Every workgroup sums the chunk partials in the same order (identical
// beta everywhere).
__global__ void __launch_bounds__(kThreads)
    normalize_kernel(double2* __restrict__ w, double2* __restrict__ z, int64_t n,
                     const double* __restrict__ part, int64_t nch, const double2* __restrict__ h1,
                     const double2* __restrict__ h2, int jh, double* __restrict__ alpha,
                     double* __restrict__ beta, int j, int* __restrict__ flag) {
  __shared__ double sh[4];
  double s = 0.0;
  for (int64_t k = threadIdx.x; k < nch; k += kThreads) s += part[k];
  const double inv = norm_scale(block_sum(s, sh), h1, h2, jh, alpha, beta, j, flag);
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  double2 a = w[i];
  a.x *= inv;
  a.y *= inv;
  w[i] = a;
  if (z && z != w) {
    double2 b = z[i];
    b.x *= inv;
    b.y *= inv;
    z[i] = b;
  }
}

// The dot product and the scaling of a short vector in one launch: one
// workgroup of 1024 threads holds up to 4 rows of w and z per thread in
// registers between the two (n = 1024 5.2 -> 3.3 us, 4096 5.2 -> 4.2 us, level
// at 8192).
constexpr int64_t kNormRows = 4096;
__global__ void __launch_bounds__(1024)
    normalize_short_kernel(double2* __restrict__ w, double2* __restrict__ z, int64_t n,
                           const double2* __restrict__ h1, const double2* __restrict__ h2, int jh,
                           double* __restrict__ alpha, double* __restrict__ beta, int j, int* __restrict__ flag) {
  __shared__ double sh[16];
  constexpr int NR = kNormRows / 1024;
  const bool two = z && z != w;
  double2 a[NR], b[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int64_t i = threadIdx.x + 1024 * r;
    a[r] = i < n ? w[i] : make_double2(0.0, 0.0);
    b[r] = !two ? a[r] : i < n ? z[i] : make_double2(0.0, 0.0);
  }
  double s = 0.0;
#pragma unroll
  for (int r = 0; r < NR; ++r) s += a[r].x * b[r].x + a[r].y * b[r].y;
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  double b2 = 0.0;
#pragma unroll
  for (int q = 0; q < 16; ++q) b2 += sh[q];
  const double inv = norm_scale(b2, h1, h2, jh, alpha, beta, j, flag);
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int64_t i = threadIdx.x + 1024 * r;
    if (i >= n) break;
    w[i] = make_double2(a[r].x * inv, a[r].y * inv);
    if (two) z[i] = make_double2(b[r].x * inv, b[r].y * inv);
  }
}

// ------------------------------------------------------- FP64 MFMA GEMM
// C (M x N) = A (M x K) * B (K x N), column-major, FP64, on
// v_mfma_f64_16x16x4f64.  Workgroup tile 64 x 64 (4 waves, each 32 x 32 =
// 2 x 2 MFMA tiles); K in steps of 4.  Lane layout of the 16x16x4 FP64
// instruction (measured on gfx950): A[i][k] in lane i + 16 k; B[k][j] in
// lane j + 16 k; result D[i][j] in lane j + 16 (i % 4), register i / 4.
typedef double dbl4 __attribute__((ext_vector_type(4)));

__global__ void __launch_bounds__(kThreads)
    dgemm_mfma_kernel(int64_t M, int N, int K, const double* __restrict__ A, int64_t lda,
                      const double* __restrict__ B, int64_t ldb, double* __restrict__ C,
                      int64_t ldc) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t m0 = (int64_t)blockIdx.x * 64 + (wave & 1) * 32;
  const int n0 = blockIdx.y * 64 + (wave >> 1) * 32;
  const int li = lane & 15, lk = lane >> 4;
  dbl4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = dbl4{0.0, 0.0, 0.0, 0.0};
  for (int k0 = 0; k0 < K; k0 += 4) {
    const int k = k0 + lk;
    double av[2], bv[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const int64_t i = m0 + a * 16 + li;
      av[a] = (i < M && k < K) ? A[(size_t)k * lda + i] : 0.0;
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int jj = n0 + b * 16 + li;
      bv[b] = (jj < N && k < K) ? B[(size_t)jj * ldb + k] : 0.0;
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
        acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], acc[a][b], 0, 0, 0);
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int jj = n0 + b * 16 + li;
      if (jj >= N) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t i = m0 + a * 16 + 4 * r + lk;
        if (i < M) C[(size_t)jj * ldc + i] = acc[a][b][r];
      }
    }
}

// Complex C (M x N) = A (M x K) * B (K x N), column-major complex128, on the
// same FP64 MFMA tile: four real products per complex one, two accumulators.
__global__ void __launch_bounds__(kThreads)
    zgemm_mfma_kernel(int64_t M, int N, int K, const double2* __restrict__ A, int64_t lda,
                      const double2* __restrict__ B, int64_t ldb, double2* __restrict__ C,
                      int64_t ldc) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t m0 = (int64_t)blockIdx.x * 64 + (wave & 1) * 32;
  const int n0 = blockIdx.y * 64 + (wave >> 1) * 32;
  const int li = lane & 15, lk = lane >> 4;
  dbl4 cr[2][2], ci[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      cr[a][b] = dbl4{0.0, 0.0, 0.0, 0.0};
      ci[a][b] = dbl4{0.0, 0.0, 0.0, 0.0};
    }
  for (int k0 = 0; k0 < K; k0 += 4) {
    const int k = k0 + lk;
    double2 av[2], bv[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const int64_t i = m0 + a * 16 + li;
      av[a] = (i < M && k < K) ? A[(size_t)k * lda + i] : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int jj = n0 + b * 16 + li;
      bv[b] = (jj < N && k < K) ? B[(size_t)jj * ldb + k] : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        cr[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a].x, bv[b].x, cr[a][b], 0, 0, 0);
        cr[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a].y, -bv[b].y, cr[a][b], 0, 0, 0);
        ci[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a].x, bv[b].y, ci[a][b], 0, 0, 0);
        ci[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a].y, bv[b].x, ci[a][b], 0, 0, 0);
      }
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int jj = n0 + b * 16 + li;
      if (jj >= N) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t i = m0 + a * 16 + 4 * r + lk;
        if (i < M) C[(size_t)jj * ldc + i] = make_double2(cr[a][b][r], ci[a][b][r]);
      }
    }
}

// ------------------------------------------------------------ small kernels
__global__ void __launch_bounds__(kThreads)
    colnorm_part_kernel(const double2* __restrict__ V, int ncol, int64_t ld, int64_t n,
                        double* __restrict__ part) {
  // grid (chunks, ceil(ncol / 4)): one column per wave
  const int64_t r0 = (int64_t)blockIdx.x * kChunk;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int c = blockIdx.y * 4 + wave;
  if (c >= ncol) return;
  double s = 0.0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t i = r0 + lane + 64 * q;
    if (i < n) {
      const double2 v = V[(size_t)c * ld + i];
      s += v.x * v.x + v.y * v.y;
    }
  }
  s = wave_sum(s);
  if (lane == 0) part[(size_t)blockIdx.x * ncol + c] = s;
}

__global__ void __launch_bounds__(kThreads)
    colsum_real_kernel(const double* __restrict__ part, int64_t nch, int ncol, double* __restrict__ h) {
  const int c = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (c >= ncol) return;
  double s = 0.0;
  for (int64_t k = lane; k < nch; k += 64) s += part[(size_t)k * ncol + c];
  s = wave_sum(s);
  if (lane == 0) h[c] = s;
}

__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}

__global__ void __launch_bounds__(kThreads)
    start_vector_kernel(double2* __restrict__ v, int64_t n, uint64_t seed) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  const uint64_t a = splitmix64(seed * 0x100000001B3ull + 2 * (uint64_t)i);
  const uint64_t b = splitmix64(seed * 0x100000001B3ull + 2 * (uint64_t)i + 1);
  v[i] = make_double2((double)(a >> 11) * 0x1.0p-53 - 0.5, (double)(b >> 11) * 0x1.0p-53 - 0.5);
}

// v[i] = sv v[i] + sum over columns c = q, q + b, q + 2b, ... < k of
// X[i + c ld] (+ ys conj(Y[i + c ld]) when Y is given)
__global__ void __launch_bounds__(kThreads)
    warm_sum_kernel(const double2* __restrict__ X, const double2* __restrict__ Y, double ys, int64_t ld, int64_t n,
                    int k, int b, int q, double sv, double2* __restrict__ v) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  double re = 0.0, im = 0.0;
  for (int c = q; c < k; c += b) {
    const double2 x = X[i + (size_t)c * ld];
    re += x.x;
    im += x.y;
    if (Y) {
      const double2 y = Y[i + (size_t)c * ld];
      re = fma(ys, y.x, re);
      im = fma(-ys, y.y, im);
    }
  }
  const double2 o = v[i];
  v[i] = make_double2(fma(sv, o.x, re), fma(sv, o.y, im));
}

// x[:, c] = -x[:, c] (n rows, column stride ld), c = blockIdx.y
__global__ void __launch_bounds__(kThreads) neg_cols_kernel(double2* __restrict__ x, int64_t ld, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  double2* p = x + (size_t)blockIdx.y * ld + i;
  *p = make_double2(-p->x, -p->y);
}

__global__ void __launch_bounds__(kThreads)
    ph_vectors_kernel(const double2* __restrict__ U, const double2* __restrict__ P, int64_t ld,
                      const double* __restrict__ omega, int64_t n, double2* __restrict__ X,
                      double2* __restrict__ Y, int64_t ldo) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int c = blockIdx.y;
  if (i >= n) return;
  const double w = omega[c];
  const double s = 0.5 / sqrt(w);
  const double2 u = U[(size_t)c * ld + i], p = P[(size_t)c * ld + i];
  X[(size_t)c * ldo + i] = make_double2(s * (w * u.x + p.x), s * (w * u.y + p.y));
  Y[(size_t)c * ldo + i] = make_double2(s * (w * u.x - p.x), -s * (w * u.y - p.y));
}

// MV[:, c] (+)= s [omega p + kp; conj(omega p - kp)], s = 1 / (2 sqrt(omega)):
// M v for v = s [omega u + p; conj(omega u - p)] from p = K1 u and kp = K2 p
// (columns of length 2 ld, top and bottom halves; add != 0 accumulates).
__global__ void __launch_bounds__(kThreads)
    ph_mvectors_kernel(const double2* __restrict__ P, const double2* __restrict__ KP, int64_t ld,
                       const double* __restrict__ omega, int64_t n, double2* __restrict__ MV, int64_t ldo,
                       int64_t ldh, int add) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int c = blockIdx.y;
  if (i >= n) return;
  const double w = omega[c];
  const double s = 0.5 / sqrt(w);
  const double2 p = P[(size_t)c * ld + i], kp = KP[(size_t)c * ld + i];
  double2 t = make_double2(s * (w * p.x + kp.x), s * (w * p.y + kp.y));
  double2 b = make_double2(s * (w * p.x - kp.x), -s * (w * p.y - kp.y));
  const size_t it = (size_t)c * ldo + i, ib = it + ldh;
  if (add) {
    const double2 t0 = MV[it], b0 = MV[ib];
    t.x += t0.x;
    t.y += t0.y;
    b.x += b0.x;
    b.y += b0.y;
  }
  MV[it] = t;
  MV[ib] = b;
}

// T[:, q] += H[:, q] (rows < cnt, columns < ncols); real_only drops Im(H).
__global__ void __launch_bounds__(kThreads)
    acc_cols_kernel(double2* __restrict__ T, int64_t ldT, const double2* __restrict__ H, int64_t ldh, int cnt,
                    int real_only) {
  const int i = blockIdx.x * kThreads + threadIdx.x;
  const int q = blockIdx.y;
  if (i >= cnt) return;
  const double2 v = H[(size_t)q * ldh + i];
  double2 t = T[(size_t)q * ldT + i];
  t.x += v.x;
  if (!real_only) t.y += v.y;
  T[(size_t)q * ldT + i] = t;
}

// ---------------------------------------------- FP64 refinement (full H)
// Columns of length 2N stored as [top (ld); bottom (ld)], column stride 2 ld.

// R[:, c] = Omega MV[:, c] - om[c] V[:, c], Omega = diag(I, -I).
__global__ void __launch_bounds__(kThreads)
    resid_h_kernel(const double2* __restrict__ MV, const double2* __restrict__ V,
                   const double* __restrict__ om, int64_t ld, int64_t n, double2* __restrict__ R) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int c = blockIdx.y;
  if (i >= n) return;
  const double w = om[c];
  const size_t t = (size_t)c * 2 * ld + i, b = t + ld;
  const double2 mt = MV[t], vt = V[t], mb = MV[b], vb = V[b];
  R[t] = make_double2(mt.x - w * vt.x, mt.y - w * vt.y);
  R[b] = make_double2(-mb.x - w * vb.x, -mb.y - w * vb.y);
}

// Diagonal correction t = (D - om)^{-1} r, D = diag(d, -d) the diagonal of H
// (two != 0) or D = diag(d) (TDA), d = diag A; denominators are kept at
// least floor in magnitude.
__global__ void __launch_bounds__(kThreads)
    precond_h_kernel(const double2* __restrict__ r, const double* __restrict__ d, double om,
                     double floor, int64_t ld, int64_t n, int two, double2* __restrict__ t) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  double dt = d[i] - om;
  if (fabs(dt) < floor) dt = dt < 0.0 ? -floor : floor;
  const double2 a = r[i];
  t[i] = make_double2(a.x / dt, a.y / dt);
  if (two) {
    double db = -d[i] - om;
    if (fabs(db) < floor) db = db < 0.0 ? -floor : floor;
    const double2 b = r[i + ld];
    t[i + ld] = make_double2(b.x / db, b.y / db);
  }
}

// X[:, c] = sqrt(om_c) top of V[:, c], Y[:, c] = sqrt(om_c) bottom (leading dimension n).
__global__ void __launch_bounds__(kThreads)
    h_out_kernel(const double2* __restrict__ V, const double* __restrict__ om, int64_t ld, int64_t n,
                 double2* __restrict__ X, double2* __restrict__ Y) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int c = blockIdx.y;
  if (i >= n) return;
  const double f = sqrt(om[c]);
  const double2 a = V[(size_t)c * 2 * ld + i], b = V[(size_t)c * 2 * ld + ld + i];
  X[(size_t)c * n + i] = make_double2(f * a.x, f * a.y);
  Y[(size_t)c * n + i] = make_double2(f * b.x, f * b.y);
}

// diag(A) in FP64 from the stored diagonal blocks (stored halved).
template <Arith AR>
__global__ void __launch_bounds__(kThreads)
    diag_a_kernel(const void* __restrict__ a, const void* __restrict__ alo, int R, int nb, int64_t n,
                  double* __restrict__ d) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  const int64_t P = i / R, r = i % R;
  const int64_t blk = P * nb - P * (P - 1) / 2;
  const size_t idx = (size_t)blk * R * R + (size_t)r * R + r;
  double v;
  if (AR == AR_C128) {
    v = static_cast<const double2*>(a)[idx].x;
  } else {
    v = (double)static_cast<const float2*>(a)[idx].x;
    if (AR == AR_HILO) v += (double)static_cast<const float2*>(alo)[idx].x;
  }
  d[i] = 2.0 * v;
}

// R[:, c] = W[:, c] - th[c] V[:, c]
__global__ void __launch_bounds__(kThreads)
    resid_cols_kernel(const double2* __restrict__ W, const double2* __restrict__ V,
                      const double* __restrict__ th, int64_t ld, int64_t n, double2* __restrict__ R) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int c = blockIdx.y;
  if (i >= n) return;
  const double t = th[c];
  const double2 w = W[(size_t)c * ld + i], v = V[(size_t)c * ld + i];
  R[(size_t)c * ld + i] = make_double2(w.x - t * v.x, w.y - t * v.y);
}

// dst[:, c] = i * scale_c * src[:, c]  (scale = 1 when sc == nullptr; per
// column 1 / sqrt(th[c]) when sqrt_inv != 0).
__global__ void __launch_bounds__(kThreads)
    times_i_kernel(const double2* __restrict__ src, int64_t lds, double2* __restrict__ dst,
                   int64_t ldd, int64_t n, const double* __restrict__ sc, int sqrt_inv) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int c = blockIdx.y;
  if (i >= n) return;
  double f = 1.0;
  if (sc) f = sqrt_inv ? 1.0 / sqrt(sc[c]) : sc[c];
  const double2 v = src[(size_t)c * lds + i];
  dst[(size_t)c * ldd + i] = make_double2(-f * v.y, f * v.x);
}

__global__ void __launch_bounds__(kThreads)
    copy_cols_kernel(const double2* __restrict__ src, int64_t lds, double2* __restrict__ dst,
                     int64_t ldd, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  dst[(size_t)blockIdx.y * ldd + i] = src[(size_t)blockIdx.y * lds + i];
}

__global__ void __launch_bounds__(kThreads)
    conj_copy_kernel(const double2* __restrict__ src, double2* __restrict__ dst, int64_t n, double sg) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  const double2 v = src[i];
  dst[i] = make_double2(sg * v.x, -sg * v.y);
}

__global__ void __launch_bounds__(kThreads)
    resid_part_kernel(const double2* __restrict__ out, const double2* __restrict__ v, int cj,
                      double so, int64_t n, double* __restrict__ part) {
  __shared__ double sh[4];
  const int64_t i = (int64_t)blockIdx.x * kChunk + threadIdx.x;
  double r2 = 0.0, v2 = 0.0;
  if (i < n) {
    const double2 o = out[i];
    double2 x = v[i];
    if (cj) x.y = -x.y;
    const double dr = o.x - so * x.x, di = o.y - so * x.y;
    r2 = dr * dr + di * di;
    v2 = x.x * x.x + x.y * x.y;
  }
  r2 = block_sum(r2, sh);
  v2 = block_sum(v2, sh);
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = r2;
    part[2 * blockIdx.x + 1] = v2;
  }
}

__global__ void __launch_bounds__(64) pair_sum_kernel(const double* __restrict__ part, int64_t nch,
                                                      double* __restrict__ res) {
  if (threadIdx.x != 0) return;
  double a = 0.0, b = 0.0;
  for (int64_t k = 0; k < nch; ++k) {
    a += part[2 * k];
    b += part[2 * k + 1];
  }
  res[0] = a;
  res[1] = b;
}

// Packed gradients on 64 x 64 tiles (I, J), I <= J, of the upper triangle:
//   G_A(i, j) = sum_c w_c (X_ic conj(X_jc) + conj(Y_ic) Y_jc),
//   G_B(i, j) = sum_c w_c (X_ic conj(Y_jc) + conj(Y_ic) X_jc),
// written packed (offset i + j (j + 1) / 2) with off-diagonal entries doubled
// and the diagonal of G_A real.  MODE 0 writes G_A (ga) and G_B (gb); MODE 1 /
// 2 instead accumulate, over the tile's entries, Re(conj(g_ij) C_ij) for the
// packed gradient entry g of G_A / G_B (doubled off the diagonal) and a packed
// component C of that block, and store the tile's sum in part[tile] (the other
// block's sums are not formed).
//
// A rank-k contraction on FP64 matrix cores (16x16x4).  With the four real
// components r = (Re x, Im x, Re y, Im y) of a pair as the k dimension of one
// instruction, r' = (Im x, -Re x, Re y, -Im y) on the row side and permutations
// of r on the column side,
//   Re G_A = r_i . r_j                       Im G_A = r'_i . (xr, xi, yi, yr)_j
//   Re G_B = r_i . (yr, yi, xr, xi)_j        Im G_B = r'_i . (yr, yi, xi, xr)_j,
// so a pair costs four instructions per 16 x 16 tile and no products beyond
// the 16 real ones of the definition.  TDA (no Y): two pairs per instruction,
// r = (Re x, Im x) of both, Re G_A = r_i . r_j, Im G_A = r'_i . r_j.  The
// column index j is the instruction's row, so a lane group holds 16
// consecutive rows i of a column and stores 256-byte segments.  Pairs pass
// through LDS in chunks of 8 (16 without Y), the next chunk's loads in flight
// under the current one's products; component rows are 80 doubles apart so
// that the 16 lanes of each component read distinct banks.
//
// Bound by the matrix cores: N = 5000, k = 64, PH (26 GFLOP, 355 us at the
// 72 TFLOP/s of a large FP64 product) 667 us with FMAs on 4 x 4 outputs per
// thread, 510 us here (TDA 396 -> 143 us);
// N = 16384, k = 16: 2033 -> 1901 us, of which the 4.3 GB written take about 870.
constexpr int kGT = 64;

template <int MODE, bool PH>
__global__ void __launch_bounds__(kThreads, 2)
    grad_tile_kernel(const double2* __restrict__ X, const double2* __restrict__ Y, int64_t ld,
                     const double* __restrict__ wgt, int k, int64_t n, double2* __restrict__ ga,
                     double2* __restrict__ gb, const double2* __restrict__ C, double* __restrict__ part) {
  constexpr int NK = 8;              // instruction k-steps per chunk
  constexpr int KP = PH ? NK : 2 * NK;  // pairs per chunk
  constexpr int LDC = 80;
  constexpr bool wantA = MODE != 2, wantB = MODE != 1 && PH;
  __shared__ double si[NK][4][LDC], sj[NK][4][LDC];
  __shared__ double sred[4];
  // tile (I, J) from the linear index over the upper triangle of tiles, column by column
  const int64_t b = blockIdx.x;
  int64_t J = (int64_t)((sqrt(8.0 * (double)b + 1.0) - 1.0) * 0.5);
  while (J * (J + 1) / 2 > b) --J;
  while ((J + 1) * (J + 2) / 2 <= b) ++J;
  const int64_t I = b - J * (J + 1) / 2;
  const int64_t i0 = I * kGT, j0 = J * kGT;
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  const int li = lane & 15, lk = lane >> 4;
  const int wi = (wave & 1) * 32, wj = (wave >> 1) * 32;  // this wave's 32 x 32 quarter

  // staging: thread t holds row t & 63, k-steps (t >> 6) + 4 e (e < 2), of each side
  const int row = t & 63, kq = t >> 6;
  const bool in_i = i0 + row < n, in_j = j0 + row < n;
  double2 pi[2][2], pj[2][2];  // [e][x, y] (TDA: [e][first, second pair])
  auto fetch = [&](int c0) {
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int c = PH ? c0 + kq + 4 * e : c0 + 2 * (kq + 4 * e) + h;
        const double2* src = PH && h ? Y : X;
        double2 vi = make_double2(0.0, 0.0), vj = vi;
        if (c < k) {
          if (in_i) {
            const double w = wgt[c];
            vi = src[(size_t)c * ld + i0 + row];
            vi = make_double2(w * vi.x, w * vi.y);
          }
          if (in_j) vj = src[(size_t)c * ld + j0 + row];
        }
        pi[e][h] = vi;
        pj[e][h] = vj;
      }
  };
  dbl4 acc[4][2][2];  // Re G_A, Im G_A, Re G_B, Im G_B
#pragma unroll
  for (int o = 0; o < 4; ++o)
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int c = 0; c < 2; ++c) acc[o][a][c] = dbl4{0.0, 0.0, 0.0, 0.0};
  // component of the lane for r' (sign on odd components) and the column permutations
  const int pr = PH ? (lk < 2 ? lk ^ 1 : lk) : lk ^ 1;
  const double sgn = (lk & 1) ? -1.0 : 1.0;
  const int p1 = PH ? (lk < 2 ? lk : lk ^ 1) : lk;  // (xr, xi, yi, yr)
  const int p2 = lk ^ 2;                            // (yr, yi, xr, xi)
  const int p3 = lk < 2 ? lk + 2 : 3 - lk;          // (yr, yi, xi, xr)

  fetch(0);
  for (int c0 = 0; c0 < k; c0 += KP) {
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        si[kq + 4 * e][2 * h][row] = pi[e][h].x;
        si[kq + 4 * e][2 * h + 1][row] = pi[e][h].y;
        sj[kq + 4 * e][2 * h][row] = pj[e][h].x;
        sj[kq + 4 * e][2 * h + 1][row] = pj[e][h].y;
      }
    __syncthreads();
    if (c0 + KP < k) fetch(c0 + KP);
#pragma unroll 2
    for (int s = 0; s < NK; ++s) {
      double ri[2], rp[2];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        ri[c] = si[s][lk][wi + 16 * c + li];
        rp[c] = sgn * si[s][pr][wi + 16 * c + li];
      }
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const int jj = wj + 16 * a + li;
        if (wantA) {
          const double q0 = sj[s][lk][jj], q1 = sj[s][p1][jj];
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            acc[0][a][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(q0, ri[c], acc[0][a][c], 0, 0, 0);
            acc[1][a][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(q1, rp[c], acc[1][a][c], 0, 0, 0);
          }
        }
        if (wantB) {
          const double q2 = sj[s][p2][jj], q3 = sj[s][p3][jj];
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            acc[2][a][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(q2, ri[c], acc[2][a][c], 0, 0, 0);
            acc[3][a][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(q3, rp[c], acc[3][a][c], 0, 0, 0);
          }
        }
      }
    }
    __syncthreads();
  }
  // entry (row i, column j): lane i + 16 (j % 4) of the tile, register j / 4
  double sum = 0.0;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t j = j0 + wj + 16 * a + 4 * r + lk;
      if (j >= n) continue;
      const int64_t off = j * (j + 1) / 2;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int64_t i = i0 + wi + 16 * c + li;
        if (i > j) continue;
        const double f = i == j ? 1.0 : 2.0;
        if (MODE == 0) {
          if (ga)
            ga[off + i] = i == j ? make_double2(acc[0][a][c][r], 0.0)
                                 : make_double2(f * acc[0][a][c][r], f * acc[1][a][c][r]);
          if (gb) gb[off + i] = make_double2(f * acc[2][a][c][r], f * acc[3][a][c][r]);
        } else {
          const double2 cv = C[off + i];
          const double gr = MODE == 1 ? acc[0][a][c][r] : acc[2][a][c][r];
          const double gi = MODE == 1 ? (i == j ? 0.0 : acc[1][a][c][r]) : acc[3][a][c][r];
          sum += f * (gr * cv.x + gi * cv.y);
        }
      }
    }
  if (MODE != 0) {
    sum = block_sum(sum, sred);
    if (t == 0) part[blockIdx.x] = sum;
  }
}

// part[block] = sum_i d_i sum_c wgt_c (|X_ci|^2 + |Y_ci|^2) over the block's rows.
__global__ void __launch_bounds__(kThreads)
    quad_diag_kernel(const double2* __restrict__ X, const double2* __restrict__ Y, int64_t ld,
                     const double* __restrict__ wgt, int k, const double* __restrict__ d, int64_t n,
                     double* __restrict__ part) {
  __shared__ double sh[4];
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  double acc = 0.0;
  if (i < n) {
    for (int c = 0; c < k; ++c) {
      const double2 x = X[(size_t)c * ld + i];
      double t = x.x * x.x + x.y * x.y;
      if (Y) {
        const double2 y = Y[(size_t)c * ld + i];
        t += y.x * y.x + y.y * y.y;
      }
      acc += wgt[c] * t;
    }
    acc *= d[i];
  }
  acc = block_sum(acc, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = acc;
}

}  // namespace

// ====================================================================== API
int choose_block(int64_t n) {
  const int cand[4] = {512, 256, 128, 64};
  for (int q = 0; q < 4; ++q) {
    const int64_t nb = (n + cand[q] - 1) / cand[q];
    if (nb * (nb + 1) / 2 >= 1024) return cand[q];
  }
  return 64;
}

void layout_blkmap_host(int nb, int2* out) {
  int64_t b = 0;
  for (int P = 0; P < nb; ++P)
    for (int Q = P; Q < nb; ++Q) out[b++] = make_int2(P, Q);
}

hipError_t matvec(const Layout& L, Arith ar, BMode bm, const MatPtrs& m, const double2* va, int conja,
                  const double2* vb, int conjb, double sb, double2* part, double2* out,
                  hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  hipError_t e;
  if (ev0) {
    e = hipEventRecord(ev0, s);
    if (e != hipSuccess) return e;
  }
  switch (L.R) {
    case 64:
      e = dispatch_ar<64>(ar, bm, L, m, va, conja, vb, conjb, sb, part, s);
      break;
    case 128:
      e = dispatch_ar<128>(ar, bm, L, m, va, conja, vb, conjb, sb, part, s);
      break;
    case 256:
      e = dispatch_ar<256>(ar, bm, L, m, va, conja, vb, conjb, sb, part, s);
      break;
    case 512:
      e = dispatch_ar<512>(ar, bm, L, m, va, conja, vb, conjb, sb, part, s);
      break;
    default:
      return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  if (ev1) {
    e = hipEventRecord(ev1, s);
    if (e != hipSuccess) return e;
  }
  const double2* rowpart = part;
  const double2* colpart = part + (size_t)L.nblk * L.R;
  const dim3 rgrid((unsigned)((L.n + 63) / 64));
  if (reduce_wide(L))
    hipLaunchKernelGGL(mv_reduce_kernel<16>, rgrid, dim3(1024), 0, s, rowpart, colpart, L.R, mv_slices(L), L.nb, L.n,
                       out, m.dc, m.dsign, va, conja);
  else
    hipLaunchKernelGGL(mv_reduce_kernel<4>, rgrid, dim3(256), 0, s, rowpart, colpart, L.R, mv_slices(L), L.nb, L.n,
                       out, m.dc, m.dsign, va, conja);
  return hipGetLastError();
}

int mv_slices(const Layout&) { return 1; }

size_t mv_part_elems(const Layout& L) { return (size_t)L.nblk * L.R * (1 + mv_slices(L)); }

size_t mh_part_elems(const Layout& L, int nh) {
  size_t mx = 0;
  for (int v = 1; v <= nh; ++v)
    mx = std::max(mx, (size_t)2 * v * L.nblk * L.R * 2 +  // row and column partials
                          (L.R >= 128 ? (size_t)2 * v * L.nb * L.R : 0));  // + staged u, w
  return mx;
}

size_t mk_part_elems(const Layout& L, int nv) {
  size_t mx = 0;
  for (int v = 1; v <= nv; ++v) {
    const int ns = L.R < mk_rows(v) ? 1 : L.R / mk_rows(v);
    mx = std::max(mx, (size_t)v * L.nblk * L.R * (1 + ns));
  }
  return mx;
}

hipError_t mh_apply(const Layout& L, Arith ar, const MatPtrs& m, int nh, const double2* V, int64_t ldv,
                    int64_t ldh, double2* part, double2* MV, double bsign, hipStream_t s, hipEvent_t ev0,
                    hipEvent_t ev1) {
  if (nh < 1 || nh > 4 || ar == AR_HI) return hipErrorInvalidValue;
  hipError_t e;
  if (ev0) {
    e = hipEventRecord(ev0, s);
    if (e != hipSuccess) return e;
  }
  switch (L.R) {
    case 64:
      e = dispatch_mh<64>(ar, nh, L, m, V, ldv, ldh, part, s);
      break;
    case 128:
      e = dispatch_mh<128>(ar, nh, L, m, V, ldv, ldh, part, s);
      break;
    case 256:
      e = dispatch_mh<256>(ar, nh, L, m, V, ldv, ldh, part, s);
      break;
    case 512:
      e = dispatch_mh<512>(ar, nh, L, m, V, ldv, ldh, part, s);
      break;
    default:
      return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  if (ev1) {
    e = hipEventRecord(ev1, s);
    if (e != hipSuccess) return e;
  }
  const double2* rowpart = part;
  const double2* colpart = part + (size_t)2 * nh * L.nblk * L.R;
  launch_mh_reduce(L, nh, 1, rowpart, colpart, MV, ldv, ldh, bsign, m, V, ldv, ldh, L.R == 64 ? 1 : 2, s);
  return hipGetLastError();
}

template <int R, int AR, int BM, int NV>
hipError_t launch_mk(const Layout& L, const MatPtrs& m, const double2* V, int64_t ldv, double sb, double2* part,
                     hipStream_t s) {
  if constexpr (R == 64) {
    launch_tile64<AR, BM == BM_CONJ ? T64_K : T64_A, NV>(L, m, V, ldv, 0, 0, nullptr, 0, sb, part, s);
  } else if constexpr (mk_on_mfma(R, AR, BM, NV)) {
    return launch_mfma<R, AR, BM == BM_CONJ ? T64_K : T64_A>(NV, L, m, V, ldv, L.n, sb, part, s);
  } else {
    using Sh = MkShape<R, AR, NV>;
    double2* rowpart = part;
    double2* colpart = part + (size_t)NV * L.nblk * R;
    hipLaunchKernelGGL((mk_block_kernel<R, AR, BM, NV>), dim3((unsigned)L.nblk, (unsigned)Sh::NS), dim3(kThreads),
                       0, s, m.a, m.alo, m.b, m.blo, L.blkmap, L.nblk, L.n, V, ldv, sb, rowpart, colpart);
  }
  return hipGetLastError();
}

template <int R, int AR, int BM>
hipError_t dispatch_mk_nv(int nv, const Layout& L, const MatPtrs& m, const double2* V, int64_t ldv, double sb,
                          double2* part, hipStream_t s) {
  switch (nv) {
    case 1:
      return launch_mk<R, AR, BM, 1>(L, m, V, ldv, sb, part, s);
    case 2:
      return launch_mk<R, AR, BM, 2>(L, m, V, ldv, sb, part, s);
    case 3:
      return launch_mk<R, AR, BM, 3>(L, m, V, ldv, sb, part, s);
    default:
      return launch_mk<R, AR, BM, 4>(L, m, V, ldv, sb, part, s);
  }
}

template <int R, int AR>
hipError_t dispatch_mk_bm(BMode bm, int nv, const Layout& L, const MatPtrs& m, const double2* V, int64_t ldv,
                          double sb, double2* part, hipStream_t s) {
  if (bm == BM_CONJ) return dispatch_mk_nv<R, AR, BM_CONJ>(nv, L, m, V, ldv, sb, part, s);
  return dispatch_mk_nv<R, AR, BM_NONE>(nv, L, m, V, ldv, sb, part, s);
}

template <int R>
hipError_t dispatch_mk(Arith ar, BMode bm, int nv, const Layout& L, const MatPtrs& m, const double2* V,
                       int64_t ldv, double sb, double2* part, hipStream_t s) {
  switch (ar) {
    case AR_C128:
      return dispatch_mk_bm<R, AR_C128>(bm, nv, L, m, V, ldv, sb, part, s);
    case AR_HI:
      return dispatch_mk_bm<R, AR_HI>(bm, nv, L, m, V, ldv, sb, part, s);
    case AR_HI64:
      return dispatch_mk_bm<R, AR_HI64>(bm, nv, L, m, V, ldv, sb, part, s);
    default:
      return dispatch_mk_bm<R, AR_HILO>(bm, nv, L, m, V, ldv, sb, part, s);
  }
}

hipError_t mk_apply(const Layout& L, Arith ar, BMode bm, const MatPtrs& m, int nv, const double2* V, int64_t ldv,
                    double sb, double2* part, double2* out, int64_t ldo, hipStream_t s, hipEvent_t ev0,
                    hipEvent_t ev1) {
  if (nv < 1 || nv > 4 || bm == BM_EXPLICIT) return hipErrorInvalidValue;
  hipError_t e;
  if (ev0) {
    e = hipEventRecord(ev0, s);
    if (e != hipSuccess) return e;
  }
  switch (L.R) {
    case 64:
      e = dispatch_mk<64>(ar, bm, nv, L, m, V, ldv, sb, part, s);
      break;
    case 128:
      e = dispatch_mk<128>(ar, bm, nv, L, m, V, ldv, sb, part, s);
      break;
    case 256:
      e = dispatch_mk<256>(ar, bm, nv, L, m, V, ldv, sb, part, s);
      break;
    case 512:
      e = dispatch_mk<512>(ar, bm, nv, L, m, V, ldv, sb, part, s);
      break;
    default:
      return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  if (ev1) {
    e = hipEventRecord(ev1, s);
    if (e != hipSuccess) return e;
  }
  // (the matrix-core pass writes one set of column partials)
  const int ns = mk_on_mfma(L.R, ar, bm, nv) || L.R < mk_rows(nv) ? 1 : L.R / mk_rows(nv);
  const double2* rowpart = part;
  const double2* colpart = part + (size_t)nv * L.nblk * L.R;
  launch_mh_reduce(L, nv, ns, rowpart, colpart, out, ldo, 0, 1.0, m, V, ldv, 0, 0, s);
  return hipGetLastError();
}

hipError_t ingest(const Layout& L, bool is_a, bool hilo, const void* src, bool src_c64, int64_t j0,
                  int64_t j1, void* dst, void* dst_lo, hipStream_t s) {
  if (j1 <= j0) return hipSuccess;
  hipLaunchKernelGGL(ingest_kernel, dim3((unsigned)(j1 - j0)), dim3(kThreads), 0, s, src,
                     (int)src_c64, j0, j0 * (j0 + 1) / 2, L.R, L.nb, (int)is_a, (int)hilo, dst,
                     dst_lo);
  return hipGetLastError();
}

// Columns per wave of the chunked dot products: 16 where the chunks and column
// groups fill the chip, else 4 (more workgroups, each one batch of loads long).
int dot_cpw(int64_t nch, int ncol) { return nch * ((ncol + 63) / 64) < 1024 ? 4 : 16; }

hipError_t cdot(const double2* V0, int n0, const double2* V1, int n1, int64_t ld, const double2* w,
                int64_t n, double2* part, double2* h, hipStream_t s) {
  const int ncol = n0 + n1;
  if (ncol == 0) return hipSuccess;
  if (n <= kDotRows) {
    hipLaunchKernelGGL(cdot_short_kernel<1>, dim3((unsigned)((ncol + 1) / 2)), dim3(1024), 0, s, V0, n0, V1, n1, ld, w, (int64_t)0, n, h);
    return hipGetLastError();
  }
  const int64_t nch = nchunks(n);
  const int cpw = dot_cpw(nch, ncol);
  hipLaunchKernelGGL(cdot_part_kernel, dim3((unsigned)nch, (unsigned)((ncol + 4 * cpw - 1) / (4 * cpw))),
                     dim3(kThreads), 0, s, V0, n0, V1, n1, ld, w, n, part, cpw);
  hipLaunchKernelGGL(colsum_kernel, dim3((unsigned)((ncol + 3) / 4)), dim3(kThreads), 0, s, part, nch, ncol, h);
  return hipGetLastError();
}

template <int NW>
hipError_t launch_cdotm(const double2* V, int ncol, int64_t ld, const double2* W, int64_t ldw, int64_t n,
                        double2* part, double2* h, hipStream_t s) {
  if (n <= kDotRows) {
    hipLaunchKernelGGL(cdot_short_kernel<NW>, dim3((unsigned)((ncol + 1) / 2)), dim3(1024), 0, s, V, ncol, nullptr, 0, ld, W, ldw, n, h);
    return hipGetLastError();
  }
  const int64_t nch = nchunks(n);
  const int cpw = dot_cpw(nch, ncol);
  hipLaunchKernelGGL(cdotm_part_kernel<NW>, dim3((unsigned)nch, (unsigned)((ncol + 4 * cpw - 1) / (4 * cpw))),
                     dim3(kThreads), 0, s, V, ncol, ld, W, ldw, n, part, cpw);
  hipLaunchKernelGGL(colsum_kernel, dim3((unsigned)((NW * ncol + 3) / 4)), dim3(kThreads), 0, s, part, nch, NW * ncol,
                     h);
  return hipGetLastError();
}

hipError_t cdotm(const double2* V, int ncol, int64_t ld, const double2* W, int64_t ldw, int nw, int64_t n,
                 double2* part, double2* h, hipStream_t s) {
  if (ncol == 0) return hipSuccess;
  switch (nw) {
    case 1:
      return launch_cdotm<1>(V, ncol, ld, W, ldw, n, part, h, s);
    case 2:
      return launch_cdotm<2>(V, ncol, ld, W, ldw, n, part, h, s);
    case 3:
      return launch_cdotm<3>(V, ncol, ld, W, ldw, n, part, h, s);
    case 4:
      return launch_cdotm<4>(V, ncol, ld, W, ldw, n, part, h, s);
    default:
      return hipErrorInvalidValue;
  }
}

// Column groups of the basis updates (cgemv_sub_kernel) by the rows n, from
// updates of two vectors by 200 columns (us, 16 / 4 / 1 groups): n = 4096
// 3.9 / 6.2 / 16.2, 10048 6.6 / 8.0 / 32, 20736 14.0 / 13.1 / 34.6, 65536
// 32.6 / 33.6 / 39.9, 200000 123 / 117 / 116.
int gemv_groups(int64_t n) { return n <= 16384 ? 16 : 4; }

// The LDS of an update: its coefficients, or the groups' sums where those are larger.
size_t gemv_lds(int ncoef, int nsums) { return std::max((size_t)ncoef, (size_t)nsums * kThreads) * sizeof(double2); }

template <int NW>
void launch_cgemvm(const double2* V, int ncol, int64_t ld, const double2* h, int ldh, double2* W, int64_t ldw,
                   int64_t n, hipStream_t s) {
  const int cg = gemv_groups(n), rows = kThreads / cg;
  const dim3 grid((unsigned)((n + rows - 1) / rows));
  const size_t lds = gemv_lds(NW * ncol, NW);
  if (cg == 16)
    hipLaunchKernelGGL((cgemvm_sub_kernel<NW, 16>), grid, dim3(kThreads), lds, s, V, ncol, ld, h, ldh, W, ldw, n);
  else
    hipLaunchKernelGGL((cgemvm_sub_kernel<NW, 4>), grid, dim3(kThreads), lds, s, V, ncol, ld, h, ldh, W, ldw, n);
}

hipError_t cgemvm_sub(const double2* V, int ncol, int64_t ld, const double2* h, int ldh, double2* W, int64_t ldw,
                      int nw, int64_t n, hipStream_t s) {
  if (ncol == 0) return hipSuccess;
  if ((size_t)nw * ncol * sizeof(double2) > 65536) {  // coefficients beyond the LDS of one group: one vector at a time
    for (int q = 0; q < nw; ++q)
      launch_cgemvm<1>(V, ncol, ld, h + (size_t)q * ldh, ldh, W + (size_t)q * ldw, ldw, n, s);
    return hipGetLastError();
  }
  switch (nw) {
    case 1:
      launch_cgemvm<1>(V, ncol, ld, h, ldh, W, ldw, n, s);
      break;
    case 2:
      launch_cgemvm<2>(V, ncol, ld, h, ldh, W, ldw, n, s);
      break;
    case 3:
      launch_cgemvm<3>(V, ncol, ld, h, ldh, W, ldw, n, s);
      break;
    case 4:
      launch_cgemvm<4>(V, ncol, ld, h, ldh, W, ldw, n, s);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <bool WithZ>
void launch_cgemv(const double2* V0, int n0, const double2* V1, int n1, const double2* P0, const double2* P1,
                  int64_t ld, const double2* h, int real_h, double2* w, double2* z, int64_t n, hipStream_t s) {
  const int cg = gemv_groups(n), rows = kThreads / cg;
  const dim3 grid((unsigned)((n + rows - 1) / rows));
  const size_t lds = gemv_lds(n0 + n1, WithZ ? 2 : 1);
  if (cg == 16)
    hipLaunchKernelGGL((cgemv_sub_kernel<WithZ, 16>), grid, dim3(kThreads), lds, s, V0, n0, V1, n1, P0, P1, ld, h,
                       real_h, w, z, n);
  else
    hipLaunchKernelGGL((cgemv_sub_kernel<WithZ, 4>), grid, dim3(kThreads), lds, s, V0, n0, V1, n1, P0, P1, ld, h,
                       real_h, w, z, n);
}

hipError_t cgemv_sub(const double2* V0, int n0, const double2* V1, int n1, const double2* P0,
                     const double2* P1, int64_t ld, const double2* h, int real_h, double2* w,
                     double2* z, int64_t n, hipStream_t s) {
  if (n0 + n1 == 0) return hipSuccess;
  if (z)
    launch_cgemv<true>(V0, n0, V1, n1, P0, P1, ld, h, real_h, w, z, n, s);
  else
    launch_cgemv<false>(V0, n0, V1, n1, P0, P1, ld, h, real_h, w, z, n, s);
  return hipGetLastError();
}

hipError_t normalize(double2* w, double2* z, int64_t n, const double2* h1, const double2* h2, int jh,
                     double* alpha, double* beta, int j, int* flag, double* part, hipStream_t s) {
  if (n <= kNormRows) {
    hipLaunchKernelGGL(normalize_short_kernel, dim3(1), dim3(1024), 0, s, w, z, n, h1, h2, jh, alpha, beta, j, flag);
    return hipGetLastError();
  }
  const int64_t nch = nchunks(n);
  hipLaunchKernelGGL(rdot_part_kernel, dim3((unsigned)nch), dim3(kThreads), 0, s, w, z ? z : w, n,
                     part);
  hipLaunchKernelGGL(normalize_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads)),
                     dim3(kThreads), 0, s, w, z, n, part, nch, h1, h2, jh, alpha, beta, j, flag);
  return hipGetLastError();
}

hipError_t scale_start(double2* w, double2* z, int64_t n, int* flag, double* part, hipStream_t s) {
  return normalize(w, z, n, nullptr, nullptr, 0, nullptr, nullptr, 0, flag, part, s);
}

hipError_t dgemm_tn_mfma(int64_t M, int N, int K, const double* A, int64_t lda, const double* B,
                         int64_t ldb, double* C, int64_t ldc, hipStream_t s) {
  if (M == 0 || N == 0) return hipSuccess;
  hipLaunchKernelGGL(dgemm_mfma_kernel, dim3((unsigned)((M + 63) / 64), (unsigned)((N + 63) / 64)),
                     dim3(kThreads), 0, s, M, N, K, A, lda, B, ldb, C, ldc);
  return hipGetLastError();
}

hipError_t colnorms(const double2* V, int ncol, int64_t ld, int64_t n, double* part, double* nrm,
                    hipStream_t s) {
  if (ncol == 0) return hipSuccess;
  const int64_t nch = nchunks(n);
  hipLaunchKernelGGL(colnorm_part_kernel, dim3((unsigned)nch, (unsigned)((ncol + 3) / 4)), dim3(kThreads), 0, s, V,
                     ncol, ld, n, part);
  hipLaunchKernelGGL(colsum_real_kernel, dim3((unsigned)((ncol + 3) / 4)), dim3(kThreads), 0, s, part, nch, ncol,
                     nrm);
  return hipGetLastError();
}

hipError_t start_vector(double2* v, int64_t n, uint64_t seed, hipStream_t s) {
  hipLaunchKernelGGL(start_vector_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads)),
                     dim3(kThreads), 0, s, v, n, seed);
  return hipGetLastError();
}

hipError_t warm_sum(const double2* X, const double2* Y, double ys, int64_t ld, int64_t n, int k, int b, int q,
                    double sv, double2* v, hipStream_t s) {
  hipLaunchKernelGGL(warm_sum_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0, s, X, Y,
                     ys, ld, n, k, b, q, sv, v);
  return hipGetLastError();
}

hipError_t neg_cols(double2* x, int64_t ld, int64_t n, int k, hipStream_t s) {
  if (k <= 0) return hipSuccess;
  hipLaunchKernelGGL(neg_cols_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads), (unsigned)k), dim3(kThreads),
                     0, s, x, ld, n);
  return hipGetLastError();
}

hipError_t ph_vectors(const double2* U, const double2* P, int64_t ld, const double* omega, int k,
                      int64_t n, double2* X, double2* Y, int64_t ldo, hipStream_t s) {
  if (k == 0) return hipSuccess;
  hipLaunchKernelGGL(ph_vectors_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads), (unsigned)k),
                     dim3(kThreads), 0, s, U, P, ld, omega, n, X, Y, ldo);
  return hipGetLastError();
}

hipError_t ph_mvectors(const double2* P, const double2* KP, int64_t ld, const double* omega, int k, int64_t n,
                       double2* MV, int64_t ldo, int64_t ldh, int add, hipStream_t s) {
  if (k == 0) return hipSuccess;
  hipLaunchKernelGGL(ph_mvectors_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads), (unsigned)k),
                     dim3(kThreads), 0, s, P, KP, ld, omega, n, MV, ldo, ldh, add);
  return hipGetLastError();
}

hipError_t acc_cols(double2* T, int64_t ldT, const double2* H, int64_t ldh, int cnt, int ncols, int real_only,
                    hipStream_t s) {
  if (cnt <= 0 || ncols <= 0) return hipSuccess;
  hipLaunchKernelGGL(acc_cols_kernel, dim3((unsigned)((cnt + kThreads - 1) / kThreads), (unsigned)ncols),
                     dim3(kThreads), 0, s, T, ldT, H, ldh, cnt, real_only);
  return hipGetLastError();
}

hipError_t zgemm_mfma(int64_t M, int N, int K, const double2* A, int64_t lda, const double2* B,
                      int64_t ldb, double2* C, int64_t ldc, hipStream_t s) {
  if (M == 0 || N == 0) return hipSuccess;
  hipLaunchKernelGGL(zgemm_mfma_kernel, dim3((unsigned)((M + 63) / 64), (unsigned)((N + 63) / 64)),
                     dim3(kThreads), 0, s, M, N, K, A, lda, B, ldb, C, ldc);
  return hipGetLastError();
}

hipError_t resid_h(const double2* MV, const double2* V, const double* om, int64_t ld, int64_t n, int ncol,
                   double2* R, hipStream_t s) {
  if (ncol == 0) return hipSuccess;
  hipLaunchKernelGGL(resid_h_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads), (unsigned)ncol),
                     dim3(kThreads), 0, s, MV, V, om, ld, n, R);
  return hipGetLastError();
}

hipError_t precond_h(const double2* r, const double* d, double om, double floor, int64_t ld, int64_t n,
                     int two, double2* t, hipStream_t s) {
  hipLaunchKernelGGL(precond_h_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0,
                     s, r, d, om, floor, ld, n, two, t);
  return hipGetLastError();
}

hipError_t h_out(const double2* V, const double* om, int64_t ld, int64_t n, int k, double2* X, double2* Y,
                 hipStream_t s) {
  if (k == 0) return hipSuccess;
  hipLaunchKernelGGL(h_out_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads), (unsigned)k),
                     dim3(kThreads), 0, s, V, om, ld, n, X, Y);
  return hipGetLastError();
}

hipError_t diag_a(const Layout& L, Arith ar, const void* a, const void* alo, double* d, hipStream_t s) {
  const dim3 g((unsigned)((L.n + kThreads - 1) / kThreads));
  if (ar == AR_C128)
    hipLaunchKernelGGL(diag_a_kernel<AR_C128>, g, dim3(kThreads), 0, s, a, alo, L.R, L.nb, L.n, d);
  else if (ar == AR_HILO)
    hipLaunchKernelGGL(diag_a_kernel<AR_HILO>, g, dim3(kThreads), 0, s, a, alo, L.R, L.nb, L.n, d);
  else
    hipLaunchKernelGGL(diag_a_kernel<AR_HI>, g, dim3(kThreads), 0, s, a, alo, L.R, L.nb, L.n, d);
  return hipGetLastError();
}

hipError_t copy_cols(const double2* src, int64_t lds, double2* dst, int64_t ldd, int64_t n, int k,
                     hipStream_t s) {
  if (k == 0) return hipSuccess;
  hipLaunchKernelGGL(copy_cols_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads), (unsigned)k),
                     dim3(kThreads), 0, s, src, lds, dst, ldd, n);
  return hipGetLastError();
}

hipError_t resid_cols(const double2* W, const double2* V, const double* th, int64_t ld, int64_t n,
                      int ncol, double2* R, hipStream_t s) {
  if (ncol == 0) return hipSuccess;
  hipLaunchKernelGGL(resid_cols_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads), (unsigned)ncol),
                     dim3(kThreads), 0, s, W, V, th, ld, n, R);
  return hipGetLastError();
}

hipError_t times_i(const double2* src, int64_t lds, double2* dst, int64_t ldd, int64_t n, int ncol,
                   const double* sc, int sqrt_inv, hipStream_t s) {
  if (ncol == 0) return hipSuccess;
  hipLaunchKernelGGL(times_i_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads), (unsigned)ncol),
                     dim3(kThreads), 0, s, src, lds, dst, ldd, n, sc, sqrt_inv);
  return hipGetLastError();
}

hipError_t conj_copy(const double2* src, double2* dst, int64_t n, double sg, hipStream_t s) {
  hipLaunchKernelGGL(conj_copy_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads)),
                     dim3(kThreads), 0, s, src, dst, n, sg);
  return hipGetLastError();
}

hipError_t resid_norms(const double2* out, const double2* v, int cj, double sgn_om, int64_t n,
                       double* part, double* res, hipStream_t s) {
  const int64_t nch = nchunks(n);
  hipLaunchKernelGGL(resid_part_kernel, dim3((unsigned)nch), dim3(kThreads), 0, s, out, v, cj,
                     sgn_om, n, part);
  hipLaunchKernelGGL(pair_sum_kernel, dim3(1), dim3(64), 0, s, part, nch, res);
  return hipGetLastError();
}

template <int MODE>
hipError_t launch_grad(const double2* X, const double2* Y, int64_t ld, const double* wgt, int k, int64_t n,
                       double2* ga, double2* gb, const double2* C, double* part, hipStream_t s) {
  const int64_t nt = (n + kGT - 1) / kGT;
  const dim3 grid((unsigned)(nt * (nt + 1) / 2));
  if (Y)
    hipLaunchKernelGGL((grad_tile_kernel<MODE, true>), grid, dim3(kThreads), 0, s, X, Y, ld, wgt, k, n, ga, gb, C,
                       part);
  else
    hipLaunchKernelGGL((grad_tile_kernel<MODE, false>), grid, dim3(kThreads), 0, s, X, Y, ld, wgt, k, n, ga, gb, C,
                       part);
  return hipGetLastError();
}

hipError_t quad_packed(const double2* X, const double2* Y, int64_t ld, const double* wgt, int k, int64_t n,
                       const double2* C, int target_b, double* part, hipStream_t s) {
  return target_b ? launch_grad<2>(X, Y, ld, wgt, k, n, nullptr, nullptr, C, part, s)
                  : launch_grad<1>(X, Y, ld, wgt, k, n, nullptr, nullptr, C, part, s);
}

hipError_t quad_diag(const double2* X, const double2* Y, int64_t ld, const double* wgt, int k,
                     const double* d, int64_t n, double* part, hipStream_t s) {
  hipLaunchKernelGGL(quad_diag_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0,
                     s, X, Y, ld, wgt, k, d, n, part);
  return hipGetLastError();
}

hipError_t grad_packed(const double2* X, const double2* Y, int64_t ld, const double* wgt, int k,
                       int64_t n, double2* ga, double2* gb, hipStream_t s) {
  return launch_grad<0>(X, Y, ld, wgt, k, n, ga, gb, nullptr, nullptr, s);
}

int64_t quad_packed_parts(int64_t n) {
  const int64_t nt = (n + kGT - 1) / kGT;
  return nt * (nt + 1) / 2;
}

hipError_t cfrac(int ph, int n, const double* alpha, const double* beta, double scale, const double* freq,
                 int nw, double eta, double2* chi, hipStream_t s) {
  if (nw <= 0) return hipSuccess;
  hipLaunchKernelGGL(cfrac_kernel, dim3((unsigned)((nw + kThreads - 1) / kThreads)), dim3(kThreads), 0, s, ph,
                     n, alpha, beta, scale, freq, nw, eta, chi);
  return hipGetLastError();
}

}  // namespace bse
