// Sums over a 64-lane wavefront by exchange steps (device code of the kernels).
// One value per sum costs 18 instructions as six shuffle-and-add steps; here
// several values share the steps, each of which halves the registers instead of
// leaving the same sum in every lane.
#pragma once

#include <hip/hip_runtime.h>

namespace bse {
namespace {

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}
// a + b after exchanging halves: lanes with bit 5 (4) of their number clear
// get a of the lane pair, the others b of it.
__device__ __forceinline__ double swap32_add(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
__device__ __forceinline__ double swap16_add(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
// The same with a DPP exchange inside rows of 16 lanes: banks (groups of four
// lanes) in BA take a of their partner, the others b.
template <int CTRL, int BA>
__device__ __forceinline__ double dpp_swap_add(double a, double b) {
  constexpr int BB = 0xf & ~BA;
  const int xl = __builtin_amdgcn_update_dpp(__double2loint(a), __double2loint(b), CTRL, 0xf, BB, false);
  const int xh = __builtin_amdgcn_update_dpp(__double2hiint(a), __double2hiint(b), CTRL, 0xf, BB, false);
  const int yl = __builtin_amdgcn_update_dpp(__double2loint(b), __double2loint(a), CTRL, 0xf, BA, false);
  const int yh = __builtin_amdgcn_update_dpp(__double2hiint(b), __double2hiint(a), CTRL, 0xf, BA, false);
  return __hiloint2double(xh, xl) + __hiloint2double(yh, yl);
}
// The same between banks 0 and 1 and banks 2 and 3: even banks get a of the
// pair, odd banks b.
__device__ __forceinline__ double bank_pair_add(double a, double b) {
  const int xl = __builtin_amdgcn_update_dpp(__double2loint(a), __double2loint(b), 0x124, 0xf, 0xa, false);
  const int xh = __builtin_amdgcn_update_dpp(__double2hiint(a), __double2hiint(b), 0x124, 0xf, 0xa, false);
  const int yl = __builtin_amdgcn_update_dpp(__double2loint(b), __double2loint(a), 0x12c, 0xf, 0x5, false);
  const int yh = __builtin_amdgcn_update_dpp(__double2hiint(b), __double2hiint(a), 0x12c, 0xf, 0x5, false);
  return __hiloint2double(xh, xl) + __hiloint2double(yh, yl);
}
// Sum of one value over the wavefront, in every lane.
__device__ __forceinline__ double wave_sum_dpp(double v) {
  v += dpp_f64<0x128>(v);  // row_ror:8
  v += dpp_f64<0x141>(v);  // row_half_mirror
  v += dpp_f64<0xB1>(v);   // lane xor 1
  v += dpp_f64<0x4E>(v);   // lane xor 2
  v = swap16_add(v, v);
  return swap32_add(v, v);
}
// Sums of N = 4, 8 or 16 values over the wavefront: every lane returns the sum
// of value wave_sum_index<N>(lane).
template <int N>
__device__ __forceinline__ double wave_sum_n(double (&v)[N]) {
  static_assert(N == 4 || N == 8 || N == 16, "4, 8 or 16 values");
#pragma unroll
  for (int i = 0; i < N / 2; ++i) v[i] = swap32_add(v[2 * i], v[2 * i + 1]);
#pragma unroll
  for (int i = 0; i < N / 4; ++i) v[i] = swap16_add(v[2 * i], v[2 * i + 1]);
  if constexpr (N >= 8) {
#pragma unroll
    for (int i = 0; i < N / 8; ++i) v[i] = dpp_swap_add<0x128, 0x3>(v[2 * i], v[2 * i + 1]);  // row_ror:8
  } else {
    v[0] += dpp_f64<0x128>(v[0]);
  }
  double s;
  if constexpr (N == 16)
    s = dpp_swap_add<0x141, 0x5>(v[0], v[1]);  // row_half_mirror
  else
    s = v[0] + dpp_f64<0x141>(v[0]);
  s += dpp_f64<0xB1>(s);  // quad_perm: lane xor 1
  s += dpp_f64<0x4E>(s);  // lane xor 2
  return s;
}
template <int N>
__device__ __forceinline__ int wave_sum_index(int lane) {
  int i = ((lane >> 5) & 1) | ((lane >> 3) & 2);
  if (N >= 8) i |= (lane >> 1) & 4;
  if (N == 16) i |= (lane << 1) & 8;
  return i;
}

}  // namespace
}  // namespace bse
