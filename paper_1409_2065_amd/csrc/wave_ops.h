// FP64 sums over the lanes of a wave by VALU lane moves.
#pragma once

#include "ccmi_internal.h"

namespace ccmi {

// A double moved between lanes by data-parallel primitives: two 32-bit VALU
// moves, against two LDS-unit permutes for a shuffle.  Every sweep ends and
// begins with sums over the block, a serial chain that bounds small problems
// and that 16 waves per CU queue up for in the LDS unit on larger ones:
// against shuffles one at a time (wave trees and block sums written out by
// one thread) a 200 x 10 FP64 solve went from 10.9 to 8.5 us per MM iteration
// and a 2000 x 500 path from 35.4 to 31.4, with the same bits.
// dpp<CTRL>(v): every
// lane reads the lane CTRL names within its row of 16 (kRor: rotation; a
// rotation by 8 is an exchange of lanes 8 apart).
constexpr int kRowShl = 0x100, kRowShr = 0x110, kRor = 0x120;
constexpr int kXor1 = 0xB1, kXor2 = 0x4E;  // quad permutations
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false),
                          __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false));
}
// The lanes 4 apart: banks (4 lanes) 0 and 2 of each row read 4 lanes up,
// banks 1 and 3 read 4 lanes down.
__device__ __forceinline__ double dpp_xor4(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  int l = __builtin_amdgcn_update_dpp(lo, lo, kRowShl + 4, 0xf, 0x5, false);
  int h = __builtin_amdgcn_update_dpp(hi, hi, kRowShl + 4, 0xf, 0x5, false);
  l = __builtin_amdgcn_update_dpp(l, lo, kRowShr + 4, 0xf, 0xa, false);
  h = __builtin_amdgcn_update_dpp(h, hi, kRowShr + 4, 0xf, 0xa, false);
  return __hiloint2double(h, l);
}
// Sum over the two halves of the wave of a (returned to lanes 0..31) and of
// b (to lanes 32..63): the upper half of a is exchanged with the lower half
// of b, and every lane adds its two values.  pair_sum16: the same between
// neighbouring rows of 16 (a to the even rows, b to the odd ones).
__device__ __forceinline__ double pair_sum32(double a, double b) {
  const auto l = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const auto h = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
}
__device__ __forceinline__ double pair_sum16(double a, double b) {
  const auto l = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
  const auto h = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
}

// Sum over the wave, in every lane: lanes 32, 16, 8, 4, 2, 1 apart add up
// in that order (after the exchange over 8 lanes the values repeat every 8,
// so the rotations by 4, 2, 1 are exchanges too).
__device__ inline double wave_sum(double v) {
  v = pair_sum32(v, v);
  v = pair_sum16(v, v);
  v += dpp<kRor + 8>(v);
  v += dpp<kRor + 4>(v);
  v += dpp<kRor + 2>(v);
  v += dpp<kRor + 1>(v);
  return v;
}

// Sums over the wave of 8 values per lane, value q's total left in lanes
// 8q .. 8q+7: the steps over 32, 16 and 8 lanes halve the values held per
// lane (value 4 b5 + 2 b4 + b3 of lane bits b), then the 8-lane groups
// reduce.  Each value is added in the order of wave_sum.  7 exchanges for 8
// values where wave_sum needs 48.
__device__ __forceinline__ double wave_sum8_groups(const double (&v)[8]) {
  double a[4], b[2];
#pragma unroll
  for (int j = 0; j < 4; ++j) a[j] = pair_sum32(v[j], v[4 + j]);
#pragma unroll
  for (int j = 0; j < 2; ++j) b[j] = pair_sum16(a[j], a[2 + j]);
  const bool hi = (threadIdx.x & 8) != 0;
  double t = (hi ? b[1] : b[0]) + dpp<kRor + 8>(hi ? b[0] : b[1]);
  t += dpp_xor4(t);
  t += dpp<kXor2>(t);
  t += dpp<kXor1>(t);
  return t;
}
// The same with value q's total returned to lane q (lanes 8..63 get some total).
__device__ inline double wave_sum8(const double (&v)[8]) {
  return __shfl(wave_sum8_groups(v), (8 * (threadIdx.x % kWave)) % kWave, kWave);
}

}  // namespace ccmi
