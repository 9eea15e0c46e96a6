// Sums over a 64-lane wave without LDS: four DPP steps add the 16 lanes of a row, two row
// broadcasts add the rows (lane 63 ends with the total), all on the vector ALU.  A butterfly of
// __shfl_xor costs two LDS permutes a step, about 800 cycles for a double; this is about 150.
#pragma once

#include <hip/hip_runtime.h>

namespace dacp {

// The value of `v` moved by a DPP control; lanes outside the row mask get 0.  (With every row in the
// mask nothing is left of the destination's old value, and the move needs none.)
template <int kCtrl, int kRowMask>
__device__ __forceinline__ int dpp_move(int v) {
  if constexpr (kRowMask == 0xf) return __builtin_amdgcn_mov_dpp(v, kCtrl, 0xf, 0xf, true);
  else return __builtin_amdgcn_update_dpp(0, v, kCtrl, kRowMask, 0xf, false);
}
template <int kCtrl, int kRowMask>
__device__ __forceinline__ double dpp_move(double v) {
  return __hiloint2double(dpp_move<kCtrl, kRowMask>(__double2hiint(v)), dpp_move<kCtrl, kRowMask>(__double2loint(v)));
}

// The same lane's value of the lane `lane` (uniform) in every lane.
__device__ __forceinline__ double read_lane(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// The wave's total, valid in lane 63: lanes of a quad, quads of 8, 8s of a row, then rows 0 + 1 and
// 2 + 3, then both.  Every lane must be active.
__device__ __forceinline__ double wave_sum_last(double v) {
  v += dpp_move<0xB1, 0xf>(v);   // quad_perm 1 0 3 2
  v += dpp_move<0x4E, 0xf>(v);   // quad_perm 2 3 0 1
  v += dpp_move<0x141, 0xf>(v);  // row_half_mirror
  v += dpp_move<0x140, 0xf>(v);  // row_mirror
  v += dpp_move<0x142, 0xa>(v);  // row_bcast15 into rows 1 and 3
  v += dpp_move<0x143, 0xc>(v);  // row_bcast31 into rows 2 and 3
  return v;
}

// The same total in every lane.
__device__ __forceinline__ double wave_sum(double v) { return read_lane(wave_sum_last(v), 63); }

}  // namespace dacp
