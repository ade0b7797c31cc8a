// Wavefront exchanges that stay in the vector unit (64 lanes, all active).
#pragma once

#include <hip/hip_runtime.h>

namespace celeste {
namespace {

// a and b with lane bit 5 (M = 32) or 4 (M = 16) exchanged: on lanes with the bit clear a keeps its
// value and b takes the partner lane's a; on lanes with it set b keeps its value and a takes the
// partner lane's b.
template <int M>
__device__ __forceinline__ void swap_half(unsigned& a, unsigned& b) {
  if constexpr (M == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
  } else {
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
  }
}

template <int M>
__device__ __forceinline__ float swap_add(float x, float y) {
  unsigned a = __float_as_uint(x), b = __float_as_uint(y);
  swap_half<M>(a, b);
  return __uint_as_float(a) + __uint_as_float(b);
}

template <int M>
__device__ __forceinline__ double swap_add(double x, double y) {
  unsigned al = __double2loint(x), ah = __double2hiint(x), bl = __double2loint(y), bh = __double2hiint(y);
  swap_half<M>(al, bl);
  swap_half<M>(ah, bh);
  return __hiloint2double((int)ah, (int)al) + __hiloint2double((int)bh, (int)bl);
}

// the partner lane's value over a DPP control: row_ror:8 (lane ^ 8), quad_perm (lane ^ 2, lane ^ 1);
// row_ror:4 is lane ^ 4 where the values repeat every 8 lanes of a row (after a sum over lane ^ 8)
constexpr int DPP_XOR8 = 0x128, DPP_ROR4 = 0x124, DPP_XOR2 = 0x4E, DPP_XOR1 = 0xB1;
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}

// Sum over the wavefront by the butterfly over lane bits 5, 4, 3, 2, 1, 0: the same bits on every
// lane (every lane adds the same pairs), about 180 cycles where the exchanges through LDS take 600.
__device__ __forceinline__ double wave_sum(double x) {
  x = swap_add<32>(x, x);
  x = swap_add<16>(x, x);
  x += dpp<DPP_XOR8>(x);
  x += dpp<DPP_ROR4>(x);
  x += dpp<DPP_XOR2>(x);
  x += dpp<DPP_XOR1>(x);
  return x;
}

__device__ __forceinline__ double wave_uniform(double x) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(x)),
                          __builtin_amdgcn_readfirstlane(__double2loint(x)));
}

// lane k's value on every lane (k uniform)
__device__ __forceinline__ double lane_value(double x, int k) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), k),
                          __builtin_amdgcn_readlane(__double2loint(x), k));
}

}  // namespace
}  // namespace celeste
