// Device helpers of the kernels on the site-operator form (parity.hip,
// site.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "parity.h"

namespace cfet {

typedef double dv2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) const dv2* lds_cptr;

__device__ __forceinline__ double2 lds_at(uint32_t byte_addr) {
  const dv2 v = *(lds_cptr)(uintptr_t)byte_addr;
  return make_double2(v.x, v.y);
}

// One DPP step of the wavefront sum: v + (v moved by the DPP pattern), rows
// outside the row mask add 0.
template <int CTRL, int ROWMASK>
__device__ __forceinline__ double w_step(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWMASK, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWMASK, 0xf, false);
  return v + __hiloint2double(hi, lo);
}

// Sum over the 64 lanes in a fixed order; lane 63 holds it.
__device__ __forceinline__ double w_sum63(double v) {
  v = w_step<0xB1, 0xf>(v);   // quad_perm [1,0,3,2]
  v = w_step<0x4E, 0xf>(v);   // quad_perm [2,3,0,1]
  v = w_step<0x141, 0xf>(v);  // row_half_mirror
  v = w_step<0x140, 0xf>(v);  // row_mirror
  v = w_step<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
  return w_step<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
}

template <bool RV>
__device__ __forceinline__ void acc_fma(double2& acc, dv2 v, double2 x) {
  if (RV) {
    acc.x = fma(v.x, x.x, acc.x);
    acc.y = fma(v.x, x.y, acc.y);
  } else {
    acc.x = fma(v.x, x.x, fma(-v.y, x.y, acc.x));
    acc.y = fma(v.x, x.y, fma(v.y, x.x, acc.y));
  }
}

}  // namespace cfet
