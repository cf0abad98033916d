// Shared by the contraction kernels: the logistic scorer of one cell.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "libnwmine.h"

namespace nwm {

// Features and logistic score of one cell (Sec. 4): S_raw = dot / l (0 for an
// empty source sentence), rho = min(l, l') / max(l, l') (1 when both
// sentences are empty), z = w0 S_raw + w1 rho + b, S = 1 / (1 + exp(-z)).
// rl, rlt are the reciprocals of l, l' (inf for 0), so rho = min(l / l',
// l' / l) = min(l rlt, l' rl); positive floats order as their bit patterns,
// so that minimum is an integer one.  An exponent past the FP32 range gives
// exp = inf and S = 0 (1 / inf), exp = 0 gives S = 1.  CHECKED = false drops
// the tests for empty sentences (every length of the tile is positive).
template <bool CHECKED>
static __device__ __forceinline__ float logistic_cell(float dot, float l, float rl, float lt, float rlt,
                                                      const nwm_scorer &sc, float &sraw) {
  const float LOG2E = 1.4426950408889634f;
  float sr = dot * rl;
  float rho = __uint_as_float(min(__float_as_uint(l * rlt), __float_as_uint(lt * rl)));
  if (CHECKED) {
    sr = l > 0.0f ? sr : 0.0f;
    rho = (l > 0.0f || lt > 0.0f) ? rho : 1.0f;
  }
  sraw = sr;
  const float z = __builtin_fmaf(sc.w0, sr, __builtin_fmaf(sc.w1, rho, sc.b));
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-z * LOG2E));
}

}  // namespace nwm
