// Top-2 records of the LM head's argmax, shared by the kernels that write and merge them.
#pragma once
#include "common.h"

namespace ad {

// Running top-2 of a set of logits: largest value v1 at index i1 (lowest index among
// equal maxima), the runner-up value v2 (equal to v1 when the maximum repeats), and
// whether a non-finite value was seen.  The merge is associative and commutative, so any
// reduction order gives the same record.  Branch-free (selects only).
struct Top2s {
  float v1;
  int i1;
  float v2;
  int bad;
};
__device__ __forceinline__ Top2s t2_merge(Top2s a, Top2s b) {
  const bool aw = (a.v1 > b.v1) | ((a.v1 == b.v1) & (a.i1 < b.i1));
  Top2s r;
  r.v1 = aw ? a.v1 : b.v1;
  r.i1 = aw ? a.i1 : b.i1;
  r.v2 = fmaxf(aw ? a.v2 : b.v2, aw ? b.v1 : a.v1);
  r.bad = a.bad | b.bad;
  return r;
}
__device__ __forceinline__ Top2s t2_shfl(Top2s t, int mask) {
  Top2s u;
  u.v1 = __shfl_xor(t.v1, mask, kWave);
  u.i1 = __shfl_xor(t.i1, mask, kWave);
  u.v2 = __shfl_xor(t.v2, mask, kWave);
  u.bad = __shfl_xor(t.bad, mask, kWave);
  return u;
}
// Rotate by N lanes inside each row of 16 lanes (DPP row_ror, no LDS round trip).
template <int N>
__device__ __forceinline__ int ror16(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x120 + N, 0xf, 0xf, false);
}
template <int N>
__device__ __forceinline__ Top2s t2_ror16(Top2s t) {
  Top2s u;
  u.v1 = __int_as_float(ror16<N>(__float_as_int(t.v1)));
  u.i1 = ror16<N>(t.i1);
  u.v2 = __int_as_float(ror16<N>(__float_as_int(t.v2)));
  u.bad = ror16<N>(t.bad);
  return u;
}
// Merge over the 16 lanes of a row: afterwards every lane holds the row's record.
__device__ __forceinline__ Top2s t2_row16(Top2s t) {
  t = t2_merge(t, t2_ror16<8>(t));
  t = t2_merge(t, t2_ror16<4>(t));
  t = t2_merge(t, t2_ror16<2>(t));
  t = t2_merge(t, t2_ror16<1>(t));
  return t;
}

}  // namespace ad
