// Sums of several values over the 64 lanes of a wave, each value's sum ending on one lane.
#pragma once

#include "polar4.h"
#include "qfs_internal.h"

namespace qfs {

// Lane l's partner's value: lane l ^ M. Within the 16-lane rows by DPP moves; across rows through
// the LDS crossbar.
template <int CTRL>
__device__ __forceinline__ float dpp_movef(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, false));
}
template <int M>
__device__ __forceinline__ double partner(double x) {
  if constexpr (M < 16) return xor_lane<M>(x);
  else return __shfl_xor(x, M);
}
template <int M>
__device__ __forceinline__ float partner(float x) {
  if constexpr (M == 1) return dpp_movef<0xB1>(x);
  else if constexpr (M == 2) return dpp_movef<0x4E>(x);
  else if constexpr (M == 4) return dpp_movef<0x1B>(dpp_movef<0x141>(x));
  else if constexpr (M == 8) return dpp_movef<0x128>(x);
  else return __shfl_xor(x, M);
}

template <int M, int C, typename R, int NV>
__device__ __forceinline__ void wave_halve(R (&v)[NV], int lane) {
  if constexpr (C >= 1) {
    const bool hi = (lane & M) != 0;
#pragma unroll
    for (int i = 0; i < C; ++i) {
      const R give = hi ? v[i] : v[C + i];
      const R keep = hi ? v[C + i] : v[i];
      v[i] = keep + partner<M>(give);
    }
  } else {
    v[0] += partner<M>(v[0]);
  }
}

// Wave sums of NV = 16, 32 or 64 values by recursive halving: at the exchange with lane ^ M
// (M = 1, 2, 4, .. 32) each lane keeps half of its values, the upper half where its bit M is set,
// and adds its partner's copy of that half; once one value is left, the sums are completed
// plainly. The many values are exchanged first, within the rows of 16 lanes by DPP moves, and
// few (NV / 16 at most) cross the rows. Lane l < NV returns the sum of value wave_sums_index(l).
template <typename R, int NV>
__device__ __forceinline__ R wave_sums(R (&v)[NV]) {
  static_assert(NV == 16 || NV == 32 || NV == 64, "16, 32 or 64 values");
  const int lane = threadIdx.x & 63;
  wave_halve<1, NV / 2>(v, lane);
  wave_halve<2, NV / 4>(v, lane);
  wave_halve<4, NV / 8>(v, lane);
  wave_halve<8, NV / 16>(v, lane);
  wave_halve<16, NV / 32>(v, lane);
  wave_halve<32, NV / 64>(v, lane);
  return v[0];
}
template <int NV>
__device__ __forceinline__ int wave_sums_index(int lane) {
  constexpr int B = NV == 16 ? 4 : NV == 32 ? 5 : 6;
  return (int)(__brev((unsigned)lane) >> (32 - B));
}

}  // namespace qfs
