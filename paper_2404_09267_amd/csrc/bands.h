// Band bits: which of a set's rectangles touch each of some columns and rows ("bands") of the
// set's extent, 32 rectangles to a word. The rectangles that can meet a query are among those
// that share a column and a row with it.
#ifndef TG_BANDS_H
#define TG_BANDS_H

#include <hip/hip_runtime.h>

#include <cstdint>

namespace tg_detail {

// The minimum over the 64 lanes of a wave, in every lane: DPP row shifts inside each row of
// 16 lanes, then row broadcasts; lane 63 ends with it. (Lanes without a source keep their
// own value.)
template <int kCtrl, int kRows>
__device__ __forceinline__ float dpp_min_step(float v) {
  const int i = __float_as_int(v);
  return fminf(v, __int_as_float(__builtin_amdgcn_update_dpp(i, i, kCtrl, kRows, 0xF, false)));
}
__device__ __forceinline__ float wave_min(float v) {
  v = dpp_min_step<0x111, 0xF>(v);  // row_shr:1
  v = dpp_min_step<0x112, 0xF>(v);  // row_shr:2
  v = dpp_min_step<0x114, 0xF>(v);  // row_shr:4
  v = dpp_min_step<0x118, 0xF>(v);  // row_shr:8
  v = dpp_min_step<0x142, 0xA>(v);  // row_bcast:15
  v = dpp_min_step<0x143, 0xC>(v);  // row_bcast:31
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// An axis of a set's extent [lo, hi] cut into bands: any finite origin and scale >= 0 serve
// (only speed depends on them), so an empty or degenerate extent puts everything in band 0.
struct BandAxis {
  float origin, scale;
};
__device__ __forceinline__ BandAxis band_axis(float lo, float hi, int bands) {
  BandAxis a;
  a.origin = __builtin_isfinite(lo) ? lo : 0.0f;
  const float s = bands * __builtin_amdgcn_rcpf(hi - lo);
  a.scale = __builtin_isfinite(s) && s > 0.0f ? s : 0.0f;
  return a;
}

// The band of coordinate v (any value): non-decreasing in v, so a rectangle [x0, x1]
// touching bands band(x0) .. band(x1) is named in the band of every point it holds.
__device__ __forceinline__ int band_of(float v, BandAxis a, int bands) {
  const float t = fmaxf(__fmul_rn(__fsub_rn(v, a.origin), a.scale), 0.0f);
  return static_cast<int>(fminf(t, static_cast<float>(bands - 1)));
}

// The 32 x 32 bit matrices held by the two halves of a wave (row l in lane l), transposed:
// five exchanges with the lane 16, 8, 4, 2, 1 away, each swapping the blocks off the
// diagonal. Turns 32 rectangles' band masks into bands' words. (30 ballots and selects for the
// same took 4 us where this takes under 1: they overflow the scalar registers.)
__device__ __forceinline__ uint32_t transpose32(uint32_t x, int lane) {
  constexpr uint32_t kLow[5] = {0x55555555u, 0x33333333u, 0x0F0F0F0Fu, 0x00FF00FFu, 0x0000FFFFu};
#pragma unroll
  for (int s = 4; s >= 0; --s) {
    const int j = 1 << s;
    const uint32_t m = kLow[s], y = __shfl_xor(x, j);
    x = (lane & j) ? (x & ~m) | (y >> j & m) : (x & m) | (y & m) << j;
  }
  return x;
}

}  // namespace tg_detail

#endif  // TG_BANDS_H
