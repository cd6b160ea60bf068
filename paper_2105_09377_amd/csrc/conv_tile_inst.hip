// One translation unit per (element type, workgroup shape) of conv_tile_kernel, so that the
// instances compile in parallel.  Built several times with different -DGS_TILE_TRAITS /
// -DGS_TILE_SHAPE / -DGS_TILE_NAME (see build.py).
#include "conv_tile_kernel.h"

#include <mutex>

namespace gs {

constexpr TileShape kShape = kTileShapes[GS_TILE_SHAPE];

template <int KH, int KW, int S, int IL, int MAXI, bool ONE>
static hipError_t launch_tile_inst(const ConvArgs& a, const TilePlan& p, hipStream_t s) {
  auto kern = conv_tile_kernel<GS_TILE_TRAITS, KH, KW, S, IL, kShape.nj, kShape.wo, kShape.wp, kShape.ks, MAXI, ONE>;
  static std::once_flag once;              // the attribute is set once, whichever thread comes first
  static hipError_t attr_status = hipSuccess;
  std::call_once(once, [&]() {
    attr_status = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, int(kLdsLimit));
  });
  if (attr_status != hipSuccess) return attr_status;
  hipLaunchKernelGGL(kern, dim3(unsigned(p.tiles)), dim3(64 * kShape.wo * kShape.wp * kShape.ks), size_t(p.lds_bytes), s, a, p.g);
  return hipGetLastError();
}

template <int KH, int KW, int S, int IL>
static hipError_t launch_tile_items(const ConvArgs& a, const TilePlan& p, hipStream_t s) {
  if constexpr (kShape.ks > 1) {
    if (p.one && p.maxi == 1) return launch_tile_inst<KH, KW, S, IL, 1, true>(a, p, s);
    if (p.one && p.maxi == 2) return launch_tile_inst<KH, KW, S, IL, 2, true>(a, p, s);
    if (p.one) return launch_tile_inst<KH, KW, S, IL, 4, true>(a, p, s);
  }
  if (p.maxi == 1) return launch_tile_inst<KH, KW, S, IL, 1, false>(a, p, s);
  if (p.maxi == 2) return launch_tile_inst<KH, KW, S, IL, 2, false>(a, p, s);
  if constexpr (kShape.nj <= 2) return launch_tile_inst<KH, KW, S, IL, 4, false>(a, p, s);
  return hipErrorInvalidValue;
}

// The plan's values are the ones that plan_tiles (conv.hip) chooses from.
hipError_t GS_TILE_NAME(const ConvArgs& a, const TilePlan& p, hipStream_t s) {
  constexpr bool kMany = kShape.nj >= 2 && kShape.ks == 1;
  if (a.Sh == 1) {
    if constexpr (kShape.nj >= 4)
      if (p.il == 4) return launch_tile_items<3, 3, 1, 4>(a, p, s);
    if constexpr (kMany)
      if (p.il == 2) return launch_tile_items<3, 3, 1, 2>(a, p, s);
    return launch_tile_items<3, 3, 1, 1>(a, p, s);
  }
  if constexpr (kMany)
    if (p.il == 2) return launch_tile_items<3, 3, 2, 2>(a, p, s);
  return launch_tile_items<3, 3, 2, 1>(a, p, s);
}

}  // namespace gs
