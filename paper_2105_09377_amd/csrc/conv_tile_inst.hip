// One translation unit per (element type, workgroup shape, window size) of conv_tile_kernel, so that the
// instances compile in parallel.  Built several times with different -DGS_TILE_TRAITS /
// -DGS_TILE_SHAPE / -DGS_TILE_K / -DGS_TILE_ODD / -DGS_TILE_NAME (see build.py).  GS_TILE_ODD: channels that do not fill
// the last chunk; not in the largest workgroups, and groups of a single chunk take the kernels for several.
#include "conv_tile_kernel.h"

#include <mutex>

namespace gs {

constexpr TileShape kShape = kTileShapes[GS_TILE_SHAPE];

template <int K, int CM, bool NAT, int S, int IL, int MAXI, bool ONE, bool PROJ = false>
static hipError_t launch_tile_inst(const ConvArgs& a, const TilePlan& p, hipStream_t s) {
  // With a projection: bfloat16, 3x3 at stride 2 (see launch_conv_with_projection).
  if constexpr (!PROJ && K == 3 && S == 2 && !GS_TILE_ODD && GS_TILE_TRAITS::kEsz == 2)
    if (a.wproj) return launch_tile_inst<K, CM, NAT, S, IL, MAXI, ONE, true>(a, p, s);
  auto kern = conv_tile_kernel<GS_TILE_TRAITS, K, K, CM, NAT, S, IL, kShape.nj, kShape.wo, kShape.wp, kShape.ks, MAXI, ONE, bool(GS_TILE_ODD), PROJ>;
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

template <int K, int CM, bool NAT, int S, int IL>
static hipError_t launch_tile_items(const ConvArgs& a, const TilePlan& p, hipStream_t s) {
  if constexpr (kShape.ks > 1 && !GS_TILE_ODD) {
    if (p.one && p.maxi == 1) return launch_tile_inst<K, CM, NAT, S, IL, 1, true>(a, p, s);
    if (p.one && p.maxi == 2) return launch_tile_inst<K, CM, NAT, S, IL, 2, true>(a, p, s);
    if (p.one) return launch_tile_inst<K, CM, NAT, S, IL, 4, true>(a, p, s);
  }
  if (p.maxi == 1) return launch_tile_inst<K, CM, NAT, S, IL, 1, false>(a, p, s);
  if (p.maxi == 2) return launch_tile_inst<K, CM, NAT, S, IL, 2, false>(a, p, s);
  if constexpr (kShape.nj <= 2) return launch_tile_inst<K, CM, NAT, S, IL, 4, false>(a, p, s);
  return hipErrorInvalidValue;
}

template <int K, int CM, bool NAT>
static hipError_t launch_tile_il(const ConvArgs& a, const TilePlan& p, hipStream_t s) {
  constexpr bool kMany = kShape.nj >= 2 && kShape.ks == 1;
  if (a.Sh == 1) {
    if constexpr (kShape.nj >= 4)
      if (p.il == 4) return launch_tile_items<K, CM, NAT, 1, 4>(a, p, s);
    if constexpr (kMany)
      if (p.il == 2) return launch_tile_items<K, CM, NAT, 1, 2>(a, p, s);
    return launch_tile_items<K, CM, NAT, 1, 1>(a, p, s);
  }
  if constexpr (kMany)
    if (p.il == 2) return launch_tile_items<K, CM, NAT, 2, 2>(a, p, s);
  return launch_tile_items<K, CM, NAT, 2, 1>(a, p, s);
}

// The plan's values are the ones that plan_tiles (conv.hip) chooses from.
hipError_t GS_TILE_NAME(const ConvArgs& a, const TilePlan& p, hipStream_t s) {
#if GS_TILE_K == 3
  return launch_tile_il<3, 1, false>(a, p, s);
#elif GS_TILE_K == 1
  return a.wblk ? launch_tile_il<1, kTileChunks, false>(a, p, s) : launch_tile_il<1, kTileChunks, true>(a, p, s);
#else
  if constexpr (kShape.nj <= 2) return launch_tile_il<5, 1, false>(a, p, s);   // (a ring of 25 taps leaves no room for more)
  return hipErrorInvalidValue;
#endif
}

}  // namespace gs
