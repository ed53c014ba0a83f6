// The attention kernel (attn_fwd_kernel.h) with its keys split over the
// wavefronts of a workgroup, for grids too small to fill the device.
//
// Eight wavefronts form G key groups of 8 / G: each group takes the same
// 256 / G query rows and every G-th key block, through K and V rings of its
// own, and the groups' (O, m, l) are merged through LDS at the end.  A query
// block then takes 1 / G of the steps, and a head has G times the blocks that a
// 256-row tile gives, so a call of a few heads keeps more CUs busy for a
// shorter time; no scratch memory and no second kernel are needed.  One
// workgroup per CU (two waves per SIMD), as its rings fill most of the LDS: the
// reason why 16-bit d = 128 stops at G = 2 (133 KB; G = 4 would need 266 KB) and
// 192-wide keys have no instance (166 KB at G = 2).
//
// What bounds it is latency: the chain of a query block's steps, each an LDS
// round trip, a row of MFMAs and the softmax that depends on them.  Measured
// against the unsplit kernel (us, B = 1, causal): d = 128 bf16 N = 2048 H = 8
// 32.5 -> 27.6, N = 8192 H = 1 107 -> 82.3 (G = 2); d = 64 N = 1000 H = 8
// 14.6 -> 10.2, N = 8192 H = 1 79.7 -> 35.9; FP8 N = 8192 H = 1 72.8 -> 36.4
// (G = 4).

#include <hip/hip_runtime.h>

#include "attn_fwd_kernel.h"
#include "attn_fwd_launch.h"

namespace qm {
namespace {

template <int DK, int DV, int DT, bool CAUSAL, int G, int LAYOUTS>
__global__ __launch_bounds__(512, 1) void attn_fwd_split_kernel(KParams p) {
  attn_fwd_body<DK, DV, DT, CAUSAL, 8 / G, G, LAYOUTS>(p);
}

template <int DK, int DV, int DT, int G, int LAYOUTS>
hipError_t launch_masks(const AttnArgs& a, const Device& dev, hipStream_t stream) {
  constexpr size_t lds = lds_bytes<DK, DV, DT, 8 / G, G>();
  static_assert(lds <= 160 * 1024, "a workgroup's rings fit the LDS");
  return a.causal ? launch_tiles<attn_fwd_split_kernel<DK, DV, DT, true, G, LAYOUTS>>(
                        a, dev, 256 / G, 512, lds, 1, stream)
                  : launch_tiles<attn_fwd_split_kernel<DK, DV, DT, false, G, LAYOUTS>>(
                        a, dev, 256 / G, 512, lds, 1, stream);
}

template <int DK, int DV, int DT, int G>
hipError_t launch_layouts(const AttnArgs& a, const Device& dev, hipStream_t stream) {
  return a.layout ? launch_masks<DK, DV, DT, G, kBnhdOnly>(a, dev, stream)
                  : launch_masks<DK, DV, DT, G, kBhndOnly>(a, dev, stream);
}

template <int D, int DT>
hipError_t launch_groups(const AttnArgs& a, const Device& dev, int groups, hipStream_t stream) {
  if constexpr (D == 64 || DT == 2) {
    if (groups == 4) return launch_layouts<D, D, DT, 4>(a, dev, stream);
  }
  return groups == 2 ? launch_layouts<D, D, DT, 2>(a, dev, stream) : hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_attn_fwd_split(const AttnArgs& a, int groups, hipStream_t stream) {
  Device dev;
  const hipError_t e = current_device(&dev);
  if (e != hipSuccess) return e;
  if (a.dtype == 2) return launch_groups<128, 2>(a, dev, groups, stream);
  if (a.d == 64) {
    return a.dtype == 0 ? launch_groups<64, 0>(a, dev, groups, stream)
                        : launch_groups<64, 1>(a, dev, groups, stream);
  }
  return a.dtype == 0 ? launch_groups<128, 0>(a, dev, groups, stream)
                      : launch_groups<128, 1>(a, dev, groups, stream);
}

}  // namespace qm
