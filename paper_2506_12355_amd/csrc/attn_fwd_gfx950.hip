// The instances of the attention kernel (attn_fwd_kernel.h), of which a call runs
// the one that attn_fwd_rules.h gives: eight wavefronts (256 query rows, one
// workgroup per CU) or four (128 rows, two or three workgroups per CU); the
// smallest grids and the 128-row instances for other tensors are in files of
// their own.

#include <hip/hip_runtime.h>

#include "attn_fwd_launch.h"
#include "attn_fwd_kernel.h"
#include "attn_fwd_rules.h"

namespace qm {
namespace {

template <int DK, int DV, int DT, bool CAUSAL, int WAVES>
__global__ __launch_bounds__(64 * WAVES, (wgs_per_cu<DK, WAVES>())) void attn_fwd_kernel(KParams p) {
  // Either layout for eight waves with four-block rings only: runtime strides spill
  // vector registers with two-block rings, and scalar ones in the four-wave FP8
  // instance (145 against 71 unmasked), whose key loop is bound by issue: N = 2048
  // H = 120 146.7 -> 144.0 us, H = 256 N = 2017 318 -> 305 unmasked; causal about 1%.
  constexpr int layouts =
      WAVES == 8 && ring_depth<DK, DV, DT, WAVES>() == 4 ? kEitherLayout : kBhndOnly;
  attn_fwd_body<DK, DV, DT, CAUSAL, WAVES, 1, layouts>(p);
}

template <int DK, int DV, int DT, bool CAUSAL, int WAVES>
hipError_t launch_instance(const AttnArgs& a, const Device& dev, hipStream_t stream) {
  constexpr size_t lds = lds_bytes<DK, DV, DT, WAVES>();
  constexpr int per_cu = wgs_per_cu<DK, WAVES>();
  static_assert(lds * per_cu <= 160 * 1024, "the workgroups of a CU fit its LDS");
  return launch_tiles<attn_fwd_kernel<DK, DV, DT, CAUSAL, WAVES>>(
      a, dev, 32 * WAVES, 64 * WAVES, lds, per_cu, stream);
}

template <int DK, int DV, int DT, int WAVES>
hipError_t launch_masks(const AttnArgs& a, const Device& dev, hipStream_t stream) {
  return a.causal ? launch_instance<DK, DV, DT, true, WAVES>(a, dev, stream)
                  : launch_instance<DK, DV, DT, false, WAVES>(a, dev, stream);
}

template <int DK, int DV, int DT>
hipError_t launch_waves(const AttnArgs& a, const Device& dev, int waves, hipStream_t stream) {
  return waves == 4 ? launch_masks<DK, DV, DT, 4>(a, dev, stream)
                    : launch_masks<DK, DV, DT, 8>(a, dev, stream);
}

}  // namespace

hipError_t launch_attn_fwd(const AttnArgs& a, hipStream_t stream) {
  Device dev;
  const hipError_t e = current_device(&dev);
  if (e != hipSuccess) return e;
  const int groups = key_groups(a, dev.cus);
  if (groups > 1) return launch_attn_fwd_split(a, groups, stream);
  // Workgroup size: eight waves (256 query rows, one workgroup per CU) or four
  // (128 rows, two or three per CU).  Both give the same bytes: a query row's
  // arithmetic does not depend on its tile.
  const int waves = a.tile_rows ? a.tile_rows / 32 : choose_waves(a, dev.cus);
  if (waves == 4 && (a.layout != 0 || a.d == 192)) return launch_attn_fwd_rows128(a, stream);
  // head dimensions (d_qk, d_v): 64/64, 128/128, 192/128; FP8: 128/128
  if (a.dtype == 2) return launch_waves<128, 128, 2>(a, dev, waves, stream);
  if (a.d == 64) {
    return a.dtype == 0 ? launch_waves<64, 64, 0>(a, dev, waves, stream)
                        : launch_waves<64, 64, 1>(a, dev, waves, stream);
  }
  if (a.d == 128) {
    return a.dtype == 0 ? launch_waves<128, 128, 0>(a, dev, waves, stream)
                        : launch_waves<128, 128, 1>(a, dev, waves, stream);
  }
  if (a.d == 192) {
    return a.dtype == 0 ? launch_masks<192, 128, 0, 8>(a, dev, stream)
                        : launch_masks<192, 128, 1, 8>(a, dev, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace qm
