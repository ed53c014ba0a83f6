// The instances of the attention kernel (attn_fwd_kernel.h) and the choice of
// one per call: eight wavefronts (256 query rows, one workgroup per CU) or four
// (128 rows, two or three workgroups per CU).

#include <hip/hip_runtime.h>

#include "attn_fwd_launch.h"
#include "attn_fwd_kernel.h"

namespace qm {
namespace {

template <int DK, int DV, int DT, bool CAUSAL, int WAVES>
__global__ __launch_bounds__(64 * WAVES, (wgs_per_cu<DK, WAVES>())) void attn_fwd_kernel(KParams p) {
  // the two-block-ring instances (192-wide keys, and four waves) take
  // [B][heads][N][w] only: runtime strides there spill registers
  constexpr int layouts = ring_depth<DK, DV, DT, WAVES>() == 4 ? kEitherLayout : kBhndOnly;
  attn_fwd_body<DK, DV, DT, CAUSAL, WAVES, 1, layouts>(p);
}

template <int DK, int DV, int DT, bool CAUSAL, int WAVES>
hipError_t launch_instance(const AttnArgs& a, const Device& dev, hipStream_t stream) {
  constexpr size_t lds = lds_bytes<DK, DV, DT, WAVES>();
  constexpr int per_cu = wgs_per_cu<DK, WAVES>();
  static_assert(lds * per_cu <= 160 * 1024, "the workgroups of a CU fit its LDS");
  // FP8: one workgroup per tile (see attn_fwd_body)
  return launch_tiles<attn_fwd_kernel<DK, DV, DT, CAUSAL, WAVES>>(
      a, dev, 32 * WAVES, 64 * WAVES, lds, per_cu, !Ops<DT>::kFp8, stream);
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
  // Workgroup size.  Eight waves (256 query rows, one workgroup per CU) keep
  // K/V tiles in LDS for the most rows; four waves (128 rows, two or three
  // workgroups per CU) let one workgroup's prologue and epilogue run beside
  // another's key loop.  That wins where workgroups are short (N <= 2048;
  // FP8, whose four-wave workgroups keep four-block rings: N <= 4096), and
  // where the 256-row workgroups, dealt out in rounds over the CUs, would
  // keep them under 80% busy (a lone four-wave workgroup in the last round
  // uses its CU better than an idle CU does).  Both give the same bytes: a
  // query row's arithmetic does not depend on its tile.  The [B][N][H][d]
  // layout and 192-wide keys run eight waves only.
  int waves = 8;
  if (a.layout == 0 && a.d != 192) {
    if (a.tile_rows == 128) {
      waves = 4;
    } else if (a.tile_rows == 0) {
      const long long nq8 = (a.N + 255) / 256;
      const long long wg8 = (a.causal ? (nq8 + 1) / 2 : nq8) * a.B * a.H;
      // the 256-row grid's work as a share of its rounds over the CUs
      const bool ragged = 5 * wg8 < 4 * ((wg8 + dev.cus - 1) / dev.cus) * (long long)dev.cus;
      // FP8 four-wave workgroups keep four-block rings and stay ahead longer
      if (a.N <= (a.dtype == 2 ? 4096 : 2048) || ragged) waves = 4;
    }
  }
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
