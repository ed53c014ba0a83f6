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
hipError_t launch_instance(const KParams& kp, hipStream_t stream) {
  constexpr size_t lds = lds_bytes<DK, DV, DT, WAVES>();
  constexpr int per_cu = wgs_per_cu<DK, WAVES>();
  static_assert(lds * per_cu <= 160 * 1024, "the workgroups of a CU fit its LDS");
  // FP8: one workgroup per tile (see attn_fwd_body)
  return launch_tiles<attn_fwd_kernel<DK, DV, DT, CAUSAL, WAVES>>(
      kp, 64 * WAVES, lds, Ops<DT>::kFp8 ? 0 : per_cu, stream);
}

template <int DK, int DV, int DT, int WAVES>
hipError_t launch_masks(const KParams& kp, bool causal, hipStream_t stream) {
  return causal ? launch_instance<DK, DV, DT, true, WAVES>(kp, stream)
                : launch_instance<DK, DV, DT, false, WAVES>(kp, stream);
}

template <int DK, int DV, int DT>
hipError_t launch_waves(const KParams& kp, bool causal, int waves, hipStream_t stream) {
  return waves == 4 ? launch_masks<DK, DV, DT, 4>(kp, causal, stream)
                    : launch_masks<DK, DV, DT, 8>(kp, causal, stream);
}

}  // namespace

hipError_t launch_attn_fwd(const AttnArgs& a, hipStream_t stream) {
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
      int dev = 0, cus = 0;
      const bool have_cus =
          hipGetDevice(&dev) == hipSuccess &&
          hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
          cus > 0;
      // the 256-row grid's work as a share of its rounds over the CUs
      const bool ragged =
          have_cus && 5 * wg8 < 4 * ((wg8 + cus - 1) / cus) * (long long)cus;
      // FP8 four-wave workgroups keep four-block rings and stay ahead longer
      if (a.N <= (a.dtype == 2 ? 4096 : 2048) || ragged) waves = 4;
    }
  }
  const KParams kp = make_params(a, 32 * waves);
  // head dimensions (d_qk, d_v): 64/64, 128/128, 192/128; FP8: 128/128
  const bool causal = a.causal != 0;
  if (a.dtype == 2) return launch_waves<128, 128, 2>(kp, causal, waves, stream);
  if (a.d == 64) {
    return a.dtype == 0 ? launch_waves<64, 64, 0>(kp, causal, waves, stream)
                        : launch_waves<64, 64, 1>(kp, causal, waves, stream);
  }
  if (a.d == 128) {
    return a.dtype == 0 ? launch_waves<128, 128, 0>(kp, causal, waves, stream)
                        : launch_waves<128, 128, 1>(kp, causal, waves, stream);
  }
  if (a.d == 192) {
    return a.dtype == 0 ? launch_masks<192, 128, 0, 8>(kp, causal, stream)
                        : launch_masks<192, 128, 1, 8>(kp, causal, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace qm
