// The instances of the attention kernel (attn_fwd_kernel.h) and the choice of
// one per call: eight wavefronts (256 query rows, one workgroup per CU) or four
// (128 rows, two or three workgroups per CU); the smallest grids and the 128-row
// instances for other tensors are in files of their own.

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

// Eight waves keep K/V tiles in LDS for the most rows; four let one workgroup's
// prologue and epilogue run beside another's key loop, which wins where
// workgroups are short, and where the 256-row tiles, dealt out in rounds over
// the CUs, would leave too many of them idle.
int choose_waves(const AttnArgs& a, int cus) {
  const auto tiles = [&](int rows) {
    const long long nq = (a.N + rows - 1) / rows;
    return (a.causal ? (nq + 1) / 2 : nq) * a.B * a.H;
  };
  const long long rounds8 = (tiles(256) + cus - 1) / cus, rounds4 = (tiles(128) + cus - 1) / cus;
  // 192-wide keys run one workgroup of either size per CU: four waves where all
  // of theirs run at once (H = 16 N = 4096 causal 104.8 -> 85.6 us; in two
  // rounds, H = 8 N = 8192 unmasked, 270 -> 300).  Short causal pairs gain
  // nothing (H = 128 N = 512 23.5 -> 23.9), single query blocks do.
  if (a.d == 192) {
    const long long blocks = (long long)((a.N + 127) / 128) * a.B * a.H;
    return blocks <= cus || (a.N >= 768 && rounds4 == 1) ? 4 : 8;
  }
  // Short sequences, us, 256 -> 128 rows at a full grid: d = 128 bf16 N = 1024
  // 133 -> 131, N = 2048 233 -> 238, causal 145 -> 142, N = 4096 440 -> 457 and
  // 247 -> 247; d = 64 N = 2048 146 -> 138, N = 4096 274 -> 267, causal
  // 156 -> 150; FP8 N = 4096 282 -> 280, causal 165 -> 161.
  if (a.N <= (a.d == 64 || a.dtype == 2 ? 4096 : a.causal ? 2048 : 1024)) return 4;
  // Longer ones: a 256-row tile takes its CU 20 units of time, two 128-row
  // tiles side by side 21, a 128-row tile that has a CU to itself 14.  (B=3 H=32
  // N=3000: 392 -> 375 us, causal 257 -> 233; B=1 H=24 N=4096 causal, whose
  // 192 tiles of 256 rows fill 192 CUs: 104 us with them, 109 with 384 halves.)
  return rounds4 / 2 * 21 + rounds4 % 2 * 14 < rounds8 * 20 ? 4 : 8;
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
