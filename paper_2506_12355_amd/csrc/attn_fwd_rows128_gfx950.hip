// The attention kernel's four-wavefront, 128-row instances (attn_fwd_kernel.h) for
// the tensors that attn_fwd_gfx950.hip has only 256-row ones for: the
// [B][N][heads][width] layout, and 192-wide keys.
//
// The layout's row strides are runtime values here, which the [B][heads][N][width]
// instances are spared (in one instance for both they cost those 1-18%).  us,
// 256 -> 128 rows, [B][N][H][d], B=32 H=16 N=512 d=128 bf16: 81.1 -> 76.1 unmasked,
// 72.1 -> 60.0 causal; FP8 62.8 -> 50.9 and 53.7 -> 44.2; d=64 H=32 103.8 -> 90.0 and
// 92.1 -> 71.4; d=128 N=1024 B=16 131.9 -> 130.5 and 91.2 -> 85.7.
//
// 192-wide keys, whose rings let only one workgroup run on a CU, gain where the
// 256-row blocks would leave CUs idle: twice the workgroups, and a wavefront that
// has its SIMD to itself runs faster.  us, B=1 bf16 causal: H=16 N=4096
// 104.8 -> 85.6, N=2048 51.5 -> 36.2; H=2 N=8192 174 -> 115.
#include <hip/hip_runtime.h>

#include "attn_fwd_kernel.h"
#include "attn_fwd_launch.h"

namespace qm {
namespace {

// Workgroups per CU: two, or three at d = 64, as for the [B][heads][N][w]
// instances; 192-wide keys' rings (83 KB) leave room for one.  (Their registers, 245
// or 252, are bounded as if two ran all the same: no instance takes more than 256.)
template <int DK>
constexpr int per_cu() {
  return DK == 64 ? 3 : DK == 128 ? 2 : 1;
}

template <int DK, int DV, int DT, bool CAUSAL, int LAYOUTS>
__global__ __launch_bounds__(256, DK == 64 ? 3 : 2) void attn_fwd_rows128_kernel(KParams p) {
  attn_fwd_body<DK, DV, DT, CAUSAL, 4, 1, LAYOUTS>(p);
}

template <int DK, int DV, int DT, int LAYOUTS>
hipError_t launch_masks(const AttnArgs& a, const Device& dev, hipStream_t stream) {
  constexpr size_t lds = lds_bytes<DK, DV, DT, 4>();
  static_assert(lds * per_cu<DK>() <= 160 * 1024, "the workgroups of a CU fit its LDS");
  return a.causal ? launch_tiles<attn_fwd_rows128_kernel<DK, DV, DT, true, LAYOUTS>>(
                        a, dev, 128, 256, lds, per_cu<DK>(), stream)
                  : launch_tiles<attn_fwd_rows128_kernel<DK, DV, DT, false, LAYOUTS>>(
                        a, dev, 128, 256, lds, per_cu<DK>(), stream);
}

}  // namespace

hipError_t launch_attn_fwd_rows128(const AttnArgs& a, hipStream_t stream) {
  Device dev;
  const hipError_t e = current_device(&dev);
  if (e != hipSuccess) return e;
  if (a.d == 192) {
    return a.dtype == 0 ? launch_masks<192, 128, 0, kBhndOnly>(a, dev, stream)
                        : launch_masks<192, 128, 1, kBhndOnly>(a, dev, stream);
  }
  if (a.dtype == 2) return launch_masks<128, 128, 2, kBnhdOnly>(a, dev, stream);
  if (a.d == 64) {
    return a.dtype == 0 ? launch_masks<64, 64, 0, kBnhdOnly>(a, dev, stream)
                        : launch_masks<64, 64, 1, kBnhdOnly>(a, dev, stream);
  }
  return a.dtype == 0 ? launch_masks<128, 128, 0, kBnhdOnly>(a, dev, stream)
                      : launch_masks<128, 128, 1, kBnhdOnly>(a, dev, stream);
}

}  // namespace qm
