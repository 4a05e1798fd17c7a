// kia_bf16.hip -- what only the bf16-output variant runs: the rounding of its
// fp32 accumulators. (The forward and backward kernels take both input types:
// bf16 inputs are one operand piece where fp32 inputs are three.)
#include "kia_device.hpp"
#include "kia_kernels.hpp"

namespace kia {

// ---------------------------------------------------------------------------
// The fp32 accumulators of dQ, dK (and dV where a split main kernel adds its
// parts up), which follow each other in the statistics, rounded once to bf16
// (nearest even), 8 elements per thread: n8 groups of 8 each, one row of
// workgroups per output. (One launch for all: three took 12 us at B1 H24 T1024
// d64, launch gaps for the most part.)
__global__ __launch_bounds__(256) void cast_bf16_kernel(const float *src, uint16_t *dq,
                                                       uint16_t *dk, uint16_t *dv, size_t n8) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n8) return;
  uint16_t *dst = blockIdx.y == 0 ? dq : (blockIdx.y == 1 ? dk : dv);
  const float *s = src + 8 * (i + blockIdx.y * n8);
  const f32x4 x = *reinterpret_cast<const f32x4 *>(s);
  const f32x4 y = *reinterpret_cast<const f32x4 *>(s + 4);
  *reinterpret_cast<uint4 *>(dst + 8 * i) =
      make_uint4(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(y[0], y[1]),
                 pack_bf16x2(y[2], y[3]));
}

}  // namespace kia
