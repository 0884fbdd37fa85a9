// 32 x 32 output tiles, two workgroups per CU: one wavefront multiplies, four load (kernel: gemm_ring.h; a file of
// its own so that the tiles compile in parallel).
#include "gemm_ring.h"

namespace lrb {
hipError_t gemm_ring32(const GemmOp& op, hipStream_t st) {
  if (gemm_rows16_ok(op)) return gemm_rows16(op, st);
  return dispatch_ring<RingTile<32, 32, 1, 1, 2, 5, 4>>(op, st);
}
}  // namespace lrb
