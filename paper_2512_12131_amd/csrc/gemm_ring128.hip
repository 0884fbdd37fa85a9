// 128 x 128 output tiles (kernel: gemm_ring.h; a file of its own so that the tiles compile in parallel): two
// workgroups of four wavefronts per CU; or one of eight with a deeper ring, for the attention's query gradient,
// whose A operand is read once from HBM (per CU 128 KB of it in flight).
#include "gemm_ring.h"

namespace lrb {
hipError_t gemm_ring128(const GemmOp& op, hipStream_t st) { return dispatch_ring<RingTile<128, 128, 2, 2, 1, 2>>(op, st); }
hipError_t gemm_ring128w(const GemmOp& op, hipStream_t st) {
  if (!op.transA || !op.transB || op.epi.kind != EPI_STORE || op.splitk != 1) return hipErrorInvalidValue;
  return launch_ring<RingTile<128, 128, 2, 4, 1, 5>, EPI_STORE, false, true, true>(op, st);
}
}  // namespace lrb
