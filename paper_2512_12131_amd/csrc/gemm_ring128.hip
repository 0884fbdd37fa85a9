// 128 x 128 output tiles, two workgroups per CU (kernel: gemm_ring.h; a file of its own so that the tiles
// compile in parallel).
#include "gemm_ring.h"

namespace lrb {
hipError_t gemm_ring128(const GemmOp& op, hipStream_t st) { return dispatch_ring<RingTile<128, 128, 2, 2, 1, 2>>(op, st); }
}  // namespace lrb
