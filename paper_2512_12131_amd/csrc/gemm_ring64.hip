// 64 x 64 output tiles, one workgroup per CU with 160 KB of loads ahead of it (kernel: gemm_ring.h; a file of its own so that the tiles
// compile in parallel).
#include "gemm_ring.h"

namespace lrb {
hipError_t gemm_ring64(const GemmOp& op, hipStream_t st) { return dispatch_ring<RingTile<64, 64, 2, 2, 2, 5>>(op, st); }
}  // namespace lrb
