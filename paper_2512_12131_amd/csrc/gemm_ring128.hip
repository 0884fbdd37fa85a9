// 128 x 128 output tiles (kernel: gemm_ring.h; a file of its own so that the tiles compile in parallel): two
// workgroups of four wavefronts per CU; or one of eight with a deeper ring, for the attention's query gradient,
// whose A operand is read once from HBM (per CU 128 KB of it in flight).
//
// gemm_stream_kernel: the same tiles, k-contiguous rows against a weight of either form, by two workgroups per CU that walk several
// each.  Bound: at short k the way into and out of a workgroup (16384 x 12288 x 128: two slices, 5 us each round of 512 tiles), at long k
// the latency of the one stage that is on its way while one is multiplied.  So a stage's operands all move to registers at once and a
// second barrier frees its slot for the stage after next, which may be the next tile's: two stages are on their way before an epilogue
// starts, and its stores drain behind the next tile's first stages.  The epilogue stages through 4 KB per wavefront beside the ring.
// us, a workgroup per tile -> stream: 16384 x 12288 x 128, plain store 124 -> 113; the SwiGLU pair of 16384 x 11008 x 128 213 -> 190,
// with g and u stored 320 -> 292; residual sum 16384 x 4096 x 128 88 -> 73; 2500 x 512 x 4096 45.6 -> 39.0, sigma' data gradients
// 2500 x 1024 x 1024 56 -> 46 and 16384 x 512 x 2048, three members 134 -> 123.
#include "gemm_ring.h"

namespace lrb {
namespace {

using Tile128 = RingTile<128, 128, 2, 2, 1, 2>;

// The epilogue's staging space beside the ring: 16 rows x 64 columns per wavefront at a time.  The XOR spreads what a cycle writes
// (one chunk of 16 rows) and reads (every second chunk of two rows) over all banks.
struct StreamStage {
  static constexpr int SR = 16, SC = 64;
  static constexpr bool STAT_IN_STAGE = false;
  static constexpr int BYTES = SR * SC * 4;
  unsigned char* p;
  __device__ __forceinline__ unsigned char* at(int row, int chunk) const { return p + row * 256 + (((chunk ^ row) & 15) << 4); }
};
constexpr int STREAM_LDS = Tile128::MAIN_BYTES + Tile128::NW * StreamStage::BYTES;
static_assert(2 * STREAM_LDS <= 160 * 1024, "two workgroups per CU");
constexpr int STREAM_WGS = 512;

template <int KIND, bool BKM>
__global__ __launch_bounds__(Tile128::NT, 2) void gemm_stream_kernel(GemmOp op, int tiles_m, int tiles_n, int total) {
  using T = Tile128;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr bool DUAL = KIND == EPI_SWIGLU_DUAL;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / T::WN, wn = wave % T::WN;
  // each XCD works through a contiguous range of tiles, its workgroups side by side
  {
    // all cache lines of the arguments at once (they come from the host's memory)
    constexpr int LINES = (sizeof(GemmOp) + 3 * sizeof(int) + 63) / 64;
    static_assert(LINES == 6, "the lines asked for below");
    const uint32_t* args = (const uint32_t*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" ::"s"(args[0]), "s"(args[16]), "s"(args[32]), "s"(args[48]), "s"(args[64]), "s"(args[80]));
  }
  const int bid = blockIdx.x, xcd = bid % NXCD, step = gridDim.x / NXCD;
  const int first = xcd * (total / NXCD) + min(xcd, total % NXCD);
  const int end = first + total / NXCD + (xcd < total % NXCD ? 1 : 0);
  const int nit1 = (op.K + BK - 1) / BK, nit = DUAL ? 2 * nit1 : nit1;
  const uint32_t sbase = (uint32_t)(uintptr_t)LRB_LDS_PTR(smem);

  // ---- loads: two stages ahead of the products, on from tile to tile ---------------------------------
  rsrc_words rsA, rsB;
  uint32_t offA[T::LA], offB[T::LB];
  int kA = 0, kB = 0;
  int pnid = first + bid / NXCD, pit = 0;                // tile and stage to be loaded next
  auto open = [&] {                                      // (behind the last tile: nothing, as zeros)
    int tm = 0, tn = 0, b = 0;
    const bool valid = pnid < end;
    if (valid) tile_of_index(pnid, tiles_m, tiles_n, tm, tn, b);
    const int m0 = tm * T::BM, n0 = tn * T::BN;
    rsA = operand_rsrc((const uint16_t*)op.A + (int64_t)b * op.sA + (int64_t)m0 * op.lda);
    rsB = operand_rsrc((const uint16_t*)op.B + (int64_t)b * op.sB + (BKM ? (int64_t)n0 : (int64_t)n0 * op.ldb));
    asm volatile("s_nop 4" : "+s"(rsA), "+s"(rsB));      // (see dma16)
    lane_offsets<T, false, T::BM>(offA, kA, op.lda, m0, valid ? op.M : 0, wave, lane);
    lane_offsets<T, BKM, T::BN>(offB, kB, op.ldb, n0, valid ? op.N : 0, wave, lane);
  };
  auto issue_one = [&](int slot, auto I) {
    constexpr int j = decltype(I)::value;
    constexpr bool is_a = j < T::LA, km = is_a ? false : BKM;
    constexpr int i = is_a ? j : j - T::LA;
    const bool other = DUAL && pit >= nit1;
    const int k0 = (other ? pit - nit1 : pit) * BK;
    uint32_t adv = (uint32_t)k0 * (km ? (uint32_t)op.ldb : 1u) * 2u;
    if (other) adv += (uint32_t)(is_a ? op.sA : op.sB) * 2u;
    const bool in = (k0 + (is_a ? kA : kB) + (km ? i * T::NWL * (512 / T::BN) : 0)) < op.K;
    const uint32_t dst = sbase + (uint32_t)(slot * T::STAGE + (is_a ? 0 : T::A_BYTES)) + (uint32_t)(wave + T::NWL * i) * 1024u;
    dma16<false>(is_a ? rsA : rsB, dst, in ? (is_a ? offA[is_a ? i : 0] : offB[is_a ? 0 : i]) + adv : RING_OOB);
  };
  auto advance = [&] {
    if (++pit == nit) {
      pit = 0;
      pnid += step;
      open();
    }
  };
  open();
#pragma unroll
  for (int s = 0; s < 2; s++) {
    static_for<T::LPS>([&](auto I) { issue_one(s, I); });
    advance();
  }

  // vector memory instructions that an epilogue certainly issues
  constexpr int OUT = DUAL ? 3 : KIND == EPI_SWIGLU_BWD || KIND == EPI_SWIGLU_FWD || KIND == EPI_ACTGRAD_A || KIND == EPI_LAXGRAD ? 2
                      : epi_writes_f32(KIND) ? 3 : 1;
  constexpr int STORES = OUT * T::TM * T::TN / (64 * 8);
  static_assert(T::LPS + STORES < 64, "vmcnt is a 6-bit counter");
  int slot = 0;
  bool stores_fly = false;
  for (int nid = first + bid / NXCD; nid < end; nid += step) {
    f32x16 acc[T::FM][T::FN];
    GateAcc<T> gate;
#pragma unroll
    for (int i = 0; i < T::FM; i++)
#pragma unroll
      for (int j = 0; j < T::FN; j++)
#pragma unroll
        for (int v = 0; v < 16; v++) acc[i][j][v] = 0.f;
    auto stage = [&](int it) {
      // This wavefront's loads of the stage have landed (behind them: the next stage's, and up to the second stage of a tile the stores of
      // the epilogue before), then everyone's
      asm volatile("" ::: "memory");
      if (stores_fly && it < 2) wait_vmcnt<T::LPS + STORES>();
      else wait_vmcnt<T::LPS>();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      bf16x8 af[4][T::FM], bf[4][T::FN];
      const unsigned char* sa = smem + slot * T::STAGE;
#pragma unroll
      for (int kk = 0; kk < 4; kk++) {
#pragma unroll
        for (int i = 0; i < T::FM; i++) af[kk][i] = ring_frag<false, T::BM, false>(sa, wm * T::TM + i * 32, kk, lane);
#pragma unroll
        for (int j = 0; j < T::FN; j++) bf[kk][j] = ring_frag<BKM, T::BN, false>(sa + T::A_BYTES, wn * T::TN + j * 32, kk, lane);
      }
      // the operands are in registers, everyone's: the slot takes the stage after next
      asm volatile("" ::: "memory");
      wait_lgkmcnt0();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      static_for<4>([&](auto KK) {
        constexpr int kk = decltype(KK)::value;
        constexpr int l0 = kk * T::LPS / 4, l1 = (kk + 1) * T::LPS / 4;
        static_for<l1 - l0>([&](auto L) { issue_one(slot, std::integral_constant<int, l0 + decltype(L)::value>{}); });
#pragma unroll
        for (int i = 0; i < T::FM; i++)
#pragma unroll
          for (int j = 0; j < T::FN; j++)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[kk][j], af[kk][i], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      });
      advance();
      slot ^= 1;
    };
    for (int it = 0; it < nit1; it++) stage(it);
    if constexpr (DUAL) {
      gate_from(gate, acc);
      for (int it = nit1; it < nit; it++) stage(it);
    }
    int tm, tn, b, elane = lane, ewave = wave;
    tile_of_index(nid, tiles_m, tiles_n, tm, tn, b);
    // (opaque copies: otherwise the epilogue's address arithmetic is moved out of the loop over tiles)
    asm volatile("" : "+v"(elane), "+s"(ewave));
    gemm_epilogue<T, KIND, false>(op, acc, StreamStage{smem + T::MAIN_BYTES + ewave * StreamStage::BYTES}, nullptr, ewave, elane, tm * T::BM,
                                  tn * T::BN, tn, tiles_n, b, b, 0, b, gate);
    stores_fly = true;
  }
  wait_vmcnt<0>();           // no load into LDS outlives its workgroup
}

template <int KIND, bool BKM>
hipError_t launch_stream(const GemmOp& op, hipStream_t st) {
  auto kern = gemm_stream_kernel<KIND, BKM>;
  // one-time opt-in to more than 64 KB of dynamic LDS (thread-safe function-local static)
  static const hipError_t attr_err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, STREAM_LDS);
  if (attr_err != hipSuccess) return attr_err;
  const int tiles_m = (op.M + 127) / 128, tiles_n = (op.N + 127) / 128;
  const int total = tiles_m * tiles_n * op.batch, wgs = total < STREAM_WGS ? (total + NXCD - 1) / NXCD * NXCD : STREAM_WGS;
  hipLaunchKernelGGL(kern, dim3(wgs), dim3(Tile128::NT), STREAM_LDS, st, op, tiles_m, tiles_n, total);
  return hipGetLastError();
}

template <bool BKM>
hipError_t dispatch_stream(const GemmOp& op, hipStream_t st) {
  switch (op.epi.kind) {
    case EPI_STORE: return launch_stream<EPI_STORE, BKM>(op, st);
    case EPI_UP: return launch_stream<EPI_UP, BKM>(op, st);
    default: break;
  }
  if constexpr (BKM) {
    switch (op.epi.kind) {
      case EPI_ACTGRAD: return launch_stream<EPI_ACTGRAD, true>(op, st);
      case EPI_ACTGRAD_A: return launch_stream<EPI_ACTGRAD_A, true>(op, st);
      case EPI_LAXGRAD: return launch_stream<EPI_LAXGRAD, true>(op, st);
      case EPI_NORMBWD: return launch_stream<EPI_NORMBWD, true>(op, st);
      case EPI_NORMBWD_O32: return launch_stream<EPI_NORMBWD_O32, true>(op, st);
      case EPI_NORMBWD_I32: return launch_stream<EPI_NORMBWD_I32, true>(op, st);
      case EPI_SWIGLU_BWD: return launch_stream<EPI_SWIGLU_BWD, true>(op, st);
      default: return hipErrorInvalidValue;
    }
  } else {
    switch (op.epi.kind) {
      case EPI_DOWN: return launch_stream<EPI_DOWN, false>(op, st);
      case EPI_DOWN_LAX: return launch_stream<EPI_DOWN_LAX, false>(op, st);
      case EPI_UP_O32: return launch_stream<EPI_UP_O32, false>(op, st);
      case EPI_UP_I32: return launch_stream<EPI_UP_I32, false>(op, st);
      case EPI_SWIGLU_FWD: return launch_stream<EPI_SWIGLU_FWD, false>(op, st);
      case EPI_SWIGLU_DUAL: return launch_stream<EPI_SWIGLU_DUAL, false>(op, st);
      default: return hipErrorInvalidValue;
    }
  }
}

}  // namespace

// As a stream of tiles, or a workgroup per tile where a launch is one round of them and k is short: one tile each gains nothing by what
// is asked for ahead and pays up to 1.3 us for it (us, a workgroup each / stream: 4096 x 2048 x 512 13.5 / 14.0, 10000 x 512 x 128 8.8 / 9.4).
hipError_t gemm_ring128(const GemmOp& op, hipStream_t st) {
  const int64_t tiles = (int64_t)((op.M + 127) / 128) * ((op.N + 127) / 128) * op.batch;
  const bool plain = op.epi.kind == EPI_STORE && !op.transB;
  if (!op.transA && op.splitk == 1 && op.k_parts == 1 && !op.epi.stat_from_a && !op.batch_inner && op.b_group == 1 &&
      tiles < (1 << 24) && (tiles > STREAM_WGS || (op.K >= 1024 && !plain)))
    return op.transB ? dispatch_stream<true>(op, st) : dispatch_stream<false>(op, st);
  return dispatch_ring<Tile128>(op, st);
}
hipError_t gemm_ring128w(const GemmOp& op, hipStream_t st) {
  if (!op.transA || !op.transB || op.epi.kind != EPI_STORE || op.splitk != 1) return hipErrorInvalidValue;
  return launch_ring<RingTile<128, 128, 2, 4, 1, 5>, EPI_STORE, false, true, true>(op, st);
}
}  // namespace lrb
