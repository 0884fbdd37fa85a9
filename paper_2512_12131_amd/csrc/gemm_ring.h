// bf16 MFMA GEMM for launches that the 256-row tiles of gemm_bf16.hip cannot spread over the chip:
// C[M,N] = epi( sum_k A[m,k] * B[n,k] ), fp32 accumulate, every epilogue of that kernel.
//
// Bound: with few output tiles per CU the time of a launch is the time one workgroup takes to walk k, and
// that is set by the latency of its global->LDS loads, not by the matrix pipes.  So the tiles are small (the
// output spreads over more CUs) and the loads run far ahead: a ring of NS LDS stages, NS - 1 of them in
// flight, one barrier per stage.  The small tiles read each operand element more often than the 256 x 256
// tile does, which is why that one keeps the launches that fill the chip (gemm_bf16_tile).
//
// Every output element is summed by the same MFMA instruction in the same k order, and from the same k slots,
// as in the 256-row kernel: which of the two kernels runs a product does not change its
// bits, so a token's result does not depend on how many tokens share the call.  The row statistics keep to that
// too: k_rowsum_parts adds the narrower row partials of these tiles up in the order in which a wider wavefront does.
//
// Measured (us, this kernel's best tile against the 256-row kernel): 777 x 1024 x 11008 37 / 172, 1031 x 256 x 1024
// 6.5 / 22, 16384 x 128 x 4096 30 / 72, 512 x 256 x 64 4.2 / 7.2.  A 64 x 64 tile takes 0.21 us per 64-wide slice: a
// wavefront's 32 x 32 block reads 2 KB of LDS per MFMA, so the LDS port (128 B per cycle) is busy for twice the
// matrix time, and the loads (one 1 KB load per ~17 cycles and CU) for as long again.  Reading all operands of a
// stage before issuing the next loads took 12 % off that; a ring of ten 16 KB stages was slower.
// A handful of rows (16 x 1024 x 4096) leaves one chain of 256 MFMAs per 32 x 32 block, 3.4 us of matrix time in
// the order that keeps a row's bits: there the 32 x 32 tile gives the chain a wavefront of its own and the loads
// to four others, 0.095 us per slice (15.0 -> 9.4 us; 16 x 4096 x 1024 6.6 -> 5.5; the same split at 64 x 64: 13.3).
//
// EPI_SWIGLU_DUAL walks the gate's product and then the up product in one stream of stages: the gate's accumulators wait as bf16
// pairs (half of the registers; what the epilogue would read back from memory), and g never leaves the chip where nobody wants it.
// Bound: the d_ff wide stores and the epilogue (16384 x 11008, k = 128, inside a block: g, then u with the epilogue 113 + 216 us,
// together 219, and 197 as a stream of tiles; with g and u stored 111 + 287 -> 292).
//
// Operand forms: k-contiguous (p[i*ld + k]) or k-major (p[k*ld + i]) for A and B independently; the k-major
// side is read through the LDS transpose read, so a data-gradient product needs no transposed weight copy.
#pragma once
#include "gemm_tile.h"

namespace lrb {
namespace {

// NL = 0: every wavefront loads its share of a stage and multiplies.  NL > 0: NL further wavefronts do nothing but
// load, the WM x WN others nothing but multiply.
template <int BM_, int BN_, int WM_, int WN_, int SUB_, int NS_, int NL_ = 0>
struct RingTile {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_;
  static constexpr int SUB = SUB_;                     // 64-wide k slices per LDS stage (one barrier per stage)
  static constexpr int NS = NS_;                       // stages in the ring
  static constexpr int NL = NL_;
  static constexpr int NW = WM * WN, NT = (NW + NL) * 64;
  static constexpr int NWL = NL > 0 ? NL : NW;         // wavefronts that load
  static constexpr int TM = BM / WM, TN = BN / WN;
  static constexpr int FM = TM / 32, FN = TN / 32;
  static constexpr int A_BYTES = BM * 128, B_BYTES = BN * 128, SLICE = A_BYTES + B_BYTES, STAGE = SUB * SLICE;
  static constexpr int LA = BM / 8 / NWL, LB = BN / 8 / NWL;   // 1 KB wavefront loads per wavefront and slice
  static constexpr int LPS = (LA + LB) * SUB;                // ... and stage
  static constexpr int CS = TN + 4;                          // fp32 row stride of the epilogue staging tile
  static constexpr int STAGE_BYTES = 32 * CS * 4;            // ... of a wavefront
  static constexpr int EPI_BYTES = NW * STAGE_BYTES;
  struct EpiStage {
    static constexpr int SR = 32, SC = TN;
    static constexpr bool STAT_IN_STAGE = false;
    unsigned char* p;
    __device__ __forceinline__ unsigned char* at(int row, int chunk) const { return p + row * (CS * 4) + chunk * 16; }
  };
  static constexpr int STAT_OFF = EPI_BYTES;
  static constexpr int MAIN_BYTES = NS * STAGE;
  static constexpr int LDS_BYTES = MAIN_BYTES > EPI_BYTES + BM * 4 ? MAIN_BYTES : EPI_BYTES + BM * 4;
  static_assert(BM / 8 % NWL == 0 && BN / 8 % NWL == 0 && NWL % 2 == 0 && FM >= 1 && FN >= 1, "tile / wavefront layout mismatch");
  static_assert(NS >= 2 && (NS - 2) * LPS < 64, "vmcnt is a 6-bit counter");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS of a CU");
  // main-loop statistics: TPR threads (of one quad of lanes) share a row, each takes 8 / TPR chunks of every slice
  static constexpr int TPR = NT / BM < 4 ? NT / BM : 4;
  static_assert(TPR == 2 || TPR == 4, "threads per tile row");
};

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

typedef uint32_t rsrc_words __attribute__((ext_vector_type(4)));

// One 1 KB global -> LDS load of a wavefront: lane L's 16 bytes land at lds + 16 L.  Inline assembly, because
// through the builtin the compiler makes later LDS reads wait for every load in flight; completion is counted
// by hand (wait_vmcnt before the barrier that publishes a stage).  No output register is written.  The compiler's hazard
// pass does not see a memory instruction in here, so the loads that follow the making of the descriptors (FIRST) make the five
// wait states themselves that have to pass between a vector write of a scalar (the v_readfirstlane of operand_rsrc) and a
// buffer instruction that reads it; a descriptor reloaded from a spill would be another.  (Five in every load: 3-5 % of a
// launch on 64 x 128 and 128 x 128 tiles; in a block of their own behind the descriptors: 16-token layer 15.2 -> 15.6 us.)
template <bool FIRST>
__device__ __forceinline__ void dma16(rsrc_words rs, uint32_t lds, uint32_t voff) {
  if constexpr (FIRST)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds), "v"(voff), "s"(rs) : "m0", "memory");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds), "v"(voff), "s"(rs) : "m0", "memory");
}
__device__ __forceinline__ rsrc_words operand_rsrc(const void* base) {
  const uint64_t a = (uint64_t)(uintptr_t)base;
  const rsrc_words r = {(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a),
                        (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xffffu)), 0x7fffffffu, 0x00020000u};
  return r;
}

// Swizzle of a k-major stage ([k][W columns], 2 W bytes per k row): the term XORed into the 16-byte chunk index
// of row k.  A transpose read takes 64 bytes out of each of four consecutive rows per half wavefront; with this
// term the four land on different 64-byte quarters of the 256 bytes of banks.  It repeats every four rows, so
// the second read of an operand (k + 4) differs from the first by a constant offset.
template <int W>
__device__ __forceinline__ int kmajor_swz(int k) {
  return W >= 128 ? (k & 3) << 2 : W == 64 ? ((k >> 1) & 1) << 2 : 0;
}

constexpr uint32_t RING_OOB = 0x80000000u;               // beyond every resource: the load delivers zeros

// A wavefront's loads of one slice of an operand: group g = lw + NWL * i covers 8 rows x 128 B
// (k-contiguous; chunk index XORed by (row / 2) % 8) or 512 / W k rows x 2 W bytes (k-major).
// i0, lim: first row (k-contiguous) or column (k-major) of the tile, and where the matrix ends.
template <class T, bool KM, int W, int NI>
__device__ __forceinline__ void lane_offsets(uint32_t (&off)[NI], int& k_of_lane, int64_t ld, int i0, int lim, int lw, int lane) {
  static_assert(NI == W / 8 / T::NWL, "loads of a wavefront");
#pragma unroll
  for (int i = 0; i < NI; i++) {
    const int g = lw + T::NWL * i;
    if constexpr (!KM) {
      const int row = g * 8 + (lane >> 3);
      const int lc = (lane & 7) ^ ((row >> 1) & 7);
      if (i == 0) k_of_lane = lc * 8;                  // the same for every i: NWL * 8 rows apart, NWL even
      off[i] = (i0 + row) < lim ? (uint32_t)(row * (int)ld + lc * 8) * 2u : RING_OOB;
    } else {
      constexpr int CPR = W / 8, RPL = 64 / CPR;
      const int krow = g * RPL + lane / CPR;
      const int lc = (lane % CPR) ^ kmajor_swz<W>(krow);
      if (i == 0) k_of_lane = krow;                    // load i: NWL * RPL rows further
      off[i] = (i0 + lc * 8) < lim ? (uint32_t)(krow * (int)ld + lc * 8) * 2u : RING_OOB;
    }
  }
}

// MFMA operands: 32 rows (lane % 32) x 8 consecutive k (k16 step kk, half lane / 32) from either layout.  BOTH: both operands are k-major.
template <bool KM, int W, bool BOTH>
__device__ __forceinline__ bf16x8 ring_frag(const unsigned char* base, int r0, int kk, int lane) {
  const int frow = lane & 31, fhalf = lane >> 5, fsw = (frow >> 1) & 7;
  if constexpr (!KM) {
    return *reinterpret_cast<const bf16x8*>(base + (r0 + frow) * 128 + (((kk * 2 + fhalf) ^ fsw) << 4));
  } else {
    // Inside 16 lanes, lane s supplies the address of 4 columns of k row s / 4 and receives column s.  Beside a
    // k-contiguous operand the lane's slots are its half's 8 consecutive k.  With two k-major operands they are
    // the two runs of four of the 256-row kernel's k-major form (k = (e / 4) * 8 + half * 4 + e % 4): the order of
    // the sum, and so the bits of the attention's query gradient, must not depend on which of the two runs.
    const int g = lane >> 4, s = lane & 15;
    const int krow = fhalf * (BOTH ? 4 : 8) + (s >> 2);
    const int col = r0 + (g & 1) * 16 + (s & 3) * 4;
    const unsigned char* p = base + (kk * 16 + krow) * (2 * W) + (((col >> 3) ^ kmajor_swz<W>(krow)) << 4) + (col & 7) * 2;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p + (BOTH ? 8 : 4) * 2 * W));
    const s16x8 r = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, r);
  }
}

// The gate's accumulators put away, and cleared for the other product.
template <class T>
__device__ __forceinline__ void gate_from(GateAcc<T>& gate, f32x16 (&acc)[T::FM][T::FN]) {
#pragma unroll
  for (int i = 0; i < T::FM; i++)
#pragma unroll
    for (int j = 0; j < T::FN; j++)
#pragma unroll
      for (int g = 0; g < 4; g++) {
        gate.v[i][j][g] = make_uint2(pack_bf16x2(acc[i][j][4 * g], acc[i][j][4 * g + 1]), pack_bf16x2(acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]));
#pragma unroll
        for (int r = 0; r < 4; r++) acc[i][j][4 * g + r] = 0.f;
      }
}

// PARTS: k runs in op.k_parts parts that are summed one by one, as split-K partials are.
// bid: this workgroup among the `total` of the product.
template <class T, int KIND, bool STAT_A, bool AKM, bool BKM, bool PARTS>
__device__ __forceinline__ void ring_product(const GemmOp& op, int kper, int tiles_m, int tiles_n, int bid, int total) {
  static_assert(!(STAT_A && AKM), "row statistics are gathered from k-contiguous rows");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / T::WN, wn = wave % T::WN;        // (of a multiplying wavefront)
  const int lw = T::NL > 0 ? wave - T::NW : wave;        // index among the loading wavefronts (below 0: not one)
  int tm, tn, bz;
  tile_of_block(bid, total, tiles_m, tiles_n, tm, tn, bz);
  if (AKM && BKM && op.causal_k) tm = tiles_m - 1 - tm;   // the longest k ranges of a batch member first
  const int m0 = tm * T::BM, n0 = tn * T::BN;
  const int b = bz / op.splitk, ks = bz % op.splitk;
  const int kbeg = ks * kper;
  int kend = min(op.K, kbeg + kper);
  if (AKM && BKM && op.causal_k) kend = min(kend, m0 + T::BM);
  const int bo = op.batch_inner > 0 ? b / op.batch_inner : 0, bi = op.batch_inner > 0 ? b % op.batch_inner : b;
  const int klen = kend > kbeg ? kend - kbeg : 0;
  constexpr int KST = T::SUB * BK, KSTEPS = T::SUB * 4;  // k elements and k16 steps per stage
  // DUAL: the stages of the gate's product, then those of the other one, in one stream
  constexpr bool DUAL = KIND == EPI_SWIGLU_DUAL;
  const int nit1 = (klen + KST - 1) / KST, nit = DUAL ? 2 * nit1 : nit1;

  const uint16_t* A = (const uint16_t*)op.A + (int64_t)bi * op.sA + (int64_t)bo * op.sAo;
  const uint16_t* B = (const uint16_t*)op.B + (int64_t)(bi / op.b_group) * op.sB + (int64_t)bo * op.sBo;
  constexpr uint32_t OOB = RING_OOB;
  const rsrc_words rsA = operand_rsrc(AKM ? A + (int64_t)kbeg * op.lda + m0 : A + (int64_t)m0 * op.lda + kbeg);
  const rsrc_words rsB = operand_rsrc(BKM ? B + (int64_t)kbeg * op.ldb + n0 : B + (int64_t)n0 * op.ldb + kbeg);
  const uint32_t sbase = (uint32_t)(uintptr_t)LRB_LDS_PTR(smem);

  uint32_t offA[T::LA], offB[T::LB];
  int kA = 0, kB = 0;        // this lane's first k inside the slice: of its chunk (k-contiguous) or its row (k-major)
  lane_offsets<T, AKM, T::BM>(offA, kA, op.lda, m0, op.M, lw, lane);
  lane_offsets<T, BKM, T::BN>(offB, kB, op.ldb, n0, op.N, lw, lane);

  // Load I (compile-time, 0 .. LPS - 1) of stage `it` into ring slot `slot`.  k past the end of the range (also
  // whole stages past it) reads as zeros, so the loop needs no tail code and the counts of loads in flight are
  // constants.
  auto issue_one = [&](int it, int slot, auto I, auto FIRST) {
    constexpr int s = decltype(I)::value / (T::LA + T::LB), j = decltype(I)::value % (T::LA + T::LB);
    constexpr bool is_a = j < T::LA, km = is_a ? AKM : BKM;
    constexpr int i = is_a ? j : j - T::LA, W = is_a ? T::BM : T::BN, RPL = 512 / W;
    const bool other = DUAL && it >= nit1;
    const int k0 = (other ? it - nit1 : it) * KST + s * BK;
    uint32_t adv = (uint32_t)k0 * (km ? (uint32_t)(is_a ? op.lda : op.ldb) : 1u) * 2u;
    if (other) adv += (uint32_t)(is_a ? op.sA : op.sB) * 2u;
    const bool in = (k0 + (is_a ? kA : kB) + (km ? i * T::NWL * RPL : 0)) < klen;
    const uint32_t dst = sbase + (uint32_t)(slot * T::STAGE + s * T::SLICE + (is_a ? 0 : T::A_BYTES)) +
                         (uint32_t)(lw + T::NWL * i) * 1024u;
    dma16<decltype(FIRST)::value>(is_a ? rsA : rsB, dst, in ? (is_a ? offA[is_a ? i : 0] : offB[is_a ? 0 : i]) + adv : OOB);   // OOB + adv stays past the resource
  };

  f32x16 acc[T::FM][T::FN];
#pragma unroll
  for (int i = 0; i < T::FM; i++)
#pragma unroll
    for (int j = 0; j < T::FN; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[i][j][v] = 0.f;
  // PARTS: sum of the finished parts; a part ends on a slice boundary
  f32x16 tot[PARTS ? T::FM : 1][PARTS ? T::FN : 1];
  const int part_slices = PARTS ? ((op.K + op.k_parts - 1) / op.k_parts + BK - 1) / BK : 0;
  int part_end = part_slices;
  if constexpr (PARTS) {
#pragma unroll
    for (int i = 0; i < T::FM; i++)
#pragma unroll
      for (int j = 0; j < T::FN; j++) tot[i][j] = acc[i][j];
  }
  // STAT_A: sum of squares of tile row tid / TPR, in the first of its TPR threads, and this thread's chunk sums of a stage.
  // That thread adds the eight chunk sums of a slice, the others' from their registers, in the order they lie in LDS, as the one
  // thread per row of the 256-row kernel does: same bits whichever tile runs.
  constexpr int CPT = 8 / T::TPR;
  float ssq = 0.f, cs[T::SUB * CPT] = {};
  auto add_chunks = [&] {
    static_for<T::SUB * 8>([&](auto C) {
      constexpr int c = decltype(C)::value % 8, j = c / CPT;   // chunk of the slice; the thread of the row that holds it
      constexpr int ctrl = T::TPR == 4 ? j * 0x55 : 0xF5;      // quad_perm [j,j,j,j] / [1,1,3,3]
      const float v = cs[decltype(C)::value / 8 * CPT + c % CPT];
      if constexpr (j == 0) ssq += v;
      else ssq += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), ctrl, 0xf, 0xf, true));
    });
  };

#pragma unroll
  for (int s = 0; s < T::NS - 1; s++)
    if (lw >= 0) static_for<T::LPS>([&](auto I) { issue_one(s, s, I, std::true_type{}); });
  int rd = 0, wr = T::NS - 1;                            // slots read from and written to
  auto stage = [&](int it) {
    // this wavefront's loads of stage `it` have landed (loads retire in order), and its reads of the stage
    // before are done; after the barrier that holds for all of them
    asm volatile("" ::: "memory");
    wait_vmcnt<(T::NS - 2) * T::LPS>();
    wait_lgkmcnt0();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if constexpr (T::NL > 0) {
      if (lw >= 0) static_for<T::LPS>([&](auto I) { issue_one(it + T::NS - 1, wr, I, std::false_type{}); });
    }
    if (T::NL == 0 || lw < 0) {
      // all operand reads of the stage first, then the next stage's loads among the MFMAs: a CU accepts one 1 KB
      // load per ~17 cycles and a wavefront issues in order, so loads in front of the reads would delay them
      bf16x8 af[KSTEPS][T::FM], bf[KSTEPS][T::FN];
#pragma unroll
      for (int kk = 0; kk < KSTEPS; kk++) {
        const unsigned char* sa = smem + rd * T::STAGE + (kk / 4) * T::SLICE;
#pragma unroll
        for (int i = 0; i < T::FM; i++) af[kk][i] = ring_frag<AKM, T::BM, AKM && BKM>(sa, wm * T::TM + i * 32, kk % 4, lane);
#pragma unroll
        for (int j = 0; j < T::FN; j++)
          bf[kk][j] = ring_frag<BKM, T::BN, AKM && BKM>(sa + T::A_BYTES, wn * T::TN + j * 32, kk % 4, lane);
      }
      asm volatile("" ::: "memory");
      static_for<KSTEPS>([&](auto KK) {
        constexpr int kk = decltype(KK)::value;
        if constexpr (PARTS && kk % 4 == 0) {
          if (it * T::SUB + kk / 4 == part_end) {
            part_end += part_slices;
#pragma unroll
            for (int i = 0; i < T::FM; i++)
#pragma unroll
              for (int j = 0; j < T::FN; j++)
#pragma unroll
                for (int v = 0; v < 16; v++) {
                  tot[i][j][v] += acc[i][j][v];
                  acc[i][j][v] = 0.f;
                }
          }
        }
        constexpr int l0 = kk * T::LPS / KSTEPS, l1 = (kk + 1) * T::LPS / KSTEPS;
        if constexpr (T::NL == 0) static_for<l1 - l0>([&](auto L) { issue_one(it + T::NS - 1, wr, std::integral_constant<int, l0 + decltype(L)::value>{}, std::false_type{}); });
#pragma unroll
        for (int i = 0; i < T::FM; i++)
#pragma unroll
          for (int j = 0; j < T::FN; j++)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[kk][j], af[kk][i], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      });
    }
    if constexpr (STAT_A) {
      // Each of a row's threads squares its chunks of the stage; the sums of the stage before are added up meanwhile.
      if (T::BM * T::TPR == T::NT || tid < T::BM * T::TPR) {
        uint4 q[T::SUB * CPT];
#pragma unroll
        for (int c = 0; c < T::SUB * CPT; c++)
          q[c] = *reinterpret_cast<const uint4*>(smem + rd * T::STAGE + c / CPT * T::SLICE + (tid / T::TPR) * 128 +
                                                 ((tid % T::TPR) * CPT + c % CPT) * 16);
        add_chunks();
#pragma unroll
        for (int c = 0; c < T::SUB * CPT; c++) cs[c] = sumsq8(q[c]);
      }
    }
    rd = rd + 1 == T::NS ? 0 : rd + 1;
    wr = wr + 1 == T::NS ? 0 : wr + 1;
  };
  for (int it = 0; it < nit1; it++) stage(it);
  GateAcc<T> gate;
  if constexpr (DUAL) {
    gate_from(gate, acc);
    for (int it = nit1; it < nit; it++) stage(it);
  }
  wait_vmcnt<0>();
  __syncthreads();           // the ring is dead from here on
  float* sStat = reinterpret_cast<float*>(smem + T::STAT_OFF);
  if constexpr (STAT_A) {
    add_chunks();            // of the last stage
    if (tid < T::BM * T::TPR && tid % T::TPR == 0) sStat[tid / T::TPR] = ssq;
    __syncthreads();
  }
  if (T::NL > 0 && lw >= 0) return;
  if constexpr (PARTS) {
#pragma unroll
    for (int i = 0; i < T::FM; i++)
#pragma unroll
      for (int j = 0; j < T::FN; j++)
#pragma unroll
        for (int v = 0; v < 16; v++) acc[i][j][v] += tot[i][j][v];
  }
  gemm_epilogue<T, KIND, STAT_A>(op, acc, typename T::EpiStage{smem + wave * T::STAGE_BYTES}, sStat, wave, lane, m0, n0, tn, tiles_n, b, bi, bo, bz, gate);
}

template <class T, int KIND, bool STAT_A, bool AKM, bool BKM, bool PARTS>
__global__ __launch_bounds__(T::NT) void gemm_ring_kernel(GemmOp op, int kper, int tiles_m, int tiles_n) {
  ring_product<T, KIND, STAT_A, AKM, BKM, PARTS>(op, kper, tiles_m, tiles_n, blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y);
}

template <class T, int KIND, bool STAT_A, bool AKM, bool BKM, bool PARTS = false>
hipError_t launch_ring(const GemmOp& op, hipStream_t st) {
  if (!PARTS && op.k_parts != 1) return hipErrorInvalidValue;
  auto kern = gemm_ring_kernel<T, KIND, STAT_A, AKM, BKM, PARTS>;
  // one-time opt-in to more than 64 KB of dynamic LDS (thread-safe function-local static)
  static const hipError_t attr_err =
      hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
  if (attr_err != hipSuccess) return attr_err;
  const int tiles_m = (op.M + T::BM - 1) / T::BM, tiles_n = (op.N + T::BN - 1) / T::BN;
  int kper = (op.K + op.splitk - 1) / op.splitk;
  kper = (kper + BK - 1) / BK * BK;    // a split ends on a slice boundary; a ragged last stage reads zeros
  hipLaunchKernelGGL(kern, tile_grid(tiles_m * tiles_n, op.batch * op.splitk), dim3(T::NT), T::LDS_BYTES, st, op, kper, tiles_m, tiles_n);
  return hipGetLastError();
}

// Every (epilogue, operand form) the sequencing code issues: forward products have both operands k-contiguous,
// data gradients a k-major weight, weight gradients and the attention's query gradient two k-major operands.
template <class T>
hipError_t dispatch_ring(const GemmOp& op, hipStream_t st) {
  const int kind = op.splitk > 1 ? (int)EPI_PARTIAL : op.epi.kind;
  const bool stat = op.epi.stat_from_a != 0;
  if (op.transA && op.transB && op.k_parts > 1) {
    // (with 64 x 64 per wavefront the second set of accumulators leaves one workgroup per CU)
    if constexpr (T::FM * T::FN < 4) {
      if (op.splitk == 1 && kind == EPI_PARTIAL) return launch_ring<T, EPI_PARTIAL, false, true, true, true>(op, st);
      if (op.splitk == 1 && kind == EPI_STORE) return launch_ring<T, EPI_STORE, false, true, true, true>(op, st);
    }
    return hipErrorInvalidValue;
  }
  if (op.transA && op.transB) {
    switch (kind) {
      case EPI_PARTIAL: return launch_ring<T, EPI_PARTIAL, false, true, true>(op, st);
      case EPI_STORE: return launch_ring<T, EPI_STORE, false, true, true>(op, st);
      default: return hipErrorInvalidValue;
    }
  }
  if (op.transB) {
    switch (kind) {
      case EPI_STORE: return launch_ring<T, EPI_STORE, false, false, true>(op, st);
      case EPI_UP: return launch_ring<T, EPI_UP, false, false, true>(op, st);
      case EPI_ACTGRAD: return launch_ring<T, EPI_ACTGRAD, false, false, true>(op, st);
      case EPI_ACTGRAD_A: return launch_ring<T, EPI_ACTGRAD_A, false, false, true>(op, st);
      case EPI_LAXGRAD: return launch_ring<T, EPI_LAXGRAD, false, false, true>(op, st);
      case EPI_NORMBWD: return launch_ring<T, EPI_NORMBWD, false, false, true>(op, st);
      case EPI_NORMBWD_O32: return launch_ring<T, EPI_NORMBWD_O32, false, false, true>(op, st);
      case EPI_NORMBWD_I32: return launch_ring<T, EPI_NORMBWD_I32, false, false, true>(op, st);
      case EPI_SWIGLU_BWD: return launch_ring<T, EPI_SWIGLU_BWD, false, false, true>(op, st);
      default: return hipErrorInvalidValue;
    }
  }
  switch (kind) {
    case EPI_STORE: return launch_ring<T, EPI_STORE, false, false, false>(op, st);
    case EPI_DOWN:
      return stat ? launch_ring<T, EPI_DOWN, true, false, false>(op, st) : launch_ring<T, EPI_DOWN, false, false, false>(op, st);
    case EPI_DOWN_LAX:
      return stat ? launch_ring<T, EPI_DOWN_LAX, true, false, false>(op, st)
                  : launch_ring<T, EPI_DOWN_LAX, false, false, false>(op, st);
    case EPI_UP: return launch_ring<T, EPI_UP, false, false, false>(op, st);
    case EPI_UP_O32: return launch_ring<T, EPI_UP_O32, false, false, false>(op, st);
    case EPI_UP_I32: return launch_ring<T, EPI_UP_I32, false, false, false>(op, st);
    case EPI_SWIGLU_FWD: return launch_ring<T, EPI_SWIGLU_FWD, false, false, false>(op, st);
    case EPI_SWIGLU_DUAL: return launch_ring<T, EPI_SWIGLU_DUAL, false, false, false>(op, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace
}  // namespace lrb
