// The 32 x 32 tile of a few rows worked as 16 x 16 pieces: C[M,N] = epi( sum_k A[m,k] * B[n,k] ), both operands
// k-contiguous, plain store or down-projection: the forward products of one layer on a handful of tokens.
//
// Bound: bytes in flight.  The weight is read once, so the time is how fast the CUs that hold a piece of it bring it in, and
// a CU accepts a 1 KB global->LDS load every 17 cycles.  A 32 x 32 tile leaves N / 32 workgroups (32 CUs for
// 16 x 1024 x 4096) and loads 16 rows of nothing; 16 x 16 pieces double the workgroups, halve what each brings in per k, and
// walk k at 16 cycles of matrix time per 32 instead of 64.  One wavefront multiplies (v_mfma_f32_16x16x32_bf16), four load
// into a ring of five stages of 256 k; the operands of a stage are read while the stage before is multiplied.
// The instruction adds its 32 products in the order of two 32 x 32 x 16 ones (measured on random operands up to k = 4096, no
// bit different), so an element has the bits that every other tile gives it.
// Measured (us, both products of a layer replayed from a graph, 32 x 32 tiles -> 16 x 16 pieces), 4096 -> 1024 -> 4096: 16 tokens
// 14.6 -> 8.5, 64 tokens 15.0 -> 10.1, 128 tokens 16.4 -> 14.8; 1024 -> 256 -> 1024: 16 tokens 8.5 -> 6.4.
#include "gemm_ring.h"

namespace lrb {
namespace {

constexpr int R16_NS = 5, R16_SLICE = 4096, R16_STAGE = 4 * R16_SLICE, R16_KST = 4 * BK, R16_LDS = R16_NS * R16_STAGE;

template <int KIND>
__global__ __launch_bounds__(320) void gemm_rows16_kernel(GemmOp op, int tiles_m, int tiles_n) {
  static_assert(KIND == EPI_STORE || KIND == EPI_DOWN, "plain store or down-projection");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tm, tn, b;
  tile_of_block(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y, tiles_m, tiles_n, tm, tn, b);
  const int m0 = tm * 16, n0 = tn * 16;
  const int bo = op.batch_inner > 0 ? b / op.batch_inner : 0, bi = op.batch_inner > 0 ? b % op.batch_inner : b;
  const uint16_t* A = (const uint16_t*)op.A + (int64_t)bi * op.sA + (int64_t)bo * op.sAo + (int64_t)m0 * op.lda;
  const uint16_t* B = (const uint16_t*)op.B + (int64_t)(bi / op.b_group) * op.sB + (int64_t)bo * op.sBo + (int64_t)n0 * op.ldb;
  const int nit = (op.K + R16_KST - 1) / R16_KST, npair = (nit + 1) / 2;   // stages; they are taken in pairs, an odd one with zeros

  if (wave > 0) {
    // Loader w takes slice w (64 k) of each stage: 16 rows of A, 16 of B, two loads of 8 rows x 128 B each.  Rows past the
    // matrix and k past the end (K is a multiple of 8) read as zeros.
    constexpr uint32_t OOB = 0x80000000u;
    const rsrc_words rsA = operand_rsrc(A), rsB = operand_rsrc(B);
    const uint32_t lds = (uint32_t)(uintptr_t)LRB_LDS_PTR(smem) + (uint32_t)(wave - 1) * R16_SLICE;
    uint32_t off[4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const int row = (i & 1) * 8 + (lane >> 3);
      const int64_t ld = i < 2 ? op.lda : op.ldb;
      const int lc = (lane & 7) ^ ((row >> 1) & 7);
      off[i] = (i < 2 ? m0 + row < op.M : n0 + row < op.N) ? (uint32_t)(row * (int)ld + lc * 8) * 2u : OOB;
    }
    auto issue = [&](int it, int slot, auto FIRST) {
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const int row = (i & 1) * 8 + (lane >> 3);
        const int k = it * R16_KST + (wave - 1) * BK, lc = (lane & 7) ^ ((row >> 1) & 7);
        dma16<decltype(FIRST)::value>(i < 2 ? rsA : rsB, lds + (uint32_t)slot * R16_STAGE + (uint32_t)i * 1024u,
                                      k + lc * 8 < op.K ? off[i] + (uint32_t)k * 2u : OOB);   // OOB + k stays past the resource
      }
    };
#pragma unroll
    for (int s = 0; s < R16_NS - 1; s++) issue(s, s, std::true_type{});
    int wr = R16_NS - 1;
    for (int it = 0; it < 2 * npair; it++) {
      wait_vmcnt<(R16_NS - 2) * 4>();                    // this wavefront's loads of stage `it` have landed
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      issue(it + R16_NS - 1, wr, std::false_type{});     // into the slot of stage it - 1, whose reads are complete
      wr = wr + 1 == R16_NS ? 0 : wr + 1;
    }
    wait_vmcnt<0>();
    return;
  }

  const int frow = lane & 15, fq = lane >> 4, fsw = (frow >> 1) & 7;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  bf16x8 fa[2][8], fb[2][8];
  int rd = 0;
  auto read = [&](auto Xc) {                             // the operands of the stage in slot rd
    constexpr int x = decltype(Xc)::value;
#pragma unroll
    for (int kk = 0; kk < 8; kk++) {
      const unsigned char* s = smem + rd * R16_STAGE + (kk >> 1) * R16_SLICE + frow * 128 + ((((kk & 1) * 4 + fq) ^ fsw) << 4);
      fa[x][kk] = *reinterpret_cast<const bf16x8*>(s);
      fb[x][kk] = *reinterpret_cast<const bf16x8*>(s + 2048);
    }
    rd = rd + 1 == R16_NS ? 0 : rd + 1;
    __builtin_amdgcn_sched_barrier(0);                   // all of them on their way before the multiplication of the stage before
  };
  auto multiply = [&](auto Xc) {
    constexpr int x = decltype(Xc)::value;
#pragma unroll
    for (int kk = 0; kk < 8; kk++) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[x][kk], fa[x][kk], acc, 0, 0, 0);
  };
  auto turn = [&] {                                      // the stage has landed; this wavefront's reads of the one before are done
    wait_lgkmcnt0();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  using X0 = std::integral_constant<int, 0>;
  using X1 = std::integral_constant<int, 1>;
  for (int p = 0; p < npair; p++) {
    turn();
    read(X0{});
    if (p > 0) multiply(X1{});
    turn();
    read(X1{});
    multiply(X0{});
  }
  multiply(X1{});

  // operands exchanged: lane -> row lane % 16, columns 4 (lane / 16) + 0..3 (N is a multiple of 8: all or none)
  const int m = m0 + frow, n = n0 + 4 * fq;
  if (m >= op.M || n >= op.N) return;
  const Epilogue& e = op.epi;
  float v[4] = {acc[0], acc[1], acc[2], acc[3]}, v2[4], none[4] = {0.f, 0.f, 0.f, 0.f};
  const float rho = e.use_rho ? rho_of(e, e.rowa[m]) : 1.f;
  const bool want2 = KIND == EPI_DOWN && e.C2 != nullptr;
  epi_math<4, KIND, true>(e.act, e.inv_d, want2, v, v2, rho, 0.f, none, none);
  auto put = [&](void* p, int64_t off, const float (&x)[4]) {
    *reinterpret_cast<uint2*>((uint16_t*)p + off) = make_uint2(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]));
  };
  put(op.C, (int64_t)bi * op.sC + (int64_t)bo * op.sCo + (int64_t)m * op.ldc + n, v);
  if (want2) put(e.C2, (int64_t)b * e.sC2 + (int64_t)m * e.ldc2 + n, v2);
}

template <int KIND>
hipError_t launch_rows16(const GemmOp& op, hipStream_t st) {
  auto kern = gemm_rows16_kernel<KIND>;
  // one-time opt-in to more than 64 KB of dynamic LDS (thread-safe function-local static)
  static const hipError_t attr_err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, R16_LDS);
  if (attr_err != hipSuccess) return attr_err;
  const int tiles_m = (op.M + 15) / 16, tiles_n = (op.N + 15) / 16;
  hipLaunchKernelGGL(kern, tile_grid(tiles_m * tiles_n, op.batch), dim3(320), R16_LDS, st, op, tiles_m, tiles_n);
  return hipGetLastError();
}

}  // namespace

// A CU holds one workgroup (two rings would be all of its LDS), so from 257 pieces on there is a second round, which only long
// k makes up for.  One product, replayed from a graph, 16 x 16 pieces / 32 x 32 tiles (us): 256 pieces, k = 64 3.2 / 3.4, 1024
// 3.5 / 4.8, 4096 5.1 / 9.9; 384 and 512 pieces, k = 64 4.7 / 3.5, 1024 5.4 / 4.9, 2048 6.7 / 6.6, 4096 8.7 / 9.9.  With at most 32
// rows two rounds are a weight of 4096 rows or more, where memory decides (8 x 8192 x 4096: 13.2 / 12.3).
bool gemm_rows16_ok(const GemmOp& op) {
  const bool kind = op.epi.kind == EPI_STORE || (op.epi.kind == EPI_DOWN && !op.epi.stat_from_a);
  const int64_t pieces = (int64_t)((op.M + 15) / 16) * ((op.N + 15) / 16) * op.batch;
  return kind && !op.transA && !op.transB && op.splitk == 1 && op.K % 8 == 0 && op.N % 8 == 0 &&
         (pieces <= 256 || (pieces <= 512 && op.K >= 3072 && op.M > 32));
}
hipError_t gemm_rows16(const GemmOp& op, hipStream_t st) {
  return op.epi.kind == EPI_STORE ? launch_rows16<EPI_STORE>(op, st) : launch_rows16<EPI_DOWN>(op, st);
}

}  // namespace lrb
