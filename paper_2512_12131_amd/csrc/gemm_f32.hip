// fp32 reference-precision GEMM: C[M,N] = epi(sum_k A(m,k) B(n,k)) for any operand orientation and
// any sizes.  This is the precision path (max|err|/RMS <= 1e-4 against the fp64 oracle): fp32 operands, fp32
// products and sums (v_mfma_f32_32x32x2_f32).  Split-K and every epilogue kind of the bf16 kernel are available,
// except row partials (callers run k_rowdot / k_rms_stat instead).
//
// Bound: latency.  The path's own sizes (hundreds of rows, ranks of 12 to 128) are a few tiles with short k, so
// the work is spread as thin as it goes: 32 x 32 output tiles, and the NW wavefronts of a workgroup share a
// tile's k, each taking every NW-th run of 32, and add their tiles up through LDS.  Operands go from global
// memory straight into the MFMA registers: a lane holds four consecutive k of one row (or column), and
// the four MFMAs of an 8-wide k group take one of the four each, which pairs the same k in A and B.
// Measured against 64 x 64 tiles through LDS with 16-deep slices and scalar FMAs: 512 x 64 x 256 29.5 -> 6.2 us; a
// layer of 512 tokens, 256 -> 64 -> 256, forward and backward 225 -> 47 us; 4096 tokens, 1024 -> 256 -> 1024
// 624 -> 283 us; 16384 tokens, 2048 -> 512 -> 2048 forward 1288 -> 1328 us (the un-transposed loads touch 32
// rows each), backward 2757 -> 2248 us.
#include "epilogue.h"

namespace lrb {
namespace {

constexpr int TB = 32;          // output tile
constexpr int KRUN = 32;        // k per wavefront and step: four groups of 8, all loads in flight together

// Four consecutive k of row `i` of an operand, zeros outside [0, lim) x [k, kend).  trans: p[k * ld + i].
// vec: p and ld keep the four of an un-transposed row on a 16-byte boundary.
__device__ __forceinline__ float4 load4(const float* p, int64_t ld, bool trans, bool vec, int i, int lim, int k, int kend) {
  float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
  if (i >= lim || k >= kend) return r;
  const int64_t sk = trans ? ld : 1;
  const float* q = p + (trans ? (int64_t)k * ld + i : (int64_t)i * ld + k);
  if (k + 4 <= kend) {
    if (vec) return *reinterpret_cast<const float4*>(q);
    r.x = q[0]; r.y = q[sk]; r.z = q[2 * sk]; r.w = q[3 * sk];
    return r;
  }
  r.x = q[0];
  if (k + 1 < kend) r.y = q[sk];
  if (k + 2 < kend) r.z = q[2 * sk];
  return r;
}

template <int KIND, int NW>
__global__ __launch_bounds__(NW * 64) void gemm_f32_kernel(GemmOp op, int kper, int tiles_n) {
  __shared__ float red[NW][TB * TB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m0 = (int)(blockIdx.x / tiles_n) * TB, n0 = (int)(blockIdx.x % tiles_n) * TB;
  const int bz = blockIdx.y;
  const int b = bz / op.splitk, ks = bz % op.splitk;
  const int kbeg = ks * kper;
  const int kend = min(op.K, kbeg + kper);
  const float* A = (const float*)op.A + (int64_t)b * op.sA;
  const float* B = (const float*)op.B + (int64_t)b * op.sB;
  const bool vecA = !op.transA && op.lda % 4 == 0 && ((uintptr_t)A & 15) == 0;   // kbeg is a multiple of 32
  const bool vecB = !op.transB && op.ldb % 4 == 0 && ((uintptr_t)B & 15) == 0;
  const int row = lane & 31, half = lane >> 5;

  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; v++) acc[v] = 0.f;
  for (int k0 = kbeg + wave * KRUN; k0 < kend; k0 += NW * KRUN) {
    float4 a[KRUN / 8], bb[KRUN / 8];
#pragma unroll
    for (int g = 0; g < KRUN / 8; g++) {
      const int k = k0 + g * 8 + half * 4;
      a[g] = load4(A, op.lda, op.transA != 0, vecA, m0 + row, op.M, k, kend);
      bb[g] = load4(B, op.ldb, op.transB != 0, vecB, n0 + row, op.N, k, kend);
    }
#pragma unroll
    for (int g = 0; g < KRUN / 8; g++) {
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[g].x, bb[g].x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[g].y, bb[g].y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[g].z, bb[g].z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[g].w, bb[g].w, acc, 0, 0, 0);
    }
  }
  // accumulator element v of a lane: row 8 (v / 4) + 4 (lane / 32) + v % 4, column lane % 32
#pragma unroll
  for (int v = 0; v < 16; v++) red[wave][(8 * (v >> 2) + 4 * half + (v & 3)) * TB + row] = acc[v];
  __syncthreads();

  const Epilogue& e = op.epi;
  for (int i = tid; i < TB * TB; i += NW * 64) {
    const int64_t gm = m0 + i / TB, gn = n0 + i % TB;
    if (gm >= op.M || gn >= op.N) continue;
    float v = red[0][i];
#pragma unroll
    for (int w = 1; w < NW; w++) v += red[w][i];
    if constexpr (KIND == EPI_PARTIAL) {
      ((float*)op.C)[((int64_t)bz * op.M + gm) * op.N + gn] = v;
    } else {
      const float rho = e.use_rho ? rho_of(e, e.rowa[gm]) : 1.f;
      const float rowb = e.rowb ? e.rowb[gm] : 0.f;
      epi_apply<float, 1, KIND>(e, op.C, op.ldc, op.sC, b, gm, gn, &v, rho, rowb);
    }
  }
}

long tiles_of(int M, int N, int batch) { return (long)((M + TB - 1) / TB) * ((N + TB - 1) / TB) * batch; }

}  // namespace

// Weight gradients (K = T): a workgroup's wavefronts already share k, so a split, which costs the finishing launch,
// only pays once each of its parts is long and the tiles alone leave most CUs idle.
int gemm_f32_pick_splitk(int M, int N, int K) {
  const long tiles = tiles_of(M, N, 1);
  long s = 1;
  while (s < 32 && tiles * s < 256 && K / (s * 2) >= 2048) s *= 2;
  return (int)s;
}

hipError_t gemm_f32(const GemmOp& op, hipStream_t st) {
  if (op.M <= 0 || op.N <= 0 || op.batch <= 0) return hipSuccess;
  const int tiles_n = (op.N + TB - 1) / TB;
  const dim3 grid((unsigned)tiles_of(op.M, op.N, 1), op.batch * op.splitk);
  int kper = (op.K + op.splitk - 1) / op.splitk;
  kper = (kper + KRUN - 1) / KRUN * KRUN;
  // 16 wavefronts per tile where they all get a run of k and the tiles do not fill the chip by themselves
  const bool wide = kper > 4 * KRUN && tiles_of(op.M, op.N, op.batch * op.splitk) <= 512;
  const int kind = op.splitk > 1 ? (int)EPI_PARTIAL : op.epi.kind;
  switch (kind) {
#define CASE(KD)                                                                             \
  case KD:                                                                                   \
    if (wide) hipLaunchKernelGGL((gemm_f32_kernel<KD, 16>), grid, dim3(1024), 0, st, op, kper, tiles_n); \
    else hipLaunchKernelGGL((gemm_f32_kernel<KD, 4>), grid, dim3(256), 0, st, op, kper, tiles_n);     \
    break;
    CASE(EPI_STORE)
    CASE(EPI_DOWN)
    CASE(EPI_UP)
    CASE(EPI_ACTGRAD)
    CASE(EPI_NORMBWD)
    CASE(EPI_PARTIAL)
    CASE(EPI_SWIGLU_BWD)
    CASE(EPI_SWIGLU_FWD)
    CASE(EPI_DOWN_LAX)
    CASE(EPI_LAXGRAD)
#undef CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace lrb
