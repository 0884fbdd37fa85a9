// fp32 reference-precision GEMM: C[M,N] = epi(sum_k A(m,k) B(n,k)) for any operand orientation and
// any sizes.  This is the precision path (max|err|/RMS <= 1e-4 against the fp64 oracle): fp32 operands, fp32
// products and sums (v_mfma_f32_32x32x2_f32).  Split-K and every epilogue kind of the bf16 kernel are available,
// except row partials (callers run k_rowdot / k_rms_stat instead).
//
// One order of summation, whatever the number of rows: k is cut into ranges (k_range()), the products of a range are added by
// the matrix instruction front to back, and the ranges' sums front to back after that.  Two kernels keep to it, so
// neither the choice between them nor how many tokens share a call shows in a row's bits.
//
// Small products are bound by latency: hundreds of rows and ranks of 12 to 128 are a few tiles with short k, so
// the work is spread as thin as it goes: 32 x 32 output tiles, and the wavefronts of a workgroup share a
// tile's k, a range each, and add their tiles up through LDS.  Operands go from global
// memory straight into the MFMA registers: a lane holds four consecutive k of one row (or column), and
// the four MFMAs of an 8-wide k group take one of the four each, which pairs the same k in A and B.
// Measured against 64 x 64 tiles through LDS with 16-deep slices and scalar FMAs: 512 x 64 x 256 29.5 -> 6.2 us; a
// layer of 512 tokens, 256 -> 64 -> 256, forward and backward 225 -> 47 us.
//
// Products that fill the chip are bound by the loads of that form (every 32 x 32 tile reads its own operands, 32 rows per
// instruction); there 64 x 64 tiles bring k through LDS.  16384 tokens, 2048 -> 512 -> 2048, forward 1330 us on the small
// form and 1259 on scalar FMAs -> 1060, backward 2266 and 2748 -> 2154.
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

// The k ranges of a sum over kper elements: at most 16 of whole runs.
__host__ __device__ constexpr int k_range(int kper) { return kper <= 4 * KRUN ? KRUN : ((kper + KRUN - 1) / KRUN + 15) / 16 * KRUN; }

__device__ __forceinline__ f32x16 mfma4(const float4& a, const float4& b, f32x16 acc) {
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b.x, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b.y, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, b.z, acc, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, b.w, acc, 0, 0, 0);
}

// accumulator element v of a lane: row 8 (v / 4) + 4 (lane / 32) + v % 4, column lane % 32 of a 32 x 32 block
__device__ __forceinline__ int acc_row(int v, int half) { return 8 * (v >> 2) + 4 * half + (v & 3); }

template <int KIND>
__device__ __forceinline__ void store_one(const GemmOp& op, int b, int bz, int64_t gm, int64_t gn, float v) {
  if (gm >= op.M || gn >= op.N) return;
  const Epilogue& e = op.epi;
  if constexpr (KIND == EPI_PARTIAL) {
    ((float*)op.C)[((int64_t)bz * op.M + gm) * op.N + gn] = v;
  } else {
    const float rho = e.use_rho ? rho_of(e, e.rowa[gm]) : 1.f;
    const float rowb = e.rowb ? e.rowb[gm] : 0.f;
    epi_apply<float, 1, KIND>(e, op.C, op.ldc, op.sC, b, gm, gn, &v, rho, rowb);
  }
}

// NW wavefronts per 32 x 32 tile, wavefront w sums range w (NW = 4: kper <= 128)
// bx, bz: output tile, batch member times k split
template <int KIND, int NW>
__device__ __forceinline__ void product_f32(const GemmOp& op, int kper, int tiles_n, int bx, int bz, float (&red)[NW][TB * TB]) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m0 = (bx / tiles_n) * TB, n0 = (bx % tiles_n) * TB;
  const int b = bz / op.splitk, ks = bz % op.splitk;
  const int kbeg = ks * kper, range = k_range(kper);
  const int kend = min(min(op.K, kbeg + kper), kbeg + (wave + 1) * range);
  const float* A = (const float*)op.A + (int64_t)b * op.sA;
  const float* B = (const float*)op.B + (int64_t)b * op.sB;
  const bool vecA = !op.transA && op.lda % 4 == 0 && ((uintptr_t)A & 15) == 0;   // kbeg is a multiple of 32
  const bool vecB = !op.transB && op.ldb % 4 == 0 && ((uintptr_t)B & 15) == 0;
  const int row = lane & 31, half = lane >> 5;

  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; v++) acc[v] = 0.f;
  for (int k0 = kbeg + wave * range; k0 < kend; k0 += KRUN) {
    float4 a[KRUN / 8], bb[KRUN / 8];
#pragma unroll
    for (int g = 0; g < KRUN / 8; g++) {
      const int k = k0 + g * 8 + half * 4;
      a[g] = load4(A, op.lda, op.transA != 0, vecA, m0 + row, op.M, k, kend);
      bb[g] = load4(B, op.ldb, op.transB != 0, vecB, n0 + row, op.N, k, kend);
    }
#pragma unroll
    for (int g = 0; g < KRUN / 8; g++) acc = mfma4(a[g], bb[g], acc);
  }
#pragma unroll
  for (int v = 0; v < 16; v++) red[wave][acc_row(v, half) * TB + row] = acc[v];
  __syncthreads();

  for (int i = tid; i < TB * TB; i += NW * 64) {
    float v = red[0][i];
#pragma unroll
    for (int w = 1; w < NW; w++) v += red[w][i];
    store_one<KIND>(op, b, bz, m0 + i / TB, n0 + i % TB, v);
  }
}

template <int KIND, int NW>
__global__ __launch_bounds__(NW * 64) void gemm_f32_kernel(GemmOp op, int kper, int tiles_n) {
  __shared__ float red[NW][TB * TB];
  product_f32<KIND, NW>(op, kper, tiles_n, blockIdx.x, blockIdx.y, red);
}

// Independent products in one launch: workgroups [first, first + count) take one.  A wavefront without a range of its own (short k)
// adds zeros, which changes no bit: a range's sum starts from +0 and is never -0.  512 tokens, 256 -> 64 -> 256, forward and
// backward in four launches instead of seven: 44.8 -> 38.8 us, of which the host's calls are most.
struct JointF32 {
  GemmOp op[JOINT_MAX];
  int first[JOINT_MAX + 1];
};
__global__ __launch_bounds__(1024) void gemm_f32_joint_kernel(JointF32) {
  const JointF32& a = *(const JointF32*)__builtin_amdgcn_kernarg_segment_ptr();   // (no copy of an array indexed at run time)
  __shared__ float red[16][TB * TB];
  int i = 0;
#pragma unroll
  for (int j = 1; j < JOINT_MAX; j++) i += (int)blockIdx.x >= a.first[j] ? 1 : 0;
  i = __builtin_amdgcn_readfirstlane(i);
  const GemmOp& op = a.op[i];
  const int tiles_n = (op.N + TB - 1) / TB, kper = (op.K + KRUN - 1) / KRUN * KRUN, bid = (int)blockIdx.x - a.first[i];
  if (op.epi.kind == EPI_PARTIAL) product_f32<EPI_PARTIAL, 16>(op, kper, tiles_n, bid, 0, red);
  else product_f32<EPI_STORE, 16>(op, kper, tiles_n, bid, 0, red);
}

// 64 x 64 tiles of 2 x 2 wavefronts; runs of 32 k go through LDS, a row's k consecutive (row stride 36: the 16 rows of a
// quarter wavefront's 16-byte reads fall on different banks), the next run's loads in registers meanwhile.
// A wavefront holds the sum of the running range and that of the ranges before it.  (128 x 128 tiles, 272 registers:
// 16384 x 512 x 2048 660 against 581 us.)
template <int KIND>
__global__ __launch_bounds__(256) void gemm_f32_tile_kernel(GemmOp op, int kper, int tiles_n) {
  constexpr int BT = 64, LS = KRUN + 4, NL = BT * KRUN / 4 / 256;   // tile side, LDS row stride, 16-byte loads per thread
  __shared__ __attribute__((aligned(16))) float sa[BT * LS], sb[BT * LS];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1;
  const int m0 = (int)(blockIdx.x / tiles_n) * BT, n0 = (int)(blockIdx.x % tiles_n) * BT;
  const int bz = blockIdx.y;
  const int b = bz / op.splitk, ks = bz % op.splitk;
  const int kbeg = ks * kper, range = k_range(kper);
  const int kend = min(op.K, kbeg + kper);
  const float* A = (const float*)op.A + (int64_t)b * op.sA;
  const float* B = (const float*)op.B + (int64_t)b * op.sB;
  const bool vecA = op.lda % 4 == 0 && ((uintptr_t)A & 15) == 0;   // kbeg, m0 and n0 are multiples of 4
  const bool vecB = op.ldb % 4 == 0 && ((uintptr_t)B & 15) == 0;
  const bool tA = op.transA != 0, tB = op.transB != 0;
  const int row = lane & 31, half = lane >> 5;

  // load j of a thread: four k of one row of the operand, or (trans) four of its rows at one k
  auto fetch = [&](const float* p, int64_t ld, bool trans, bool vec, int i0, int lim, int k0, float4 (&r)[NL]) {
#pragma unroll
    for (int j = 0; j < NL; j++) {
      const int idx = tid + 256 * j;
      r[j] = trans ? load4(p, ld, false, vec, k0 + idx / (BT / 4), kend, i0 + idx % (BT / 4) * 4, lim)
                   : load4(p, ld, false, vec, i0 + idx / (KRUN / 4), lim, k0 + idx % (KRUN / 4) * 4, kend);
    }
  };
  auto put = [&](float* s, bool trans, const float4 (&r)[NL]) {
#pragma unroll
    for (int j = 0; j < NL; j++) {
      const int idx = tid + 256 * j;
      if (trans) {
        float* q = s + idx % (BT / 4) * 4 * LS + idx / (BT / 4);
        q[0] = r[j].x; q[LS] = r[j].y; q[2 * LS] = r[j].z; q[3 * LS] = r[j].w;
      } else {
        *reinterpret_cast<float4*>(s + idx / (KRUN / 4) * LS + idx % (KRUN / 4) * 4) = r[j];
      }
    }
  };
  f32x16 acc, tot;
#pragma unroll
  for (int v = 0; v < 16; v++) acc[v] = tot[v] = 0.f;
  float4 ra[NL], rb[NL];
  fetch(A, op.lda, tA, vecA, m0, op.M, kbeg, ra);
  fetch(B, op.ldb, tB, vecB, n0, op.N, kbeg, rb);
  int range_end = kbeg + range;
  for (int k0 = kbeg; k0 < kend; k0 += KRUN) {
    if (k0 == range_end) {
      range_end += range;
#pragma unroll
      for (int v = 0; v < 16; v++) {
        tot[v] += acc[v];
        acc[v] = 0.f;
      }
    }
    __syncthreads();       // everyone has read the run before
    put(sa, tA, ra);
    put(sb, tB, rb);
    __syncthreads();
    fetch(A, op.lda, tA, vecA, m0, op.M, k0 + KRUN, ra);   // (past the end: zeros, not loaded)
    fetch(B, op.ldb, tB, vecB, n0, op.N, k0 + KRUN, rb);
#pragma unroll
    for (int g = 0; g < KRUN / 8; g++)
      acc = mfma4(*reinterpret_cast<const float4*>(sa + (wm * 32 + row) * LS + g * 8 + half * 4),
                  *reinterpret_cast<const float4*>(sb + (wn * 32 + row) * LS + g * 8 + half * 4), acc);
  }
#pragma unroll
  for (int v = 0; v < 16; v++) store_one<KIND>(op, b, bz, m0 + wm * 32 + acc_row(v, half), n0 + wn * 32 + row, tot[v] + acc[v]);
}

long tiles_of(int M, int N, int side) { return (long)((M + side - 1) / side) * ((N + side - 1) / side); }

template <int KIND>
hipError_t run(const GemmOp& op, int kper, int side, hipStream_t st) {
  const int tiles_n = (op.N + side - 1) / side;
  const dim3 grid((unsigned)tiles_of(op.M, op.N, side), op.batch * op.splitk);
  if (side == 64) hipLaunchKernelGGL(gemm_f32_tile_kernel<KIND>, grid, dim3(256), 0, st, op, kper, tiles_n);
  else if (kper > 4 * KRUN) hipLaunchKernelGGL((gemm_f32_kernel<KIND, 16>), grid, dim3(1024), 0, st, op, kper, tiles_n);
  else hipLaunchKernelGGL((gemm_f32_kernel<KIND, 4>), grid, dim3(256), 0, st, op, kper, tiles_n);
  return hipGetLastError();
}

}  // namespace

// Weight gradients (K = T): a workgroup's wavefronts already share k, so a split, which costs the finishing launch,
// only pays once each of its parts is long and the tiles alone leave most CUs idle.
int gemm_f32_pick_splitk(int M, int N, int K) {
  const long tiles = tiles_of(M, N, TB);
  long s = 1;
  while (s < 32 && tiles * s < 256 && K / (s * 2) >= 2048) s *= 2;
  return (int)s;
}

hipError_t gemm_f32(const GemmOp& op, hipStream_t st) {
  if (op.M <= 0 || op.N <= 0 || op.batch <= 0) return hipSuccess;
  int kper = (op.K + op.splitk - 1) / op.splitk;
  kper = (kper + KRUN - 1) / KRUN * KRUN;
  // 64 x 64 tiles from two per CU on (both ways, us): 4096 x 512 x 2048, 512 of them, 165 / 143 (k-major B) and 185 / 183;
  // 16384 x 512 x 2048 724 / 581; 2048 x 512 x 2048, 256 of them, 94 / 140
  const int side = tiles_of(op.M, op.N, 64) * op.batch * op.splitk >= 512 ? 64 : TB;
  switch (op.splitk > 1 ? (int)EPI_PARTIAL : op.epi.kind) {
#define CASE(KD) case KD: return run<KD>(op, kper, side, st);
    CASE(EPI_STORE)
    CASE(EPI_DOWN)
    CASE(EPI_UP)
    CASE(EPI_ACTGRAD)
    CASE(EPI_ACTGRAD_A)
    CASE(EPI_NORMBWD)
    CASE(EPI_PARTIAL)
    CASE(EPI_SWIGLU_BWD)
    CASE(EPI_SWIGLU_FWD)
    CASE(EPI_DOWN_LAX)
    CASE(EPI_LAXGRAD)
#undef CASE
    default: return hipErrorInvalidValue;
  }
}

hipError_t gemm_f32_many(const GemmOp* ops, int n, hipStream_t st) {
  // Together where all their 32 x 32 tiles find a place at once (two workgroups of 16 wavefronts per CU): what such products
  // cost is the launch.
  bool ok = n > 1 && n <= JOINT_MAX;
  long wgs = 0;
  JointF32 a;
  for (int i = 0; ok && i < n; i++) {
    const GemmOp& op = ops[i];
    ok = op.splitk == 1 && op.batch == 1 && (op.epi.kind == EPI_PARTIAL || op.epi.kind == EPI_STORE) && op.M > 0 && op.N > 0 &&
         tiles_of(op.M, op.N, 64) < 512;
    a.op[i] = op;
    a.first[i] = (int)wgs;
    if (ok) wgs += tiles_of(op.M, op.N, TB);
  }
  if (ok && wgs <= 512) {
    for (int i = n; i <= JOINT_MAX; i++) a.first[i] = (int)wgs;
    hipLaunchKernelGGL(gemm_f32_joint_kernel, dim3((unsigned)wgs), dim3(1024), 0, st, a);
    return hipGetLastError();
  }
  for (int i = 0; i < n; i++) {
    const hipError_t e = gemm_f32(ops[i], st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace lrb
