// Memory-bound kernels: per-token statistics, RMSNorm apply / backward, sigma at rank r, SwiGLU
// forward / backward, transposes and the small reductions that finish weight gradients.
// bf16 tensors move as 16-byte vectors (8 elements per lane, 1 KB per wavefront instruction);
// fp32 tensors (precision path, arbitrary sizes) move element-wise.  All arithmetic is fp32.
// The forms the block uses (dense bf16 tensors, rows of at most 4096 elements) reach memory through
// buffer resources sized to what a workgroup or a row owns, so that they need no bounds branches: with
// a test per vector the compiler puts a full memory wait inside every branch and a lane's loads go one
// round trip after the other.  Also here: the rotary embedding and the LaX variant's rank-r sum.
#include "epilogue.h"

namespace lrb {
namespace {

template <int DT> struct St;
template <> struct St<LR_F32> { using T = float; static constexpr int NV = 1; };
template <> struct St<LR_BF16> { using T = bf16_t; static constexpr int NV = 8; };

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// ---- S[t] = sum_j x[t,j]^2 : one wavefront per row ---------------------------------------------
// (Many short wavefronts read faster here than fewer wavefronts with more rows or vectors each.)
template <int DT>
__device__ __forceinline__ void rms_stat_rows(int block, const void* x, int64_t ldx, float* stat, int64_t T, int64_t d) {
  using S = St<DT>;
  using IO = VecIO<typename S::T, S::NV>;
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)block * 4 + (threadIdx.x >> 6);
  if (row >= T) return;
  float s = 0.f;
  // four vectors per lane in flight before the arithmetic
  constexpr int U = 4;
  for (int64_t c0 = 0; c0 < d; c0 += U * 64 * S::NV) {
    float v[U][S::NV];
#pragma unroll
    for (int j = 0; j < U; j++) {
      const int64_t c = c0 + (j * 64 + lane) * S::NV;
      if (c < d) IO::load_nt(x, row * ldx + c, v[j]);
    }
#pragma unroll
    for (int j = 0; j < U; j++) {
      const int64_t c = c0 + (j * 64 + lane) * S::NV;
      if (c < d) {
#pragma unroll
        for (int i = 0; i < S::NV; i++) s = fmaf(v[j][i], v[j][i], s);
      }
    }
  }
  s = wave_sum(s);
  if (lane == 0) stat[row] = s;
}
template <int DT>
__global__ __launch_bounds__(256) void rms_stat_kernel(const void* x, int64_t ldx, float* stat, int64_t T, int64_t d) {
  rms_stat_rows<DT>((int)blockIdx.x, x, ldx, stat, T, d);
}

// Columns scaled by gamma, of one or two matrices of equal width (rows1 = 0: one): a block folds both of its norms' gammas in one
// launch.  Workgroup `block` of `blocks`.
template <int DT>
__device__ __forceinline__ void scale_cols_part(const ScaleCols& p, int block, int blocks) {
  using S = St<DT>;
  using IO = VecIO<typename S::T, S::NV>;
  const int64_t cpr = p.cols / S::NV, total0 = p.rows0 * cpr, total = total0 + p.rows1 * cpr;
  for (int64_t j = (int64_t)block * 256 + threadIdx.x; j < total; j += (int64_t)blocks * 256) {
    const bool second = j >= total0;
    const int64_t i = second ? j - total0 : j;
    const int64_t c = (i % cpr) * S::NV, off = (i / cpr) * p.cols + c;
    float wv[S::NV], gv[S::NV];
    IO::load(second ? p.w1 : p.w0, off, wv);
    IO::load(second ? p.gamma1 : p.gamma0, c, gv);
#pragma unroll
    for (int k = 0; k < S::NV; k++) wv[k] *= gv[k];
    IO::store(second ? p.out1 : p.out0, off, wv);
  }
}
template <int DT>
__global__ __launch_bounds__(256) void scale_cols_kernel(ScaleCols p) {
  scale_cols_part<DT>(p, (int)blockIdx.x, (int)gridDim.x);
}
// A normed group folds its gamma and takes the rows' statistic: neither waits for the other (777 rows of 4096 beside 5120 x 4096
// weights 14.5 + 6.3 -> 15.4 us, 16384 rows of 2048 beside 1536 x 2048 5.7 + 12.0 -> 14.6, and one way in and out less).
template <int DT>
__global__ __launch_bounds__(256) void scale_cols_rms_stat_kernel(ScaleCols p, int stat_blocks, const void* x, int64_t ldx, float* stat,
                                                                  int64_t T, int64_t d) {
  if ((int)blockIdx.x < stat_blocks) rms_stat_rows<DT>((int)blockIdx.x, x, ldx, stat, T, d);
  else scale_cols_part<DT>(p, (int)blockIdx.x - stat_blocks, (int)gridDim.x - stat_blocks);
}

template <int DT>
__global__ __launch_bounds__(256) void rmsnorm_apply_kernel(const void* x, int64_t ldx, const void* gamma,
                                                            const float* stat, float eps, void* out, int64_t ldo,
                                                            int64_t T, int64_t d, int64_t d_div) {
  // d: row width; d_div: the width the statistic was taken over (differs from d when the rows are the
  // summed partial products of a feature-sharded projection); gamma may be null (no scale)
  using S = St<DT>;
  using IO = VecIO<typename S::T, S::NV>;
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= T) return;
  const float rho = rsqrtf(stat[row] / (float)d_div + eps);
  for (int64_t c = lane * S::NV; c < d; c += 64 * S::NV) {
    float v[S::NV], g[S::NV];
    IO::load(x, row * ldx + c, v);
#pragma unroll
    for (int i = 0; i < S::NV; i++) g[i] = 1.f;
    if (gamma) IO::load(gamma, c, g);
#pragma unroll
    for (int i = 0; i < S::NV; i++) v[i] = v[i] * g[i] * rho;
    IO::store(out, row * ldo + c, v);
  }
}

// ---- reverse mode of RMSNorm ----------------------------------------------------------------------
// One workgroup owns RB consecutive rows.  Phase A: each wavefront reduces c = mean_j(dn*n) for its
// rows.  Phase B: column super-chunks of 64*NV*IT columns; each lane keeps the column partial sums
// of dxhat*n for its columns across the workgroup's rows, writes dx, and the four wavefronts'
// partials are added through LDS into dgamma_part[blockIdx][.].
constexpr int NB_RB = 64;
constexpr int NB_IT = 4;

template <int DT>
__global__ __launch_bounds__(256) void rmsnorm_bwd_kernel(const void* x, int64_t ldx, const void* gamma,
                                                          const float* stat, float eps, const void* dxh,
                                                          int64_t lddxh, const void* dres, int64_t lddres, void* dx,
                                                          int64_t lddx, float* dgpart, int64_t T, int64_t d) {
  using S = St<DT>;
  using IO = VecIO<typename S::T, S::NV>;
  constexpr int NV = S::NV;
  __shared__ float sc[NB_RB];
  __shared__ float sred[4][64 * NV];  // one it-slice of a super-chunk at a time
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t row0 = (int64_t)blockIdx.x * NB_RB;
  const float inv_d = 1.f / (float)d;
  for (int r = wave; r < NB_RB; r += 4) {
    const int64_t row = row0 + r;
    if (row >= T) break;
    const float rho = rsqrtf(stat[row] * inv_d + eps);
    float s = 0.f;
    for (int64_t c = lane * NV; c < d; c += 64 * NV) {
      float xv[NV], gv[NV], dv[NV];
      IO::load(x, row * ldx + c, xv);
      IO::load(gamma, c, gv);
      IO::load(dxh, row * lddxh + c, dv);
#pragma unroll
      for (int i = 0; i < NV; i++) s = fmaf(dv[i] * gv[i], xv[i] * rho, s);
    }
    s = wave_sum(s);
    if (lane == 0) sc[r] = s * inv_d;
  }
  __syncthreads();
  constexpr int SUPER = 64 * NV * NB_IT;
  for (int64_t cb = 0; cb < d; cb += SUPER) {
    float acc[NB_IT][NV];
#pragma unroll
    for (int it = 0; it < NB_IT; it++)
#pragma unroll
      for (int i = 0; i < NV; i++) acc[it][i] = 0.f;
    for (int r = wave; r < NB_RB; r += 4) {
      const int64_t row = row0 + r;
      if (row >= T) break;
      const float rho = rsqrtf(stat[row] * inv_d + eps);
      const float c = sc[r];
#pragma unroll
      for (int it = 0; it < NB_IT; it++) {
        const int64_t col = cb + (int64_t)it * 64 * NV + lane * NV;
        if (col < d) {
          float xv[NV], gv[NV], dv[NV], o[NV];
          IO::load(x, row * ldx + col, xv);
          IO::load(gamma, col, gv);
          IO::load(dxh, row * lddxh + col, dv);
#pragma unroll
          for (int i = 0; i < NV; i++) {
            const float n = xv[i] * rho;
            o[i] = (dv[i] * gv[i] - n * c) * rho;
            acc[it][i] = fmaf(dv[i], n, acc[it][i]);
          }
          if (dres) {
            float rv[NV];
            IO::load(dres, row * lddres + col, rv);
#pragma unroll
            for (int i = 0; i < NV; i++) o[i] += rv[i];
          }
          IO::store(dx, row * lddx + col, o);
        }
      }
    }
    // add the four wavefronts' column partials, one it-slice at a time
#pragma unroll
    for (int it = 0; it < NB_IT; it++) {
#pragma unroll
      for (int i = 0; i < NV; i++) sred[wave][lane * NV + i] = acc[it][i];
      __syncthreads();
      for (int e = threadIdx.x; e < 64 * NV; e += 256) {
        const int64_t col = cb + (int64_t)it * 64 * NV + e;
        if (col < d) dgpart[(int64_t)blockIdx.x * d + col] = sred[0][e] + sred[1][e] + sred[2][e] + sred[3][e];
      }
      __syncthreads();
    }
  }
}

// bf16, d <= 512 * NIT: a wavefront holds a whole row of x, dxhat and the residual gradient in
// registers (packed, as loaded), so every tensor is read exactly once: reduce c, then write dx and add
// the row into the lane's column partials of dgamma.  Same partial layout as the kernel above; the rows
// of a workgroup are interleaved with those of the others, so that the workgroups in flight together
// sweep one contiguous window of each tensor.
// All global accesses of the row loop go through buffer resources that span exactly one row (and
// nothing, for an absent residual): columns past d read as zeros and are dropped on store without a
// branch, so the loop body is straight-line code and all of a row's loads are in flight together.  (With a
// bounds test per vector the compiler had put a full wait for memory between the vectors of the
// second phase: 4.5 instead of the rate below.)
// What bounds it below one workgroup per CU and on narrow rows is a wavefront's way from one row to the next: 16 rows in a
// chain, each a wait for memory, then some 20 instructions per column slot.  So NIT follows the width (one kernel of eight
// slices for every width spent 3 us per row, also on 256 columns), and AHEAD keeps the next row on its way in a second set
// of registers.  Measured, launch and sum of the partials included, before and after: 49.6 -> 16.2 us (8192 x 512),
// 101.5 -> 45.7 us (32768 x 1024), 59.7 -> 43.9 us (16384 x 2048: 6.1 TB/s), 58.5 -> 43.9 us (8192 x 3072), 61.2 ->
// 56.6 us (8192 x 4096).  A row that is not there is left out, not worked on as zeros (one row of 2176 columns 7.2 -> 5.4 us).
template <int NIT, bool AHEAD>
__global__ __launch_bounds__(256, AHEAD ? 1 : 2) void rmsnorm_bwd_row_kernel(
    const uint16_t* x, int64_t ldx, const uint16_t* gamma, const float* stat, float eps, const uint16_t* dxh, int64_t lddxh,
    const uint16_t* dres, int64_t lddres, uint16_t* dx, int64_t lddx, float* dgpart, int64_t T, int64_t d, int rows_per_wg,
    int64_t nparts) {
  // LDS: gamma (staged once per workgroup: re-reading it here costs no registers and, unlike a global
  // re-read, does not queue behind the row's stores), then each wavefront's column partials of dgamma
  // (kept here rather than in 64 registers per lane, which the row data needs)
  extern __shared__ __align__(16) unsigned char rn_smem[];
  uint4* sgam = reinterpret_cast<uint4*>(rn_smem);                           // [NIT * 64]
  float4* sacc = reinterpret_cast<float4*>(rn_smem + NIT * 64 * 16);          // [4][NIT * 64][2]
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const float inv_d = 1.f / (float)d;
  const uint32_t row_bytes = (uint32_t)d * 2u;
  // cache policy of the streamed tensors: non-temporal loads; the stores with the default policy (measured:
  // 5.8 against 5.6 TB/s with non-temporal stores, and the reverse for the loads)
  constexpr int NT_ = 2, ST_ = 0;
  auto row_rsrc = [&](const uint16_t* base, int64_t row, int64_t ld) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)(base ? base + row * ld : nullptr), 0, base ? row_bytes : 0u,
                                             0x00020000);
  };
  for (int e = threadIdx.x; e < NIT * 64; e += 256)
    sgam[e] = (int64_t)e * 8 < d ? *reinterpret_cast<const uint4*>(gamma + (int64_t)e * 8) : make_uint4(0, 0, 0, 0);
  float4* myacc = sacc + (wave * NIT * 64 + lane) * 2;      // + it * 128: this lane's 8 columns of slice it
#pragma unroll
  for (int it = 0; it < NIT; it++) {
    myacc[it * 128] = make_float4(0.f, 0.f, 0.f, 0.f);
    myacc[it * 128 + 1] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  __syncthreads();
  auto u4 = [](const u32x4_t& t) { return make_uint4(t.x, t.y, t.z, t.w); };
  // A row past the last one, asked for ahead, has empty resources; nobody works on it.
  struct Row { u32x4_t x[NIT], d[NIT], r[NIT]; float ss; };
  auto row_at = [&](int r) { return ((int64_t)r * gridDim.x + blockIdx.x) * 4 + wave; };
  auto fetch = [&](int r, Row& q) {
    const int64_t row = row_at(r);
    const bool there = r < rows_per_wg / 4 && row < T;
    const __amdgpu_buffer_rsrc_t rsX = row_rsrc(there ? x : nullptr, row, ldx),
                                 rsD = row_rsrc(there ? dxh : nullptr, row, lddxh),
                                 rsR = row_rsrc(there ? dres : nullptr, row, lddres);
    q.ss = there ? stat[row] : 1.f;
#pragma unroll
    for (int it = 0; it < NIT; it++) {
      const int off = (it * 64 + lane) * 16;
      q.x[it] = __builtin_amdgcn_raw_buffer_load_b128(rsX, off, 0, NT_);
      q.d[it] = __builtin_amdgcn_raw_buffer_load_b128(rsD, off, 0, NT_);
    }
#pragma unroll
    for (int it = 0; it < NIT; it++) q.r[it] = __builtin_amdgcn_raw_buffer_load_b128(rsR, (it * 64 + lane) * 16, 0, NT_);
  };
  auto work = [&](int r, const Row& q) {
    const int64_t row = row_at(r);
    const __amdgpu_buffer_rsrc_t rsO = row_rsrc(row < T ? dx : nullptr, row, lddx);
    const float rho = rsqrtf(q.ss * inv_d + eps);
    float s = 0.f;
#pragma unroll
    for (int it = 0; it < NIT; it++) {
      float xv[8], gv[8], dv[8];
      unpack8(u4(q.x[it]), xv); unpack8(sgam[it * 64 + lane], gv); unpack8(u4(q.d[it]), dv);
#pragma unroll
      for (int i = 0; i < 8; i++) s = fmaf(dv[i] * gv[i], xv[i] * rho, s);
      // keeps the compiler from fetching and unpacking every slice's gamma at once (registers)
      if (it % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    }
    const float c = wave_sum(s) * inv_d;
#pragma unroll
    for (int it = 0; it < NIT; it++) {
      float xv[8], gv[8], dv[8], rv[8], o[8];
      if (it % 2 == 0) __builtin_amdgcn_sched_barrier(0);
      unpack8(u4(q.x[it]), xv); unpack8(sgam[it * 64 + lane], gv); unpack8(u4(q.d[it]), dv); unpack8(u4(q.r[it]), rv);
      float4 a0 = myacc[it * 128], a1 = myacc[it * 128 + 1];
      float a[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
#pragma unroll
      for (int i = 0; i < 8; i++) {
        const float n = xv[i] * rho;
        o[i] = (dv[i] * gv[i] - n * c) * rho + rv[i];
        a[i] = fmaf(dv[i], n, a[i]);
      }
      myacc[it * 128] = make_float4(a[0], a[1], a[2], a[3]);
      myacc[it * 128 + 1] = make_float4(a[4], a[5], a[6], a[7]);
      const uint4 ov = pack8(o);
      __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{ov.x, ov.y, ov.z, ov.w}, rsO, (it * 64 + lane) * 16, 0, ST_);
    }
  };
  Row qa, qb;
  if constexpr (AHEAD) {
    fetch(0, qa);
    for (int r = 0; r < rows_per_wg / 4; r += 2) {           // (an even number: rows_per_wg is a multiple of NB_RB)
      if (row_at(r) >= T) break;
      fetch(r + 1, qb);
      __builtin_amdgcn_sched_barrier(0);
      work(r, qa);
      if (row_at(r + 1) >= T) break;
      fetch(r + 2, qa);
      __builtin_amdgcn_sched_barrier(0);
      work(r + 1, qb);
    }
  } else {
    for (int r = 0; r < rows_per_wg / 4; r++) {
      if (row_at(r) >= T) break;
      fetch(r, qa);
      work(r, qa);
    }
  }
  // add the four wavefronts' column partials
  __syncthreads();
  const float* fa = reinterpret_cast<const float*>(sacc);
  for (int e = threadIdx.x; e < NIT * 512; e += 256) {
    if (e < d) {
      dgpart[(int64_t)blockIdx.x * d + e] = fa[e] + fa[NIT * 512 + e] + fa[2 * NIT * 512 + e] + fa[3 * NIT * 512 + e];
      // the caller adds up nparts rows of partials: those that no workgroup owns hold zeros
      for (int64_t pr = (int64_t)blockIdx.x + gridDim.x; pr < nparts; pr += gridDim.x) dgpart[pr * d + e] = 0.f;
    }
  }
}
constexpr int rn_row_lds(int nit) { return nit * 64 * 16 + 4 * nit * 512 * 4; }   // gamma + four sets of partials

// ---- elementwise on [T, n] with leading dimensions -------------------------------------------
// Each workgroup owns one contiguous run of EW_U x 256 vectors and issues all of its loads before the
// arithmetic; loads and stores are non-temporal.  (Measured on this chip: 6.3 TB/s for a two-input,
// one-output kernel, against 5.2 TB/s for a grid-stride loop with one vector in flight per lane.)
constexpr int EW_U = 4;
template <int DT>
__global__ __launch_bounds__(256) void act_fwd_kernel(const void* z, int64_t ldz, void* a, int64_t lda, int64_t T,
                                                      int64_t n, int act) {
  using S = St<DT>;
  using IO = VecIO<typename S::T, S::NV>;
  const int64_t cpr = n / S::NV;  // vectors per row
  const int64_t total = T * cpr;
  const int64_t base = (int64_t)blockIdx.x * (256 * EW_U) + threadIdx.x;
  float v[EW_U][S::NV];
#pragma unroll
  for (int j = 0; j < EW_U; j++) {
    const int64_t i = base + j * 256;
    if (i < total) IO::load_nt(z, (i / cpr) * ldz + (i % cpr) * S::NV, v[j]);
  }
#pragma unroll
  for (int j = 0; j < EW_U; j++) {
    const int64_t i = base + j * 256;
    if (i < total) {
#pragma unroll
      for (int k = 0; k < S::NV; k++) v[j][k] = act_f(v[j][k], act);
      IO::store_nt(a, (i / cpr) * lda + (i % cpr) * S::NV, v[j]);
    }
  }
}

template <int DT>
__global__ __launch_bounds__(256) void swiglu_fwd_kernel(const void* g, const void* u, void* m, int64_t ld, int64_t T,
                                                         int64_t f) {
  using S = St<DT>;
  using IO = VecIO<typename S::T, S::NV>;
  const int64_t cpr = f / S::NV, total = T * cpr;
  const int64_t base = (int64_t)blockIdx.x * (256 * EW_U) + threadIdx.x;
  float gv[EW_U][S::NV], uv[EW_U][S::NV];
#pragma unroll
  for (int j = 0; j < EW_U; j++) {
    const int64_t i = base + j * 256;
    if (i < total) {
      const int64_t off = (i / cpr) * ld + (i % cpr) * S::NV;
      IO::load_nt(g, off, gv[j]);
      IO::load_nt(u, off, uv[j]);
    }
  }
#pragma unroll
  for (int j = 0; j < EW_U; j++) {
    const int64_t i = base + j * 256;
    if (i < total) {
#pragma unroll
      for (int k = 0; k < S::NV; k++) gv[j][k] = silu_f(gv[j][k]) * uv[j][k];
      IO::store_nt(m, (i / cpr) * ld + (i % cpr) * S::NV, gv[j]);
    }
  }
}

constexpr int EW_U3 = 2;   // three inputs, two outputs: fewer vectors per lane keep the register count down
template <int DT>
__global__ __launch_bounds__(256) void swiglu_bwd_kernel(const void* g, const void* u, const void* dm, void* dg,
                                                         void* du, int64_t ld, int64_t T, int64_t f) {
  using S = St<DT>;
  using IO = VecIO<typename S::T, S::NV>;
  const int64_t cpr = f / S::NV, total = T * cpr;
  const int64_t base = (int64_t)blockIdx.x * (256 * EW_U3) + threadIdx.x;
  float gv[EW_U3][S::NV], uv[EW_U3][S::NV], dv[EW_U3][S::NV];
#pragma unroll
  for (int j = 0; j < EW_U3; j++) {
    const int64_t i = base + j * 256;
    if (i < total) {
      const int64_t off = (i / cpr) * ld + (i % cpr) * S::NV;
      IO::load_nt(g, off, gv[j]);
      IO::load_nt(u, off, uv[j]);
      IO::load_nt(dm, off, dv[j]);
    }
  }
#pragma unroll
  for (int j = 0; j < EW_U3; j++) {
    const int64_t i = base + j * 256;
    if (i < total) {
      const int64_t off = (i / cpr) * ld + (i % cpr) * S::NV;
      float o1[S::NV], o2[S::NV];
#pragma unroll
      for (int k = 0; k < S::NV; k++) {
        o1[k] = dv[j][k] * uv[j][k] * silu_prime_f(gv[j][k]);
        o2[k] = dv[j][k] * silu_f(gv[j][k]);
      }
      IO::store_nt(dg, off, o1);
      IO::store_nt(du, off, o2);
    }
  }
}

// ---- the same three maps for dense bf16 tensors (row pitch = row length), the form the block uses ------
// The tensor is one flat array; a workgroup owns the 256 * U vectors from byte blockIdx.x * CHUNK on and
// reaches them through a buffer resource that starts there and ends at the chunk's or the tensor's end,
// whichever comes first: the tail needs no bounds test, the body is straight-line code, and all loads of
// a lane are in flight before the first is used.  (With a test per vector the compiler waits for each
// vector's load inside its branch, one memory round trip after the other.)
constexpr int DENSE_U = 4, DENSE_U3 = 4;   // vectors per lane: one / two inputs, three inputs (measured best)
constexpr int NT_POLICY = 2;   // buffer cache policy: non-temporal, loads and stores (for these kernels default-policy
                               // stores measured 4 - 5 % slower, unlike the row kernel above)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t chunk_rsrc(const void* p, int64_t total_bytes, int64_t chunk_bytes) {
  const int64_t start = (int64_t)blockIdx.x * chunk_bytes;
  const int64_t left = total_bytes - start;
  return __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)p + start), 0,
                                           (uint32_t)(left < chunk_bytes ? left : chunk_bytes), 0x00020000);
}
__device__ __forceinline__ void unpack8v(const u32x4_t& t, float* v) { unpack8(make_uint4(t.x, t.y, t.z, t.w), v); }
__device__ __forceinline__ u32x4_t pack8v(const float* v) {
  const uint4 q = pack8(v);
  return u32x4_t{q.x, q.y, q.z, q.w};
}

template <int U>
__global__ __launch_bounds__(256) void act_fwd_dense_kernel(const void* z, void* a, int64_t total_bytes, int act) {
  constexpr int64_t CHUNK = 256 * U * 16;
  const __amdgpu_buffer_rsrc_t rz = chunk_rsrc(z, total_bytes, CHUNK), ra = chunk_rsrc(a, total_bytes, CHUNK);
  u32x4_t q[U];
#pragma unroll
  for (int j = 0; j < U; j++) q[j] = __builtin_amdgcn_raw_buffer_load_b128(rz, (j * 256 + (int)threadIdx.x) * 16, 0, NT_POLICY);
#pragma unroll
  for (int j = 0; j < U; j++) {
    float v[8];
    unpack8v(q[j], v);
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = act_f(v[k], act);
    __builtin_amdgcn_raw_buffer_store_b128(pack8v(v), ra, (j * 256 + (int)threadIdx.x) * 16, 0, NT_POLICY);
  }
}

// The rank-r activations of a block's layers, rebuilt from the checkpoints in one launch (a launch per layer is
// what a small block waits for: four of 2.4 us at 512 tokens): sigma(z), or z + h_{i-1} where the LaX variant
// hands an h.  Workgroups [first[i], first[i + 1]) take segment i; those from `act_blocks` on fold the norms' gammas into the
// weights of the call (512 tokens, rank 64, 256 features: 4.2 + 2.4 -> 3.9 us).
template <int U>
__global__ __launch_bounds__(256) void act_layers_kernel(ActLayers p, int act, int act_blocks, ScaleCols fold) {
  if ((int)blockIdx.x >= act_blocks) {
    scale_cols_part<LR_BF16>(fold, (int)blockIdx.x - act_blocks, (int)gridDim.x - act_blocks);
    return;
  }
  constexpr int64_t CHUNK = 256 * U * 16;
  int i = 0;
  while (i + 1 < p.n && (int)blockIdx.x >= p.first[i + 1]) i++;
  const int64_t start = (int64_t)((int)blockIdx.x - p.first[i]) * CHUNK, left = p.bytes[i] - start;
  const uint32_t size = (uint32_t)(left < CHUNK ? left : CHUNK);
  auto rsrc = [&](const void* q) { return __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)q + start), 0, size, 0x00020000); };
  const __amdgpu_buffer_rsrc_t rz = rsrc(p.z[i]), ra = rsrc(p.a[i]);
  u32x4_t q[U], hq[U];
#pragma unroll
  for (int j = 0; j < U; j++) q[j] = __builtin_amdgcn_raw_buffer_load_b128(rz, (j * 256 + (int)threadIdx.x) * 16, 0, NT_POLICY);
  const bool add = p.h[i] != nullptr;
  if (add) {
    const __amdgpu_buffer_rsrc_t rh = rsrc(p.h[i]);
#pragma unroll
    for (int j = 0; j < U; j++) hq[j] = __builtin_amdgcn_raw_buffer_load_b128(rh, (j * 256 + (int)threadIdx.x) * 16, 0, NT_POLICY);
  }
#pragma unroll
  for (int j = 0; j < U; j++) {
    float v[8], h[8];
    unpack8v(q[j], v);
    if (add) {
      unpack8v(hq[j], h);
#pragma unroll
      for (int k = 0; k < 8; k++) v[k] += h[k];
    } else {
#pragma unroll
      for (int k = 0; k < 8; k++) v[k] = act_f(v[k], act);
    }
    __builtin_amdgcn_raw_buffer_store_b128(pack8v(v), ra, (j * 256 + (int)threadIdx.x) * 16, 0, NT_POLICY);
  }
}

template <int U>
__global__ __launch_bounds__(256) void swiglu_fwd_dense_kernel(const void* g, const void* u, void* m, int64_t total_bytes) {
  constexpr int64_t CHUNK = 256 * U * 16;
  const __amdgpu_buffer_rsrc_t rg = chunk_rsrc(g, total_bytes, CHUNK), ru = chunk_rsrc(u, total_bytes, CHUNK),
                               rm = chunk_rsrc(m, total_bytes, CHUNK);
  u32x4_t gq[U], uq[U];
#pragma unroll
  for (int j = 0; j < U; j++) {
    const int off = (j * 256 + (int)threadIdx.x) * 16;
    gq[j] = __builtin_amdgcn_raw_buffer_load_b128(rg, off, 0, NT_POLICY);
    uq[j] = __builtin_amdgcn_raw_buffer_load_b128(ru, off, 0, NT_POLICY);
  }
#pragma unroll
  for (int j = 0; j < U; j++) {
    float gv[8], uv[8];
    unpack8v(gq[j], gv);
    unpack8v(uq[j], uv);
#pragma unroll
    for (int k = 0; k < 8; k++) gv[k] = silu_f(gv[k]) * uv[k];
    __builtin_amdgcn_raw_buffer_store_b128(pack8v(gv), rm, (j * 256 + (int)threadIdx.x) * 16, 0, NT_POLICY);
  }
}

template <int U>
__global__ __launch_bounds__(256) void swiglu_bwd_dense_kernel(const void* g, const void* u, const void* dm, void* dg,
                                                               void* du, int64_t total_bytes) {
  constexpr int64_t CHUNK = 256 * U * 16;
  const __amdgpu_buffer_rsrc_t rg = chunk_rsrc(g, total_bytes, CHUNK), ru = chunk_rsrc(u, total_bytes, CHUNK),
                               rd = chunk_rsrc(dm, total_bytes, CHUNK), rdg = chunk_rsrc(dg, total_bytes, CHUNK),
                               rdu = chunk_rsrc(du, total_bytes, CHUNK);
  u32x4_t gq[U], uq[U], dq[U];
#pragma unroll
  for (int j = 0; j < U; j++) {
    const int off = (j * 256 + (int)threadIdx.x) * 16;
    gq[j] = __builtin_amdgcn_raw_buffer_load_b128(rg, off, 0, NT_POLICY);
    uq[j] = __builtin_amdgcn_raw_buffer_load_b128(ru, off, 0, NT_POLICY);
    dq[j] = __builtin_amdgcn_raw_buffer_load_b128(rd, off, 0, NT_POLICY);
  }
#pragma unroll
  for (int j = 0; j < U; j++) {
    float gv[8], uv[8], dv[8], o1[8], o2[8];
    unpack8v(gq[j], gv);
    unpack8v(uq[j], uv);
    unpack8v(dq[j], dv);
#pragma unroll
    for (int k = 0; k < 8; k++) {
      o1[k] = dv[k] * uv[k] * silu_prime_f(gv[k]);
      o2[k] = dv[k] * silu_f(gv[k]);
    }
    const int off = (j * 256 + (int)threadIdx.x) * 16;
    __builtin_amdgcn_raw_buffer_store_b128(pack8v(o1), rdg, off, 0, NT_POLICY);
    __builtin_amdgcn_raw_buffer_store_b128(pack8v(o2), rdu, off, 0, NT_POLICY);
  }
}

// ---- rotary position embedding, in place, heads of 128 (rotate-half form) -----------------------
// x[rows, ld], head h in columns 128 h ..; the pair (v[i], v[i + 64]) of the row at position p = row % S
// is turned by the angle whose cosine and sine the caller tabulated as cs[p, i], sn[p, i] ([S, 64] fp32).
// One lane owns 8 consecutive i of one head: two 16-byte loads, two 16-byte stores.  sgn = -1 applies the
// transpose (the backward of the rotation).  x1, ld1, H1: a second tensor of as many rows, the keys beside the queries (H1 = 0: none;
// 777 rows, 32 and 8 heads: 5.1 + 4.6 -> 5.6 us).
__global__ __launch_bounds__(256) void rope128_kernel(uint16_t* x, int64_t ld, int H, uint16_t* x1, int64_t ld1, int H1,
                                                      const float* __restrict__ cs, const float* __restrict__ sn, int64_t rows, int S,
                                                      float sgn) {
  int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= rows * H * 8) {
    idx -= rows * H * 8;
    x = x1; ld = ld1; H = H1;
    if (idx >= rows * H * 8) return;
  }
  const int c8 = (int)(idx & 7) * 8;
  const int64_t rh = idx >> 3;
  const int h = (int)(rh % H);
  const int64_t row = rh / H;
  const int p = (int)(row % S);
  uint16_t* ptr = x + row * ld + (int64_t)h * 128 + c8;
  float lo[8], hi[8], c[8], s[8];
  unpack8(*reinterpret_cast<const uint4*>(ptr), lo);
  unpack8(*reinterpret_cast<const uint4*>(ptr + 64), hi);
  const float4* cp = reinterpret_cast<const float4*>(cs + (int64_t)p * 64 + c8);
  const float4* sp = reinterpret_cast<const float4*>(sn + (int64_t)p * 64 + c8);
  const float4 c0 = cp[0], c1 = cp[1], s0 = sp[0], s1 = sp[1];
  c[0] = c0.x; c[1] = c0.y; c[2] = c0.z; c[3] = c0.w; c[4] = c1.x; c[5] = c1.y; c[6] = c1.z; c[7] = c1.w;
  s[0] = s0.x; s[1] = s0.y; s[2] = s0.z; s[3] = s0.w; s[4] = s1.x; s[5] = s1.y; s[6] = s1.z; s[7] = s1.w;
  float olo[8], ohi[8];
#pragma unroll
  for (int i = 0; i < 8; i++) {
    const float si = s[i] * sgn;
    olo[i] = lo[i] * c[i] - hi[i] * si;
    ohi[i] = hi[i] * c[i] + lo[i] * si;
  }
  *reinterpret_cast<uint4*>(ptr) = pack8(olo);
  *reinterpret_cast<uint4*>(ptr + 64) = pack8(ohi);
}

// ---- transpose: out[c, r] = in[r, c]; 64x64 tiles through LDS.  Output columns rows..pad_to-1
// are written as zeros, so a transposed activation can serve as a k-contiguous GEMM operand whose
// k extent is rounded up to the 16-byte vector.
template <typename E>
__global__ __launch_bounds__(256) void transpose_kernel(const E* in, int64_t ld_in, int64_t s_in, E* out, int64_t ld_out, int64_t s_out,
                                                        int64_t rows, int64_t cols, int64_t pad_to) {
  __shared__ E tile[64][64 + 2];
  in += blockIdx.z * s_in; out += blockIdx.z * s_out;
  const int64_t r0 = (int64_t)blockIdx.y * 64, c0 = (int64_t)blockIdx.x * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int i = ty; i < 64; i += 4) {
    const int64_t r = r0 + i, c = c0 + tx;
    if (r < rows && c < cols) tile[i][tx] = in[r * ld_in + c];
  }
  __syncthreads();
  for (int i = ty; i < 64; i += 4) {
    const int64_t c = c0 + i, r = r0 + tx;
    if (c < cols) {
      if (r < rows) out[c * ld_out + r] = tile[tx][i];
      else if (r < pad_to) out[c * ld_out + r] = (E)0;
    }
  }
}

// 16-bit elements, all extents and pitches multiples of 8: global accesses are 16-byte vectors on both
// sides (a 2-byte-per-lane access moves 128 bytes per wavefront instruction, a 16-byte one 1 KB); the
// element shuffle happens between LDS and registers.  Tile: 64 input rows x 64 input columns.
__global__ __launch_bounds__(256) void transpose16_vec_kernel(const uint16_t* in, int64_t ld_in, int64_t s_in, uint16_t* out, int64_t ld_out,
                                                              int64_t s_out, int64_t rows, int64_t cols, int64_t pad_to) {
  __shared__ uint16_t tile[64][64 + 8];   // pitch 144 bytes: 16-byte aligned rows, column walks spread over banks
  in += blockIdx.z * s_in; out += blockIdx.z * s_out;
  const int64_t r0 = (int64_t)blockIdx.y * 64, c0 = (int64_t)blockIdx.x * 64;
  const int t = threadIdx.x;
#pragma unroll
  for (int k = 0; k < 2; k++) {           // 64 rows x 8 vectors
    const int v = t + k * 256, i = v >> 3, cv = (v & 7) * 8;
    const int64_t r = r0 + i, c = c0 + cv;
    uint4 q = make_uint4(0, 0, 0, 0);
    if (r < rows && c < cols) q = *reinterpret_cast<const uint4*>(in + r * ld_in + c);
    *reinterpret_cast<uint4*>(&tile[i][cv]) = q;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 2; k++) {           // 64 output rows (input columns) x 8 vectors of 8 input rows
    const int v = t + k * 256, i = v >> 3, rv = (v & 7) * 8;
    const int64_t c = c0 + i, r = r0 + rv;
    if (c < cols && r < pad_to) {
      uint16_t e[8];
#pragma unroll
      for (int j = 0; j < 8; j++) e[j] = tile[rv + j][i];   // rows past `rows` were staged as zeros
      uint4 q;
      q.x = e[0] | ((uint32_t)e[1] << 16); q.y = e[2] | ((uint32_t)e[3] << 16);
      q.z = e[4] | ((uint32_t)e[5] << 16); q.w = e[6] | ((uint32_t)e[7] << 16);
      *reinterpret_cast<uint4*>(out + c * ld_out + r) = q;
    }
  }
}

// Row partials -> row sums: eight lanes per row, lane l loads the units l, l + 8, ...  A unit that arrives as two or
// four partials is added up pairwise first, the order in which a wavefront that owns all its columns adds its
// quads of lanes; the units are then added front to back, each lane taking the others' from their registers.
// The sum has the same bits whichever tile wrote the partials.  Bound by launch and latency (8 MB at
// most); one thread per row left most CUs without a wavefront (4.8 us at 16384 rows x 8 partials).
__global__ __launch_bounds__(256) void rowsum_parts_kernel(const float* part, int64_t ld, int members, int slabs,
                                                           int per_unit, int units, float* out, int64_t M) {
  const int l = threadIdx.x & 7;
  const int64_t m = (int64_t)blockIdx.x * 32 + (threadIdx.x >> 3);
  float s = 0.f;
  for (int i0 = 0; i0 < members * units; i0 += 8) {
    const int i = i0 + l;
    float u = 0.f;
    if (m < M && i < members * units) {
      const int g = i / units, c0 = (i % units) * per_unit;
      const float* p = part + m * ld + g * slabs + c0;
      auto at = [&](int j) { return j < per_unit && c0 + j < slabs ? p[j] : 0.f; };
      u = (at(0) + at(1)) + (at(2) + at(3));
    }
#pragma unroll
    for (int j = 0; j < 8; j++) s += __shfl(u, j, 8);
  }
  if (m < M && l == 0) out[m] = s;
}

template <int DT>
__global__ __launch_bounds__(256) void rowdot_kernel(const void* a, int64_t lda, const void* b, int64_t ldb,
                                                     float* out, int64_t M, int64_t N) {
  using S = St<DT>;
  using IO = VecIO<typename S::T, S::NV>;
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= M) return;
  float s = 0.f;
  for (int64_t c = lane * S::NV; c < N; c += 64 * S::NV) {
    float av[S::NV], bv[S::NV];
    IO::load(a, row * lda + c, av);
    IO::load(b, row * ldb + c, bv);
#pragma unroll
    for (int i = 0; i < S::NV; i++) s = fmaf(av[i], bv[i], s);
  }
  s = wave_sum(s);
  if (lane == 0) out[row] = s;
}

// ---- finish a split-K weight gradient ------------------------------------------------------------
// Sums the nsplit fp32 partials of one 8-column (bf16) / 1-column (fp32) vector of the gradient, scales, accumulates, stores;
// s[] is the sum, front to back.  The loads of up to eight partials are issued together instead of one dependent round trip per
// partial (16 partials of 2048 x 512 in the narrow kernel below: 16.6 -> 14.0 us).  NS > 0: the number of partials is known at compile time; NS = 0 takes any count.
template <int DT, typename OT, int NS>
__device__ __forceinline__ void finish_vector(const float* part, int nsplit, int64_t count, int64_t off, const float* cs, void* dw,
                                              int accumulate, float* s) {
  constexpr int NV = St<DT>::NV;
  using OIO = VecIO<OT, NV>;
  using PIO = VecIO<float, NV>;
  // partials sp0 .. sp0 + G - 1, added to s (FIRST: the first of them starts it)
  auto take = [&](auto Gc, auto FIRST, int sp0) {
    constexpr int G = decltype(Gc)::value, first = decltype(FIRST)::value;
    float t[G][NV];
#pragma unroll
    for (int g = 0; g < G; g++) PIO::load(part, (int64_t)(sp0 + g) * count + off, t[g]);
    if constexpr (first) {
#pragma unroll
      for (int i = 0; i < NV; i++) s[i] = t[0][i];
    }
#pragma unroll
    for (int g = first; g < G; g++)
#pragma unroll
      for (int i = 0; i < NV; i++) s[i] += t[g][i];
  };
  using std::integral_constant;
  if constexpr (NS > 0) {
    take(integral_constant<int, NS>{}, integral_constant<int, 1>{}, 0);
  } else {
    constexpr integral_constant<int, 0> more{};
    int sp = nsplit >= 8 ? 8 : 1;
    if (nsplit >= 8) take(integral_constant<int, 8>{}, integral_constant<int, 1>{}, 0);
    else take(integral_constant<int, 1>{}, integral_constant<int, 1>{}, 0);
    for (; sp + 8 <= nsplit; sp += 8) take(integral_constant<int, 8>{}, more, sp);
    if (nsplit - sp >= 4) { take(integral_constant<int, 4>{}, more, sp); sp += 4; }
    if (nsplit - sp >= 2) { take(integral_constant<int, 2>{}, more, sp); sp += 2; }
    if (nsplit - sp >= 1) take(integral_constant<int, 1>{}, more, sp);
  }
  float o[NV];
#pragma unroll
  for (int i = 0; i < NV; i++) o[i] = s[i] * cs[i];
  if (accumulate) {
    float old[NV];
    OIO::load(dw, off, old);
#pragma unroll
    for (int i = 0; i < NV; i++) o[i] += old[i];
  }
  OIO::store(dw, off, o);
}

// One thread per vector of one row.  When dgamma partials are wanted a workgroup covers 32 rows of a
// 64-vector column strip: its 4 wavefronts take rows r, r+4, ... and add their column sums through LDS.
constexpr int WF_RB = 32;  // rows per dgamma partial
template <int DT, typename OT, bool DG, int NS>
__global__ __launch_bounds__(256) void wgrad_finish_kernel(const float* part, int nsplit, int64_t rows, int64_t cols,
                                                           void* dw, const void* colscale, const void* wdg,
                                                           float* dgpart, int accumulate) {
  constexpr int NV = St<DT>::NV;
  using IO = VecIO<typename St<DT>::T, NV>;
  __shared__ float sred[DG ? 4 * 64 * NV : 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t count = rows * cols;
  float cs[NV], dg[NV], s[NV];
#pragma unroll
  for (int i = 0; i < NV; i++) { cs[i] = 1.f; dg[i] = 0.f; }
  if constexpr (!DG) {
    const int64_t vpr = cols / NV;                               // vectors per row
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v >= rows * vpr) return;
    const int64_t r = v / vpr, c = (v % vpr) * NV;
    if (colscale) IO::load(colscale, c, cs);
    finish_vector<DT, OT, NS>(part, nsplit, count, r * cols + c, cs, dw, accumulate, s);
  } else {
    const int64_t c = ((int64_t)blockIdx.x * 64 + lane) * NV;
    const bool cok = c < cols;
    if (cok && colscale) IO::load(colscale, c, cs);
    const int64_t rbeg = (int64_t)blockIdx.y * WF_RB, rend = min(rows, rbeg + WF_RB);
    if (cok)
      for (int64_t r = rbeg + wave; r < rend; r += 4) {
        float wv[NV];
        IO::load(wdg, r * cols + c, wv);
        finish_vector<DT, OT, NS>(part, nsplit, count, r * cols + c, cs, dw, accumulate, s);
#pragma unroll
        for (int i = 0; i < NV; i++) dg[i] = fmaf(wv[i], s[i], dg[i]);
      }
#pragma unroll
    for (int i = 0; i < NV; i++) sred[(wave * 64 + lane) * NV + i] = dg[i];
    __syncthreads();
    if (wave == 0 && cok) {
#pragma unroll
      for (int i = 0; i < NV; i++)
        dgpart[(int64_t)blockIdx.y * cols + c + i] = sred[lane * NV + i] + sred[(64 + lane) * NV + i] +
                                                     sred[(128 + lane) * NV + i] + sred[(192 + lane) * NV + i];
    }
  }
}

// The same with dgamma partials where few strips leave CUs idle: 32 rows x 16 vectors per workgroup, every vector on a
// thread of its own instead of eight rows in turn, the column sums afterwards from LDS.  They are added in the
// wide kernel's order (four classes of rows r, r+4, ..., then the classes), so the choice does not show in dgamma.
constexpr int WF_NS = 16;  // vectors per strip
template <int DT, typename OT, int NS>
__global__ __launch_bounds__(256) void wgrad_finish_narrow_kernel(const float* part, int nsplit, int64_t rows, int64_t cols,
                                                                  void* dw, const void* colscale, const void* wdg,
                                                                  float* dgpart, int accumulate) {
  constexpr int NV = St<DT>::NV, W = WF_NS * NV;
  using IO = VecIO<typename St<DT>::T, NV>;
  __shared__ float ssum[WF_RB * W], sw[WF_RB * W], sclass[4 * W];
  const int tid = threadIdx.x, v = tid % WF_NS;
  const int64_t count = rows * cols, c0 = (int64_t)blockIdx.x * W, c = c0 + v * NV;
  const int64_t rbeg = (int64_t)blockIdx.y * WF_RB;
  const int nrows = (int)min((int64_t)WF_RB, rows - rbeg);
  float cs[NV];
#pragma unroll
  for (int i = 0; i < NV; i++) cs[i] = 1.f;
  if (c < cols) {
    if (colscale) IO::load(colscale, c, cs);
#pragma unroll
    for (int rr = tid / WF_NS; rr < WF_RB; rr += 256 / WF_NS) {
      if (rr >= nrows) continue;
      const int64_t off = (rbeg + rr) * cols + c;
      float s[NV], wv[NV];
      IO::load(wdg, off, wv);
      finish_vector<DT, OT, NS>(part, nsplit, count, off, cs, dw, accumulate, s);
#pragma unroll
      for (int i = 0; i < NV; i++) {
        ssum[rr * W + v * NV + i] = s[i];
        sw[rr * W + v * NV + i] = wv[i];
      }
    }
  }
  __syncthreads();
  for (int i = tid; i < 4 * W; i += 256) {
    const int q = i / W, col = i % W;
    float dg = 0.f;
    if (c0 + col < cols)
      for (int rr = q; rr < nrows; rr += 4) dg = fmaf(sw[rr * W + col], ssum[rr * W + col], dg);
    sclass[i] = dg;
  }
  __syncthreads();
  if (tid < W && c0 + tid < cols)
    dgpart[(int64_t)blockIdx.y * cols + c0 + tid] = sclass[tid] + sclass[W + tid] + sclass[2 * W + tid] + sclass[3 * W + tid];
}

// The whole pass behind a norm, dgamma included, where a gradient has few rows and partials: a workgroup takes 32 columns of all rows, the
// sums of 32 rows stay in LDS and are added up there, in the order of the two kernels that otherwise share the work.  Bound by its way
// in and out like those, of which it saves one; a thread takes every 64th row (bf16; fp32, one column per thread: every 8th) and its
// partials one after the other, on as many workgroups as there are strips of 32 columns, which costs more than the launch where there are
// several such rows or many partials.  us, two launches / this one, by rows (256 columns; 64 to 1024 differ by 0.7 at most) and
// partials, right behind what writes them:
//   bf16   64: 1 5.2 / 3.0, 32 10.5 / 8.0      128: 1 5.3 / 3.8, 12 7.5 / 7.2, 16 8.1 / 8.6, 32 11.0 / 13.3
//         160: 1 5.2 / 5.0, 4 5.8 / 6.1        192: 1 5.4 / 5.0, 2 5.4 / 5.6, 16 8.5 / 12.5       256: 1 5.4 / 5.7, 32 12.7 / 25.3
//   fp32   16: 1 3.8 / 2.6, 16 4.6 / 4.2        32: 1 4.3 / 3.4, 4 4.4 / 4.0, 8 4.5 / 5.0          64: 1 4.4 / 4.9, 16 5.9 / 9.1
constexpr int WHOLE_ROWS = 192, WHOLE_COLS = 1024;
inline bool finish_whole(int64_t rows, int64_t cols, int nsplit, int dt) {
  if (cols > WHOLE_COLS) return false;
  if (dt == LR_F32) return nsplit <= (rows <= 16 ? 16 : rows <= 32 ? 4 : 0);
  return rows <= 64 || nsplit <= (rows <= 128 ? 12 : rows <= WHOLE_ROWS ? 1 : 0);
}
template <int DT, typename OT>
__global__ __launch_bounds__(256) void wgrad_finish_whole_kernel(const float* part, int nsplit, int64_t rows, int64_t cols, void* dw,
                                                                 const void* colscale, const void* wdg, void* dgamma, int accumulate) {
  constexpr int NV = St<DT>::NV, W = 32, VS = W / NV, CH = 128;
  using IO = VecIO<typename St<DT>::T, NV>;
  using OIO = VecIO<OT, 1>;
  __shared__ float ssum[CH * W], sw[CH * W], sclass[CH / WF_RB * 4 * W], spart[WHOLE_ROWS / WF_RB * W];
  const int tid = threadIdx.x, v = tid % VS;
  const int64_t count = rows * cols, c0 = (int64_t)blockIdx.x * W, c = c0 + v * NV;
  float cs[NV];
#pragma unroll
  for (int i = 0; i < NV; i++) cs[i] = 1.f;
  if (c < cols && colscale) IO::load(colscale, c, cs);
  for (int r0 = 0; r0 < (int)rows; r0 += CH) {
    const int nrows = min(CH, (int)rows - r0);
    if (c < cols)
      for (int rr = tid / VS; rr < nrows; rr += 256 / VS) {
        const int64_t off = (int64_t)(r0 + rr) * cols + c;
        float s[NV], wv[NV];
        IO::load(wdg, off, wv);
        switch (nsplit) {
          case 1: finish_vector<DT, OT, 1>(part, nsplit, count, off, cs, dw, accumulate, s); break;
          case 2: finish_vector<DT, OT, 2>(part, nsplit, count, off, cs, dw, accumulate, s); break;
          case 4: finish_vector<DT, OT, 4>(part, nsplit, count, off, cs, dw, accumulate, s); break;
          default: finish_vector<DT, OT, 0>(part, nsplit, count, off, cs, dw, accumulate, s); break;
        }
#pragma unroll
        for (int i = 0; i < NV; i++) {
          ssum[rr * W + v * NV + i] = s[i];
          sw[rr * W + v * NV + i] = wv[i];
        }
      }
    __syncthreads();
    for (int i = tid; i < CH / WF_RB * 4 * W; i += 256) {
      const int col = i % W, first = i / (4 * W) * WF_RB, last = min(nrows, first + WF_RB);
      float dg = 0.f;
      if (c0 + col < cols)
        for (int rr = first + i / W % 4; rr < last; rr += 4) dg = fmaf(sw[rr * W + col], ssum[rr * W + col], dg);
      sclass[i] = dg;
    }
    __syncthreads();
    for (int i = tid; i < CH / WF_RB * W; i += 256) {
      const float* q = sclass + i / W * 4 * W + i % W;
      if (r0 / WF_RB + i / W < WHOLE_ROWS / WF_RB) spart[r0 / WF_RB * W + i] = q[0] + q[W] + q[2 * W] + q[3 * W];
    }
  }
  __syncthreads();
  if (tid >= W || c0 + tid >= cols) return;
  float s = 0.f;
  for (int p = 0; p < (int)((rows + WF_RB - 1) / WF_RB); p++) s += spart[p * W + tid];
  if (accumulate) {
    float o;
    OIO::load(dgamma, c0 + tid, &o);
    s += o;
  }
  OIO::store(dgamma, c0 + tid, &s);
}

// Several gradients in one launch, one thread per vector as above.  Bound by launches: a gradient of a small or mid-sized
// block is some hundred KB, whose pass takes 4 us of which most is the way in and out, and a backward has nine.
struct FinishMany {
  FinishJob job[FINISH_MAX];
  int first[FINISH_MAX + 1];    // workgroups [first[i], first[i + 1]) take job i
};
template <typename OT>
__global__ __launch_bounds__(256) void wgrad_finish_many_kernel(FinishMany, int accumulate) {
  // (read where the dispatch left them: an array indexed by the workgroup's job, not copied to the stack)
  const FinishMany& a = *(const FinishMany*)__builtin_amdgcn_kernarg_segment_ptr();
  constexpr int NV = St<LR_BF16>::NV;
  int j = 0;
#pragma unroll
  for (int i = 1; i < FINISH_MAX; i++) j += (int)blockIdx.x >= a.first[i] ? 1 : 0;
  j = __builtin_amdgcn_readfirstlane(j);
  const float* part = a.job[j].part;
  const int nsplit = a.job[j].nsplit;
  const int64_t count = a.job[j].count, off = ((int64_t)((int)blockIdx.x - a.first[j]) * 256 + threadIdx.x) * NV;
  if (off >= count) return;
  float cs[NV], s[NV];
#pragma unroll
  for (int i = 0; i < NV; i++) cs[i] = 1.f;
  switch (nsplit) {
    case 1: finish_vector<LR_BF16, OT, 1>(part, nsplit, count, off, cs, a.job[j].dw, accumulate, s); break;
    case 2: finish_vector<LR_BF16, OT, 2>(part, nsplit, count, off, cs, a.job[j].dw, accumulate, s); break;
    case 3: finish_vector<LR_BF16, OT, 3>(part, nsplit, count, off, cs, a.job[j].dw, accumulate, s); break;
    case 4: finish_vector<LR_BF16, OT, 4>(part, nsplit, count, off, cs, a.job[j].dw, accumulate, s); break;
    default: finish_vector<LR_BF16, OT, 0>(part, nsplit, count, off, cs, a.job[j].dw, accumulate, s); break;
  }
}

// Column sums of a few hundred partial rows, front to back: 16 columns (a 64-byte run) per workgroup, 16 threads per
// column that bring every 16th row into LDS, from where one of them adds the column up.  Bound by the latency of
// the loads: a thread per column walked all rows one after the other from a handful of workgroups (96 x 4096: 26 us).
template <typename OT>
__global__ __launch_bounds__(256) void colsum_parts_kernel(const float* part, int64_t nparts, int64_t cols, void* out,
                                                           int accumulate) {
  using IO = VecIO<OT, 1>;
  constexpr int NR = 128;
  __shared__ float rowsv[NR][17];
  const int ci = threadIdx.x & 15, pi = threadIdx.x >> 4;
  const int64_t c = (int64_t)blockIdx.x * 16 + ci;
  float s = 0.f;
  for (int64_t p0 = 0; p0 < nparts; p0 += NR) {
#pragma unroll
    for (int i = 0; i < NR / 16; i++) {
      const int64_t p = p0 + pi + i * 16;
      rowsv[pi + i * 16][ci] = c < cols && p < nparts ? part[p * cols + c] : 0.f;
    }
    __syncthreads();
    if (pi == 0) {
      const int n16 = (int)min((int64_t)NR, nparts - p0 + 15) / 16;
      for (int j = 0; j < n16; j++)
#pragma unroll
        for (int i = 0; i < 16; i++) s += rowsv[j * 16 + i][ci];   // (rows past the end are zeros)
    }
    __syncthreads();
  }
  if (pi != 0 || c >= cols) return;
  if (accumulate) {
    float o;
    IO::load(out, c, &o);
    s += o;
  }
  IO::store(out, c, &s);
}

// one workgroup per run of `per` items
inline unsigned grid_chunks(int64_t total, int per) { return (unsigned)((total + per - 1) / per); }
inline int grid1d(int64_t total, int cap = 256 * 32) {
  int64_t g = (total + 255) / 256;
  if (g > cap) g = cap;
  if (g < 1) g = 1;
  return (int)g;
}
inline unsigned scale_blocks(const ScaleCols& p, int dt) {
  if (p.rows0 + p.rows1 <= 0 || p.cols <= 0) return 0;
  return (unsigned)grid1d((p.rows0 + p.rows1) * (p.cols / (dt == LR_BF16 ? 8 : 1)));
}

}  // namespace

#define DISPATCH_DT(dt, KERNEL, grid, block, st, ...)                                              \
  do {                                                                                             \
    if ((dt) == LR_F32) hipLaunchKernelGGL(KERNEL<LR_F32>, grid, block, 0, st, __VA_ARGS__);       \
    else hipLaunchKernelGGL(KERNEL<LR_BF16>, grid, block, 0, st, __VA_ARGS__);                     \
    return hipGetLastError();                                                                      \
  } while (0)

hipError_t k_rms_stat(const void* x, int64_t ldx, float* stat, int64_t T, int64_t d, int dt, hipStream_t st) {
  if (T <= 0) return hipSuccess;
  DISPATCH_DT(dt, rms_stat_kernel, dim3((T + 3) / 4), dim3(256), st, x, ldx, stat, T, d);
}
hipError_t k_rmsnorm_apply(const void* x, int64_t ldx, const void* gamma, const float* stat, float eps, void* xhat,
                           int64_t ldo, int64_t T, int64_t d, int dt, hipStream_t st) {
  if (T <= 0) return hipSuccess;
  DISPATCH_DT(dt, rmsnorm_apply_kernel, dim3((T + 3) / 4), dim3(256), st, x, ldx, gamma, stat, eps, xhat, ldo, T, d, d);
}
hipError_t k_row_rms_scale(const void* h, int64_t ldh, const float* stat, int64_t d_total, float eps, void* out,
                           int64_t ldo, int64_t T, int64_t n, int dt, hipStream_t st) {
  if (T <= 0) return hipSuccess;
  DISPATCH_DT(dt, rmsnorm_apply_kernel, dim3((T + 3) / 4), dim3(256), st, h, ldh, (const void*)nullptr, stat, eps, out, ldo,
              T, n, d_total);
}
int64_t k_rmsnorm_bwd_parts(int64_t T) { return (T + NB_RB - 1) / NB_RB; }
hipError_t k_rmsnorm_bwd(const void* x, int64_t ldx, const void* gamma, const float* stat, float eps,
                         const void* dxhat, int64_t lddxh, const void* dres, int64_t lddres, void* dx, int64_t lddx,
                         float* dgamma_part, int64_t T, int64_t d, int dt, hipStream_t st) {
  if (T <= 0) return hipSuccess;
  if (dt == LR_BF16 && d <= 4096) {   // a row fits a wavefront's registers: single pass over every tensor
    // Rows per workgroup: a multiple of NB_RB chosen so that the launch is about one workgroup per CU
    // (measured at T = 32768: 6.1 TB/s with 256 workgroups of 128 rows against 5.8 with 512 of 64; 128
    // workgroups of 256 rows leave half the chip idle, 4.7).  The partial buffer keeps one row per NB_RB
    // rows of the input, whatever the launch.
    const int64_t nparts = k_rmsnorm_bwd_parts(T);
    int64_t mult = T / ((int64_t)NB_RB * 256);
    if (mult < 1) mult = 1;
    const int rows_per_wg = (int)(mult * NB_RB);
    const unsigned grid = (unsigned)((T + rows_per_wg - 1) / rows_per_wg);
    const auto launch = [&](auto nit, auto ahead) -> hipError_t {
      constexpr int NIT = decltype(nit)::value;
      const auto kernel = rmsnorm_bwd_row_kernel<NIT, decltype(ahead)::value>;
      // one-time opt-in to more than 64 KB of dynamic LDS (thread-safe static initialisation)
      static const hipError_t attr_err =
          hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, rn_row_lds(NIT));
      if (attr_err != hipSuccess) return attr_err;
      hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), rn_row_lds(NIT), st, (const uint16_t*)x, ldx,
                         (const uint16_t*)gamma, stat, eps, (const uint16_t*)dxhat, lddxh, (const uint16_t*)dres, lddres,
                         (uint16_t*)dx, lddx, dgamma_part, T, d, rows_per_wg, nparts);
      return hipGetLastError();
    };
    // The narrowest kernel that holds the row.  The widest with both sets of rows takes 300 registers, one workgroup per CU:
    // measured at d = 4096 against one set, 55.9 / 61.8 us with 128 workgroups, 50.2 / 52.2 with 19, 46.4 / 46.0 with 10, 47.0 / 45.3
    // with one, 92.3 / 91.4 with 256 and 196 / 194 with more, so at both ends it keeps to one set.
    const std::true_type ahead;
    if (d <= 512) return launch(std::integral_constant<int, 1>{}, ahead);
    if (d <= 1024) return launch(std::integral_constant<int, 2>{}, ahead);
    if (d <= 1536) return launch(std::integral_constant<int, 3>{}, ahead);
    if (d <= 2048) return launch(std::integral_constant<int, 4>{}, ahead);
    if (d <= 3072) return launch(std::integral_constant<int, 6>{}, ahead);
    return grid >= 16 && grid < 256 ? launch(std::integral_constant<int, 8>{}, ahead)
                                    : launch(std::integral_constant<int, 8>{}, std::false_type{});
  }
  DISPATCH_DT(dt, rmsnorm_bwd_kernel, dim3(k_rmsnorm_bwd_parts(T)), dim3(256), st, x, ldx, gamma, stat, eps, dxhat,
              lddxh, dres, lddres, dx, lddx, dgamma_part, T, d);
}
hipError_t k_act_fwd(const void* z, int64_t ldz, void* a, int64_t lda, int64_t T, int64_t n, int act, int dt,
                     hipStream_t st) {
  if (T <= 0 || n <= 0) return hipSuccess;
  if (dt == LR_BF16 && ldz == n && lda == n) {
    const int64_t bytes = T * n * 2;
    hipLaunchKernelGGL(act_fwd_dense_kernel<DENSE_U>, dim3(grid_chunks(bytes / 16, 256 * DENSE_U)), dim3(256), 0, st, z, a, bytes, act);
    return hipGetLastError();
  }
  const int nv = dt == LR_BF16 ? 8 : 1;
  DISPATCH_DT(dt, act_fwd_kernel, dim3(grid_chunks(T * (n / nv), 256 * EW_U)), dim3(256), st, z, ldz, a, lda, T, n, act);
}
hipError_t k_rope128_bf16(void* x, int64_t ld, int H, void* x1, int64_t ld1, int H1, const float* cos_tab, const float* sin_tab,
                          int64_t rows, int S, int inverse, hipStream_t st) {
  if (rows <= 0 || H <= 0) return hipSuccess;
  const int64_t items = rows * (H + H1) * 8;
  hipLaunchKernelGGL(rope128_kernel, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, st, (uint16_t*)x, ld, H, (uint16_t*)x1, ld1, H1,
                     cos_tab, sin_tab, rows, S, inverse ? -1.f : 1.f);
  return hipGetLastError();
}
hipError_t k_act_layers_bf16(ActLayers p, int act, const ScaleCols* fold, hipStream_t st) {
  unsigned grid = 0;
  for (int i = 0; i < p.n; i++) {
    p.first[i] = (int)grid;
    grid += grid_chunks(p.bytes[i] / 16, 256 * DENSE_U);
  }
  const int act_blocks = (int)grid;
  if (fold) grid += scale_blocks(*fold, LR_BF16);
  if (grid == 0) return hipSuccess;
  hipLaunchKernelGGL(act_layers_kernel<DENSE_U>, dim3(grid), dim3(256), 0, st, p, act, act_blocks, fold ? *fold : ScaleCols{});
  return hipGetLastError();
}
hipError_t k_swiglu_fwd(const void* g, const void* u, void* m, int64_t ld, int64_t T, int64_t f, int dt,
                        hipStream_t st) {
  if (T <= 0 || f <= 0) return hipSuccess;
  if (dt == LR_BF16 && ld == f) {
    const int64_t bytes = T * f * 2;
    hipLaunchKernelGGL(swiglu_fwd_dense_kernel<DENSE_U>, dim3(grid_chunks(bytes / 16, 256 * DENSE_U)), dim3(256), 0, st, g, u, m, bytes);
    return hipGetLastError();
  }
  const int nv = dt == LR_BF16 ? 8 : 1;
  DISPATCH_DT(dt, swiglu_fwd_kernel, dim3(grid_chunks(T * (f / nv), 256 * EW_U)), dim3(256), st, g, u, m, ld, T, f);
}
hipError_t k_swiglu_bwd(const void* g, const void* u, const void* dm, void* dg, void* du, int64_t ld, int64_t T,
                        int64_t f, int dt, hipStream_t st) {
  if (T <= 0 || f <= 0) return hipSuccess;
  if (dt == LR_BF16 && ld == f) {
    const int64_t bytes = T * f * 2;
    hipLaunchKernelGGL(swiglu_bwd_dense_kernel<DENSE_U3>, dim3(grid_chunks(bytes / 16, 256 * DENSE_U3)), dim3(256), 0, st, g, u, dm, dg, du, bytes);
    return hipGetLastError();
  }
  const int nv = dt == LR_BF16 ? 8 : 1;
  DISPATCH_DT(dt, swiglu_bwd_kernel, dim3(grid_chunks(T * (f / nv), 256 * EW_U3)), dim3(256), st, g, u, dm, dg, du, ld, T, f);
}
hipError_t k_transpose(const void* in, int64_t ld_in, int64_t s_in, void* out, int64_t ld_out, int64_t s_out, int64_t rows, int64_t cols,
                       int n, int dt, hipStream_t st) {
  if (rows <= 0 || cols <= 0 || n <= 0) return hipSuccess;
  const int64_t pad_to = ld_out;  // the whole output row is owned by the destination buffer
  dim3 grid((cols + 63) / 64, (pad_to + 63) / 64, n);
  if (dt == LR_F32)
    hipLaunchKernelGGL(transpose_kernel<float>, grid, dim3(256), 0, st, (const float*)in, ld_in, s_in, (float*)out, ld_out, s_out,
                       rows, cols, pad_to);
  else if (rows % 8 == 0 && cols % 8 == 0 && ld_in % 8 == 0 && ld_out % 8 == 0 && ((uintptr_t)in & 15) == 0 &&
           ((uintptr_t)out & 15) == 0 && (n == 1 || (s_in % 8 == 0 && s_out % 8 == 0)))
    hipLaunchKernelGGL(transpose16_vec_kernel, grid, dim3(256), 0, st, (const uint16_t*)in, ld_in, s_in, (uint16_t*)out, ld_out, s_out,
                       rows, cols, pad_to);
  else
    hipLaunchKernelGGL(transpose_kernel<uint16_t>, grid, dim3(256), 0, st, (const uint16_t*)in, ld_in, s_in, (uint16_t*)out, ld_out, s_out,
                       rows, cols, pad_to);
  return hipGetLastError();
}
hipError_t k_rowsum_parts(const float* part, int64_t ld, int members, const RowParts& rp, float* out, int64_t M,
                          hipStream_t st) {
  if (M <= 0) return hipSuccess;
  hipLaunchKernelGGL(rowsum_parts_kernel, dim3((M + 31) / 32), dim3(256), 0, st, part, ld, members, rp.slabs, rp.per_unit, rp.units,
                     out, M);
  return hipGetLastError();
}
hipError_t k_rowdot(const void* a, int64_t lda, const void* b, int64_t ldb, float* out, int64_t M, int64_t N, int dt,
                    hipStream_t st) {
  if (M <= 0) return hipSuccess;
  DISPATCH_DT(dt, rowdot_kernel, dim3((M + 3) / 4), dim3(256), st, a, lda, b, ldb, out, M, N);
}
hipError_t k_scale_cols(const ScaleCols& p, int dt, hipStream_t st) {
  const unsigned blocks = scale_blocks(p, dt);
  if (!blocks) return hipSuccess;
  DISPATCH_DT(dt, scale_cols_kernel, dim3(blocks), dim3(256), st, p);
}
hipError_t k_scale_cols_rms_stat(const ScaleCols& p, const void* x, int64_t ldx, float* stat, int64_t T, int64_t d, int dt, hipStream_t st) {
  const unsigned blocks = scale_blocks(p, dt), stat_blocks = T > 0 ? (unsigned)((T + 3) / 4) : 0;
  if (!blocks || !stat_blocks) {
    const hipError_t e = k_scale_cols(p, dt, st);
    return e != hipSuccess ? e : k_rms_stat(x, ldx, stat, T, d, dt, st);
  }
  DISPATCH_DT(dt, scale_cols_rms_stat_kernel, dim3(stat_blocks + blocks), dim3(256), st, p, (int)stat_blocks, x, ldx, stat, T, d);
}
int64_t k_wgrad_dgamma_parts(int64_t rows) { return (rows + WF_RB - 1) / WF_RB; }
hipError_t k_wgrad_finish(const float* part, int nsplit, int64_t rows, int64_t cols, void* dw, const void* colscale,
                          const void* w_for_dgamma, float* dgamma_part, void* dgamma, int accumulate, int dt, int out_dt,
                          hipStream_t st) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  const int nv = dt == LR_BF16 ? 8 : 1;
  const bool dg = w_for_dgamma != nullptr && dgamma_part != nullptr;
  if (dg && finish_whole(rows, cols, nsplit, dt) && (dt == LR_BF16 || out_dt == LR_F32)) {
    const dim3 grid((unsigned)((cols + 31) / 32));
#define LRB_WHOLE(DT_, OT_)                                                                                                         \
  hipLaunchKernelGGL((wgrad_finish_whole_kernel<DT_, OT_>), grid, dim3(256), 0, st, part, nsplit, rows, cols, dw, colscale, w_for_dgamma, \
                     dgamma, accumulate)
    if (dt == LR_F32) LRB_WHOLE(LR_F32, float);
    else if (out_dt == LR_F32) LRB_WHOLE(LR_BF16, float);
    else LRB_WHOLE(LR_BF16, bf16_t);
#undef LRB_WHOLE
    return hipGetLastError();
  }
  const int64_t blocks = (rows + WF_RB - 1) / WF_RB;
  // narrow strips where 64-vector ones would leave CUs without two workgroups (3072 x 512, five splits: 96 workgroups
  // took 20 us; 3072 x 4096: 768 workgroups read at 5.4 TB/s)
  const bool narrow = dg && (cols / nv + 63) / 64 * blocks < 512;
  dim3 grid = narrow ? dim3((unsigned)((cols / nv + WF_NS - 1) / WF_NS), (unsigned)blocks)
              : dg   ? dim3((unsigned)((cols / nv + 63) / 64), (unsigned)blocks)
                     : dim3((unsigned)((rows * (cols / nv) + 255) / 256));
#define LRB_WF2(DT_, OT_, NS_)                                                                                   \
  do {                                                                                                           \
    if (narrow)                                                                                                  \
      hipLaunchKernelGGL((wgrad_finish_narrow_kernel<DT_, OT_, NS_>), grid, dim3(256), 0, st, part, nsplit, rows, cols, dw, \
                         colscale, w_for_dgamma, dgamma_part, accumulate);                                      \
    else if (dg)                                                                                                 \
      hipLaunchKernelGGL((wgrad_finish_kernel<DT_, OT_, true, NS_>), grid, dim3(256), 0, st, part, nsplit, rows, cols, dw, \
                         colscale, w_for_dgamma, dgamma_part, accumulate);                                      \
    else                                                                                                         \
      hipLaunchKernelGGL((wgrad_finish_kernel<DT_, OT_, false, NS_>), grid, dim3(256), 0, st, part, nsplit, rows, cols, dw, \
                         colscale, w_for_dgamma, dgamma_part, accumulate);                                      \
  } while (0)
#define LRB_WF(DT_, OT_)                                                                                         \
  do {                                                                                                           \
    switch (nsplit) {                                                                                            \
      case 1: LRB_WF2(DT_, OT_, 1); break;                                                                       \
      case 2: LRB_WF2(DT_, OT_, 2); break;                                                                       \
      case 3: LRB_WF2(DT_, OT_, 3); break;                                                                       \
      case 4: LRB_WF2(DT_, OT_, 4); break;                                                                       \
      case 8: LRB_WF2(DT_, OT_, 8); break;                                                                       \
      default: LRB_WF2(DT_, OT_, 0); break;                                                                      \
    }                                                                                                            \
  } while (0)
  if (dt == LR_F32) LRB_WF(LR_F32, float);
  else if (out_dt == LR_F32) LRB_WF(LR_BF16, float);
  else LRB_WF(LR_BF16, bf16_t);
#undef LRB_WF
#undef LRB_WF2
  const hipError_t e = hipGetLastError();
  return e != hipSuccess || !dg ? e : k_colsum_parts(dgamma_part, blocks, cols, dgamma, accumulate, out_dt, st);
}
hipError_t k_wgrad_finish_many(const FinishJob* jobs, int n, int accumulate, int out_dt, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  if (n > FINISH_MAX) return hipErrorInvalidValue;
  FinishMany a;
  int wgs = 0;
  for (int i = 0; i < FINISH_MAX; i++) {
    a.first[i] = wgs;
    a.job[i] = i < n ? jobs[i] : FinishJob{nullptr, 1, 0, nullptr};
    wgs += (int)((a.job[i].count / St<LR_BF16>::NV + 255) / 256);
  }
  a.first[FINISH_MAX] = wgs;
  if (out_dt == LR_F32) hipLaunchKernelGGL(wgrad_finish_many_kernel<float>, dim3((unsigned)wgs), dim3(256), 0, st, a, accumulate);
  else hipLaunchKernelGGL(wgrad_finish_many_kernel<bf16_t>, dim3((unsigned)wgs), dim3(256), 0, st, a, accumulate);
  return hipGetLastError();
}
hipError_t k_colsum_parts(const float* part, int64_t nparts, int64_t cols, void* out, int accumulate, int out_dt,
                          hipStream_t st) {
  if (cols <= 0) return hipSuccess;
  if (out_dt == LR_F32)
    hipLaunchKernelGGL(colsum_parts_kernel<float>, dim3((cols + 15) / 16), dim3(256), 0, st, part, nparts, cols, out,
                       accumulate);
  else
    hipLaunchKernelGGL(colsum_parts_kernel<bf16_t>, dim3((cols + 15) / 16), dim3(256), 0, st, part, nparts, cols,
                       out, accumulate);
  return hipGetLastError();
}

}  // namespace lrb
