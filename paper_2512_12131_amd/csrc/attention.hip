// Causal multi-head attention, head_dim 128, bf16 in / fp32 softmax, for gfx950.
//
// Forward (one workgroup = 4 or 8 wavefronts x 32 queries of one (batch, head), for one query block and
// its causal mirror; K/V stream through LDS in 64-key tiles, double buffered):
//   S^T = K Q^T      MFMA, A = K rows from LDS, B = Q rows kept in registers for the whole kernel
//   online softmax   per query = per lane column of the S^T accumulators (one exchange of the wavefront's halves)
//   O^T += V^T P^T   MFMA, B = P^T straight from the softmax registers, A = V^T through the LDS
//                    transpose read (ds_read_b64_tr_b16), so V is stored as it arrives: [key][h]
// Working on the transposed problem is what lets the probabilities feed the second MFMA without
// leaving registers: the 32x32 accumulator layout (lane = column, 16 rows in 4-row groups) is, up
// to a fixed permutation of the k slots that the V^T loads follow, the B-operand layout.
//
// Backward, free of atomics and therefore deterministic, with D[q] = sum_h dO[q,h] O[q,h] and
// lse * log2(e) from a small preprocessing kernel:
//   dkv kernel - workgroup owns 128 keys, streams 64-query tiles from the diagonal on:
//                S = Q K^T, dP = dO V^T, dV^T += dO^T P, dK^T += Q^T dS;
//                in launches that leave CUs idle it also stores scale * dS^T (bf16, [key][query] per
//                (batch, head)), and dQ = (scale dS^T)^T K is then one causal k-major GEMM
//                (gemm_bf16.hip): the scores are formed once, 5 GEMM units in all
//   dq kernel  - the form without that workspace (work for the whole chip; S not a multiple of 8, or
//                too large): same walk as the forward (workgroup owns queries, streams keys): S^T,
//                dP^T = V dO^T, dS^T = P^T*(dP^T - D), dQ^T += K^T dS^T; 7 units together with the
//                dkv kernel
//
// Grouped-query form (fewer key / value heads than query heads, H / Hkv consecutive query heads per
// key / value head): the same kernels with K and V addressed by head / group and their own row stride.
// The dkv kernel then writes one dK and one dV contribution per query head into the workspace and a
// last kernel adds up each group; the dQ GEMM runs per batch element with (key / value head, head in
// group) as its two batch levels.  Multi-head attention is the case of groups of one.
#include "common.h"

namespace lrb {
namespace {

constexpr int HD = 128;
constexpr int KT = 64;            // keys (or queries, in the dkv kernel) per streamed tile
constexpr float LOG2E = 1.4426950408889634f;

typedef short s16x4 __attribute__((ext_vector_type(4)));

// raw v_exp_f32 (2^x): the arguments here are differences to a running maximum, never denormal-critical
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ bf16x8 lds_b128(const unsigned char* p) { return *reinterpret_cast<const bf16x8*>(p); }

// 8 consecutive accumulator values (v = t*8 .. t*8+7) packed as the bf16 B operand of one k16 step.
__device__ __forceinline__ bf16x8 pack_acc_half(const f32x16& a, int t) {
  uint4 q;
  q.x = pack_bf16x2(a[t * 8 + 0], a[t * 8 + 1]);
  q.y = pack_bf16x2(a[t * 8 + 2], a[t * 8 + 3]);
  q.z = pack_bf16x2(a[t * 8 + 4], a[t * 8 + 5]);
  q.w = pack_bf16x2(a[t * 8 + 6], a[t * 8 + 7]);
  return __builtin_bit_cast(bf16x8, q);
}

// Row index of accumulator element v inside a 32-row block.
__device__ __forceinline__ int acc_row(int v, int lane) { return 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); }

// Query-row fragments kept in registers: B operand (rows = queries) for all 8 k16 steps over h.
template <int MB>
__device__ __forceinline__ void load_row_frags(bf16x8 (&f)[MB][8], const uint16_t* base, int64_t ld, int row0,
                                               int nrows, int lane) {
#pragma unroll
  for (int mb = 0; mb < MB; mb++) {
    const int row = row0 + mb * 32 + (lane & 31);
    const bool ok = row < nrows;
#pragma unroll
    for (int ks = 0; ks < 8; ks++) {
      uint4 q = ok ? *reinterpret_cast<const uint4*>(base + (int64_t)row * ld + ks * 16 + (lane >> 5) * 8)
                   : make_uint4(0, 0, 0, 0);
      f[mb][ks] = __builtin_bit_cast(bf16x8, q);
    }
  }
}

// Writes a transposed accumulator block set acc[hb][.] (rows = h, column = the lane's token) as
// out[token][h], 4 consecutive h (8 bytes) at a time, scaled by `mul`.
__device__ __forceinline__ void store_acc_T(uint16_t* out_row, const f32x16 (&acc)[4], float mul, int lane) {
#pragma unroll
  for (int hb = 0; hb < 4; hb++)
#pragma unroll
    for (int g4 = 0; g4 < 4; g4++) {
      const int h = hb * 32 + 8 * g4 + 4 * (lane >> 5);
      uint2 w;
      w.x = pack_bf16x2(acc[hb][g4 * 4 + 0] * mul, acc[hb][g4 * 4 + 1] * mul);
      w.y = pack_bf16x2(acc[hb][g4 * 4 + 2] * mul, acc[hb][g4 * 4 + 3] * mul);
      *reinterpret_cast<uint2*>(out_row + h) = w;
    }
}

// ----------------------------------------------------------------------------------------------
// 64-row x 128-column bf16 tiles moved global -> LDS without passing through registers.
// One buffer_load_dwordx4 ... lds per wavefront writes 1 KB = 4 tile rows of 256 bytes; lane L's 16
// bytes land at base + 16 L, i.e. row L/16, physical chunk L%16.  Rows are not padded; instead the
// 16-byte chunks of a row are XOR-swizzled and each lane fetches the logical chunk that belongs in its
// slot.  Two swizzles, one per read pattern:
//   SWZ_ROW16  chunk ^ (row % 16)        16 consecutive rows x one logical chunk (ds_read_b128 of
//                                        MFMA operand rows) cover all 64 banks
//   SWZ_ROW4   chunk ^ ((row % 4) * 4)   4 consecutive rows x 64 bytes (the LDS transpose read)
//                                        cover all 64 banks
// Rows at or past `nrows` are fetched with an out-of-range offset: the load returns zeros.
// ----------------------------------------------------------------------------------------------
constexpr int TILE_BYTES = KT * HD * 2;
constexpr uint32_t DMA_OOB = 0x80000000u;
enum { SWZ_ROW16 = 0, SWZ_ROW4 = 1, SWZ_BOTH = 2 };
//   SWZ_BOTH   chunk ^ ((row % 4) * 4 + (row / 4) % 4)   serves both read patterns of a tile that is
//                                        needed row-wise and transposed: 16 consecutive rows see 16
//                                        different terms, 4 consecutive rows 4 different 64-byte groups
#define LRB_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

// Buffer resource as four scalar words: base address, stride 0, size in bytes, data format word.
typedef uint32_t rsrc_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  const uint64_t a = (uint64_t)(uintptr_t)base;
  rsrc_t r = {(uint32_t)a, (uint32_t)(a >> 32) & 0xffffu, bytes, 0x00020000u};
  // Five wait states have to pass between a vector write of a scalar (v_readfirstlane) and a buffer instruction that reads
  // it; the compiler does not look for buffer instructions inside lds_dma's assembly.
  asm volatile("s_nop 4" : "+s"(r));
  return r;
}
__device__ __forceinline__ rsrc_t tile_rsrc(const uint16_t* base) { return make_rsrc(base, 0x7fffffffu); }

// One global -> LDS load of BYTES (4 or 16) per lane: lane L's data lands at lds + BYTES * L.  Issued
// as inline assembly on purpose: through the builtin the compiler treats every later LDS read as a
// possible read of this load's destination and makes it wait for ALL global loads in flight, i.e. the
// tile being worked on would wait for the next tile's loads.  Completion is tracked by hand instead
// (wait_vm0 before the barrier that publishes a tile).  `lds` must be wavefront-uniform.
template <int BYTES>
__device__ __forceinline__ void lds_dma(rsrc_t rs, const unsigned char* lds, uint32_t voff) {
  const uint32_t m0v = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)LRB_LDS_PTR(lds));
  if constexpr (BYTES == 16)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(m0v), "v"(voff), "s"(rs) : "m0", "memory");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" ::"s"(m0v), "v"(voff), "s"(rs) : "m0", "memory");
}

// Per-lane byte offsets (row * ld + logical chunk) of the 16 / NW wavefront loads that a wavefront of
// an NW-wavefront workgroup contributes to one tile.
template <int SWZ, int NL>
__device__ __forceinline__ void dma_lane_offsets(uint32_t (&off)[NL], int (&row)[NL], int64_t ld, int wave, int lane) {
  constexpr int NW = 16 / NL;
#pragma unroll
  for (int i = 0; i < NL; i++) {
    const int r = (i * NW + wave) * 4 + (lane >> 4);
    const int pc = lane & 15;
    const int lc = SWZ == SWZ_ROW16 ? (pc ^ (r & 15))
                 : SWZ == SWZ_ROW4 ? (pc ^ ((r & 3) << 2))
                                   : (pc ^ (((r & 3) << 2) | ((r >> 2) & 3)));
    row[i] = r;
    off[i] = (uint32_t)(r * (int)ld + lc * 8) * 2u;
  }
}
template <int NL>
__device__ __forceinline__ void dma_tile(rsrc_t rs, unsigned char* tile, const uint32_t (&off)[NL],
                                         const int (&row)[NL], int row0, int nrows, int64_t ld, int wave) {
  constexpr int NW = 16 / NL;
  const uint32_t base = (uint32_t)row0 * (uint32_t)ld * 2u;
#pragma unroll
  for (int i = 0; i < NL; i++) {
    const uint32_t o = (row0 + row[i]) < nrows ? base + off[i] : DMA_OOB;
    lds_dma<16>(rs, tile + (i * NW + wave) * 1024, o);
  }
}
// s_waitcnt vmcnt(0) alone (gfx9 encoding), and lgkmcnt(0) alone
__device__ __forceinline__ void wait_vm0() { __builtin_amdgcn_s_waitcnt(0x0f70); }
__device__ __forceinline__ void wait_lgkm0() { __builtin_amdgcn_s_waitcnt(0xc07f); }
// s_waitcnt vmcnt(N) alone, N < 64: bits 3:0 and 15:14 hold vmcnt, the other counters stay at "no wait"
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 15) | ((N >> 4) << 14));
}

// A operand (32 rows = tile rows r0 + lane%32, k slots = logical chunk ks*2 + lane/32) from a
// SWZ_ROW16 tile.  r0 is a multiple of 16, so the swizzle term depends on the lane only.
__device__ __forceinline__ bf16x8 swz_row_frag(const unsigned char* tile, int r0, int ks, int lane) {
  const int row = r0 + (lane & 31);
  return lds_b128(tile + row * 256 + (((ks * 2 + (lane >> 5)) ^ (lane & 15)) << 4));
}
// Transposed A operand from a SWZ_ROW4 tile stored [k][col]: rows = columns c0..c0+31 (c0 a multiple
// of 32), k slots (half = lane / 32, e = 0..7) = tile rows k0 + (e/4)*8 + half*4 + e%4 (k0 a multiple
// of 16), which is the row order of a 32x32 accumulator.  Inside each group of 16 lanes the transpose
// read hands lane i the i-th 16-bit column of the 4 x 16 block that the 16 lanes fetched as 4 rows x
// 4 lanes x 8 bytes.
__device__ __forceinline__ bf16x8 swz_tr_frag(const unsigned char* tile, int k0, int c0, int lane) {
  const int g = lane >> 4, s = lane & 15;
  const int rl = (g >> 1) * 4 + (s >> 2);                       // row inside the 16-row group; rl % 4 = s / 4
  const int chunk = (c0 >> 3) + (g & 1) * 2 + ((s & 3) >> 1);   // logical 16-byte chunk
  const unsigned char* p0 = tile + (k0 + rl) * 256 + ((chunk ^ ((s >> 2) << 2)) << 4) + (s & 1) * 8;
  const unsigned char* p1 = p0 + 8 * 256;
  s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p0));
  s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p1));
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  s16x8 r = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(bf16x8, r);
}

// The same two operand reads for a SWZ_BOTH tile (r0 and k0 multiples of 16, c0 a multiple of 32).
__device__ __forceinline__ bf16x8 both_row_frag(const unsigned char* tile, int r0, int ks, int lane) {
  const int l31 = lane & 31;
  const int f = ((l31 & 3) << 2) | ((l31 >> 2) & 3);
  return lds_b128(tile + (r0 + l31) * 256 + (((ks * 2 + (lane >> 5)) ^ f) << 4));
}
__device__ __forceinline__ bf16x8 both_tr_frag(const unsigned char* tile, int k0, int c0, int lane) {
  const int g = lane >> 4, s = lane & 15;
  const int rl = (g >> 1) * 4 + (s >> 2);
  const int f0 = ((s >> 2) << 2) | (g >> 1);                    // rows k0 + rl; rows + 8 flip bit 1 of the term
  const int chunk = (c0 >> 3) + (g & 1) * 2 + ((s & 3) >> 1);
  const unsigned char* rowp = tile + (k0 + rl) * 256 + (s & 1) * 8;
  s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(rowp + ((chunk ^ f0) << 4)));
  s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (s16x4 __attribute__((address_space(3)))*)(rowp + 8 * 256 + ((chunk ^ f0 ^ 2) << 4)));
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  s16x8 r = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(bf16x8, r);
}

// The hardware deals consecutive workgroup ids to the 8 XCDs in rotation.  This maps the id back so
// that each XCD works through a contiguous range of (batch, head, block) triples, block fastest: the
// workgroups that stream the same head's K / V (or Q / dO) tiles then share one XCD's L2 instead of
// every XCD fetching every head.
struct WgCoord { int x, head, b; };
__device__ __forceinline__ WgCoord wg_coord() {
  const int nx = gridDim.x, H = gridDim.y;
  const int total = nx * H * (int)gridDim.z;
  const int lin = (int)blockIdx.x + nx * ((int)blockIdx.y + H * (int)blockIdx.z);
  const int xcd = lin % 8, loc = lin / 8;
  const int base = total / 8, rem = total % 8;
  const int v = xcd * base + (xcd < rem ? xcd : rem) + loc;
  WgCoord c;
  c.x = v % nx;
  c.head = (v / nx) % H;
  c.b = v / (nx * H);
  return c;
}

constexpr int FWD_LDS = 4 * TILE_BYTES;   // K and V, double buffered

// Compile-time loop over std::integral_constant indices: register arrays indexed by them stay in registers.
template <int N, class F, int I = 0>
__device__ __forceinline__ void unroll_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    unroll_for<N, F, I + 1>(static_cast<F&&>(f));
  }
}
// Buffer resource of S rows of 256 bytes, ld elements apart: rows at or past S are out of range by themselves.
__device__ __forceinline__ rsrc_t rows_rsrc(const uint16_t* base, int S, int64_t ld) {
  return make_rsrc(base, (uint32_t)(S - 1) * (uint32_t)ld * 2u + 256u);
}
// The same resource from byte `off` on (scalar arithmetic only); empty, so that loads deliver zeros, where !valid.
__device__ __forceinline__ rsrc_t rsrc_from(rsrc_t r, uint32_t off, bool valid) {
  const uint64_t a = (((uint64_t)r.y << 32) | r.x) + (valid ? off : 0u);
  return rsrc_t{(uint32_t)a, (uint32_t)(a >> 32), valid ? r.z - off : 0u, r.w};
}
// lds_dma<16> with the LDS address as a number
__device__ __forceinline__ void lds_dma_at(rsrc_t rs, uint32_t lds, uint32_t voff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds), "v"(voff), "s"(rs) : "m0", "memory");
}
__device__ __forceinline__ void lds_dma4_at(rsrc_t rs, uint32_t lds, uint32_t voff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" ::"s"(lds), "v"(voff), "s"(rs) : "m0", "memory");
}
// max / sum of the two lanes l and l + 32
__device__ __forceinline__ float half_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// ----------------------------------------------------------------------------------------------
// forward
// ----------------------------------------------------------------------------------------------
// Bound: the issue of vector ALU work beside the MFMAs, and in long runs the chip's power.  An iteration works on two key
// tiles: the scores of tile j + 1 (16 MFMAs) and the output of tile j (16 MFMAs) with the softmax of tile j and the maximum of
// the new scores threaded between them, one MFMA and a share of the rest per slot, so that a wavefront's matrix and
// vector work overlap and its LDS operands are read some MFMAs ahead.  (One tile at a time - scores, softmax, output -
// the phases of the two wavefronts of a SIMD did not overlap enough: matrix pipes 41 % busy, now 52 %.)  One barrier per
// iteration, in the middle, where the K operands have been read and no V operand yet: each load then has a whole iteration to land.
// The loop over the unmasked tiles is unrolled by two, its score registers swapping roles; the branches (masks, odd
// tiles, the end) stay outside, which is what lets the compiler keep every tuple in place (246 registers, no copies).
// Sustained, one tile at a time -> now (us): 4 x 4096 tokens, 32 heads 627 -> 555; 8 x 2048, 16 heads 175 -> 157;
// 2 x 2047, 32 / 8 heads 89.9 -> 79; 777 tokens, 32 / 8 heads 23.5 -> 19.9; 4 x 4096, 4 heads 93.8 -> 78.
// A tile past the last one is not asked for where that costs a scalar branch outside the main loop (128 x 64 tokens, 16 heads:
// 32.7 -> 31.0).
constexpr int FWD_D = 4;        // LDS operands are read this many MFMAs ahead (2, 4, 8: within 2 %)
constexpr int FWD_BAR = 12;     // slot of the barrier: the last operand of the score product has been read
// elements of the softmax done by the end of slot s: each bf16x8 operand is whole when its MFMAs come (slots 16, 20, 24, 28)
constexpr int fwd_elems(int s) { return s < 0 ? 0 : s < 16 ? 5 * (s + 1) / 4 : s < 28 ? 5 + s : 32; }

template <int NW>
__global__ __launch_bounds__(NW * 64, 2) void attn_fwd_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                                                       const uint16_t* __restrict__ v, uint16_t* __restrict__ o,
                                                       float* __restrict__ lse, int64_t ld, int64_t ldkv, int grp, int S,
                                                       int H, float scale) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int BQ = NW * 32, NL = 16 / NW;             // queries per block, 1 KB loads per wavefront and tile
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nqb = (S + BQ - 1) / BQ;
  const WgCoord wg = wg_coord();
  const int head = wg.head, b = wg.b;
  const int64_t tok0 = (int64_t)b * S;
  const uint16_t* qb = q + tok0 * ld + head * HD;
  // grouped-query attention: grp consecutive query heads share key / value head head / grp (rows of ldkv)
  const int kvh = head / grp;
  const rsrc_t rsK = rows_rsrc(k + tok0 * ldkv + kvh * HD, S, ldkv);
  const rsrc_t rsV = rows_rsrc(v + tok0 * ldkv + kvh * HD, S, ldkv);
  const float c = scale * LOG2E;
  uint32_t offK[NL], offV[NL];
  {
    int row[NL];
    dma_lane_offsets<SWZ_ROW16, NL>(offK, row, ldkv, wave, lane);
    dma_lane_offsets<SWZ_ROW4, NL>(offV, row, ldkv, wave, lane);
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)LRB_LDS_PTR(smem) + (uint32_t)wave * 1024u;
  // load i of key tile t into its slot (K: slots 0, 1, V: slots 2, 3); a tile past the last one: every lane out of range
  auto dma = [&](bool isV, int t, int ntiles, int i) {
    lds_dma_at(rsrc_from(isV ? rsV : rsK, (uint32_t)t * (uint32_t)(KT * 2) * (uint32_t)ldkv, t < ntiles),
               lds0 + (uint32_t)((isV ? 2 : 0) + (t & 1)) * TILE_BYTES + (uint32_t)(i * NW) * 1024u, isV ? offV[i] : offK[i]);
  };

  // Causal work grows linearly with the query block index.  Every workgroup takes one block from the
  // late end and its mirror image from the early end, so that all workgroups of the launch do the
  // same amount of work (the hardware deals workgroups to the XCDs in strict rotation: unequal
  // workgroups leave most of the chip waiting for the XCD that drew the heavy ones).  A launch that gives
  // every block a CU of its own is not paired (grid.x = the number of blocks).
  for (int pass = 0; pass < 2; pass++) {
  const int qblk = pass == 0 ? nqb - 1 - wg.x : wg.x;
  // unpaired launch, or odd block count: the middle block has no mirror
  if (pass == 1 && ((int)gridDim.x == nqb || qblk >= nqb - 1 - wg.x)) break;
  const int q0 = qblk * BQ;
  const int qw0 = q0 + wave * 32;                        // first query of this wavefront
  const int kv_end = min(S, q0 + BQ);                    // causal: keys up to the block's last query
  const int ntiles = (kv_end + KT - 1) / KT;
  const int ntw = qw0 < S ? min(ntiles, (qw0 + 31) / KT + 1) : 0;   // ... and up to this wavefront's

  __syncthreads();                                       // the pass before is done with the slots
#pragma unroll
  for (int i = 0; i < NL; i++) dma(false, 0, ntiles, i);
#pragma unroll
  for (int i = 0; i < NL; i++) dma(true, 0, ntiles, i);
  if (ntiles > 1) {
#pragma unroll
    for (int i = 0; i < NL; i++) dma(false, 1, ntiles, i);
  }
  bf16x8 qf[1][8];
  load_row_frags<1>(qf, qb, ld, qw0, S, lane);

  f32x16 oacc[4], st[2];                                 // st: scores (S^T) of the tile whose softmax comes next
#pragma unroll
  for (int hb = 0; hb < 4; hb++)
#pragma unroll
    for (int e = 0; e < 16; e++) oacc[hb][e] = 0.f;
#pragma unroll
  for (int nb = 0; nb < 2; nb++)
#pragma unroll
    for (int e = 0; e < 16; e++) st[nb][e] = 0.f;
  float mrun = -INFINITY, lrun = 0.f, alpha = 1.f, mc = 0.f;
  bf16x8 fr[FWD_D];                                      // operands read ahead, slot s in fr[s % FWD_D]

  // operand of MFMA slot s: 0..15 scores (k16 step s / 2, key block s % 2), 16..31 output (16 keys each four slots)
  auto read_frag = [&](auto Sc, const unsigned char* sK, const unsigned char* sV) {
    constexpr int s = decltype(Sc)::value;
    if constexpr (s < 16) fr[s % FWD_D] = swz_row_frag(sK, (s & 1) * 32, s >> 1, lane);
    else fr[s % FWD_D] = swz_tr_frag(sV, ((s - 16) >> 2) * 16, (s & 3) * 32, lane);
  };
  // maximum of a tile's scores, mx where no key is masked; else (diagonal / tail tile) masks them first
  auto masked_max = [&](f32x16 (&x)[2], int key0, float mx) -> float {
    if ((key0 + KT - 1 > qw0) || (key0 + KT > S)) {      // wavefront-uniform
      const int lim = min(qw0 + (lane & 31) + 1, S) - key0 - 4 * (lane >> 5);   // first masked key, less the lane's rows
      mx = -INFINITY;
#pragma unroll
      for (int nb = 0; nb < 2; nb++)
#pragma unroll
        for (int e = 0; e < 16; e++) {
          x[nb][e] = nb * 32 + acc_row(e, 0) >= lim ? -INFINITY : x[nb][e];
          mx = fmaxf(mx, x[nb][e]);
        }
    }
    return mx;
  };
  // running maximum over the new scores: the factor of what is there already, and the exponents' common term
  auto new_max = [&](float mx) {
    const float mnew = fmaxf(mrun, half_max(mx));        // finite: key 0 is visible to every query
    alpha = fast_exp2((mrun - mnew) * c);
    mrun = mnew;
    mc = mnew * c;
  };

  wait_vm0();
  __syncthreads();
  if (ntw > 0) {                                         // scores of the first tile
    unroll_for<FWD_D>([&](auto I) { read_frag(I, smem, smem); });
    unroll_for<16>([&](auto I) {
      constexpr int s = decltype(I)::value;
      st[s & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[s % FWD_D], qf[0][s >> 1], st[s & 1], 0, 0, 0);
      if constexpr (s + FWD_D < 16) read_frag(std::integral_constant<int, s + FWD_D>{}, smem, smem);
    });
    float mx = -INFINITY;
#pragma unroll
    for (int nb = 0; nb < 2; nb++)
#pragma unroll
      for (int e = 0; e < 16; e++) mx = fmaxf(mx, st[nb][e]);
    new_max(masked_max(st, 0, mx));
    if (ntw > 1) unroll_for<FWD_D>([&](auto I) { read_frag(I, smem + TILE_BYTES, smem); });
  }
  wait_lgkm0();
  __builtin_amdgcn_s_barrier();                          // nobody reads K's first tile any more
  if (ntiles > 2) {
#pragma unroll
    for (int i = 0; i < NL; i++) dma(false, 2, ntiles, i);
  }

  // all of this workgroup's reads of K(j + 1) and V(j - 1) are done, K(j + 2) and V(j) have landed
  auto turn = [&] {
    wait_lgkm0();
    wait_vm0();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  auto next_loads = [&](int j, int i) {                  // into the slots just left
    if (i < NL) dma(true, j + 1, ntiles, i);
    else dma(false, j + 3, ntiles, i - NL);
  };
  // the running maximum settles after the first tiles: skip the rescale when no lane needs it
  auto rescale = [&] {
    if (__builtin_amdgcn_ballot_w64(alpha != 1.f) != 0) {
#pragma unroll
      for (int hb = 0; hb < 4; hb++)
#pragma unroll
        for (int e = 0; e < 16; e++) oacc[hb][e] *= alpha;
    }
  };
  uint32_t pw[16];                                       // the probabilities as bf16 pairs: two operands per key block
  float rs = 0.f, plow = 0.f;
  // elements F .. T - 1 of the softmax (key block e / 16, accumulator row e % 16)
  auto softmax_to = [&](const f32x16 (&x)[2], auto Fc, auto Tc) {
    constexpr int f = decltype(Fc)::value, t = decltype(Tc)::value;
    unroll_for<t - f>([&](auto I) {
      constexpr int e = f + decltype(I)::value;
      const float p = fast_exp2(fmaf(x[e >> 4][e & 15], c, -mc));
      rs += p;
      if constexpr (e & 1) pw[e >> 1] = pack_bf16x2(plow, p);
      else plow = p;
    });
  };
  auto pv = [&](auto Sc) {                               // output MFMA of slot s
    constexpr int s = decltype(Sc)::value, kk = (s - 16) >> 2;
    const bf16x8 pf = __builtin_bit_cast(bf16x8, make_uint4(pw[kk * 4], pw[kk * 4 + 1], pw[kk * 4 + 2], pw[kk * 4 + 3]));
    oacc[s & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[s % FWD_D], pf, oacc[s & 3], 0, 0, 0);
  };
  // softmax and output of tile j (scores sc), scores of tile j + 1 (into sn); par = j % 2.  MASK: tile j + 1 may be the diagonal
  // or the tail tile (the last one of the wavefront).
  auto iteration = [&](int j, auto par, auto MASK, f32x16 (&sc)[2], f32x16 (&sn)[2]) {
    const unsigned char* sK1 = smem + (par ^ 1) * TILE_BYTES;              // K of tile j + 1
    const unsigned char* sK2 = smem + par * TILE_BYTES;                    // K of tile j + 2
    const unsigned char* sV = smem + (2 + par) * TILE_BYTES;               // V of tile j
    rescale();
    rs = 0.f;
#pragma unroll
    for (int nb = 0; nb < 2; nb++)
#pragma unroll
      for (int e = 0; e < 16; e++) sn[nb][e] = 0.f;
    float mx0 = -INFINITY, mx1 = -INFINITY;
    unroll_for<32>([&](auto Sc) {
      constexpr int s = decltype(Sc)::value;
      if constexpr (s < 16)
        sn[s & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[s % FWD_D], qf[0][s >> 1], sn[s & 1], 0, 0, 0);
      else pv(Sc);
      if constexpr (s == FWD_BAR) turn();
      // operands: V only from behind the barrier, then K of the tile after next
      unroll_for<32>([&](auto I) {
        constexpr int t = decltype(I)::value + FWD_D;               // target slot
        constexpr int at = t - FWD_D < FWD_BAR && t >= 16 ? FWD_BAR : t - FWD_D;
        if constexpr (at == s) {
          if constexpr (t < 32) read_frag(std::integral_constant<int, t>{}, sK1, sV);
          else read_frag(std::integral_constant<int, t - 32>{}, sK2, sV);
        }
      });
      if constexpr (s > FWD_BAR && s <= FWD_BAR + 2 * NL) next_loads(j, s - FWD_BAR - 1);
      softmax_to(sc, std::integral_constant<int, fwd_elems(s - 1)>{}, std::integral_constant<int, fwd_elems(s)>{});
      if constexpr (s >= 18 && s < 26) {                            // maximum of the new scores
        constexpr int e = (s - 18) * 2;
        mx0 = fmaxf(fmaxf(mx0, sn[0][e]), sn[0][e + 1]);
        mx1 = fmaxf(fmaxf(mx1, sn[1][e]), sn[1][e + 1]);
      }
      // (the sums stay in this block: moved down to their use they would keep every element alive)
      if constexpr (fwd_elems(s - 1) != fwd_elems(s)) asm volatile("" : "+v"(rs));
      if constexpr (s == 25) asm volatile("" : "+v"(mx0), "+v"(mx1));
      __builtin_amdgcn_sched_barrier(0);
    });
    lrun = lrun * alpha + rs;
    float mx = fmaxf(mx0, mx1);
    if constexpr (decltype(MASK)::value) mx = masked_max(sn, (j + 1) * KT, mx);
    new_max(mx);
  };
  int j = 0;
  f32x16 s2[2];
  for (; j + 3 < ntw; j += 2) {
    iteration(j, std::integral_constant<int, 0>{}, std::false_type{}, st, s2);
    iteration(j + 1, std::integral_constant<int, 1>{}, std::false_type{}, s2, st);
  }
  for (; j + 1 < ntw; j++) {
    iteration(j, j & 1, std::true_type{}, st, s2);
#pragma unroll
    for (int nb = 0; nb < 2; nb++) st[nb] = s2[nb];
  }
  if (j < ntw) {                                         // this wavefront's last tile
    const unsigned char* sV = smem + (2 + (j & 1)) * TILE_BYTES;
    rescale();
    rs = 0.f;
    turn();
    unroll_for<FWD_D>([&](auto I) { read_frag(std::integral_constant<int, 16 + decltype(I)::value>{}, smem, sV); });
    if (j + 1 < ntiles) {
#pragma unroll
      for (int i = 0; i < 2 * NL; i++) next_loads(j, i);
    }
    softmax_to(st, std::integral_constant<int, 0>{}, std::integral_constant<int, 16>{});
    unroll_for<16>([&](auto I) {
      constexpr int s = 16 + decltype(I)::value;
      pv(std::integral_constant<int, s>{});
      if constexpr (s + FWD_D < 32) read_frag(std::integral_constant<int, s + FWD_D>{}, smem, sV);
      if constexpr (s < 24) softmax_to(st, std::integral_constant<int, 16 + (s - 16) * 2>{}, std::integral_constant<int, 18 + (s - 16) * 2>{});
    });
    lrun = lrun * alpha + rs;
    j++;
  }
  for (; j < ntiles; j++) {                              // nothing left for this wavefront but its share of the loads
    turn();
    if (j + 1 < ntiles) {
#pragma unroll
      for (int i = 0; i < 2 * NL; i++) next_loads(j, i);
    }
  }

  {
    const int qi = qw0 + (lane & 31);
    const float l = half_sum(lrun);
    if (qi < S) {
      store_acc_T(o + (tok0 + qi) * ld + head * HD, oacc, 1.f / l, lane);
      if (lane < 32) lse[((int64_t)b * H + head) * S + qi] = mrun * scale + logf(l);
    }
  }
  }  // pass
  wait_vm0();                                            // no load into LDS outlives the workgroup
}

// ----------------------------------------------------------------------------------------------
// D[b, head, q] = sum_h dO[q, h] * O[q, h] : 16 lanes per (token, head); also lse2 = lse * log2(e)
// ----------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void attn_dot_kernel(const uint16_t* __restrict__ dout, const uint16_t* __restrict__ o,
                                                       const float* __restrict__ lse, float* __restrict__ D,
                                                       float* __restrict__ lse2, int64_t ld, int S, int H,
                                                       int64_t total) {
  const int64_t item = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 4;   // (token, head) pair
  const int sub = threadIdx.x & 15;
  float s = 0.f;
  int64_t tok = 0;
  int head = 0;
  if (item < total) {
    tok = item / H;
    head = (int)(item % H);
    const int64_t off = tok * ld + head * HD + sub * 8;
    float a[8], bb[8];
    unpack8(*reinterpret_cast<const uint4*>(dout + off), a);
    unpack8(*reinterpret_cast<const uint4*>(o + off), bb);
#pragma unroll
    for (int i = 0; i < 8; i++) s = fmaf(a[i], bb[i], s);
  }
  s += __shfl_xor(s, 1);
  s += __shfl_xor(s, 2);
  s += __shfl_xor(s, 4);
  s += __shfl_xor(s, 8);
  if (item < total && sub == 0) {
    const int64_t bidx = tok / S, qi = tok % S;
    D[(bidx * H + head) * S + qi] = s;
    lse2[(bidx * H + head) * S + qi] = lse[(bidx * H + head) * S + qi] * LOG2E;   // exponent offset in base 2
  }
}

// ----------------------------------------------------------------------------------------------
// backward, dQ: workgroup owns NW x 32 queries, streams 64-key tiles of K and V
//
// Bound: instruction issue beside the MFMAs, and the LDS port (every operand read feeds one MFMA, as in the forward).  With 32
// queries a wavefront holds Q, dO, dQ and the scores of two 32-key blocks in 250 registers, so two of them share a SIMD, and the
// elements of one block are threaded between the MFMAs of the next block's S and dP and its own outputs (the kernels above do the
// same).  Four LDS stages: a tile's loads have two tiles' time to land; one barrier per tile.
// Only a wavefront's last block lies on the diagonal; it is the only one that is masked, outside the loop.
// Whole backward, us, 64 queries per wavefront, one wavefront per SIMD and one block after the other -> now: 2 x 2047 tokens, 32 / 8
// heads 315 -> 275 (this kernel 173 -> 125); 1 x 777, 32 / 8 heads 71.6 -> 63.5; 4 x 4095, 8 heads 502 -> 449; 13 x 641, 32 heads
// 496 -> 400; 1 x 3333, 16 heads 281 -> 195; 1 x 333, 32 / 8 heads 45.4 -> 41.4.
// ----------------------------------------------------------------------------------------------
constexpr int DQ_NS = 4;                                   // ring of key tiles: two in use, two on their way
constexpr int DQ_LDS = DQ_NS * 2 * TILE_BYTES;

constexpr int DQ_BAR = 5;       // slot of the barrier in the stage of a tile's first block
// elements of dS done by the end of slot s: their operands are whole when their MFMAs come (slots 16, 20)
constexpr int dq_elems(int s) { return s < 0 ? 0 : s < 20 ? 4 * (s + 1) / 5 : 16; }

// SCALED: dS is scaled before it is rounded, as where it is stored (attn_bwd_dkv_kernel): dQ then has the bits of the product that
// reads it there, whose order over the keys is this one.
template <int NW, bool SCALED>
__global__ __launch_bounds__(NW * 64, NW / 4) void attn_bwd_dq_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                                                          const uint16_t* __restrict__ v,
                                                          const uint16_t* __restrict__ dout,
                                                          const float* __restrict__ lse2, const float* __restrict__ D,
                                                          uint16_t* __restrict__ dq, int64_t ld, int64_t ldkv, int grp, int S, int H,
                                                          float scale) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int BQ = NW * 32, NL = 16 / NW;                // queries per block, 1 KB loads per wavefront, tile and operand
  constexpr int DQ_D = NW == 8 ? 4 : 8;                    // LDS operands are read this many MFMAs ahead (8 of 8 wavefronts: spills)
  // the wavefront index as a scalar: everything derived from it (LDS slots, tile rows) is scalar arithmetic
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nqb = (S + BQ - 1) / BQ;
  const WgCoord wg = wg_coord();
  const int head = wg.head, b = wg.b;
  const int64_t tok0 = (int64_t)b * S;
  const int64_t hoff = head * HD, kvoff = (head / grp) * HD;   // the key / value head this query head's group shares
  const float c = scale * LOG2E;
  // K is needed row-wise (S^T) and transposed (dQ^T), V row-wise (dP^T): one LDS copy each, in the
  // swizzle that serves both reads, written by direct-to-LDS loads.
  const rsrc_t rsK = rows_rsrc(k + tok0 * ldkv + kvoff, S, ldkv);
  const rsrc_t rsV = rows_rsrc(v + tok0 * ldkv + kvoff, S, ldkv);
  uint32_t offT[NL];
  {
    int row[NL];
    dma_lane_offsets<SWZ_BOTH, NL>(offT, row, ldkv, wave, lane);
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)LRB_LDS_PTR(smem) + (uint32_t)wave * 1024u;
  // Operand addresses inside a SWZ_BOTH tile (both_row_frag, both_tr_frag): the lane's part, from which the k16 step or the 32
  // columns differ by an XOR, and rows by a constant.
  uint32_t rowl, trl;
  {
    const int l31 = lane & 31, f = ((l31 & 3) << 2) | ((l31 >> 2) & 3), g = lane >> 4, s = lane & 15;
    rowl = (uint32_t)(l31 * 256 + (((lane >> 5) ^ f) << 4));
    trl = (uint32_t)(((g >> 1) * 4 + (s >> 2)) * 256 + ((((g & 1) * 2 + ((s & 3) >> 1)) ^ (((s >> 2) << 2) | (g >> 1))) << 4) + (s & 1) * 8);
  }
  // one query block from the late end and its mirror image from the early end: equal work per workgroup
  for (int pass = 0; pass < 2; pass++) {
  const int qblk = pass == 0 ? nqb - 1 - wg.x : wg.x;
  if (pass == 1 && ((int)gridDim.x == nqb || qblk >= nqb - 1 - wg.x)) break;   // (unpaired launch: see the forward)
  const int q0 = qblk * BQ;
  const int qw0 = q0 + wave * 32;
  const int ntiles = (min(S, q0 + BQ) + KT - 1) / KT;      // causal: keys up to the block's last query
  const int nb = qw0 < S ? qw0 / 32 + 1 : 0;               // 32-key blocks up to this wavefront's diagonal
  // load i of the 2 NL of key tile t (K, then V); a tile past the last one: every lane out of range, so that every tile costs
  // every wavefront the same number of loads
  auto dma = [&](int t, int i) {
    lds_dma_at(rsrc_from(i < NL ? rsK : rsV, (uint32_t)t * (uint32_t)(KT * 2) * (uint32_t)ldkv, t < ntiles),
               lds0 + (uint32_t)(t % DQ_NS) * (2 * TILE_BYTES) + (uint32_t)((i / NL) * TILE_BYTES + (i % NL) * NW * 1024), offT[i % NL]);
  };
  __syncthreads();                                         // the pass before is done with the ring

  // Q and dO rows of this wavefront stay in registers (B operands).
  bf16x8 qf[1][8], dof[1][8];
  load_row_frags<1>(qf, q + tok0 * ld + hoff, ld, qw0, S, lane);
  load_row_frags<1>(dof, dout + tok0 * ld + hoff, ld, qw0, S, lane);
  const int qi = qw0 + (lane & 31);                        // this lane's query
  const int64_t sidx = ((int64_t)b * H + head) * S + min(qi, S - 1);
  float lsq = lse2[sidx], Dq = D[sidx];
#pragma unroll
  for (int t = 0; t < 3; t++)
#pragma unroll
    for (int i = 0; i < 2 * NL; i++) dma(t, i);

  f32x16 acc[4];                                           // dQ^T
#pragma unroll
  for (int hb = 0; hb < 4; hb++)
#pragma unroll
    for (int e = 0; e < 16; e++) acc[hb][e] = 0.f;
  wait_vm<4 * NL>();                                       // the first of the three tiles has landed
  __builtin_amdgcn_s_barrier();
  asm volatile("" : "+v"(lsq), "+v"(Dq) : : "memory");     // (used here, so that no wait for them stays in the loop)

  struct Scores { f32x16 s, dp; };                         // rows = keys of a 32-key block, column = query: S^T and dP^T
  Scores sa, sb;                                           // of a tile's first and second block
  bf16x8 fr[DQ_D];                                         // operands read ahead, slot s in fr[s % DQ_D]
  uint32_t dw[8];                                          // dS as bf16 pairs: two operands
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  auto tile = [&](int t) -> uint32_t { return (uint32_t)(t % DQ_NS) * (2 * TILE_BYTES); };
  // operand of slot s: 0..15 the next block's rows (k16 step s / 2, K then V), 16..23 the current block's columns of K (16 keys
  // each four slots)
  auto read_frag = [&](auto Sc, uint32_t cur, auto CRB, uint32_t nxt, auto NRB) {
    constexpr int s = decltype(Sc)::value;
    if constexpr (s < 16) {
      fr[s % DQ_D] = lds_b128(smem + ((nxt + rowl) ^ (uint32_t)((s >> 1) << 5)) + (s & 1) * TILE_BYTES + decltype(NRB)::value * 8192);
    } else {
      typedef short s16x8 __attribute__((ext_vector_type(8)));
      constexpr int off = decltype(CRB)::value * 8192 + ((s - 16) >> 2) * 4096;
      const uint32_t at = (cur + trl) ^ (uint32_t)((s & 3) << 6);
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(smem + at + off));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(smem + (at ^ 32u) + off + 2048));
      const s16x8 r = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      fr[s % DQ_D] = __builtin_bit_cast(bf16x8, r);
    }
  };
  auto mfma = [&](auto Sc, Scores& nx) {
    constexpr int s = decltype(Sc)::value;
    constexpr f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const bf16x8 f = fr[s % DQ_D];
    if constexpr (s < 16) {
      if constexpr (s & 1) nx.dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, dof[0][s >> 1], s < 2 ? zero : nx.dp, 0, 0, 0);
      else nx.s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, qf[0][s >> 1], s < 2 ? zero : nx.s, 0, 0, 0);
    } else {
      constexpr int t = (s - 16) >> 2, hb = s & 3;
      const bf16x8 x = __builtin_bit_cast(bf16x8, make_uint4(dw[t * 4], dw[t * 4 + 1], dw[t * 4 + 2], dw[t * 4 + 3]));
      acc[hb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, x, acc[hb], 0, 0, 0);
    }
  };
  // elements F .. T - 1 of dS^T = P^T * (dP^T - D) of the current block, whose first key is kb0
  float dlow = 0.f;
  auto elements = [&](auto Fc, auto Tc, auto MASK, const Scores& x, int kb0) {
    constexpr int f = decltype(Fc)::value, t = decltype(Tc)::value;
    unroll_for<t - f>([&](auto I) {
      constexpr int e = f + decltype(I)::value;
      float p = fast_exp2(fmaf(x.s[e], c, -lsq));
      if constexpr (decltype(MASK)::value) p = kb0 + acc_row(e, lane) > qi ? 0.f : p;
      const float ds = (SCALED ? p * scale : p) * (x.dp[e] - Dq);
      if constexpr (e & 1) dw[e >> 1] = pack_bf16x2(dlow, ds);
      else dlow = ds;
    });
  };
  // this wavefront's loads of tile t + 1 have landed (behind them are the next tile's, and loads retire in order), then
  // everyone's, and everyone has left tile t - 1, whose slot is loaded anew
  auto meet = [&] {
    wait_vm<2 * NL>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // Elements and outputs of the current block (half CRB of tile t) with the scores of the next one (half 1 - CRB, tile t or
  // t + 1) between them.  The first operands were read by the stage before, and this one reads those of the stage after.
  auto stage = [&](int t, auto CRB, const Scores& cu, Scores& nx) {
    constexpr int crb = decltype(CRB)::value;
    using Other = std::integral_constant<int, crb ^ 1>;
    const uint32_t cur = tile(t), after = tile(t + 1);     // after: of the stage after, half 1 of tile t + 1, or half 0 of it
    const uint32_t nxt = crb ? after : cur;
    // Slots in pairs, the operand that was asked for last first: one wait serves both.
    unroll_for<12>([&](auto Uc) {
      constexpr int u = decltype(Uc)::value, s = 2 * u + 1;
      mfma(std::integral_constant<int, s>{}, nx);
      mfma(std::integral_constant<int, s - 1>{}, nx);
      if constexpr (crb == 0 && s == DQ_BAR) meet();
      unroll_for<2>([&](auto I) {
        constexpr int r = s - 1 + decltype(I)::value;
        if constexpr (crb == 0 && r > DQ_BAR && r <= DQ_BAR + 2 * NL) dma(t + 3, r - DQ_BAR - 1);
        if constexpr (r + DQ_D < 24) read_frag(std::integral_constant<int, r + DQ_D>{}, cur, CRB, nxt, Other{});
        else read_frag(std::integral_constant<int, r + DQ_D - 24>{}, cur, CRB, after, CRB);
      });
      elements(std::integral_constant<int, dq_elems(s - 2)>{}, std::integral_constant<int, dq_elems(s)>{}, std::false_type{}, cu, 0);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  // the diagonal block, at cur and from key kb0 on, whose scores are there
  auto last = [&](uint32_t cur, int kb0, const Scores& x) {
    Scores none;
    unroll_for<DQ_D>([&](auto I) { read_frag(std::integral_constant<int, 16 + decltype(I)::value>{}, cur, I0{}, cur, I0{}); });
    elements(I0{}, std::integral_constant<int, 8>{}, std::true_type{}, x, kb0);
    __builtin_amdgcn_sched_barrier(0);
    elements(std::integral_constant<int, 8>{}, std::integral_constant<int, 16>{}, std::true_type{}, x, kb0);
    __builtin_amdgcn_sched_barrier(0);
    unroll_for<8>([&](auto I) {
      constexpr int s = 16 + decltype(I)::value;
      mfma(std::integral_constant<int, s>{}, none);
      if constexpr (s + DQ_D < 24) read_frag(std::integral_constant<int, s + DQ_D>{}, cur, I0{}, cur, I0{});
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  int t = 0;
  if (nb > 0) {
    unroll_for<DQ_D>([&](auto I) { read_frag(I, 0, I0{}, 0, I0{}); });    // scores of the first block
    unroll_for<16>([&](auto Sc) {
      constexpr int s = decltype(Sc)::value;
      mfma(Sc, sa);
      if constexpr (s + DQ_D < 16) read_frag(std::integral_constant<int, s + DQ_D>{}, 0, I0{}, 0, I0{});
    });
    unroll_for<DQ_D>([&](auto I) { read_frag(I, 0, I0{}, 0, I1{}); });    // (unused where there is no second block)
    for (; 2 * t + 2 < nb; t++) {
      stage(t, I0{}, sa, sb);
      stage(t, I1{}, sb, sa);
    }
    const int odd = 2 * t + 1 < nb;                        // one more block before the diagonal
    if (odd) {
      stage(t, I0{}, sa, sb);
      sa = sb;
    } else {
      meet();
#pragma unroll
      for (int i = 0; i < 2 * NL; i++) dma(t + 3, i);
    }
    __builtin_amdgcn_sched_barrier(0);
    last(tile(t) + (uint32_t)odd * 8192u, t * KT + odd * 32, sa);
    t++;
  }
  for (; t < ntiles; t++) {                                // nothing left for this wavefront but its share of the loads
    meet();
#pragma unroll
    for (int i = 0; i < 2 * NL; i++) dma(t + 3, i);
  }
  if (qi < S) store_acc_T(dq + (tok0 + qi) * ld + hoff, acc, SCALED ? 1.f : scale, lane);
  }  // pass
  wait_vm0();                                              // no load into LDS outlives the workgroup
}

// ----------------------------------------------------------------------------------------------
// backward, dK and dV: workgroup owns 4 x 32 keys, streams 64-query tiles of Q and dO
// ----------------------------------------------------------------------------------------------
constexpr int DKV_STAGE = 2 * TILE_BYTES + 2 * KT * 4;     // Q tile, dO tile, lse2[64], D[64]
constexpr int DKV_LDS = 2 * DKV_STAGE;

// NB 32-key blocks per wavefront: every Q / dO operand read from LDS feeds NB MFMAs.  With NB = 1 the
// four wavefronts together need 128 bytes of LDS operands per clock to keep the matrix pipes busy,
// which is all the LDS delivers; NB = 2 halves that (the accumulators then fill the AGPR file).
// WRITE_DS: the kernel also leaves scale * dS^T, as bf16 [key][query] per (batch, head), in `dst`; the
// query gradient is then one k-major GEMM dQ = (scale dS^T)^T K over it, instead of a second kernel
// that forms S, dP and dS all over again.  Everything a row tile of that GEMM reads is written here:
// key k's row holds every query from 256 * floor(k / 256) on, zeros where the query precedes the key.
template <int NB, bool WRITE_DS>
__global__ __launch_bounds__(256) void attn_bwd_dkv_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                                                           const uint16_t* __restrict__ v,
                                                           const uint16_t* __restrict__ dout,
                                                           const float* __restrict__ lse2, const float* __restrict__ D,
                                                           uint16_t* __restrict__ dk, uint16_t* __restrict__ dv,
                                                           uint16_t* __restrict__ dst, int64_t ld, int64_t ldkv, int64_t lddkv, int grp, int S, int H,
                                                           float scale) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int BN = 4 * NB * 32;
  // the wavefront index as a scalar: everything derived from it (LDS slots, tile rows) is scalar arithmetic
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nkb = (S + BN - 1) / BN;
  const WgCoord wg = wg_coord();
  const int head = wg.head, b = wg.b;
  const int64_t tok0 = (int64_t)b * S;
  const int64_t hoff = head * HD;
  const float c = scale * LOG2E;
  // Q and dO tiles are needed row-wise (S, dP) and transposed (dK^T, dV^T): one LDS copy each, in the
  // swizzle that serves both reads, written by direct-to-LDS loads.
  const rsrc_t rsQ = tile_rsrc(q + tok0 * ld + hoff);
  const rsrc_t rsO = tile_rsrc(dout + tok0 * ld + hoff);
  const rsrc_t rsL = make_rsrc(lse2 + ((int64_t)b * H + head) * S, (uint32_t)S * 4u);
  const rsrc_t rsD = make_rsrc(D + ((int64_t)b * H + head) * S, (uint32_t)S * 4u);
  uint32_t offT[4];
  int rowT[4];
  dma_lane_offsets<SWZ_BOTH, 4>(offT, rowT, ld, wave, lane);
  // all loads of one 64-query tile: 4 + 4 tile loads per wavefront; wavefronts 0 and 1 also fetch the
  // tile's 64 row scalars (out-of-range rows read as zeros: the resource ends at S)
  auto dma_stage = [&](int st, int j) {
    unsigned char* p = smem + st * DKV_STAGE;
    dma_tile<4>(rsQ, p, offT, rowT, j * KT, S, ld, wave);
    dma_tile<4>(rsO, p + TILE_BYTES, offT, rowT, j * KT, S, ld, wave);
    if (wave == 0)
      lds_dma<4>(rsL, p + 2 * TILE_BYTES, (uint32_t)(j * KT + lane) * 4u);
    if (wave == 1)
      lds_dma<4>(rsD, p + 2 * TILE_BYTES + KT * 4, (uint32_t)(j * KT + lane) * 4u);
  };

  // one key block from the early end (most queries) and its mirror image from the late end: equal
  // work per workgroup
  // dS^T of this (batch, head): S rows of S bf16.  A packed k16 fragment holds, for the lane's key row,
  // queries 4h..4h+3 and 8+4h..8+4h+3 (h = lane / 32); lanes l and l + 32 exchange one half each, after
  // which a lane owns 8 consecutive queries and stores them with one 16-byte access.  Rows past S fall
  // outside the resource, queries past S (a multiple of 8) are given an offset that does.
  const __amdgpu_buffer_rsrc_t rsS = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(WRITE_DS ? dst + ((int64_t)b * H + head) * S * S : nullptr), 0, WRITE_DS ? (uint32_t)S * (uint32_t)S * 2u : 0u,
      0x00020000);
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  auto store_ds = [&](const bf16x8& f, int key, int q16) {
    const uint4 w = __builtin_bit_cast(uint4, f);
    // swap(a, b): lanes 32..63 of a <-> lanes 0..31 of b
    const auto sx = __builtin_amdgcn_permlane32_swap(w.x, w.z, false, false);
    const auto sy = __builtin_amdgcn_permlane32_swap(w.y, w.w, false, false);
    const int q0 = q16 + 8 * (lane >> 5);
    const uint32_t o = q0 < S ? (uint32_t)key * (uint32_t)S * 2u + (uint32_t)q0 * 2u : DMA_OOB;
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{sx[0], sy[0], sx[1], sy[1]}, rsS, (int)o, 0, 0);
  };
  const bf16x8 zero_frag = __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0));

  for (int pass = 0; pass < 2; pass++) {
  const int kblk = pass == 0 ? wg.x : nkb - 1 - wg.x;
  if (pass == 1 && ((int)gridDim.x == nkb || kblk <= wg.x)) break;   // (unpaired launch: see the forward)
  const int n0 = kblk * BN;
  const int nw0 = n0 + wave * NB * 32;
  if constexpr (WRITE_DS) {
    // queries between the start of the enclosing 256-row tile and this key block: zeros
    for (int qz = (n0 / 256) * 256; qz < n0; qz += 16)
#pragma unroll
      for (int nb = 0; nb < NB; nb++) store_ds(zero_frag, nw0 + nb * 32 + (lane & 31), qz);
  }

  // K and V rows of this wavefront stay in registers (B operands).
  bf16x8 kf[NB][8], vf[NB][8];
  // (grouped-query attention: the group's shared key / value head, rows of ldkv; dk and dv below are
  // this query head's contribution, laid out like q)
  load_row_frags<NB>(kf, k + tok0 * ldkv + (head / grp) * HD, ldkv, nw0, S, lane);
  load_row_frags<NB>(vf, v + tok0 * ldkv + (head / grp) * HD, ldkv, nw0, S, lane);

  f32x16 akv[2][NB][4];                                    // [0] = dK^T, [1] = dV^T
#pragma unroll
  for (int w = 0; w < 2; w++)
#pragma unroll
    for (int nb = 0; nb < NB; nb++)
#pragma unroll
      for (int hb = 0; hb < 4; hb++)
#pragma unroll
        for (int e = 0; e < 16; e++) akv[w][nb][hb][e] = 0.f;

  const int jbeg = n0 / KT;                                // causal: first query tile that sees key n0
  const int jend = (S + KT - 1) / KT;
  dma_stage(0, jbeg);
  wait_vm0();
  __syncthreads();

  for (int j = jbeg; j < jend; j++) {
    const int cur = (j - jbeg) & 1;
    if (j + 1 < jend) dma_stage(cur ^ 1, j + 1);           // lands while this tile is worked on
    const unsigned char* sQ = smem + cur * DKV_STAGE;
    const unsigned char* sO = sQ + TILE_BYTES;
    const float* sl = reinterpret_cast<const float*>(sO + TILE_BYTES);
    const float* sd = sl + KT;
    const int qt0 = j * KT;
    // one 32-query block at a time; blocks entirely before this wavefront's keys are skipped, blocks
    // entirely after them need no mask
#pragma unroll 1
    for (int qb2 = 0; qb2 < 2; qb2++) {
      const int qb0 = qt0 + qb2 * 32;
      if (qb0 + 31 < nw0 || qb0 >= S) {
        if constexpr (WRITE_DS) {   // not computed, but a row tile of the dQ GEMM reads it: zeros
#pragma unroll
          for (int t = 0; t < 2; t++)
#pragma unroll
            for (int nb = 0; nb < NB; nb++) store_ds(zero_frag, nw0 + nb * 32 + (lane & 31), qb0 + t * 16);
        }
        continue;
      }
      f32x16 st[NB], dp[NB];                               // rows = queries, column = key
#pragma unroll
      for (int nb = 0; nb < NB; nb++)
#pragma unroll
        for (int e = 0; e < 16; e++) { st[nb][e] = 0.f; dp[nb][e] = 0.f; }
#pragma unroll
      for (int ks = 0; ks < 8; ks++) {
        const bf16x8 qfr = both_row_frag(sQ, qb2 * 32, ks, lane), dfr = both_row_frag(sO, qb2 * 32, ks, lane);
#pragma unroll
        for (int nb = 0; nb < NB; nb++) {
          st[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qfr, kf[nb][ks], st[nb], 0, 0, 0);
          dp[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dfr, vf[nb][ks], dp[nb], 0, 0, 0);
        }
      }
      float4 slv[4], sdv[4];                               // rows 8 g + 4 (lane / 32) + 0..3, g = 0..3
#pragma unroll
      for (int g4 = 0; g4 < 4; g4++) {
        slv[g4] = *reinterpret_cast<const float4*>(sl + qb2 * 32 + 8 * g4 + 4 * (lane >> 5));
        sdv[g4] = *reinterpret_cast<const float4*>(sd + qb2 * 32 + 8 * g4 + 4 * (lane >> 5));
      }
      const bool need_mask = (qb0 < nw0 + NB * 32 - 1) || (qb0 + 32 > S);
      // the element loop exists twice, with and without the mask, under one wavefront-uniform branch
      // (left to the compiler, the test was repeated per element and split the loop into 16 blocks)
      auto elements = [&](auto MASKED) {
#pragma unroll
        for (int nb = 0; nb < NB; nb++) {
          const int ni = nw0 + nb * 32 + (lane & 31);
#pragma unroll
          for (int e = 0; e < 16; e++) {
            const float lv = e % 4 == 0 ? slv[e / 4].x : e % 4 == 1 ? slv[e / 4].y : e % 4 == 2 ? slv[e / 4].z : slv[e / 4].w;
            const float dvv = e % 4 == 0 ? sdv[e / 4].x : e % 4 == 1 ? sdv[e / 4].y : e % 4 == 2 ? sdv[e / 4].z : sdv[e / 4].w;
            float p = fast_exp2(fmaf(st[nb][e], c, -lv));
            if constexpr (decltype(MASKED)::value) {
              const int qi = qb0 + acc_row(e, lane);
              p = (ni > qi || qi >= S) ? 0.f : p;
            }
            st[nb][e] = p;                                   // P
            if constexpr (WRITE_DS) dp[nb][e] = (p * scale) * (dp[nb][e] - dvv);   // scale * dS
            else dp[nb][e] = p * (dp[nb][e] - dvv);          // dS
          }
        }
      };
      if (need_mask) {
        asm volatile("" ::: "memory");
        elements(std::true_type{});
      } else {
        elements(std::false_type{});
      }
#pragma unroll
      for (int t = 0; t < 2; t++) {
        bf16x8 pf[NB], dsf[NB];
#pragma unroll
        for (int nb = 0; nb < NB; nb++) { pf[nb] = pack_acc_half(st[nb], t); dsf[nb] = pack_acc_half(dp[nb], t); }
        if constexpr (WRITE_DS) {
#pragma unroll
          for (int nb = 0; nb < NB; nb++) store_ds(dsf[nb], nw0 + nb * 32 + (lane & 31), qb0 + t * 16);
        }
#pragma unroll
        for (int hb = 0; hb < 4; hb++) {
          const bf16x8 dtf = both_tr_frag(sO, qb2 * 32 + t * 16, hb * 32, lane);
          const bf16x8 qtf = both_tr_frag(sQ, qb2 * 32 + t * 16, hb * 32, lane);
#pragma unroll
          for (int nb = 0; nb < NB; nb++) {
            akv[1][nb][hb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dtf, pf[nb], akv[1][nb][hb], 0, 0, 0);
            akv[0][nb][hb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qtf, dsf[nb], akv[0][nb][hb], 0, 0, 0);
          }
        }
      }
    }
    // The next tile's loads were issued before this tile's dS^T stores (4 * NB per wavefront, issued on
    // every path) and memory operations retire in order: waiting until at most that many are
    // outstanding covers the loads without waiting for the stores to be acknowledged.
    if constexpr (WRITE_DS) wait_vm<4 * NB>();
    else wait_vm0();
    __syncthreads();
  }
#pragma unroll
  for (int nb = 0; nb < NB; nb++) {
    const int ni = nw0 + nb * 32 + (lane & 31);
    if (ni < S) {
      store_acc_T(dk + (tok0 + ni) * lddkv + hoff, akv[0][nb], WRITE_DS ? 1.f : scale, lane);
      store_acc_T(dv + (tok0 + ni) * lddkv + hoff, akv[1][nb], 1.f, lane);
    }
  }
  }  // pass
}

// ----------------------------------------------------------------------------------------------
// The same for long sequences without the score gradient: the elementwise work of a 32-query block threaded between the
// MFMAs of the next block's S and dP and its own outputs, two MFMAs and a share of it per pair of slots.
//
// Bound: instruction issue.  One wavefront per SIMD (its accumulators and K / V operands take 240 registers) issues an
// instruction every four cycles at best, about 310 of them per block for 32 MFMAs of 32 cycles each; what was lost beside that was the
// wait for the phases of a block to follow each other.  Four LDS stages, so that a tile's loads have two tiles' time to
// land; the diagonal tiles, the last one and anything shorter than three full tiles go one block at a time.
// Backward, us, before -> now: 2 x 2047 tokens, 32 / 8 heads 345 -> 327; 2 x 3333, 16 / 4 heads 484 -> 439; 4 x 1501, 16 heads
// 260 -> 247; 777, 32 / 8 heads 129.5 -> 125.8; below that it is slower (4 x 300, 8 heads 64 -> 67), and with the score gradient
// stored as well, where the dQ product waits on memory, the whole backward gained nothing at 2048 tokens (628 / 628).
// Paired key blocks share a CU's time with others, and there it takes longer sequences to pay (whole backward, this kernel against the
// other: 8 x 779 tokens, 32 heads +3.3 %, 4 x 923, 32 / 8 heads +2.6, 6 x 1045, 32 / 8 heads -2.5, 8 x 1129, 32 heads -1.7;
// a workgroup per block: 14 x 774, 1 head -6.3, 14 x 943, 2 heads -6.1).
// ----------------------------------------------------------------------------------------------
constexpr int LDKV_MIN_S = 768, LDKV_MIN_S_PAIRED = 1024;
constexpr int LDKV_NS = 4;                                 // ring of stages: two tiles in use, two on their way
constexpr int LDKV_LDS = LDKV_NS * DKV_STAGE + KT * 4;     // (and a place for what nobody reads)
constexpr int DKV_D = 8;        // LDS operands are read this many MFMAs ahead
constexpr int DKV_BAR = 5;      // slot of the barrier in the stage of a tile's first block
// elements of P and dS done by the end of slot s: their operands are whole when their MFMAs come (slots 16, 24)
constexpr int dkv_elems(int s) { return s < 0 ? 0 : s < 16 ? 5 * (s + 1) / 8 : s < 22 ? s - 5 : 16; }

__global__ __launch_bounds__(256) void attn_bwd_dkv_long_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                                                           const uint16_t* __restrict__ v,
                                                           const uint16_t* __restrict__ dout,
                                                           const float* __restrict__ lse2, const float* __restrict__ D,
                                                           uint16_t* __restrict__ dk, uint16_t* __restrict__ dv,
                                                           int64_t ld, int64_t ldkv, int64_t lddkv, int grp, int S, int H, float scale) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int BN = 128;
  // the wavefront index as a scalar: everything derived from it (LDS slots, tile rows) is scalar arithmetic
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nkb = (S + BN - 1) / BN;
  const WgCoord wg = wg_coord();
  const int head = wg.head, b = wg.b;
  const int64_t tok0 = (int64_t)b * S;
  const int64_t hoff = head * HD;
  const float c = scale * LOG2E;
  // Q and dO tiles are needed row-wise (S, dP) and transposed (dK^T, dV^T): one LDS copy each, in the
  // swizzle that serves both reads, written by direct-to-LDS loads.
  const rsrc_t rsQ = rows_rsrc(q + tok0 * ld + hoff, S, ld);
  const rsrc_t rsO = rows_rsrc(dout + tok0 * ld + hoff, S, ld);
  const rsrc_t rsLD = make_rsrc((wave == 0 ? lse2 : D) + ((int64_t)b * H + head) * S, wave < 2 ? (uint32_t)S * 4u : 0u);
  uint32_t offT[4];
  {
    int row[4];
    dma_lane_offsets<SWZ_BOTH, 4>(offT, row, ld, wave, lane);
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)LRB_LDS_PTR(smem);
  const int jend = (S + KT - 1) / KT;
  // Load i of the 9 of 64-query tile j (4 of Q, 4 of dO; the ninth fetches the tile's 64 row scalars: lse2 by wavefront 0, D by
  // wavefront 1, nothing by the others).  Rows past S, and whole tiles past it, read as zeros: no branches, and every tile
  // costs every wavefront the same number of loads.
  auto dma = [&](int slot, int j, int i) {
    const bool valid = j < jend;
    const uint32_t p = lds0 + (uint32_t)slot * DKV_STAGE;
    const uint32_t off = (uint32_t)j * (uint32_t)(KT * 2) * (uint32_t)ld;
    if (i < 4) lds_dma_at(rsrc_from(rsQ, off, valid), p + (uint32_t)(i * 4 + wave) * 1024u, offT[i]);
    else if (i < 8) lds_dma_at(rsrc_from(rsO, off, valid), p + TILE_BYTES + (uint32_t)((i - 4) * 4 + wave) * 1024u, offT[i - 4]);
    else lds_dma4_at(rsLD, wave < 2 ? p + 2 * TILE_BYTES + (uint32_t)wave * (KT * 4) : lds0 + LDKV_NS * DKV_STAGE, (uint32_t)(j * KT + lane) * 4u);
  };

  // one key block from the early end (most queries) and its mirror image from the late end: equal
  // work per workgroup
  for (int pass = 0; pass < 2; pass++) {
  const int kblk = pass == 0 ? wg.x : nkb - 1 - wg.x;
  if (pass == 1 && ((int)gridDim.x == nkb || kblk <= wg.x)) break;   // (unpaired launch: see the forward)
  const int n0 = kblk * BN;
  const int nw0 = n0 + wave * 32;
  const int ni = nw0 + (lane & 31);                        // this lane's key
  __syncthreads();                                         // the pass before is done with the ring

  // K and V rows of this wavefront stay in registers (B operands).
  bf16x8 kf[1][8], vf[1][8];
  // (grouped-query attention: the group's shared key / value head, rows of ldkv; dk and dv below are
  // this query head's contribution, laid out like q)
  load_row_frags<1>(kf, k + tok0 * ldkv + (head / grp) * HD, ldkv, nw0, S, lane);
  load_row_frags<1>(vf, v + tok0 * ldkv + (head / grp) * HD, ldkv, nw0, S, lane);

  f32x16 akv[2][4];                                        // [0] = dK^T, [1] = dV^T
#pragma unroll
  for (int w = 0; w < 2; w++)
#pragma unroll
    for (int hb = 0; hb < 4; hb++)
#pragma unroll
      for (int e = 0; e < 16; e++) akv[w][hb][e] = 0.f;

  const int jbeg = n0 / KT;                                // causal: first query tile that sees key n0
  const int nt = jend - jbeg;
#pragma unroll
  for (int t = 0; t < 3; t++)
#pragma unroll
    for (int i = 0; i < 9; i++) dma(t, jbeg + t, i);
  wait_vm<18>();                                           // the first of the three tiles has landed
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");

  struct Scores { f32x16 s, dp; };                         // rows = queries of a 32-query block, column = key: S and dP, then P and dS
  Scores sa, sb;                                           // of a tile's first and second block
#pragma unroll
  for (int e = 0; e < 16; e++) { sa.s[e] = 0.f; sa.dp[e] = 0.f; sb.s[e] = 0.f; sb.dp[e] = 0.f; }
  bf16x8 fr[DKV_D];                                        // operands read ahead, slot s in fr[s % DKV_D]
  float4 slv[4], sdv[4];                                   // lse2 and D of the current block: rows 8 g + 4 (lane / 32) + 0..3
  uint32_t pw[8], dw[8];                                   // P and dS as bf16 pairs: two operands each

  auto tile = [&](int t) -> const unsigned char* { return smem + (t % LDKV_NS) * DKV_STAGE; };   // t: tile of this pass
  auto read_scalars = [&](auto Gc, const unsigned char* tp, int rb) {
    constexpr int g4 = decltype(Gc)::value;
    const float* sl = reinterpret_cast<const float*>(tp + 2 * TILE_BYTES);
    if constexpr (g4 < 4) slv[g4] = *reinterpret_cast<const float4*>(sl + rb * 32 + 8 * g4 + 4 * (lane >> 5));
    else sdv[g4 - 4] = *reinterpret_cast<const float4*>(sl + KT + rb * 32 + 8 * (g4 - 4) + 4 * (lane >> 5));
  };
  // operand of slot s: 0..15 the next block's rows (k16 step s / 2, Q then dO), 16..31 the current block's columns
  // (16 queries each eight slots, 32 columns each two, dO then Q)
  auto read_frag = [&](auto Sc, const unsigned char* cur, int crb, const unsigned char* nxt, int nrb) {
    constexpr int s = decltype(Sc)::value;
    if constexpr (s < 16) fr[s % DKV_D] = both_row_frag(nxt + (s & 1) * TILE_BYTES, nrb * 32, s >> 1, lane);
    else fr[s % DKV_D] = both_tr_frag(cur + ((s & 1) ^ 1) * TILE_BYTES, crb * 32 + ((s - 16) >> 3) * 16, ((s >> 1) & 3) * 32, lane);
  };
  auto mfma = [&](auto Sc, Scores& nx) {
    constexpr int s = decltype(Sc)::value;
    const bf16x8 f = fr[s % DKV_D];
    if constexpr (s < 16) {
      if constexpr (s & 1) nx.dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, vf[0][s >> 1], nx.dp, 0, 0, 0);
      else nx.s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, kf[0][s >> 1], nx.s, 0, 0, 0);
    } else {
      constexpr int t = (s - 16) >> 3, hb = (s >> 1) & 3, w = (s & 1) ^ 1;
      const uint32_t* x = w ? pw : dw;
      const bf16x8 pf = __builtin_bit_cast(bf16x8, make_uint4(x[t * 4], x[t * 4 + 1], x[t * 4 + 2], x[t * 4 + 3]));
      akv[w][hb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, pf, akv[w][hb], 0, 0, 0);
    }
  };
  auto clear = [&](Scores& x) {
#pragma unroll
    for (int e = 0; e < 16; e++) { x.s[e] = 0.f; x.dp[e] = 0.f; }
  };
  // elements F .. T - 1 of the current block, whose first query is qb0
  float plow = 0.f, dlow = 0.f;
  auto elements = [&](auto Fc, auto Tc, auto MASK, const Scores& x, int qb0) {
    constexpr int f = decltype(Fc)::value, t = decltype(Tc)::value;
    unroll_for<t - f>([&](auto I) {
      constexpr int e = f + decltype(I)::value, g = e >> 2, r = e & 3;
      const float lv = r == 0 ? slv[g].x : r == 1 ? slv[g].y : r == 2 ? slv[g].z : slv[g].w;
      const float dvv = r == 0 ? sdv[g].x : r == 1 ? sdv[g].y : r == 2 ? sdv[g].z : sdv[g].w;
      float p = fast_exp2(fmaf(x.s[e], c, -lv));
      if constexpr (decltype(MASK)::value) {
        const int qi = qb0 + acc_row(e, lane);
        p = (ni > qi || qi >= S) ? 0.f : p;
      }
      const float ds = p * (x.dp[e] - dvv);
      if constexpr (e & 1) {
        pw[e >> 1] = pack_bf16x2(plow, p);
        dw[e >> 1] = pack_bf16x2(dlow, ds);
      } else {
        plow = p;
        dlow = ds;
      }
    });
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;

  // Elements and outputs of the current block (of tile t, half crb) with the scores of the next one (half 1 - crb, tile t or
  // t + 1) between them.  The first operands and the scalars were read by the stage before, and this one reads those of the
  // stage after; the stage of a tile's first half holds its barrier and the loads of the tile after next but one.
  auto stage = [&](int t, auto CRB, const Scores& cu, Scores& nx) {
    constexpr int crb = decltype(CRB)::value;
    constexpr bool bar = crb == 0;
    const unsigned char* cur = tile(t);
    const unsigned char* nxt = crb ? tile(t + 1) : cur;
    const unsigned char* after = tile(t + 1);              // of the stage after: half 1 of tile t + 1, or half 0 of it
    const int qb0 = (jbeg + t) * KT + crb * 32;
    clear(nx);
    // Slots in pairs, the operand that was asked for last first: one wait serves both.
    unroll_for<16>([&](auto Uc) {
      constexpr int u = decltype(Uc)::value, s = 2 * u + 1;
      mfma(std::integral_constant<int, s>{}, nx);
      mfma(std::integral_constant<int, s - 1>{}, nx);
      if constexpr (bar && s == DKV_BAR) {
        // All loads of tile t + 1 have landed (behind them are the next tile's nine, and loads retire in order).  Everyone
        // has left tile t - 1, whose slot is loaded anew.
        wait_vm<9>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      }
      unroll_for<2>([&](auto I) {
        constexpr int r = s - 1 + decltype(I)::value;
        if constexpr (bar && r > DKV_BAR && r <= DKV_BAR + 9) dma((t + 3) % LDKV_NS, jbeg + t + 3, r - DKV_BAR - 1);
        if constexpr (r + DKV_D < 32) read_frag(std::integral_constant<int, r + DKV_D>{}, cur, crb, nxt, crb ^ 1);
        else read_frag(std::integral_constant<int, r + DKV_D - 32>{}, cur, crb, after, crb);
        if constexpr (r >= 23 && r < 31) read_scalars(std::integral_constant<int, r - 23>{}, nxt, crb ^ 1);
      });
      elements(std::integral_constant<int, dkv_elems(s - 2)>{}, std::integral_constant<int, dkv_elems(s)>{}, std::false_type{}, cu, qb0);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  // one block at a time: its scores,
  auto scores = [&](const unsigned char* tp, int rb, Scores& x) {
    clear(x);
    unroll_for<DKV_D>([&](auto I) { read_frag(I, tp, 0, tp, rb); });
    unroll_for<16>([&](auto Sc) {
      constexpr int s = decltype(Sc)::value;
      mfma(Sc, x);
      if constexpr (s + DKV_D < 16) read_frag(std::integral_constant<int, s + DKV_D>{}, tp, 0, tp, rb);
    });
  };
  // then its elements and outputs
  auto outputs = [&](const unsigned char* tp, int rb, int qb0, Scores& x) {
    unroll_for<8>([&](auto G) { read_scalars(G, tp, rb); });
    unroll_for<DKV_D>([&](auto I) { read_frag(std::integral_constant<int, 16 + decltype(I)::value>{}, tp, rb, tp, 0); });
    elements(I0{}, std::integral_constant<int, 16>{}, std::true_type{}, x, qb0);
    unroll_for<16>([&](auto I) {
      constexpr int s = 16 + decltype(I)::value;
      mfma(std::integral_constant<int, s>{}, x);
      if constexpr (s + DKV_D < 32) read_frag(std::integral_constant<int, s + DKV_D>{}, tp, rb, tp, 0);
    });
  };

  for (int t = 0; t < nt;) {
    if (t >= 2 && t + 3 < nt) {
      // full tiles behind every wavefront's diagonal (three blocks in) and before the last; three of them at least, since the
      // accumulators change registers on the way in and out
      scores(tile(t), 0, sa);
      unroll_for<8>([&](auto G) { read_scalars(G, tile(t), 0); });
      unroll_for<DKV_D>([&](auto I) { read_frag(I, tile(t), 0, tile(t), 1); });
      do {
        stage(t, I0{}, sa, sb);
        stage(t, I1{}, sb, sa);
        t++;
      } while (t + 1 < nt);
      continue;
    }
    wait_vm<9>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < 9; i++) dma((t + 3) % LDKV_NS, jbeg + t + 3, i);
#pragma unroll 1
    for (int rb = 0; rb < 2; rb++) {
      const int qb0 = (jbeg + t) * KT + rb * 32;
      if (qb0 + 31 < nw0 || qb0 >= S) continue;            // before this wavefront's keys, or not there
      scores(tile(t), rb, sa);
      outputs(tile(t), rb, qb0, sa);
    }
    t++;
  }
  if (ni < S) {
    store_acc_T(dk + (tok0 + ni) * lddkv + hoff, akv[0], scale, lane);
    store_acc_T(dv + (tok0 + ni) * lddkv + hoff, akv[1], 1.f, lane);
  }
  }  // pass
  wait_vm0();                                              // no load into LDS outlives the workgroup
}

// ----------------------------------------------------------------------------------------------
// backward, dK and dV by pairs of wavefronts that share KB blocks of 32 keys and walk 32-query blocks together, one forming S, P and dV,
// the other dP, dS and dK: 256 keys per workgroup where the score gradient is formed twice and there is work for the chip (dkv_pairs
// below), 128 where it is stored and a workgroup has a CU to itself
//
// Bound: what one wavefront of a SIMD does while the other's MFMAs run.  A wavefront that does all of a key block's work holds dK,
// dV, K and V of 32 keys (192 registers): it is alone on its SIMD, its MFMAs and its vector arithmetic follow each other (matrix pipes
// 35 % busy in the kernel above), and each MFMA needs an operand of its own from LDS.  Split by what is formed, a wavefront holds one
// of dK and dV and one of K and V, and that of 64 keys (192 registers again): every operand read from LDS feeds two MFMAs, and the
// wavefronts w and w + 4 of a pair sit on one SIMD.  What passes between them is P, as the fp32 values that dS is formed
// from (8 KB per block, twice buffered): one barrier per block.  The sums over queries and over h are those of the other
// dK / dV kernels, in the same order: the same bits.
// Whole backward, us, the other kernels -> this one: 2 x 2047 tokens, 32 / 8 heads 338 -> 308; 2 x 1501, 32 heads 245 -> 224; 4 x 4095, 8
// heads 524 -> 497; 1 x 12001, 8 heads 1237 -> 1147; 16 x 300, 16 heads 115 -> 101; 16 x 500, 32 heads 327 -> 316.
// With the score gradient stored as well the stores were what 256 keys waited for (8 x 2048, 16 heads 621 -> 634): not done.  128
// keys leave registers for a read-ahead of six operands (of two: 1 x 4096 tokens, 4 heads 166 -> 169) and wait for the stores of
// three blocks before only.
// ----------------------------------------------------------------------------------------------
constexpr int PAIR_NS = 5;                                       // ring of 32-query blocks: one or two in use, three on their way
constexpr int PAIR_BLOCK = 2 * 32 * HD * 2 + 512;                // Q rows, dO rows, lse2, D (64 entries each, 32 used)
constexpr int PAIR_X = PAIR_NS * PAIR_BLOCK;                     // P of the four pairs, two blocks
constexpr int PAIR_NONE = PAIR_X + 2 * 4 * 8192;                 // a place for what nobody reads
constexpr int PAIR_LDS = PAIR_NONE + 256;
static_assert(PAIR_BLOCK % 256 == 0 && PAIR_LDS <= 160 * 1024, "LDS of a CU");

template <int KB, bool SCALED, bool WRITE_DS>
__global__ __launch_bounds__(512) void attn_bwd_dkv_pair_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                                                                const uint16_t* __restrict__ v, const uint16_t* __restrict__ dout,
                                                                const float* __restrict__ lse2, const float* __restrict__ D,
                                                                uint16_t* __restrict__ dk, uint16_t* __restrict__ dv,
                                                                uint16_t* __restrict__ dst, int64_t ld, int64_t ldkv, int64_t lddkv, int grp, int S, int H,
                                                                float scale) {
  extern __shared__ __attribute__((aligned(256))) unsigned char smem[];
  static_assert(!WRITE_DS || SCALED, "what is stored is scaled");
  constexpr int BN = 128 * KB;
  constexpr int PAIR_D = KB == 2 ? 2 : 6;                  // LDS operands are read this many groups of KB MFMAs ahead
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pair = wave & 3;
  const bool second = wave >= 4;                           // dP, dS, dK; otherwise S, P, dV
  const int nkb = (S + BN - 1) / BN;
  const WgCoord wg = wg_coord();
  const int head = wg.head, b = wg.b;
  const int64_t tok0 = (int64_t)b * S, hoff = head * HD, kvoff = (head / grp) * HD;
  const float c = scale * LOG2E;
  const rsrc_t rsQ = rows_rsrc(q + tok0 * ld + hoff, S, ld);
  const rsrc_t rsO = rows_rsrc(dout + tok0 * ld + hoff, S, ld);
  const rsrc_t rsLD = make_rsrc((wave == 0 ? lse2 : D) + ((int64_t)b * H + head) * S, (wave & 3) == 0 ? (uint32_t)S * 4u : 0u);
  uint32_t offT[2];
  {
    int row[2];
    dma_lane_offsets<SWZ_BOTH, 2>(offT, row, ld, wave, lane);
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)LRB_LDS_PTR(smem);
  const int qblocks = (S + 31) / 32;
  // The three loads of a wavefront for 32-query block qb (of the sequence): four rows of Q, four of dO, the scalars or nothing.
  // Rows past S, and whole blocks past it, read as zeros.
  auto dma = [&](int slot, int qb) {
    const bool valid = qb < qblocks;
    const uint32_t p = lds0 + (uint32_t)slot * PAIR_BLOCK, off = (uint32_t)qb * 64u * (uint32_t)ld;
    lds_dma_at(rsrc_from(rsQ, off, valid), p + (uint32_t)wave * 1024u, offT[0]);
    lds_dma_at(rsrc_from(rsO, off, valid), p + 8192u + (uint32_t)wave * 1024u, offT[0]);
    lds_dma4_at(rsLD, (wave & 3) == 0 ? p + 16384u + (uint32_t)(wave >> 2) * 256u : lds0 + PAIR_NONE, (uint32_t)(qb * 32 + lane) * 4u);
  };
  // dS^T of this (batch, head), see attn_bwd_dkv_kernel
  const __amdgpu_buffer_rsrc_t rsS = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(WRITE_DS ? dst + ((int64_t)b * H + head) * S * S : nullptr), 0, WRITE_DS ? (uint32_t)S * (uint32_t)S * 2u : 0u, 0x00020000);
  auto store_ds = [&](const bf16x8& f, int key, int q16) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const uint4 w = __builtin_bit_cast(uint4, f);
    const auto sx = __builtin_amdgcn_permlane32_swap(w.x, w.z, false, false);
    const auto sy = __builtin_amdgcn_permlane32_swap(w.y, w.w, false, false);
    const int q0 = q16 + 8 * (lane >> 5);
    const uint32_t o = q0 < S ? (uint32_t)key * (uint32_t)S * 2u + (uint32_t)q0 * 2u : DMA_OOB;
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{sx[0], sy[0], sx[1], sy[1]}, rsS, (int)o, 0, 0);
  };
  const bf16x8 zero_frag = __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0));
  uint32_t rowl, trl;
  {
    const int l31 = lane & 31, f = ((l31 & 3) << 2) | ((l31 >> 2) & 3), g = lane >> 4, s = lane & 15;
    rowl = (uint32_t)(l31 * 256 + (((lane >> 5) ^ f) << 4));
    trl = (uint32_t)(((g >> 1) * 4 + (s >> 2)) * 256 + ((((g & 1) * 2 + ((s & 3) >> 1)) ^ (((s >> 2) << 2) | (g >> 1))) << 4) + (s & 1) * 8);
  }
  // one key block from the early end (most queries) and its mirror image from the late end: equal work per workgroup
  for (int pass = 0; pass < 2; pass++) {
    const int kblk = pass == 0 ? wg.x : nkb - 1 - wg.x;
    if (pass == 1 && ((int)gridDim.x == nkb || kblk <= wg.x)) break;   // (unpaired launch: see the forward)
    const int n0 = kblk * BN, nw0 = n0 + pair * 32 * KB;
    wait_vm0();                                            // the pass before: its last loads, and everyone done with the ring
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    // what the dQ product reads of queries before this key block: zeros
    if (WRITE_DS && second)
      for (int qz = n0 / 256 * 256; qz < n0; qz += 16)
#pragma unroll
        for (int nb = 0; nb < KB; nb++) store_ds(zero_frag, nw0 + nb * 32 + (lane & 31), qz);
    // K or V rows of the pair's keys stay in registers (B operands); rows past S read as zeros.
    bf16x8 kv[KB][8];
    {
      const __amdgpu_buffer_rsrc_t rsKV = __builtin_amdgcn_make_buffer_rsrc(
          (void*)((second ? v : k) + tok0 * ldkv + kvoff), 0, (uint32_t)(S - 1) * (uint32_t)ldkv * 2u + 256u, 0x00020000);
      const uint32_t off = (uint32_t)(nw0 + (lane & 31)) * (uint32_t)ldkv * 2u + (uint32_t)(lane >> 5) * 16u;
#pragma unroll
      for (int nb = 0; nb < KB; nb++)
#pragma unroll
        for (int ks = 0; ks < 8; ks++)
          kv[nb][ks] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
              rsKV, (int)(off + (uint32_t)(nb * 32) * (uint32_t)ldkv * 2u + (uint32_t)ks * 32u), 0, 0));
    }
    f32x16 acc[KB][4];                                     // dK^T or dV^T
#pragma unroll
    for (int nb = 0; nb < KB; nb++)
#pragma unroll
      for (int hb = 0; hb < 4; hb++)
#pragma unroll
        for (int e = 0; e < 16; e++) acc[nb][hb][e] = 0.f;
    const int qb0 = n0 / 32, n = qblocks - qb0;            // causal: the first block that sees key n0, how many there are
    for (int i = 0; i < PAIR_NS - 1; i++) dma(i, qb0 + i);
    wait_vm<9>();                                          // block 0 has landed
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    int slot = 0, spare = PAIR_NS - 1;                     // of block i, and where block i + 4 goes

    // Operand addresses inside a SWZ_BOTH block (both_row_frag, both_tr_frag): the lane's part, from which the k16 step or the
    // 32 columns differ by an XOR.  (Blocks are multiples of 256 bytes; with the block added first nothing but the lane's part
    // is kept over the loop.)
    auto row_frag = [&](uint32_t blk, int ks) -> bf16x8 { return lds_b128(smem + ((blk + rowl) ^ (uint32_t)(ks << 5))); };
    auto tr_frag = [&](uint32_t blk, int t, int hb) -> bf16x8 {
      typedef short s16x8 __attribute__((ext_vector_type(8)));
      const uint32_t at = (blk + trl) ^ (uint32_t)(hb << 6);
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(smem + at + t * 4096));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(smem + (at ^ 32u) + t * 4096 + 2048));
      const s16x8 r = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      return __builtin_bit_cast(bf16x8, r);
    };
    // scores of the block at blk (its Q or dO rows): 32 queries x 32 NB keys
    auto scores = [&](uint32_t blk, f32x16 (&x)[KB], auto NB) {
#pragma unroll
      for (int nb = 0; nb < decltype(NB)::value; nb++)
#pragma unroll
        for (int e = 0; e < 16; e++) x[nb][e] = 0.f;
      bf16x8 f[PAIR_D + 1];
      unroll_for<PAIR_D>([&](auto I) { f[decltype(I)::value] = row_frag(blk, decltype(I)::value); });
      unroll_for<8>([&](auto I) {
        constexpr int ks = decltype(I)::value;
        if constexpr (ks + PAIR_D < 8) f[(ks + PAIR_D) % (PAIR_D + 1)] = row_frag(blk, ks + PAIR_D);
#pragma unroll
        for (int nb = 0; nb < decltype(NB)::value; nb++)
          x[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[ks % (PAIR_D + 1)], kv[nb][ks], x[nb], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    // acc += columns of the block at blk (its dO or Q rows) times what was made of the scores
    auto outputs = [&](uint32_t blk, const bf16x8 (&w)[KB][2], auto NB) {
      bf16x8 f[PAIR_D + 1];
      unroll_for<PAIR_D>([&](auto I) { f[decltype(I)::value] = tr_frag(blk, decltype(I)::value >> 2, decltype(I)::value & 3); });
      unroll_for<8>([&](auto I) {
        constexpr int s = decltype(I)::value, a = s + PAIR_D;
        if constexpr (a < 8) f[a % (PAIR_D + 1)] = tr_frag(blk, a >> 2, a & 3);
#pragma unroll
        for (int nb = 0; nb < decltype(NB)::value; nb++)
          acc[nb][s & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[s % (PAIR_D + 1)], w[nb][s >> 2], acc[nb][s & 3], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    // Between the first and the second half of block i: this wavefront's loads of block i + 1 have landed, everyone is done
    // with block i - 1.  Behind those loads lie the ones of two more blocks, and from block 3 on (STORES) what three blocks stored.
    auto meet = [&](int i, auto STORES) {
      wait_lgkm0();
      if (decltype(STORES)::value && i >= 3) wait_vm<6 + 3 * 2 * KB>();
      else wait_vm<6>();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      dma(spare, qb0 + i + PAIR_NS - 1);
    };
    auto next = [&]() {
      spare = slot;
      slot = slot + 1 == PAIR_NS ? 0 : slot + 1;
    };
    // Blocks of this pass: those before the pair's keys, the one that sees the first 32 of them (and only those: what the other 32
    // would add is 0 times it, NaN where it is not finite), the one with the other 32 keys' diagonal, whole ones, perhaps one with
    // the last queries.  Loops of their own: a branch around part of a block's work would have the accumulators change registers.
    const int skip = min(pair * KB, n), half = KB == 2 ? min(skip + 1, n) : skip, diag = min(skip + KB, n), whole = max(diag, S / 32 - qb0);
    constexpr std::integral_constant<int, 1> one{};
    constexpr std::integral_constant<int, KB> all{};
    constexpr std::false_type none{};
    constexpr std::integral_constant<bool, WRITE_DS> stores{};
    int i = 0;
    for (; i < skip; i++) {
      if (second) meet(i, stores);
      else meet(i, none);
      if constexpr (WRITE_DS) {
        if (second)
#pragma unroll
          for (int t = 0; t < 2; t++)
#pragma unroll
            for (int nb = 0; nb < KB; nb++) store_ds(zero_frag, nw0 + nb * 32 + (lane & 31), (qb0 + i) * 32 + t * 16);
      }
      next();
    }
    if (!second) {
      auto block = [&](auto MASKED, auto NB) {
        const uint32_t blk = (uint32_t)slot * PAIR_BLOCK;
        f32x16 x[KB];
        scores(blk, x, NB);
        const float* sl = reinterpret_cast<const float*>(smem + blk + 16384);
        unsigned char* xp = smem + PAIR_X + (i & 1) * 32768 + pair * 8192 + lane * 16;
        bf16x8 w[KB][2];
        unroll_for<4>([&](auto G) {
          constexpr int g = decltype(G)::value;
          const f32x4 lv = *reinterpret_cast<const f32x4*>(sl + 8 * g + 4 * (lane >> 5));
#pragma unroll
          for (int nb = 0; nb < decltype(NB)::value; nb++) {
            f32x4 p;
#pragma unroll
            for (int r = 0; r < 4; r++) {
              p[r] = fast_exp2(fmaf(x[nb][4 * g + r], c, -lv[r]));
              if constexpr (decltype(MASKED)::value) {
                const int qi = (qb0 + i) * 32 + acc_row(4 * g + r, lane), ni = nw0 + nb * 32 + (lane & 31);
                p[r] = (ni > qi || qi >= S) ? 0.f : p[r];
              }
            }
            *reinterpret_cast<f32x4*>(xp + (nb * 4 + g) * 1024) = p;
#pragma unroll
            for (int r = 0; r < 4; r++) x[nb][4 * g + r] = p[r];
          }
          if constexpr (g & 1)
#pragma unroll
            for (int nb = 0; nb < decltype(NB)::value; nb++) w[nb][g >> 1] = pack_acc_half(x[nb], g >> 1);
          __builtin_amdgcn_sched_barrier(0);
        });
        meet(i, none);
        outputs(blk + 8192, w, NB);
        next();
      };
      if constexpr (KB == 2)
        for (; i < half; i++) block(std::true_type{}, one);
      for (; i < diag; i++) block(std::true_type{}, all);
      for (; i < whole; i++) block(std::false_type{}, all);
      for (; i < n; i++) block(std::true_type{}, all);
    } else {
      auto block = [&](auto NB) {
        const uint32_t blk = (uint32_t)slot * PAIR_BLOCK;
        f32x16 x[KB];
        scores(blk + 8192, x, NB);
        meet(i, stores);
        const float* sd = reinterpret_cast<const float*>(smem + blk + 16384 + 256);
        const unsigned char* xp = smem + PAIR_X + (i & 1) * 32768 + pair * 8192 + lane * 16;
        bf16x8 w[KB][2];
        unroll_for<4>([&](auto G) {
          constexpr int g = decltype(G)::value;
          const f32x4 dvv = *reinterpret_cast<const f32x4*>(sd + 8 * g + 4 * (lane >> 5));
#pragma unroll
          for (int nb = 0; nb < decltype(NB)::value; nb++) {
            const f32x4 p = *reinterpret_cast<const f32x4*>(xp + (nb * 4 + g) * 1024);
#pragma unroll
            for (int r = 0; r < 4; r++) x[nb][4 * g + r] = (SCALED ? p[r] * scale : p[r]) * (x[nb][4 * g + r] - dvv[r]);   // dS
          }
          if constexpr (g & 1)
#pragma unroll
            for (int nb = 0; nb < decltype(NB)::value; nb++) w[nb][g >> 1] = pack_acc_half(x[nb], g >> 1);
          __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (WRITE_DS) {   // (as many stores for every block: the waits above count them)
          static_assert(KB == 1, "a block with the first 32 keys alone stores less");
#pragma unroll
          for (int t = 0; t < 2; t++) store_ds(w[0][t], nw0 + (lane & 31), (qb0 + i) * 32 + t * 16);
        }
        outputs(blk, w, NB);
        next();
      };
      if constexpr (KB == 2)
        for (; i < half; i++) block(one);
      for (; i < n; i++) block(all);
    }
#pragma unroll
    for (int nb = 0; nb < KB; nb++) {
      const int ni = nw0 + nb * 32 + (lane & 31);
      if (ni < S) store_acc_T((second ? dk : dv) + (tok0 + ni) * lddkv + hoff, acc[nb], second && !SCALED ? scale : 1.f, lane);
    }
  }  // pass
  wait_vm0();                                              // no load into LDS outlives the workgroup
}

// Grouped-query attention: a key / value head's gradient is the sum of the contributions of the grp
// query heads that share it.  part: two [T, H * HD] bf16 tensors (dK, then dV contributions, one per
// query head), out: dk / dv [T, ldkv].  One thread adds grp 16-byte vectors in fp32.
__global__ __launch_bounds__(256) void attn_group_sum_kernel(const uint16_t* __restrict__ part, int64_t part_elems,
                                                             uint16_t* __restrict__ dk, uint16_t* __restrict__ dv,
                                                             int64_t ldkv, int grp, int H, int64_t T) {
  const int Hkv = H / grp;
  const int64_t item = (int64_t)blockIdx.x * 256 + threadIdx.x;   // (token, kv head, 16-byte chunk)
  if (item >= T * Hkv * (HD / 8)) return;
  const int ch = (int)(item % (HD / 8));
  const int kvh = (int)((item / (HD / 8)) % Hkv);
  const int64_t t = item / ((int64_t)(HD / 8) * Hkv);
  const uint16_t* src = part + (int64_t)blockIdx.y * part_elems + t * ((int64_t)H * HD) + (int64_t)kvh * grp * HD + ch * 8;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int g = 0; g < grp; g++) {
    float v[8];
    unpack8(*reinterpret_cast<const uint4*>(src + g * HD), v);
#pragma unroll
    for (int e = 0; e < 8; e++) acc[e] += v[e];
  }
  uint16_t* dst = (blockIdx.y == 0 ? dk : dv) + t * ldkv + kvh * HD + ch * 8;
  *reinterpret_cast<uint4*>(dst) = pack8(acc);
}

template <class K>
hipError_t set_lds(K kern, int bytes) {
  return hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

}  // namespace

hipError_t attention_fwd_bf16(const void* q, const void* k, const void* v, void* o, float* lse, int64_t ld, int B,
                              int S, int H, int hd, int causal, hipStream_t st) {
  return attention_gqa_fwd_bf16(q, k, v, o, lse, ld, ld, B, S, H, H, hd, causal, st);
}

// Hkv key / value heads (rows of ldkv elements) serve H query heads, H / Hkv consecutive ones each.
hipError_t attention_gqa_fwd_bf16(const void* q, const void* k, const void* v, void* o, float* lse, int64_t ld,
                                  int64_t ldkv, int B, int S, int H, int Hkv, int hd, int causal, hipStream_t st) {
  if (hd != HD || !causal) return hipErrorNotSupported;
  if (Hkv <= 0 || H % Hkv != 0) return hipErrorInvalidValue;
  const int grp = H / Hkv;
  // 32-bit buffer offsets per (batch, head)
  if ((int64_t)S * ld * 2 >= (int64_t)0x7fffffff || (int64_t)S * ldkv * 2 >= (int64_t)0x7fffffff) return hipErrorNotSupported;
  auto launch = [&](auto NWc) {
    constexpr int NW = decltype(NWc)::value, BQ = NW * 32;
    // one-time opt-in to more than 64 KB of dynamic LDS (thread-safe static initialisation)
    static const hipError_t attr_err = set_lds(attn_fwd_kernel<NW>, FWD_LDS);
    if (attr_err != hipSuccess) return attr_err;
    const int nqb = (S + BQ - 1) / BQ;
    // Each workgroup: one query block and its mirror; or one block, where each finds a CU free: the launch then takes
    // as long as its longest block instead of a pair (2 x 256 tokens, 2 heads: 18.3 -> 12.3 us).  With two
    // unpaired workgroups per CU the late blocks meet on some CUs (4 x 4096 tokens, 4 heads: 110 -> 135 us).
    dim3 grid((int64_t)nqb * H * B <= 256 ? nqb : (nqb + 1) / 2, H, B);
    hipLaunchKernelGGL(attn_fwd_kernel<NW>, grid, dim3(NW * 64), FWD_LDS, st, (const uint16_t*)q, (const uint16_t*)k,
                       (const uint16_t*)v, (uint16_t*)o, lse, ld, ldkv, grp, S, H, 1.f / sqrtf((float)hd));
    return hipGetLastError();
  };
  // 4 wavefronts: a block's wavefronts walk its keys together, so in one of 8 those of the first half wait for those of the second, and
  // the chip fills less evenly (us, 4 / 8, inputs warm: 128 x 64 tokens, 16 heads 31.0 / 47.4, 16 x 1024 95 / 103, 7 x 1280, 32 heads
  // 131 / 155, 8 x 2048, 16 heads 155 / 158, 4 x 4096, 32 heads 552 / 568).  8 where every CU gets one such pair of blocks and no more,
  // which is as many wavefronts as two workgroups of 4 but fetches a key tile once for them, not twice: no faster warm (2 x 2047, 32 / 8
  // heads 83.5 / 82.8, 4 x 2047, 16 heads 81.5 / 83.0), but with the inputs in memory (91.4 / 90.3, 94.0 / 88.9; 1 x 4096, 32
  // heads 150.6 / 146.2; the first with its backward 431 / 424).  Fewer blocks than 8, or an odd one out: behind in both (us, cold,
  // 1 x 1600, 64 / 8 heads 66.3 / 71.4, 1 x 2349, 32 / 8 heads 79.1 / 84.2).
  const int wide = (S + 255) / 256;
  const int64_t pairs = (int64_t)(wide / 2) * H * B;
  return wide >= 8 && wide % 2 == 0 && pairs >= 224 && pairs <= 256 ? launch(std::integral_constant<int, 8>{})
                                                                    : launch(std::integral_constant<int, 4>{});
}

// The backward runs in one of two forms.  With the score gradient kept (S a multiple of 8, and
// B * H * S^2 bf16 values within the cap below): the dK / dV kernel also writes scale * dS^T and dQ is
// one k-major GEMM over it, 5 GEMM units in all.  Otherwise: a second kernel recomputes S, dP and dS for
// dQ, 7 units and no large workspace.  Where the pairs of wavefronts find work for the whole chip (dkv_pairs), forming the
// score gradient twice is faster than the way through memory, and the kernels round it where the first form does: the same
// bits.  Whole backward, us, kept -> formed twice: 4 x 4096 tokens, 32 heads 2098 -> 1841; 8 x 2048, 16 heads 644 -> 542; 1 x 8192, 16 heads
// 980 -> 853; 8 x 1024, 16 heads 204 -> 178; 16 x 264, 32 heads 157 -> 152; elsewhere 2 x 1536, 16 heads 106 / 115; 1 x 2048, 8 heads 99 / 104,
// 128 x 128, 16 heads 243 / 280.
constexpr size_t DS_WS_CAP = (size_t)24 << 30;
static bool keep_ds(int B, int S, int H) {
  return S % 8 == 0 && (int64_t)S * S * 2 < (int64_t)0x7fffffff && (size_t)B * H * S * S * 2 <= DS_WS_CAP;
}

// 256 keys per workgroup, in pairs of blocks, or 128: a workgroup of twice the keys takes 0.91 to 0.97 of two workgroups' time, so it
// pays where the launch is half as many rounds of the chip or fewer, and from 144 workgroups on (fewer were not measured).  Whole
// backward, this kernel against the others, % (rounds, this one's first): 2 x 2047 tokens, 32 heads -8.9 (1, 2), 2 x 2999, 12 heads -8.5
// (1, 2), 16 x 259, 32 heads -9.3 (2, 4), 7 x 1283, 32 heads -6.2 (3, 6); 8 x 1129, 32 heads -3.8 (3, 5), 20 x 1001, 16 heads -1.8 (3, 5),
// 3 x 1801, 32 heads +1.4 (2, 3), 16 x 700, 16 heads +3.9 (2, 3), 1 x 6001, 24 heads +7.1 (2, 3), 13 x 641, 32 heads +8.8 (4, 5), 1 x 3333,
// 16 heads, a block per workgroup, +17 (1, 1).
static bool dkv_pairs(int S, int64_t heads) {
  const int64_t wide = (S + 255) / 256, wgs = (wide + 1) / 2 * heads, other = ((S + 127) / 128 + 1) / 2 * heads;
  return wide * heads > 256 && wgs >= 144 && 2 * ((wgs + 255) / 256) <= (other + 255) / 256;
}

// The room for the score gradient: the most that a call of as many heads stores for up to B * S tokens in sequences of up to S, so that
// a workspace for more tokens serves for fewer, which may store it where more form it twice (4 x 4096 tokens, 32 heads: 3.4 GB, for
// 5 x 3272; its own would be 4.3).  dkv_pairs sees of S only the number of 256-key blocks, so of those with as
// many the longest sequence counts: `longest` while b of them fit, then what the tokens leave to each.
static size_t ds_bytes(int B, int S, int H) {
  if (!keep_ds(B, S, H)) return 0;
  const int64_t tokens = (int64_t)B * S;
  size_t most = 0;
  auto one = [&](int64_t b, int64_t s) { return (size_t)b * H * s * s * 2; };
  for (int wide = (S + 255) / 256; wide > 0; wide--) {
    const int64_t longest = S < wide * 256 ? S : wide * 256, fit = tokens / longest;
    if ((size_t)tokens * H * longest * 2 <= most) break;
    for (int64_t b = fit; b > 0 && one(b, longest) > most; b--)
      if (!dkv_pairs((int)longest, b * H)) most = one(b, longest);
    for (int64_t b = fit + 1; tokens / b > (wide - 1) * 256 && one(b, tokens / b) > most; b++)
      if (!dkv_pairs((int)longest, b * H)) most = one(b, tokens / b);
  }
  return (most + 255) / 256 * 256;
}
// D and the base-2 exponent offsets lse * log2(e), both [B, H, S] fp32; then dS^T [B, H, S, S] bf16
size_t attention_bwd_ws_bytes(int B, int S, int H, int hd) { return attention_gqa_bwd_ws_bytes(B, S, H, H, hd); }
// ... and, with fewer key / value heads than query heads, the per-query-head contributions to dK and dV
// (two [B * S, H * hd] bf16 tensors) that a last kernel adds up group by group
size_t attention_gqa_bwd_ws_bytes(int B, int S, int H, int Hkv, int hd) {
  const size_t small = (2 * (size_t)B * H * S * sizeof(float) + 255) / 256 * 256;
  return small + ds_bytes(B, S, H) + (Hkv < H ? 2 * (size_t)B * S * H * HD * 2 : 0);
}

constexpr int DKV_NB = 1;   // 32-key blocks per wavefront in the dK/dV kernel

hipError_t attention_bwd_bf16(const void* q, const void* k, const void* v, const void* o, const void* dout,
                              const float* lse, void* dq, void* dk, void* dv, int64_t ld, int B, int S, int H, int hd,
                              int causal, void* ws, hipStream_t st) {
  return attention_gqa_bwd_bf16(q, k, v, o, dout, lse, dq, dk, dv, ld, ld, B, S, H, H, hd, causal, ws, st);
}

hipError_t attention_gqa_bwd_bf16(const void* q, const void* k, const void* v, const void* o, const void* dout,
                                  const float* lse, void* dq, void* dk, void* dv, int64_t ld, int64_t ldkv, int B, int S,
                                  int H, int Hkv, int hd, int causal, void* ws, hipStream_t st) {
  if (hd != HD || !causal) return hipErrorNotSupported;
  if (Hkv <= 0 || H % Hkv != 0) return hipErrorInvalidValue;
  const int grp = H / Hkv;
  // 32-bit buffer offsets per (batch, head)
  if ((int64_t)S * ld * 2 >= (int64_t)0x7fffffff || (int64_t)S * ldkv * 2 >= (int64_t)0x7fffffff) return hipErrorNotSupported;
  static const hipError_t attr_err = [] {
    hipError_t e = set_lds(attn_bwd_dq_kernel<4, false>, DQ_LDS);
    if (e == hipSuccess) e = set_lds(attn_bwd_dq_kernel<8, false>, DQ_LDS);
    if (e == hipSuccess) e = set_lds(attn_bwd_dq_kernel<8, true>, DQ_LDS);
    if (e == hipSuccess) e = set_lds(attn_bwd_dkv_long_kernel, LDKV_LDS);
    if (e == hipSuccess) e = set_lds(attn_bwd_dkv_pair_kernel<2, false, false>, PAIR_LDS);
    if (e == hipSuccess) e = set_lds(attn_bwd_dkv_pair_kernel<2, true, false>, PAIR_LDS);
    if (e == hipSuccess) e = set_lds(attn_bwd_dkv_pair_kernel<1, true, true>, PAIR_LDS);
    if (e == hipSuccess) e = set_lds(attn_bwd_dkv_kernel<DKV_NB, false>, DKV_LDS);
    if (e == hipSuccess) e = set_lds(attn_bwd_dkv_kernel<DKV_NB, true>, DKV_LDS);
    return e;
  }();
  if (attr_err != hipSuccess) return attr_err;
  float* D = (float*)ws;
  const int64_t items = (int64_t)B * S * H;
  float* lse2 = D + items;
  hipLaunchKernelGGL(attn_dot_kernel, dim3((unsigned)((items * 16 + 255) / 256)), dim3(256), 0, st,
                     (const uint16_t*)dout, (const uint16_t*)o, lse, D, lse2, ld, S, H, items);
  const float scale = 1.f / sqrtf((float)hd);
  const int nkb = (S + 127) / 128;   // paired or not as in the forward (29.6 -> 18.6 us)
  const dim3 kv_grid((int64_t)nkb * H * B <= 256 ? nkb : (nkb + 1) / 2, H, B);
  const size_t small = (2 * (size_t)items * sizeof(float) + 255) / 256 * 256;
  // where the dK / dV kernel writes: the outputs themselves, or (fewer key / value heads than query
  // heads) one contribution per query head, added up at the end
  const int64_t T = (int64_t)B * S, part_elems = T * H * HD;
  uint16_t* part = (uint16_t*)((char*)ws + small + ds_bytes(B, S, H));
  uint16_t* dk_w = grp > 1 ? part : (uint16_t*)dk;
  uint16_t* dv_w = grp > 1 ? part + part_elems : (uint16_t*)dv;
  const int64_t lddkv = grp > 1 ? (int64_t)H * HD : ldkv;
  auto group_sum = [&]() -> hipError_t {
    if (grp == 1) return hipSuccess;
    const int64_t n = T * Hkv * (HD / 8);
    hipLaunchKernelGGL(attn_group_sum_kernel, dim3((unsigned)((n + 255) / 256), 2), dim3(256), 0, st, (const uint16_t*)part,
                       part_elems, (uint16_t*)dk, (uint16_t*)dv, ldkv, grp, H, T);
    return hipGetLastError();
  };
  const int64_t heads = (int64_t)H * B;
  const bool pairs = dkv_pairs(S, heads), kept = keep_ds(B, S, H);
  if (kept && !pairs) {
    uint16_t* dst = (uint16_t*)((char*)ws + small);
    // Pairs of wavefronts put two on a SIMD where a workgroup has a CU to itself (whole backward, us, four wavefronts / four pairs:
    // 1 x 2048 tokens, 8 heads 100 / 92.3, 1 x 4096, 4 heads 181 / 165.8, 1 x 776, 32 heads 58.6 / 55.4, 2 x 1536, 16 heads
    // 107.8 / 100.8, 4 x 1024, 16 heads 92.9 / 90.1).  They lose where two workgroups of four fit beside each other (8 x 1280, 16
    // heads 315 / 322), and on few long sequences that fill the chip (4 x 4096, 4 heads 258.8 / 276.1; 2 x 2048, 16 heads 152 / 161).
    if (nkb * heads <= 256 || (nkb * heads <= 512 && S <= 1536))
      hipLaunchKernelGGL((attn_bwd_dkv_pair_kernel<1, true, true>), kv_grid, dim3(512), PAIR_LDS, st, (const uint16_t*)q,
                         (const uint16_t*)k, (const uint16_t*)v, (const uint16_t*)dout, lse2, D, dk_w, dv_w, dst, ld, ldkv,
                         lddkv, grp, S, H, scale);
    else
      hipLaunchKernelGGL((attn_bwd_dkv_kernel<DKV_NB, true>), kv_grid, dim3(256), DKV_LDS, st, (const uint16_t*)q,
                         (const uint16_t*)k, (const uint16_t*)v, (const uint16_t*)dout, lse2, D, dk_w, dv_w, dst, ld, ldkv,
                         lddkv, grp, S, H, scale);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // dQ[q, :] = sum_key (scale dS^T)[key, q] * K[key, :], per (batch, head): both operands k-major, the
    // key range of a row tile cut at its last query; one launch, batch index = (batch element, head), the
    // heads of a group on the same K
    GemmOp op;
    op.lda = S; op.transA = 1; op.ldb = ldkv; op.transB = 1; op.ldc = ld;
    op.M = S; op.N = HD; op.K = S; op.causal_k = 1;
    op.epi.kind = EPI_STORE;
    op.A = dst; op.sA = (int64_t)S * S; op.sAo = (int64_t)H * S * S;
    op.B = k; op.sB = HD; op.sBo = (int64_t)S * ldkv; op.b_group = grp;
    op.C = dq; op.sC = HD; op.sCo = (int64_t)S * ld;
    op.batch = B * H; op.batch_inner = H;
    e = gemm_bf16_untimed(op, st);
    return e != hipSuccess ? e : group_sum();
  }
  // dQ: a block of 256 queries and its mirror per workgroup; where that leaves CUs idle a block each, and of 128 queries where
  // those find a CU each.  Of few long blocks of 256 the last ones decide, so from 1024 tokens on they are halved and paired
  // (whole backward, us, a block of 256 each / 128 and its mirror: 4 x 4095 tokens, 4 heads 279 / 253, 1 x 3333, 16 heads 216 / 195,
  // 4 x 1501, 8 heads 121 / 112, 2 x 1031, 16 heads 95.1 / 93.3; 4 x 700, 12 heads 76 / 78).
  auto dq_launch = [&](auto NWc, auto SCALED, bool paired) {
    constexpr int NW = decltype(NWc)::value;
    const int n = (S + NW * 32 - 1) / (NW * 32);
    hipLaunchKernelGGL((attn_bwd_dq_kernel<NW, decltype(SCALED)::value>), dim3(paired ? (n + 1) / 2 : n, H, B), dim3(NW * 64), DQ_LDS, st,
                       (const uint16_t*)q, (const uint16_t*)k, (const uint16_t*)v, (const uint16_t*)dout, lse2, D, (uint16_t*)dq, ld,
                       ldkv, grp, S, H, scale);
  };
  using Four = std::integral_constant<int, 4>;
  using Eight = std::integral_constant<int, 8>;
  if (pairs && kept) dq_launch(Eight{}, std::true_type{}, true);   // (pairs: more than 256 blocks of 256)
  else if ((S + 127) / 128 * heads <= 256) dq_launch(Four{}, std::false_type{}, false);
  else if (S >= 1024 && (S + 255) / 256 * heads <= 256) dq_launch(Four{}, std::false_type{}, true);
  else dq_launch(Eight{}, std::false_type{}, (S + 255) / 256 * heads > 256);
  auto pair_launch = [&](auto SCALED) {
    hipLaunchKernelGGL((attn_bwd_dkv_pair_kernel<2, decltype(SCALED)::value, false>), dim3(((S + 255) / 256 + 1) / 2, H, B), dim3(512),
                       PAIR_LDS, st, (const uint16_t*)q, (const uint16_t*)k, (const uint16_t*)v, (const uint16_t*)dout, lse2, D, dk_w, dv_w,
                       (uint16_t*)nullptr, ld, ldkv, lddkv, grp, S, H, scale);
  };
  if (pairs && kept) pair_launch(std::true_type{});
  else if (pairs) pair_launch(std::false_type{});
  else if (S >= ((int)kv_grid.x == nkb ? LDKV_MIN_S : LDKV_MIN_S_PAIRED))
    hipLaunchKernelGGL(attn_bwd_dkv_long_kernel, kv_grid, dim3(256), LDKV_LDS, st, (const uint16_t*)q, (const uint16_t*)k,
                       (const uint16_t*)v, (const uint16_t*)dout, lse2, D, dk_w, dv_w, ld, ldkv, lddkv, grp, S, H, scale);
  else
    hipLaunchKernelGGL((attn_bwd_dkv_kernel<DKV_NB, false>), kv_grid, dim3(256), DKV_LDS, st, (const uint16_t*)q,
                       (const uint16_t*)k, (const uint16_t*)v, (const uint16_t*)dout, lse2, D, dk_w, dv_w,
                       (uint16_t*)nullptr, ld, ldkv, lddkv, grp, S, H, scale);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return group_sum();
}

}  // namespace lrb
