// What the bf16 MFMA GEMM kernels share: compile-time loops, wait counts, the workgroup -> tile map and the
// epilogue that carries an accumulator tile through LDS into row-contiguous global vectors.
#pragma once
#include <type_traits>

#include "epilogue.h"

namespace lrb {
namespace {

constexpr int BK = 64;          // k elements per LDS stage: 128-byte rows, i.e. whole cache lines per request
constexpr int NXCD = 8;

// Compile-time loop: the body receives std::integral_constant indices, so register arrays indexed
// by them never turn into scratch memory, whatever the unroller decides.
template <int N, class F, int I = 0>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, F, I + 1>(static_cast<F&&>(f));
  }
}

__device__ __forceinline__ float sumsq8(const uint4& q) {
  float v[8];
  unpack8(q, v);
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 8; i++) s = fmaf(v[i], v[i], s);
  return s;
}

// s_waitcnt vmcnt(N) with the other counters left alone (gfx9 encoding: vmcnt in bits 3:0 and 15:14).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0f70);
}
__device__ __forceinline__ void wait_lgkmcnt0() { __builtin_amdgcn_s_waitcnt(0xc07f); }

// Sum over aligned groups of N = 4 or 8 consecutive lanes, every lane receiving the total, with
// data-parallel-primitive moves (register file only): neighbours inside a quad, then the mirror image
// inside 8 lanes.  (A butterfly of __shfl_xor goes through the LDS crossbar: three
// dependent round trips per row partial.)
template <int N>
__device__ __forceinline__ float lane_group_sum(float x) {
  static_assert(N == 4 || N == 8, "lane group size");
  auto dpp = [](float v, auto CTRL) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(CTRL)::value, 0xf, 0xf, false));
  };
  x += dpp(x, std::integral_constant<int, 0xB1>{});    // quad_perm [1,0,3,2]
  x += dpp(x, std::integral_constant<int, 0x4E>{});    // quad_perm [2,3,0,1]
  if constexpr (N == 8) x += dpp(x, std::integral_constant<int, 0x141>{});   // row_half_mirror: lane i <-> 7 - i
  return x;
}

// The output tile with index nid of a launch: consecutive indexes form compact panels (PM tiles tall), keeping the A
// rows and B rows they share in one L2; (batch member, k split) slowest.
__device__ __forceinline__ void tile_of_index(int nid, int tiles_m, int tiles_n, int& tm, int& tn, int& bz) {
  const int tiles = tiles_m * tiles_n;
  bz = nid / tiles;
  const int tid_ = nid % tiles;
  constexpr int PM = 8;
  const int per_panel = PM * tiles_n;
  const int panel = tid_ / per_panel, within = tid_ % per_panel;
  const int pm_eff = min(PM, tiles_m - panel * PM);
  tn = within / pm_eff;
  tm = panel * PM + within % pm_eff;
}

// Maps the linear workgroup id to an output tile so that the workgroups that the hardware deals round-robin to one
// XCD form a contiguous range of tiles.
// The range runs over the whole launch: an XCD then works on tiles of one batch member and one k range at a time,
// which is what lets its workgroups share operand slices.
__device__ __forceinline__ void tile_of_block(int bid, int total, int tiles_m, int tiles_n, int& tm, int& tn, int& bz) {
  const int xcd = bid % NXCD, loc = bid / NXCD;
  const int base = total / NXCD, rem = total % NXCD;
  tile_of_index(xcd * base + (xcd < rem ? xcd : rem) + loc, tiles_m, tiles_n, tm, tn, bz);
}

// The launch grid of `tiles` output tiles for each of `members` batch members times k splits.  The kernels number their
// workgroups through both dimensions, so where the members are more than the second may have, all go into the first.
inline dim3 tile_grid(int tiles, int members) {
  return members <= 65535 ? dim3((unsigned)tiles, (unsigned)members) : dim3((unsigned)tiles * (unsigned)members);
}

#define LRB_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

// ---- epilogue ---------------------------------------------------------------------------------
// Called by every wavefront that holds accumulators once they are final and its staging space is free.
// Tile type T: BM rows; WN wavefronts across, each with an FM x FN arrangement of 32x32 MFMA blocks (TM x TN), of
// which Stage::SR rows of Stage::SC columns are staged at a time: 32 of all columns, or 16 of 64.  stage.at(row, chunk): where
// 16-byte chunk `chunk` of staged row `row` lies.  (m0, n0): first row / column of the output tile, tn its column
// index, b / (bi, bo) / bz: batch member, its two-level split, batch member times k split.  sStat: the row
// statistics gathered in the main loop (STAT_A); STAT_IN_STAGE: they lie in the staging space.  accg: the gate's accumulators as
// bf16 pairs (EPI_SWIGLU_DUAL): [row block][column block][four columns of a run].
template <class T>
struct GateAcc { uint2 v[T::FM][T::FN][4]; };
template <class T, int KIND, bool STAT_A, class Stage>
__device__ __forceinline__ void gemm_epilogue(const GemmOp& op, f32x16 (&acc)[T::FM][T::FN], const Stage& stage,
                                              const float* sStat, int wave, int lane, int m0, int n0, int tn,
                                              int tiles_n, int b, int bi, int bo, int bz, const GateAcc<T>& accg = GateAcc<T>()) {
  const int wm = wave / T::WN, wn = wave % T::WN;
  // The wavefront's sub-tile leaves in passes of RPP rows and SC columns.  Everything the passes touch
  // in global memory goes through buffer resources that start at the tile's first row and end after
  // its last valid row: rows past M (and, by an out-of-range offset, columns past N) read as zeros and
  // are dropped on store, an absent auxiliary tile is a resource of size zero.  The pass code is
  // therefore free of branches, which is what lets the compiler count the loads in flight exactly: the
  // auxiliary tiles an epilogue reads (residual, z, x, g, u) are fetched PF passes ahead into a small
  // register ring, and each pass waits only for its own.
  const Epilogue& e = op.epi;
  constexpr int LPR = Stage::SC / 8;            // lanes per output row
  constexpr int RPP = 64 / LPR;             // rows per pass
  constexpr int PPS = Stage::SR / RPP;          // passes per staged piece
  constexpr int NJ = T::TN / Stage::SC;         // pieces side by side
  constexpr int NH = 32 / Stage::SR;            // pieces of an MFMA block's rows
  constexpr int NQ = T::FM * NH * NJ * PPS; // passes per wavefront
  static_assert(Stage::SR == 32 ? NJ == 1 : Stage::SR == 16 && Stage::SC == 64, "staging forms");
  // which auxiliary tiles a kind can read at all, and the prefetch distance in passes: kinds with one
  // auxiliary tile keep eight of its 16-byte vectors in flight per lane, kinds with two keep four of each
  // BASE: the formula; R_F32: the R tile is fp32 (two 16-byte vectors per lane and pass); O32: the primary
  // output is also written un-rounded, as fp32, into C32
  constexpr int BASE = epi_base(KIND);
  constexpr bool R_F32 = epi_r_is_f32(KIND), O32 = epi_writes_f32(KIND);
  constexpr bool DUAL = KIND == EPI_SWIGLU_DUAL;
  constexpr bool HAS_R = DUAL ? false : BASE == EPI_UP || BASE == EPI_ACTGRAD || BASE == EPI_NORMBWD || BASE == EPI_SWIGLU_BWD ||
                         BASE == EPI_SWIGLU_FWD || BASE == EPI_DOWN_LAX || BASE == EPI_LAXGRAD;
  constexpr bool HAS_R2 = BASE == EPI_NORMBWD || BASE == EPI_SWIGLU_BWD || BASE == EPI_LAXGRAD;
  constexpr int PF = (HAS_R2 || R_F32) ? 4 : 8;
  constexpr uint32_t EOOB = 0x80000000u;
  const int cg = lane % LPR, rsub = lane / LPR;
  const int rows_valid = min(T::BM, op.M - m0);
  const int coln = n0 + wn * T::TN + cg * 8;                         // first of this lane's 8 columns (leftmost piece)
  auto tile_rsrc = [&](const void* base, int64_t batch_off, int64_t ld, int esz) {
    const char* p = base ? (const char*)base + (batch_off + (int64_t)m0 * ld) * esz : nullptr;
    return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, base ? (uint32_t)rows_valid * (uint32_t)ld * (uint32_t)esz : 0u,
                                             0x00020000);
  };
  auto row_rsrc = [&](const float* base) {   // per-row fp32 scalars of the tile's rows
    return __builtin_amdgcn_make_buffer_rsrc((void*)(base ? base + m0 : nullptr), 0, base ? (uint32_t)rows_valid * 4u : 0u,
                                             0x00020000);
  };
  constexpr bool PARTIAL = KIND == EPI_PARTIAL;
  // C: bf16 [batch][M][ldc]; fp32 split-K partials: [batch * split][M][N]
  const __amdgpu_buffer_rsrc_t rsC = PARTIAL
      ? __builtin_amdgcn_make_buffer_rsrc((void*)((char*)op.C + ((int64_t)bz * op.M + m0) * op.N * 4), 0,
                                          (uint32_t)rows_valid * (uint32_t)op.N * 4u, 0x00020000)
      : tile_rsrc(op.C, (int64_t)bi * op.sC + (int64_t)bo * op.sCo, op.ldc, 2);
  const __amdgpu_buffer_rsrc_t rsC2 = tile_rsrc(PARTIAL ? nullptr : e.C2, (int64_t)b * e.sC2, e.ldc2, 2);
  const bool use_r = !PARTIAL && epi_reads_r<BASE>(e), use_r2 = !PARTIAL && epi_reads_r2<BASE>(e);
  const __amdgpu_buffer_rsrc_t rsR = tile_rsrc(use_r ? e.R : nullptr, (int64_t)b * e.sR, e.ldr, R_F32 ? 4 : 2);   // (DUAL: g, written)
  const __amdgpu_buffer_rsrc_t rsC32 = tile_rsrc(O32 ? e.C32 : nullptr, 0, e.ldc32, 4);
  const __amdgpu_buffer_rsrc_t rsR2 = tile_rsrc(use_r2 ? e.R2 : nullptr, (int64_t)b * e.sR2, e.ldr2, 2);
  const __amdgpu_buffer_rsrc_t rsRowA = row_rsrc((!PARTIAL && e.use_rho && !STAT_A) ? e.rowa : nullptr);
  const __amdgpu_buffer_rsrc_t rsRowB = row_rsrc(!PARTIAL ? e.rowb : nullptr);
  const int ldC = PARTIAL ? op.N * 4 : (int)op.ldc * 2;               // row pitches in bytes
  const int ldC2 = (int)e.ldc2 * 2, ldR = (int)e.ldr * (R_F32 ? 4 : 2), ldR2 = (int)e.ldr2 * 2, ldC32 = (int)e.ldc32 * 4;
  // byte offset inside a row of this lane's columns of piece jj, for elements of es bytes
  auto col_off = [&](int jj, uint32_t es) -> uint32_t {
    return coln + jj * Stage::SC < op.N ? (uint32_t)(coln + jj * Stage::SC) * es : EOOB;
  };
  const bool want2 = KIND == EPI_SWIGLU_BWD || BASE == EPI_SWIGLU_FWD || KIND == EPI_DOWN_LAX || KIND == EPI_LAXGRAD ||
                     KIND == EPI_ACTGRAD_A || (KIND == EPI_DOWN && e.C2 != nullptr);
  const bool use_rho = !PARTIAL && e.use_rho;
  const bool rho_sqrt = e.rho_sqrt != 0;
  // row partials [M, rowpart_ld] and the statistic [M]: one lane per row writes, the others (and rows
  // past M) are given an out-of-range offset
  constexpr bool ROWPART = BASE == EPI_UP || BASE == EPI_ACTGRAD || BASE == EPI_LAXGRAD;
  const __amdgpu_buffer_rsrc_t rsPart = __builtin_amdgcn_make_buffer_rsrc(
      (void*)((ROWPART && e.rowpart) ? e.rowpart + (int64_t)m0 * e.rowpart_ld : nullptr), 0,
      (ROWPART && e.rowpart) ? (uint32_t)rows_valid * (uint32_t)e.rowpart_ld * 4u : 0u, 0x00020000);
  const int ldPart = ROWPART ? (int)e.rowpart_ld * 4 : 0;
  // one partial per 64 columns (32 where the wavefront's sub-tile has no more): SPW of them per wavefront and row
  constexpr int LPP = T::TN < 64 ? T::TN / 8 : 8, SPW = T::TN / (LPP * 8);
  const uint32_t colPart =
      cg % LPP == 0 ? (uint32_t)(e.rowpart_off + ((b * tiles_n + tn) * T::WN + wn) * SPW + cg / LPP) * 4u : EOOB;
  const bool write_stat = STAT_A && e.stat_out && tn == 0 && wn == 0 && b == 0;
  const __amdgpu_buffer_rsrc_t rsStat = row_rsrc(write_stat ? e.stat_out : nullptr);
  const uint32_t colStat = cg == 0 ? 0u : EOOB;
  const int act = e.act;
  const float inv_d = e.inv_d, eps = e.eps;
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  u32x4 auxr[PF], auxr2[PF], auxr3[R_F32 ? PF : 1];   // auxr3: columns 4..7 of an fp32 R tile
  uint4 gate[DUAL ? PPS : 1];                   // DUAL: g as stored, of the staged piece
  // pass q: MFMA block row i, piece h of its rows, piece jj across, p-th run of RPP rows
  auto row_of = [&](int q) {                                       // row inside the tile
    return wm * T::TM + (q / (NH * NJ * PPS)) * 32 + (q / (NJ * PPS) % NH) * Stage::SR + (q % PPS) * RPP + rsub;
  };
  auto across = [](int q) { return q / PPS % NJ; };
  // per-row scalars, fetched with the auxiliary tiles; where there is none, all before the first pass: behind stores that a branch
  // may leave out, the compiler cannot count, and their waits were for everything, the next tile's slices included (EPI_DOWN)
  constexpr int PR = STAT_A || !HAS_R ? NQ : PF;
  float ssv[PR], rbv[PR];
  constexpr bool ROWS = !PARTIAL && !STAT_A && BASE != EPI_STORE && BASE != EPI_UP && BASE != EPI_SWIGLU_BWD && BASE != EPI_SWIGLU_FWD;
  auto fetch_row = [&](int q, float& ss, float& rb) {
    const int lm = row_of(q);
    if constexpr (ROWS) {
      if (use_rho) ss = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsRowA, lm * 4, 0, 0));
    }
    if constexpr (BASE == EPI_NORMBWD) rb = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsRowB, lm * 4, 0, 0));
  };
  auto fetch = [&](int q, u32x4& ar, u32x4& ar2, u32x4& ar3) {
    const int lm = row_of(q);
    if constexpr (R_F32) {
      const uint32_t off = (uint32_t)(lm * ldR) + col_off(across(q), 4u);
      ar = __builtin_amdgcn_raw_buffer_load_b128(rsR, (int)off, 0, 0);
      ar3 = __builtin_amdgcn_raw_buffer_load_b128(rsR, (int)(off + 16u), 0, 0);
    } else if constexpr (HAS_R) {
      ar = __builtin_amdgcn_raw_buffer_load_b128(rsR, (int)((uint32_t)(lm * ldR) + col_off(across(q), 2u)), 0, 0);
    }
    if constexpr (HAS_R2) ar2 = __builtin_amdgcn_raw_buffer_load_b128(rsR2, (int)((uint32_t)(lm * ldR2) + col_off(across(q), 2u)), 0, 0);
  };
  static_for<PF>([&](auto Q) {
    constexpr int q = decltype(Q)::value;
    auxr[q] = u32x4{0u, 0u, 0u, 0u};
    auxr2[q] = u32x4{0u, 0u, 0u, 0u};
    if constexpr (R_F32) auxr3[q] = u32x4{0u, 0u, 0u, 0u};
    if constexpr (q < NQ) fetch(q, auxr[q], auxr2[q], auxr3[R_F32 ? q : 0]);
  });
  static_for<(PR < NQ ? PR : NQ)>([&](auto Q) {
    constexpr int q = decltype(Q)::value;
    ssv[q] = 0.f;
    rbv[q] = 0.f;
    fetch_row(q, ssv[q], rbv[q]);
  });
  if constexpr (STAT_A)
    static_for<NQ>([&](auto Q) { ssv[decltype(Q)::value] = sStat[row_of(decltype(Q)::value)]; });
  if constexpr (STAT_A && Stage::STAT_IN_STAGE) {   // read by all before anyone writes there
    wait_lgkmcnt0();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  }
  static_for<NQ>([&](auto Q) {
    constexpr int q = decltype(Q)::value;
    constexpr int i = q / (NH * NJ * PPS), h = q / (NJ * PPS) % NH, jj = q / PPS % NJ, p = q % PPS;
    // the accumulators hold the transposed 32x32 block (the MFMA is issued with its operands
    // exchanged): lane -> row lane%32, registers 4g..4g+3 -> columns 8g + 4*(lane/32) + 0..3, so a lane
    // stages four consecutive columns with one 16-byte write.
    // No barrier: the staging region belongs to this wavefront alone and a wavefront's LDS
    // operations complete in order.
    if constexpr (Stage::SR == 16 && h == 0 && jj == 0 && p == 0) {
      // Rows 0..15 of two neighbouring MFMA blocks come together: lanes 16..31 and 48..63 of the left block (its rows
      // 16..31) change places with lanes 0..15 and 32..47 of the right one.  Then lane -> row lane%16, block (lane/16)%2.
      static_for<T::FN / 2>([&](auto J) {
        constexpr int j = decltype(J)::value;
#pragma unroll
        for (int v = 0; v < 16; v++) {
          const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[i][2 * j][v]), __float_as_uint(acc[i][2 * j + 1][v]),
                                                           false, false);
          acc[i][2 * j][v] = __uint_as_float(sw[0]);
          acc[i][2 * j + 1][v] = __uint_as_float(sw[1]);
        }
      });
    }
    if constexpr (DUAL && p == 0) {
      // the gate's piece through the staging space first: rows of eight columns, rounded as they are stored
      if constexpr (Stage::SR == 32) {
        static_for<T::FN>([&](auto J) {
#pragma unroll
          for (int g = 0; g < 4; g++)
            *reinterpret_cast<uint2*>(stage.at(lane & 31, decltype(J)::value * 4 + g) + (lane >> 5) * 8) = accg.v[i][decltype(J)::value][g];
        });
      } else {
#pragma unroll
        for (int g = 0; g < 4; g++) {
          // (as below: rows 0..15 of two neighbouring blocks, then their rows 16..31)
          const uint2 l = accg.v[i][2 * jj][g], r = accg.v[i][2 * jj + 1][g];
          const auto sx = __builtin_amdgcn_permlane16_swap(l.x, r.x, false, false), sy = __builtin_amdgcn_permlane16_swap(l.y, r.y, false, false);
          *reinterpret_cast<uint2*>(stage.at(lane & 15, (lane >> 4 & 1) * 4 + g) + (lane >> 5) * 8) = make_uint2(sx[h], sy[h]);
        }
      }
#pragma unroll
      for (int pp = 0; pp < PPS; pp++) gate[pp] = *reinterpret_cast<const uint4*>(stage.at(pp * RPP + rsub, cg));
    }
    if constexpr (p == 0) {
      auto put = [&](int row, int chunk, const f32x16& a) {
#pragma unroll
        for (int g = 0; g < 4; g++)
          *reinterpret_cast<f32x4*>(stage.at(row, chunk + 2 * g)) = f32x4{a[4 * g], a[4 * g + 1], a[4 * g + 2], a[4 * g + 3]};
      };
      if constexpr (Stage::SR == 32)
        static_for<T::FN>([&](auto J) { put(lane & 31, decltype(J)::value * 8 + (lane >> 5), acc[i][decltype(J)::value]); });
      else
        put(lane & 15, (lane >> 4 & 1) * 8 + (lane >> 5), acc[i][2 * jj + h]);
    }
    const int rl = p * RPP + rsub;                // row inside the piece
    const int lm = row_of(q);                     // row inside the block tile
    float v[8];
    {
      // (vector types: of a struct's member accesses the compiler would make each wait for the LDS loads in flight)
      const f32x4 lo = *reinterpret_cast<const f32x4*>(stage.at(rl, 2 * cg));
      const f32x4 hi = *reinterpret_cast<const f32x4*>(stage.at(rl, 2 * cg + 1));
      v[0] = lo.x; v[1] = lo.y; v[2] = lo.z; v[3] = lo.w;
      v[4] = hi.x; v[5] = hi.y; v[6] = hi.z; v[7] = hi.w;
    }
    if constexpr (PARTIAL) {
      const uint32_t off = (uint32_t)(lm * ldC) + col_off(jj, 4u);
      const u32x4 lo = {__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])};
      const u32x4 hi = {__float_as_uint(v[4]), __float_as_uint(v[5]), __float_as_uint(v[6]), __float_as_uint(v[7])};
      __builtin_amdgcn_raw_buffer_store_b128(lo, rsC, (int)off, 0, 0);
      __builtin_amdgcn_raw_buffer_store_b128(hi, rsC, (int)(off + 16u), 0, 0);
    } else {
      float rho = 1.f, rowb = 0.f;
      if (use_rho) {
        const float ss = ssv[q % PR];
        rho = rho_sqrt ? sqrtf(ss * inv_d + eps) : rsqrtf(ss * inv_d + eps);
      }
      if constexpr (BASE == EPI_NORMBWD) rowb = rbv[q % PR];
      float r[8], r2[8], v2[8];
      if constexpr (R_F32) {
        const u32x4 a0 = auxr[q % PF], a1 = auxr3[q % PF];
        r[0] = __uint_as_float(a0.x); r[1] = __uint_as_float(a0.y); r[2] = __uint_as_float(a0.z); r[3] = __uint_as_float(a0.w);
        r[4] = __uint_as_float(a1.x); r[5] = __uint_as_float(a1.y); r[6] = __uint_as_float(a1.z); r[7] = __uint_as_float(a1.w);
      } else if constexpr (DUAL) {
        unpack8(gate[p], r);
        const u32x4 gv = {gate[p].x, gate[p].y, gate[p].z, gate[p].w};
        __builtin_amdgcn_raw_buffer_store_b128(gv, rsR, (int)((uint32_t)(lm * ldR) + col_off(jj, 2u)), 0, 0);
      } else {
        unpack8(make_uint4(auxr[q % PF].x, auxr[q % PF].y, auxr[q % PF].z, auxr[q % PF].w), r);
      }
      unpack8(make_uint4(auxr2[q % PF].x, auxr2[q % PF].y, auxr2[q % PF].z, auxr2[q % PF].w), r2);
      float part = epi_math<8, BASE, true>(act, inv_d, want2, v, v2, rho, rowb, r, r2);
      if constexpr (O32) {
        const u32x4 lo = {__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])};
        const u32x4 hi = {__float_as_uint(v[4]), __float_as_uint(v[5]), __float_as_uint(v[6]), __float_as_uint(v[7])};
        const uint32_t off = (uint32_t)(lm * ldC32) + col_off(jj, 4u);
        __builtin_amdgcn_raw_buffer_store_b128(lo, rsC32, (int)off, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b128(hi, rsC32, (int)(off + 16u), 0, 0);
      }
      {
        const uint4 o = pack8(v);
        const u32x4 ov = {o.x, o.y, o.z, o.w};
        __builtin_amdgcn_raw_buffer_store_b128(ov, rsC, (int)((uint32_t)(lm * ldC) + col_off(jj, 2u)), 0, 0);
      }
      if (want2) {
        const uint4 o = pack8(v2);
        const u32x4 ov = {o.x, o.y, o.z, o.w};
        __builtin_amdgcn_raw_buffer_store_b128(ov, rsC2, (int)((uint32_t)(lm * ldC2) + col_off(jj, 2u)), 0, 0);
      }
      if constexpr (q + PR < NQ) fetch_row(q + PR, ssv[q % PR], rbv[q % PR]);
      if constexpr (q + PF < NQ) fetch(q + PF, auxr[q % PF], auxr2[q % PF], auxr3[R_F32 ? q % PF : 0]);
      if constexpr (ROWPART) {
        part = lane_group_sum<LPP>(part);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(part), rsPart, (int)((uint32_t)(lm * ldPart) + colPart + jj * (Stage::SC / (LPP * 8)) * 4), 0, 0);
      }
      if constexpr (STAT_A && jj == 0)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(ssv[q]), rsStat, (int)((uint32_t)(lm * 4) + colStat), 0, 0);
    }
  });
}

}  // namespace
}  // namespace lrb
