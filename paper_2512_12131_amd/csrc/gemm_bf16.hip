// bf16 MFMA GEMM for gfx950:  C[M,N] = epi( sum_k A[m,k] * B[n,k] ), fp32 accumulate.
//
// The 256-row tiles, and the choice between them and the smaller ones of gemm_ring.h.
//
// Two operand forms.  k-contiguous ("NT": the forward projections x.W^T, and those data gradients that run on
// these tiles, on a transposed copy of the weight; the smaller tiles read it in place): slices land in LDS as
// [row][k] and the MFMA operands are plain 16-byte reads.  k-major (weight gradients, which reduce over tokens): slices
// land as [k][column] and the operands are gathered with the LDS transpose read.  The k-major form with
// a plain bf16 store, batched with two-level strides and with the k range of a row tile cut at its last
// row, also computes the attention's query gradient from the stored score gradient.
//
// Work decomposition: one workgroup owns a BM x BN output tile at a time, WM x WN wavefronts each own a
// (BM/WM) x (BN/WN) sub-tile built from 32x32x16 MFMA blocks (256x256 by 8 wavefronts, two per SIMD,
// or 256x128 by 4).  The k loop moves 64-wide slices straight from global memory into LDS
// (buffer_load ... lds, no register staging, whole 128-byte cache lines per row) through a ring of
// three A slots and two B slots, one workgroup barrier per slice, the loads of a slice spread over
// its four k16 steps; the 16-byte chunk index of a row is XOR-swizzled so that the MFMA-operand reads
// spread over all banks.  The accumulator tile (held transposed: the MFMAs are issued with their
// operands exchanged) leaves through LDS as well, so that every global access of the epilogue (C, the
// auxiliary tiles it reads, the secondary output) is a row-contiguous 16-byte vector through a per-tile
// buffer resource, without branches.  Workgroups map to tiles XCD by XCD in compact panels and all walk k front to back, so that
// the tiles resident in one XCD share operand slices in its L2.
//
// A launch has at most one workgroup per CU, and a workgroup walks all its tiles in one stream of slices.  (The causal product of
// the attention keeps a workgroup per tile: see launch.)  What bounds
// a launch with k of 512 or 1024 is the time outside the main loop: with a workgroup per tile 9 us of each 33 us (K = 1024,
// plain store) went into its start, the wait for its first slices and the drain of its stores, with the matrix pipes idle.
// Now the first two slices of the next tile are under way before the epilogue starts, and the epilogue's stores drain behind
// the next tile's first slice.  us, a workgroup per tile -> one stream (inside a block step):
//   16384 x 11008 x 1024, plain store        341 -> 304      same, SwiGLU forward            442 -> 385
//   16384 x  4096 x 1024, three members      366 -> 342      same, SwiGLU backward           543 -> 478
//   16384 x  2048 x  512, three members      113 -> 106      11008 x 1024 x 16384 k-major    349 -> 337
// Launches of one tile per CU have nothing to stream to and take what they took: 16384 x 1024 x 4096 111.1 -> 108.7, 777 x 11008 x 1024 27.8 ->
// 27.6, k of one slice 1024 x 12288 x 64 12.2 -> 11.8; up to 5 % longer is the re-forward's residual sum over a short k (16384 x 1024 x 256
// 25.2 -> 26.4).
// The four-kilobyte staging space that this leaves a wavefront gives the epilogue rows of 128 bytes.  Rows of 256 through the free B slot
// as well, with slice 1 of B loaded behind the epilogue, lost the gain (350 -> 350: its wait includes the stores); rows of 64
// bytes (one MFMA block at a time) made epilogues that read tiles up to 30 % slower.  Where rows start between cache lines a piece spans
// two of them: SwiGLU with u stored, 16384 x 5464 x 512 into a caller's dense rows, 213 -> 218 (in a workspace rows start on lines).
// A workgroup's share of tiles is fixed, and a CU is not free for another stream's workgroups before the launch ends (up to 500 us; with
// a workgroup per tile, a tile's time).  Beside a chain of attention forwards (4096 tokens, 4 heads) a group forward of 16384 tokens
// takes 1155 -> 949 us and each of them 105 -> 125; beside a kernel that holds 64 CUs for 0.5 ms at a time 1910 -> 1815.
#include <vector>

#include "gemm_tile.h"

namespace lrb {
namespace {

constexpr int NSA = 3;          // LDS slots of the A operand's slices: loads get two slices of lead
constexpr int NSB = 2;          // LDS slots of the B operand's slices: loads get one slice of lead
constexpr int NCU = 256;        // workgroups of a launch with more tiles than that: one per CU

template <int BM_, int BN_, int WM_, int WN_>
struct Tile {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_;
  static constexpr int NW = WM * WN, NT = NW * 64;
  static constexpr int TM = BM / WM, TN = BN / WN;
  static constexpr int FM = TM / 32, FN = TN / 32;
  static constexpr int A_BYTES = BM * 128, B_BYTES = BN * 128, STAGE = A_BYTES + B_BYTES;
  static constexpr int WLOADS = (BM + BN) / 8 / NW;   // 1 KB wavefront loads (8 rows x 128 B) per wavefront per stage
  static constexpr int WLOADS_A = BM / 8 / NW;        // the first WLOADS_A of them fetch A rows, the rest B rows
  static constexpr int MAIN_BYTES = NSA * A_BYTES + NSB * B_BYTES;
  static constexpr int LDS_BYTES = MAIN_BYTES;
  // The epilogue stages 16 rows x 64 columns per wavefront at a time (rows of a whole cache line of bf16), in four 1 KB pieces of
  // the free A slot that the wavefront's own global->LDS loads fill: what it has read back it may load over, without a
  // word to the others.  The XOR spreads what a cycle writes (one chunk of 16 rows) and reads (every second chunk of two
  // rows) over all banks.
  struct EpiStage {
    static constexpr int SR = 16, SC = 64;
    static constexpr bool STAT_IN_STAGE = true;
    unsigned char* p;
    __device__ __forceinline__ unsigned char* at(int row, int chunk) const {
      return p + (row >> 2) * (NW * 1024) + (row & 3) * 256 + ((chunk ^ row) << 4);
    }
  };
  // Behind the last tile all of LDS is free: whole rows of the wavefront's sub-tile.  The fp32 row stride is = 4 (mod 64), so the
  // 16 rows that one cycle of a 16-byte-per-lane write touches fall on 16 different groups of four banks.
  static constexpr int LAST_CS = TN + 4, LAST_BYTES = 32 * LAST_CS * 4;
  struct LastStage {
    static constexpr int SR = 32, SC = TN;
    static constexpr bool STAT_IN_STAGE = false;
    unsigned char* p;
    __device__ __forceinline__ unsigned char* at(int row, int chunk) const { return p + row * (LAST_CS * 4) + chunk * 16; }
  };
  static_assert(NW * LAST_BYTES <= LDS_BYTES, "staging of the last tile");
  static_assert(WLOADS_A >= 4, "a wavefront stages 4 KB in pieces of its own");
  static_assert(BM / 8 % NW == 0 && BN / 8 % NW == 0 && FM >= 1 && FN >= 1 && BM <= NT,
                "tile / wavefront layout mismatch");
};

// KM = false: operands k-contiguous, A[m][k], B[n][k].
// KM = true:  operands k-major,      A[k][m], B[k][n]  (weight gradients: k runs over tokens).  The
//             slices are stored in LDS as they arrive, [k][m], and the MFMA operands are gathered
//             with the LDS transpose read, so no transposed copy of an activation is ever written.
template <class T, int KIND, bool STAT_A, bool KM>
__global__ __launch_bounds__(T::NT) void gemm_bf16_kernel(GemmOp op, int kper, int tiles_m, int tiles_n, int total, int stagger) {
  static_assert(!KM || ((KIND == EPI_PARTIAL || KIND == EPI_STORE) && !STAT_A && T::BM == 256 && T::BN % 128 == 0),
                "the k-major form serves split-K weight gradients and plain stores");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / T::WN, wn = wave % T::WN;

  // All cache lines of the arguments at once: they come from the host's memory, and the code ahead of the first loads, which asks for them
  // as it needs them, waited 4 (plain store) to 9 times (EPI_DOWN) one after the other.  us, then -> now (a workgroup per tile, with 3 waits):
  // 8192 x 1536 x 2048 60.9 -> 59.5 (62.6), residual sums 16384 x 1024 x 256 27.7 -> 27.3 (26.5), 8000 x 2048 x 320 35.9 -> 34.8 (35.2).
  {
    constexpr int LINES = (sizeof(GemmOp) + 5 * sizeof(int) + 63) / 64;
    static_assert(LINES == 6, "the lines asked for below");
    const uint32_t* args = (const uint32_t*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" ::"s"(args[0]), "s"(args[16]), "s"(args[32]), "s"(args[48]), "s"(args[64]), "s"(args[80]));
  }

  // ---- tiles of this workgroup -----------------------------------------------------------------
  // The hardware deals workgroups round-robin to the XCDs; each XCD works through a contiguous range of tiles, its
  // workgroups side by side.
  const int bid = blockIdx.x + gridDim.x * blockIdx.y, nwg = gridDim.x * gridDim.y;
  const int xcd = bid % NXCD;
  const int step = nwg / NXCD + (xcd < nwg % NXCD ? 1 : 0);             // workgroups on this XCD
  // (see launch)
  for (int i = 0; i < xcd * stagger; i++) __builtin_amdgcn_s_sleep(16);
  const int tiles_first = xcd * (total / NXCD) + min(xcd, total % NXCD);
  const int tiles_end = tiles_first + total / NXCD + (xcd < total % NXCD ? 1 : 0);

  // Where a tile's slices come from.  rec_*: bytes behind base_* that may be read; what lies beyond (rows past the
  // matrix, or everything for the tile after the last one) arrives as zeros.
  struct Source {
    const uint16_t *base_a, *base_b;
    uint32_t rec_a, rec_b;
    int klen, nk;                        // k elements, 64-wide slices
    int m0, n0, tn, b, bi, bo, bz;
  };
  // At least one slice, and two where a tile follows another: two slices of the next tile are under way before an epilogue, and may not
  // reach into a third.  (Two for all, us: 1024 x 12288 x 64 12.1 -> 13.2, 4096 x 4096 x 40 13.6 -> 14.6.)
  const int nk_min = total > nwg ? 2 : 1;
  auto source = [&](int nid) -> Source {
    Source s;
    int tm;
    tile_of_index(nid, tiles_m, tiles_n, tm, s.tn, s.bz);
    if (KM && op.causal_k) tm = tiles_m - 1 - tm;   // the longest k ranges of a batch member first
    s.m0 = tm * T::BM;
    s.n0 = s.tn * T::BN;
    s.b = s.bz / op.splitk;
    const int kbeg = s.bz % op.splitk * kper;
    int kend = min(op.K, kbeg + kper);
    if (KM && op.causal_k) kend = min(kend, s.m0 + T::BM);
    s.klen = max(kend - kbeg, 0);
    s.nk = max((s.klen + BK - 1) / BK, nk_min);
    // element offsets of this batch entry's operands
    s.bo = op.batch_inner > 0 ? s.b / op.batch_inner : 0;
    s.bi = op.batch_inner > 0 ? s.b % op.batch_inner : s.b;
    const uint16_t* A = (const uint16_t*)op.A + (int64_t)s.bi * op.sA + (int64_t)s.bo * op.sAo;
    const uint16_t* B = (const uint16_t*)op.B + (int64_t)(s.bi / op.b_group) * op.sB + (int64_t)s.bo * op.sBo;
    s.base_a = KM ? A + (int64_t)kbeg * op.lda + s.m0 : A + (int64_t)s.m0 * op.lda + kbeg;
    s.base_b = KM ? B + (int64_t)kbeg * op.ldb + s.n0 : B + (int64_t)s.n0 * op.ldb + kbeg;
    // first to last element of the tile's rows, k-contiguous: [rows][klen], k-major: [klen][columns]
    auto extent = [&](int64_t rows, int64_t cols, int64_t ld) -> uint32_t {
      return s.klen > 0 ? (uint32_t)min((int64_t)0x7fffffff, ((rows - 1) * ld + cols) * 2) : 0u;
    };
    s.rec_a = KM ? extent(s.klen, op.M - s.m0, op.lda) : extent(min(T::BM, op.M - s.m0), s.klen, op.lda);
    s.rec_b = KM ? extent(s.klen, op.N - s.n0, op.ldb) : extent(min(T::BN, op.N - s.n0), s.klen, op.ldb);
    return s;
  };
  int nid = tiles_first + bid / NXCD;
  Source cur = source(nid), nxt = cur;

  // ---- global -> LDS, without passing through registers ---------------------------------------
  // One buffer_load_dwordx4 ... lds per wavefront moves 8 tile rows x 128 bytes (1 KB, eight whole
  // cache lines): lane L's 16 bytes land at LDS base + 16 L, i.e. tile row L/8, physical chunk L%8.
  // The 16-byte chunks of a row are stored XOR-swizzled by (row/2)%8, so each lane fetches the logical
  // chunk that belongs in its slot; MFMA operand reads (32 rows x one logical chunk) then spread over
  // all banks.  A lane whose chunk lies outside the matrix (row tail, k tail) uses an offset past the
  // resource size: the load returns zeros and zeros are what reaches LDS.
  // k-contiguous form: 8 rows x 128 B per wavefront load; k-major form: 2 k-rows x 512 B (BM = 256
  // columns) or 4 k-rows x 256 B (128 columns).  In both, the 16-byte chunk index inside a row is
  // XOR-swizzled so that the operand reads spread over the banks.
  // Swizzle of the k-contiguous form: physical chunk = logical chunk ^ ((row / 2) % 8).  An LDS row is
  // 128 bytes, half of the 64 x 4-byte banks, so rows 2i and 2i+1 lie side by side in one bank line;
  // with this term the 16 rows that one cycle of a 16-byte-per-lane read touches (16 lanes) fall on
  // 16 different 16-byte bank groups.  The 1 KB group index g = wave + NW * i keeps its parity over i
  // (NW is even), so one swizzle value per lane serves all of its loads.
  // k-major: rows past k lie behind the resource's end; a column chunk past the matrix is left out (read into the next k-row it
  // would only feed rows or columns that are not stored, but it costs its bytes: dQ of 9 x 1032 tokens, 32 heads, 8 of the last
  // tile's 256 rows in the matrix, 149 us against 133).  A lane's columns are the same in all its loads: NW * RPL is a multiple of 8.
  // The offsets below hold for every slice of every tile; a slice's own offset is added per lane.  (Advancing the resource's base
  // instead saves a vector addition per load, but its chains of scalar instructions stand between a slice's barrier and its first
  // MFMA: 90 scalar instructions per slice against 65, 2 % of a launch.  us, base advanced -> offset added: 1000 x 11008 x 1024
  // 28.1 -> 27.3, 16384 x 11008 x 1024 in a block step 311 -> 306, 16384 x 1024 x 4096 109.9 -> 107.1.)
  constexpr uint32_t OOB = 0x80000000u;
  static_assert(T::NW % 2 == 0 && (T::BM / 8) % 2 == 0, "row parity of a lane must not depend on the load index");
  const int lrow = lane >> 3, lchunk = (lane & 7) ^ (((wave & 1) << 2) | (lrow >> 1));
  uint32_t goff[T::WLOADS];
  int kcol_a = 0, kcol_b = 0;                            // first column of this lane's chunks (k-major)
#pragma unroll
  for (int i = 0; i < T::WLOADS; i++) {
    const bool isA = i < T::WLOADS_A;
    const int g = wave + T::NW * i - (isA ? 0 : T::BM / 8);   // 1 KB group of the operand
    const int64_t ld = isA ? op.lda : op.ldb;
    int64_t off;
    if constexpr (!KM) {
      off = ((g * 8 + lrow) * ld + lchunk * 8) * 2;
    } else {
      const int CPR = (isA ? T::BM : T::BN) / 8, RPL = 64 / CPR;       // chunks per k-row, k-rows per wavefront load
      const int krow = g * RPL + lane / CPR;
      const int col = ((lane % CPR) ^ (((krow & 7) << 2) & (CPR - 1))) * 8;
      (isA ? kcol_a : kcol_b) = col;
      off = (krow * ld + col) * 2;
    }
    goff[i] = off < (int64_t)OOB ? (uint32_t)off : OOB;
  }
  // Every workgroup walks its k range in the same order, front to back.  The workgroups of an XCD
  // that share A rows or B rows (one panel of tiles) then want the same k slice at about the same time,
  // and all but the first request for it hit in that XCD's L2: walking from staggered starting slices
  // instead multiplied the traffic out of L2 by 3.6 and cost 12-18% of the GEMM rate.  The fixed order
  // also makes the summation order of a token row independent of how sequences are batched.
  // Slots: A slices cycle through NSA slots at the bottom of LDS, B slices through NSB above, on from tile to tile.
  // a0, a1, a2: slots of slices kt, kt + 1, kt + 2 (and of kt - 1); b0, b1 those of kt, kt + 1.
  uint32_t a0 = 0, a1 = T::A_BYTES, a2 = 2 * T::A_BYTES, b0 = NSA * T::A_BYTES, b1 = b0 + T::B_BYTES;
  constexpr int WLOADS_B = T::WLOADS - T::WLOADS_A;
  // issue_ab(kt, dst, IS_A, HALF): HALF = 0 / 1 issues the first / second half of the operand's loads of
  // slice kt of this tile, or past its end of the next one, HALF = 2 all of them
  auto issue_ab = [&](int kt, uint32_t slot, auto IS_A, auto HALF) {
    constexpr bool isA = decltype(IS_A)::value;
    constexpr int half = decltype(HALF)::value;
    const bool here = kt < cur.nk;
    const int ks = here ? kt : kt - cur.nk, klen = here ? cur.klen : nxt.klen;
    const uint32_t skip = (uint32_t)ks * (uint32_t)(KM ? BK * 2 * (isA ? op.lda : op.ldb) : BK * 2);     // bytes before this slice
    const uint32_t rec = here ? (isA ? cur.rec_a : cur.rec_b) : (isA ? nxt.rec_a : nxt.rec_b);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(here ? (isA ? cur.base_a : cur.base_b) : (isA ? nxt.base_a : nxt.base_b)), 0, rec, 0x00020000);
    // chunks past the end of k or of the columns (k-major form) read as zeros.  (k-major, whole slices past the end of k: skip may
    // have wrapped.  Elsewhere offset and skip are each below 2 GB or OOB, and their sum is past the resource or right.)
    bool inside;
    if constexpr (KM)
      inside = ks * BK < klen && (isA ? kcol_a + (here ? cur.m0 : nxt.m0) : kcol_b + (here ? cur.n0 : nxt.n0)) < (isA ? op.M : op.N);
    else
      inside = ks * BK + lchunk * 8 < klen;
    const uint32_t mask = inside ? 0u : OOB;
    unsigned char* dst = smem + slot + wave * 1024;
    constexpr int F0 = isA ? 0 : T::WLOADS_A, F1 = isA ? T::WLOADS_A : T::WLOADS;   // the operand's loads
    constexpr int I0 = half == 1 ? (F0 + F1) / 2 : F0, I1 = half == 0 ? (F0 + F1) / 2 : F1;
#pragma unroll
    for (int i = I0; i < I1; i++)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, LRB_LDS_PTR(dst + (i - F0) * (T::NW * 1024)), 16,
                                               (int)((goff[i] + skip) | mask), 0, 0, 0);
  };
  using Half0 = std::integral_constant<int, 0>;
  using Half1 = std::integral_constant<int, 1>;
  using Whole = std::integral_constant<int, 2>;

  f32x16 acc[T::FM][T::FN];

  // MFMA operand addressing: row = lane%32 of a 32-row block, logical chunk kk*2 + lane/32
  const int frow = lane & 31, fk = lane >> 5, fsw = (frow >> 1) & 7;
  bf16x8 af[2][T::FM], bf[2][T::FN];
  // k-major form, transpose reads.  Inside each group of 16 lanes, lane s supplies the address of 4
  // consecutive columns of k-row (s/4) and receives column s of the 4 x 16 block; two reads (k-rows +0 and
  // +8) give the 8 k slots of a lane: slot (half, e) -> k = kk*16 + (e/4)*8 + half*4 + e%4, the same
  // assignment for both operands.  The lane-dependent part of every fragment address (k-row inside a
  // k16 step, swizzled column chunk) does not change over the main loop and is computed once; the slot
  // of the slice is added per fragment, the k16 step and the +8 rows ride in the instruction's offset.
  uint32_t troffA[KM ? T::FM : 1], troffB[KM ? T::FN : 1];
  if constexpr (KM) {
    const int g = lane >> 4, sl = lane & 15;
    const int krow0 = (g >> 1) * 4 + (sl >> 2);
    const int ksw = (krow0 & 7) << 2;                     // (krow0 + 8 n) & 7 is the same
    const int cin = (g & 1) * 16 + (sl & 3) * 4;          // column inside the 32-column block
    auto lane_off = [&](int pitch, int col, int swz) {
      return (uint32_t)(krow0 * pitch + ((((col >> 3) ^ swz) << 4) + (col & 7) * 2));
    };
#pragma unroll
    for (int i = 0; i < T::FM; i++) troffA[i] = lane_off(T::BM * 2, wm * T::TM + i * 32 + cin, ksw);
#pragma unroll
    for (int j2 = 0; j2 < T::FN; j2++) troffB[j2] = lane_off(T::BN * 2, wn * T::TN + j2 * 32 + cin, ksw & (T::BN / 8 - 1));
  }
  auto load_frags = [&](int buf, uint32_t slot_a, uint32_t slot_b, auto KKc) {
    constexpr int kk = decltype(KKc)::value;
    if constexpr (!KM) {
      const unsigned char* sa = smem + slot_a + (wm * T::TM + frow) * 128;
      const unsigned char* sb = smem + slot_b + (wn * T::TN + frow) * 128;
      const int coff = ((kk * 2 + fk) ^ fsw) << 4;
#pragma unroll
      for (int i = 0; i < T::FM; i++) af[buf][i] = *reinterpret_cast<const bf16x8*>(sa + i * 32 * 128 + coff);
#pragma unroll
      for (int j = 0; j < T::FN; j++) bf[buf][j] = *reinterpret_cast<const bf16x8*>(sb + j * 32 * 128 + coff);
    } else {
      typedef short s16x4 __attribute__((ext_vector_type(4)));
      typedef short s16x8 __attribute__((ext_vector_type(8)));
      // The transpose reads are issued as inline assembly.  Through the builtin, the compiler cannot
      // tell them from a read of the slot that the global->LDS loads in flight are writing, and puts a
      // wait for ALL outstanding global loads in front of each group of reads (which throws away the
      // two slices of load lead).  The price: the compiler does not wait for their results either, so
      // every k16 step of this form ends with an explicit wait for the LDS counter behind a scheduling
      // barrier (see the main loop).
      const uint32_t slotA = (uint32_t)(uintptr_t)LRB_LDS_PTR(smem + slot_a);
      const uint32_t slotB = (uint32_t)(uintptr_t)LRB_LDS_PTR(smem + slot_b);
      auto tr_pair = [&](uint32_t addr, auto PITCH) -> bf16x8 {
        constexpr int o0 = kk * 16 * decltype(PITCH)::value, o1 = o0 + 8 * decltype(PITCH)::value;
        static_assert(o1 < 65536, "LDS instruction offset field");
        s16x4 lo, hi;
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(addr), "n"(o0) : "memory");
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(addr), "n"(o1) : "memory");
        s16x8 r = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        return __builtin_bit_cast(bf16x8, r);
      };
#pragma unroll
      for (int i = 0; i < T::FM; i++) af[buf][i] = tr_pair(slotA + troffA[i], std::integral_constant<int, T::BM * 2>{});
#pragma unroll
      for (int j = 0; j < T::FN; j++) bf[buf][j] = tr_pair(slotB + troffB[j], std::integral_constant<int, T::BN * 2>{});
    }
  };
  // first operands of a tile (the reads of the k-major form are waited for here)
  auto first_frags = [&]() {
    load_frags(0, a0, b0, std::integral_constant<int, 0>{});
    if constexpr (KM) {
      wait_lgkmcnt0();
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto mfma_step = [&](int buf, auto ZERO) {
    constexpr f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < T::FM; i++)
#pragma unroll
      for (int j = 0; j < T::FN; j++)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[buf][j], af[buf][i], decltype(ZERO)::value ? zero : acc[i][j], 0, 0, 0);
  };
  // STAT_A: thread t accumulates the sum of squares of tile row t from the LDS copy, chunk by chunk as they lie there
  // (the ring kernels share a row among threads and add its chunks up in this order)
  float ssq = 0.f;
  auto stat_row = [&](int half) {
    if constexpr (STAT_A) {
      if (tid < T::BM) {
        const unsigned char* sr = smem + a0 + tid * 128 + half * 64;
#pragma unroll
        for (int c = 0; c < 4; c++) ssq += sumsq8(*reinterpret_cast<const uint4*>(sr + c * 16));
      }
    }
  };

  // ---- main loop ---------------------------------------------------------------------------------
  // Slice kt (64 wide) is multiplied in four k16 steps.  While step s runs, the operands of step s+1
  // are read from LDS.  Before step 3 a barrier establishes that every wavefront's part of slice
  // kt+1 has landed and that nobody reads slice kt's slots any more (the step-3 operands are in
  // registers).
  // The global->LDS loads are spread evenly over the four steps, because the CU's address/texture
  // path accepts about one 1 KB wavefront load per 23 cycles: issued in one burst they block the
  // issuing wavefronts (and with them their MFMAs) for most of a step.  LDS holds 3 slots for A
  // slices and 2 for B slices (5 x 32 KB), which allows this order inside iteration kt:
  //   step 0: second half of B(kt+1)      -> the slot B(kt-1) left at the previous barrier
  //   step 1, 2: the halves of A(kt+2)    -> the slot A(kt-1) left at the previous barrier
  //   barrier (needs A(kt+1), B(kt+1); loads retire in order, so A(kt+2) alone may stay in flight)
  //   step 3: first half of B(kt+2)       -> the slot B(kt) just left
  // The loop body is branch free: slices past the end of k are the next tile's, or, after the last tile, "loaded" with
  // every lane out of range (zeros into a slot nobody reads again), so the wait counts are compile-time constants.
  // Slices 0 and 1 of the next tile are on their way before this tile's epilogue starts, which stages through the one A
  // slot that then is free.  They do not wait for its stores either: slice 0 lets those fly.
  // Instruction interleave: a wavefront issues in order, and an MFMA occupies the matrix pipe for
  // 32 cycles during which the same wavefront may issue other work.  The scheduler is therefore
  // told to thread the LDS reads and global->LDS loads between the MFMAs instead of issuing them
  // in a burst while the matrix pipe idles.
  constexpr int MPR = (T::FM * T::FN) / (T::FM + T::FN);   // MFMAs per LDS operand read
  constexpr int HLA = T::WLOADS_A / 2, HLB = WLOADS_B / 2; // loads per half slice of A, of B
  constexpr std::true_type OPA{};
  constexpr std::false_type OPB{};
  // vector memory instructions that a wavefront's epilogue certainly issues behind the loads of slice 1 of the next tile
  constexpr int STORES = T::TM * T::TN / (64 * 8) * (KIND == EPI_PARTIAL ? 2 : 1);
  static_assert(T::WLOADS_A + STORES < 64, "vmcnt is a 6-bit counter");
  bool stores_fly = false;          // there was an epilogue
  // FIRST: slice 0 of a tile.  B(1) is on its way already, the accumulators start at zero.
  auto slice = [&](int kt, auto FIRST) {
    constexpr bool first = decltype(FIRST)::value;
    static_for<3>([&](auto KK) {
      constexpr int kk = decltype(KK)::value;
      load_frags((kk + 1) & 1, a0, b0, std::integral_constant<int, kk + 1>{});
      if constexpr (kk == 0 && !first) issue_ab(kt + 1, b1, OPB, Half1{});
      if constexpr (kk == 1) issue_ab(kt + 2, a2, OPA, Half0{});
      if constexpr (kk == 2) issue_ab(kt + 2, a2, OPA, Half1{});
      if constexpr (kk < 2) stat_row(kk);
      mfma_step(kk & 1, std::integral_constant<bool, first && kk == 0>{});
      constexpr int NL = kk > 0 ? HLA : first ? 0 : HLB;
#pragma unroll
      for (int i = 0; i < T::FM + T::FN; i++) {
        __builtin_amdgcn_sched_group_barrier(0x008, MPR, 0);   // MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, KM ? 2 : 1, 0);     // DS read
        if (i * NL / (T::FM + T::FN) != (i + 1) * NL / (T::FM + T::FN))
          __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   // VMEM read (global -> LDS)
      }
      if constexpr (KM) {
        __builtin_amdgcn_sched_barrier(0);
        wait_lgkmcnt0();                   // the next step's operands (inline-assembly reads) have arrived
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    if (first && stores_fly) wait_vmcnt<T::WLOADS_A + STORES>();
    else wait_vmcnt<T::WLOADS_A>();        // A(kt+1), B(kt+1) of this wavefront landed; A(kt+2) may fly
    wait_lgkmcnt0();                       // and its reads of slice kt's slots are complete
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    issue_ab(kt + 2, b0, OPB, Half0{});
    load_frags(0, a1, b1, std::integral_constant<int, 0>{});
    mfma_step(1, std::false_type{});
#pragma unroll
    for (int i = 0; i < T::FM + T::FN; i++) {
      __builtin_amdgcn_sched_group_barrier(0x008, MPR, 0);   // MFMA
      __builtin_amdgcn_sched_group_barrier(0x100, KM ? 2 : 1, 0);     // DS read
      if (i * HLB / (T::FM + T::FN) != (i + 1) * HLB / (T::FM + T::FN))
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   // VMEM read (global -> LDS)
    }
    if constexpr (KM) {
      __builtin_amdgcn_sched_barrier(0);
      wait_lgkmcnt0();
    }
    __builtin_amdgcn_sched_barrier(0);
    const uint32_t a = a0, b = b0;
    a0 = a1; a1 = a2; a2 = a;
    b0 = b1; b1 = b;
  };
  issue_ab(0, a0, OPA, Whole{});
  issue_ab(0, b0, OPB, Whole{});
  issue_ab(1, a1, OPA, Whole{});
  issue_ab(1, b1, OPB, Whole{});
  wait_vmcnt<T::WLOADS>();          // A(0), B(0) landed; A(1) and B(1) may fly
  __builtin_amdgcn_s_barrier();
  while (true) {
    const int nid_next = nid + step;
    const bool more = nid_next < tiles_end;
    if (more) {
      nxt = source(nid_next);
    } else {
      nxt.rec_a = 0;
      nxt.rec_b = 0;
      nxt.klen = 0;
    }
    first_frags();
    slice(0, std::true_type{});
    for (int kt = 1; kt < cur.nk; kt++) slice(kt, std::false_type{});
    // (opaque copies: otherwise the epilogue's address arithmetic is moved out of the loop over tiles, and spilled)
    int elane = lane, ewave = wave;
    asm volatile("" : "+v"(elane), "+s"(ewave));
    // Of the kinds only EPI_UP_O32 gains by whole rows for its last tile: its fp32 copy then leaves in runs of 512 bytes.  us, a
    // workgroup per tile / pieces of 64 columns / whole rows last: 8192 x 2048 x 512 49.2 / 51.6 / 49.7, 8192 x 4096 x 1024 119.6 /
    // 123.3 / 119.4, 16384 x 4096 x 1024 235.3 / 239.1 / 235.7.  Others, pieces / whole rows: plain stores 1000 x 11008 x 1024
    // 33.1 / 33.3, EPI_DOWN 16384 x 1024 x 2048 70.1 / 71.1, EPI_NORMBWD_O32 8192 x 2048 x 1024 63.0 / 65.7.
    if (KIND == EPI_UP_O32 && !more) {
      wait_vmcnt<0>();             // this wavefront's loads past the last tile have written their zeros, then everyone's
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      gemm_epilogue<T, KIND, STAT_A>(op, acc, typename T::LastStage{smem + wave * T::LAST_BYTES}, nullptr, ewave, elane, cur.m0, cur.n0,
                                     cur.tn, tiles_n, cur.b, cur.bi, cur.bo, cur.bz);
      return;
    }
    issue_ab(cur.nk + 1, b1, OPB, Half1{});
    __builtin_amdgcn_sched_barrier(0);
    // ---- epilogue: a2 is the free slot -------------------------------------------------------------
    if constexpr (STAT_A) {
      float* sStat = reinterpret_cast<float*>(smem + a2);
      if (tid < T::BM) sStat[tid] = ssq;
      ssq = 0.f;
      wait_lgkmcnt0();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    }
    gemm_epilogue<T, KIND, STAT_A>(op, acc, typename T::EpiStage{smem + a2 + wave * 1024},
                                   reinterpret_cast<const float*>(smem + a2), ewave, elane, cur.m0, cur.n0, cur.tn, tiles_n, cur.b,
                                   cur.bi, cur.bo, cur.bz);
    if (!more) break;
    stores_fly = true;
    nid = nid_next;
    cur = nxt;
  }
  wait_vmcnt<STORES>();          // no load into LDS outlives its workgroup
}

// ---------------------------------------------------------------------------------------------
template <class T, int KIND, bool STAT_A, bool KM = false>
hipError_t launch(const GemmOp& op, hipStream_t st) {
  // one-time opt-in to > 64 KB of dynamic LDS for this instantiation (a function-local static: its
  // initialisation is thread-safe and runs once per process; a failure is reported by every launch)
  auto kern = gemm_bf16_kernel<T, KIND, STAT_A, KM>;
  static const hipError_t attr_err =
      hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
  if (attr_err != hipSuccess) return attr_err;
  const int tiles_m = (op.M + T::BM - 1) / T::BM, tiles_n = (op.N + T::BN - 1) / T::BN;
  int kper = (op.K + op.splitk - 1) / op.splitk;
  kper = (kper + BK - 1) / BK * BK;
  const int64_t total = (int64_t)tiles_m * tiles_n * op.batch * op.splitk;
  // causal k ranges differ from tile to tile: a workgroup each, dealt out as CUs become free
  const dim3 grid = op.causal_k || total <= NCU ? tile_grid(tiles_m * tiles_n, op.batch * op.splitk) : dim3(NCU);
  // SwiGLU epilogues move up to 512 KB per tile, 134 MB of a round of 256 tiles, 25 of its 48 us at k = 1024, with the matrix pipes
  // idle; then all main loops leave memory idle.  The XCDs start 768 cycles per slice of k apart (in units of 1024), 3/8 of the matrix
  // time of a slice, and one's epilogues run beside the others' main loops: up to 6 us off a round, for a last XCD that starts 7 x 768
  // cycles per slice of k late (36 us at k = 1024).  So it takes rounds enough, and more of them for longer k.  Against starting together,
  // 311 launches of 8192 to 16384 tokens x 2752 .. 16384 over k of 256 .. 2048: of the 145 under the rule none is more than 1.2 % slower,
  // on average the forward is 2.1 % faster and the reverse, which moves more, 1.7 %.  us, together -> apart, forward: five rounds 8192 x
  // 10240 x 512 129 -> 138, six 12288 x 8192 x 512 149 -> 154, seven 16384 x 7168 x 512 181 -> 178, eight 16384 x 8192 x 512 222 -> 213,
  // with u stored 278 -> 263; reverse: five 8192 x 10240 x 512 180 -> 184, six 8192 x 12264 x 512 242 -> 231.  The rounds for a k: 16384 x
  // 8192 x 1024 (half a round per slice) 303 -> 297, 8192 x 11008 x 1024 (0.31) 214 -> 222, 16384 x 11008 x 2048 (0.31) 637 -> 681; the
  // line is at 9/16.
  // Half and a quarter of the delay gain less (16384 x 8192 x 512 222 -> 220, 223).  Of other kinds the start costs more than it
  // gives (16384 x 4096 x 2048, norm's reverse 341 -> 350, plain stores of k = 1024 320 -> 340).
  const int nk = kper / BK;
  const int64_t rounds = total / NCU;
  const bool enough = KIND == EPI_SWIGLU_FWD ? rounds >= 7 : KIND == EPI_SWIGLU_BWD && rounds >= 6;
  const int stagger = enough && grid.y == 1 && rounds * 16 >= nk * 9 ? nk * 3 / 4 : 0;
  hipLaunchKernelGGL(kern, grid, dim3(T::NT), T::LDS_BYTES, st, op, kper, tiles_m, tiles_n, (int)total, stagger);
  return hipGetLastError();
}

using TileBig = Tile<256, 256, 4, 2>;   // 8 waves, 64x128 per wave
using TileMid = Tile<256, 128, 2, 2>;   // 4 waves, 128x64 per wave (two k-major operands)

template <class T>
hipError_t dispatch(const GemmOp& op, hipStream_t st) {
  const int kind = op.splitk > 1 ? (int)EPI_PARTIAL : op.epi.kind;
  switch (kind) {
    case EPI_STORE: return launch<T, EPI_STORE, false>(op, st);
    case EPI_DOWN:
      return op.epi.stat_from_a ? launch<T, EPI_DOWN, true>(op, st) : launch<T, EPI_DOWN, false>(op, st);
    case EPI_UP: return launch<T, EPI_UP, false>(op, st);
    case EPI_ACTGRAD: return launch<T, EPI_ACTGRAD, false>(op, st);
    case EPI_ACTGRAD_A: return launch<T, EPI_ACTGRAD_A, false>(op, st);
    case EPI_NORMBWD: return launch<T, EPI_NORMBWD, false>(op, st);
    case EPI_PARTIAL: return launch<T, EPI_PARTIAL, false>(op, st);
    case EPI_SWIGLU_BWD: return launch<T, EPI_SWIGLU_BWD, false>(op, st);
    case EPI_SWIGLU_FWD: return launch<T, EPI_SWIGLU_FWD, false>(op, st);
    case EPI_DOWN_LAX:
      return op.epi.stat_from_a ? launch<T, EPI_DOWN_LAX, true>(op, st) : launch<T, EPI_DOWN_LAX, false>(op, st);
    case EPI_LAXGRAD: return launch<T, EPI_LAXGRAD, false>(op, st);
    case EPI_UP_O32: return launch<T, EPI_UP_O32, false>(op, st);
    case EPI_UP_I32: return launch<T, EPI_UP_I32, false>(op, st);
    case EPI_NORMBWD_O32: return launch<T, EPI_NORMBWD_O32, false>(op, st);
    case EPI_NORMBWD_I32: return launch<T, EPI_NORMBWD_I32, false>(op, st);
    default: return hipErrorInvalidValue;
  }
}

// ---- which tile runs a launch --------------------------------------------------------------------
// Estimated microseconds of a launch.  A tile kind runs `slots` workgroups at a time; a round of them takes a
// fixed time f (pipeline fill), the epilogue g * e + h * e and nk 64-wide k slices of s0 + s1 each, where s1 and g
// are what the slices and the epilogue lose to each other when every slot is busy (they scale with the share
// of slots in use) and e is the traffic of the epilogue in units of one bf16 output.  The rows of T256, R64, R64X128 and R128
// are least-squares fits of the relative error over 1770 launches with k-contiguous operands (M 64 .. 16384, N 64 ..
// 11008, K 64 .. 11008, nine epilogue kinds), T256X128's over the plain stores among them; R32's is its measured slice time
// and start-up, set by hand.  All of these ran a workgroup per tile.  Against 1648 launches of the kernels as they are, T256 and R128 as
// streams among them (888 forward products, M from 16; 400 data gradients; 360 weight gradients), the estimates of tiles within 1.5 times
// the best are off by 7-17 % rms, 2-8 % too slow on average (data gradients on ring tiles 6 % too fast to 2 % too slow).  R128 as a stream
// is 10 % (forward) and 4 % (data gradients) faster than its estimate, T256 as one 2 to 15 %.  Taking the estimated best loses 0.9 %
// (forward) and 1.4 % (data gradients) in the geometric mean against the measured best, 28 % in the worst launch (16384 x 4096 x 256
// with the fp32 copy of the output: T256 184 us, R128 143), 13-23 % for weights 11008 wide on 256 and 1024 rows (R64X128 taken, R128
// faster); the 256-row tiles alone take 2.27 times as long as that over the forward products.  Forward products on R32 of up to
// 256 pieces of 16 x 16 run as those (gemm_rows16.hip): up to twice as fast with long k, which the estimate does not know (off by 32 %
// rms there).  What the lines amount to, with both sides measured (us, plain stores):
//   a handful of rows: one chain of k per CU        16 x 1024 x 4096:   T256 67.1   R64    14.6   R32 5.1
//   few tiles, the loads' latency decides          777 x 1024 x 4096:   T256 67.2   R64    16.4   R32 25.7
//   half the CUs idle under T256                 16384 x 512 x 2048:   T256 43.4   R128   35.1
//   N = 128 leaves T256 half its columns         16384 x 128 x 4096:   T256 70.0   R64x128 28.2
//   few tiles and short k                         8192 x 512 x 256:   T256 10.6   R64x128 6.8
//   the chip full                                16384 x 4096 x 256:   T256 46.2   R128   51.5
//                                                16384 x 4096 x 2048:  T256 214.4  R128   263.7
struct TileCost {
  int bm, bn, slots;
  float a, f, s0, s1, g, h;
};
constexpr TileCost kTileCost[] = {
    {0, 0, 0, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f},
    {256, 256, 256, 0.82f, 3.82f, 0.876f, 0.591f, 4.68f, 0.703f},   // GEMM_T256
    {256, 128, 256, 3.02f, 2.24f, 0.689f, 0.231f, 1.98f, 0.f},      // GEMM_T256X128
    {64, 64, 256, 1.89f, 1.80f, 0.169f, 0.029f, 0.22f, 0.141f},     // GEMM_R64
    {64, 128, 512, 2.08f, 1.38f, 0.231f, 0.306f, 1.05f, 0.095f},    // GEMM_R64X128
    {128, 128, 512, 2.48f, 0.80f, 0.479f, 0.451f, 2.42f, 0.142f},   // GEMM_R128
    {32, 32, 512, 2.00f, 1.00f, 0.095f, 0.080f, 0.30f, 0.140f},     // GEMM_R32
    {128, 128, 256, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f},                  // GEMM_R128W: causal products, chosen by rule below
};
// bf16-output equivalents an epilogue moves (reads and writes, secondary outputs included)
float epi_traffic(int kind) {
  switch (kind) {
    case EPI_STORE: return 1.f;
    case EPI_DOWN: case EPI_UP: case EPI_ACTGRAD: case EPI_PARTIAL: return 2.f;
    case EPI_UP_I32: case EPI_NORMBWD: case EPI_SWIGLU_FWD: case EPI_DOWN_LAX:
    case EPI_ACTGRAD_A: return 3.f;
    case EPI_UP_O32: case EPI_NORMBWD_I32: case EPI_SWIGLU_BWD: case EPI_LAXGRAD: return 4.f;
    default: return 5.f;   // EPI_NORMBWD_O32
  }
}
float epi_traffic(const GemmOp& op) {
  if (op.epi.kind == EPI_SWIGLU_DUAL) return 1.f + (op.epi.R ? 1.f : 0.f) + (op.C ? 1.f : 0.f);
  return epi_traffic(op.epi.kind);
}
// k slices of one workgroup
int op_slices(const GemmOp& op) {
  return (((op.K + op.splitk - 1) / op.splitk) + BK - 1) / BK * (op.epi.kind == EPI_SWIGLU_DUAL ? 2 : 1);
}
// nk: k slices of one workgroup; members: batch members times k splits; slice: factor on the slice time
float tile_time(int tile, int M, int N, int nk, int members, float e, float slice = 1.f) {
  const TileCost& c = kTileCost[tile];
  const long wgs = (long)((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn) * members;
  const long full = wgs / c.slots;
  const float u = (float)(wgs % c.slots) / (float)c.slots;
  float t = c.a + (float)full * (c.f + (c.g + c.h) * e + (float)nk * slice * (c.s0 + c.s1));
  if (u > 0.f) t += c.f + (c.g * u + c.h) * e + (float)nk * slice * (c.s0 + c.s1 * u);
  return t;
}
// From the end of one launch to the start of the next (see gemm_bf16_join_tile).
constexpr float kLaunchGap = 1.5f;
// The smaller tiles have to be estimated 7.5 % faster than T256 before they are taken: the estimate's own error.
constexpr float kRingMargin = 1.075f;
// What a slice costs more with two k-major operands.  The 256-row kernels pay for their transpose reads.  The ring
// tiles read 128 or 256 bytes per k row where those read 512, which shows when the rows come from HBM (2048 x 512
// over 16384 tokens: R64x128 in 4 splits 60 us, T256 in 16 splits 45 us plus 6 us more in the finishing pass).  With these
// factors the estimates of 360 weight gradients (512 .. 16384 tokens) are 8, 0, 11, 10, 11 and 5 % too slow on average.
constexpr float kKMajorSlice[] = {0.f, 1.13f, 1.05f, 1.5f, 1.5f, 1.3f, 1.5f};

}  // namespace

bool gemm_bf16_mixed_ok(const GemmOp& op) {
  return !op.transA && op.transB && op.splitk == 1 && gemm_bf16_tile(op) >= GEMM_R64;
}

int gemm_bf16_tile(const GemmOp& op) {
  if (op.tile != GEMM_TILE_AUTO) return op.tile;
  if (op.splitk > 1 || op.epi.kind == EPI_PARTIAL) return GEMM_T256;   // weight gradients come with a plan
  const bool dual = op.epi.kind == EPI_SWIGLU_DUAL;
  // a k-major weight is read in place in whole 8-column chunks, within the 2 GB a buffer resource addresses
  if (op.transB && !op.transA && (op.N % 8 || op.K % 8 || (int64_t)op.K * op.ldb * 2 >= 0x7fffffffLL)) return GEMM_T256;
  // Causal k ranges: tiles of unequal length, for which the estimate has no term.  Where the 256-row tiles give less
  // than two rounds their longest decides, and finer ones even them out (attention backward of 4 x 4096 tokens, 4
  // heads: 83 us on T256X128, 71 on R128W; 1 x 1024 tokens, 32 heads: 18.8 / 13.4); with more rounds the larger
  // tile reads less (4 x 4096 tokens, 32 heads: 553 / 583).  Fewer tiles than half the CUs: as any product.
  if (op.causal_k) {
    const int64_t members = (int64_t)((op.N + 127) / 128) * op.batch;
    if ((op.M + 255) / 256 * members >= 512) return GEMM_T256X128;
    if ((op.M + 127) / 128 * members >= 128) return GEMM_R128W;
  }
  const int nk = op_slices(op);
  const float e = epi_traffic(op);
  const bool km = op.transA && op.transB;
  float best = dual ? 1e30f : tile_time(GEMM_T256, op.M, op.N, nk, op.batch, e, km ? kKMajorSlice[GEMM_T256] : 1.f);
  // T256 with a k-major weight first writes a transposed copy, of all batch members in one launch (three of 1024 x 512: 14.4 us as
  // three, 5.0 as one).  Its price is that of a launch per member: without it three of 512 x 2048 under 16384 tokens came out even
  // (157 us with the copy, 157 on R128) for a launch more.
  if (op.transB && !op.transA) best += (float)op.batch * (2.5f + (float)op.N * (float)op.K * (4.f / 4e6f));
  int tile = GEMM_T256;
  if (km) {
    const float c = tile_time(GEMM_T256X128, op.M, op.N, nk, op.batch, e, kKMajorSlice[GEMM_T256X128]);
    if (c < best) {
      best = c;
      tile = GEMM_T256X128;
    }
  }
  for (int t = GEMM_R64; t <= GEMM_R32; t++) {
    const float c = tile_time(t, op.M, op.N, nk, op.batch, e, km ? kKMajorSlice[t] : 1.f);
    if (c * (tile < GEMM_R64 ? kRingMargin : 1.f) < best) {
      best = c;
      tile = t;
    }
  }
  return tile;
}

void gemm_bf16_tile_size(int tile, int* rows, int* cols) {
  *rows = kTileCost[tile].bm;
  *cols = kTileCost[tile].bn;
}

RowParts gemm_bf16_rowparts(const GemmOp& op) {
  const int tile = gemm_bf16_tile(op), bn = kTileCost[tile].bn;
  const int width = bn <= 64 ? 32 : 64;                            // columns per partial (gemm_tile.h)
  // The order in which a row's columns are added may not depend on the tile, so it is fixed by N: units of 128
  // columns, or of 64 for a narrow N that does not fill 256-column tiles.
  const int unit = op.N > 128 && (op.N % 256 == 0 || op.N > 512) ? 128 : 64;
  return RowParts{(op.N + bn - 1) / bn * (bn / width), unit / width, (op.N + unit - 1) / unit};
}

int gemm_bf16_rowpart_slabs_max(GemmOp op, std::initializer_list<int> kinds) {
  int most = 0;
  op.tile = GEMM_TILE_AUTO;
  for (int kind : kinds) {
    op.epi.kind = kind;
    const int s = gemm_bf16_rowparts(op).slabs;
    if (s > most) most = s;
  }
  return most;
}

int gemm_bf16_wgrad_max_splits(int64_t K) {
  const int64_t nk = (K + BK - 1) / BK;
  return nk < 16 ? 1 : nk / 8 < 64 ? (int)(nk / 8) : 64;   // at least 8 slices per split
}

int gemm_bf16_wgrad_splits(int M, int N, int K) {
  // The splits are part of the result: the fp32 sum over the tokens is their sums added up.  So they follow from the shape
  // alone, whatever tile runs them, whether the gradient is added to and how many equal ones share a launch.
  // With one 256-row tile per CU a launch runs in ceil(workgroups / 256) rounds, each as long as one workgroup: its
  // k slices plus a fixed cost (pipeline fill, the fp32 partial tile it writes, its share of the fold) worth
  // about 8 slices.  The split count with the smallest estimate; ties go to fewer splits (less partial traffic).
  const int bm = 256, bn = N > 128 && (N % 256 == 0 || N > 512) ? 256 : 128;
  const long tiles = (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn);
  const int nk = (K + BK - 1) / BK;
  const int maxs = gemm_bf16_wgrad_max_splits(K);
  int best = 1;
  long best_cost = -1;
  for (int s = 1; s <= maxs; s++) {
    const long rounds = (tiles * s + 255) / 256;
    const long cost = rounds * ((nk + s - 1) / s + 8) * 16 + s;   // "+ s": the tie-break
    if (best_cost < 0 || cost < best_cost) { best_cost = cost; best = s; }
  }
  return best;
}

WgradPlan gemm_bf16_plan_wgrad(int M, int N, int K, int batch, bool direct) {
  // A split launch writes an fp32 partial per split, which the finishing pass reads (7 TB/s).  The ring tiles can instead add
  // the parts up in registers, where the shape spreads over the chip without a split (256 x 1024 over 1031 tokens, two
  // parts: 6.6 us against 7.0 + 2.7); what is left is at most a finishing pass over one partial.
  const int nk = (K + BK - 1) / BK, splits = gemm_bf16_wgrad_splits(M, N, K);
  WgradPlan best{GEMM_T256, splits, 1};
  float best_t = -1.f;
  for (int tile = GEMM_T256; tile <= GEMM_R32; tile++)
    for (int s : {splits, 1}) {
      if (s < splits && (tile < GEMM_R64 || tile == GEMM_R128)) continue;   // (gemm_ring.h)
      float t = tile_time(tile, M, N, (nk + s - 1) / s, batch * s, 2.f, kKMajorSlice[tile]);
      if (s > 1 || !direct) t += (float)batch * (2.f + (float)(s + 1) * (float)M * (float)N * (4.f / 7e6f));
      if (best_t < 0.f || t < best_t) {
        best_t = t;
        best = WgradPlan{tile, s, splits / s};
      }
    }
  return best;
}

// ---- optional timing of launches (for the benchmark's roofline figures) --------------------------
// When enabled, every gemm_bf16 launch (and whatever else the sequencing code brackets with
// launch_timer_open / close) sits between two HIP events on its stream; the elapsed time between them is
// the time the stream spent in that launch.  Off by default; the events are created by launch_timer_begin
// and released when the session is read out, never on the compute path.  Process-global and not
// thread-safe: a measurement aid for a single-threaded benchmark, not part of the compute contract.
namespace {
struct LaunchTimer {
  bool on = false;
  std::vector<hipEvent_t> ev;
  std::vector<lr_launch_record> rec;
  size_t used = 0;
} g_timer;

void timer_release() {
  for (auto& e : g_timer.ev)
    if (e) (void)hipEventDestroy(e);
  g_timer.ev.clear();
  g_timer.rec.clear();
  g_timer.used = 0;
  g_timer.on = false;
}
}  // namespace

int launch_timer_begin(int max_launches) {
  if (g_timer.on || max_launches <= 0) return -1;
  g_timer.ev.assign((size_t)max_launches * 2, nullptr);
  for (auto& e : g_timer.ev)
    if (hipEventCreate(&e) != hipSuccess) {
      e = nullptr;
      timer_release();          // destroys the events created so far
      return -1;
    }
  g_timer.rec.assign((size_t)max_launches, lr_launch_record{});
  g_timer.used = 0;
  g_timer.on = true;
  return 0;
}

int launch_timer_open(int tag, int M, int N, int K, int batch, double flops, hipStream_t st) {
  if (!g_timer.on || g_timer.used >= g_timer.rec.size()) return -1;
  const int slot = (int)g_timer.used++;
  lr_launch_record& r = g_timer.rec[slot];
  r.tag = tag; r.M = M; r.N = N; r.K = K; r.batch = batch; r.flops = flops; r.ms = 0.f;
  (void)hipEventRecord(g_timer.ev[2 * slot], st);
  return slot;
}

void launch_timer_close(int slot, hipStream_t st) {
  if (slot >= 0 && g_timer.on) (void)hipEventRecord(g_timer.ev[2 * slot + 1], st);
}

int launch_timer_end(lr_launch_record* out, int max_records, int* n_records) {
  if (!g_timer.on) return -1;
  const size_t n = g_timer.used;
  if (n > 0) (void)hipEventSynchronize(g_timer.ev[2 * n - 1]);
  int w = 0;
  for (size_t i = 0; i < n; i++) {
    float ms = 0.f;
    (void)hipEventElapsedTime(&ms, g_timer.ev[2 * i], g_timer.ev[2 * i + 1]);
    g_timer.rec[i].ms = ms;
    if (out && w < max_records) out[w++] = g_timer.rec[i];
  }
  if (n_records) *n_records = (int)n;
  timer_release();
  return 0;
}

hipError_t gemm_bf16(const GemmOp& op, hipStream_t st) {
  if (!g_timer.on || op.M <= 0 || op.N <= 0 || op.batch <= 0) return gemm_bf16_untimed(op, st);
  // two k-major operands: a weight gradient, also where it stores bf16 itself; EPI_ACTGRAD_A: the class of EPI_ACTGRAD
  const int tag = op.splitk > 1 || (op.transA && op.transB) ? (int)EPI_PARTIAL : op.epi.kind == EPI_ACTGRAD_A ? (int)EPI_ACTGRAD : op.epi.kind;
  const int slot = launch_timer_open(tag, op.M, op.N, op.K, op.batch, 2.0 * op.M * op.N * (double)op.K * op.batch, st);
  hipError_t e = gemm_bf16_untimed(op, st);
  launch_timer_close(slot, st);
  return e;
}

int gemm_bf16_join_tile(const GemmOp* ops, int n) {
  // Apart, each on its best tile, a launch each; or together on 32 x 32 or 64 x 64 tiles, the workgroups of all
  // sharing the chip: as long as the longest workgroup or, where all of their work is more, as that and three quarters of the longest
  // one (they are not alike: what a slot still holds when the others are empty).
  // Against 11106 backward calls of a layer or group (1 .. 6000 tokens, weights 16 .. 4096 wide, written or added to), each measured
  // apart and joined on either tile: the choice loses 1.0 % to the best of the three in the geometric mean and saves 31 % of the
  // call against apart; 165 calls are more than 3 % slower than apart.  (With half of the longest 1.02 %, 229 calls, with all of it
  // 1.04 %, 98 calls; without the gap between launches 1.06 %, 47 calls, with twice as much 1.11 %, 288.  A linear fit of all
  // terms loses 0.6 % here but makes small blocks, whose chains of launches these calls do not show, up to 6 % slower.)  Some of
  // them, us, apart / 32 x 32 / 64 x 64 tiles:
  //   layer 12 tokens 2872 -> 400 -> 1760: 20.0 / 21.8 / 18.5        439 tokens 3000 -> 288 -> 864: 22.6 / 29.7 / 21.5
  //         1059 tokens 64 -> 48 -> 288:   19.0 / 10.7 / 12.4        3380 tokens 2088 -> 72 -> 72:  30.1 / 65.7 / 41.1
  //   group 2 x 82 tokens 240 -> 344 -> 1480: 19.8 / 17.9 / 18.2     1 x 557 tokens 392 -> 184 -> 504: 28.4 / 24.9 / 25.7
  if (n < 2 || n > JOINT_MAX || g_timer.on) return 0;
  float apart = 0.f, joint[2] = {0.f, 0.f}, longest[2] = {0.f, 0.f};
  const int tiles[2] = {GEMM_R32, GEMM_R64};
  for (int i = 0; i < n; i++) {
    const GemmOp& op = ops[i];
    if (!gemm_bf16_joint_ok(op)) return 0;
    const int best = op.tile != GEMM_TILE_AUTO ? op.tile : gemm_bf16_tile(op), members = op.batch * op.splitk;
    const int nk = op_slices(op);
    const bool km = op.transA && op.transB;
    const float e = epi_traffic(op);
    apart += tile_time(best, op.M, op.N, nk, members, e, km ? kKMajorSlice[best] : 1.f) + kLaunchGap;
    for (int t = 0; t < 2; t++) {
      const TileCost& c = kTileCost[tiles[t]];
      const float slice = km ? kKMajorSlice[tiles[t]] : 1.f;
      const float wgs = (float)((op.M + c.bm - 1) / c.bm) * (float)((op.N + c.bn - 1) / c.bn) * (float)members;
      const float one = c.f + (c.g + c.h) * e + (float)nk * slice * (c.s0 + c.s1);
      joint[t] += wgs * one / (float)c.slots;
      if (one > longest[t]) longest[t] = one;
    }
  }
  for (int t = 0; t < 2; t++)
    joint[t] = kTileCost[tiles[t]].a + kLaunchGap + (joint[t] > longest[t] ? joint[t] + 0.75f * longest[t] : longest[t]);
  const int t = joint[0] <= joint[1] ? 0 : 1;
  return joint[t] < apart ? tiles[t] : 0;
}

int gemm_bf16_dual_tile(const GemmOp& op) {
  // Apart, the gate's tile goes to memory and comes back, and a launch ends in between; together, both products run on the tiles of
  // gemm_ring.h, which read an operand element more often.  Block forwards (only m stored) and backwards (g and u too) of 256 to
  // 16384 tokens, 2 to 32 heads, rank 64 to 1024, replayed from graphs, us, apart -> together:
  //   256 tokens, 2 heads, r 64: 54.0 -> 50.8, 101 -> 98              777, 16 heads, r 128: 104 -> 98, 259 -> 257
  //   3000, 16 heads, r 512: 319 -> 298, 937 -> 925                   16384, 32 heads, r 128: 1320 -> 1188, 3779 -> 3716
  //   16384, 16 heads, r 512: 1045 -> 1023, 2992 -> 2995              16384, 32 heads, r 1024: 2787 -> 2853, 7855 -> 8040
  // 256-row tiles read less, which shows when the weights come from memory: where they run both products, together has to be estimated a
  // quarter faster (777 tokens, 32 heads, r 1024: 0.78 of the estimate, warm 285 / 285, weights cold 298 -> 303; 5000, 16 heads, r 512:
  // 0.69, 409 -> 395).  As streams of 2.5 rounds and more they are also faster than their estimate: a third (8192, 16 heads, r 512:
  // 0.69, forward 577 -> 599; 16384, 16 heads, r 512: 0.66).
  if (g_timer.on || op.epi.kind != EPI_SWIGLU_DUAL || op.transA || op.transB || op.splitk != 1 || op.batch != 1 || op.N % 8 || op.K % 8 ||
      (op.sA + 128 * op.lda + op.K) * 2 >= 0x7fffffffLL || (op.sB + 128 * op.ldb + op.K) * 2 >= 0x7fffffffLL)
    return 0;
  const int tile = gemm_bf16_tile(op), nk = op_slices(op);
  GemmOp one = op;
  float apart = kLaunchGap;
  bool t256 = true;
  for (int kind : {EPI_STORE, EPI_SWIGLU_FWD}) {
    one.epi.kind = kind;
    const int t = gemm_bf16_tile(one);
    t256 = t256 && t == GEMM_T256;
    apart += tile_time(t, op.M, op.N, nk / 2, 1, epi_traffic(kind) + (kind == EPI_SWIGLU_FWD && op.C ? 1.f : 0.f));
  }
  const bool rounds = (int64_t)((op.M + 255) / 256) * ((op.N + 255) / 256) * 2 > 5 * NCU;
  return tile_time(tile, op.M, op.N, nk, 1, epi_traffic(op)) < apart * (!t256 ? 1.f : rounds ? 0.68f : 0.75f) ? tile : 0;
}

hipError_t gemm_bf16_many(const GemmOp* ops, int n, hipStream_t st) {
  const int tile = gemm_bf16_join_tile(ops, n);
  if (tile) return gemm_bf16_joint(tile, ops, n, st);
  for (int i = 0; i < n; i++) {
    const hipError_t e = gemm_bf16(ops[i], st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

bool gemm_bf16_kmajor_ok(const GemmOp& op) {
  // both operands k-major, whole 8-column chunks, offsets within the 2 GB a buffer resource addresses
  const bool wgrad = op.epi.kind == EPI_PARTIAL;
  const bool plain = op.splitk == 1 && op.epi.kind == EPI_STORE;
  return op.transA && op.transB && (wgrad || plain) && op.M % 8 == 0 && op.N % 8 == 0 &&
         (int64_t)op.K * op.lda * 2 < 0x7fffffffLL && (int64_t)op.K * op.ldb * 2 < 0x7fffffffLL;
}

hipError_t gemm_bf16_untimed(const GemmOp& op, hipStream_t st) {
  if (op.M <= 0 || op.N <= 0 || op.batch <= 0) return hipSuccess;
  const bool km = op.transA && op.transB;
  if (km && !gemm_bf16_kmajor_ok(op)) return hipErrorInvalidValue;
  if (op.transA != op.transB && !gemm_bf16_mixed_ok(op)) return hipErrorInvalidValue;
  if (op.epi.stat_from_a && op.splitk > 1) return hipErrorInvalidValue;
  if (op.k_parts > 1 && gemm_bf16_tile(op) < GEMM_R64) return hipErrorInvalidValue;
  switch (gemm_bf16_tile(op)) {
    case GEMM_R64: return gemm_ring64(op, st);
    case GEMM_R64X128: return gemm_ring64x128(op, st);
    case GEMM_R128: return gemm_ring128(op, st);
    case GEMM_R32: return gemm_ring32(op, st);
    case GEMM_R128W: return gemm_ring128w(op, st);
    default: break;
  }
  if (!km) return dispatch<TileBig>(op, st);
  const bool store = op.epi.kind == EPI_STORE && op.splitk == 1;
  if (gemm_bf16_tile(op) == GEMM_T256X128)
    return store ? launch<TileMid, EPI_STORE, false, true>(op, st) : launch<TileMid, EPI_PARTIAL, false, true>(op, st);
  return store ? launch<TileBig, EPI_STORE, false, true>(op, st) : launch<TileBig, EPI_PARTIAL, false, true>(op, st);
}

}  // namespace lrb
