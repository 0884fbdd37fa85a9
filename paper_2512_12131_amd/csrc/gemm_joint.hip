// Independent bf16 products in one launch, on the small tiles of gemm_ring.h.
//
// Bound: launches.  Products of a few hundred rows take 4 to 8 us each, of which half is the way to the first and from the
// last workgroup; a launch costs the host another 3.3 us, so a chain of them is as long as the slower of the two.  Here up
// to JOINT_MAX products that do not depend on each other share a grid: workgroups [first, first + count) take one,
// each as its own launch would run it (same tile function, same order of summation, same bits).
// Measured, with sigma(z) written by the data gradient's epilogue instead of a pass of its own (a layer's backward in two
// launches instead of five): 1031 tokens, 1024 -> 256 -> 768, forward and backward 48.4 -> 40.4 us.
#include "gemm_ring.h"

namespace lrb {
namespace {

// operand form (T: k-major, N: k-contiguous A; N: k-major, T: k-contiguous B) and epilogue
enum JointForm : int {
  JF_NONE = -1, JF_TT_PARTIAL, JF_TT_PARTIAL_PARTS, JF_TT_STORE, JF_TT_STORE_PARTS,
  JF_NN_STORE, JF_NN_ACTGRAD, JF_NN_LAXGRAD, JF_NN_SWIGLU_BWD, JF_NN_NORMBWD_O32, JF_NN_NORMBWD_I32, JF_NT_STORE, JF_NT_UP, JF_NT_SWIGLU_DUAL
};

struct JointArgs {
  GemmOp op[JOINT_MAX];
  int form[JOINT_MAX], first[JOINT_MAX + 1], tiles_m[JOINT_MAX], tiles_n[JOINT_MAX], kper[JOINT_MAX];
};

// The arguments are read where the dispatch left them: an array indexed by the workgroup's product, not copied to the stack.
template <class T>
__global__ __launch_bounds__(T::NT) void gemm_joint_kernel(JointArgs) {
  const JointArgs& a = *(const JointArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  int i = 0;
#pragma unroll
  for (int j = 1; j < JOINT_MAX; j++) i += (int)blockIdx.x >= a.first[j] ? 1 : 0;
  i = __builtin_amdgcn_readfirstlane(i);
  const GemmOp& op = a.op[i];
  const int bid = (int)blockIdx.x - a.first[i], total = a.first[i + 1] - a.first[i];
  const int tm = a.tiles_m[i], tn = a.tiles_n[i], kper = a.kper[i];
  switch (a.form[i]) {
    case JF_TT_PARTIAL: ring_product<T, EPI_PARTIAL, false, true, true, false>(op, kper, tm, tn, bid, total); break;
    case JF_TT_PARTIAL_PARTS: ring_product<T, EPI_PARTIAL, false, true, true, true>(op, kper, tm, tn, bid, total); break;
    case JF_TT_STORE: ring_product<T, EPI_STORE, false, true, true, false>(op, kper, tm, tn, bid, total); break;
    case JF_TT_STORE_PARTS: ring_product<T, EPI_STORE, false, true, true, true>(op, kper, tm, tn, bid, total); break;
    case JF_NN_STORE: ring_product<T, EPI_STORE, false, false, true, false>(op, kper, tm, tn, bid, total); break;
    case JF_NN_ACTGRAD: ring_product<T, EPI_ACTGRAD, false, false, true, false>(op, kper, tm, tn, bid, total); break;
    case JF_NN_LAXGRAD: ring_product<T, EPI_LAXGRAD, false, false, true, false>(op, kper, tm, tn, bid, total); break;
    case JF_NN_SWIGLU_BWD: ring_product<T, EPI_SWIGLU_BWD, false, false, true, false>(op, kper, tm, tn, bid, total); break;
    case JF_NN_NORMBWD_O32: ring_product<T, EPI_NORMBWD_O32, false, false, true, false>(op, kper, tm, tn, bid, total); break;
    case JF_NN_NORMBWD_I32: ring_product<T, EPI_NORMBWD_I32, false, false, true, false>(op, kper, tm, tn, bid, total); break;
    case JF_NT_STORE: ring_product<T, EPI_STORE, false, false, false, false>(op, kper, tm, tn, bid, total); break;
    case JF_NT_UP: ring_product<T, EPI_UP, false, false, false, false>(op, kper, tm, tn, bid, total); break;
    case JF_NT_SWIGLU_DUAL: ring_product<T, EPI_SWIGLU_DUAL, false, false, false, false>(op, kper, tm, tn, bid, total); break;
    default: break;
  }
}

JointForm form_of(const GemmOp& op) {
  if (op.epi.stat_from_a || op.causal_k || op.batch_inner || op.M <= 0 || op.N <= 0 || op.batch <= 0) return JF_NONE;
  const int kind = op.epi.kind;
  if (op.transA && op.transB) {
    if (!gemm_bf16_kmajor_ok(op) || (op.splitk > 1 && (kind != EPI_PARTIAL || op.k_parts > 1))) return JF_NONE;
    if (kind == EPI_PARTIAL) return op.k_parts > 1 ? JF_TT_PARTIAL_PARTS : JF_TT_PARTIAL;
    return op.k_parts > 1 ? JF_TT_STORE_PARTS : JF_TT_STORE;
  }
  if (op.transA || op.splitk != 1 || op.k_parts != 1 || op.N % 8 || op.K % 8) return JF_NONE;
  if (!op.transB) return kind == EPI_STORE ? JF_NT_STORE : kind == EPI_UP ? JF_NT_UP : kind == EPI_SWIGLU_DUAL ? JF_NT_SWIGLU_DUAL : JF_NONE;
  // a k-major weight beside k-contiguous rows: in place under the conditions of gemm_bf16_tile
  if ((int64_t)op.K * op.ldb * 2 >= 0x7fffffffLL) return JF_NONE;
  switch (kind) {
    case EPI_STORE: return JF_NN_STORE;
    case EPI_ACTGRAD: return JF_NN_ACTGRAD;
    case EPI_LAXGRAD: return JF_NN_LAXGRAD;
    case EPI_SWIGLU_BWD: return JF_NN_SWIGLU_BWD;
    case EPI_NORMBWD_O32: return JF_NN_NORMBWD_O32;
    case EPI_NORMBWD_I32: return JF_NN_NORMBWD_I32;
    default: return JF_NONE;
  }
}

template <class T>
hipError_t launch_joint(const GemmOp* ops, int n, hipStream_t st) {
  auto kern = gemm_joint_kernel<T>;
  // one-time opt-in to more than 64 KB of dynamic LDS (thread-safe function-local static)
  static const hipError_t attr_err =
      hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
  if (attr_err != hipSuccess) return attr_err;
  JointArgs a;
  int wgs = 0;
  for (int i = 0; i < JOINT_MAX; i++) {
    a.first[i] = wgs;
    a.form[i] = JF_NONE;
    a.tiles_m[i] = a.tiles_n[i] = a.kper[i] = 0;
    if (i >= n) continue;
    a.op[i] = ops[i];
    a.form[i] = form_of(ops[i]);
    if (a.form[i] == JF_NONE) return hipErrorInvalidValue;
    a.tiles_m[i] = (ops[i].M + T::BM - 1) / T::BM;
    a.tiles_n[i] = (ops[i].N + T::BN - 1) / T::BN;
    a.kper[i] = ((ops[i].K + ops[i].splitk - 1) / ops[i].splitk + BK - 1) / BK * BK;
    wgs += a.tiles_m[i] * a.tiles_n[i] * ops[i].batch * ops[i].splitk;
  }
  a.first[JOINT_MAX] = wgs;
  hipLaunchKernelGGL(kern, dim3((unsigned)wgs), dim3(T::NT), T::LDS_BYTES, st, a);
  return hipGetLastError();
}

}  // namespace

bool gemm_bf16_joint_ok(const GemmOp& op) { return form_of(op) != JF_NONE; }
hipError_t gemm_bf16_joint(int tile, const GemmOp* in, int n, hipStream_t st) {
  if (n <= 0 || n > JOINT_MAX) return hipErrorInvalidValue;
  // The longest workgroups first: started last they run alone behind the others (4 tokens, two members 328 -> 464 -> 3408, a
  // data gradient of 54 slices beside weight gradients of one: 27.9 us, apart 20).  A gate's and up pair walks k twice.
  auto walk = [](const GemmOp& op) { return (int64_t)op.K * (op.epi.kind == EPI_SWIGLU_DUAL ? 2 : 1); };
  GemmOp ops[JOINT_MAX];
  for (int i = 0; i < n; i++) {
    int j = i;
    for (; j > 0 && walk(ops[j - 1]) * in[i].splitk < walk(in[i]) * ops[j - 1].splitk; j--) ops[j] = ops[j - 1];
    ops[j] = in[i];
  }
  if (tile == GEMM_R32) return launch_joint<RingTile<32, 32, 1, 1, 2, 5, 4>>(ops, n, st);
  return tile == GEMM_R64 ? launch_joint<RingTile<64, 64, 2, 2, 2, 5>>(ops, n, st) : hipErrorInvalidValue;
}

}  // namespace lrb
