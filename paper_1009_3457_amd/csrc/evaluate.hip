// The whole evaluation (tree, P2M .. P2P) and its reverse pass as one call
// each, on one workspace: what a caller of the separate stages would enqueue,
// without its host work between them and with the passes over the points
// that only join two stages taken out.  Points and charges are sorted
// along with the tree, L2P overwrites its sums instead of adding to cleared arrays, and
// the near field adds them up and leaves the results in the caller's order.
// 4096 points, depth 4, p = 8: 7 launches where the stages take 17, and with
// one call from Python where there are 11, 67 us an evaluation against 156;
// 2^20 points, depth 8, p = 12: 302 us against 374.
#include <algorithm>

#include "fmm2d_internal.h"

namespace fmm2d {

namespace {

// Consecutive arrays on 256-byte boundaries of one buffer; with base NULL
// only the size counts.
struct Carver {
  char *base;
  size_t used = 0;
  explicit Carver(void *p) : base(static_cast<char *>(p)) {}
  template <typename T>
  T *take(int64_t n) {
    T *p = reinterpret_cast<T *>(base + used);
    used += tree_ws::align256(size_t(n) * sizeof(T));
    return p;
  }
};

// What a reverse pass needs of the forward one: both trees and their points
// in leaf order.  nt < 0: the sources are the targets and share them.
struct Plan {
  uint32_t *flags;  // domain flags of the sources' and the targets' tree
  int32_t *ls, *perm, *tls, *tperm;
  float *xs, *qs, *ts;
  size_t bytes;
  Plan(void *p, int64_t n, int64_t nt, int depth) {
    Carver c(p);
    const int64_t nleaf = int64_t(1) << (2 * depth);
    flags = c.take<uint32_t>(2);
    ls = tls = c.take<int32_t>(nleaf + 1);
    perm = tperm = c.take<int32_t>(n);
    xs = ts = c.take<float>(2 * n);
    qs = c.take<float>(n);
    if (nt >= 0) {
      tls = c.take<int32_t>(nleaf + 1);
      tperm = c.take<int32_t>(nt);
      ts = c.take<float>(2 * nt);
    }
    bytes = c.used;
  }
};

struct ForwardWs {
  float *M, *Lm, *bm, *phi, *field;
  double *L, *b;
  void *tree;  // shares the expansions' memory: the trees are built before them
  size_t bytes;
  ForwardWs(void *p, int64_t n, int64_t nt, int depth, int order) {
    const int64_t nb = level_off(depth + 1), m = nt < 0 ? n : nt;
    Carver c(p);
    tree = p;
    M = c.take<float>(2 * nb * order);
    Lm = c.take<float>(2 * nb * order);
    bm = c.take<float>(2 * nb);
    L = c.take<double>(2 * nb * order);
    b = c.take<double>(2 * nb);
    phi = c.take<float>(2 * m);
    field = c.take<float>(2 * m);
    bytes = std::max(c.used, sort_points_ws_bytes(std::max(n, m)));
  }
};

struct BackwardWs {
  float *cphi, *cfield, *gLm, *gbm, *gM, *gq, *G;
  double *gL, *gb;
  size_t bytes;
  BackwardWs(void *p, int64_t n, int64_t nt, int depth, int order) {
    const int64_t nb = level_off(depth + 1), m = nt < 0 ? n : nt;
    Carver c(p);
    cphi = c.take<float>(2 * m);
    cfield = c.take<float>(2 * m);
    gL = c.take<double>(2 * nb * order);
    gb = c.take<double>(2 * nb);
    gLm = c.take<float>(2 * nb * order);
    gbm = c.take<float>(2 * nb);
    gM = c.take<float>(2 * nb * order);
    gq = c.take<float>(n);
    G = c.take<float>(2 * n);
    bytes = c.used;
  }
};

// Sorted conjugates of the cotangents that are present.
__global__ void sort_cotangents_kernel(const float2 *__restrict__ gphi, const float2 *__restrict__ gfield,
                                       const int32_t *__restrict__ perm, int64_t n, float2 *__restrict__ cphi,
                                       float2 *__restrict__ cfield) {
  const int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (i >= n) return;
  const int64_t j = perm[i];
  if (gphi) {
    const float2 v = gphi[j];
    cphi[i] = make_float2(v.x, -v.y);
  }
  if (gfield) {
    const float2 v = gfield[j];
    cfield[i] = make_float2(v.x, -v.y);
  }
}

inline unsigned blocks_of(int64_t n) { return unsigned((n + 255) / 256); }

int check_sizes(const char *fn, int64_t n, int64_t nt, int depth, int p) {
  if (depth < 2 || depth > kMaxDepth) return set_error(FMM2D_EDEPTH, "%s: depth %d outside 2..%d", fn, depth, kMaxDepth);
  if (!p_supported(p)) return set_error(FMM2D_EUNSUPPORTED_P, "%s: p = %d not in {8, 12, 16, 20}", fn, p);
  const int64_t end = int64_t(1) << 31;
  if (n < 1 || n >= end || nt == 0 || nt < -1 || nt >= end)
    return set_error(FMM2D_EINVAL, "%s: n = %lld or nt = %lld out of range", fn, (long long)n, (long long)nt);
  return FMM2D_OK;
}

int check_buffer(const char *fn, const char *what, const void *p, size_t bytes, size_t need) {
  if (p == nullptr) return set_error(FMM2D_EINVAL, "%s: %s is NULL", fn, what);
  if (reinterpret_cast<uintptr_t>(p) % 16 != 0) return set_error(FMM2D_EINVAL, "%s: %s not 16-byte aligned", fn, what);
  if (bytes < need) return set_error(FMM2D_EWORKSPACE, "%s: %s has %zu bytes, %zu needed", fn, what, bytes, need);
  return FMM2D_OK;
}

#define TRY(expr)                    \
  do {                               \
    const int rc_ = (expr);          \
    if (rc_ != FMM2D_OK) return rc_; \
  } while (0)

}  // namespace

}  // namespace fmm2d

using namespace fmm2d;

extern "C" {

size_t fmm2d_evaluate_plan_bytes(int64_t n, int64_t nt, int depth) {
  clear_error();
  if (check_sizes("fmm2d_evaluate_plan_bytes", n, nt, depth, 8) != FMM2D_OK) return 0;
  return Plan(nullptr, n, nt, depth).bytes;
}

size_t fmm2d_evaluate_workspace(int64_t n, int64_t nt, int depth, int p) {
  clear_error();
  if (check_sizes("fmm2d_evaluate_workspace", n, nt, depth, p) != FMM2D_OK) return 0;
  return ForwardWs(nullptr, n, nt, depth, p).bytes;
}

size_t fmm2d_evaluate_backward_workspace(int64_t n, int64_t nt, int depth, int p) {
  clear_error();
  if (check_sizes("fmm2d_evaluate_backward_workspace", n, nt, depth, p) != FMM2D_OK) return 0;
  return BackwardWs(nullptr, n, nt, depth, p).bytes;
}

int fmm2d_evaluate(const float *xy, const float *q, int64_t n, const float *txy, int64_t nt, int depth, int p,
                   int precision, const void *ops, size_t ops_bytes, void *plan, size_t plan_bytes, float *phi,
                   float *field, void *ws, size_t ws_bytes, hipStream_t stream) {
  const char *fn = "fmm2d_evaluate";
  clear_error();
  TRY(check_sizes(fn, n, nt, depth, p));
  if (!xy || !q || !phi || !field || (nt > 0 && !txy)) return set_error(FMM2D_EINVAL, "%s: NULL pointer", fn);
  const Plan pl(plan, n, nt, depth);
  const ForwardWs w(ws, n, nt, depth, p);
  TRY(check_buffer(fn, "plan", plan, plan_bytes, pl.bytes));
  TRY(check_buffer(fn, "ws", ws, ws_bytes, w.bytes));
  if (ops_bytes < m2l_ops_bytes(p, precision) || m2l_ops_bytes(p, precision) == 0 || !ops)
    return set_error(FMM2D_EINVAL, "%s: no operator bank for p = %d, precision %d", fn, p, precision);

  TRY(launch_sort_points(xy, q, n, depth, pl.perm, pl.ls, pl.flags, pl.xs, pl.qs, w.tree, stream));
  if (nt > 0)
    TRY(launch_sort_points(txy, nullptr, nt, depth, pl.tperm, pl.tls, pl.flags + 1, pl.ts, nullptr, w.tree, stream));
  const int64_t m = nt < 0 ? n : nt;
  TRY(launch_p2m(pl.xs, pl.qs, pl.ls, depth, p, w.M, stream));
  // M2L starts at level 2: ceil((depth - 2) / 3) launches for ceil(depth / 3)
  TRY(launch_m2m(w.M, depth, 2, p, stream));
  TRY(fmm2d_m2l(w.M, w.Lm, w.bm, depth, p, 2, depth, precision, ops, ops_bytes, stream));
  TRY(launch_l2l(w.Lm, w.bm, w.L, w.b, depth, p, stream));
  TRY(launch_l2p(pl.ts, pl.tls, m, w.L, w.b, depth, p, w.phi, w.field, false, stream));
  return launch_p2p(pl.xs, pl.qs, pl.ls, pl.ts, pl.tls, m, depth, w.phi, w.field, pl.tperm, phi, field, stream);
}

int fmm2d_evaluate_backward(const void *plan, size_t plan_bytes, int64_t n, int64_t nt, int depth, int p,
                            int precision, const void *ops, size_t ops_bytes, const float *gphi, const float *gfield,
                            float *gq, float *gxy, void *ws, size_t ws_bytes, hipStream_t stream) {
  const char *fn = "fmm2d_evaluate_backward";
  clear_error();
  TRY(check_sizes(fn, n, nt, depth, p));
  if ((!gphi && !gfield) || !gq || !gxy) return set_error(FMM2D_EINVAL, "%s: NULL pointer", fn);
  const Plan pl(const_cast<void *>(plan), n, nt, depth);
  const BackwardWs w(ws, n, nt, depth, p);
  TRY(check_buffer(fn, "plan", plan, plan_bytes, pl.bytes));
  TRY(check_buffer(fn, "ws", ws, ws_bytes, w.bytes));
  if (ops_bytes < m2l_ops_bytes(p, precision) || m2l_ops_bytes(p, precision) == 0 || !ops)
    return set_error(FMM2D_EINVAL, "%s: no operator bank for p = %d, precision %d", fn, p, precision);

  const int64_t m = nt < 0 ? n : nt;
  float *cphi = gphi ? w.cphi : nullptr, *cfield = gfield ? w.cfield : nullptr;
  hipLaunchKernelGGL(sort_cotangents_kernel, dim3(blocks_of(m)), dim3(256), 0, stream,
                     reinterpret_cast<const float2 *>(gphi), reinterpret_cast<const float2 *>(gfield), pl.tperm, m,
                     reinterpret_cast<float2 *>(cphi), reinterpret_cast<float2 *>(cfield));
  TRY(launch_l2p_backward(pl.ts, pl.tls, cphi, cfield, depth, p, w.gL, w.gb, stream));
  TRY(launch_l2l_backward(w.gL, w.gb, w.gLm, w.gbm, depth, p, stream));
  TRY(fmm2d_m2l_backward(w.gLm, w.gbm, w.gM, depth, p, 2, depth, precision, ops, ops_bytes, stream));
  TRY(launch_m2m_backward(w.gM, depth, p, stream));
  TRY(launch_p2m_backward(pl.xs, pl.qs, pl.ls, n, depth, p, w.gM, w.gq, w.G, stream));
  return launch_p2p_backward(pl.xs, pl.qs, pl.ls, n, pl.ts, pl.tls, depth, cphi, cfield, w.gq, w.G, pl.perm, gq, gxy,
                             stream);
}

}  // extern "C"
