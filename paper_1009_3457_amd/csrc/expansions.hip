// Upward sweep (P2M, M2M), L2L and L2P (Sec. 2.1, stages 2-4) in the scaled
// basis of fmm2d.h, and the plain transposes of each for gradients.  L2L and
// L2P run in FP64 (the deep-level accumulation of local expansions).
//
// Leaf stages (P2M, L2P^T) sum powers over a leaf's points: a few lanes share
// a leaf, each with a strided part of its points and all the sums in
// registers.  Shifts between a box and its parent (M2M, L2L and transposes)
// are bound by latency on the few boxes of the upper levels, so one launch
// takes up to three levels, a workgroup per subtree.
#include "fmm2d_internal.h"

namespace fmm2d {

// Find the leaf of sorted item i: the largest m with ls[m] <= i.
__device__ inline int64_t leaf_of(const int32_t *__restrict__ ls, int64_t nleaf, int64_t i) {
  int64_t lo = 0, hi = nleaf;  // invariant: ls[lo] <= i < ls[hi]
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (int64_t(ls[mid]) <= i) lo = mid;
    else hi = mid;
  }
  return lo;
}

// body(m) for the leaf m of sorted item t at `z`: the leaf the tree build
// assigns to z (floor of z 2^depth, clamped), confirmed against the leaf
// ranges; once more for the leaf that a search of the ranges finds when they
// disagree.  The body's reads are not to wait for the ranges': it returns a
// value that it ends with, and the ranges are compared after that.
template <typename F>
__device__ __forceinline__ void at_leaf(float2 z, const int32_t *__restrict__ ls, int64_t nleaf, int depth, int64_t t,
                                        F body) {
  const float side = float(1 << depth);  // z 2^depth is exact in FP32
  const int lim = (1 << depth) - 1;
  const int ix = min(max(int(floorf(z.x * side)), 0), lim), iy = min(max(int(floorf(z.y * side)), 0), lim);
  int64_t m = morton2(uint32_t(ix), uint32_t(iy));
  int32_t s0 = ls[m], s1 = ls[m + 1];
  const float last = body(m);
  asm volatile("" : "+v"(s0), "+v"(s1) : "v"(last));
  if (int64_t(s0) > t || t >= int64_t(s1)) body(leaf_of(ls, nleaf, t));
}

// (x - c)/h for a point and the centre of leaf m at level `depth`.
__device__ inline float2 scaled_offset(float2 p, uint32_t m, int depth) {
  uint32_t ix, iy;
  unmorton2(m, ix, iy);
  const float h = ldexpf(1.f, -depth);
  const float cx = (float(ix) + 0.5f) * h, cy = (float(iy) + 0.5f) * h;
  return make_float2((p.x - cx) * float(1 << depth), (p.y - cy) * float(1 << depth));
}

// ----------------------------------------------------- sums over a leaf --
//
// LANES consecutive lanes share a leaf; lane r takes its points r, r + LANES,
// ...  With one thread a leaf, 2.5e5 clustered points in 16384 leaves gave
// 256 waves that waited for their fullest leaf: P2M 58 us against 10, L2P^T
// 113 against 18 (p = 16).  At 2^24 points, depth 10, p = 20: 374 against 131
// and 629 against 338.  4 lanes keep the sums' exchange small against the
// points' work; trees of few leaves take 16 to fill the chip.
static int leaf_lanes(int64_t nleaf) { return nleaf < 65536 ? 16 : 4; }

// v of another lane of the row of 16 (DPP control CTRL).
template <int CTRL>
__device__ inline float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ inline double dpp(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// Sum over the leaf's lanes; every lane ends with the total.  The mirrors of
// 8 and 16 lanes stand for an exchange of halves: their lanes agree by then.
template <int LANES, typename T>
__device__ inline T lanes_sum(T v) {
  static_assert(LANES == 4 || LANES == 16, "quads or rows");
  v += dpp<0xb1>(v);   // quad_perm 1 0 3 2
  v += dpp<0x4e>(v);   // quad_perm 2 3 0 1
  if constexpr (LANES == 16) {
    v += dpp<0x141>(v);  // row_half_mirror
    v += dpp<0x140>(v);  // row_mirror
  }
  return v;
}

// The leaf's coefficients from its lanes' sums: lane r writes coefficients r,
// r + LANES, ..., so that the lanes write consecutive addresses.
template <int P, int LANES, typename T, typename T2>
__device__ inline void store_sums(const T (&ar)[P], const T (&ai)[P], T2 *__restrict__ out, int r) {
#pragma unroll
  for (int k0 = 0; k0 < P; k0 += LANES) {
    T x = ar[k0], y = ai[k0];
#pragma unroll
    for (int e = 1; e < LANES; ++e) {
      if (k0 + e >= P) break;
      x = r == e ? ar[k0 + e] : x;
      y = r == e ? ai[k0 + e] : y;
    }
    if (k0 + r < P) out[k0 + r] = T2{x, y};
  }
}

// ------------------------------------------------------------------ P2M --

template <int P, int LANES>
__global__ __launch_bounds__(256) void p2m_kernel(const float2 *__restrict__ xy, const float *__restrict__ q,
                                                  const int32_t *__restrict__ ls, int depth, float2 *__restrict__ M) {
  const int64_t nleaf = int64_t(1) << (2 * depth);
  const int64_t m = (blockIdx.x * int64_t(256) + threadIdx.x) / LANES;
  if (m >= nleaf) return;  // whole leaves
  const int r = threadIdx.x % LANES;
  float ar[P], ai[P];
#pragma unroll
  for (int k = 0; k < P; ++k) ar[k] = ai[k] = 0.f;
  // counted down: an index that steps past the end may pass 2^31
  const int64_t first = ls[m] + int64_t(r);
  xy += first;
  q += first;
  for (int32_t left = ls[m + 1] - ls[m] - r; left > 0; left -= LANES, xy += LANES, q += LANES) {
    const float2 w = scaled_offset(*xy, uint32_t(m), depth);
    float pr = *q, pi = 0.f;  // q w^k
#pragma unroll
    for (int k = 0; k < P; ++k) {
      ar[k] += pr;
      ai[k] += pi;
      const float tr = pr * w.x - pi * w.y;
      pi = pr * w.y + pi * w.x;
      pr = tr;
    }
  }
#pragma unroll
  for (int k = 0; k < P; ++k) {
    ar[k] = lanes_sum<LANES>(ar[k]);
    ai[k] = lanes_sum<LANES>(ai[k]);
  }
  store_sums<P, LANES>(ar, ai, M + (level_off(depth) + m) * P, r);
}

// P2M^T and its z-derivative for every sorted source.
template <int P>
__global__ void p2m_backward_kernel(const float2 *__restrict__ xy, const float *__restrict__ q,
                                    const int32_t *__restrict__ ls, int64_t n, int depth,
                                    const float2 *__restrict__ gM, float *__restrict__ gq, float2 *__restrict__ G) {
  const int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  const int64_t nleaf = int64_t(1) << (2 * depth);
  if (i >= n) return;
  const float2 z = xy[i];
  const float sc = q[i] * float(1 << depth);  // q / h
  const int32_t end = ls[nleaf];
  float qr, dr, di;
  at_leaf(z, ls, nleaf, depth, i, [&](int64_t m) {
    const float2 w = scaled_offset(z, uint32_t(m), depth);
    const float2 *g = gM + (level_off(depth) + m) * P;
    qr = dr = di = 0.f;
    float pr = 1.f, pi = 0.f;  // w^k
#pragma unroll
    for (int k = 0; k < P; ++k) {
      qr += g[k].x * pr - g[k].y * pi;
      if (k + 1 < P) {  // d/dz of gM_{k+1} w^{k+1} = (k+1) gM_{k+1} w^k
        dr += float(k + 1) * (g[k + 1].x * pr - g[k + 1].y * pi);
        di += float(k + 1) * (g[k + 1].x * pi + g[k + 1].y * pr);
      }
      const float tr = pr * w.x - pi * w.y;
      pi = pr * w.y + pi * w.x;
      pr = tr;
    }
    return qr;
  });
  if (i >= int64_t(end)) return;
  gq[i] = qr;
  G[i] = make_float2(sc * dr, sc * di);
}

// ------------------------------------------------------- shifts by u --
//
// A shift between a box and its parent applies the binomial matrix of the
// offset u = (+-1 +- i)/2 (child centre minus parent centre, in child
// widths).  With rho = (1 + i)/2 the offsets of children 0..3 are -rho,
// conj(rho), -conj(rho), rho, and rho^m is real for m = 0, imaginary for
// m = 2, and x (1 + i) or x (1 - i) for m = 1 or 3 (mod 4).  So up,
//     sum_c u_c^m a_c = r(m) V_(m mod 4),   r(m) real,
//     V_0 = P + Q, V_2 = i (P - Q)                of P = a_3 + a_0, Q = a_1 + a_2,
//     V_1 = (P + Q) + i (P - Q), V_3 = (P + Q) - i (P - Q)
//                                                 of P = a_3 - a_0, Q = a_1 - a_2,
// one real multiple of a complex value a coefficient pair for all four
// children together (2 multiply-adds against 16), and down, the sums of
// r(m) t over each class of m give the four children the same way.
//
// Tables: w(k, j) = 2^-k C(k, j) r(k - j) for j <= k, zero above, both ways
// round, and column kB of `down`: 2^-(m+1) r(m+1) / (m+1) (the step of b).
// All but that column are exact in FP32.
constexpr int kMaxP = 20, kB = kMaxP;

template <typename T>
struct ShiftTable {
  T up[kMaxP][kMaxP];        // [j][k]
  T down[kMaxP][kMaxP + 1];  // [k][j]
};

template <typename T>
constexpr ShiftTable<T> shift_table() {
  ShiftTable<T> t{};
  double r[kMaxP + 1] = {1.0};  // the real factor of rho^m: Re rho^m, or Im where that is 0
  double x = 1.0, y = 0.0;
  for (int m = 1; m <= kMaxP; ++m) {
    const double nx = 0.5 * (x - y);
    y = 0.5 * (x + y);
    x = nx;
    r[m] = m % 4 == 2 ? y : x;
  }
  double half = 1.0;  // 2^-k
  for (int k = 0; k < kMaxP; ++k) {
    double c = 1.0;  // C(k, j)
    for (int j = 0; j <= k; ++j) {
      t.up[j][k] = t.down[k][j] = T(half * c * r[k - j]);
      c = c * double(k - j) / double(j + 1);
    }
    half *= 0.5;
    t.down[k][kB] = T(half * r[k + 1] / double(k + 1));
  }
  return t;
}

__constant__ ShiftTable<float> kShiftF = shift_table<float>();
__constant__ ShiftTable<double> kShiftD = shift_table<double>();

template <typename T>
__device__ inline const ShiftTable<T> &shifts() {
  if constexpr (sizeof(T) == 4) return kShiftF;
  else return kShiftD;
}

template <typename T>
struct Pair;
template <>
struct Pair<float> {
  using type = float2;
};
template <>
struct Pair<double> {
  using type = double2;
};

// One launch a level, a thread a box, left the upper levels at 6 us each:
// M2M 46 us against 12 at depth 8 (p = 12), L2L 42 against 16, L2L^T 87
// against 26; at depth 10, p = 20: 164 against 120, 367 against 316, 469
// against 351, where the FP64 arrays bound them (L2L moves 0.6 GB, 125 us).
constexpr int kSpan = 3;                      // levels of one launch, at most
constexpr int kSub = 1 << (2 * (kSpan - 1));  // parents of a subtree's widest step
// a thread per parent and coefficient (and b) of the widest step
constexpr int shift_threads(int p) { return (kSub * (p + 1) + 63) / 64 * 64; }

// Up: `a` holds [num_boxes][P]; the levels root + span - 1 .. root are formed
// from their children, scaled by `scale`; one workgroup per box of level
// `root`.  With b, b(parent) = sum b(child), and the parent takes the
// transpose of the step of b (L2L^T).  a32 and b32 (or NULL) take the FP32
// values of the levels formed and, with `leaves`, of the level below them.
template <typename T, int P, bool WITH_B>
__global__ __launch_bounds__(shift_threads(P)) void shift_up_kernel(typename Pair<T>::type *__restrict__ a,
                                                                    typename Pair<T>::type *__restrict__ b,
                                                                    float2 *__restrict__ a32,
                                                                    float2 *__restrict__ b32, int root, int span,
                                                                    bool leaves, T scale) {
  using T2 = typename Pair<T>::type;
  __shared__ T2 comb[kSub][4][P + 1];  // V_0..V_3; column P: of b
  __shared__ T2 cur[kSub][P + 1];      // the step's parents: the next step's children
  const ShiftTable<T> &w = shifts<T>();
  constexpr int N = WITH_B ? P + 1 : P;
  const int64_t box = blockIdx.x;
  for (int s = span - 1; s >= 0; --s) {
    const int np = 1 << (2 * s);  // parents of this subtree at level root + s
    const int64_t par0 = level_off(root + s) + (box << (2 * s));
    const int64_t ch0 = level_off(root + s + 1) + (box << (2 * s + 2));
    for (int it = threadIdx.x; it < np * N; it += blockDim.x) {
      const int i = it / N, j = it - i * N;
      T2 v[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (s == span - 1) v[c] = j < P ? a[(ch0 + 4 * i + c) * P + j] : b[ch0 + 4 * i + c];
        else v[c] = cur[4 * i + c][j];
      }
      if (a32 && leaves && s == span - 1) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
          *(j < P ? a32 + (ch0 + 4 * i + c) * P + j : b32 + ch0 + 4 * i + c) = make_float2(float(v[c].x), float(v[c].y));
      }
      const T2 pe = {v[3].x + v[0].x, v[3].y + v[0].y}, qe = {v[1].x + v[2].x, v[1].y + v[2].y};
      const T2 po = {v[3].x - v[0].x, v[3].y - v[0].y}, qo = {v[1].x - v[2].x, v[1].y - v[2].y};
      const T2 eo = {po.x + qo.x, po.y + qo.y}, dn = {po.x - qo.x, po.y - qo.y};
      comb[i][0][j] = {pe.x + qe.x, pe.y + qe.y};
      comb[i][1][j] = {eo.x - dn.y, eo.y + dn.x};
      comb[i][2][j] = {qe.y - pe.y, pe.x - qe.x};
      comb[i][3][j] = {eo.x + dn.y, eo.y - dn.x};
    }
    __syncthreads();
    for (int it = threadIdx.x; it < np * N; it += blockDim.x) {
      const int i = it / N, k = it - i * N;
      if (WITH_B && k == P) {
        const T2 t = comb[i][0][P];
        cur[i][P] = t;
        b[par0 + i] = t;
        if (a32) b32[par0 + i] = make_float2(float(t.x), float(t.y));
        continue;
      }
      // V of class (k - j) mod 4 for j = 0..3 (mod 4)
      const T2 *v[4] = {comb[i][k & 3], comb[i][(k - 1) & 3], comb[i][(k - 2) & 3], comb[i][(k - 3) & 3]};
      T re = 0, im = 0;
#pragma unroll
      for (int j = 0; j < P; ++j) {
        const T2 t = v[j & 3][j];
        const T x = w.up[j][k];
        re += x * t.x;
        im += x * t.y;
      }
      re *= scale;
      im *= scale;
      if (WITH_B) {  // power k + 1
        const T2 t = comb[i][(k + 1) & 3][P];
        const T x = w.down[k][kB];
        re += x * t.x;
        im += x * t.y;
      }
      cur[i][k] = {re, im};
      a[(par0 + i) * P + k] = {re, im};
      if (a32) a32[(par0 + i) * P + k] = make_float2(float(re), float(im));
    }
    __syncthreads();
  }
}

// The four children's values of coefficient column `col` from their parent's
// coefficients t[0..P); n: the coefficient's index (-1 for b).
// (Scalars throughout: selecting between vector values sent them through
// scratch memory, 652 us against 442 at depth 10, p = 20; loops unrolled less and the widest
// step's loads issued first made it 317.)
template <typename T, int P, typename T2>
__device__ inline void down_sums(const ShiftTable<T> &w, const T2 *t, int col, int n, T (&vx)[4], T (&vy)[4]) {
  T ax[4] = {0, 0, 0, 0}, ay[4] = {0, 0, 0, 0};  // by m mod 4
#pragma unroll 2  // whole, the table's loads take 130 registers at p = 20
  for (int m = 0; m < P; m += 4) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const T x = w.down[m + r][col];
      const T2 u = t[m + r];
      ax[r] += x * u.x;
      ay[r] += x * u.y;
    }
  }
  // class r = (m - n) mod 4 is a[(n + r) mod 4]
  const bool n1 = n & 1, n2 = n & 2;
  T hx[4], hy[4], sx[4], sy[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const T x0 = ax[r], x1 = ax[(r + 1) & 3], y0 = ay[r], y1 = ay[(r + 1) & 3];
    hx[r] = n1 ? x1 : x0;
    hy[r] = n1 ? y1 : y0;
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const T x0 = hx[r], x1 = hx[(r + 2) & 3], y0 = hy[r], y1 = hy[(r + 2) & 3];
    sx[r] = n2 ? x1 : x0;
    sy[r] = n2 ? y1 : y0;
  }
  // A = sum of Re rho^m t, B = of Im rho^m t; children A +- i B, odd classes
  // with the sign of (-1)^m
  const T aox = sx[1] + sx[3], aoy = sy[1] + sy[3], box = sx[1] - sx[3], boy = sy[1] - sy[3];
  const T apx = sx[0] + aox, apy = sy[0] + aoy, amx = sx[0] - aox, amy = sy[0] - aoy;
  const T bpx = sx[2] + box, bpy = sy[2] + boy, bmx = sx[2] - box, bmy = sy[2] - boy;
  vx[0] = amx - bmy, vy[0] = amy + bmx;
  vx[1] = apx + bpy, vy[1] = apy - bpx;
  vx[2] = amx + bmy, vy[2] = amy - bmx;
  vx[3] = apx - bpy, vy[3] = apy + bpx;
}

// M2M^T, in place: gM(child) += the shift of gM(parent), levels root + 1 ..
// root + span; one workgroup per box of level `root`.
template <int P>
__global__ __launch_bounds__(shift_threads(P)) void m2m_backward_kernel(float2 *__restrict__ gM, int root, int span) {
  __shared__ float2 buf[2][kSub][P];
  const int64_t box = blockIdx.x;
  for (int j = threadIdx.x; j < P; j += blockDim.x) buf[0][0][j] = gM[(level_off(root) + box) * P + j];
  __syncthreads();
  for (int s = 0; s < span; ++s) {
    const int np = 1 << (2 * s);
    const int64_t ch0 = level_off(root + s + 1) + (box << (2 * s + 2));
    float2(*cur)[P] = buf[s & 1], (*next)[P] = buf[(s + 1) & 1];
    for (int it = threadIdx.x; it < np * P; it += blockDim.x) {
      const int i = it / P, n = it - i * P;
      float2 own[4];
      float vx[4], vy[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) own[c] = gM[(ch0 + 4 * i + c) * P + n];
      down_sums<float, P>(kShiftF, cur[i], n, n, vx, vy);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float2 o = make_float2(own[c].x + vx[c], own[c].y + vy[c]);
        gM[(ch0 + 4 * i + c) * P + n] = o;
        if (s + 1 < span) next[4 * i + c][n] = o;
      }
    }
    __syncthreads();
  }
}

// L2L: L(child) = Lm2l(child) + shift of L(parent), and b with it, levels
// root + 1 .. root + span.  root = 2 also forms its own level (no parent) and
// clears the levels above, which hold no local expansion.
template <int P>
__global__ __launch_bounds__(shift_threads(P)) void l2l_kernel(const float2 *__restrict__ Lm2l,
                                                               const float2 *__restrict__ bm2l,
                                                               double2 *__restrict__ L, double2 *__restrict__ b,
                                                               int root, int span) {
  __shared__ double2 buf[2][kSub][P + 1];  // column P: b
  const int64_t box = blockIdx.x;
  const int N = b ? P + 1 : P;
  // Lm2l and bm2l of the widest step's children load while the steps above
  // run; a thread has one item a step
  const auto load_own = [&](int s, float2(&own)[4]) {
    const int i = int(threadIdx.x) / N, n = int(threadIdx.x) - i * N;
    const int64_t ch0 = level_off(root + s + 1) + (box << (2 * s + 2)) + 4 * i;
#pragma unroll
    for (int c = 0; c < 4; ++c) own[c] = *(n == P ? bm2l + ch0 + c : Lm2l + (ch0 + c) * P + n);
  };
  float2 wide[4] = {};
  if (span > 0 && int(threadIdx.x) < N << (2 * span - 2)) load_own(span - 1, wide);
  if (root == 2 && box == 0) {
    for (int e = threadIdx.x; e < 5 * P; e += blockDim.x) L[e] = {0.0, 0.0};
    if (b && threadIdx.x < 5) b[threadIdx.x] = {0.0, 0.0};
  }
  for (int n = threadIdx.x; n < N; n += blockDim.x) {
    const int64_t at = level_off(root) + box;
    double2 v;
    if (root == 2) {
      const float2 o = n < P ? Lm2l[at * P + n] : bm2l[at];
      v = {o.x, o.y};
      if (n < P) L[at * P + n] = v;
      else b[at] = v;
    } else {
      v = n < P ? L[at * P + n] : b[at];
    }
    buf[0][0][n] = v;
  }
  __syncthreads();
  for (int s = 0; s < span; ++s) {
    const int np = 1 << (2 * s);
    const int64_t ch0 = level_off(root + s + 1) + (box << (2 * s + 2));
    double2(*cur)[P + 1] = buf[s & 1], (*next)[P + 1] = buf[(s + 1) & 1];
    const int it = threadIdx.x;
    if (it < np * N) {
      const int i = it / N, n = it - i * N;
      const bool is_b = n == P;
      float2 own[4] = {wide[0], wide[1], wide[2], wide[3]};
      if (s + 1 < span) load_own(s, own);
      double vx[4], vy[4];
      down_sums<double, P>(kShiftD, cur[i], is_b ? kB : n, is_b ? -1 : n, vx, vy);
      const double sc = is_b ? 1.0 : 0.5;  // 2^-(m+1) = 2^-m / 2; b's column has it
      const double bx = is_b ? cur[i][P].x : 0.0, by = is_b ? cur[i][P].y : 0.0;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const double2 o = {bx + sc * vx[c] + own[c].x, by + sc * vy[c] + own[c].y};
        const int64_t at = ch0 + 4 * i + c;
        *(is_b ? b + at : L + at * P + n) = o;
        if (s + 1 < span) next[4 * i + c][n] = o;
      }
    }
    __syncthreads();
  }
}

__global__ void f64_to_f32_kernel(const double2 *__restrict__ a, float2 *__restrict__ b, int64_t n) {
  const int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (i >= n) return;
  const double2 v = a[i];
  b[i] = make_float2(float(v.x), float(v.y));
}

// ------------------------------------------------------------------ L2P --
// Two Horner schemes in w (the field's, and phi's with coefficients
// L_n / (n + 1)), one target a thread; targets of a leaf read the same lines.
// Bound by the latency of its chain of reads, then by memory: with the leaf
// confirmed ahead of its coefficients 387 us at 2^24 targets, p = 20, now 313
// (1.0 GB, 207 us at the rate of a large copy); 4e6, p = 16: 59 and 53.
// ADD: into phi and field, else they are overwritten.

template <int P, bool ADD>
__global__ void l2p_kernel(const float2 *__restrict__ txy, const int32_t *__restrict__ tls, int64_t nt, int depth,
                           const double2 *__restrict__ L, const double2 *__restrict__ b, float2 *__restrict__ phi,
                           float2 *__restrict__ field) {
  const int64_t t = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  const int64_t nleaf = int64_t(1) << (2 * depth);
  if (t >= nt) return;
  const float2 z = txy[t];
  const int32_t end = tls[nleaf];
  const double h = ldexp(1.0, -depth), ih = ldexp(1.0, depth);  // exact
  double fr, fi, pr, pi;
  at_leaf(z, tls, nleaf, depth, t, [&](int64_t m) {
    uint32_t ix, iy;
    unmorton2(uint32_t(m), ix, iy);
    const double wr = (double(z.x) - (double(ix) + 0.5) * h) * ih;
    const double wi = (double(z.y) - (double(iy) + 0.5) * h) * ih;
    const double2 *Ll = L + (level_off(depth) + m) * P;
    const double2 bb = b ? b[level_off(depth) + m] : make_double2(0.0, 0.0);
    fr = fi = pr = pi = 0.0;
#pragma unroll
    for (int n = P - 1; n >= 0; --n) {
      const double2 ln = Ll[n];
      constexpr double one = 1.0;
      const double inv = one / double(n + 1);
      const double tr = fma(fr, wr, fma(-fi, wi, ln.x)), ti = fma(fr, wi, fma(fi, wr, ln.y));
      fr = tr, fi = ti;
      const double ur = fma(pr, wr, fma(-pi, wi, inv * ln.x)), ui = fma(pr, wi, fma(pi, wr, inv * ln.y));
      pr = ur, pi = ui;
    }
    const double br = pr * wr - pi * wi, bi = pr * wi + pi * wr;  // times w
    pr = b ? br + bb.x : br, pi = b ? bi + bb.y : bi;
    return float(pr);
  });
  if (t >= int64_t(end)) return;
  if (field) {
    const float2 o = ADD ? field[t] : make_float2(0.f, 0.f);
    field[t] = make_float2(o.x + float(fr * ih), o.y + float(fi * ih));
  }
  if (phi) {
    const float2 o = ADD ? phi[t] : make_float2(0.f, 0.f);
    phi[t] = make_float2(o.x + float(pr), o.y + float(pi));
  }
}

// L2P^T: gL_n = sum_t [cphi w^(n+1)/(n+1) + cfield w^n / h], gb = sum_t cphi.
// The sums of cphi w^(n+1) take their 1/(n+1) once at the end.
template <int P, int LANES, bool CPHI, bool CF>
__global__ __launch_bounds__(256) void l2p_backward_kernel(const float2 *__restrict__ txy,
                                                           const int32_t *__restrict__ tls, int depth,
                                                           const float2 *__restrict__ cphi,
                                                           const float2 *__restrict__ cfield,
                                                           double2 *__restrict__ gL, double2 *__restrict__ gb) {
  const int64_t nleaf = int64_t(1) << (2 * depth);
  const int64_t m = (blockIdx.x * int64_t(256) + threadIdx.x) / LANES;
  if (m >= nleaf) return;  // whole leaves
  const int r = threadIdx.x % LANES;
  uint32_t ix, iy;
  unmorton2(uint32_t(m), ix, iy);
  const double h = ldexp(1.0, -depth), ih = ldexp(1.0, depth);  // exact
  const double cx = (double(ix) + 0.5) * h, cy = (double(iy) + 0.5) * h;
  double ar[P], ai[P];
#pragma unroll
  for (int n = 0; n < P; ++n) ar[n] = ai[n] = 0.0;
  double sbr = 0.0, sbi = 0.0;
  const int64_t first = tls[m] + int64_t(r);
  txy += first;
  cphi += CPHI ? first : 0;
  cfield += CF ? first : 0;
  for (int32_t left = tls[m + 1] - tls[m] - r; left > 0; left -= LANES, txy += LANES) {
    const float2 z = *txy;
    const double wr = (double(z.x) - cx) * ih, wi = (double(z.y) - cy) * ih;
    double cr = 0.0, ci = 0.0, dr = 0.0, di = 0.0;  // cphi w^n, cfield w^n / h
    if (CPHI) {
      const float2 c = *cphi;
      cphi += LANES;
      cr = c.x, ci = c.y;
      sbr += cr, sbi += ci;
    }
    if (CF) {
      const float2 c = *cfield;
      cfield += LANES;
      dr = double(c.x) * ih, di = double(c.y) * ih;
    }
#pragma unroll
    for (int n = 0; n < P; ++n) {
      if (CF) {
        ar[n] += dr;
        ai[n] += di;
        const double tr = dr * wr - di * wi;
        di = dr * wi + di * wr;
        dr = tr;
      }
      if (CPHI) {
        const double tr = cr * wr - ci * wi;
        ci = cr * wi + ci * wr;
        cr = tr;
        constexpr double one = 1.0;
        const double inv = CF ? one / double(n + 1) : one;
        ar[n] = fma(inv, cr, ar[n]);
        ai[n] = fma(inv, ci, ai[n]);
      }
    }
  }
#pragma unroll
  for (int n = 0; n < P; ++n) {
    constexpr double one = 1.0;
    const double inv = CPHI && !CF ? one / double(n + 1) : one;
    ar[n] = inv * lanes_sum<LANES>(ar[n]);
    ai[n] = inv * lanes_sum<LANES>(ai[n]);
  }
  store_sums<P, LANES>(ar, ai, gL + (level_off(depth) + m) * P, r);
  if (gb) {
    sbr = lanes_sum<LANES>(sbr);
    sbi = lanes_sum<LANES>(sbi);
    if (r == 0) gb[level_off(depth) + m] = make_double2(sbr, sbi);
  }
}

// ------------------------------------------------------------- launchers --

static inline unsigned blocks_for(int64_t n, int bs = 256) { return unsigned((n + bs - 1) / bs); }

// f<P> for the order p
#define FOR_P(f, ...)                 \
  switch (p) {                        \
    case 8: f<8>(__VA_ARGS__); break;   \
    case 12: f<12>(__VA_ARGS__); break; \
    case 16: f<16>(__VA_ARGS__); break; \
    case 20: f<20>(__VA_ARGS__); break; \
  }

template <int P>
static void p2m_p(const float2 *x, const float *q, const int32_t *ls, int depth, float2 *M, hipStream_t s) {
  const int64_t nleaf = int64_t(1) << (2 * depth);
  const int lanes = leaf_lanes(nleaf);
  const dim3 g(blocks_for(nleaf * lanes)), bl(256);
  if (lanes == 16) hipLaunchKernelGGL((p2m_kernel<P, 16>), g, bl, 0, s, x, q, ls, depth, M);
  else hipLaunchKernelGGL((p2m_kernel<P, 4>), g, bl, 0, s, x, q, ls, depth, M);
}

int launch_p2m(const float *xy, const float *q, const int32_t *ls, int depth, int p, float *M, hipStream_t s) {
  FOR_P(p2m_p, reinterpret_cast<const float2 *>(xy), q, ls, depth, reinterpret_cast<float2 *>(M), s)
  return check_launch("p2m");
}

template <int P>
static void p2m_backward_p(const float2 *x, const float *q, const int32_t *ls, int64_t n, int depth, const float2 *gM,
                           float *gq, float2 *G, hipStream_t s) {
  hipLaunchKernelGGL(p2m_backward_kernel<P>, dim3(blocks_for(n)), dim3(256), 0, s, x, q, ls, n, depth, gM, gq, G);
}

int launch_p2m_backward(const float *xy, const float *q, const int32_t *ls, int64_t n, int depth, int p,
                        const float *gM, float *gq, float *G, hipStream_t s) {
  if (n == 0) return FMM2D_OK;
  FOR_P(p2m_backward_p, reinterpret_cast<const float2 *>(xy), q, ls, n, depth, reinterpret_cast<const float2 *>(gM),
        gq, reinterpret_cast<float2 *>(G), s)
  return check_launch("p2m_backward");
}

// Levels bottom - 1 .. top from the level `bottom`, up to kSpan a launch.
template <typename T, int P, bool WITH_B>
static void sweep_up(typename Pair<T>::type *a, typename Pair<T>::type *b, float2 *a32, float2 *b32, int bottom,
                     int top, T scale, hipStream_t s) {
  for (bool leaves = true; bottom > top; leaves = false) {
    const int span = bottom - top < kSpan ? bottom - top : kSpan, root = bottom - span;
    hipLaunchKernelGGL((shift_up_kernel<T, P, WITH_B>), dim3(1u << (2 * root)), dim3(shift_threads(P)), 0, s, a, b,
                       a32, b32, root, span, leaves, scale);
    bottom = root;
  }
}

template <int P>
static void m2m_p(float2 *M, int depth, int top, hipStream_t s) {
  sweep_up<float, P, false>(M, nullptr, nullptr, nullptr, depth, top, 1.f, s);
}

int launch_m2m(float *M, int depth, int top, int p, hipStream_t s) {
  FOR_P(m2m_p, reinterpret_cast<float2 *>(M), depth, top, s)
  return check_launch("m2m");
}

// Calls f(root, span) for the levels 3 .. depth from level 2 down, the short
// span first: the deepest launch is the large one and takes whole subtrees.
template <typename F>
static void sweep_down(int depth, F f) {
  int root = 2, span = (depth - 2) % kSpan;
  if (span == 0 && depth > 2) span = kSpan;
  do {
    f(root, span);
    root += span;
    span = kSpan;
  } while (root < depth);
}

template <int P>
static void m2m_backward_p(float2 *g, int depth, hipStream_t s) {
  if (depth < 3) return;
  sweep_down(depth, [&](int root, int span) {
    hipLaunchKernelGGL(m2m_backward_kernel<P>, dim3(1u << (2 * root)), dim3(shift_threads(P)), 0, s, g, root, span);
  });
}

int launch_m2m_backward(float *gM, int depth, int p, hipStream_t s) {
  FOR_P(m2m_backward_p, reinterpret_cast<float2 *>(gM), depth, s)
  return check_launch("m2m_backward");
}

template <int P>
static void l2l_p(const float2 *Lm, const float2 *bm, double2 *L, double2 *b, int depth, hipStream_t s) {
  sweep_down(depth, [&](int root, int span) {
    hipLaunchKernelGGL(l2l_kernel<P>, dim3(1u << (2 * root)), dim3(shift_threads(P)), 0, s, Lm, bm, L, b, root, span);
  });
}

int launch_l2l(const float *Lm2l, const float *bm2l, double *L, double *b, int depth, int p, hipStream_t s) {
  FOR_P(l2l_p, reinterpret_cast<const float2 *>(Lm2l), reinterpret_cast<const float2 *>(bm2l),
        reinterpret_cast<double2 *>(L), reinterpret_cast<double2 *>(b), depth, s)
  return check_launch("l2l");
}

template <int P>
static void l2l_backward_p(double2 *g, double2 *gb, float2 *g32, float2 *gb32, int depth, hipStream_t s) {
  if (depth == 2) {  // the leaf level is the top one: only its FP32 values
    const int64_t o = level_off(2), nb = 16;
    hipLaunchKernelGGL(f64_to_f32_kernel, dim3(blocks_for(nb * P)), dim3(256), 0, s, g + o * P, g32 + o * P, nb * P);
    if (gb) hipLaunchKernelGGL(f64_to_f32_kernel, dim3(1), dim3(256), 0, s, gb + o, gb32 + o, nb);
  } else if (gb) {
    sweep_up<double, P, true>(g, gb, g32, gb32, depth, 2, 0.5, s);
  } else {
    sweep_up<double, P, false>(g, gb, g32, gb32, depth, 2, 0.5, s);
  }
}

int launch_l2l_backward(double *gL, double *gb, float *gLm2l, float *gbm2l, int depth, int p, hipStream_t s) {
  double2 *g = reinterpret_cast<double2 *>(gL);
  FOR_P(l2l_backward_p, g, reinterpret_cast<double2 *>(gb), reinterpret_cast<float2 *>(gLm2l),
        reinterpret_cast<float2 *>(gbm2l), depth, s)
  return check_launch("l2l_backward");
}

template <int P>
static void l2p_p(const float2 *t, const int32_t *tls, int64_t nt, const double2 *L, const double2 *b, int depth,
                  float2 *ph, float2 *fi, bool add, hipStream_t s) {
  const dim3 g(blocks_for(nt)), bl(256);
  if (add) hipLaunchKernelGGL((l2p_kernel<P, true>), g, bl, 0, s, t, tls, nt, depth, L, b, ph, fi);
  else hipLaunchKernelGGL((l2p_kernel<P, false>), g, bl, 0, s, t, tls, nt, depth, L, b, ph, fi);
}

int launch_l2p(const float *txy, const int32_t *tls, int64_t nt, const double *L, const double *b, int depth, int p,
               float *phi, float *field, bool add, hipStream_t s) {
  if (nt == 0) return FMM2D_OK;
  FOR_P(l2p_p, reinterpret_cast<const float2 *>(txy), tls, nt, reinterpret_cast<const double2 *>(L),
        reinterpret_cast<const double2 *>(b), depth, reinterpret_cast<float2 *>(phi),
        reinterpret_cast<float2 *>(field), add, s)
  return check_launch("l2p");
}

template <int P>
static void l2p_backward_p(const float2 *t, const int32_t *tls, const float2 *cp, const float2 *cf, int depth,
                           double2 *g, double2 *gb, hipStream_t s) {
  const int64_t nleaf = int64_t(1) << (2 * depth);
  const int lanes = leaf_lanes(nleaf);
  const dim3 gr(blocks_for(nleaf * lanes)), bl(256);
#define LAUNCH(LANES, CP, CF) \
  hipLaunchKernelGGL((l2p_backward_kernel<P, LANES, CP, CF>), gr, bl, 0, s, t, tls, depth, cp, cf, g, gb)
  if (lanes == 16) {
    if (cp && cf) LAUNCH(16, true, true);
    else if (cp) LAUNCH(16, true, false);
    else if (cf) LAUNCH(16, false, true);
    else LAUNCH(16, false, false);
  } else {
    if (cp && cf) LAUNCH(4, true, true);
    else if (cp) LAUNCH(4, true, false);
    else if (cf) LAUNCH(4, false, true);
    else LAUNCH(4, false, false);
  }
#undef LAUNCH
}

int launch_l2p_backward(const float *txy, const int32_t *tls, const float *cphi, const float *cfield, int depth,
                        int p, double *gL, double *gb, hipStream_t s) {
  FOR_P(l2p_backward_p, reinterpret_cast<const float2 *>(txy), tls, reinterpret_cast<const float2 *>(cphi),
        reinterpret_cast<const float2 *>(cfield), depth, reinterpret_cast<double2 *>(gL),
        reinterpret_cast<double2 *>(gb), s)
  return check_launch("l2p_backward");
}

}  // namespace fmm2d
