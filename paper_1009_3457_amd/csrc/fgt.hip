// Fast Gauss transform, Hermite stage (Sec. 2.2; Sec. 4.2): the coefficients
// of Eq. (eqn:A_alpha) per box and their evaluation, Eq. (eqn:hermite), at
// the targets, in two dimensions on the 4^depth boxes of the uniform grid.
//
// Evaluation has two paths.  With a workspace, and where the cost rule below
// says so, the series of a box's (2K+1)^2 neighbours are first re-expanded
// into one Taylor polynomial about the box's centre (one separable
// contraction per axis on FP32 matrix instructions), and each target then
// evaluates its own box's polynomial: see "Taylor path" below.
//
// The direct path evaluates, for a target and one box, the bilinear form
//     sum_{a,b<p} h_a(t1) A_ab h_b(t2),   t = (y - s_B) / (sqrt(2) sigma),
// p^2 multiply-adds on one box's coefficient matrix after two Hermite-function
// recurrences.  One target per lane; every lane of a wave visits the same box
// at the same time, so the box's coefficients are wave-uniform and come in
// through scalar loads, feeding the multiply-adds as scalar operands: no LDS
// and no vector memory traffic in the inner loop.  A wave covers either the
// bounding rectangle of its targets' (2K+1)^2 neighbourhoods, each lane
// masked to its own neighbourhood, or each distinct target box in turn,
// whichever visits fewer boxes.  Targets sorted by box (Morton order) keep a
// wave within one or two adjacent boxes, where the rectangle costs about 6%
// over the lanes' own neighbourhoods.
#include <algorithm>
#include <cmath>

#include "fgt2d.h"
#include "fmm2d_internal.h"

namespace fmm2d {

namespace {

// ------------------------------------------------------- coefficients --

// A[box][a][b] = 1/(a! b!) sum_j q_j s1^a s2^b, s = (x_j - s_B) / (sqrt(2) sigma),
// FP64 sums rounded once, by one of two kernels.
//
// Boxes of many sources: the (a, j) x (j, b) product of the sources' powers
// on FP64 matrix instructions, one wave per box.  Sources go 32 at a time:
// each lane forms the powers of one source on one axis (P - 1 products) and
// leaves them in the wave's LDS slice, rows kPowRow doubles apart so that the
// 16 rows of a fragment read fall into different banks; 4 sources a k-step
// then meet in one 16x16x4 product.  The next 32 sources load meanwhile.
//
// Boxes of few sources: a thread per (box, a) forms q s1^a anew for each
// source and sums it over b in registers; no lane waits for a wave's latency
// with nothing to do.
//
// 65536 boxes of 100 sources, p = 12: 92 us by products, 204 by threads; 2^20
// boxes of 0.3 sources, p = 5: 219 and 34.  Up to depth 7 products take all
// boxes: few as they are, the two are level there (9 and 8 us at p = 5, two
// sources a box).  Past it the mean of 64 consecutive boxes decides, at the
// sources a box where the two meet (16 and 40 at p = 9, 8 and 16 at p = 12, 4
// and 16 at p = 16 are either side of it for 65536 to 2^20 boxes; about 80 at p = 5);
// a box's own count would have both kernels at work on every wave's
// boxes near that line (61 us for 38 at p = 12, 16 sources a box).  A box of
// twice that line is left to products whatever its neighbours have, as its
// threads would be waited for (0.4 us a source).
constexpr int kPowRow = 34;
template <int P>
constexpr uint32_t kMeet = 1900 / (P * P) < 128 ? 1900 / (P * P) : 128;
constexpr int kThreadsFrom = 8;  // depth

// Whether products form a box of `count` sources, `around` those of its 64.
template <int P>
__device__ __forceinline__ bool by_products(uint32_t count, uint32_t around) {
  return around > 64 * kMeet<P> || count > 2 * kMeet<P>;
}

template <int P>
__global__ __launch_bounds__(256) void fgt_coeffs_few_kernel(const float2 *__restrict__ xy, const float *__restrict__ q,
                                                             const int32_t *__restrict__ ls, int depth, double scale,
                                                             float *__restrict__ A) {
  const int64_t nbox = int64_t(1) << (2 * depth);
  const int64_t e = blockIdx.x * int64_t(256) + threadIdx.x;
  if (e >= nbox * P) return;
  const int64_t m = e / P;
  const int a = int(e - m * P);
  const int32_t jb = ls[m], je = ls[m + 1];
  const int64_t m64 = m & ~int64_t(63);
  if (by_products<P>(uint32_t(je - jb), uint32_t(ls[m64 + 64] - ls[m64]))) return;
  uint32_t bx, by;
  unmorton2(uint32_t(m), bx, by);
  const double w = ldexp(1.0, -depth);
  const double c1 = (double(bx) + 0.5) * w, c2 = (double(by) + 0.5) * w;
  double acc[P];
#pragma unroll
  for (int b = 0; b < P; ++b) acc[b] = 0.0;
  float2 xn = make_float2(0.f, 0.f);
  float qn = 0.f;
  if (jb < je) xn = xy[jb], qn = q[jb];
  for (int32_t j = jb; j < je; ++j) {
    const double s1 = (double(xn.x) - c1) * scale, s2 = (double(xn.y) - c2) * scale;
    double p = double(qn);  // q s1^a, then times s2^b
    if (j + 1 < je) xn = xy[j + 1], qn = q[j + 1];
    for (int i = 0; i < a; ++i) p *= s1;
#pragma unroll
    for (int b = 0; b < P; ++b) {
      acc[b] += p;
      p *= s2;
    }
  }
  double f = 1.0;  // a! b!
  for (int i = 2; i <= a; ++i) f *= double(i);
  float *out = A + (m * P + a) * P;
#pragma unroll
  for (int b = 0; b < P; ++b) {
    if (b >= 2) f *= double(b);
    out[b] = float(acc[b] / f);
  }
}

// G > 1: a wave looks at G boxes, far apart so that a cluster's go to many
// waves (consecutive ones: 3e6 points, half of them in a 20th of each axis,
// 640 us for 250), and takes those that fgt_coeffs_few_kernel leaves; the
// first sources of the next of them load while a box is finished.
template <int P, int G>
__global__ __launch_bounds__(256) void fgt_coeffs_kernel(const float2 *__restrict__ xy, const float *__restrict__ q,
                                                         const int32_t *__restrict__ ls, int depth, double scale,
                                                         float *__restrict__ A) {
  __shared__ double pow12[4][2][P * kPowRow];  // [wave][axis][power][source]
  const int64_t nbox = int64_t(1) << (2 * depth);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t stride = nbox / G, m0 = blockIdx.x * int64_t(4) + wave;  // box b of the wave's: m0 + b stride
  if (m0 >= stride) return;
  const double w = ldexp(1.0, -depth);
  const int axis = lane >> 5, src = lane & 31;
  double *mine = pow12[wave][axis] + src;
  typedef double d4 __attribute__((ext_vector_type(4)));
  const int row = lane & 15, kq = lane >> 4;
  // rows and columns past P repeat row 0 and are not stored
  const double *w1 = pow12[wave][0] + (row < P ? row : 0) * kPowRow + kq;
  const double *w2 = pow12[wave][1] + (row < P ? row : 0) * kPowRow + kq;
  const float *co = reinterpret_cast<const float *>(xy) + axis;
  // lane b: the sources of box b of the wave's; unsigned: a step may pass 2^31
  const int64_t mine_at = m0 + (G == 1 ? 0 : min(lane, G - 1)) * stride;
  const uint32_t begins = ls[mine_at], ends = ls[mine_at + 1];
  uint64_t left = 1;
  if constexpr (G > 1) {
    const int64_t m64 = mine_at & ~int64_t(63);
    left = __ballot(lane < G && by_products<P>(ends - begins, uint32_t(ls[m64 + 64] - ls[m64])));
  }
  if (left == 0) return;
  int box = __ffsll(static_cast<long long>(left)) - 1;
  uint32_t jb = __builtin_amdgcn_readlane(begins, box), je = __builtin_amdgcn_readlane(ends, box);
  float xn = 0.f, qn = 0.f;
  if (jb + src < je) xn = co[2 * int64_t(jb + src)], qn = q[jb + src];
  for (;;) {
    left &= left - 1;
    const int next = left ? __ffsll(static_cast<long long>(left)) - 1 : box;
    const uint32_t nb = left ? __builtin_amdgcn_readlane(begins, next) : je, ne = __builtin_amdgcn_readlane(ends, next);
    uint32_t bx, by;
    const int64_t m = m0 + box * stride;
    unmorton2(uint32_t(m), bx, by);
    const double c = (double(axis ? by : bx) + 0.5) * w;
    d4 acc = {0.0, 0.0, 0.0, 0.0};
    if (jb == je && nb + src < ne) xn = co[2 * int64_t(nb + src)], qn = q[nb + src];  // an empty box among full ones
    for (uint32_t j0 = jb; j0 < je; j0 += 32) {
      const int cnt = int(min(32u, je - j0));
      const bool live = src < cnt;  // a source past the end has charge 0
      const double s = live ? (double(xn) - c) * scale : 0.0;
      double p = !live ? 0.0 : axis ? 1.0 : double(qn);  // q s1^a, s2^b
#pragma unroll
      for (int a = 0; a < P; ++a) {
        mine[a * kPowRow] = p;
        p *= s;
      }
      const bool last = je - j0 <= 32u;
      const uint32_t jn = (last ? nb : j0 + 32) + src;
      if (jn < (last ? ne : je)) xn = co[2 * int64_t(jn)], qn = q[jn];
      __builtin_amdgcn_wave_barrier();  // the wave's LDS accesses complete in order
      for (int k = 0; k < cnt; k += 4) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(w1[k], w2[k], acc, 0, 0, 0);
      __builtin_amdgcn_wave_barrier();
    }
    if (row < P) {
      double fb = 1.0;  // b!
      for (int i = 2; i <= row; ++i) fb *= double(i);
      float *out = A + m * (P * P) + row;
      double fa = 1.0;  // a!
      int done = 1;
#pragma unroll
      for (int e = 0; e < 4; ++e) {  // D: row a = 4 e + lane / 16, column b = lane % 16
        const int a = 4 * e + kq;
        for (; done < a; ++done) fa *= double(done + 1);
        if (a < P) out[a * P] = float(acc[e] / (fa * fb));
      }
    }
    if (left == 0) return;
    box = next;
    jb = nb;
    je = ne;
  }
}

// --------------------------------------------------------- evaluation --

// h_n(t) = exp(-t^2) H_n(t) for n < P by H_{n+1} = 2t H_n - 2n H_{n-1}, with
// e = exp(-t^2) already applied (zero masks the lane).
template <int P>
__device__ __forceinline__ void hermite_fns(float t, float e, float (&h)[P]) {
  const float tt = 2.f * t;
  h[0] = e;
  if (P > 1) h[1] = tt * e;
#pragma unroll
  for (int n = 1; n + 1 < P; ++n) h[n + 1] = fmaf(tt, h[n], -2.f * float(n) * h[n - 1]);
}

__device__ __forceinline__ float gauss(float t) { return __expf(-t * t); }

__device__ __forceinline__ int wave_min(int v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v = min(v, __shfl_xor(v, m));
  return __builtin_amdgcn_readfirstlane(v);
}

__device__ __forceinline__ int wave_max(int v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v = max(v, __shfl_xor(v, m));
  return __builtin_amdgcn_readfirstlane(v);
}

// acc += sum_a h1[a] sum_b Ab[a][b] h2[b]; Ab is wave-uniform.
template <int P>
__device__ __forceinline__ float bilinear(const float *__restrict__ Ab, const float (&h1)[P], const float (&h2)[P],
                                          float acc) {
#pragma unroll
  for (int a = 0; a < P; ++a) {
    float v = 0.f;
#pragma unroll
    for (int b = 0; b < P; ++b) v = fmaf(Ab[a * P + b], h2[b], v);
    acc = fmaf(h1[a], v, acc);
  }
  return acc;
}

// Box columns per strip of the sweep: h1 of a strip's columns stays in
// registers while the rows go by, so h1 is formed once per column and h2
// once per strip and row, against h1 once per box.  For p >= 10 the
// strips were slower (8.9-9.3 ms against 8.3 ms at p = 12, 6.5M targets):
// a box's p^2 coefficients then fill the scalar registers and the unrolled
// strip holds back their loads, so those orders sweep box by box (1).
template <int P>
constexpr int kStrip = P <= 9 ? 4 : 1;

// Sum over boxes (i, j), x0 <= i <= x1, y0 <= j <= y1 (all wave-uniform);
// a lane takes box (i, j) only if |i - bx| <= K and |j - by| <= K and sel.
template <int P>
__device__ __forceinline__ float sweep(const float *__restrict__ A, float2 y, int bx, int by, bool sel, int K,
                                       int x0, int x1, int y0, int y1, float wb, float inv_s, float acc) {
  constexpr int W = kStrip<P>;
  if constexpr (W == 1) {
    for (int j = y0; j <= y1; ++j) {
      const float t2 = (y.y - (float(j) + 0.5f) * wb) * inv_s;
      const bool row = sel && abs(j - by) <= K;
      float h2[P];
      hermite_fns<P>(t2, row ? gauss(t2) : 0.f, h2);
      for (int i = x0; i <= x1; ++i) {
        const float t1 = (y.x - (float(i) + 0.5f) * wb) * inv_s;
        const bool in = abs(i - bx) <= K;
        float h1[P];
        hermite_fns<P>(t1, in ? gauss(t1) : 0.f, h1);
        const float *Ab = A + int64_t(morton2(uint32_t(i), uint32_t(j))) * (P * P);
        acc = bilinear<P>(Ab, h1, h2, acc);
      }
    }
    return acc;
  }
  for (int i0 = x0; i0 <= x1; i0 += W) {
    float h1[W][P];
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const int i = i0 + w;  // past x1: never used
      const float t1 = (y.x - (float(i) + 0.5f) * wb) * inv_s;
      const bool in = abs(i - bx) <= K;
      hermite_fns<P>(t1, in ? gauss(t1) : 0.f, h1[w]);
    }
    for (int j = y0; j <= y1; ++j) {
      const float t2 = (y.y - (float(j) + 0.5f) * wb) * inv_s;
      const bool row = sel && abs(j - by) <= K;
      float h2[P];
      hermite_fns<P>(t2, row ? gauss(t2) : 0.f, h2);
#pragma unroll
      for (int w = 0; w < W; ++w) {
        if (i0 + w > x1) break;  // wave-uniform: no coefficients past the rectangle
        const float *Ab = A + int64_t(morton2(uint32_t(i0 + w), uint32_t(j))) * (P * P);
        acc = bilinear<P>(Ab, h1[w], h2, acc);
      }
    }
  }
  return acc;
}

// Box coordinate of a target, clamped (fminf/fmaxf also map NaN into the grid).
__device__ __forceinline__ int clamped_box(float v, float fs) {
  return int(fminf(fmaxf(floorf(v * fs), 0.f), fs - 1.f));
}

// Blocks are dispatched to the 8 XCDs in turn (b mod 8).  Each XCD takes a
// contiguous eighth of the (box-ordered) targets, so the coefficient boxes
// that neighbouring waves visit are fetched once into that XCD's L2.
__device__ __forceinline__ int64_t xcd_block() {
  const int64_t nb = gridDim.x, b = blockIdx.x;
  return (nb % 8 == 0) ? (b % 8) * (nb / 8) + b / 8 : b;
}

// The sum over the neighbourhood of one target per lane.
template <int P>
__device__ __forceinline__ float eval_wave(const float2 y, int depth, float inv_s, int K,
                                           const float *__restrict__ A) {
  const int side = 1 << depth;
  const float fs = float(side), wb = 1.f / fs;  // exact powers of two
  const int bx = clamped_box(y.x, fs), by = clamped_box(y.y, fs);

  // option 1: the bounding rectangle of the wave's neighbourhoods
  const int x0 = max(wave_min(bx) - K, 0), x1 = min(wave_max(bx) + K, side - 1);
  const int y0 = max(wave_min(by) - K, 0), y1 = min(wave_max(by) + K, side - 1);
  const int64_t rect = int64_t(x1 - x0 + 1) * (y1 - y0 + 1);
  // option 2: each distinct target box with its own clipped neighbourhood
  const int key = bx | (by << 16);
  int64_t per_box = 0;
  uint64_t left = __ballot(1);
  while (left) {
    const int k = __builtin_amdgcn_readfirstlane(__shfl(key, __ffsll(static_cast<long long>(left)) - 1));
    const int kx = k & 0xffff, ky = k >> 16;
    per_box += int64_t(min(kx + K, side - 1) - max(kx - K, 0) + 1) * (min(ky + K, side - 1) - max(ky - K, 0) + 1);
    left &= ~__ballot(key == k);
  }

  float acc = 0.f;
  if (rect <= per_box) {
    acc = sweep<P>(A, y, bx, by, true, K, x0, x1, y0, y1, wb, inv_s, acc);
  } else {
    left = __ballot(1);
    while (left) {
      const int k = __builtin_amdgcn_readfirstlane(__shfl(key, __ffsll(static_cast<long long>(left)) - 1));
      const int kx = k & 0xffff, ky = k >> 16;
      acc = sweep<P>(A, y, bx, by, key == k, K, max(kx - K, 0), min(kx + K, side - 1), max(ky - K, 0),
                     min(ky + K, side - 1), wb, inv_s, acc);
      left &= ~__ballot(key == k);
    }
  }
  return acc;
}

template <int P>
__global__ __launch_bounds__(256) void fgt_eval_kernel(const float2 *__restrict__ txy, int64_t nt, int depth,
                                                       float inv_s, int K, const float *__restrict__ A,
                                                       const int32_t *__restrict__ place, float *__restrict__ G) {
  const int64_t t0 = (xcd_block() * 4 + (threadIdx.x >> 6)) * 64;
  if (t0 >= nt) return;  // whole wave
  const int64_t t = t0 + (threadIdx.x & 63);
  const bool act = t < nt;
  const float2 y = txy[act ? t : t0];  // idle lanes follow lane 0's target
  const float acc = eval_wave<P>(y, depth, inv_s, K, A);
  if (act) G[place ? place[t] : t] = acc;
}

// --------------------------------------------------------- Taylor path --
//
// With delta the target's offset from its own box's centre and o = B - T the
// offset of a source box, both in units of sqrt(2) sigma after the factor
// r = 2^-depth / (sqrt(2) sigma), t = delta - r o, and h_n' = -h_{n+1} gives
//     h_a(delta - r o) = sum_m u^m T_o[m][a],   u = 2 delta / r in [-1, 1],
//     T_o[m][a] = (-r/2)^m / m! h_{a+m}(-r o).
// So the sum over the (2K+1)^2 boxes is a polynomial in (u1, u2) whose
// coefficients separate over the axes:
//     W(tx, by)[m1][b] = sum_ox sum_a T_ox[m1][a] A(tx + ox, by)[a][b]
//     C(tx, ty)[m2][m1] = sum_oy sum_b T_oy[m2][b] W(tx, ty + oy)[m1][b]
// (2K+1) 2 p q^2-sized products per box instead of (2K+1)^2 p^2 per target.
//
// q is the smallest even order whose remainder on one axis is at most 2^-25 for
// a unit charge: with |s|, |delta| <= r/2 and
// Cramer's |h_n| <= 1.0865 2^(n/2) sqrt(n!), it is at most
// R = 1.0865 sum_{m>=q} (r/2)^m/m! sum_{a<p} (r/2)^a/a! 2^((a+m)/2) sqrt((a+m)!).
// An axis's own sum is at most F = 1 + rho, rho the truncation to p terms, so
// the product of both is off by at most R (2F + R), 2^-24 (1 + rho): an ulp of
// the Gaussian's peak.  (The largest found, over r = 0.2 .. 1.3 and p = 5 .. 16,
// is 0.41 2^-25.)
// r = 1/2 takes q = 12; past r = 1 (p = 12) 16 terms don't reach it and the
// call stays on the direct path.  T is formed in FP64 and rounded once, both
// contractions and the polynomial (a Horner scheme in u, which is exact) run
// in FP32, as the direct path does, with far shorter sums: the error against FP64
// fell from 6.3e-7 to 3.0e-7 (6.5M targets, p = 12; FP64 products would give
// 0.6e-7 at 170 us an axis instead of 66 to 75).  Evaluation at 6.5M targets,
// p = 12, K = 8, 65536 boxes: 8400 us directly, 215 us here (66 + 75 for the
// two axes, 64 for the targets, 10 for the table and the outside check).

constexpr int kMaxQ = 16;

__global__ __launch_bounds__(256) void fgt_taylor_table_kernel(int p, int ks, int K, double r, float *__restrict__ T,
                                                               uint32_t *__restrict__ outside) {
  // T[o + K][k-step][lane]: the A fragment of v_mfma_f32_16x16x4_f32, row
  // m = lane % 16, column a = 4 k-step + lane / 16 (zero for a >= p)
  const int e = threadIdx.x, lane = e & 63, step = e >> 6;
  if (blockIdx.x == 0 && e == 0) *outside = 0u;
  if (step >= ks) return;
  const int m = lane & 15, a = 4 * step + (lane >> 4);
  const double t = -r * double(int(blockIdx.x) - K);
  double h0 = exp(-t * t), h1 = 2.0 * t * h0;  // h_n, h_{n+1}
  double f = 1.0;                              // (-r/2)^m / m!
  for (int n = 0; n < a + m; ++n) {
    const double h2 = 2.0 * t * h1 - 2.0 * double(n + 1) * h0;
    h0 = h1;
    h1 = h2;
  }
  for (int i = 1; i <= m; ++i) f *= -0.5 * r / double(i);
  T[(int64_t(blockIdx.x) * ks + step) * 64 + lane] = a < p ? float(f * h0) : 0.f;
}

// One axis of the re-expansion: out[m] of column c of box x is
// sum_{o, k} T_o[m][k] in(x + o)[k][c], for `tiles` boxes in a line.
//   AXIS 0 (along x): in = A (Morton order, p x p, column b, k = a, out = W)
//   AXIS 1 (along y): in = W ([tx][ty][m1][b], column m1, k = b, out = C)
// A workgroup takes TX boxes of one line; their columns are the N dimension
// of 16x16x4 FP32 products, 16 columns a tile, up to 4 tiles a wave, the
// T fragments and the line's boxes (TX + kOffsets - 1 of them) in LDS.
// Bound by the matrix pipe, 32 cycles a product, which vector instructions
// share: so boxes are padded to whole k-steps on the way into LDS, and the
// loop is products, LDS reads and one address add a tile.
// TX = 16 amortises the halo (2x at K = 8) once a grid has enough lines;
// TX = 4 gives a 16 x 16 grid 64 workgroups instead of 16.
constexpr int kOffsets = 9;  // offsets per LDS fill: 21 KB at p = 12

template <int P, int AXIS>
struct AxisShape {
  static constexpr int kSteps = (P + 3) / 4, kP4 = 4 * kSteps;
  // LDS: AXIS 0 [k padded][b], AXIS 1 [m1][k padded + 1]: an odd stride puts
  // the 16 columns of a fragment read into different banks
  static constexpr int kRow = kP4 + 1;
  static __host__ __device__ int lds_len(int q) { return AXIS == 0 ? kP4 * P : q * kRow; }
  static __host__ __device__ size_t lds_bytes(int tx, int no, int q) {
    return (size_t(no) * kSteps * 64 + size_t(tx + no - 1) * lds_len(q)) * sizeof(float);
  }
};

// NT: tiles per wave, without branches around the products (with them the
// accumulators went through register copies at every product, twice the
// time).
template <int P, int AXIS, int TX, int NT>
__global__ __launch_bounds__(256) void fgt_axis_kernel(const float *__restrict__ in, int depth, int q, int K,
                                                       const float *__restrict__ T, float *__restrict__ out) {
  using S = AxisShape<P, AXIS>;
  constexpr int KS = S::kSteps, P4 = S::kP4;
  extern __shared__ __align__(16) float lds[];
  const int side = 1 << depth;
  const int len = AXIS == 0 ? P * P : q * P;  // floats per box
  const int plen = S::lds_len(q);             // floats per box in LDS
  const int ncol = AXIS == 0 ? P : q;         // columns per box
  constexpr int cstride = AXIS == 0 ? 1 : S::kRow, kstride = AXIS == 0 ? P : 1;
  const int nfill = min(kOffsets, 2 * K + 1);
  float *sT = lds;
  float *sB = lds + nfill * KS * 64;
  const int segs = (side + TX - 1) / TX;
  const int line = int(blockIdx.x) / segs, x0 = (int(blockIdx.x) % segs) * TX;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, kq = lane >> 4;
  // this wave's tiles wave, wave + 4, ...: each lane's column
  typedef float f4 __attribute__((ext_vector_type(4)));
  f4 acc[NT];
  int base[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    acc[i] = f4{0.f, 0.f, 0.f, 0.f};
    const int c = min((wave + 4 * i) * 16 + (lane & 15), TX * ncol - 1);
    base[i] = (c / ncol) * plen + (c % ncol) * cstride + kq * kstride;
  }

  if (P4 != P) {  // the padding stays zero
    for (int e = threadIdx.x; e < (TX + nfill - 1) * plen; e += 256) sB[e] = 0.f;
  }
  // A fill: kOffsets offsets' fragments and the boxes they reach, NB boxes a
  // wave.  Its loads are all under way at once, and while the fill before is
  // multiplied: with two boxes at a time 76 us an axis at depth 8, p = 12, now
  // 66 and 75; 11 and 7 us at depth 4, p = 9, now 5.4 and 5.9.
  constexpr int NB = (TX + kOffsets + 2) / 4, NV = (kMaxQ * P + 63) / 64, NTV = (kOffsets * KS + 3) / 4;
  float v[NB][NV], tv[NTV];
  const auto load = [&](int o0) {
    const int no = min(kOffsets, K - o0 + 1);
#pragma unroll
    for (int i = 0; i < NTV; ++i) {
      const int e = threadIdx.x + i * 256;
      tv[i] = e < no * KS * 64 ? T[int64_t(o0 + K) * KS * 64 + e] : 0.f;
    }
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const int j = wave + 4 * n, x = x0 + o0 + j;
      const bool ok = j < TX + no - 1 && x >= 0 && x < side;
      const int64_t box = AXIS == 0 ? int64_t(morton2(uint32_t(ok ? x : 0), uint32_t(line)))
                                    : int64_t(line) * side + (ok ? x : 0);
      const float *src = in + box * len;
#pragma unroll
      for (int i = 0; i < NV; ++i) v[n][i] = ok && i * 64 + lane < len ? src[i * 64 + lane] : 0.f;
    }
  };
  load(-K);
  for (int o0 = -K; o0 <= K; o0 += kOffsets) {
    const int no = min(kOffsets, K - o0 + 1);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NTV; ++i) {
      const int e = threadIdx.x + i * 256;
      if (e < no * KS * 64) sT[e] = tv[i];
    }
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const int j = wave + 4 * n;
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int w = i * 64 + lane;
        if (j < TX + no - 1 && w < len) sB[j * plen + (AXIS == 0 ? w : (w / P) * S::kRow + w % P)] = v[n][i];
      }
    }
    if (o0 + kOffsets <= K) load(o0 + kOffsets);
    __syncthreads();
    const float *tp = sT + lane, *bp = sB;
    for (int o = 0; o < no; ++o, tp += KS * 64, bp += plen) {
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const float t = tp[s * 64];
#pragma unroll
        for (int i = 0; i < NT; ++i)
          acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(t, bp[base[i] + s * 4 * kstride], acc[i], 0, 0, 0);
      }
    }
  }
  // D: row m = 4 (lane / 16) + e of register e, column lane % 16
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const int col = (wave + 4 * i) * 16 + (lane & 15);
    const int x = x0 + col / ncol, c = col % ncol;
    if (col >= TX * ncol || x >= side) continue;
    float *o = AXIS == 0 ? out + (int64_t(x) * side + line) * q * P + c
                         : out + int64_t(morton2(uint32_t(line), uint32_t(x))) * q * q + c;
    const int rs = AXIS == 0 ? P : q;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int m = 4 * kq + e;
      if (m < q) o[m * rs] = acc[i][e];
    }
  }
}

// sum_{m2} u2^m2 sum_{m1} C[m2][m1] u1^m1
template <int Q>
__device__ __forceinline__ float horner2(const float *__restrict__ C, float u1, float u2) {
  float acc = 0.f;
#pragma unroll
  for (int m2 = Q - 1; m2 >= 0; --m2) {
    float v = C[m2 * Q + Q - 1];
#pragma unroll
    for (int m1 = Q - 2; m1 >= 0; --m1) v = fmaf(v, u1, C[m2 * Q + m1]);
    acc = fmaf(acc, u2, v);
  }
  return acc;
}

// One target per lane.  The first boxes of a wave are taken one at a time
// with wave-uniform (scalar-loaded) coefficients; targets sorted by box leave
// nothing after that.  Lanes left after kUniformBoxes boxes (unsorted
// targets) read their own box's coefficients: q^2 / 4 gathered lines cost a
// wave about as much as 6 uniform boxes.  Targets outside the unit square
// raise `outside` and are left to fgt_eval_outside_kernel.  With a place the
// result goes there directly: 4-byte writes in random order are what bounds
// the kernel then (6.5e6 targets: 133 us, against 66 in order and 100 for a
// scatter afterwards).
constexpr int kUniformBoxes = 6;

template <int Q>
__global__ __launch_bounds__(256) void fgt_taylor_eval_kernel(const float2 *__restrict__ txy, int64_t nt, int depth,
                                                              const float *__restrict__ C,
                                                              const int32_t *__restrict__ place, float *__restrict__ G,
                                                              uint32_t *__restrict__ outside) {
  const int64_t t0 = (xcd_block() * 4 + (threadIdx.x >> 6)) * 64;
  if (t0 >= nt) return;  // whole wave
  const int64_t t = t0 + (threadIdx.x & 63);
  const bool act = t < nt;
  const float2 y = txy[act ? t : t0];  // idle lanes follow lane 0's target
  const int64_t to = act && place ? place[t] : t;
  const float fs = float(1 << depth);
  const int bx = clamped_box(y.x, fs), by = clamped_box(y.y, fs);
  const float u1 = 2.f * (y.x * fs - (float(bx) + 0.5f)), u2 = 2.f * (y.y * fs - (float(by) + 0.5f));
  const bool in = y.x >= 0.f && y.x <= 1.f && y.y >= 0.f && y.y <= 1.f;
  if (__ballot(!in) != 0ull && (threadIdx.x & 63) == 0) atomicOr(outside, 1u);
  const uint32_t key = morton2(uint32_t(bx), uint32_t(by));
  float acc = 0.f;
  uint64_t left = __ballot(1);
  for (int i = 0; i < kUniformBoxes && left; ++i) {
    const uint32_t k = __builtin_amdgcn_readfirstlane(__shfl(key, __ffsll(static_cast<long long>(left)) - 1));
    const float v = horner2<Q>(C + int64_t(k) * (Q * Q), u1, u2);
    acc = key == k ? v : acc;
    left &= ~__ballot(key == k);
  }
  if ((left >> (threadIdx.x & 63)) & 1) acc = horner2<Q>(C + int64_t(key) * (Q * Q), u1, u2);
  if (act) G[to] = acc;
}

// Targets outside the unit square (the polynomial holds inside the box only):
// the direct sum, for the waves that have one.  Returns at once when no
// target raised the flag.
template <int P>
__global__ __launch_bounds__(256) void fgt_eval_outside_kernel(const float2 *__restrict__ txy, int64_t nt, int depth,
                                                               float inv_s, int K, const float *__restrict__ A,
                                                               const uint32_t *__restrict__ outside,
                                                               const int32_t *__restrict__ place,
                                                               float *__restrict__ G) {
  if (*outside == 0u) return;
  const int lane = threadIdx.x & 63;
  const int64_t step = int64_t(gridDim.x) * 256;
  for (int64_t t0 = (int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6)) * 64; t0 < nt; t0 += step) {
    const int64_t t = t0 + lane;
    float2 y = txy[t < nt ? t : t0];
    const bool need = t < nt && !(y.x >= 0.f && y.x <= 1.f && y.y >= 0.f && y.y <= 1.f);
    const uint64_t mask = __ballot(need);
    if (mask == 0ull) continue;
    const int first = __ffsll(static_cast<long long>(mask)) - 1;
    const float fx = __shfl(y.x, first), fy = __shfl(y.y, first);
    if (!need) y = make_float2(fx, fy);  // the other lanes follow the first such target
    const float acc = eval_wave<P>(y, depth, inv_s, K, A);
    if (need) G[place ? place[t] : t] = acc;
  }
}

inline unsigned blocks_of(int64_t work) { return unsigned((work + 255) / 256); }

template <int P>
void launch_coeffs_p(const float *xy, const float *q, const int32_t *ls, int depth, double scale, float *A,
                     hipStream_t s) {
  const int64_t nbox = int64_t(1) << (2 * depth);
  const float2 *x = reinterpret_cast<const float2 *>(xy);
#define LAUNCH(G) \
  hipLaunchKernelGGL((fgt_coeffs_kernel<P, G>), dim3(unsigned((nbox / G + 3) / 4)), dim3(256), 0, s, x, q, ls, depth, scale, A)
  if (depth < kThreadsFrom) {
    LAUNCH(1);
    return;
  }
  hipLaunchKernelGGL(fgt_coeffs_few_kernel<P>, dim3(blocks_of(nbox * P)), dim3(256), 0, s, x, q, ls, depth, scale, A);
  if (depth == 8) LAUNCH(4);
  else if (depth <= 10) LAUNCH(16);
  else LAUNCH(64);
#undef LAUNCH
}

template <int P>
void launch_eval_p(const float *txy, int64_t nt, int depth, float inv_s, int K, const float *A, const int32_t *place,
                   float *G, hipStream_t s) {
  hipLaunchKernelGGL(fgt_eval_kernel<P>, dim3(blocks_of(nt)), dim3(256), 0, s,
                     reinterpret_cast<const float2 *>(txy), nt, depth, inv_s, K, A, place, G);
}

// Order of the Taylor path (0: 16 terms are not enough).  any: for an A that
// need not fall off as the coefficients do.  The remainder of h_a is then held
// against Cramer's bound of h_a itself, as tau_a = sum_{m>=q} (r/2)^m/m!
// 2^(m/2) sqrt((a+m)!/a!), largest at a = p - 1, and that of a product of two
// is at most tau (2 + tau) of their bounds: 2^-23 at most, less than the
// direct sum's own rounding (4e-7 to 3e-6 of the largest |G|; with the
// coefficients' order an A of equal entries came out 7.8e-6 off for 1.0e-6
// directly at r = 1, p = 12).
int taylor_order(double r, int p, bool any) {
  constexpr int kLast = 40;  // terms past it are far below the rest
  struct Bounds {
    double e[kLast + FGT2D_MAX_P];  // 2^(n/2) sqrt(n!)
    Bounds() {
      for (int n = 0; n < kLast + FGT2D_MAX_P; ++n) e[n] = std::exp2(0.5 * n) * std::sqrt(std::tgamma(double(n) + 1.0));
    }
  };
  static const Bounds bounds;  // formed once: its gamma functions took 45 us of a call
  const double *e = bounds.e;
  double t[kLast + 1] = {1.0};  // (r/2)^m / m!
  for (int m = 1; m <= kLast; ++m) t[m] = t[m - 1] * (0.5 * r / double(m));
  double rem = 0.0, tau = 0.0;
  int q = 0;
  for (int m = kLast; m >= 4; --m) {  // remainder of order m, smallest terms first
    double row = 0.0;
    for (int a = 0; a < p; ++a) row += t[a] * e[a + m];
    rem += 1.0865 * t[m] * row;
    tau += t[m] * (e[p - 1 + m] / e[p - 1]);
    if (m > kMaxQ || (m & 1)) continue;
    if (!(rem <= 0x1p-25) || (any && !(tau * (2.0 + tau) <= 0x1p-23))) break;
    q = m;
  }
  return q;
}

// Order q of the Taylor path for a call, 0 where the direct path is the
// better one, by estimated microseconds.  The direct path does about
// (2K+1)^2 (p^2 + 4p) multiply-adds a target, and takes at least one wave's
// time of them, on as many boxes as the grid has.  The Taylor path has five
// launches, (2K+1) matrix products of 16 p4 (p + q) a box (p4: p rounded up
// to 4) and q^2 a target.  Rates measured at 65536 boxes, p = 12, K = 8:
// 8400 us directly; 150 us of matrix products and 64 us at the targets.  Of
// 1126 calls timed on both paths, 1 to 2.6e6 targets, depths 2 to 8, p 2 to 16,
// K 1 to 16, sorted and not, those that take the Taylor path are all
// faster by it; without the grid's limit 60 on 16 boxes were not (19 us
// directly, 32 by the polynomial, K = 3).  The estimate of the direct path is
// low where a wave's targets lie in many boxes: such calls (65536 targets in
// as many boxes: 7400 us, 160) may still take it.
int taylor_q(int64_t nt, int depth, int p, float sigma, int K, bool any) {
  const double r = std::ldexp(1.0, -depth) / (std::sqrt(2.0) * double(sigma));
  if (!(r <= 4.0)) return 0;
  const int q = taylor_order(r, p, any);
  if (q == 0) return 0;
  const double w = 2.0 * K + 1.0, boxes = std::ldexp(1.0, 2 * depth), p4 = double((p + 3) / 4 * 4);
  const double side = std::ldexp(1.0, depth), reach = std::min(w, side);
  const double box = double(p) * p + 4.0 * p;  // multiply-adds of a direct target in one box
  const double direct = 2.0 + std::max(reach * reach * box * 4.6 / 2400.0, double(nt) * w * w * box / 40e6);
  const double taylor = 10.4 + 0.1 * p + boxes * w * 16.0 * p4 * (p + q) / 30e6 + double(nt) * q * q / 13e6;
  return taylor < direct ? q : 0;
}

struct TaylorWs {
  size_t table, w, c, flag, bytes;  // byte offsets, total
};

TaylorWs taylor_ws(int depth, int p, int q, int K) {
  const auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  const size_t nbox = size_t(1) << (2 * depth), ks = size_t(p + 3) / 4;
  TaylorWs l;
  l.table = 0;
  l.w = up((2 * size_t(K) + 1) * ks * 64 * sizeof(float));
  l.c = l.w + up(nbox * size_t(q) * size_t(p) * sizeof(float));
  l.flag = l.c + up(nbox * size_t(q) * size_t(q) * sizeof(float));
  l.bytes = l.flag + 256;
  return l;
}

// Boxes of one workgroup: 16 from 64 lines on, 4 below (see fgt_axis_kernel).
template <int P, int AXIS>
void launch_axis(const float *in, int depth, int q, int K, const float *T, float *out, hipStream_t s) {
  const int side = 1 << depth;
  const int tx = depth >= 6 ? 16 : 4;
  const unsigned grid = unsigned(side) * unsigned((side + tx - 1) / tx);
  const size_t lds = AxisShape<P, AXIS>::lds_bytes(tx, std::min(kOffsets, 2 * K + 1), q);
  const dim3 g(grid), bl(256);
#define LAUNCH(TX, NT) hipLaunchKernelGGL((fgt_axis_kernel<P, AXIS, TX, NT>), g, bl, lds, s, in, depth, q, K, T, out)
  if (tx == 4) LAUNCH(4, 1);
  else if constexpr (AXIS == 0) LAUNCH(16, (P + 3) / 4);
  else if (q <= 4) LAUNCH(16, 1);
  else if (q <= 8) LAUNCH(16, 2);
  else if (q <= 12) LAUNCH(16, 3);
  else LAUNCH(16, 4);
#undef LAUNCH
}

template <int P>
void launch_axes_p(const float *A, int depth, int q, int K, const float *T, float *W, float *C, hipStream_t s) {
  launch_axis<P, 0>(A, depth, q, K, T, W, s);
  launch_axis<P, 1>(W, depth, q, K, T, C, s);
}

template <int P>
void launch_outside_p(const float *txy, int64_t nt, int depth, float inv_s, int K, const float *A,
                      const uint32_t *outside, const int32_t *place, float *G, hipStream_t s) {
  const int64_t nb = (nt + 255) / 256;
  hipLaunchKernelGGL(fgt_eval_outside_kernel<P>, dim3(unsigned(nb < 2048 ? nb : 2048)), dim3(256), 0, s,
                     reinterpret_cast<const float2 *>(txy), nt, depth, inv_s, K, A, outside, place, G);
}

#define FGT_FOR_EACH_P(X) \
  X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)

int check_fgt_common(const char *fn, int depth, int p, float sigma) {
  if (depth < 0 || depth > kMaxDepth) return set_error(FMM2D_EDEPTH, "%s: depth %d outside 0..%d", fn, depth, kMaxDepth);
  if (p < 1 || p > FGT2D_MAX_P) return set_error(FMM2D_EUNSUPPORTED_P, "%s: p = %d outside 1..%d", fn, p, FGT2D_MAX_P);
  if (!(sigma > 0.f) || !std::isfinite(sigma)) return set_error(FMM2D_EINVAL, "%s: sigma must be finite and > 0", fn);
  return FMM2D_OK;
}

}  // namespace

}  // namespace fmm2d

using namespace fmm2d;

extern "C" {

int fgt2d_hermite_coeffs(const float *xy_sorted, const float *q_sorted, const int32_t *leaf_start, int depth, int p,
                         float sigma, float *A, hipStream_t stream) {
  const char *fn = "fgt2d_hermite_coeffs";
  clear_error();
  const int rc = check_fgt_common(fn, depth, p, sigma);
  if (rc != FMM2D_OK) return rc;
  if (!xy_sorted || !q_sorted || !leaf_start || !A) return set_error(FMM2D_EINVAL, "%s: NULL pointer", fn);
  const double scale = 1.0 / (std::sqrt(2.0) * double(sigma));
  switch (p) {
#define X(P_) \
  case P_: launch_coeffs_p<P_>(xy_sorted, q_sorted, leaf_start, depth, scale, A, stream); break;
    FGT_FOR_EACH_P(X)
#undef X
  }
  return check_launch(fn);
}

static int check_eval(const char *fn, const float *txy, int64_t nt, int depth, int p, float sigma, int K,
                      const float *A, const float *G) {
  const int rc = check_fgt_common(fn, depth, p, sigma);
  if (rc != FMM2D_OK) return rc;
  if (nt < 0 || nt >= (int64_t(1) << 31)) return set_error(FMM2D_EINVAL, "%s: nt out of range", fn);
  if (K < 0 || K >= (1 << depth))
    return set_error(FMM2D_EINVAL, "%s: K = %d outside 0..%d", fn, K, (1 << depth) - 1);
  if (!A) return set_error(FMM2D_EINVAL, "%s: A is NULL", fn);
  if (nt > 0 && (!txy || !G)) return set_error(FMM2D_EINVAL, "%s: NULL pointer", fn);
  return FMM2D_OK;
}

static int eval_direct(const char *fn, const float *txy, int64_t nt, int depth, int p, float sigma, int K,
                       const float *A, const int32_t *place, float *G, hipStream_t stream) {
  const float inv_s = float(1.0 / (std::sqrt(2.0) * double(sigma)));
  switch (p) {
#define X(P_) \
  case P_: launch_eval_p<P_>(txy, nt, depth, inv_s, K, A, place, G, stream); break;
    FGT_FOR_EACH_P(X)
#undef X
  }
  return check_launch(fn);
}

int fgt2d_hermite_eval(const float *txy, int64_t nt, int depth, int p, float sigma, int K, const float *A, float *G,
                       hipStream_t stream) {
  const char *fn = "fgt2d_hermite_eval";
  clear_error();
  const int rc = check_eval(fn, txy, nt, depth, p, sigma, K, A, G);
  if (rc != FMM2D_OK || nt == 0) return rc;
  return eval_direct(fn, txy, nt, depth, p, sigma, K, A, nullptr, G, stream);
}

static size_t eval_workspace(const char *fn, int64_t nt, int depth, int p, float sigma, int K, bool any) {
  clear_error();
  if (check_fgt_common(fn, depth, p, sigma) != FMM2D_OK) return 0;
  if (nt <= 0 || nt >= (int64_t(1) << 31) || K < 0 || K >= (1 << depth)) return 0;
  const int q = taylor_q(nt, depth, p, sigma, K, any);
  return q ? taylor_ws(depth, p, q, K).bytes : 0;
}

size_t fgt2d_hermite_eval_workspace(int64_t nt, int depth, int p, float sigma, int K) {
  return eval_workspace("fgt2d_hermite_eval_workspace", nt, depth, p, sigma, K, false);
}

size_t fgt2d_hermite_eval_any_workspace(int64_t nt, int depth, int p, float sigma, int K) {
  return eval_workspace("fgt2d_hermite_eval_any_workspace", nt, depth, p, sigma, K, true);
}

static int eval_ws(const char *fn, const float *txy, int64_t nt, int depth, int p, float sigma, int K, bool any,
                   const float *A, const int32_t *place, float *G, void *ws, size_t ws_bytes, hipStream_t stream) {
  const int q = taylor_q(nt, depth, p, sigma, K, any);
  if (q == 0 || ws == nullptr) return eval_direct(fn, txy, nt, depth, p, sigma, K, A, place, G, stream);
  const TaylorWs l = taylor_ws(depth, p, q, K);
  if (ws_bytes < l.bytes)
    return set_error(FMM2D_EWORKSPACE, "%s: workspace of %zu bytes, %zu needed", fn, ws_bytes, l.bytes);
  if (reinterpret_cast<uintptr_t>(ws) % 16 != 0) return set_error(FMM2D_EINVAL, "%s: ws not 16-byte aligned", fn);
  char *base = static_cast<char *>(ws);
  float *T = reinterpret_cast<float *>(base + l.table);
  float *W = reinterpret_cast<float *>(base + l.w);
  float *C = reinterpret_cast<float *>(base + l.c);
  uint32_t *outside = reinterpret_cast<uint32_t *>(base + l.flag);
  const double r = std::ldexp(1.0, -depth) / (std::sqrt(2.0) * double(sigma));
  const int ks = (p + 3) / 4;
  hipLaunchKernelGGL(fgt_taylor_table_kernel, dim3(unsigned(2 * K + 1)), dim3(256), 0, stream, p, ks, K, r, T, outside);
  switch (p) {
#define X(P_) \
  case P_: launch_axes_p<P_>(A, depth, q, K, T, W, C, stream); break;
    FGT_FOR_EACH_P(X)
#undef X
  }
  const float2 *t = reinterpret_cast<const float2 *>(txy);
  const dim3 grid(blocks_of(nt)), block(256);
  switch (q) {
#define X(Q_) \
  case Q_: hipLaunchKernelGGL(fgt_taylor_eval_kernel<Q_>, grid, block, 0, stream, t, nt, depth, C, place, G, outside); break;
    X(4) X(6) X(8) X(10) X(12) X(14) X(16)
#undef X
  }
  const float inv_s = float(1.0 / (std::sqrt(2.0) * double(sigma)));
  switch (p) {
#define X(P_) \
  case P_: launch_outside_p<P_>(txy, nt, depth, inv_s, K, A, outside, place, G, stream); break;
    FGT_FOR_EACH_P(X)
#undef X
  }
  return check_launch(fn);
}

int fgt2d_hermite_eval_ws(const float *txy, int64_t nt, int depth, int p, float sigma, int K, const float *A, float *G,
                          void *ws, size_t ws_bytes, hipStream_t stream) {
  const char *fn = "fgt2d_hermite_eval_ws";
  clear_error();
  const int rc = check_eval(fn, txy, nt, depth, p, sigma, K, A, G);
  if (rc != FMM2D_OK || nt == 0) return rc;
  return eval_ws(fn, txy, nt, depth, p, sigma, K, false, A, nullptr, G, ws, ws_bytes, stream);
}

int fgt2d_hermite_eval_place(const float *txy, int64_t nt, int depth, int p, float sigma, int K, const float *A,
                             const int32_t *place, float *G, void *ws, size_t ws_bytes, hipStream_t stream) {
  const char *fn = "fgt2d_hermite_eval_place";
  clear_error();
  const int rc = check_eval(fn, txy, nt, depth, p, sigma, K, A, G);
  if (rc != FMM2D_OK) return rc;
  if (nt == 0) return set_error(FMM2D_EINVAL, "%s: no targets", fn);
  if (!place) return set_error(FMM2D_EINVAL, "%s: place is NULL", fn);
  return eval_ws(fn, txy, nt, depth, p, sigma, K, false, A, place, G, ws, ws_bytes, stream);
}

int fgt2d_hermite_eval_any(const float *txy, int64_t nt, int depth, int p, float sigma, int K, const float *A,
                           const int32_t *place, float *G, void *ws, size_t ws_bytes, hipStream_t stream) {
  const char *fn = "fgt2d_hermite_eval_any";
  clear_error();
  const int rc = check_eval(fn, txy, nt, depth, p, sigma, K, A, G);
  if (rc != FMM2D_OK || nt == 0) return rc;
  return eval_ws(fn, txy, nt, depth, p, sigma, K, true, A, place, G, ws, ws_bytes, stream);
}

}  // extern "C"
