// Whole Lawson solves of small 2D problems in one workgroup (the time loop on the
// device). For n1, n2 <= 64 a step is ~1 MFLOP: launched kernel by kernel it is bound
// by launch latency, so one workgroup keeps the state and the stage vectors in LDS and
// each lane's factor operands and stencil coefficients in registers for the whole solve,
// and runs every step -- the remainder stencil (eq. (eq:nonlin), flux form, the same
// arithmetic as the grid kernel), the two mode products (FP64 MFMA) and the stage
// combinations -- with workgroup barriers between the phases.
//
// One CU bounds a solve, by its matrix cores and its LDS. Per step and vector the products of
// the exponentials themselves hold each SIMD for 2 x 4096 clocks. Where both axes are
// centrosymmetric (see fold_factor) they halve: the vector is kept folded along both axes as
// four 32 x 32 quadrants (even/odd mirror combinations of rows and columns), on which every
// product is block diagonal. A thread owns two rows of mirror quadruples for the whole solve:
// state and face coefficients stay in registers, and folding and unfolding are sums within the
// thread. Eight waves of 256 registers; a wave has a 16 x 32 strip of every product, so that an
// operand read from LDS serves two matrix instructions. Sixteen waves of 128 registers took
// 4.65 (LE) and 11.5 us (Lawson2b, spilling) per step at 63 x 63 against 4.6 and 8.8.
// Measured per step at 63 x 63: folded 4.6 us (LE) and 8.8 us (Lawson2b), plain 6.4 and 13.1 us;
// one 16 x 16 tile a wave with every factor plain took 7.3 and 13.5 us.
#include <cfloat>

#include "mm_internal.h"

namespace mm {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int NS = 64;              // largest n1, n2
constexpr int THS = 512;
constexpr int QH = NS / 2;          // folded positions per axis, quadrant edge
constexpr int QP = NS + 2;          // row pitch: 16 rows of 2 consecutive values fill all banks once
constexpr int QB = NS * QP;         // one vector
constexpr int QR = (NS + 2) * QP;   // one grid with its zero border
constexpr int PS = NS + 1;          // plain form: row pitch in doubles, pitch of a
constexpr int PA = NS + 2;

// the wave's two 16 x 16 output tiles (side by side) of the 64 x 64 grid
__device__ __forceinline__ int tile_row() { return (threadIdx.x >> 7) * 16; }
__device__ __forceinline__ int tile_col() { return ((threadIdx.x >> 6) & 1) * QH; }

// ------------------------------------------------------------------------------------
// Folded form.

// This lane's operands of the folded products along one axis of n points: row c = 16 j + lane%16
// of Es (waves of the left half, tile_col() = 0) or Ed (right half), f[j][kk] =
// E[c][4 kk + lane/16], zero beyond the folded length.
struct FoldFrags {
  double f[2][8];

  __device__ __forceinline__ void load(const double* __restrict__ Ef, int n) {
    const int lane = threadIdx.x & 63, lg = lane >> 4, lr = lane & 15, h = (threadIdx.x >> 6) & 1;
    const int m = n - n / 2, ld = fold_ld(n);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        const int c = 16 * j + lr, k = 4 * kk + lg;
        f[j][kk] = (c < m && k < m) ? Ef[(c + h * m) * ld + k] : 0.0;
      }
  }
};

// Y[c][r] <- sum_k X[r][k] F[c][k] for NV vectors, transposed on the way out: two in turn
// contract both axes and restore the order, and every read and write of the pitch-QP rows is free
// of bank conflicts. f: folded length of
// the contracted axis.
template <int NV>
__device__ __forceinline__ void fold_product(double* const (&Y)[NV], const double* const (&X)[NV], const FoldFrags& F,
                                             int f) {
  const int lane = threadIdx.x & 63, lg = lane >> 4, lr = lane & 15, wm = tile_row(), wn = tile_col();
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    double x[8];
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) x[kk] = X[v][(wm + lr) * QP + wn + 4 * kk + lg];
    d4 acc[2] = {d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}};
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      if (4 * kk >= f) continue;   // (uniform)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[kk], F.f[j][kk], acc[j], 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int t = 0; t < 4; ++t) Y[v][(wn + 16 * j + lr) * QP + wm + 4 * t + lg] = acc[j][t];
  }
  __syncthreads();
}

// A thread's points: rows r0 = 2 (tid / 32) and r0 + 1 (s = 0, 1), each of them a quadruple of
// mirror points: point m = 4 s + 2 b + a at column q1 or (a) n1-1-q1 and row r0 + s or (b)
// n2-1-r0-s. On the middle line of an odd axis mirrored points coincide: both hold the same
// value, and folding counts it once.
struct Points {
  int at[8];                      // positions in the bordered grid
  double cxp[8], cxm[8], cy[4][3];   // face coefficients (mean of a, less the extracted part); cy of the
                                     // pair 2 b + a: outside of s = 0, between, outside of s = 1
  bool on[2], mid1, mid2[2];
  int fold_at;                    // position of row r0's even-even value in a folded vector

  __device__ __forceinline__ void init(const SmallArgs& p) {
    const int n1 = p.n1, n2 = p.n2, q1 = threadIdx.x & (QH - 1), r0 = 2 * (threadIdx.x / QH);
    fold_at = r0 * QP + q1;
    mid1 = 2 * q1 == n1 - 1;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      on[s] = 2 * q1 < n1 && 2 * (r0 + s) < n2;
      mid2[s] = 2 * (r0 + s) == n2 - 1;
    }
    const double la = p.lam_amax;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      // (without points: at the first one)
      const bool o = on[m >> 2];
      const int r = r0 + (m >> 2), i1 = !o ? 0 : (m & 1) ? n1 - 1 - q1 : q1, i2 = !o ? 0 : (m & 2) ? n2 - 1 - r : r;
      at[m] = (i2 + 1) * QP + i1 + 1;
      const double* a = p.a + (int64_t)(i2 + 1) * (n1 + 2) + i1 + 1;
      const double ac = a[0];
      cxp[m] = 0.5 * (ac + a[1]) - la;
      cxm[m] = 0.5 * (ac + a[-1]) - la;
      const double yp = 0.5 * (ac + a[n1 + 2]) - la, ym = 0.5 * (ac + a[-(n1 + 2)]) - la;
      // s = 0 of a mirrored pair lies above s = 1
      if (m < 4) {
        cy[m & 3][0] = (m & 2) ? yp : ym;
        cy[m & 3][1] = (m & 2) ? ym : yp;
      } else {
        cy[m & 3][2] = (m & 2) ? ym : yp;
      }
    }
  }

  // g at the pair k = 2 b + a (points k and 4 + k) of the grid U, whose values there are u
  __device__ __forceinline__ void g(double (&out)[2], const SmallArgs& p, const double* U, int k, double u0,
                                    double u1) const {
    const double *x0 = U + at[k], *x1 = U + at[4 + k];
    const int step = (k & 2) ? -QP : QP;   // from s = 0 to s = 1
    const double v0 = x0[-step], v3 = x1[step];
    // (a pair cut by the middle of the grid has its neighbour in the mirrored half)
    const double v2 = on[1] ? u1 : x0[step];
    const double xm0 = x0[-1], xp0 = x0[1], xm1 = x1[-1], xp1 = x1[1];
    const double sg = (k & 2) ? -1.0 : 1.0;
    out[0] = (cxp[k] * (xp0 - u0) - cxm[k] * (u0 - xm0)) * p.ih2[0] + p.cadv[0] * (xp0 - xm0);
    out[0] += (cy[k][1] * (v2 - u0) - cy[k][0] * (u0 - v0)) * p.ih2[1] + sg * p.cadv[1] * (v2 - v0);
    out[0] += p.r0 + u0 * (p.r1 + u0 * (p.r2 + u0 * p.r3));
    out[1] = (cxp[4 + k] * (xp1 - u1) - cxm[4 + k] * (u1 - xm1)) * p.ih2[0] + p.cadv[0] * (xp1 - xm1);
    out[1] += (cy[k][2] * (v3 - u1) - cy[k][1] * (u1 - u0)) * p.ih2[1] + sg * p.cadv[1] * (v3 - u0);
    out[1] += p.r0 + u1 * (p.r1 + u1 * (p.r2 + u1 * p.r3));
  }

  // grid values into U, and the border beyond n1 and n2 (which a vector in the same buffer
  // overwrites) back to zero
  __device__ __forceinline__ void put(double* U, const double (&u)[8], int n1, int n2) const {
#pragma unroll
    for (int s = 0; s < 2; ++s)
      if (on[s]) {
#pragma unroll
        for (int k = 0; k < 4; ++k) U[at[4 * s + k]] = u[4 * s + k];
        if ((threadIdx.x & (QH - 1)) == 0) U[at[4 * s] + n1] = U[at[4 * s + 2] + n1] = 0.0;
      }
    if (on[0] && threadIdx.x / QH == 0) U[at[0] + n2 * QP] = U[at[1] + n2 * QP] = 0.0;
  }

  // v folded along both axes into V
  __device__ __forceinline__ void fold(double* V, const double (&v)[8]) const {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const double* w = v + 4 * s;
      const double w0 = on[s] ? w[0] : 0.0, w1 = on[s] && !mid1 ? w[1] : 0.0, w2 = on[s] && !mid2[s] ? w[2] : 0.0,
                   w3 = on[s] && !mid1 && !mid2[s] ? w[3] : 0.0;
      const double s0 = w0 + w1, d0 = w0 - w1, s1 = w2 + w3, d1 = w2 - w3;
      double* x = V + fold_at + s * QP;
      x[0] = s0 + s1;
      x[QH] = d0 + d1;
      x[QH * QP] = s0 - s1;
      x[QH * QP + QH] = d0 - d1;
    }
  }

  // the grid values of the folded vector V
  __device__ __forceinline__ void unfold(double (&v)[8], const double* V) const {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      double* w = v + 4 * s;
      const double* x = V + fold_at + s * QP;
      const double ee = x[0], eo = x[QH], oe = x[QH * QP], oo = x[QH * QP + QH];
      const double e0 = ee + eo, e1 = ee - eo, o0 = oe + oo, o1 = oe - oo;
      w[0] = e0 + o0;
      w[1] = mid1 ? w[0] : e1 + o1;
      w[2] = mid2[s] ? w[0] : e0 - o0;
      w[3] = mid1 ? w[2] : mid2[s] ? w[1] : e1 - o1;
    }
  }

  __device__ __forceinline__ bool bad(const double (&u)[8]) const {
    bool b = false;
#pragma unroll
    for (int m = 0; m < 8; ++m) b |= on[m >> 2] && !(fabs(u[m]) <= DBL_MAX);
    return b;
  }
};

// LE (L2B = 0) or Lawson2b (L2B = 1), nsteps steps of u (global, n2 x n1) in place. Four (LE) or
// five barriers a step; Lawson2b's products use the buffers of the two grids, which are idle then.
template <int L2B>
__device__ __forceinline__ void lawson_small2d_fold(const SmallArgs& p, double* lds) {
  const int n1 = p.n1, n2 = p.n2, f1 = n1 - n1 / 2, f2 = n2 - n2 / 2;
  FoldFrags F1, F2;
  F1.load(p.Ef1, n1);
  F2.load(p.Ef2, n2);
  Points q;
  q.init(p);
  for (int e = threadIdx.x; e < 2 * QB + (L2B ? 2 : 1) * QR; e += THS) lds[e] = 0.0;
  __syncthreads();
  double u[8];
#pragma unroll
  for (int m = 0; m < 8; ++m) u[m] = p.u[(q.at[m] / QP - 1) * n1 + q.at[m] % QP - 1];
  q.put(lds + (L2B ? QR + 2 * QB : 0), u, n1, n2);
  __syncthreads();
  const double tau = p.tau;
  bool bad = false;
  for (int it = 0; it < p.nsteps; ++it) {
    // (opaque, so that the buffers' lane addresses are not all kept in registers over the loop)
    int z = 0;
    asm volatile("" : "+s"(z));
    // R1: grid (LE: the state; Lawson2b: the first stage); A, B: vectors; R2: Lawson2b's grid of
    // the state; S: the state's grid
    double *const R1 = lds + z, *const A = R1 + QR, *const B = A + QB, *const R2 = B + QB, *const S = L2B ? R2 : R1;
    double v[8], w[8];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      double g[2];
      q.g(g, p, S, k, u[k], u[4 + k]);
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        v[4 * s + k] = u[4 * s + k] + tau * g[s];
        w[4 * s + k] = u[4 * s + k] + 0.5 * tau * g[s];
      }
    }
    q.fold(A, v);
    if (L2B) q.fold(B, w);
    __syncthreads();
    if constexpr (L2B) {
      // U = e^{tau A} v, W = e^{tau A} w; u+ = W + tau/2 g(U)
      // (inside the grids' top and left borders, which stay zero)
      fold_product<2>({R1 + QP + 1, R2 + QP + 1}, {A, B}, F1, f1);
      fold_product<2>({A, B}, {R1 + QP + 1, R2 + QP + 1}, F2, f2);
      q.unfold(v, A);
      q.unfold(w, B);
      q.put(R1, v, n1, n2);
      __syncthreads();
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        double g[2];
        q.g(g, p, R1, k, v[k], v[4 + k]);
#pragma unroll
        for (int s = 0; s < 2; ++s) u[4 * s + k] = w[4 * s + k] + 0.5 * tau * g[s];
      }
    } else {
      // u+ = e^{tau A} v
      fold_product<1>({B}, {A}, F1, f1);
      fold_product<1>({A}, {B}, F2, f2);
      q.unfold(u, A);
    }
    bad |= q.bad(u);
    q.put(S, u, n1, n2);
    __syncthreads();
  }
#pragma unroll
  for (int m = 0; m < 8; ++m)
    if (q.on[m >> 2]) p.u[(q.at[m] / QP - 1) * n1 + q.at[m] % QP - 1] = u[m];
  if (bad && p.flag) p.flag[0] = 1;
}

// ------------------------------------------------------------------------------------
// Plain form: products of the exponentials themselves.

// g at interior point (i2, i1) from the LDS grid U (zero outside [0,n2) x [0,n1)) and
// the LDS copy of a ((n2+2) x (n1+2) nodes, pitch PA).
__device__ __forceinline__ double g_small(const SmallArgs& p, const double* U, const double* A, int i2, int i1) {
  const int n1 = p.n1, n2 = p.n2;
  const double uc = U[i2 * PS + i1];
  const double uxm = (i1 > 0) ? U[i2 * PS + i1 - 1] : 0.0;
  const double uxp = (i1 + 1 < n1) ? U[i2 * PS + i1 + 1] : 0.0;
  const double uym = (i2 > 0) ? U[(i2 - 1) * PS + i1] : 0.0;
  const double uyp = (i2 + 1 < n2) ? U[(i2 + 1) * PS + i1] : 0.0;
  const int ia = (i1 + 1) + PA * (i2 + 1);
  const double ac = A[ia], axm = A[ia - 1], axp = A[ia + 1], aym = A[ia - PA], ayp = A[ia + PA];
  const double la = p.lam_amax;
  double g = ((0.5 * (ac + axp) - la) * (uxp - uc) - (0.5 * (ac + axm) - la) * (uc - uxm)) * p.ih2[0] +
             p.cadv[0] * (uxp - uxm);
  g += ((0.5 * (ac + ayp) - la) * (uyp - uc) - (0.5 * (ac + aym) - la) * (uc - uym)) * p.ih2[1] +
       p.cadv[1] * (uyp - uym);
  g += p.r0 + uc * (p.r1 + uc * (p.r2 + uc * p.r3));
  return g;
}

// The factor operand of this lane for all 16 k-steps of a 64-long contraction (zero
// beyond n), loaded once per solve: f[kk] = E[r0 + lane%16][4 kk + lane/16].
struct Frags {
  double f[16];

  __device__ __forceinline__ void load(const double* __restrict__ E, int n, int r0) {
    const int lane = threadIdx.x & 63, lg = lane >> 4, lr = lane & 15;
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      const int r = r0 + lr, k = 4 * kk + lg;
      f[kk] = (r < n && k < n) ? E[r * n + k] : 0.0;
    }
  }
};

// Mode products of one workgroup on 64 x 64 LDS tiles (zero beyond n), factor operands
// from registers:
//   mode 1:  Y[i2][j1] <- sum_k X[i2][k] E1[j1][k]      (F = E1 rows j1 of this wave's two tiles)
//   mode 2:  Y[j2][i1] <- sum_k E2[j2][k] X[k][i1]      (F[0] = E2 rows j2 of this wave)
// Each wave computes its two 16 x 16 tiles into registers; with Y = X (IN_PLACE) a
// barrier before the write-back lets the product overwrite its own input. Returns whether a
// value of the lane is not finite.
template <int MODE, bool IN_PLACE>
__device__ __forceinline__ bool mode_product(double* Y, const double* X, const Frags* F, int m1, int m2) {
  const int lane = threadIdx.x & 63;
  const int wm = tile_row(), wn = tile_col();
  const int lg = lane >> 4, lr = lane & 15;
  d4 acc[2] = {d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}};
#pragma unroll
  for (int kk = 0; kk < 16; ++kk) {
    const int k = 4 * kk + lg;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const double av = (MODE == 1) ? X[(wm + lr) * PS + k] : F[0].f[kk];          // X[i2][k] or E2[j2][k]
      const double bv = (MODE == 1) ? F[j].f[kk] : X[k * PS + wn + 16 * j + lr];   // E1[j1][k] or X[k][i1]
      acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc[j], 0, 0, 0);
    }
  }
  if (IN_PLACE) __syncthreads();   // every wave has read X
  bool bad = false;
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int r = wm + 4 * t + lg, c = wn + 16 * j + lr;
      const double y = (r < m2 && c < m1) ? acc[j][t] : 0.0;
      bad |= !(fabs(y) <= DBL_MAX);
      Y[r * PS + c] = y;
    }
  __syncthreads();
  return bad;
}

// LE (L2B = 0) or Lawson2b (L2B = 1), nsteps steps of u (global, n2 x n1) in place.
template <int L2B>
__device__ __forceinline__ void lawson_small2d_plain(const SmallArgs& p, double* lds) {
  double* const Us = lds;
  double* const As = Us + NS * PS;
  double* const V1 = As + PA * PA;
  double* const V2 = V1 + NS * PS;   // Lawson2b only
  const int n1 = p.n1, n2 = p.n2, tid = threadIdx.x;
  // factor operands for the whole solve: mode 1 uses E1 rows of the wave's columns, mode 2 E2
  // rows of the wave's rows
  Frags F1[2], F2[1];
  F1[0].load(p.E1, n1, tile_col());
  F1[1].load(p.E1, n1, tile_col() + 16);
  F2[0].load(p.E2, n2, tile_row());
  for (int e = tid; e < NS * PS; e += THS) {
    const int i2 = e / PS, i1 = e % PS;
    Us[e] = (i2 < n2 && i1 < n1) ? p.u[i2 * n1 + i1] : 0.0;
    V1[e] = 0.0;
    if (L2B) V2[e] = 0.0;
  }
  for (int e = tid; e < (n2 + 2) * (n1 + 2); e += THS) {
    const int j2 = e / (n1 + 2), j1 = e % (n1 + 2);
    As[j2 * PA + j1] = p.a[e];
  }
  __syncthreads();
  const double tau = p.tau;
  bool bad = false;
  // a thread's points: every THS-th in row-major order
  const int first2 = tid / n1, first1 = tid % n1, step2 = THS / n1, step1 = THS % n1;
  const auto advance = [&](int& i2, int& i1) {
    i2 += step2;
    i1 += step1;
    if (i1 >= n1) {
      i1 -= n1;
      ++i2;
    }
  };
  for (int it = 0; it < p.nsteps; ++it) {
    // first stage vectors: v1 = u + tau g(u) (LE and L2b), v2 = u + tau/2 g(u) (L2b)
    for (int i2 = first2, i1 = first1; i2 < n2; advance(i2, i1)) {
      const double g = g_small(p, Us, As, i2, i1);
      const double u = Us[i2 * PS + i1];
      V1[i2 * PS + i1] = u + tau * g;
      if (L2B) V2[i2 * PS + i1] = u + 0.5 * tau * g;
    }
    __syncthreads();
    mode_product<1, true>(V1, V1, F1, n1, n2);
    if (!L2B) {
      // u+ = e^{tau A} v1
      bad |= mode_product<2, false>(Us, V1, F2, n1, n2);
    } else {
      // U = e^{tau A} v1, W = e^{tau A} v2; u+ = W + tau/2 g(U)
      mode_product<2, true>(V1, V1, F2, n1, n2);
      mode_product<1, true>(V2, V2, F1, n1, n2);
      mode_product<2, true>(V2, V2, F2, n1, n2);
      for (int i2 = first2, i1 = first1; i2 < n2; advance(i2, i1)) {
        const double o = V2[i2 * PS + i1] + 0.5 * tau * g_small(p, V1, As, i2, i1);
        bad |= !(fabs(o) <= DBL_MAX);
        Us[i2 * PS + i1] = o;
      }
      __syncthreads();
    }
  }
  for (int i2 = first2, i1 = first1; i2 < n2; advance(i2, i1)) p.u[i2 * n1 + i1] = Us[i2 * PS + i1];
  if (bad && p.flag) p.flag[0] = 1;
}

}  // namespace

// One solve per workgroup: blockIdx.x selects the problem (its own sizes, factors,
// coefficients, step count and form). A single solve is launched the same way with one
// entry, so a problem's result does not depend on whether it ran alone or in a group.
template <int L2B>
__global__ __launch_bounds__(THS) void lawson_small2d_batch(SmallBatch b) {
  constexpr int kFold = 2 * QB + (L2B ? 2 : 1) * QR, kPlain = PA * PA + (L2B ? 3 : 2) * NS * PS;
  __shared__ double lds[kFold > kPlain ? kFold : kPlain];
  const SmallArgs& p = b.a[blockIdx.x];
  if (p.Ef1)
    lawson_small2d_fold<L2B>(p, lds);
  else
    lawson_small2d_plain<L2B>(p, lds);
}

bool small2d_fits(int d, int n1, int n2) { return d == 2 && n1 >= 1 && n2 >= 1 && n1 <= NS && n2 <= NS; }

hipError_t launch_lawson_small2d(const SmallArgs& a, bool l2b, hipStream_t s) {
  return launch_lawson_small2d_batch(&a, 1, l2b, s);
}

hipError_t launch_lawson_small2d_batch(const SmallArgs* a, int count, bool l2b, hipStream_t s) {
  if (count < 1 || count > kMaxSmallBatch) return hipErrorInvalidValue;
  SmallBatch b;
  for (int i = 0; i < count; ++i) {
    if (a[i].n1 < 1 || a[i].n2 < 1 || a[i].n1 > NS || a[i].n2 > NS || a[i].nsteps < 0 ||
        !a[i].Ef1 != !a[i].Ef2)
      return hipErrorInvalidValue;
    b.a[i] = a[i];
  }
  if (l2b)
    lawson_small2d_batch<1><<<count, THS, 0, s>>>(b);
  else
    lawson_small2d_batch<0><<<count, THS, 0, s>>>(b);
  return hipGetLastError();
}

}  // namespace mm
