// Functions of tau A in the folded sine basis (gfx950, FP64).
//
// On axes with zero Dirichlet data at both ends and no advection moved into A, A_mu is a
// symmetric Toeplitz tridiagonal with the orthogonal symmetric eigenvector matrix
// S_jk = sqrt(2/N) sin(j k pi / N), N = n + 1, j, k = 1..n, and the eigenvalues
// -4 lam a_max/h^2 sin^2(k pi / (2N)). A function of tau A = tau (A_1 (+) A_2 (+) A_3) -- an
// exponential, a phi function or a quadrature sum of exponentials -- is then S_3 S_2 S_1,
// a pointwise scaling and S_1 S_2 S_3: six mode products, however many exponentials the
// function sums (the quadrature of phi1 by q nodes: 3q products of exponentials).
// S is not centrosymmetric, but its odd columns (k = 1, 3, ..) are symmetric and its even
// columns antisymmetric under j -> N - j. With s, d the folded sums and differences of a
// fiber (m = n/2 mirror pairs, f = n - m positions) the coefficients are
//   a_i = sum_r S_{2i+1,r} s_r  (i < f)      b_i = sum_r S_{2i+2,r} d_r  (i < m).
// The folded mode products write a_i + b_i at i and a_i - b_i at n - 1 - i; so the
// transformed array holds the coefficients rotated by 45 degrees in every mirror pair, and
// the folded products of regfac.hip and contract.hip serve both directions unchanged: the
// inverse folds the rotated pairs to 2a and 2b, with the halves in its factor. Only the
// scaling below has to undo and redo the rotation, on the up to eight mirrored positions
// of one octant at a time.
#include "mm_internal.h"

#include <algorithm>

namespace mm {

namespace {

// sin(j k pi / N) from the residue of j k mod 2N, reduced to the first quadrant
__device__ double sine_entry(int64_t j, int64_t k, int N) {
  int64_t r = (j * k) % (2 * (int64_t)N);
  const bool neg = r > N;
  if (neg) r -= N;
  if (2 * r > N) r = N - r;
  const double v = sinpi((double)r / (double)N);
  return neg ? -v : v;
}

// Factors [Es; Ed] (rows of fold_ld(n)) of the transform (fwd) and of its inverse (inv), the
// eigenvalues ev[k] and the exponentials tab[j n + k] = exp(theta_j tau ev[k]), j = 0..q
__global__ void sine_setup(double* __restrict__ fwd, double* __restrict__ inv, double* __restrict__ ev,
                           double* __restrict__ tab, int n, double diff, double tau, SineNodes nodes) {
  const int N = n + 1, m = n >> 1, f = n - m, ld = fold_ld(n);
  const double c = sqrt(2.0 / N);
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < f * ld; e += gridDim.x * blockDim.x) {
    const int i = e / ld, r = e - i * ld;
    double fs = 0.0, fd = 0.0, bs = 0.0, bd = 0.0;
    if (r < f) {
      // transform: row = coefficient i (eigenvectors 2i+1, 2i+2), column = position r
      fs = c * sine_entry(2 * i + 1, r + 1, N);
      if (i < m && r < m) fd = c * sine_entry(2 * i + 2, r + 1, N);
      // inverse: row = position i, column = coefficient r
      bs = (r < m ? 0.5 : 1.0) * c * sine_entry(i + 1, 2 * r + 1, N);
      if (i < m && r < m) bd = 0.5 * c * sine_entry(i + 1, 2 * r + 2, N);
    }
    fwd[e] = fs;
    fwd[f * ld + e] = fd;
    inv[e] = bs;
    inv[f * ld + e] = bd;
  }
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x) {
    const double h = sinpi((k + 1) / (2.0 * N)), v = -4.0 * diff * h * h;
    ev[k] = v;
    for (int j = 0; j <= nodes.q; ++j) tab[(int64_t)j * n + k] = exp(nodes.theta[j] * tau * v);
  }
}

// exp, phi1(z) = (e^z - 1)/z, phi2(z) = (e^z - 1 - z)/z^2 (series below |z| = 1/2, where the
// closed form cancels), 1
__device__ double sine_fn(int f, double z) {
  if (f == MM_EIG_EXP) return exp(z);
  if (f == MM_EIG_PHI1) return z == 0.0 ? 1.0 : expm1(z) / z;
  if (f == MM_EIG_PHI2) {
    if (fabs(z) < 0.5) {
      double term = 0.5, acc = 0.0;
#pragma unroll 1
      for (int k = 0; k < 24; ++k) {
        acc += term;
        term *= z / (k + 3);
      }
      return acc;
    }
    return (expm1(z) - z) / (z * z);
  }
  return 1.0;
}

// out = ca f_a(tau L) a + cb f_b(tau L) b (B: with b) on the rotated coefficients of one
// octant. A thread's octant (i1, i2, i3), i_mu < f_mu, holds the positions i_mu or n_mu - 1 -
// i_mu of every axis (one position where they coincide); slot t = t1 + 2 t2 + 4 t3 of the
// rotated-back values is the coefficient with index 2 i_mu + t_mu along axis mu.
// TAB: exponentials from the 1D tables (a product of three entries; the phi1 quadrature
// sums q such products); otherwise the functions are evaluated at z.
// Bound by its traffic, 16 bytes per point (24 with b): 383^3 250-340 us, 3.6-4 TB/s; 127^3
// 13-15 us.
template <int D, bool B, bool TAB>
__global__ __launch_bounds__(256) void sine_scale_kernel(SineScaleArgs p) {
  constexpr int NT = D == 3 ? 8 : 4;
  const int n1 = p.n[0], n2 = p.n[1], n3 = D == 3 ? p.n[2] : 1;
  const int f1 = n1 - n1 / 2, f2 = n2 - n2 / 2, f3 = n3 - n3 / 2;
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= (int64_t)f1 * f2 * f3) return;
  const int i1 = (int)(e % f1);
  const int64_t r = e / f1;
  const int i2 = (int)(r % f2), i3 = (int)(r / f2);
  // (a middle position has no mirror: its slots with t_mu = 1 are unused)
  const bool pair[3] = {n1 - 1 - i1 != i1, n2 - 1 - i2 != i2, D == 3 && n3 - 1 - i3 != i3};
  bool used[NT];
  int64_t idx[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int t1 = t & 1, t2 = (t >> 1) & 1, t3 = t >> 2;
    used[t] = (!t1 || pair[0]) && (!t2 || pair[1]) && (!t3 || pair[2]);
    const int x1 = t1 ? n1 - 1 - i1 : i1, x2 = t2 ? n2 - 1 - i2 : i2, x3 = t3 ? n3 - 1 - i3 : i3;
    idx[t] = ((int64_t)x3 * n2 + x2) * n1 + x1;
  }
  // position pairs (u at i, v at the mirror) to coefficients ((u + v)/2, (u - v)/2), or back
  auto rotate = [&](double (&v)[NT], double h) {
#pragma unroll
    for (int ax = 0; ax < D; ++ax) {
      if (!pair[ax]) continue;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (t & (1 << ax)) continue;
        const double x = v[t], y = v[t | (1 << ax)];
        v[t] = h * (x + y);
        v[t | (1 << ax)] = h * (x - y);
      }
    }
  };
  double va[NT], vb[NT], fa[NT], fb[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    va[t] = used[t] ? p.a[idx[t]] : 0.0;
    if (B) vb[t] = used[t] ? p.b[idx[t]] : 0.0;
    fa[t] = 0.0;
    fb[t] = 0.0;
  }
  // coefficient index along each axis (clamped where a slot is unused)
  const int k1[2] = {2 * i1, min(2 * i1 + 1, n1 - 1)}, k2[2] = {2 * i2, min(2 * i2 + 1, n2 - 1)},
            k3[2] = {2 * i3, min(2 * i3 + 1, n3 - 1)};
  if (TAB) {
    for (int j = 0; j <= p.q; ++j) {
      const double wa = p.ca * (p.fa == MM_EIG_EXP ? (j == 0) : j > 0 ? p.weight[j] : 0.0);
      const double wb = B ? p.cb * (p.fb == MM_EIG_EXP ? (j == 0) : j > 0 ? p.weight[j] : 0.0) : 0.0;
      if (wa == 0.0 && wb == 0.0) continue;
      const double* t1 = p.tab[0] + (int64_t)j * n1;
      const double* t2 = p.tab[1] + (int64_t)j * n2;
      const double* t3 = D == 3 ? p.tab[2] + (int64_t)j * n3 : nullptr;
      const double x1[2] = {t1[k1[0]], t1[k1[1]]}, x2[2] = {t2[k2[0]], t2[k2[1]]};
      double x3[2] = {1.0, 1.0};
      if (D == 3) {
        x3[0] = t3[k3[0]];
        x3[1] = t3[k3[1]];
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const double x = x1[t & 1] * x2[(t >> 1) & 1] * (D == 3 ? x3[t >> 2] : 1.0);
        fa[t] += wa * x;
        if (B) fb[t] += wb * x;
      }
    }
  } else {
    const double e1[2] = {p.ev[0][k1[0]], p.ev[0][k1[1]]}, e2[2] = {p.ev[1][k2[0]], p.ev[1][k2[1]]};
    double e3[2] = {0.0, 0.0};
    if (D == 3) {
      e3[0] = p.ev[2][k3[0]];
      e3[1] = p.ev[2][k3[1]];
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const double z = p.tau * (e1[t & 1] + e2[(t >> 1) & 1] + (D == 3 ? e3[t >> 2] : 0.0));
      fa[t] = p.ca * sine_fn(p.fa, z);
      if (B) fb[t] = p.cb * sine_fn(p.fb, z);
    }
  }
  rotate(va, 0.5);
  if (B) rotate(vb, 0.5);
#pragma unroll
  for (int t = 0; t < NT; ++t) va[t] = B ? fa[t] * va[t] + fb[t] * vb[t] : fa[t] * va[t];
  rotate(va, 1.0);
#pragma unroll
  for (int t = 0; t < NT; ++t)
    if (used[t]) p.out[idx[t]] = va[t];
}

}  // namespace

hipError_t launch_sine_setup(double* fwd, double* inv, double* ev, double* tab, int n, double diff, double tau,
                             const SineNodes& nodes, hipStream_t s) {
  if (!fwd || !inv || !ev || !tab || n < 1 || nodes.q < 0 || nodes.q >= kMaxGroups) return hipErrorInvalidValue;
  const int f = n - n / 2;
  const int blocks = std::min(1024, (f * fold_ld(n) + 255) / 256);
  sine_setup<<<blocks, 256, 0, s>>>(fwd, inv, ev, tab, n, diff, tau, nodes);
  return hipGetLastError();
}

hipError_t launch_sine_scale(int d, const SineScaleArgs& a, hipStream_t s) {
  if (!a.out || !a.a || (d != 2 && d != 3)) return hipErrorInvalidValue;
  int64_t cnt = 1;
  for (int mu = 0; mu < d; ++mu) cnt *= a.n[mu] - a.n[mu] / 2;
  const dim3 grid((unsigned)((cnt + 255) / 256)), block(256);
  const bool tab = a.q > 0;
  if (tab && ((a.fa != MM_EIG_EXP && a.fa != MM_EIG_QUAD) || (a.b && a.fb != MM_EIG_EXP && a.fb != MM_EIG_QUAD)))
    return hipErrorInvalidValue;
  if (!tab && (a.fa == MM_EIG_QUAD || (a.b && a.fb == MM_EIG_QUAD))) return hipErrorInvalidValue;
  auto go = [&](auto kernel) { kernel<<<grid, block, 0, s>>>(a); };
  if (d == 3) {
    if (a.b)
      tab ? go(sine_scale_kernel<3, true, true>) : go(sine_scale_kernel<3, true, false>);
    else
      tab ? go(sine_scale_kernel<3, false, true>) : go(sine_scale_kernel<3, false, false>);
  } else {
    if (a.b)
      tab ? go(sine_scale_kernel<2, true, true>) : go(sine_scale_kernel<2, true, false>);
    else
      tab ? go(sine_scale_kernel<2, false, true>) : go(sine_scale_kernel<2, false, false>);
  }
  return hipGetLastError();
}

}  // namespace mm
