// Stage evaluation and the first two mode products of an x3 slab in one workgroup (gfx950,
// FP64, grids with n1, n2 <= 64).
//
// On such grids a slab's x1-x2 plane fits LDS with its coefficient, and the separate passes
// (remainder stencil, product along x1, product along x2) are each bound by what they cost
// before their first product: a launch, the load latency, the store of an intermediate
// that the next one reads back. Here a workgroup evaluates the stage vector of one slab
// (the remainder reads the planes above and below straight from memory), multiplies it by
// E1 along x1 and by E2 along x2 in LDS, and writes the result once; the product along x3
// follows as a mode product of its own. 60^3: 12-13.5 us for one or two vectors, against
// 5.2 us of stencil and 5-6 us per product and vector. Without a remainder the slab is read, multiplied
// twice and written (launch_slab_action). 2 T waves, T = ceil(max(n1, n2)/16), each with the
// factor rows of one tile of either product in registers.
#include <cfloat>

#include "mm_internal.h"

#include <algorithm>

namespace mm {

typedef double d4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int kSlabMax = 64;
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));

// What a slab costs before its first product is bound by the number of vector memory
// instructions: points go in pairs along x1 (16-byte loads), all loads are unconditional
// (clamped into the arrays) and issued together.
// CN: column tiles of x1 that a workgroup computes (T, or half of them, rounded up: blockIdx.z
// selects the half, and each evaluates the whole stage vector).
template <int T, int CN>
__global__ __launch_bounds__(128 * T, 2) void slab_products(SlabArgs p) {
  constexpr int K = 16 * T;        // padded length of both axes
  constexpr int PU = K + 3;        // LDS pitch of the plane with its ghost ring (odd)
  constexpr int NT = 128 * T;
  const int v = blockIdx.y, z = blockIdx.x;
  const int n1 = p.n1, n2 = p.n2, n3 = p.n3;
  __shared__ double U[(K + 2) * PU], A[(K + 2) * PU];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lg = lane >> 4, lr = lane & 15;
  const int c0 = CN * blockIdx.z;            // first column tile
  // first product: column tile c0 + wave mod CN, row tiles ot1 + j 2T/CN; second: row tile
  // wave mod T, column tiles c0 + wave / T + 2 j
  const int ft1 = c0 + wave % CN, ot1 = wave / CN, ft2 = wave % T, ot2 = c0 + wave / T;
  constexpr int S1 = 2 * T / CN;

  const int plane = n1 * n2, dof = plane * n3;
  const int t2 = n1 + 2, t3 = t2 * (n2 + 2);
  const double* __restrict__ u = p.u;
  const double* __restrict__ a = p.a;
  const bool eval = p.c[v] != 0.0 || p.raw;   // the remainder is needed
  const bool flux = eval && !p.nondiv;        // and the coefficient's neighbours
  // values i, i + 1 of u (the pair at the last value of all is moved one back)
  auto pair = [&](int i) {
    const int c = min(i, dof - 2);
    d2u q = *reinterpret_cast<const d2u*>(u + c);
    q.x = c == i ? q.x : q.y;
    return q;
  };
  // pair i of this thread: row y, columns x, x + 1 (columns 2 (tid mod K/2), T rows NT / (K/2)
  // apart)
  const int x = 2 * (tid % (K / 2)), y0 = tid / (K / 2);
  constexpr int DY = NT / (K / 2);
  const int xc = min(x, n1 - 1);
  d2u uc[T], um[T], up[T], ac[T], am[T], ap[T];
  const int lo = z > 0 ? plane : 0, hi = z + 1 < n3 ? plane : 0;
#pragma unroll
  for (int i = 0; i < T; ++i) {
    const int yc = min(y0 + i * DY, n2 - 1);
    const int iu = plane * z + yc * n1 + xc, ia = t3 * (z + 1) + (yc + 1) * t2 + xc + 1;
    uc[i] = pair(iu);
    if (eval) {
      um[i] = pair(iu - lo);
      up[i] = pair(iu + hi);
      ac[i] = *reinterpret_cast<const d2u*>(a + ia);
      if (flux) {
        am[i] = *reinterpret_cast<const d2u*>(a + ia - t3);
        ap[i] = *reinterpret_cast<const d2u*>(a + ia + t3);
      }
    }
  }
  // the boundary nodes of a around the plane
  const int ring = 2 * t2 + 2 * n2;
  const int rx = tid < 2 * t2 ? tid % t2 : (tid - 2 * t2) % 2 * (n1 + 1);
  const int ry = tid < 2 * t2 ? tid / t2 * (n2 + 1) : (tid - 2 * t2) / 2 + 1;
  double ar = 0.0;
  if (flux && tid < ring) ar = a[t3 * (z + 1) + ry * t2 + rx];
  // factor rows 16 ft + lr of a tile: element 4 b + s is k = 16 b + 4 lg + s (zero past the axis)
  auto rows = [&](double (&f)[4 * T], const double* E, int n, int ft) {
    const int r = min(16 * ft + lr, n - 1), last = n * n - 2;
#pragma unroll
    for (int h = 0; h < 2 * T; ++h) {
      const int k = 16 * (h >> 1) + 4 * lg + 2 * (h & 1), i = r * n + k, c = min(i, last);
      const d2u q = *reinterpret_cast<const d2u*>(E + c);
      f[2 * h] = k < n ? (c == i ? q.x : q.y) : 0.0;
      f[2 * h + 1] = k + 1 < n ? q.y : 0.0;
    }
  };
  // LDS: the plane of u with zeros around it and beyond the axes, the plane of a with its
  // boundary nodes
#pragma unroll
  for (int i = 0; i < T; ++i) {
    const int y = y0 + i * DY;
    double* q = U + (y + 1) * PU + x + 1;
    uc[i].x = x < n1 && y < n2 ? uc[i].x : 0.0;
    uc[i].y = x + 1 < n1 && y < n2 ? uc[i].y : 0.0;
    q[0] = uc[i].x;
    q[1] = uc[i].y;
    if (flux && y < n2) {   // (the ring is written by its own threads below)
      double* b = A + (y + 1) * PU + x + 1;
      if (x < n1) b[0] = ac[i].x;
      if (x + 1 < n1) b[1] = ac[i].y;
    }
  }
  for (int e = tid; e < 4 * (K + 2); e += NT) {
    const int side = e / (K + 2), k = e - side * (K + 2);
    U[side == 0 ? k : side == 1 ? (K + 1) * PU + k : side == 2 ? k * PU : k * PU + K + 1] = 0.0;
  }
  if (flux && tid < ring) A[ry * PU + rx] = ar;
  double f1[4 * T], f2[4 * T];
  rows(f1, p.E1[v], n1, ft1);
  __syncthreads();
  if (eval) {
    bool bad = false;
    const bool mz = p.neu[2] && z == n3 - 1;
    const double base = p.base[v] ? 1.0 : 0.0, c = p.c[v];
    d2u val[T];
#pragma unroll
    for (int i = 0; i < T; ++i) {
      const int y = y0 + i * DY;
      val[i] = d2u{0.0, 0.0};
      if (x >= n1 || y >= n2) continue;
      const double* q = U + (y + 1) * PU + x + 1;
      const double* b = A + (y + 1) * PU + x + 1;
      const double ux[4] = {q[-1], uc[i].x, uc[i].y, q[2]};
      const double ax[4] = {flux ? b[-1] : 0.0, ac[i].x, ac[i].y, flux ? b[2] : 0.0};
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        if (x + e >= n1) continue;
        const double u0 = ux[e + 1], a0 = ax[e + 1];
        const double uxm = ux[e], uxp = p.neu[0] && x + e == n1 - 1 ? uxm : ux[e + 2];
        const double uym = q[e - PU], uyp = p.neu[1] && y == n2 - 1 ? uym : q[e + PU];
        const double uzm = lo ? um[i][e] : 0.0, uzp = mz ? uzm : hi ? up[i][e] : 0.0;
        // (the arithmetic of the remainder stencil; the reaction is shared with raw)
        const double react = p.r0 + u0 * (p.r1 + u0 * (p.r2 + u0 * p.r3));
        auto remainder = [&](double la, const double (&cadv)[3]) {
          double s;
          if (p.nondiv) {
            const double cc = a0 - la;
            s = cc * (uxp - 2.0 * u0 + uxm) * p.ih2[0] + cadv[0] * (uxp - uxm);
            s += cc * (uyp - 2.0 * u0 + uym) * p.ih2[1] + cadv[1] * (uyp - uym);
            s += cc * (uzp - 2.0 * u0 + uzm) * p.ih2[2] + cadv[2] * (uzp - uzm);
          } else {
            // (a's own right neighbour is the pair's second value or the node after it)
            const double axp = e == 0 ? (x + 1 < n1 ? ax[2] : b[1]) : ax[3];
            s = ((0.5 * (a0 + axp) - la) * (uxp - u0) - (0.5 * (a0 + ax[e]) - la) * (u0 - uxm)) * p.ih2[0] +
                cadv[0] * (uxp - uxm);
            s += ((0.5 * (a0 + b[e + PU]) - la) * (uyp - u0) - (0.5 * (a0 + b[e - PU]) - la) * (u0 - uym)) * p.ih2[1] +
                 cadv[1] * (uyp - uym);
            s += ((0.5 * (a0 + ap[i][e]) - la) * (uzp - u0) - (0.5 * (a0 + am[i][e]) - la) * (u0 - uzm)) * p.ih2[2] +
                 cadv[2] * (uzp - uzm);
          }
          return s + react;
        };
        const int idx = plane * z + y * n1 + x + e;
        double s = remainder(p.lam_amax, p.cadv);
        if (p.sub) s -= p.sub[idx];
        val[i][e] = base * u0 + c * s;
        bad |= !(fabs(val[i][e]) <= DBL_MAX);
        if (p.raw && v == 0 && c0 == 0) p.raw[idx] = remainder(p.raw_lam_amax, p.raw_cadv);
      }
    }
    __syncthreads();   // every thread has read the plane
#pragma unroll
    for (int i = 0; i < T; ++i) {
      const int y = y0 + i * DY;
      double* q = U + (y + 1) * PU + x + 1;
      q[0] = val[i].x;
      q[1] = val[i].y;
    }
    if (p.flag && bad) p.flag[0] = 1;
    __syncthreads();
  }
  rows(f2, p.E2[v], n2, ft2);   // (in flight under the first product)

  // X[i2][j1] <- sum_k X[i2][k] E1[j1][k]
  double* X = U + PU + 1;
  constexpr int NJ = (CN + 1) / 2;
  d4 acc[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) acc[j] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int kk = 0; kk < 4 * T; ++kk)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int r = 16 * min(ot1 + S1 * j, T - 1), k = 16 * (kk >> 2) + 4 * lg + (kk & 3);
      acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(X[(r + lr) * PU + k], f1[kk], acc[j], 0, 0, 0);
    }
  __syncthreads();   // every wave has read X
  // f64 16x16 layout: lane l, element t holds row 4t + l/16, column l%16
#pragma unroll
  for (int j = 0; j < NJ; ++j)
    if (ot1 + S1 * j < T && ft1 < T)
#pragma unroll
      for (int t = 0; t < 4; ++t) X[(16 * (ot1 + S1 * j) + 4 * t + lg) * PU + 16 * ft1 + lr] = acc[j][t];
  __syncthreads();
  // out[j2][i1] = sum_k E2[j2][k] X[k][i1]
#pragma unroll
  for (int j = 0; j < NJ; ++j) acc[j] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int kk = 0; kk < 4 * T; ++kk)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int c = 16 * min(ot2 + 2 * j, T - 1), k = 16 * (kk >> 2) + 4 * lg + (kk & 3);
      acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(f2[kk], X[k * PU + c + lr], acc[j], 0, 0, 0);
    }
  double* out = p.out[v] + (int64_t)plane * z;
#pragma unroll
  for (int j = 0; j < NJ; ++j)
    if (ot2 + 2 * j < min(c0 + CN, T))
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int y = 16 * ft2 + 4 * t + lg, x = 16 * (ot2 + 2 * j) + lr;
        if (y < n2 && x < n1) __builtin_nontemporal_store(acc[j][t], out + y * n1 + x);
      }
}

}  // namespace

bool slab_fits(int d, int n1, int n2, int n3) {
  return d == 3 && n1 >= 2 && n2 >= 2 && n3 >= 1 && n1 <= kSlabMax && n2 <= kSlabMax && n3 <= 65535;
}

hipError_t launch_slab_action(const double* u, const double* E1, const double* E2, double* out, int n1, int n2, int n3,
                              hipStream_t s) {
  SlabArgs a{};
  a.u = a.a = u;   // (without a remainder the coefficient is not read)
  a.n1 = n1;
  a.n2 = n2;
  a.n3 = n3;
  a.base[0] = 1;
  a.E1[0] = E1;
  a.E2[0] = E2;
  a.out[0] = out;
  return launch_slab(a, 1, s);
}

hipError_t launch_slab(const SlabArgs& a, int nvec, hipStream_t s) {
  if (nvec < 1 || nvec > 2 || !a.u || !a.a || !slab_fits(3, a.n1, a.n2, a.n3)) return hipErrorInvalidValue;
  for (int v = 0; v < nvec; ++v)
    if (!a.E1[v] || !a.E2[v] || !a.out[v]) return hipErrorInvalidValue;
  const int T = (std::max(a.n1, a.n2) + 15) / 16;
  // two workgroups per slab while that leaves each a compute unit of its own (60^3, SL2: 41.1 ->
  // 38.9 us per step)
  const bool split = T > 1 && 2 * a.n3 * nvec <= 256;
  const dim3 grid(a.n3, nvec, split ? 2 : 1), block(128 * T);
  auto go = [&](auto kernel) { kernel<<<grid, block, 0, s>>>(a); };
  switch (T) {
    case 1: go(slab_products<1, 1>); break;
    case 2: split ? go(slab_products<2, 1>) : go(slab_products<2, 2>); break;
    case 3: split ? go(slab_products<3, 2>) : go(slab_products<3, 3>); break;
    default: split ? go(slab_products<4, 2>) : go(slab_products<4, 4>); break;
  }
  return hipGetLastError();
}

}  // namespace mm
