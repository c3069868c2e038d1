// Sums of mode products of small periodic 2D grids as independent tasks of one launch (gfx950,
// FP64, axes of 2 to 256 points).
//
// A step of such a problem is a chain of 256 x 256 x 256 products and pointwise passes, each
// worth well under a microsecond of the chip, so the step is bound by the number of launches
// and by what one costs: the tiled kernel's serial chain of K chunks, 9-12 us per product. A
// task here is one output array that is a sum of up to two mode products (along x1 or x2,
// any inputs) with a pointwise epilogue: the flux of the spectral remainder, or a stage
// combination with the reaction. A launch takes up to three tasks; a workgroup computes one
// 16 x 16 tile of one task, its four waves sharing the k blocks of the task's products. A
// wave loads all its fragments at once, straight into registers (two row operands as 16-byte
// pairs of consecutive k), so a launch has one load latency, up to 32 matrix instructions
// per wave and one sum over the waves in LDS. 256^2: 5-7.5 us per launch of one or two tasks
// (three with two products each 13.5), against 9-12 us per product and 1.5-3 per pointwise
// pass.
#include <cfloat>

#include "mm_internal.h"

#include <algorithm>

namespace mm {

typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));
typedef double d4 __attribute__((ext_vector_type(4)));

namespace {

// four consecutive values base[k..k+3] of a row of n (zero past the row; n >= 2)
__device__ __forceinline__ void row4(double (&f)[4], const double* __restrict__ base, int k, int n) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int i = k + 2 * h, c = min(i, n - 2);
    const d2u q = *reinterpret_cast<const d2u*>(base + c);
    f[2 * h] = i < n ? (c == i ? q.x : q.y) : 0.0;
    f[2 * h + 1] = i + 1 < n ? q.y : 0.0;
  }
}

// NB: k blocks of 16 per wave
template <int NB>
__global__ __launch_bounds__(256, NB > 4 ? 2 : 4) void periodic_products(PeriodicBatch batch) {
  const PeriodicTask& p = batch.t[blockIdx.y];
  const int n1 = batch.n1, n2 = batch.n2;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lg = lane >> 4, lr = lane & 15;
  const int nt1 = (n1 + 15) / 16;
  const int r0 = 16 * (blockIdx.x / nt1), c0 = 16 * (blockIdx.x % nt1);   // x2 rows, x1 columns
  const int row = min(r0 + lr, n2 - 1), col = min(c0 + lr, n1 - 1);

  // block i of this wave: products' k blocks wave + 4 i, the first product's first
  const int b0 = p.M[0] ? ((p.mode[0] ? n2 : n1) + 15) / 16 : 0;
  const int b1 = p.M[1] ? ((p.mode[1] ? n2 : n1) + 15) / 16 : 0;
  double fa[NB][4], fb[NB][4];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int b = wave + 4 * i;
#pragma unroll
    for (int s = 0; s < 4; ++s) fa[i][s] = fb[i][s] = 0.0;
    if (b >= b0 + b1) continue;
    const int q = b >= b0;
    const double* __restrict__ M = p.M[q];
    const double* __restrict__ X = p.X[q];
    const int k = 16 * (q ? b - b0 : b) + 4 * lg;
    if (p.mode[q] == 0) {   // X[row][k] M[col][k]
      row4(fa[i], X + row * n1, k, n1);
      row4(fb[i], M + col * n1, k, n1);
    } else {                // M[row][k] X[k][col]
      row4(fa[i], M + row * n2, k, n2);
#pragma unroll
      for (int s = 0; s < 4; ++s) fb[i][s] = X[min(k + s, n2 - 1) * n1 + col];
#pragma unroll
      for (int s = 0; s < 4; ++s) fb[i][s] = k + s < n2 ? fb[i][s] : 0.0;
    }
  }
  // the epilogue's operands of this lane's output element: element t = wave of the f64 16x16
  // layout (lane l, element t: row 4t + l/16, column l%16)
  const int er = r0 + 4 * wave + lg, ec = c0 + lr;
  const bool live = er < n2 && ec < n1;
  const int e = min(er, n2 - 1) * n1 + min(ec, n1 - 1);
  const double ca = p.coef ? p.coef[e] - p.coef0 : p.scale;
  const double cu = p.flux_u ? p.flux_u[e] * ((p.vel ? p.vel[e] : p.vel_const) - p.vel0) : 0.0;
  const double ru = p.react ? p.react[e] : 0.0;
  const double sb = p.sub ? p.sub[e] : 0.0;
  const double ba0 = p.base[0] ? p.base[0][e] : 0.0, ba1 = p.base[1] ? p.base[1][e] : 0.0;

  d4 acc[2] = {d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}};
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int s = 0; s < 4; ++s)
      acc[s & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[i][s], fb[i][s], acc[s & 1], 0, 0, 0);
  __shared__ double part[4][4][64];
#pragma unroll
  for (int t = 0; t < 4; ++t) part[wave][t][lane] = acc[0][t] + acc[1][t];
  __syncthreads();
  double v = 0.0;
#pragma unroll
  for (int w = 0; w < 4; ++w) v += part[w][wave][lane];
  double g = ca * v + cu;
  if (p.react) g += p.r[0] + ru * (p.r[1] + ru * (p.r[2] + ru * p.r[3]));
  if (p.sub) g -= sb;
  const double o0 = p.base[0] ? ba0 + p.c[0] * g : p.c[0] * g;
  if (live) {
    p.out[0][e] = o0;
    if (p.flag && !(fabs(o0) <= DBL_MAX)) p.flag[0] = 1;
    if (p.out[1]) p.out[1][e] = p.base[1] ? ba1 + p.c[1] * g : p.c[1] * g;
  }
}

}  // namespace

bool periodic_fits(int d, int n1, int n2) { return d == 2 && n1 >= 2 && n2 >= 2 && n1 <= 256 && n2 <= 256; }

hipError_t launch_periodic(const PeriodicTask* t, int count, int n1, int n2, hipStream_t s) {
  if (count < 1 || count > kMaxPeriodicTasks || !periodic_fits(2, n1, n2)) return hipErrorInvalidValue;
  PeriodicBatch b{};
  b.n1 = n1;
  b.n2 = n2;
  int blocks = 1;
  for (int i = 0; i < count; ++i) {
    if (!t[i].out[0] || !t[i].M[0]) return hipErrorInvalidValue;
    int nb = 0;
    for (int q = 0; q < 2; ++q) {
      if (!t[i].M[q]) continue;
      if (!t[i].X[q] || t[i].mode[q] < 0 || t[i].mode[q] > 1) return hipErrorInvalidValue;
      nb += ((t[i].mode[q] ? n2 : n1) + 15) / 16;
    }
    blocks = std::max(blocks, (nb + 3) / 4);
    b.t[i] = t[i];
  }
  const dim3 grid((unsigned)(((n1 + 15) / 16) * ((n2 + 15) / 16)), (unsigned)count);
  if (blocks <= 2)
    periodic_products<2><<<grid, 256, 0, s>>>(b);
  else if (blocks <= 4)
    periodic_products<4><<<grid, 256, 0, s>>>(b);
  else if (blocks <= 6)
    periodic_products<6><<<grid, 256, 0, s>>>(b);
  else
    periodic_products<8><<<grid, 256, 0, s>>>(b);
  return hipGetLastError();
}

}  // namespace mm
