// FP64 mode products with the factor held in registers (gfx950).
//
// What bounds the tiled kernels of contract.hip on these products is not the matrix unit:
// each of their workgroups re-reads factor and grid tiles in short K chunks, with a
// barrier, LDS stores and fragment reads of both operands per chunk. But a factor is
// small: the rows [Es; Ed] of a folded 255-point axis are 262 KB, half the register file
// of one compute unit. So a wave keeps the factor rows of its 16 output positions over
// the whole contraction in registers for its lifetime, and the workgroup walks over tiles
// of grid fibers: every grid value is loaded once, staged in LDS over the whole K range
// as the sums s and differences d, and read as fragments by the row waves. One barrier per
// tile instead of one per chunk, half the LDS reads per MFMA, no factor traffic.
//
// Work split: RW row waves of 16 output positions each (16 rows of Es and the same of Ed)
// x WC column waves of NC 16-fiber units. Workgroups are persistent; the next tile's loads
// are in flight through the current tile's products. Fibers of modes 2/3 are cut into
// units of 16 columns per slab, so that a ragged slab wastes at most 15 columns, and the
// rows are padded to 16 folded positions (the tiled kernel: 64); a tile takes NC WC
// consecutive units.
//
// Measured (two stacked 255^3 vectors, rows of 256; kernel alone): 145-153 us per product
// against 190-202 of the tiled kernel, 56-59 TFLOP/s executed; the products alone (no grid
// traffic) run 124 us, the grid traffic alone 106-117 us (530 MB; a copy of that size
// 98 us). 127^3: 17-18 against 20-21 us, bound by the start of a workgroup (its first
// tile and factor rows) and the traffic, with four tiles per compute unit in all; 130 x 129
// x 127: 24-26 against 28-58 us (f = 65 pads to 80 rows instead of 128).
// Results are bit for bit those of gemm_f64_fold: every output sums over k in blocks of 8
// with k = 2g + s in lane group g at step s.
#include "mm_internal.h"

#include <algorithm>
#include <type_traits>

namespace mm {

typedef double d2 __attribute__((ext_vector_type(2)));
typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));
typedef unsigned u2 __attribute__((ext_vector_type(2)));
typedef unsigned u4 __attribute__((ext_vector_type(4)));

namespace {

// Grid operands go through buffer descriptors: a lane offset plus a uniform offset per
// access, both 32-bit, and accesses past `bytes` are dropped by the hardware, so that a
// masked store is a store to offset kOut (operands are below 2 GB: checked at launch).
constexpr unsigned kOut = 0x80000000u;
constexpr unsigned kOperandBytes = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t operand(const void* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, kOperandBytes, 0x00020000);
}
__device__ __forceinline__ d2 load2(__amdgpu_buffer_rsrc_t r, unsigned off, unsigned uniform) {
  return __builtin_bit_cast(d2, __builtin_amdgcn_raw_buffer_load_b128(r, off, uniform, 0));
}
__device__ __forceinline__ double load1(__amdgpu_buffer_rsrc_t r, unsigned off, unsigned uniform) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off, uniform, 0));
}
template <bool NT>
__device__ __forceinline__ void store1(__amdgpu_buffer_rsrc_t r, unsigned off, unsigned uniform, double v) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), r, off, uniform, NT ? 2 /* nontemporal */ : 0);
}

// position of the k pair (2u, 2u + 1) in an LDS row, in pairs: a lane group reads its pair
// of step block h at pair 4h + lg (folded: natural order; plain: lane group g takes
// k = 16 b + 4g + {0, 1} at block 2b and 16 b + 4g + {2, 3} at block 2b + 1)
template <int FOLD>
__device__ __forceinline__ int pair_slot(int u) {
  return FOLD ? u : (u & ~7) | ((u & 1) << 2) | ((u & 7) >> 1);
}
// first k of lane group lg at step block h
template <int FOLD>
__device__ __forceinline__ int frag_k(int h, int lg) {
  return FOLD ? 8 * h + 2 * lg : 16 * (h >> 1) + 4 * lg + 2 * (h & 1);
}

}  // namespace

// H: step blocks of 8 k (folded: f <= 8H; plain: K <= 8H, H even)
template <int BT, int FOLD, int H, int RW, int WC, int NC, int WPE, int LATE>
__global__ __launch_bounds__(64 * RW * WC, WPE) void gemm_f64_regs(GemmArgs p) {
  constexpr int NT = 64 * RW * WC;
  constexpr int CT = NC * WC;              // units (16 fibers) per tile
  constexpr int TC = 16 * CT;              // fibers per tile
  constexpr int KP = 4 * H;                // k pairs
  // LDS rows of one fiber, in doubles: 16-byte pairs at pitch 2 (2H + 1), twice an odd
  // number, so that the fragment reads (16 fibers x 2 lane groups per half wave) fall on
  // distinct 16-byte slots
  constexpr int PK = 8 * H + 4;
  constexpr int NS = FOLD ? 2 : 1;         // staged values per position (s and d, or x)
  constexpr int KPM = H <= 16 ? 8 * ((H + 1) / 2) : 128;   // staged k pairs (mode 1: threads per fiber)
  constexpr int KI = NT / (TC / 2);        // modes 2/3: k pairs per pass
  constexpr int FI = NT / KPM;             // mode 1: fibers per pass
  static_assert(BT || (NT % KPM == 0 && TC % FI == 0), "mode 1 staging covers whole fibers");
  constexpr int NI = BT ? (KP + KI - 1) / KI : TC / FI;
  __shared__ __attribute__((aligned(16))) double Gs[2][NS][TC * PK];

  const int L = blockIdx.x;
  const int P = (L & 7) * p.per_xcd + (L >> 3);
  if (P >= p.total) return;
  const int RG = p.tiles_m;                // row groups
  const int W = p.tiles_n;                 // workers per problem and row group
  const int rg = P % RG, gw = P / RG, w = gw % W, g = gw / W;
  const int n = p.K, m = n >> 1, f = FOLD ? n - m : n;
  const int M = p.M, N = p.N;
  const int fibers = BT ? N : M;           // per slab
  const int rows = FOLD ? f : (BT ? M : N);   // output positions
  const int ldx = BT ? p.ldb : p.lda, ldc = p.ldc;
  const double* __restrict__ X = (const double*)(BT ? p.B[g] : p.A[g]);
  double* __restrict__ C = (double*)p.C[g];
  const double* __restrict__ Cadd = p.Cadd[g];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave % RW, wc = wave / RW;
  const int lg = lane >> 4, lr = lane & 15;
  const int r0 = 16 * (rg * RW + wr);      // first output position of this wave

  // units: slab b = unit / upb, fibers 16 (unit % upb) ..; every position that moves from
  // tile to tile advances by W CT units without a division
  const int upb = (fibers + 15) >> 4;
  const int units = upb * p.inner;
  const int step = W * CT, stepb = step / upb, stepc = step - stepb * upb;
  auto advance = [&](int& b, int& c) {
    b += stepb;
    c += stepc;
    if (c >= upb) {
      c -= upb;
      ++b;
    }
  };

  // Staging. Modes 2/3: a thread covers one column pair of the tile (eight consecutive
  // pairs per unit: 16-byte loads) and the k pairs tk + i KI; mode 1: the k pair tk of the
  // fibers tc + i FI. Byte offsets are 32-bit (checked at launch).
  // Modes 2/3: the last pair of a slab of odd N starts at its last column where the row
  // continues (padding), else one column before (shift).
  constexpr int NV = BT ? 2 * NS : NS;     // 16-byte loads per item
  const int tc = BT ? tid % (TC / 2) : tid / KPM;
  const int tk = BT ? tid / (TC / 2) : tid % KPM;
  const bool shift = BT && (N & 1) && ldx == N;
  const int cmax = (N & 1) && !shift ? N - 1 : N - 2;
  int ub, uc;   // modes 2/3: unit of the thread's columns; mode 1: ub the row of fiber tc
  if (BT) {
    const int unit = w * CT + (tc >> 3);
    ub = unit / upb;
    uc = unit - ub * upb;
  } else {
    ub = 16 * w * CT + tc;
    uc = 0;
  }
  // one item's grid values: modes 2/3: x(k), x(k+1) of two columns and their mirrors;
  // mode 1: the pair x(k), x(k+1) and the mirror pair (in reverse order)
  struct Item {
    d2 v[NV];
  };
  bool odd = false;   // the thread's column pair was moved one column back
  auto kpair = [&](int i) { return BT ? tk + i * KI : tk; };
  auto idle = [&](int i) { return BT ? (i + 1) * KI > KP && kpair(i) >= KP : KPM != KP && tk >= KP; };
  // Byte offsets of the thread's first k and of its mirror in a fiber; items differ by
  // uniform amounts, which go into the scalar base of the load. Folded: no k is clamped,
  // as with n >= 17 and 8 (H - 2) < f the staged positions k < 8H and their mirrors lie
  // inside the fiber. Plain: k is clamped to the fiber.
  const unsigned ks = BT ? 8u * (unsigned)ldx : 8u;
  constexpr int DK = BT ? 2 * KI * (NI - 1) + 1 : 0;   // the last k of a thread - its first
  const unsigned kb = 2u * (unsigned)tk * ks;
  // (mode 1: the pair x[n-2-k], x[n-1-k])
  const unsigned mb = (unsigned)(n - (BT ? 1 : 2) - DK) * ks - kb;
  const __amdgpu_buffer_rsrc_t xr = operand(X), cr = operand(C), ar = operand(Cadd);
  unsigned foff = 0;   // modes 2/3: offset of the thread's columns in the tile being loaded
  auto position = [&]() {
    if (BT) {
      const int c = 16 * uc + 2 * (tc & 7);
      // (units past the last: clamped to the last slab, feeding masked outputs)
      foff = (unsigned)min(ub, p.inner - 1) * (8u * (unsigned)p.sB) + 8u * (unsigned)min(c, cmax);
      odd = shift && c == N - 1;
      advance(ub, uc);
    }
  };
  auto load = [&](int i, Item& q) {
    if (idle(i)) return;
    if (BT) {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int dk = 2 * KI * i + s;
        if (FOLD) {
          q.v[s] = load2(xr, foff + kb, (unsigned)dk * ks);
          q.v[NV - 2 + s] = load2(xr, foff + mb, (unsigned)(DK - dk) * ks);
        } else {
          q.v[s] = load2(xr, foff + min(kb + (unsigned)dk * ks, (unsigned)(n - 1) * ks), 0);
        }
      }
    } else {
      const unsigned o = (unsigned)min(ub + i * FI, M - 1) * (8u * (unsigned)ldx);
      if (FOLD) {
        q.v[0] = load2(xr, o + kb, 0);
        q.v[NV - 1] = load2(xr, o + mb, 0);
      } else {   // (the pair at n - 1 of an odd K: one back)
        q.v[0] = load2(xr, o + min(kb, 8u * (unsigned)(n - 2)), 0);
      }
      if (i == NI - 1) ub += 16 * step;
    }
  };
  const int lo = (BT ? 2 * tc : tc) * PK;
  // part c of item i (modes 2/3: one of its two columns) into the LDS tile
  auto store = [&](int buf, int i, int c, const Item& q) {
    if (idle(i)) return;
    double* G0 = &Gs[buf][0][0] + lo;
    constexpr int GS = TC * PK;            // d tile after the s tile
    const int k = 2 * kpair(i), slot = 2 * pair_slot<FOLD>(kpair(i));
    d2 v[NS];
    if (BT) {
      double x[NV];
#pragma unroll
      for (int t = 0; t < NV; ++t) x[t] = q.v[t][c];
      if (c == 0 && shift) {   // (wave-uniform; the lane's choice is a select)
#pragma unroll
        for (int t = 0; t < NV; ++t) x[t] = odd ? q.v[t].y : q.v[t].x;
      }
      if (FOLD) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          v[0][s] = x[s] + x[NV - 2 + s];
          v[NS - 1][s] = x[s] - x[NV - 2 + s];
        }
        // (wave-uniform: some k of the wave's items is not below the middle)
        if (!(2 * ((64 * wave + 63) / (TC / 2) + i * KI) + 1 < m)) {
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            v[0][s] = k + s < m ? v[0][s] : k + s < f ? x[s] : 0.0;
            v[NS - 1][s] = k + s < m ? v[NS - 1][s] : 0.0;
          }
        }
      } else {
        v[0] = d2{k < n ? x[0] : 0.0, k + 1 < n ? x[1] : 0.0};
      }
#pragma unroll
      for (int t = 0; t < NS; ++t) *reinterpret_cast<d2*>(G0 + t * GS + c * PK + slot) = v[t];
    } else {
      if (FOLD) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const double x0 = q.v[0][s], x1 = q.v[NV - 1][1 - s];
          v[0][s] = k + s < m ? x0 + x1 : k + s < f ? x0 : 0.0;
          v[NS - 1][s] = k + s < m ? x0 - x1 : 0.0;
        }
      } else {
        v[0].x = k + 1 < n ? q.v[0].x : k < n ? q.v[0].y : 0.0;
        v[0].y = k + 1 < n ? q.v[0].y : 0.0;
      }
#pragma unroll
      for (int t = 0; t < NS; ++t) *reinterpret_cast<d2*>(G0 + t * GS + i * FI * PK + slot) = v[t];
    }
  };
  constexpr int NP = BT ? 2 : 1;           // parts of an item

  // output units of this wave (uniform)
  int ob[NC], oc[NC];
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    const int unit = w * CT + wc * NC + j;
    ob[j] = unit / upb;
    oc[j] = unit - ob[j] * upb;
  }
  // f64 16x16 layout: lane l, element t holds row 4t + l/16, column l%16 (modes 2/3: rows
  // are positions, columns fibers; mode 1 the reverse): a store covers four 128-byte runs.
  // Byte offsets of element 0 (and, modes 2/3, of the mirror of element 3, mode 1 of element
  // 0) from the unit's first value; element t is t st away (modes 2/3, mirror: 3 - t).
  d4 acc[NS][NC];
  const unsigned o0 = 8u * (unsigned)(BT ? (r0 + lg) * ldc + lr : lg * ldc + r0 + lr);
  const unsigned o1 = 8u * (unsigned)(BT ? (n - 13 - r0 - lg) * ldc + lr : lg * ldc + n - 1 - r0 - lr);
  // unit j of the results: its byte offset in C and its fibers (0 past the last unit)
  unsigned rb[NC];
  int rl[NC];
  auto results_of_tile = [&]() {
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      rb[j] = 8u * ((unsigned)ob[j] * (unsigned)p.sC + 16u * (unsigned)oc[j] * (BT ? 1u : (unsigned)ldc));
      rl[j] = ob[j] < p.inner ? fibers - 16 * oc[j] : 0;
      advance(ob[j], oc[j]);
    }
  };
  const bool whole_rows = r0 + 15 < (FOLD ? m : rows);   // every row exists and has a mirror
  const unsigned st = 32u * (unsigned)ldc;
  // lane offsets of element t and of its mirror (kOut where there is none) and their
  // uniform offsets (the mirror rows of modes 2/3 run downwards: from element 3)
  auto lane0 = [&](int j, int t) {
    const bool live = (BT ? lr : 4 * t + lg) < rl[j];
    return live && (whole_rows || (BT ? r0 + 4 * t + lg : r0 + lr) < rows) ? o0 : kOut;
  };
  auto lane1 = [&](int j, int t) {
    const bool live = (BT ? lr : 4 * t + lg) < rl[j];
    return live && (whole_rows || (BT ? r0 + 4 * t + lg : r0 + lr) < m) ? o1 : kOut;
  };
  // element t of unit j of y to C (alpha = 1, nothing added)
  auto write = [&](const d4 (&y)[NS][NC], int j, int t, auto stream) {
    constexpr bool NT = decltype(stream)::value;
    const double a = y[0][j][t], b = FOLD ? y[NS - 1][j][t] : 0.0;
    store1<NT>(cr, lane0(j, t), rb[j] + t * st, FOLD ? a + b : a);
    if (FOLD) store1<NT>(cr, lane1(j, t), rb[j] + (BT ? 3 - t : t) * st, a - b);
  };
  // the tile's results with alpha and the added term (all its loads in flight together; a load
  // at kOut gives zero)
  auto write_scaled = [&](auto stream) {
    constexpr bool NT = decltype(stream)::value;
    const double alpha = p.alpha, beta = p.beta;
    double x[NC][4][NS];
#pragma unroll
    for (int j = 0; j < NC; ++j)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        x[j][t][0] = x[j][t][NS - 1] = 0.0;
        if (Cadd) {
          x[j][t][0] = load1(ar, lane0(j, t), rb[j] + t * st);
          if (FOLD) x[j][t][NS - 1] = load1(ar, lane1(j, t), rb[j] + (BT ? 3 - t : t) * st);
        }
      }
#pragma unroll
    for (int j = 0; j < NC; ++j)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const double a = acc[0][j][t], b = FOLD ? acc[NS - 1][j][t] : 0.0;
        const double y0 = alpha * (FOLD ? a + b : a), y1 = alpha * (a - b);
        store1<NT>(cr, lane0(j, t), rb[j] + t * st, Cadd ? y0 + beta * x[j][t][0] : y0);
        if (FOLD) store1<NT>(cr, lane1(j, t), rb[j] + (BT ? 3 - t : t) * st, Cadd ? y1 + beta * x[j][t][NS - 1] : y1);
      }
  };

  // first tile: its loads in flight before the factor's
  double F[NS][2 * H];
  {
    Item q[NI];
    position();
#pragma unroll
    for (int i = 0; i < NI; ++i) load(i, q[i]);
    __builtin_amdgcn_sched_barrier(0);
    // this wave's factor rows for its lifetime
    const int ldf = FOLD ? p.ldf : (BT ? p.lda : p.ldb);
    const double* Fq = FOLD ? p.Ff[g] : (const double*)(BT ? p.A[g] : p.B[g]);
    // (rows past the last feed masked outputs)
    const int row = min(r0 + lr, rows - 1);
#pragma unroll
    for (int q = 0; q < NS; ++q)
#pragma unroll
      for (int h = 0; h < H; ++h) {
        const int k = frag_k<FOLD>(h, lg);
        const double* src = Fq + (int64_t)(row + q * f) * ldf;
        if (FOLD) {   // (row padding is zero up to ldf, an even stride)
          const d2 v = k < ldf ? *reinterpret_cast<const d2*>(src + k) : d2{0.0, 0.0};
          F[q][2 * h] = v.x;
          F[q][2 * h + 1] = v.y;
        } else {   // (pairs past the row are clamped into the factor, its last pair one back)
          const int64_t i = (int64_t)row * ldf + k, last = (int64_t)(rows - 1) * ldf + n - 2, c = i < last ? i : last;
          const d2 v = *reinterpret_cast<const d2u*>(Fq + c);
          F[q][2 * h] = k < n ? (c == i ? v.x : v.y) : 0.0;
          F[q][2 * h + 1] = k + 1 < n ? v.y : 0.0;
        }
      }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int c = 0; c < NP; ++c) store(0, i, c, q[i]);
  }
  __syncthreads();
  // One tile per round. The matrix unit and the vector ALU exclude each other on FP64, and a
  // wave that multiplies keeps a younger wave of its SIMD from issuing anything else until
  // it is done, so separate phases for loads and staging leave the matrix unit idle. They
  // are therefore cut into pieces that stand between the products: the next tile's items
  // are loaded at the first steps and staged at the last ones.
  // Fragment steps e alternate between two register sets: a set is read again right after
  // its products are issued, two steps ahead, so that the products of the other set cover the
  // LDS latency (the scheduling barriers keep this order). With one unit per wave a step is
  // a step block of both tiles, whose products alternate between the two accumulators (a
  // product that follows on its own accumulator waits for it); with more units a step is
  // one tile's part of a block.
  constexpr int NB = NC == 1 ? NS : 1;     // tiles per step
  constexpr int T = NS * H / NB;
  const bool plain_out = p.alpha == 1.0 && !Cadd;
  int cur = 0;
  auto products = [&](auto with_next) {
    constexpr bool MORE = decltype(with_next)::value;
    const double* gs = &Gs[cur][0][0] + (wc * NC * 16 + lr) * PK + 2 * lg;
    d2 x[2][NB][NC];
    Item q[NI];
    auto fetch = [&](int e) {
      const int h = e * NB / NS;
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int j = 0; j < NC; ++j)
          x[e & 1][b][j] =
              *reinterpret_cast<const d2*>(gs + ((e * NB + b) % NS) * TC * PK + j * 16 * PK + 8 * h);
    };
    fetch(0);
    fetch(1);
    if (MORE) position();
#pragma unroll
    for (int t = 0; t < NS; ++t)
#pragma unroll
      for (int j = 0; j < NC; ++j) acc[t][j] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int e = 0; e < T; ++e) {
      const int h = e * NB / NS;
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int j = 0; j < NC; ++j) {
            const int t = (e * NB + b) % NS;
            const double f = F[t][2 * h + s], v = x[e & 1][b][j][s];
            acc[t][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(BT ? f : v, BT ? v : f, acc[t][j], 0, 0, 0);
          }
      __builtin_amdgcn_sched_barrier(0);
      if (e + 2 < T) fetch(e + 2);
      if (MORE) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          if (e == std::min(i, T - 1)) load(i, q[i]);
#pragma unroll
          for (int c = 0; c < NP; ++c)
            if (e == std::max(T - NI * NP + i * NP + c, std::min(i, T - 1))) store(cur ^ 1, i, c, q[i]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    results_of_tile();
  };
  auto write_all = [&]() {
    auto go = [&](auto stream) {
      if (!plain_out) {
        write_scaled(stream);
      } else {
#pragma unroll
        for (int r = 0; r < 4 * NC; ++r) write(acc, r / 4, r % 4, stream);
      }
    };
    if (p.stream_out)
      go(std::true_type{});
    else
      go(std::false_type{});
  };
  int u0 = w * CT;
  if (LATE && ((wave >> 2) & 1)) {
    // the younger wave of a SIMD stores a tile's results at the start of the next round,
    // under the older wave's products, instead of between its own products and the barrier
    bool prev = false;
    for (; u0 + step < units; u0 += step) {
      __builtin_amdgcn_s_setprio(3);
      if (prev) write_all();
      __builtin_amdgcn_s_setprio(0);
      products(std::true_type{});
      prev = true;
      __syncthreads();
      cur ^= 1;
    }
    if (prev) write_all();
  } else {
    for (; u0 + step < units; u0 += step) {
      products(std::true_type{});
      write_all();
      __syncthreads();
      cur ^= 1;
    }
  }
  products(std::false_type{});
  write_all();
}

namespace {

// Workgroup shapes by row tiles RW: WC column waves of NC units and at least WPE waves per
// SIMD (the register budget: 512 / WPE). From five row tiles on, one workgroup per compute
// unit has two or three waves per SIMD (LATE); below, several workgroups share the unit.
// Beyond eight row tiles a wave's factor rows take 144 to 256 registers: one wave per SIMD,
// row groups of four row tiles, each of which reads the grid tile (neighbouring workgroups:
// the second and third time from L2).
template <int FOLD, int H>
struct Shape {
  static constexpr int RT = (H + 1) / 2;   // row tiles of a square factor (folded: of f <= 8H)
  static constexpr int RW = RT > 8 ? 4 : RT;
  static constexpr int WC = RT == 1 ? 4 : RT == 2 || RT == 5 || RT == 6 ? 2 : 1;
  static constexpr int NC = FOLD && (RT == 3 || RT == 4) ? 2 : 1;
  static constexpr int WPE = !FOLD ? 4 : RT > 8 ? 1 : RT >= 7 || RT == 4 ? 2 : RT >= 3 ? 3 : 4;
  static constexpr int LATE = RT >= 5 && RT <= 8;
};

// Outputs are stored past the caches, with two exceptions. Small ones that a tiled product reads
// next: on few tiles its chain of K chunks waits for each load. Along 2700 points after 65 (1.4 MB)
// it takes 98 us on cached values and 118 on streamed ones; along 4000 after 176 (5.6 MB) the
// Lawson-Euler step takes 188 and 206. And large ones in rows that begin and end inside 128-byte
// lines, whose parts would go to memory one by one: an exponential action on 255^3 takes 333 us
// streamed and 269 cached, on 191^3 151 and 125, on 143^3 (23 MB) 71 and 67; 110^3 (11 MB) ETD2RK
// steps 202 and 209, 127^3 254 in either form. Large outputs in whole lines gain nothing from the
// caches (255^3 Lawson2b steps 635 us streamed, 647 cached).
constexpr int64_t kCachedBytes = 6 << 20, kPartialLineBytes = 16 << 20;

template <int BT, int FOLD, int H>
hipError_t launch_regs_h(GemmArgs& g, hipStream_t s) {
  typedef Shape<FOLD, H> S;
  constexpr int CT = S::NC * S::WC;
  const int n = g.K, f = FOLD ? n - n / 2 : n;
  const int rows = FOLD ? f : (BT ? g.M : g.N);
  const int64_t units = (int64_t)(((BT ? g.N : g.M) + 15) / 16) * g.inner;
  const int RG = (rows + 16 * S::RW - 1) / (16 * S::RW);
  const int64_t tiles = (units + CT - 1) / CT;
  // workgroups per compute unit: by waves (WPE per SIMD) and by LDS
  constexpr int lds = 2 * (FOLD ? 2 : 1) * 16 * CT * (8 * H + 4) * 8;
  constexpr int occ = std::max(1, std::min(4 * S::WPE / (S::RW * S::WC), 160 * 1024 / lds));
  const int64_t slots = std::max<int64_t>(1, 256 * occ / (RG * g.groups));
  const int64_t W = std::min(tiles, slots);
  if (units >= ((int64_t)1 << 28)) return hipErrorInvalidValue;
  g.tiles_m = RG;
  g.tiles_n = (int)W;
  g.total = (int)(RG * W * g.groups);
  g.per_xcd = (g.total + 7) / 8;
  const int64_t bytes = 8 * units * 16 * n * g.groups;
  g.stream_out = !(g.chunked_next && bytes <= kCachedBytes) && !(g.ldc % 16 != 0 && bytes > kPartialLineBytes);
  const auto kernel = gemm_f64_regs<BT, FOLD, H, S::RW, S::WC, S::NC, S::WPE, S::LATE>;
  kernel<<<dim3(8 * g.per_xcd), dim3(64 * S::RW * S::WC), 0, s>>>(g);
  return hipGetLastError();
}

template <int BT>
hipError_t launch_fold_bt(GemmArgs& g, hipStream_t s) {
  const int f = g.K - g.K / 2;
  switch ((f + 7) / 8) {
    case 2: return launch_regs_h<BT, 1, 2>(g, s);
    case 3: return launch_regs_h<BT, 1, 3>(g, s);
    case 4: return launch_regs_h<BT, 1, 4>(g, s);
    case 5: return launch_regs_h<BT, 1, 5>(g, s);
    case 6: return launch_regs_h<BT, 1, 6>(g, s);
    case 7: return launch_regs_h<BT, 1, 7>(g, s);
    case 8: return launch_regs_h<BT, 1, 8>(g, s);
    case 9: return launch_regs_h<BT, 1, 9>(g, s);
    case 10: return launch_regs_h<BT, 1, 10>(g, s);
    case 11: return launch_regs_h<BT, 1, 11>(g, s);
    case 12: return launch_regs_h<BT, 1, 12>(g, s);
    case 13: return launch_regs_h<BT, 1, 13>(g, s);
    case 14: return launch_regs_h<BT, 1, 14>(g, s);
    case 15: return launch_regs_h<BT, 1, 15>(g, s);
    case 16: return launch_regs_h<BT, 1, 16>(g, s);
    case 17:
    case 18: return launch_regs_h<BT, 1, 18>(g, s);
    case 19:
    case 20: return launch_regs_h<BT, 1, 20>(g, s);
    case 21:
    case 22: return launch_regs_h<BT, 1, 22>(g, s);
    case 23:
    case 24: return launch_regs_h<BT, 1, 24>(g, s);
    case 25:
    case 26: return launch_regs_h<BT, 1, 26>(g, s);
    case 27:
    case 28: return launch_regs_h<BT, 1, 28>(g, s);
    case 29:
    case 30: return launch_regs_h<BT, 1, 30>(g, s);
    case 31:
    case 32: return launch_regs_h<BT, 1, 32>(g, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

namespace {

// 32-bit byte offsets of the grid operands
bool offsets_fit(const GemmArgs& g) {
  const int64_t lim = (int64_t)1 << 28;   // values
  const int64_t in = g.b_trans ? (g.inner - 1) * g.sB + (int64_t)g.K * g.ldb : (int64_t)g.M * g.lda;
  const int64_t out = g.b_trans ? (g.inner - 1) * g.sC + (int64_t)g.M * g.ldc : (int64_t)g.M * g.ldc;
  return in < lim && out < lim;
}

template <int BT>
hipError_t launch_plain_bt(GemmArgs& g, hipStream_t s) {
  switch ((g.K + 15) / 16) {
    case 2: return launch_regs_h<BT, 0, 4>(g, s);
    case 3: return launch_regs_h<BT, 0, 6>(g, s);
    case 4: return launch_regs_h<BT, 0, 8>(g, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// Plain products of square factors of 17 to 64 points: the tiled kernel walks a serial chain of
// K chunks, each with its load latency on a launch this small; here all of K is loaded at
// once. Up to 16 points the tiled kernel has a single chunk and is no slower (a phi1 action on
// 16^3 by six products and a scaling 18.9 us in a replayed graph, 20.6 with this kernel).
bool plain_regs_fits(const GemmArgs& g) {
  return g.fold_blocks <= 1 && g.K >= 17 && g.K <= 64 && (g.b_trans ? g.M : g.N) == g.K && (!g.b_trans || g.N >= 2) &&
         g.sA == 0 && !g.in_f32 && !g.out_f32 && offsets_fit(g);
}

hipError_t launch_plain_regs(GemmArgs& g, hipStream_t s) {
  return g.b_trans ? launch_plain_bt<1>(g, s) : launch_plain_bt<0>(g, s);
}

// Up to 128 folded positions the register-held kernel is a faster folded one than the tiled
// kernel at every size. Beyond, with one wave per SIMD, it wins where the tiled kernel's
// 128 x 64 tiles do not fill the chip (512 of them): two 511 x 511 vectors 14.5 us per
// product against 22-24 (plain 32-tiles), but 383^3 in unpadded rows 430-495 us against
// 480-505 alone and 5% behind in the ETD2RK step.
constexpr int64_t kWideMaxTiles = 512;

bool fold_regs_fits(const GemmArgs& g) {
  const int n = g.K;
  if (g.fold_blocks > 1 || n < 17 || n > 512 || (g.b_trans && g.N < 2)) return false;
  if (n > 256 && fold_tiles(g) >= kWideMaxTiles) return false;
  return offsets_fit(g);
}

// Where it is the faster one than the plain product. On few units of 16 fibers either kernel is a
// single round of workgroups, and time is a workgroup's own: its factor rows, its first tile and
// its chain. Up to 64 folded positions (and beyond 128: row groups of four waves) the
// register-held kernel is no slower then; with five or six row tiles it takes 10.4-11 us at 144 points
// and 13 at 176 against 10 and 11 of the plain one, until the latter needs further rounds (12.5 and
// 14.3 us at 256 units); with seven or eight 11-12.6 against 12-13.4. Factor rows a multiple of 128
// bytes apart take it another 3-4 us to load (160 points 14.1 against 10.5 us, 191 17.6 against 11.4,
// 224 13.7 against 12.4, 255 16 against 13.1).
constexpr int64_t kNarrowUnits = 192, kNarrowAlignedUnits = 352, kAlignedUnits = 160;

bool fold_regs_pays(const GemmArgs& g, int groups) {
  if (!fold_regs_fits(g)) return false;
  const int f = g.K - g.K / 2;
  if (f <= 64 || f > 128) return true;
  const bool aligned = fold_ld(g.K) % 16 == 0;
  const int64_t least = f <= 96 ? (aligned ? kNarrowAlignedUnits : kNarrowUnits) : aligned ? kAlignedUnits : 0;
  return ((int64_t)((g.b_trans ? g.N : g.M) + 15) / 16) * g.inner * groups >= least;
}

hipError_t launch_fold_regs(GemmArgs& g, hipStream_t s) {
  return g.b_trans ? launch_fold_bt<1>(g, s) : launch_fold_bt<0>(g, s);
}

}  // namespace mm
