// Self-consistent field of the particle step (arXiv:2110.14494: Sec. 2.5
// Poisson's equation and E = -grad phi, Sec. 2.3 boundary conditions,
// Sec. 2.1.4 time step).
//
// * Space charge rho = e (n_+ - n_e - n_-) from the three int64 fixed-point
//   density grids (2^-32 electrons per unit), lap phi = -rho / eps0.
// * phi = 0 on the two z faces (Dirichlet), zero normal derivative on the x
//   and y faces (homogeneous Neumann): 7-point stencil on cell centres with
//   ghost cells (Dirichlet ghost = -phi of the boundary cell, Neumann ghost =
//   phi).  The caller's field is the applied field; the field the electrons
//   see is E_applied - grad phi (central differences, same ghosts).
// * Geometric multigrid as defect correction: the defect of the potential is
//   computed in double precision, the correction solved by one V(2,2) cycle in
//   single precision (red-black Gauss-Seidel smoothing, restriction by the
//   mean of the 8 children, trilinear prolongation with the error's ghost
//   rules, every dimension halved while all are even and above 2, the levels
//   of at most 4096 cells run by one block in LDS) and added to the potential; the
//   iteration converges to the double-precision solution of the discrete
//   system while the cycles move half the bytes.  All passes are
//   HBM-streaming stencils.
// * Time-step ingredients: the 90 % speed quantile by a three-pass radix
//   selection on |v|^2 keys (exact), the densest cell (largest fixed-point
//   density, first in x-fastest order), and the sum of the weights.
#include <hip/hip_runtime.h>

#include <climits>
#include <type_traits>

#include "pcmcc_field.hpp"
#include "pcmcc_internal.hpp"

namespace pcmcc {

namespace {

__device__ __forceinline__ size_t idx3(int i, int j, int k, int nx, int ny) {
  return ((size_t)k * ny + j) * nx + i;
}

// Non-negative doubles compare like their bit patterns.
__device__ __forceinline__ void atomic_max_pos(unsigned long long* a, double v) {
  atomicMax(a, (unsigned long long)__double_as_longlong(v));
}

__device__ __forceinline__ double wave_max(double v) {
  for (int d = 32; d > 0; d >>= 1) v = fmax(v, __shfl_xor(v, d, 64));
  return v;
}

// Largest non-negative value of the block into *a (one atomic per block).
__device__ __forceinline__ void block_max_to(unsigned long long* a, double v) {
  __shared__ double s_w[16];
  v = wave_max(v);
  const int wid = threadIdx.x / 64, nw = (blockDim.x + 63) / 64;
  if ((threadIdx.x & 63) == 0) s_w[wid] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double m = 0.0;
    for (int w = 0; w < nw; ++w) m = fmax(m, s_w[w]);
    if (m > 0.0) atomic_max_pos(a, m);
  }
}

// Sum of the neighbours present and the diagonal of the stencil at (i,j,k):
// a missing x/y neighbour is a Neumann ghost (diagonal 6 -> one less), a
// missing z neighbour a Dirichlet ghost (one more).  The six loads are issued
// together (a missing neighbour reads the cell itself and is then replaced by
// zero) and summed in the order -x, +x, -y, +y, -z, +z.
template <class T>
__device__ __forceinline__ T nb_sum(const T* u, int i, int j, int k, int nx, int ny, int nz, T& diag) {
  const size_t c = idx3(i, j, k, nx, ny);
  const size_t sy = (size_t)nx, sz = (size_t)nx * ny;
  const bool xm = i > 0, xp = i < nx - 1, ym = j > 0, yp = j < ny - 1, zm = k > 0, zp = k < nz - 1;
  const T a = u[xm ? c - 1 : c], b = u[xp ? c + 1 : c];
  const T e = u[ym ? c - sy : c], f = u[yp ? c + sy : c];
  const T g = u[zm ? c - sz : c], h = u[zp ? c + sz : c];
  T s = 0;
  s += xm ? a : T(0);
  s += xp ? b : T(0);
  s += ym ? e : T(0);
  s += yp ? f : T(0);
  s += zm ? g : T(0);
  s += zp ? h : T(0);
  diag = (T)(6 - (int)!xm - (int)!xp - (int)!ym - (int)!yp + (int)!zm + (int)!zp);
  return s;
}

// Storage of a level's u and f.  A level swept by launches (above
// kMgCoarseMax cells, so that every dimension is even) is split by colour:
// the red cells ((i + j + k) even) fill the first half and the black cells the
// second, each in natural order at index c / 2 (c the natural index; nx is
// even, so every pair 2m, 2m + 1 of a row holds one cell of each colour, and
// both are number m of their colour's row).  A half sweep then streams the
// other colour and its own right-hand side: half the bytes of the natural
// layout, and V consecutive cells of a colour have their neighbours in V
// consecutive cells of the other, so a thread takes V of them (4, or 2 or 1
// where nx / 2 is not divisible) with vector loads: five rows, one more cell
// at the end, and the right-hand side for four results, instead of seven
// loads and as many addresses for one (half sweep at 256^3: 30 -> 17.3 us,
// 96 MiB at 5.8 TB/s; 128^3: 8.4 -> 4.1 us).  The levels of the tail kernel are in natural order.
template <int V>
struct Item {
  int j, k, m0;      // row, and the first of the item's V numbers in it
  size_t base, row;  // index of m0 within a colour's half; cells of a colour per row
  size_t plane, half;
  bool in;
};
template <int V>
__device__ __forceinline__ Item<V> item_of(unsigned q, int nx, int ny, int nz) {
  const unsigned nq = (unsigned)nx / (2u * V), row = q / nq;
  Item<V> t;
  t.m0 = (int)(q - row * nq) * V;
  t.k = (int)(row / (unsigned)ny);
  t.j = (int)(row - (unsigned)t.k * (unsigned)ny);
  t.row = (size_t)nx / 2;
  t.plane = t.row * ny;
  t.half = t.plane * nz;
  t.base = (size_t)row * t.row + t.m0;
  t.in = t.k < nz;
  return t;
}

// V consecutive floats (16- or 8-byte aligned for V = 4 and 2).
template <int V>
__device__ __forceinline__ void load_v(const float* p, float (&o)[V]) {
  if constexpr (V == 4) {
    const float4 v = *reinterpret_cast<const float4*>(p);
    o[0] = v.x;
    o[1] = v.y;
    o[2] = v.z;
    o[3] = v.w;
  } else if constexpr (V == 2) {
    const float2 v = *reinterpret_cast<const float2*>(p);
    o[0] = v.x;
    o[1] = v.y;
  } else {
    o[0] = *p;
  }
}
template <int V>
__device__ __forceinline__ void store_v(float* p, const float (&o)[V]) {
  if constexpr (V == 4)
    *reinterpret_cast<float4*>(p) = make_float4(o[0], o[1], o[2], o[3]);
  else if constexpr (V == 2)
    *reinterpret_cast<float2*>(p) = make_float2(o[0], o[1]);
  else
    *p = o[0];
}

// Sum of the neighbours present and the diagonal (as nb_sum) of the item's
// cells of colour `color`; O: the other colour's half.  mid receives the other
// colour's cells of the same row.
template <int V>
__device__ __forceinline__ void nb_sum_v(const float* O, const Item<V>& t, int nx, int ny, int nz, int color,
                                         float (&s)[V], float (&diag)[V], float (&mid)[V]) {
  const int odd = (t.j + t.k + color) & 1;  // the cells are i = 2 m + odd
  const bool ym = t.j > 0, yp = t.j < ny - 1, zm = t.k > 0, zp = t.k < nz - 1;
  float e, f[V], g[V], h[V], l[V];
  load_v(O + t.base, mid);
  // the x neighbour beyond the item's own row cells (a missing one reads a
  // cell of the item and is then replaced by zero)
  const bool xe = odd ? 2 * (t.m0 + V) < nx : t.m0 > 0;
  e = O[odd ? (xe ? t.base + V : t.base) : (xe ? t.base - 1 : t.base)];
  load_v(O + (ym ? t.base - t.row : t.base), f);
  load_v(O + (yp ? t.base + t.row : t.base), g);
  load_v(O + (zm ? t.base - t.plane : t.base), h);
  load_v(O + (zp ? t.base + t.plane : t.base), l);
  e = xe ? e : 0.0f;
#pragma unroll
  for (int q = 0; q < V; ++q) {
    const float a = odd ? mid[q] : (q > 0 ? mid[q > 0 ? q - 1 : 0] : e);
    const float b = odd ? (q < V - 1 ? mid[q < V - 1 ? q + 1 : q] : e) : mid[q];
    float w = 0.0f;
    w += a;
    w += b;
    w += ym ? f[q] : 0.0f;
    w += yp ? g[q] : 0.0f;
    w += zm ? h[q] : 0.0f;
    w += zp ? l[q] : 0.0f;
    s[q] = w;
    const int i = 2 * (t.m0 + q) + odd;
    diag[q] = (float)(6 - (int)!(i > 0) - (int)!(i < nx - 1) - (int)!ym - (int)!yp + (int)!zm + (int)!zp);
  }
}

// Diagonal alone.
__device__ __forceinline__ float diag_at(int i, int j, int k, int nx, int ny, int nz) {
  return (float)(6 - (int)!(i > 0) - (int)!(i < nx - 1) - (int)!(j > 0) - (int)!(j < ny - 1) + (int)!(k > 0) +
                 (int)!(k < nz - 1));
}

// Neighbour sum of one red cell of a split level (the restriction's).
__device__ __forceinline__ float nb_sum_red(const float* u, size_t half, int i, int j, int k, int nx, int ny, int nz,
                                            float& diag) {
  const size_t c = idx3(i, j, k, nx, ny);
  const size_t sy = (size_t)nx, sz = (size_t)nx * ny;
  const float* O = u + half;  // the neighbours are black
  const bool xm = i > 0, xp = i < nx - 1, ym = j > 0, yp = j < ny - 1, zm = k > 0, zp = k < nz - 1;
  const float a = O[(xm ? c - 1 : c) >> 1], b = O[(xp ? c + 1 : c) >> 1];
  const float e = O[(ym ? c - sy : c) >> 1], f = O[(yp ? c + sy : c) >> 1];
  const float g = O[(zm ? c - sz : c) >> 1], h = O[(zp ? c + sz : c) >> 1];
  float s = 0.0f;
  s += xm ? a : 0.0f;
  s += xp ? b : 0.0f;
  s += ym ? e : 0.0f;
  s += yp ? f : 0.0f;
  s += zm ? g : 0.0f;
  s += zp ? h : 0.0f;
  diag = diag_at(i, j, k, nx, ny, nz);
  return s;
}

}  // namespace

// Right-hand side of the finest level and its largest magnitude.
__global__ void k_sc_rhs(const int64_t* __restrict__ np, const int64_t* __restrict__ ne,
                         const int64_t* __restrict__ nn, size_t n, double scale, double* __restrict__ f,
                         unsigned long long* fmax_bits) {
#pragma clang fp contract(off)
  double m = 0.0;
  for (size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x; c < n; c += (size_t)gridDim.x * blockDim.x) {
    const double v = (((double)np[c] - (double)ne[c]) - (double)nn[c]) * scale;
    f[c] = v;
    m = fmax(m, fabs(v));
  }
  block_max_to(fmax_bits, m);
}

// The level kernels are stencils over rows handed out in XCD-local runs
// (xcd_block).

// One red-black Gauss-Seidel half sweep: cells with (i + j + k) % 2 == color.
// kZero: the correction starts from zero (the first red half sweep of a level;
// nothing is read of it, and the black half need not be cleared, since the
// next half sweep writes it from the red one).
template <int V, bool kZero>
__global__ __launch_bounds__(kMgThreads) void k_mg_smooth(float* __restrict__ u, const float* __restrict__ f, int nx,
                                                          int ny, int nz, float h2, int color) {
#pragma clang fp contract(off)
  const Item<V> t = item_of<V>(xcd_block() * kMgThreads + threadIdx.x, nx, ny, nz);
  if (!t.in) return;
  float s[V], d[V], fv[V], r[V];
  const size_t c = (color ? t.half : 0) + t.base;
  load_v(f + c, fv);
  if constexpr (kZero) {
    const int odd = (t.j + t.k + color) & 1;
#pragma unroll
    for (int q = 0; q < V; ++q) {
      s[q] = 0.0f;
      d[q] = diag_at(2 * (t.m0 + q) + odd, t.j, t.k, nx, ny, nz);
    }
  } else {
    float mid[V];
    nb_sum_v(u + (color ? 0 : t.half), t, nx, ny, nz, color, s, d, mid);
  }
#pragma unroll
  for (int q = 0; q < V; ++q) r[q] = (s[q] - h2 * fv[q]) / d[q];
  store_v(u + c, r);
}

// Residual r = f - L u of the 8 children of every coarse cell, averaged into
// the coarse right-hand side.  The restriction follows the pre-smoothing,
// whose last half sweep relaxed the black cells ((i + j + k) odd): their
// residual is zero up to rounding, so only the four red children are summed
// (child offsets 000, 110, 101, 011).  kCoarseSplit: the coarse level is
// swept by launches too.
template <bool kCoarseSplit>
__global__ __launch_bounds__(kRowThreads) void k_mg_restrict(const float* __restrict__ u,
                                                             const float* __restrict__ f, int nx, int ny, int nz,
                                                             float inv_h2, float* __restrict__ fc) {
#pragma clang fp contract(off)
  const size_t half = (size_t)nx * ny * nz / 2;
  const int cx = nx / 2, cy = ny / 2, cz = nz / 2;
  const RowPos P = row_pos(cx, cy);
  const int I = P.x0 + (int)threadIdx.x, J = P.j, K = P.k;
  if (I < cx) {
    float acc = 0.0f;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (((q ^ (q >> 1) ^ (q >> 2)) & 1) != 0) continue;
      const int i = 2 * I + (q & 1), j = 2 * J + ((q >> 1) & 1), k = 2 * K + (q >> 2);
      float d;
      const float s = nb_sum_red(u, half, i, j, k, nx, ny, nz, d);
      const size_t c = idx3(i, j, k, nx, ny) >> 1;
      acc += f[c] - (s - d * u[c]) * inv_h2;
    }
    const size_t C = idx3(I, J, K, cx, cy);
    fc[kCoarseSplit ? (((I + J + K) & 1) ? (size_t)cx * cy * cz / 2 : 0) + (C >> 1) : C] = 0.125f * acc;
  }
}

// Coarse value with the error's ghost rule outside the grid (natural order).
__device__ __forceinline__ float coarse_at(const float* U, int I, int J, int K, int cx, int cy, int cz) {
  float sgn = 1.0f;
  I = min(max(I, 0), cx - 1);
  J = min(max(J, 0), cy - 1);
  if (K < 0) {
    K = 0;
    sgn = -1.0f;
  } else if (K >= cz) {
    K = cz - 1;
    sgn = -1.0f;
  }
  return sgn * U[idx3(I, J, K, cx, cy)];
}

// Coarse cells m0 .. m0 + V - 1 of row (J, K), and the one before or after
// them (`after`), with the ghost rule.
template <int V, bool kCoarseSplit>
__device__ __forceinline__ void coarse_row(const float* U, int m0, bool after, int J, int K, int cx, int cy, int cz,
                                           float (&a)[V], float& e) {
  J = min(max(J, 0), cy - 1);
  const float sgn = K < 0 || K >= cz ? -1.0f : 1.0f;
  K = min(max(K, 0), cz - 1);
  const int me = min(max(after ? m0 + V : m0 - 1, 0), cx - 1);
  const size_t row = ((size_t)K * cy + J) * cx;
  if constexpr (!kCoarseSplit) {
    load_v(U + row + m0, a);
    e = U[row + me];
  } else {
    const size_t half = (size_t)cx * cy * cz / 2;
    const int par = (J + K) & 1;  // parity of the row's cell 0
    if constexpr (V >= 2) {       // m0 is even
      float r[V / 2], b[V / 2];
      load_v(U + ((row + m0) >> 1), r);
      load_v(U + half + ((row + m0) >> 1), b);
#pragma unroll
      for (int q = 0; q < V / 2; ++q) {
        a[2 * q] = par ? b[q] : r[q];
        a[2 * q + 1] = par ? r[q] : b[q];
      }
    } else {
      a[0] = U[((par + m0) & 1 ? half : 0) + ((row + m0) >> 1)];
    }
    e = U[((par + me) & 1 ? half : 0) + ((row + me) >> 1)];
  }
#pragma unroll
  for (int q = 0; q < V; ++q) a[q] = sgn * a[q];
  e = sgn * e;
}

// u_fine += trilinear interpolation of the coarse correction, on the black
// cells only: the red half sweep that follows overwrites the red cells without
// reading them (49 -> 19 us at 256^3).
template <int V, bool kCoarseSplit>
__global__ __launch_bounds__(kMgThreads) void k_mg_prolong(float* __restrict__ u, const float* __restrict__ U, int nx,
                                                           int ny, int nz) {
#pragma clang fp contract(off)
  const Item<V> t = item_of<V>(xcd_block() * kMgThreads + threadIdx.x, nx, ny, nz);
  if (!t.in) return;
  const int cx = nx / 2, cy = ny / 2, cz = nz / 2;
  const int J = t.j >> 1, K = t.k >> 1;
  const int J2 = J + ((t.j & 1) ? 1 : -1), K2 = K + ((t.k & 1) ? 1 : -1);
  const bool after = ((t.j + t.k + 1) & 1) != 0;  // the black cells are i = 2 m + after
  float a0[V], a1[V], a2[V], a3[V], e0, e1, e2, e3, w[V];
  float* p = u + t.half + t.base;
  coarse_row<V, kCoarseSplit>(U, t.m0, after, J, K, cx, cy, cz, a0, e0);
  coarse_row<V, kCoarseSplit>(U, t.m0, after, J2, K, cx, cy, cz, a1, e1);
  coarse_row<V, kCoarseSplit>(U, t.m0, after, J, K2, cx, cy, cz, a2, e2);
  coarse_row<V, kCoarseSplit>(U, t.m0, after, J2, K2, cx, cy, cz, a3, e3);
  load_v(p, w);
  auto next = [&](const float (&a)[V], float e, int q) {  // the column next to q on the cell's side
    return after ? (q < V - 1 ? a[q < V - 1 ? q + 1 : q] : e) : (q > 0 ? a[q > 0 ? q - 1 : 0] : e);
  };
#pragma unroll
  for (int q = 0; q < V; ++q) {
    const float v = 27.0f * a0[q] + 9.0f * (next(a0, e0, q) + a1[q] + a2[q]) +
                    3.0f * (next(a1, e1, q) + next(a2, e2, q) + a3[q]) + next(a3, e3, q);
    w[q] += v * (1.0f / 64.0f);
  }
  store_v(p, w);
}

// The levels of a V(2,2) cycle from the first one of at most kMgCoarseMax
// cells down to the coarsest, run by one block with every level in LDS (the
// same arithmetic as the level kernels; one launch instead of about eleven
// per level).  The coarsest level is solved directly (tail_direct), or by
// `coarse_iters` red-black sweeps.
constexpr int kMgTailCells = 4696;  // >= kMgCoarseMax * (1 + 1/8 + 1/64 + ...)
constexpr int kMgDirectMat = 4096;  // entries of the direct solve's three transform matrices
struct MgTailArgs {
  float* u;        // the first tail level's correction (global; starts at zero)
  const float* f;  // its right-hand side (global)
  int first, levels, coarse_iters;
  int direct;      // 1: the coarsest level is solved directly
  MgDims d[kMgMaxLevels];
  float h2[kMgMaxLevels];
  float inv_h2[kMgMaxLevels];
};

constexpr int kTailThreads = 1024;

// Block-wide barrier, or for a wave on its own the ordering of its LDS
// accesses alone.
template <bool kWave>
__device__ __forceinline__ void tail_sync() {
  if constexpr (kWave) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  } else {
    __syncthreads();
  }
}

// `iters` red-black sweeps of a level of even nx, at most two cells of a
// colour per thread (kWave: one, by one wave).  The neighbours' places, the
// right-hand side and the reciprocal diagonal of a thread's cells are formed
// once for all sweeps; a missing neighbour reads `zero`, a word of LDS that
// holds 0.  x / d is x r, corrected by the exact remainder: the correctly
// rounded quotient, since r is the rounded 1 / d (Markstein), as the plain
// division gives.
template <bool kWave>
__device__ void tail_sweeps(float* u, const float* f, MgDims d, float h2, int iters, int zero) {
#pragma clang fp contract(off)
  constexpr int kR = kWave ? 1 : 2, kN = kWave ? 64 : kTailThreads;
  const int hx = d.nx >> 1, n = d.nx * d.ny * d.nz, nh = n >> 1, plane = d.nx * d.ny;
  int at[2][kR], nb[2][kR][6];
  float hf[2][kR], dg[2][kR], rd[2][kR];
#pragma unroll
  for (int color = 0; color < 2; ++color)
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      const int q = (int)threadIdx.x + r * kN;
      at[color][r] = -1;
      if (q < nh) {
        const int row = q / hx, k = row / d.ny, j = row - k * d.ny;
        const int i = 2 * (q - row * hx) + ((j + k + color) & 1);
        const int c = row * d.nx + i;
        at[color][r] = c;
        nb[color][r][0] = i > 0 ? c - 1 : zero;
        nb[color][r][1] = i < d.nx - 1 ? c + 1 : zero;
        nb[color][r][2] = j > 0 ? c - d.nx : zero;
        nb[color][r][3] = j < d.ny - 1 ? c + d.nx : zero;
        nb[color][r][4] = k > 0 ? c - plane : zero;
        nb[color][r][5] = k < d.nz - 1 ? c + plane : zero;
        hf[color][r] = h2 * f[c];
        dg[color][r] = diag_at(i, j, k, d.nx, d.ny, d.nz);
        rd[color][r] = 1.0f / dg[color][r];
      }
    }
  for (int it = 0; it < iters; ++it)
#pragma unroll
    for (int color = 0; color < 2; ++color) {
#pragma unroll
      for (int r = 0; r < kR; ++r)
        if (at[color][r] >= 0) {
          const int* b = nb[color][r];
          float s = 0.0f;
          s += u[b[0]];
          s += u[b[1]];
          s += u[b[2]];
          s += u[b[3]];
          s += u[b[4]];
          s += u[b[5]];
          const float x = s - hf[color][r];
          const float q = x * rd[color][r];
          u[at[color][r]] = fmaf(fmaf(-dg[color][r], q, x), rd[color][r], q);
        }
      tail_sync<kWave>();
    }
}

// Residual of level (u, f, d) averaged into the coarse right-hand side fc (red
// children only, as in k_mg_restrict), the coarse correction cleared.
template <bool kWave>
__device__ void tail_restrict(const float* u, const float* f, MgDims d, float inv_h2, float* uc, float* fc) {
#pragma clang fp contract(off)
  constexpr int kN = kWave ? 64 : kTailThreads;
  const int cx = d.nx / 2, cy = d.ny / 2, nc = cx * cy * (d.nz / 2);
  for (int C = threadIdx.x; C < nc; C += kN) {
    const int row = C / cx, I = C - row * cx, K = row / cy, J = row - K * cy;
    float acc = 0.0f;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (((q ^ (q >> 1) ^ (q >> 2)) & 1) != 0) continue;
      const int i = 2 * I + (q & 1), j = 2 * J + ((q >> 1) & 1), k = 2 * K + (q >> 2);
      float dg;
      const float s = nb_sum(u, i, j, k, d.nx, d.ny, d.nz, dg);
      const int c = (k * d.ny + j) * d.nx + i;
      acc += f[c] - (s - dg * u[c]) * inv_h2;
    }
    fc[C] = 0.125f * acc;
    uc[C] = 0.0f;
  }
  tail_sync<kWave>();
}

// u += trilinear interpolation of the coarse correction, black cells only (as
// k_mg_prolong).
template <bool kWave>
__device__ void tail_prolong(float* u, MgDims d, const float* U) {
#pragma clang fp contract(off)
  constexpr int kN = kWave ? 64 : kTailThreads;
  const int cx = d.nx / 2, cy = d.ny / 2, cz = d.nz / 2, hx = cx, nh = (d.nx * d.ny * d.nz) >> 1;
  for (int q = threadIdx.x; q < nh; q += kN) {
    const int row = q / hx, k = row / d.ny, j = row - k * d.ny;
    const int I = q - row * hx, i = 2 * I + ((j + k + 1) & 1), J = j >> 1, K = k >> 1;
    const int I2 = I + ((i & 1) ? 1 : -1), J2 = J + ((j & 1) ? 1 : -1), K2 = K + ((k & 1) ? 1 : -1);
    const float v = 27.0f * coarse_at(U, I, J, K, cx, cy, cz) +
                    9.0f * (coarse_at(U, I2, J, K, cx, cy, cz) + coarse_at(U, I, J2, K, cx, cy, cz) +
                            coarse_at(U, I, J, K2, cx, cy, cz)) +
                    3.0f * (coarse_at(U, I2, J2, K, cx, cy, cz) + coarse_at(U, I2, J, K2, cx, cy, cz) +
                            coarse_at(U, I, J2, K2, cx, cy, cz)) +
                    coarse_at(U, I2, J2, K2, cx, cy, cz);
    u[row * d.nx + i] += v * (1.0f / 64.0f);
  }
  tail_sync<kWave>();
}

__device__ void tail_smooth(float* u, const float* f, MgDims d, float h2, int color) {
#pragma clang fp contract(off)
  const int n = d.nx * d.ny * d.nz;
  if ((d.nx & 1) == 0) {  // threads visit the cells of the colour only
    const int hx = d.nx >> 1;
    for (int q = threadIdx.x; q < (n >> 1); q += blockDim.x) {
      const int row = q / hx, j = row % d.ny, k = row / d.ny;
      const int i = 2 * (q - row * hx) + ((j + k + color) & 1);
      const int c = (k * d.ny + j) * d.nx + i;
      float dg;
      const float s = nb_sum(u, i, j, k, d.nx, d.ny, d.nz, dg);
      u[c] = (s - h2 * f[c]) / dg;
    }
  } else {
    for (int c = threadIdx.x; c < n; c += blockDim.x) {
      const int i = c % d.nx, j = (c / d.nx) % d.ny, k = c / (d.nx * d.ny);
      if (((i + j + k) & 1) != color) continue;
      float dg;
      const float s = nb_sum(u, i, j, k, d.nx, d.ny, d.nz, dg);
      u[c] = (s - h2 * f[c]) / dg;
    }
  }
  __syncthreads();
}

// Direct solve of the coarsest level: its stencil is a sum of one-dimensional
// ones whose eigenvectors are known in closed form, cosines cos(pi k (i + 1/2)
// / n) along x and y (Neumann ghosts) and sines sin(pi (k + 1) (i + 1/2) / n)
// along z (Dirichlet ghosts), with eigenvalues -4 sin^2(pi k / 2n) and
// -4 sin^2(pi (k + 1) / 2n).  Three transforms, a division by the summed
// eigenvalues and the three transforms back, in double precision: cells x
// (nx + ny + nz) multiply-adds each way.  Red-black sweeps need some 4 m^2 of
// them for a grid of m cells a side: a 15x11x13 level took 3.4 ms a cycle
// that way (nine tenths of a fluid step on 240x176x208 cells), the whole tail
// kernel takes 23 us with the direct solve.
__device__ void tail_direct(float* u, const float* f, MgDims d, float h2, double* w0, double* w1, double* mat) {
  const int nx = d.nx, ny = d.ny, nz = d.nz, n = nx * ny * nz;
  double *mx = mat, *my = mx + nx * nx, *mz = my + ny * ny;
  for (int e = threadIdx.x; e < nx * nx + ny * ny + nz * nz; e += blockDim.x) {
    const int q = e < nx * nx ? e : (e < nx * nx + ny * ny ? e - nx * nx : e - nx * nx - ny * ny);
    const int m = e < nx * nx ? nx : (e < nx * nx + ny * ny ? ny : nz);
    const bool sine = e >= nx * nx + ny * ny;
    const int k = q / m, i = q - k * m;
    const double a = (double)((sine ? k + 1 : k) * (2 * i + 1)) / (double)(2 * m);
    const bool edge = sine ? k == m - 1 : k == 0;
    mat[e] = (sine ? sinpi(a) : cospi(a)) * sqrt((edge ? 1.0 : 2.0) / (double)m);
  }
  for (int c = threadIdx.x; c < n; c += blockDim.x) w0[c] = (double)f[c];
  __syncthreads();
  // one transform along an axis of length m and stride st: forward, row k of
  // M against the line; back, column i of M
  auto pass = [&](const double* a, double* b, const double* M, int m, int st, bool fwd, auto&& put) {
    for (int c = threadIdx.x; c < n; c += blockDim.x) {
      const int k = (c / st) % m;
      const double* line = a + (c - k * st);
      double s = 0.0;
      for (int i = 0; i < m; ++i) s = fma(fwd ? M[k * m + i] : M[i * m + k], line[i * st], s);
      put(b, c, s);
    }
    __syncthreads();
  };
  auto keep = [](double* b, int c, double s) { b[c] = s; };
  pass(w0, w1, mx, nx, 1, true, keep);
  pass(w1, w0, my, ny, nx, true, keep);
  pass(w0, w1, mz, nz, nx * ny, true, [&](double* b, int c, double s) {
    const int i = c % nx, j = (c / nx) % ny, k = c / (nx * ny);
    const double a = sinpi((double)i / (2 * nx)), e = sinpi((double)j / (2 * ny));
    const double g = sinpi((double)(k + 1) / (2 * nz));
    b[c] = -s * (double)h2 / (4.0 * (a * a + e * e + g * g));
  });
  pass(w1, w0, mz, nz, nx * ny, false, keep);
  pass(w0, w1, my, ny, nx, false, keep);
  pass(w1, w0, mx, nx, 1, false, [&](double*, int c, double s) { u[c] = (float)s; });
}

// From the first level of at most 128 cells on (if the coarsest is swept) one
// wave runs the cycle alone: its LDS accesses need no block barrier, and these
// levels' half sweeps, 48 of 64 for a 16^3 tail, are a chain of latencies
// anyway.  16^3 to 2^3: 44 us with a block barrier and fresh index arithmetic for
// every half sweep and 512 threads, 26 us so.
__global__ __launch_bounds__(kTailThreads) void k_mg_tail(MgTailArgs A) {
#pragma clang fp contract(off)
  __shared__ double s_w[2 * kMgCoarseMax + kMgDirectMat];  // direct solve: two work grids, the matrices
  __shared__ float s_u[kMgTailCells + 1];                  // the last word is zero
  __shared__ float s_f[kMgTailCells];
  __shared__ int off[kMgMaxLevels];  // level offsets in s_u / s_f
  if (threadIdx.x == 0) {
    int o = 0;
    for (int l = A.first; l < A.levels; ++l) {
      off[l] = o;
      o += A.d[l].nx * A.d[l].ny * A.d[l].nz;
    }
    s_u[kMgTailCells] = 0.0f;
  }
  const MgDims d0 = A.d[A.first];
  const int n0 = d0.nx * d0.ny * d0.nz;
  for (int c = threadIdx.x; c < n0; c += kTailThreads) {
    s_u[c] = 0.0f;
    s_f[c] = A.f[c];
  }
  __syncthreads();
  const int last = A.levels - 1;
  auto zero = [&](int l) { return kMgTailCells - off[l]; };  // the zero word, from a level's u
  int wave = A.levels;                                       // first level that one wave runs
  if (!A.direct && (A.d[last].nx & 1) == 0)
    for (wave = A.first; A.d[wave].nx * A.d[wave].ny * A.d[wave].nz > 128 && wave < last;) ++wave;
  if (wave == last && A.d[last].nx * A.d[last].ny * A.d[last].nz > 128) wave = A.levels;
  int l = A.first;
  for (; l < last && l < wave; ++l) {  // down: pre-smoothing, restriction
    tail_sweeps<false>(s_u + off[l], s_f + off[l], A.d[l], A.h2[l], 2, zero(l));
    tail_restrict<false>(s_u + off[l], s_f + off[l], A.d[l], A.inv_h2[l], s_u + off[l + 1], s_f + off[l + 1]);
  }
  if (l == wave) {
    if (threadIdx.x < 64) {
      for (; l < last; ++l) {
        tail_sweeps<true>(s_u + off[l], s_f + off[l], A.d[l], A.h2[l], 2, zero(l));
        tail_restrict<true>(s_u + off[l], s_f + off[l], A.d[l], A.inv_h2[l], s_u + off[l + 1], s_f + off[l + 1]);
      }
      tail_sweeps<true>(s_u + off[last], s_f + off[last], A.d[last], A.h2[last], A.coarse_iters, zero(last));
      for (l = last - 1; l >= wave; --l) {
        tail_prolong<true>(s_u + off[l], A.d[l], s_u + off[l + 1]);
        tail_sweeps<true>(s_u + off[l], s_f + off[l], A.d[l], A.h2[l], 2, zero(l));
      }
    }
    __syncthreads();
    l = wave - 1;
  } else {
    if (A.direct)
      tail_direct(s_u + off[last], s_f + off[last], A.d[last], A.h2[last], s_w, s_w + kMgCoarseMax,
                  s_w + 2 * kMgCoarseMax);
    else
      for (int it = 0; it < A.coarse_iters; ++it)
        for (int color = 0; color < 2; ++color)
          tail_smooth(s_u + off[last], s_f + off[last], A.d[last], A.h2[last], color);
    l = last - 1;
  }
  for (; l >= A.first; --l) {  // up: prolongation, post-smoothing
    tail_prolong<false>(s_u + off[l], A.d[l], s_u + off[l + 1]);
    tail_sweeps<false>(s_u + off[l], s_f + off[l], A.d[l], A.h2[l], 2, zero(l));
  }
  for (int c = threadIdx.x; c < n0; c += kTailThreads) A.u[c] = s_u[c];
}

// Two consecutive cells of a row (nx is even).  kAligned: the caller's potential
// lies on 16 bytes, so that they load as one; it need not.
template <bool kAligned>
__device__ __forceinline__ void load_2(const double* p, double& a, double& b) {
  if constexpr (kAligned) {
    const double2 v = *reinterpret_cast<const double2*>(p);
    a = v.x;
    b = v.y;
  } else {
    a = p[0];
    b = p[1];
  }
}

// The block's largest |defect| to its entry of part.
__device__ __forceinline__ void defect_max(double m, double* part) {
  __shared__ double s_w[kMgThreads / 64];
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) s_w[threadIdx.x / 64] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < (int)blockDim.x / 64; ++w) m = fmax(m, s_w[w]);
    part[blockIdx.x] = m;
  }
}

// Defect of the potential, r = rhs - L phi in double precision: stored in
// single precision as the right-hand side of the correction cycle; a block's
// largest magnitude goes to part[block] (k_max_parts reduces them:
// one same-address atomic per block would serialise in the memory-side
// atomic unit).  A thread takes a pair of cells of a row, one of each colour:
// pairs load as 16 bytes and the lanes of a wave read consecutive ones (108 ->
// 84 us at 256^3 with 268 MB to read; four pairs a thread leave 64-byte strides
// between the lanes, 112 us).
template <bool kAligned>
__global__ __launch_bounds__(kMgThreads) void k_mg_defect(const double* __restrict__ phi,
                                                          const double* __restrict__ rhs, int nx, int ny, int nz,
                                                          double inv_h2, float* __restrict__ r,
                                                          double* __restrict__ part) {
#pragma clang fp contract(off)
  const Item<1> t = item_of<1>(xcd_block() * kMgThreads + threadIdx.x, nx, ny, nz);
  double m = 0.0;
  if (t.in) {
    const size_t c = 2 * t.base, sy = (size_t)nx, sz = (size_t)nx * ny;
    const int i0 = 2 * t.m0;
    const bool ym = t.j > 0, yp = t.j < ny - 1, zm = t.k > 0, zp = t.k < nz - 1;
    const bool xm = i0 > 0, xp = i0 + 2 < nx;
    double p[2], e[2], f[2], g[2], h[2], b[2], v[2];
    load_2<kAligned>(phi + c, p[0], p[1]);
    const double l = phi[xm ? c - 1 : c], n = phi[xp ? c + 2 : c];
    load_2<kAligned>(phi + (ym ? c - sy : c), e[0], e[1]);
    load_2<kAligned>(phi + (yp ? c + sy : c), f[0], f[1]);
    load_2<kAligned>(phi + (zm ? c - sz : c), g[0], g[1]);
    load_2<kAligned>(phi + (zp ? c + sz : c), h[0], h[1]);
    load_2<true>(rhs + c, b[0], b[1]);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      double s = 0.0;
      s += q ? p[0] : (xm ? l : 0.0);
      s += q ? (xp ? n : 0.0) : p[1];
      s += ym ? e[q] : 0.0;
      s += yp ? f[q] : 0.0;
      s += zm ? g[q] : 0.0;
      s += zp ? h[q] : 0.0;
      const double d = (double)diag_at(i0 + q, t.j, t.k, nx, ny, nz);
      v[q] = b[q] - (s - d * p[q]) * inv_h2;
      m = fmax(m, fabs(v[q]));
    }
    const bool odd = ((t.j + t.k) & 1) != 0;  // the pair's first cell is black
    r[t.base] = (float)(odd ? v[1] : v[0]);
    r[t.half + t.base] = (float)(odd ? v[0] : v[1]);
  }
  defect_max(m, part);
}

// The same for a finest level that the tail kernel runs (natural order).
__global__ __launch_bounds__(kMgThreads) void k_mg_defect_natural(const double* __restrict__ phi,
                                                                  const double* __restrict__ rhs, int nx, int ny,
                                                                  int nz, double inv_h2, float* __restrict__ r,
                                                                  double* __restrict__ part) {
#pragma clang fp contract(off)
  const unsigned c = blockIdx.x * kMgThreads + threadIdx.x, n = (unsigned)nx * (unsigned)ny * (unsigned)nz;
  double m = 0.0;
  if (c < n) {
    const int i = (int)(c % (unsigned)nx), j = (int)(c / (unsigned)nx % (unsigned)ny);
    const int k = (int)(c / (unsigned)nx / (unsigned)ny);
    double d;
    const double s = nb_sum(phi, i, j, k, nx, ny, nz, d);
    const double v = rhs[c] - (s - d * phi[c]) * inv_h2;
    r[c] = (float)v;
    m = fabs(v);
  }
  defect_max(m, part);
}

// Largest of n non-negative partial maxima, stored as its bit pattern.
__global__ __launch_bounds__(1024) void k_max_parts(const double* __restrict__ part, unsigned n,
                                                    unsigned long long* out) {
  __shared__ double s_w[16];
  double m = 0.0;
#pragma unroll 8
  for (unsigned q = threadIdx.x; q < n; q += 1024) m = fmax(m, part[q]);
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) s_w[threadIdx.x / 64] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < (int)blockDim.x / 64; ++w) m = fmax(m, s_w[w]);
    *out = (unsigned long long)__double_as_longlong(m);
  }
}

// phi += the correction, with the cycle's last half sweep: the black cells are
// relaxed here, from the red ones, and go into phi without being stored (the
// next cycle starts from zero): 30 + 60 -> 50 us at 256^3.
template <bool kAligned>
__global__ __launch_bounds__(kMgThreads) void k_mg_last(double* __restrict__ phi, const float* __restrict__ u,
                                                        const float* __restrict__ f, int nx, int ny, int nz,
                                                        float h2) {
#pragma clang fp contract(off)
  const Item<1> t = item_of<1>(xcd_block() * kMgThreads + threadIdx.x, nx, ny, nz);
  if (!t.in) return;
  float s[1], d[1], red[1];
  double p[2];
  double* at = phi + 2 * t.base;
  const float fv = f[t.half + t.base];
  load_2<kAligned>(at, p[0], p[1]);
  nb_sum_v(u, t, nx, ny, nz, 1, s, d, red);
  const bool odd = ((t.j + t.k) & 1) != 0;  // the pair's first cell is black
  const float black = (s[0] - h2 * fv) / d[0];
  p[0] += (double)(odd ? black : red[0]);
  p[1] += (double)(odd ? red[0] : black);
  if constexpr (kAligned) {
    *reinterpret_cast<double2*>(at) = make_double2(p[0], p[1]);
  } else {
    at[0] = p[0];
    at[1] = p[1];
  }
}

// phi += the correction in natural order (a finest level that the tail runs).
__global__ void k_mg_correct_natural(double* __restrict__ phi, const float* __restrict__ e, unsigned n) {
  const unsigned c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c < n) phi[c] += (double)e[c];
}

// Start value of the next solve from the last two solutions: phi <- phi +
// r (phi - prev) (linear in time, r the ratio of the coming to the last time
// step), prev <- the old phi.
__global__ void k_extrapolate(double* __restrict__ phi, double* __restrict__ prev, double r, size_t n) {
#pragma clang fp contract(off)
  for (size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x; c < n; c += (size_t)gridDim.x * blockDim.x) {
    const double t = phi[c];
    phi[c] = t + r * (t - prev[c]);
    prev[c] = t;
  }
}

// E = E_applied - grad phi at the centres (central differences with ghosts).
__global__ __launch_bounds__(kRowThreads) void k_sc_field(const float4* __restrict__ Ea, const double* __restrict__ phi,
                                                  int nx, int ny, int nz, double two_dx, float4* __restrict__ E) {
#pragma clang fp contract(off)
  const size_t sy = (size_t)nx, sz = (size_t)nx * ny;
  const RowPos P = row_pos(nx, ny);
  const int i = P.x0 + (int)threadIdx.x, j = P.j, k = P.k;
  if (i < nx) {
    const size_t c = idx3(i, j, k, nx, ny);
    const double p = phi[c];
    const double xm = i > 0 ? phi[c - 1] : p, xp = i < nx - 1 ? phi[c + 1] : p;
    const double ym = j > 0 ? phi[c - sy] : p, yp = j < ny - 1 ? phi[c + sy] : p;
    const double zm = k > 0 ? phi[c - sz] : -p, zp = k < nz - 1 ? phi[c + sz] : -p;
    const float4 a = Ea[c];
    E[c] = make_float4((float)((double)a.x - (xp - xm) / two_dx), (float)((double)a.y - (yp - ym) / two_dx),
                       (float)((double)a.z - (zp - zm) / two_dx), 0.0f);
  }
}

// ---------------------------------------------------------------------------
// Time-step ingredients.

__device__ __forceinline__ uint32_t speed_key(float vx, float vy, float vz) {
#pragma clang fp contract(off)
  const double a = (double)vx, b = (double)vy, c = (double)vz;
  return __float_as_uint((float)((a * a + b * b) + c * c));
}

// Radix-selection pass: histogram of the key bits [shift, shift + bits) of
// the particles whose higher bits equal the state's prefix.
__global__ __launch_bounds__(256) void k_sel_hist(const float* __restrict__ vx, const float* __restrict__ vy,
                                                  const float* __restrict__ vz, const int64_t* n_dev,
                                                  const SelState* st, int shift, int bits,
                                                  unsigned* __restrict__ hist) {
  __shared__ unsigned h[1 << 12];
  const int nb = 1 << bits;
  for (int b = threadIdx.x; b < nb; b += blockDim.x) h[b] = 0;
  __syncthreads();
  const uint64_t n = (uint64_t)*n_dev;
  const int hi = shift + bits;
  const uint32_t want = st->prefix;
  for (uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t key = speed_key(vx[p], vy[p], vz[p]);
    if (hi >= 32 || (key >> hi) == (want >> hi)) atomicAdd(&h[(key >> shift) & (uint32_t)(nb - 1)], 1u);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < nb; b += blockDim.x)
    if (h[b]) atomicAdd(&hist[b], h[b]);
}

// Picks the bin holding the wanted rank (one wave: each lane sums a
// contiguous chunk of bins, a prefix over the lanes finds the chunk, its lane
// the bin); the first pass sets the rank ceil(9 n / 10) from the count.  The
// histogram is cleared for the next pass.
__global__ __launch_bounds__(64) void k_sel_pick(const int64_t* n_dev, unsigned* __restrict__ hist, SelState* st,
                                                 int shift, int bits, int first) {
  const int lane = threadIdx.x;
  const int nb = 1 << bits, per = nb / 64;
  uint64_t rank = first ? ((uint64_t)*n_dev ? (9 * (uint64_t)*n_dev + 9) / 10 : 0) : st->rank;
  uint64_t mine = 0;
  for (int b = lane * per; b < (lane + 1) * per; ++b) mine += hist[b];
  uint64_t incl = mine;
  for (int d = 1; d < 64; d <<= 1) {
    const uint64_t o = __shfl_up(incl, d, 64);
    if (lane >= d) incl += o;
  }
  const uint64_t excl = incl - mine;
  const bool here = rank > 0 && excl < rank && rank <= incl;
  if (here) {
    uint64_t acc = excl;
    for (int b = lane * per; b < (lane + 1) * per; ++b) {
      const uint64_t h = hist[b];
      if (acc + h >= rank) {
        st->prefix = (first ? 0u : st->prefix) | ((uint32_t)b << shift);
        st->rank = rank - acc;
        break;
      }
      acc += h;
    }
  }
  if (lane == 0 && first && rank == 0) {
    st->prefix = 0;
    st->rank = 0;
  }
  __syncthreads();
  for (int b = lane; b < nb; b += 64) hist[b] = 0;
}

// Largest fixed-point electron density, then the first cell holding it.
__global__ void k_ne_max(const int64_t* __restrict__ ne, size_t n, long long* out) {
  __shared__ long long s_w[16];
  long long m = LLONG_MIN;
  for (size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x; c < n; c += (size_t)gridDim.x * blockDim.x)
    m = max(m, (long long)ne[c]);
  for (int d = 32; d > 0; d >>= 1) m = max(m, (long long)__shfl_xor(m, d, 64));
  if ((threadIdx.x & 63) == 0) s_w[threadIdx.x / 64] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < (int)(blockDim.x + 63) / 64; ++w) m = max(m, s_w[w]);
    atomicMax(out, max(m, s_w[0]));
  }
}

__global__ void k_ne_first(const int64_t* __restrict__ ne, size_t n, const long long* mx,
                           unsigned long long* first) {
  const long long m = *mx;
  for (size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x; c < n; c += (size_t)gridDim.x * blockDim.x)
    if ((long long)ne[c] == m) atomicMin(first, (unsigned long long)c);
}

__global__ void k_weight_sum(const float* __restrict__ w, const int64_t* n_dev, double* out) {
  const uint64_t n = (uint64_t)*n_dev;
  double s = 0.0;
  for (uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (uint64_t)gridDim.x * blockDim.x)
    s += (double)w[p];
  for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d, 64);
  if ((threadIdx.x & 63) == 0 && s != 0.0) atomicAdd(out, s);
}

// ---------------------------------------------------------------------------
// Host launchers.


static unsigned grid_for(size_t n, unsigned cap = 16384) {
  const size_t b = (n + 255) / 256;
  return (unsigned)(b < cap ? (b > 0 ? b : 1) : cap);
}

int mg_levels(int nx, int ny, int nz, MgDims* dims) {
  int L = 0;
  dims[L++] = MgDims{nx, ny, nz};
  while (L < kMgMaxLevels && nx % 2 == 0 && ny % 2 == 0 && nz % 2 == 0 && nx > 2 && ny > 2 && nz > 2) {
    nx /= 2;
    ny /= 2;
    nz /= 2;
    dims[L++] = MgDims{nx, ny, nz};
  }
  return L;
}

hipError_t launch_sc_rhs(const int64_t* np, const int64_t* ne, const int64_t* nn, size_t n, double scale, double* f,
                         unsigned long long* fmax, hipStream_t s) {
  hipLaunchKernelGGL(k_sc_rhs, dim3(grid_for(n, 2048)), dim3(256), 0, s, np, ne, nn, n, scale, f, fmax);
  return hipGetLastError();
}

// A level is stored split by colour and swept by launches above
// kMgCoarseMax cells.
static bool split_level(const MgDims& d) { return (size_t)d.nx * d.ny * d.nz > (size_t)kMgCoarseMax; }

static bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

// Cells of a colour per thread of the split kernels.
static int mg_width(int nx) { return nx % 8 == 0 ? 4 : (nx % 4 == 0 ? 2 : 1); }

static unsigned mg_blocks(const MgDims& d, int width) {
  const size_t items = (size_t)(d.nx / (2 * width)) * d.ny * d.nz;
  return (unsigned)((items + kMgThreads - 1) / kMgThreads);
}

size_t defect_blocks(int nx, int ny, int nz) {
  const MgDims d{nx, ny, nz};
  return split_level(d) ? mg_blocks(d, 1) : ((size_t)nx * ny * nz + kMgThreads - 1) / kMgThreads;
}

// Runs body(std::integral_constant<int, V>) for the level's width.
template <class Body>
static void with_width(int nx, Body&& body) {
  switch (mg_width(nx)) {
    case 4: body(std::integral_constant<int, 4>{}); break;
    case 2: body(std::integral_constant<int, 2>{}); break;
    default: body(std::integral_constant<int, 1>{}); break;
  }
}

// One V(2,2) cycle of the correction from level l down (u[l], f[l]: the
// level's single-precision arrays); on a split finest level its last half
// sweep adds the correction to phi.
static hipError_t mg_vcycle(const MgWork& W, int l, hipStream_t s) {
  const MgDims d = W.dims[l];
  const double h = W.dx * (double)(1 << l);
  const float h2 = (float)(h * h);
  if ((size_t)d.nx * d.ny * d.nz <= (size_t)kMgCoarseMax) {
    MgTailArgs A{};
    A.u = W.u[l];
    A.f = W.f[l];
    A.first = l;
    A.levels = W.levels;
    size_t cells = 0;
    for (int q = l; q < W.levels; ++q) {
      cells += (size_t)W.dims[q].nx * W.dims[q].ny * W.dims[q].nz;
      const double hq = W.dx * (double)(1 << q);
      A.d[q] = W.dims[q];
      A.h2[q] = (float)(hq * hq);
      A.inv_h2[q] = 1.0f / A.h2[q];
    }
    const MgDims dl = W.dims[W.levels - 1];
    const int m = dl.nx > dl.ny ? (dl.nx > dl.nz ? dl.nx : dl.nz) : (dl.ny > dl.nz ? dl.ny : dl.nz);
    int iters = 4 * m * m;  // enough red-black sweeps for a grid of m cells a side
    A.coarse_iters = iters < 16 ? 16 : (iters > 4096 ? 4096 : iters);
    // Sweeps stay for the grids of at most 2 cells a side that every power of
    // two ends in (16 sweeps of 8 cells reach rounding in about 4 us) and
    // for a side too long for the matrices in LDS.
    A.direct = m > 2 && dl.nx * dl.nx + dl.ny * dl.ny + dl.nz * dl.nz <= kMgDirectMat;
    if (cells > (size_t)kMgTailCells) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_mg_tail, dim3(1), dim3(kTailThreads), 0, s, A);
    return hipGetLastError();
  }
  const MgDims dc = W.dims[l + 1];
  const bool coarse_split = split_level(dc);
  const dim3 gs(mg_blocks(d, mg_width(d.nx))), bs(kMgThreads);
  with_width(d.nx, [&](auto w) {
    constexpr int V = decltype(w)::value;
    hipLaunchKernelGGL((k_mg_smooth<V, true>), gs, bs, 0, s, W.u[l], W.f[l], d.nx, d.ny, d.nz, h2, 0);
    for (int q = 1; q < 4; ++q)
      hipLaunchKernelGGL((k_mg_smooth<V, false>), gs, bs, 0, s, W.u[l], W.f[l], d.nx, d.ny, d.nz, h2, q & 1);
  });
  const dim3 gr = row_grid(dc.nx, dc.ny, dc.nz);
  if (coarse_split)
    hipLaunchKernelGGL(k_mg_restrict<true>, gr, dim3(kRowThreads), 0, s, W.u[l], W.f[l], d.nx, d.ny, d.nz, 1.0f / h2,
                       W.f[l + 1]);
  else
    hipLaunchKernelGGL(k_mg_restrict<false>, gr, dim3(kRowThreads), 0, s, W.u[l], W.f[l], d.nx, d.ny, d.nz, 1.0f / h2,
                       W.f[l + 1]);
  const hipError_t e = mg_vcycle(W, l + 1, s);
  if (e != hipSuccess) return e;
  with_width(d.nx, [&](auto w) {
    constexpr int V = decltype(w)::value;
    if (coarse_split)
      hipLaunchKernelGGL((k_mg_prolong<V, true>), gs, bs, 0, s, W.u[l], W.u[l + 1], d.nx, d.ny, d.nz);
    else
      hipLaunchKernelGGL((k_mg_prolong<V, false>), gs, bs, 0, s, W.u[l], W.u[l + 1], d.nx, d.ny, d.nz);
    for (int q = 0; q < 3; ++q)
      hipLaunchKernelGGL((k_mg_smooth<V, false>), gs, bs, 0, s, W.u[l], W.f[l], d.nx, d.ny, d.nz, h2, q & 1);
    if (l == 0)
      hipLaunchKernelGGL(aligned16(W.phi) ? k_mg_last<true> : k_mg_last<false>, dim3(mg_blocks(d, 1)), bs, 0, s, W.phi,
                         W.u[0], W.f[0], d.nx, d.ny, d.nz, h2);
    else
      hipLaunchKernelGGL((k_mg_smooth<V, false>), gs, bs, 0, s, W.u[l], W.f[l], d.nx, d.ny, d.nz, h2, 1);
  });
  return hipGetLastError();
}

// One cycle for the defect in f[0], added to the potential.
hipError_t launch_cycle(const MgWork& W, hipStream_t s) {
  const MgDims d = W.dims[0];
  const hipError_t e = mg_vcycle(W, 0, s);
  if (e != hipSuccess || split_level(d)) return e;
  const unsigned n = (unsigned)d.nx * (unsigned)d.ny * (unsigned)d.nz;
  hipLaunchKernelGGL(k_mg_correct_natural, dim3((n + 255) / 256), dim3(256), 0, s, W.phi, W.u[0], n);
  return hipGetLastError();
}

hipError_t launch_defect(const MgWork& W, unsigned long long* rmax, hipStream_t s) {
  const MgDims d = W.dims[0];
  const unsigned nb = (unsigned)defect_blocks(d.nx, d.ny, d.nz);
  const double ih2 = 1.0 / (W.dx * W.dx);
  if (split_level(d))
    hipLaunchKernelGGL(aligned16(W.phi) ? k_mg_defect<true> : k_mg_defect<false>, dim3(nb), dim3(kMgThreads), 0, s,
                       W.phi, W.rhs, d.nx, d.ny, d.nz, ih2, W.f[0], W.part);
  else
    hipLaunchKernelGGL(k_mg_defect_natural, dim3(nb), dim3(kMgThreads), 0, s, W.phi, W.rhs, d.nx, d.ny, d.nz, ih2,
                       W.f[0], W.part);
  hipLaunchKernelGGL(k_max_parts, dim3(1), dim3(1024), 0, s, W.part, nb, rmax);
  return hipGetLastError();
}

hipError_t launch_extrapolate(double* phi, double* prev, double r, size_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_extrapolate, dim3(grid_for(n, 4096)), dim3(256), 0, s, phi, prev, r, n);
  return hipGetLastError();
}

hipError_t launch_sc_field(const float4* Ea, const double* phi, int nx, int ny, int nz, double dx, float4* E,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_sc_field, row_grid(nx, ny, nz), dim3(kRowThreads), 0, s, Ea, phi, nx, ny, nz, 2.0 * dx, E);
  return hipGetLastError();
}

hipError_t launch_speed_select(const float* vx, const float* vy, const float* vz, const int64_t* n_dev, uint64_t n,
                               SelState* st, unsigned* hist, hipStream_t s) {
  const unsigned g = grid_for(n, 1024);
  const int shifts[3] = {20, 8, 0}, bits[3] = {12, 12, 8};
  for (int pass = 0; pass < 3; ++pass) {
    if (pass == 0) {  // the first pick sets the rank; the histogram needs the prefix 0
      hipError_t e = hipMemsetAsync(st, 0, sizeof(SelState), s);
      if (e == hipSuccess) e = hipMemsetAsync(hist, 0, (1u << 12) * sizeof(unsigned), s);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_sel_hist, dim3(g), dim3(256), 0, s, vx, vy, vz, n_dev, st, shifts[pass], bits[pass], hist);
    hipLaunchKernelGGL(k_sel_pick, dim3(1), dim3(64), 0, s, n_dev, hist, st, shifts[pass], bits[pass],
                       pass == 0 ? 1 : 0);
  }
  return hipGetLastError();
}

hipError_t launch_densest(const int64_t* ne, size_t n, long long* mx, unsigned long long* first, hipStream_t s) {
  hipLaunchKernelGGL(k_ne_max, dim3(grid_for(n, 2048)), dim3(256), 0, s, ne, n, mx);
  hipLaunchKernelGGL(k_ne_first, dim3(grid_for(n)), dim3(256), 0, s, ne, n, mx, first);
  return hipGetLastError();
}

hipError_t launch_weight_sum(const float* w, const int64_t* n_dev, uint64_t n, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_weight_sum, dim3(grid_for(n, 2048)), dim3(256), 0, s, w, n_dev, out);
  return hipGetLastError();
}

}  // namespace pcmcc
