// Drift-diffusion-reaction fluid step with the local field approximation
// (arXiv:2110.14494 Sec. 2.2): electrons with Koren-limited advective fluxes
// and central diffusive fluxes, ionization / attachment sources, immobile
// ions, Heun's method with the space-charge field recomputed for the
// predicted densities, and the fluid time-step limits.
//
// * Electrons drift with v = -mu E; flux = v n_face - D (n_R - n_L) / dx;
//   dn_e/dt = -div(flux) + (alpha - eta) mu |E| n_e; positive ions gain
//   alpha mu |E| n_e, negative ions eta mu |E| n_e.
// * Face field = mean of the two cells' field vectors; mu and D from its
//   magnitude; the upwind face density adds half the Koren-limited slope
//   (slope form, psi(r) = max(0, min(2r, (1 + 2r) / 3, 2))).
// * Densities have homogeneous Neumann boundaries as mirror ghost cells
//   (n_-1 = n_0, n_-2 = n_1); a ghost cell's field is the boundary cell's.
// * Transport data: tables of mu N, D N, alpha / N, eta / N on log-spaced E/N
//   nodes, linear in ln(E/N), held constant outside.
// No flux array: one pass over the densities and fields per stage.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "pcmcc_field.hpp"
#include "pcmcc_internal.hpp"

namespace pcmcc {

namespace {

__device__ __forceinline__ int mirror(int i, int m) {
  i = i < 0 ? -i - 1 : (i >= m ? 2 * m - i - 1 : i);
  return min(max(i, 0), m - 1);
}

// Table position of a field of squared magnitude E2: u = (ln(E/N in Td) -
// ln_lo) (n - 1) / ln_span with ln(E/N) = ln(E2) / 2 + ln(1e21 / N), clamped.
// (Reciprocals and logarithms of the constants are precomputed: the kernel
// multiplies where the definition divides, a difference of an ulp or so.)
struct TabPos {
  int i;
  double f;
};
__device__ __forceinline__ TabPos tab_pos(const FluidTab& T, double E2) {
#pragma clang fp contract(off)
  double u = (0.5 * log(fmax(E2, 1e-300)) + T.ln_td - T.ln_lo) * T.pos_scale;
  u = fmin(fmax(u, 0.0), (double)(T.n - 1));
  const int i = min((int)floor(u), T.n - 2);
  return TabPos{i, u - (double)i};
}
__device__ __forceinline__ double tab_at(const TabPos& p, const double* v) {
#pragma clang fp contract(off)
  return (1.0 - p.f) * v[p.i] + p.f * v[p.i + 1];
}

// Koren-limited slope from the upwind slope a and the downwind slope b.
__device__ __forceinline__ double koren(double a, double b) {
#pragma clang fp contract(off)
  if (!(a * b > 0.0)) return 0.0;
  const double aa = fabs(a), ab = fabs(b);
  const double m = fmin(fmin(2.0 * ab, (aa + 2.0 * ab) * (1.0 / 3.0)), 2.0 * aa);
  return a > 0.0 ? m : -m;
}

__device__ __forceinline__ double3 e3(float4 e) { return make_double3((double)e.x, (double)e.y, (double)e.z); }

}  // namespace

// Flux along axis ax through the face between cells L and R.
__device__ __forceinline__ double face_flux(const FluidArgs& A, double nLL, double nL, double nR, double nRR,
                                            const double3& EL, const double3& ER, int ax, double inv_dx) {
#pragma clang fp contract(off)
  const double3 Ef = make_double3(0.5 * (EL.x + ER.x), 0.5 * (EL.y + ER.y), 0.5 * (EL.z + ER.z));
  const TabPos tp = tab_pos(A.T, (Ef.x * Ef.x + Ef.y * Ef.y) + Ef.z * Ef.z);
  const double mu = tab_at(tp, A.T.muN) * A.T.inv_gas_N;
  const double D = tab_at(tp, A.T.DN) * A.T.inv_gas_N;
  const double v = -mu * (ax == 0 ? Ef.x : (ax == 1 ? Ef.y : Ef.z));
  const double up = v >= 0.0 ? nL + 0.5 * koren(nL - nLL, nR - nL) : nR + 0.5 * koren(nR - nRR, nL - nR);
  return v * up - D * (nR - nL) * inv_dx;
}

// That between cells p-1 and p of a row of m cells; n and E point at the
// row's first cell.
__device__ __forceinline__ double face_of_row(const FluidArgs& A, const double* __restrict__ n,
                                              const float4* __restrict__ E, int ax, size_t stride, int p, int m,
                                              double inv_dx) {
  return face_flux(A, n[(size_t)mirror(p - 2, m) * stride], n[(size_t)mirror(p - 1, m) * stride],
                   n[(size_t)mirror(p, m) * stride], n[(size_t)mirror(p + 1, m) * stride],
                   e3(E[(size_t)max(p - 1, 0) * stride]), e3(E[(size_t)min(p, m - 1) * stride]), ax, inv_dx);
}

// One Heun stage on cell c of field Ec, given div(flux).  Stage 1: k1 = F(n0);
// out = n0 + dt k1.  Stage 2: n0 += dt/2 (k1 + F(n_s)) in place (n_s: the
// predicted densities, n_c that of the cell).
__device__ __forceinline__ void stage_cell(const FluidArgs& A, int stage, size_t c, const double3& Ec, double n_c,
                                           double div) {
#pragma clang fp contract(off)
  const double E2 = (Ec.x * Ec.x + Ec.y * Ec.y) + Ec.z * Ec.z;
  const double Emag = sqrt(E2);
  const TabPos tp = tab_pos(A.T, E2);
  const double mu = tab_at(tp, A.T.muN) * A.T.inv_gas_N;
  const double alpha = tab_at(tp, A.T.aN) * A.T.gas_N;
  const double eta = tab_at(tp, A.T.eN) * A.T.gas_N;
  const double rate = mu * Emag * n_c;
  const double ke = -div + (alpha - eta) * rate, kp = alpha * rate, kn = eta * rate;
  if (stage == 1) {
    A.k1e[c] = ke;
    A.k1p[c] = kp;
    A.k1n[c] = kn;
    A.se[c] = A.ne[c] + A.dt * ke;
    A.sp[c] = A.np[c] + A.dt * kp;
    A.sn[c] = A.nn[c] + A.dt * kn;
  } else {
    const double h = 0.5 * A.dt;
    A.ne[c] = A.ne[c] + h * (A.k1e[c] + ke);
    A.np[c] = A.np[c] + h * (A.k1p[c] + kp);
    A.nn[c] = A.nn[c] + h * (A.k1n[c] + kn);
  }
}

// A thread per cell, which forms its six face fluxes (each face twice), rows
// handed out in XCD-local runs.
__global__ __launch_bounds__(kRowThreads) void k_fl_stage(FluidArgs A, int stage) {
#pragma clang fp contract(off)
  const int nx = A.nx, ny = A.ny, nz = A.nz;
  const RowPos P = row_pos(nx, ny);
  const int i = P.x0 + (int)threadIdx.x, j = P.j, k = P.k;
  if (i >= nx) return;
  const double* __restrict__ n = stage == 1 ? A.ne : A.se;
  const size_t c = ((size_t)k * ny + j) * nx + i;
  const double3 Ec = e3(A.E[c]);
  const double inv_dx = 1.0 / A.dx;
  double div = 0.0;
  const int dims[3] = {nx, ny, nz};
  const int pos[3] = {i, j, k};
  const size_t stride[3] = {1, (size_t)nx, (size_t)nx * ny};
  for (int ax = 0; ax < 3; ++ax) {
    const int m = dims[ax], p = pos[ax];
    const size_t base = c - (size_t)p * stride[ax];
    double nv[5];  // cells p-2 .. p+2 along the axis (mirror ghosts)
#pragma unroll
    for (int q = 0; q < 5; ++q) nv[q] = n[base + (size_t)mirror(p - 2 + q, m) * stride[ax]];
    const double3 Em = p > 0 ? e3(A.E[c - stride[ax]]) : Ec;
    const double3 Ep = p < m - 1 ? e3(A.E[c + stride[ax]]) : Ec;
    double fl[2];
#pragma unroll
    for (int side = 0; side < 2; ++side) {  // face between cells (p-1+side) and (p+side)
      fl[side] = face_flux(A, nv[side], nv[side + 1], nv[side + 2], nv[side + 3], side ? Ec : Em, side ? Ep : Ec, ax,
                           inv_dx);
    }
    div += (fl[1] - fl[0]) * inv_dx;
  }
  stage_cell(A, stage, c, Ec, n[c], div);
}

// The same on large grids, where the stage's arrays (90 B a cell) outgrow the
// 256 MB memory-side cache and k_fl_stage, whose neighbours' rows are read by
// other blocks, waits for memory: a wave takes 64 cells of kFlY rows and kFlZ
// planes.  It takes the upper x face of a cell from the next lane (those of
// the last cells from one evaluation for all its rows and planes, a lane
// each), carries the upper z face on to the next plane and the upper y faces,
// through LDS that each lane has for itself, to the next row: 5 evaluations of
// the transport tables a cell instead of 7.  All go through one copy of the
// code (63 registers, 8 waves a SIMD; unrolled 157 registers and 500 us).
// Bound by the chain of loads, logarithm and table loads: without tables and
// logarithms 291 us.  486 -> 390 us for 240 x 176 x 208 cells; 470 -> 320 us
// for 192^3 and 260 -> 190 us for 144^3, but 104 -> 125 us for 128^3: from
// kFlMarchCells on.
constexpr size_t kFlMarchCells = (size_t)5 << 19;
constexpr int kFlY = 2, kFlZ = 4;
__global__ __launch_bounds__(64, 8) void k_fl_march(FluidArgs A, int stage) {
#pragma clang fp contract(off)
  __shared__ double s_y[kFlZ][64];
  const int nx = A.nx, ny = A.ny, nz = A.nz;
  const unsigned L = xcd_block(), tx = (unsigned)((nx + 63) / 64), ty = (unsigned)((ny + kFlY - 1) / kFlY);
  const int lane = threadIdx.x;
  const int x0 = (int)(L % tx) * 64, j0 = (int)(L / tx % ty) * kFlY, k0 = (int)(L / tx / ty) * kFlZ;
  const int i = x0 + lane, j1 = min(ny, j0 + kFlY), k1 = min(nz, k0 + kFlZ);
  const double* __restrict__ n = stage == 1 ? A.ne : A.se;
  const size_t sy = (size_t)nx, sz = (size_t)nx * ny;
  const double inv_dx = 1.0 / A.dx;
  double last_x = 0.0, flz = 0.0;
  if (x0 + 64 <= nx && j0 + lane % kFlY < j1 && k0 + lane / kFlY < k1) {  // lanes of the rows and planes there are
    const size_t r = (size_t)(k0 + lane / kFlY) * sz + (size_t)(j0 + lane % kFlY) * sy;
    last_x = face_of_row(A, n + r, A.E + r, 0, 1, x0 + 64, nx, inv_dx);
  }
  for (int j = j0; j < j1; ++j) {
    for (int k = k0; k < k1; ++k) {
      const size_t r = (size_t)k * sz + (size_t)j * sy, c = r + i;
      double div = 0.0, fly = j > j0 ? s_y[k - k0][lane] : 0.0;
      // faces: lower z and y (first plane and row alone), lower x, upper y, upper z
#pragma unroll 1
      for (int f = k == k0 ? 0 : (j == j0 ? 1 : 2); f < 5; ++f) {
        if (f == 1 && j > j0) continue;
        const int ax = f == 0 || f == 4 ? 2 : (f == 2 ? 0 : 1);
        const int p = f == 0 ? k : (f == 1 ? j : (f == 2 ? i : (f == 3 ? j + 1 : k + 1)));
        const int m = ax == 0 ? nx : (ax == 1 ? ny : nz);
        const size_t stride = ax == 0 ? 1 : (ax == 1 ? sy : sz);
        const size_t first = ax == 0 ? r : (ax == 1 ? (size_t)k * sz + i : (size_t)j * sy + i);
        double fl = 0.0;
        if (i < nx || (i == nx && ax == 0)) fl = face_of_row(A, n + first, A.E + first, ax, stride, p, m, inv_dx);
        if (f == 0) flz = fl;
        if (f == 1) fly = fl;
        if (f == 2) {
          const double next_x = __shfl_down(fl, 1), end_x = __shfl(last_x, (k - k0) * kFlY + j - j0);
          div += ((lane == 63 ? end_x : next_x) - fl) * inv_dx;
        }
        if (f == 3) {
          div += (fl - fly) * inv_dx;
          s_y[k - k0][lane] = fl;
        }
        if (f == 4) {
          div += (fl - flz) * inv_dx;
          flz = fl;
        }
      }
      if (i < nx) {
        stage_cell(A, stage, c, e3(A.E[c]), n[c], div);
      }
    }
  }
}

// Poisson right-hand side from the double densities: -e ((n+ - n_e) - n-) / eps0.
__global__ void k_fl_rhs(const double* __restrict__ np, const double* __restrict__ ne,
                         const double* __restrict__ nn, size_t n, double* __restrict__ f,
                         unsigned long long* fmax_bits) {
#pragma clang fp contract(off)
  __shared__ double s_w[4];
  double m = 0.0;
  for (size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x; c < n; c += (size_t)gridDim.x * blockDim.x) {
    const double q = ((np[c] - ne[c]) - nn[c]) * kFlQe;
    const double v = -q / kFlEps0;
    f[c] = v;
    m = fmax(m, fabs(v));
  }
  for (int d = 32; d > 0; d >>= 1) m = fmax(m, __shfl_xor(m, d, 64));
  if ((threadIdx.x & 63) == 0) s_w[threadIdx.x / 64] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < (int)blockDim.x / 64; ++w) m = fmax(m, s_w[w]);
    if (m > 0.0) atomicMax(fmax_bits, (unsigned long long)__double_as_longlong(m));
  }
}

// Time-step inputs: max of 2 N_dim D / dx^2 + sum |v_i| / dx and of e n mu / eps0.
__global__ __launch_bounds__(256) void k_fl_dt(const double* __restrict__ ne, const float4* __restrict__ E,
                                               size_t n, FluidTab T, double dx, unsigned long long* out) {
#pragma clang fp contract(off)
  __shared__ double s_c[4], s_d[4];
  double mc = 0.0, md = 0.0;
  for (size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x; c < n; c += (size_t)gridDim.x * blockDim.x) {
    const double3 e = e3(E[c]);
    const TabPos tp = tab_pos(T, (e.x * e.x + e.y * e.y) + e.z * e.z);
    const double mu = tab_at(tp, T.muN) * T.inv_gas_N;
    const double D = tab_at(tp, T.DN) * T.inv_gas_N;
    const double cfl = 2.0 * 3.0 * D / (dx * dx) + (mu * ((fabs(e.x) + fabs(e.y)) + fabs(e.z))) / dx;
    const double drt = kFlQe * ne[c] * mu / kFlEps0;
    mc = fmax(mc, cfl);
    md = fmax(md, drt);
  }
  for (int d = 32; d > 0; d >>= 1) {
    mc = fmax(mc, __shfl_xor(mc, d, 64));
    md = fmax(md, __shfl_xor(md, d, 64));
  }
  if ((threadIdx.x & 63) == 0) {
    s_c[threadIdx.x / 64] = mc;
    s_d[threadIdx.x / 64] = md;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < (int)blockDim.x / 64; ++w) {
      mc = fmax(mc, s_c[w]);
      md = fmax(md, s_d[w]);
    }
    if (mc > 0.0) atomicMax(&out[0], (unsigned long long)__double_as_longlong(mc));
    if (md > 0.0) atomicMax(&out[1], (unsigned long long)__double_as_longlong(md));
  }
}

static unsigned fl_blocks(size_t n) {
  const size_t b = (n + 255) / 256;
  return (unsigned)(b < 2048 ? (b > 0 ? b : 1) : 2048);
}

hipError_t launch_fluid_stage(const FluidArgs& A, int stage, hipStream_t s) {
  if ((size_t)A.nx * A.ny * A.nz < kFlMarchCells) {
    hipLaunchKernelGGL(k_fl_stage, row_grid(A.nx, A.ny, A.nz), dim3(kRowThreads), 0, s, A, stage);
    return hipGetLastError();
  }
  const size_t blocks = (size_t)((A.nx + 63) / 64) * (size_t)((A.ny + kFlY - 1) / kFlY) *
                        (size_t)((A.nz + kFlZ - 1) / kFlZ);
  hipLaunchKernelGGL(k_fl_march, dim3((unsigned)blocks), dim3(64), 0, s, A, stage);
  return hipGetLastError();
}

hipError_t launch_fluid_rhs(const double* np, const double* ne, const double* nn, size_t n, double* f,
                            unsigned long long* fmax_bits, hipStream_t s) {
  hipLaunchKernelGGL(k_fl_rhs, dim3(fl_blocks(n)), dim3(256), 0, s, np, ne, nn, n, f, fmax_bits);
  return hipGetLastError();
}

hipError_t launch_fluid_dt(const double* ne, const float4* E, size_t n, const FluidTab& T, double dx,
                           unsigned long long* out, hipStream_t s) {
  hipLaunchKernelGGL(k_fl_dt, dim3(fl_blocks(n)), dim3(256), 0, s, ne, E, n, T, dx, out);
  return hipGetLastError();
}

}  // namespace pcmcc
