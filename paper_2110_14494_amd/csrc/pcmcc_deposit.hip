// Charge deposit (arXiv:2110.14494 Sec. 2.1.3): trilinear weighting of each
// particle's charge to the 8 nearest cell centres.
//
// Fixed-point rule (both paths): weights in double precision without
// contraction, each corner rounded to 2^-32 fixed point and the last corner
// taking the remainder, so the integer sum is independent of order and
// exactly conserves round(w 2^32) per particle.
//
// Range: a particle's charge must fit one corner (0 <= w < 2^31) and every
// cell sum must stay within int64 (2^31 electrons).  Every addition, in LDS
// and in global memory, checks its own signed overflow from the value the
// atomic returns; as the corner charges are non-negative (the remainder
// corner can be a few units below zero) a cell whose sum leaves the range
// overflows in one of them.  Either case raises range_err and drops nothing
// else: the caller reports the error and rho is then unspecified.
//
// Two schedules of the same sums:
//  * direct: one thread per particle, 8 global int64 atomics;
//  * binned (large inputs): the grid is cut into tiles of 8^3 cells, the
//    particles are counted per tile (per-block LDS hash of tiles, one global
//    atomic per block and tile), scattered into tile order (a block reserves
//    its place in each of its tiles with one atomic), and then summed
//    per tile in an LDS int64 buffer of 9^3 cells (the tile plus its upper
//    neighbour layer) that is flushed once per block and tile.  Global
//    atomics drop from 8 per particle to about 8 per thousand particles in
//    dense regions: device-wide int64 atomics are executed at the memory
//    side and were the limit of the direct schedule.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "pcmcc_internal.hpp"

namespace pcmcc {

constexpr int kTile = 8;                                // cells per tile edge
constexpr int kTileBuf = kTile + 1;                     // with the upper neighbour layer
constexpr int kTileCells = kTileBuf * kTileBuf * kTileBuf;
constexpr int kBinThreads = 1024;
constexpr int kBinPer = 8;                              // particles per thread, count and scatter
constexpr int kBinRange = kBinThreads * kBinPer;        // particles per block
constexpr int kSortPer = 16;                            // particles per thread of the particle sort
constexpr int kSortRange = kBinThreads * kSortPer;
constexpr int kScanTile = 4096;                         // tile counts per block of the prefix sum
// Sorted particles per block of the accumulation: an even share over 2^14
// blocks, between the limits (a block's flush costs up to 729 global atomics,
// and few blocks leave the chip idle: with 2^15 particles a block, 9e5
// particles took 485 us in 29 blocks, 142 us so; 2^24 470 and 341, 1e8 1600 and
// 917 us).
constexpr uint32_t kAccMin = 1024, kAccMax = 32768;
static uint32_t acc_range(uint64_t n) {
  const uint64_t r = (n / 16384 + 255) / 256 * 256;
  return (uint32_t)(r < kAccMin ? kAccMin : (r < kAccMax ? r : kAccMax));
}
constexpr uint32_t kEmpty = 0xFFFFFFFFu;

// Lower and upper centre index of one axis, clamped to the grid, and the
// weights (1 - f, f).
__device__ __forceinline__ void dep_axis(double p, double o, double inv_dx, int n, int ic[2], double W[2]) {
#pragma clang fp contract(off)
  double u = (p - o) * inv_dx - 0.5;
  u = fmin(fmax(u, -1.0), (double)n);
  const double fl = floor(u);
  const double f = u - fl;
  const int i = (int)fl;
  ic[0] = min(max(i, 0), n - 1);
  ic[1] = min(max(i + 1, 0), n - 1);
  W[0] = 1.0 - f;
  W[1] = f;
}

// Cells (lower/upper per axis) and fixed-point charges of the 8 corners in
// (dz, dy, dx) order.  A weight outside [0, 2^31) raises range_err and
// deposits nothing.
__device__ __forceinline__ void corner_charges(const DepositGeom& g, float x, float y, float z, float w, int ic[3][2],
                                               long long q[8]) {
#pragma clang fp contract(off)
  double W[3][2];
  dep_axis((double)x, g.x0, g.inv_dx, g.nx, ic[0], W[0]);
  dep_axis((double)y, g.y0, g.inv_dx, g.ny, ic[1], W[1]);
  dep_axis((double)z, g.z0, g.inv_dx, g.nz, ic[2], W[2]);
  double wd = (double)w;
  if (!(wd >= 0.0 && wd < 2147483648.0)) {
    atomicOr(g.range_err, 1u);
    wd = 0.0;
  }
  const long long qw = __double2ll_rn(wd * 4294967296.0);
  long long given = 0;
#pragma unroll
  for (int c = 0; c < 7; ++c) {
    const int dz = c >> 2, dy = (c >> 1) & 1, dx = c & 1;
    const double frac = (W[0][dx] * W[1][dy]) * W[2][dz];
    q[c] = __double2ll_rn((wd * frac) * 4294967296.0);
    given += q[c];
  }
  q[7] = qw - given;
}

__device__ __forceinline__ size_t cell_index(const DepositGeom& g, int i, int j, int k) {
  return ((size_t)k * g.ny + j) * g.nx + i;
}

// rho[i] += v (int64, global or LDS), raising *err on signed overflow.
__device__ __forceinline__ void add_checked(unsigned long long* a, long long v, unsigned* err) {
  const long long old = (long long)atomicAdd(a, (unsigned long long)v);
  const long long res = (long long)((unsigned long long)old + (unsigned long long)v);
  if (((old ^ res) & (v ^ res)) < 0) atomicOr(err, 1u);
}

__global__ void k_deposit(const float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ z,
                          const float* __restrict__ w, const int64_t* n_dev, DepositGeom g,
                          unsigned long long* rho) {
  const uint64_t n = (uint64_t)*n_dev;
  for (uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (uint64_t)gridDim.x * blockDim.x) {
    int ic[3][2];
    long long q[8];
    corner_charges(g, x[p], y[p], z[p], w[p], ic, q);
#pragma unroll
    for (int c = 0; c < 8; ++c)
      add_checked(&rho[cell_index(g, ic[0][c & 1], ic[1][(c >> 1) & 1], ic[2][c >> 2])], q[c], g.range_err);
  }
}

// ---------------------------------------------------------------------------
// Binned schedule.

struct TileGeom {
  DepositGeom g;
  int tx, ty, tz;  // tiles per axis
};

// Tile of a particle: the one holding its lower (clamped) centre indices.
__device__ __forceinline__ uint32_t tile_of(const TileGeom& T, float x, float y, float z) {
  int ic[2];
  double W[2];
  dep_axis((double)x, T.g.x0, T.g.inv_dx, T.g.nx, ic, W);
  const int i = ic[0] / kTile;
  dep_axis((double)y, T.g.y0, T.g.inv_dx, T.g.ny, ic, W);
  const int j = ic[0] / kTile;
  dep_axis((double)z, T.g.z0, T.g.inv_dx, T.g.nz, ic, W);
  const int k = ic[0] / kTile;
  return ((uint32_t)k * T.ty + j) * T.tx + i;
}

// A block's table of tiles in LDS: open addressing over N = 2^k entries, at
// least as many as the block has particles, so it never fills.
template <int N>
struct TileTable {
  uint32_t key[N];
  uint32_t cnt[N];
};

template <int N>
__device__ __forceinline__ void table_clear(TileTable<N>& H) {
  for (int e = threadIdx.x; e < N; e += kBinThreads) {
    H.key[e] = kEmpty;
    H.cnt[e] = 0;
  }
}

// Entry of tile t, inserting it if new.
template <int N>
__device__ __forceinline__ uint32_t table_insert(TileTable<N>& H, uint32_t t) {
  uint32_t h = (t * 2654435761u) >> (32 - __builtin_ctz(N));
  for (;;) {
    const uint32_t old = atomicCAS(&H.key[h], kEmpty, t);
    if (old == kEmpty || old == t) return h;
    h = (h + 1) & (N - 1);
  }
}

// Counts tile t in (lanes with `valid`); returns the particle's entry and its
// number within it.  Where many lanes hold the first lane's tile (particles
// that come in tile order), they take one insertion and one addition
// together: 64 lanes on one LDS word are served one after the other.
template <int N>
__device__ __forceinline__ uint2 table_count(TileTable<N>& H, uint32_t t, bool valid) {
  const uint64_t act = __ballot(valid);
  if (act == 0) return make_uint2(0u, 0u);
  const int lane = (int)__lane_id(), lead = __ffsll((unsigned long long)act) - 1;
  const uint32_t t0 = (uint32_t)__builtin_amdgcn_readlane((int)t, lead);
  const uint64_t same = __ballot(valid && t == t0);
  uint2 r = make_uint2(0u, 0u);
  if (__popcll(same) >= 8) {
    if (lane == lead) {
      r.x = table_insert(H, t0);
      r.y = atomicAdd(&H.cnt[r.x], (uint32_t)__popcll(same));
    }
    const uint32_t e = (uint32_t)__builtin_amdgcn_readlane((int)r.x, lead);
    const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)r.y, lead);
    const uint32_t below = __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u);
    r = make_uint2(e, b + __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), below));
    valid = valid && !((same >> lane) & 1);
  }
  if (valid) {
    const uint32_t e = table_insert(H, t);
    r = make_uint2(e, atomicAdd(&H.cnt[e], 1u));
  }
  return r;
}

// Pass 1: particles per tile; block b covers [b kBinRange, (b + 1) kBinRange).
__global__ __launch_bounds__(kBinThreads) void k_dep_count(const float* __restrict__ x, const float* __restrict__ y,
                                                           const float* __restrict__ z, uint64_t n, TileGeom T,
                                                           uint32_t* __restrict__ tile_count) {
  __shared__ TileTable<kBinRange> H;
  table_clear(H);
  __syncthreads();
  const uint64_t p0 = (uint64_t)blockIdx.x * kBinRange + threadIdx.x;
#pragma unroll 2
  for (int q = 0; q < kBinPer; ++q) {
    const uint64_t p = p0 + (uint64_t)q * kBinThreads;
    const bool valid = p < n;
    (void)table_count(H, valid ? tile_of(T, x[p], y[p], z[p]) : 0u, valid);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < kBinRange; e += kBinThreads)
    if (H.key[e] != kEmpty) atomicAdd(&tile_count[H.key[e]], H.cnt[e]);
}

// Exclusive prefix sum of the tile counts: start[t] and start[n_tiles] = the
// total; the counts become the tiles' write positions (equal to start).  Two
// launches: sums of kScanTile counts each, then every block adds the sums
// before its own (one block for 2^18 tiles took 445 us, these two 8).
__global__ __launch_bounds__(kBinThreads) void k_dep_sums(const uint32_t* __restrict__ count, uint32_t n_tiles,
                                                          uint32_t* __restrict__ sums) {
  __shared__ uint32_t s_w[kBinThreads / 64];
  const uint32_t a = blockIdx.x * kScanTile + threadIdx.x * 4;
  uint32_t s = 0;
  for (uint32_t t = a; t < a + 4; ++t) s += t < n_tiles ? count[t] : 0u;
  for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d, 64);
  if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0;
    for (int w = 0; w < kBinThreads / 64; ++w) t += s_w[w];
    sums[blockIdx.x] = t;
  }
}

__global__ __launch_bounds__(kBinThreads) void k_dep_scan(uint32_t* __restrict__ count, uint32_t n_tiles,
                                                          const uint32_t* __restrict__ sums,
                                                          uint32_t* __restrict__ start) {
  __shared__ uint32_t s_w[kBinThreads / 64], s_before;
  const int lane = (int)__lane_id(), wave = (int)(threadIdx.x >> 6);
  uint32_t b = 0;
  for (uint32_t q = threadIdx.x; q < blockIdx.x; q += kBinThreads) b += sums[q];
  for (int d = 32; d > 0; d >>= 1) b += __shfl_xor(b, d, 64);
  if (lane == 0) s_w[wave] = b;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0;
    for (int w = 0; w < kBinThreads / 64; ++w) t += s_w[w];
    s_before = t;
  }
  __syncthreads();
  const uint32_t a = blockIdx.x * kScanTile + threadIdx.x * 4;
  uint32_t c[4], s = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    c[q] = a + q < n_tiles ? count[a + q] : 0u;
    s += c[q];
  }
  uint32_t incl = s;
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = __shfl_up(incl, d, 64);
    if (lane >= d) incl += o;
  }
  if (lane == 63) s_w[wave] = incl;
  __syncthreads();
  uint32_t run = s_before + incl - s;
  for (int w = 0; w < wave; ++w) run += s_w[w];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (a + q < n_tiles) {
      start[a + q] = run;
      count[a + q] = run;
      run += c[q];
      if (a + q == n_tiles - 1) start[n_tiles] = run;
    }
  }
}

// Pass 2: scatter (x, y, z, w) into tile order.  pos: the tiles' write
// positions, advanced by each block by its particles of the tile.
__global__ __launch_bounds__(kBinThreads) void k_dep_scatter(const float* __restrict__ x, const float* __restrict__ y,
                                                             const float* __restrict__ z, const float* __restrict__ w,
                                                             uint64_t n, TileGeom T, uint32_t* __restrict__ pos,
                                                             float4* __restrict__ sorted) {
  __shared__ TileTable<kBinRange> H;
  table_clear(H);
  __syncthreads();
  const uint64_t p0 = (uint64_t)blockIdx.x * kBinRange + threadIdx.x;
  float4 v[kBinPer];
  uint2 er[kBinPer];
#pragma unroll
  for (int q = 0; q < kBinPer; ++q) {
    const uint64_t p = p0 + (uint64_t)q * kBinThreads;
    const bool valid = p < n;
    v[q] = valid ? make_float4(x[p], y[p], z[p], w[p]) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    er[q] = table_count(H, valid ? tile_of(T, v[q].x, v[q].y, v[q].z) : 0u, valid);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < kBinRange; e += kBinThreads)
    if (H.key[e] != kEmpty) H.cnt[e] = atomicAdd(&pos[H.key[e]], H.cnt[e]);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kBinPer; ++q)
    if (p0 + (uint64_t)q * kBinThreads < n) sorted[H.cnt[er[q].x] + er[q].y] = v[q];
}

// Particle sort by tile (the step loop's start order): the count and scan
// passes above, then every array of a particle moved to its tile's range.
// Within a tile the order follows the atomics and is not fixed.
//
// A block brings its 2^14 particles into tile order in LDS, one array after
// the other, and writes them from there, so that the particles a block has of
// one tile leave as one run of consecutive words (12 particles of an
// unordered streamer head on 512^3 cells).  Each lane writing its own
// particle's eight words from a block of 2^12 left a partly written line per
// word: 8.6 ms for 2^26 particles (72 bytes each: 0.9 ms at the HBM rate),
// 2.5 ms so.
struct SortLds {
  union {
    TileTable<kSortRange> H;
    struct {
      uint32_t val[kSortRange];
      uint32_t dst[kSortRange];
    } out;
  };
  uint32_t wave_sum[kBinThreads / 64];
};

__global__ __launch_bounds__(kBinThreads) void k_sort_scatter(Soa src, uint64_t n, TileGeom T,
                                                              uint32_t* __restrict__ pos, Soa dst) {
  __shared__ SortLds S;
  table_clear(S.H);
  __syncthreads();
  const uint64_t b0 = (uint64_t)blockIdx.x * kSortRange, p0 = b0 + threadIdx.x;
  const uint32_t m = (uint32_t)(n - b0 < (uint64_t)kSortRange ? n - b0 : (uint64_t)kSortRange);
  uint2 er[kSortPer];
#pragma unroll
  for (int q = 0; q < kSortPer; ++q) {
    const uint64_t p = p0 + (uint64_t)q * kBinThreads;
    const bool valid = p < n;
    er[q] = table_count(S.H, valid ? tile_of(T, src.x[p], src.y[p], src.z[p]) : 0u, valid);
  }
  __syncthreads();
  // the entries' first ranks in the block (in table order) and their places in
  // the tiles' ranges
  const int lane = (int)__lane_id(), wave = (int)(threadIdx.x >> 6);
  const int e0 = (int)threadIdx.x * kSortPer;
  uint32_t sum = 0;
#pragma unroll
  for (int q = 0; q < kSortPer; ++q) sum += S.H.cnt[e0 + q];
  uint32_t incl = sum;
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = __shfl_up(incl, d, 64);
    if (lane >= d) incl += o;
  }
  if (lane == 63) S.wave_sum[wave] = incl;
  __syncthreads();
  uint32_t run = incl - sum;
  for (int w = 0; w < wave; ++w) run += S.wave_sum[w];
#pragma unroll 4
  for (int q = 0; q < kSortPer; ++q) {
    const uint32_t t = S.H.key[e0 + q], c = S.H.cnt[e0 + q];
    if (t != kEmpty) {
      S.H.key[e0 + q] = atomicAdd(&pos[t], c);
      S.H.cnt[e0 + q] = run;
      run += c;
    }
  }
  __syncthreads();
  // each particle's rank in the block and its destination
  uint32_t rank[kSortPer], to[kSortPer];
#pragma unroll
  for (int q = 0; q < kSortPer; ++q) {
    rank[q] = S.H.cnt[er[q].x] + er[q].y;
    to[q] = S.H.key[er[q].x] + er[q].y;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kSortPer; ++q)
    if (p0 + (uint64_t)q * kBinThreads < n) S.out.dst[rank[q]] = to[q];
  // one 4-byte array at a time (an id's two halves likewise)
  auto move = [&](const uint32_t* from, uint32_t* into, int stride, int half) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSortPer; ++q) {
      const uint64_t p = p0 + (uint64_t)q * kBinThreads;
      if (p < n) S.out.val[rank[q]] = from[p * stride + half];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSortPer; ++q) {
      const uint32_t r = threadIdx.x + q * kBinThreads;
      if (r < m) into[(size_t)S.out.dst[r] * stride + half] = S.out.val[r];
    }
  };
  const float* const f[7] = {src.x, src.y, src.z, src.vx, src.vy, src.vz, src.w};
  float* const t[7] = {dst.x, dst.y, dst.z, dst.vx, dst.vy, dst.vz, dst.w};
#pragma unroll 1
  for (int a = 0; a < 7; ++a)
    move(reinterpret_cast<const uint32_t*>(f[a]), reinterpret_cast<uint32_t*>(t[a]), 1, 0);
#pragma unroll 1
  for (int h = 0; h < 2; ++h) move(reinterpret_cast<const uint32_t*>(src.id), reinterpret_cast<uint32_t*>(dst.id), 2, h);
}

// One tile run [cur, e) of sorted particles into the LDS buffer of the tile
// at (oi, oj, ok).  The plain pass adds without overflow checks (it cannot
// overflow while the run carries fewer than 2^31 electrons, which the caller
// checks with the returned weight sum) and sends a corner outside the buffer
// to rho directly; the checked pass repeats only the LDS part.
template <bool kChecked>
__device__ __forceinline__ double accum_run(const float4* __restrict__ sorted, uint64_t cur, uint64_t e,
                                            const TileGeom& T, int oi, int oj, int ok, unsigned long long* acc,
                                            unsigned long long* rho) {
  double wsum = 0.0;
  for (uint64_t p = cur + threadIdx.x; p < e; p += blockDim.x) {
    const float4 v = sorted[p];
    int ic[3][2];
    long long q[8];
    corner_charges(T.g, v.x, v.y, v.z, v.w, ic, q);
    if (v.w >= 0.0f) wsum += (double)v.w;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const int ci = ic[0][c & 1], cj = ic[1][(c >> 1) & 1], ck = ic[2][c >> 2];
      const int li = ci - oi, lj = cj - oj, lk = ck - ok;
      if ((unsigned)li < (unsigned)kTileBuf && (unsigned)lj < (unsigned)kTileBuf && (unsigned)lk < (unsigned)kTileBuf) {
        unsigned long long* a = &acc[(lk * kTileBuf + lj) * kTileBuf + li];
        if (kChecked)
          add_checked(a, q[c], T.g.range_err);
        else
          atomicAdd(a, (unsigned long long)q[c]);
      } else if (!kChecked) {  // a particle outside its tile's buffer: never expected, kept exact
        add_checked(&rho[cell_index(T.g, ci, cj, ck)], q[c], T.g.range_err);
      }
    }
  }
  return wsum;
}

// A tile run carrying this many electrons or more is summed again with
// overflow checks (2^31 electrons is the int64 limit of one cell).
constexpr double kAccGuard = 1073741824.0;

// Pass 3: per-tile sums.  Block b covers sorted particles
// [b range, (b + 1) range), one tile at a time.
__global__ __launch_bounds__(256) void k_dep_accum(const float4* __restrict__ sorted, uint64_t n, uint32_t range,
                                                    TileGeom T, const uint32_t* __restrict__ start,
                                                    unsigned long long* rho) {
  __shared__ unsigned long long acc[kTileCells];
  __shared__ uint32_t s_tile;
  __shared__ uint64_t s_end;
  __shared__ double s_wsum;
  for (int c = threadIdx.x; c < kTileCells; c += blockDim.x) acc[c] = 0;
  uint64_t cur = (uint64_t)blockIdx.x * range;
  const uint64_t end = cur + range < n ? cur + range : n;
  while (cur < end) {
    if (threadIdx.x == 0) {
      const float4 q = sorted[cur];
      const uint32_t t = tile_of(T, q.x, q.y, q.z);
      s_tile = t;
      // the run of tile t ends at start[t + 1] (at least one particle on)
      uint64_t te = start[t + 1];
      te = te > cur ? te : cur + 1;
      s_end = te < end ? te : end;
      s_wsum = 0.0;
    }
    __syncthreads();
    const uint32_t t = s_tile;
    const uint64_t e = s_end;
    const int oi = (int)(t % T.tx) * kTile;
    const int oj = (int)((t / T.tx) % T.ty) * kTile;
    const int ok = (int)(t / ((uint32_t)T.tx * T.ty)) * kTile;
    const double ws = accum_run<false>(sorted, cur, e, T, oi, oj, ok, acc, rho);
    if (ws > 0.0) atomicAdd(&s_wsum, ws);
    __syncthreads();
    if (s_wsum >= kAccGuard) {  // block-uniform
      for (int c = threadIdx.x; c < kTileCells; c += blockDim.x) acc[c] = 0;
      __syncthreads();
      accum_run<true>(sorted, cur, e, T, oi, oj, ok, acc, rho);
    }
    __syncthreads();
    for (int c = threadIdx.x; c < kTileCells; c += blockDim.x) {
      const unsigned long long v = acc[c];
      if (v != 0) {
        const int ci = oi + c % kTileBuf, cj = oj + (c / kTileBuf) % kTileBuf, ck = ok + c / (kTileBuf * kTileBuf);
        if (ci < T.g.nx && cj < T.g.ny && ck < T.g.nz)
          add_checked(&rho[cell_index(T.g, ci, cj, ck)], (long long)v, T.g.range_err);
        acc[c] = 0;
      }
    }
    __syncthreads();
    cur = e;
  }
}

// ---------------------------------------------------------------------------

// Sets n words to v (a kernel rather than a memset node, so that the deposit
// may be recorded into a graph).
__global__ void k_fill_u32(uint32_t* __restrict__ p, uint64_t n, uint32_t v) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

hipError_t launch_fill_u32(uint32_t* p, uint64_t n, uint32_t v, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  const uint64_t blocks = std::min<uint64_t>((n + 255) / 256, 1024);
  hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, stream, p, n, v);
  return hipGetLastError();
}

hipError_t launch_deposit(const float* x, const float* y, const float* z, const float* w, const int64_t* n_dev,
                          const DepositGeom& g, int64_t* rho, hipStream_t stream) {
  hipLaunchKernelGGL(k_deposit, dim3(4096), dim3(256), 0, stream, x, y, z, w, n_dev, g,
                     (unsigned long long*)rho);
  return hipGetLastError();
}

DepositNeeds deposit_needs(const DepositGeom& g, uint64_t n) {
  DepositNeeds d;
  d.binned = n >= kDepositBinnedMin;
  const uint64_t tx = ((uint64_t)g.nx + kTile - 1) / kTile, ty = ((uint64_t)g.ny + kTile - 1) / kTile,
                 tz = ((uint64_t)g.nz + kTile - 1) / kTile;
  d.n_tiles = tx * ty * tz;
  d.scan_sums = (d.n_tiles + kScanTile - 1) / kScanTile;
  d.sorted = n;
  return d;
}

// Tile geometry of g, the particles of (x, y, z) counted per tile and the
// counts turned into starts and write positions.
static hipError_t count_tiles(const float* x, const float* y, const float* z, uint64_t n, const DepositGeom& g,
                              const DepositWork& W, TileGeom& T, hipStream_t stream) {
  T.g = g;
  T.tx = (g.nx + kTile - 1) / kTile;
  T.ty = (g.ny + kTile - 1) / kTile;
  T.tz = (g.nz + kTile - 1) / kTile;
  const uint32_t n_tiles = (uint32_t)T.tx * T.ty * T.tz;
  hipError_t e = launch_fill_u32(W.tile_count, n_tiles, 0u, stream);
  if (e != hipSuccess) return e;
  const dim3 nb((unsigned)((n + kBinRange - 1) / kBinRange)), ns((n_tiles + kScanTile - 1) / kScanTile);
  hipLaunchKernelGGL(k_dep_count, nb, dim3(kBinThreads), 0, stream, x, y, z, n, T, W.tile_count);
  hipLaunchKernelGGL(k_dep_sums, ns, dim3(kBinThreads), 0, stream, W.tile_count, n_tiles, W.tile_start + n_tiles + 1);
  hipLaunchKernelGGL(k_dep_scan, ns, dim3(kBinThreads), 0, stream, W.tile_count, n_tiles, W.tile_start + n_tiles + 1,
                     W.tile_start);
  return hipGetLastError();
}

hipError_t launch_sort_tiles(const Soa& src, uint64_t n, const DepositGeom& g, const DepositWork& W, const Soa& dst,
                             hipStream_t stream) {
  if (n == 0) return hipSuccess;
  TileGeom T;
  const hipError_t e = count_tiles(src.x, src.y, src.z, n, g, W, T, stream);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_sort_scatter, dim3((unsigned)((n + kSortRange - 1) / kSortRange)), dim3(kBinThreads), 0, stream,
                     src, n, T, W.tile_count, dst);
  return hipGetLastError();
}

hipError_t launch_deposit_binned(const float* x, const float* y, const float* z, const float* w, uint64_t n,
                                 const DepositGeom& g, int64_t* rho, const DepositWork& W, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  TileGeom T;
  const hipError_t e = count_tiles(x, y, z, n, g, W, T, stream);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_dep_scatter, dim3((unsigned)((n + kBinRange - 1) / kBinRange)), dim3(kBinThreads), 0, stream, x,
                     y, z, w, n, T, W.tile_count, W.sorted);
  const uint32_t range = acc_range(n);
  hipLaunchKernelGGL(k_dep_accum, dim3((unsigned)((n + range - 1) / range)), dim3(256), 0, stream, W.sorted, n, range,
                     T, W.tile_start, (unsigned long long*)rho);
  return hipGetLastError();
}

}  // namespace pcmcc
