// Coefficient surrogate: a 1 -> 64 -> 64 -> 6 perceptron (tanh hidden
// layers) that maps standardised ln(E/N) to standardised log swarm
// coefficients (the inputs of the fluid model of arXiv:2110.14494 Sec. 2.2,
// computed by the swarms of Sec. 2.2.2).
//
//  * training (FP32): forward and backward over 16-point tiles held in LDS,
//    gradients reduced in a fixed order (bit-reproducible), full-batch Adam
//    with a cosine learning rate; one cooperative launch runs every epoch;
//  * inference (BF16 weights and activations, FP32 accumulation): the 64x64
//    layer and the output layer run on MFMA (v_mfma_f32_32x32x16_bf16); the
//    first layer is computed per lane straight into the MFMA operand layout;
//    a hidden activation is carried as s = (1 + tanh z) / 2, the logistic
//    function of 2 z, which the next layer absorbs into its bias;
//    the outputs flagged for a point's E/N cell fall back to interpolation
//    of the swarm table.
// Parameter vector (4678 floats): W1[64,1], b1[64], W2[64,64], b2[64],
// W3[6,64], b3[6], row-major.
#include <hip/hip_runtime.h>

#include "pcmcc_internal.hpp"

namespace pcmcc {

constexpr int kH = 64, kOut = 6;
constexpr unsigned kAllOut = (1u << kOut) - 1u;  // fallback mask with every output
constexpr int OFF_W1 = 0, OFF_B1 = 64, OFF_W2 = 128, OFF_B2 = 128 + 4096, OFF_W3 = OFF_B2 + 64,
              OFF_B3 = OFF_W3 + 384;
static_assert(OFF_B3 + 6 == kMlpParams, "parameter packing");

// ---------------------------------------------------------------------------
// Training: one tile of kTile points through forward and backward.  The three
// 64-wide products (layer 2, its input gradient, its weight gradient) run on
// register tiles: a thread holds kRP x 4 (or 4 x 4) outputs and reads its two
// operands as vectors from LDS copies laid out so that the lanes of a wave
// read consecutive words; the operands are therefore kept in both orders.
// Everything is in a fixed order, so results are reproducible.  Bound by
// latency: the stages of a tile depend on each other, and one block a compute
// unit runs each as a few hundred instructions.  A thread per output
// reading two LDS words per multiply-add, the layer's weights with all lanes
// on one bank, and 64-point tiles took 163 us an epoch for 1792 points (28
// blocks); 32-point tiles of this form take 33 us (56 blocks, 17.6 us of
// it the tile, 5.2 the parameters, 9.8 the reduction and two barriers), and
// 16-point tiles 27 us (112 blocks), 24.5 us since the compiler knows the
// vector loads' alignment.
constexpr int kTile = kMlpTile, kTP = kTile + 4;
constexpr int kRP = kTile / 16;  // points of a thread's register tile
struct alignas(16) MlpLds {  // W2, W2T, H1 and D2 are read four floats at a time
  float W2[kH][kH];      // [j][k]
  float W2T[kH][kH + 4];  // [k][j]
  float H1[kTile][kH];
  float H1T[kH][kTP];  // [k][p]
  float D2[kTile][kH];
  float D2T[kH][kTP];  // [j][p]
  float H2[kTile][kH + 1];  // later the gradient at layer 1
  float W1[kH], b1[kH], b2[kH], W3[kOut][kH], b3[kOut];
  float x[kTile];
  float dy[kTile][kOut];
  float red[256];
};
static_assert(offsetof(MlpLds, W2T) % 16 == 0 && offsetof(MlpLds, H1) % 16 == 0 && offsetof(MlpLds, D2) % 16 == 0 &&
                  sizeof(MlpLds::W2[0]) % 16 == 0 && sizeof(MlpLds::W2T[0]) % 16 == 0 &&
                  sizeof(MlpLds::H1[0]) % 16 == 0 && sizeof(MlpLds::D2[0]) % 16 == 0 && alignof(MlpLds) == 16,
              "rows of vector loads");

// Small-parameter gradients a thread owns: W3 entries tid and tid + 256 (of
// 384), one of b3, b2, and one of W1 or b1.
struct MlpAcc {
  float W2[4][4];  // rows 4 (tid / 16) .., columns 4 (tid % 16) ..
  float W3[2], b3, b2, l1;
  float loss;
};

__device__ __forceinline__ void load_params(MlpLds& L, const float* P) {
  const int tid = threadIdx.x;
  for (int e = tid; e < kH * kH; e += 256) {
    const float w = P[OFF_W2 + e];
    L.W2[e >> 6][e & 63] = w;
    L.W2T[e & 63][e >> 6] = w;
  }
  if (tid < kH) {
    L.W1[tid] = P[OFF_W1 + tid];
    L.b1[tid] = P[OFF_B1 + tid];
    L.b2[tid] = P[OFF_B2 + tid];
  }
  for (int e = tid; e < kOut * kH; e += 256) L.W3[e >> 6][e & 63] = P[OFF_W3 + e];
  if (tid < kOut) L.b3[tid] = P[OFF_B3 + tid];
}

__device__ __forceinline__ void tile_grad(MlpLds& L, const float* __restrict__ x, const float* __restrict__ t,
                                          const float* __restrict__ m, int64_t n, int64_t p0, float inv_cnt,
                                          MlpAcc& G) {
  const int tid = threadIdx.x;
  if (tid < kTile) L.x[tid] = (p0 + tid < n) ? x[p0 + tid] : 0.0f;
  __syncthreads();
  // h1 = tanh(W1 x + b1)
#pragma unroll
  for (int e = tid; e < kTile * kH; e += 256) {
    const int p = e >> 6, k = e & 63;
    const float h = tanhf(fmaf(L.W1[k], L.x[p], L.b1[k]));
    L.H1[p][k] = h;
    L.H1T[k][p] = h;
  }
  __syncthreads();
  const int q0 = 4 * (tid & 15), r0 = kRP * (tid >> 4);  // this thread's 4 features and kRP points
  // h2 = tanh(W2 h1 + b2)
  {
    float a[kRP][4];
#pragma unroll
    for (int r = 0; r < kRP; ++r)
#pragma unroll
      for (int c = 0; c < 4; ++c) a[r][c] = L.b2[q0 + c];
#pragma unroll 16
    for (int k = 0; k < kH; ++k) {
      const float4 w = *reinterpret_cast<const float4*>(&L.W2T[k][q0]);
#pragma unroll
      for (int r = 0; r < kRP; ++r) {
        const float h = L.H1T[k][r0 + r];
        a[r][0] = fmaf(w.x, h, a[r][0]);
        a[r][1] = fmaf(w.y, h, a[r][1]);
        a[r][2] = fmaf(w.z, h, a[r][2]);
        a[r][3] = fmaf(w.w, h, a[r][3]);
      }
    }
#pragma unroll
    for (int r = 0; r < kRP; ++r)
#pragma unroll
      for (int c = 0; c < 4; ++c) L.H2[r0 + r][q0 + c] = tanhf(a[r][c]);
  }
  __syncthreads();
  // y = W3 h2 + b3; masked residual; dL/dy
  if (tid < kTile * kOut) {
    const int p = tid / kOut, o = tid % kOut;
    const int64_t q = p0 + p;
    float mk = 0.0f, tg = 0.0f;
    if (q < n) {
      mk = m[q * kOut + o];
      tg = t[q * kOut + o];
    }
    float a = L.b3[o];
#pragma unroll 16
    for (int j = 0; j < kH; ++j) a = fmaf(L.W3[o][j], L.H2[p][j], a);
    float r = 0.0f;
    if (q < n) r = mk * (a - tg);
    G.loss = fmaf(r, r, G.loss);
    L.dy[p][o] = 2.0f * r * inv_cnt;
  }
  __syncthreads();
  // dW3, db3
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int e = tid + 256 * u;
    if (e < kOut * kH) {
      const int o = e >> 6, j = e & 63;
      float g = 0.0f;
#pragma unroll 8
      for (int p = 0; p < kTile; ++p) g = fmaf(L.dy[p][o], L.H2[p][j], g);
      G.W3[u] += g;
    } else if (e - kOut * kH < kOut) {
      float g = 0.0f;
      for (int p = 0; p < kTile; ++p) g += L.dy[p][e - kOut * kH];
      G.b3 += g;
    }
  }
  // dz2 = (W3^T dy) (1 - h2^2)
#pragma unroll
  for (int e = tid; e < kTile * kH; e += 256) {
    const int p = e >> 6, j = e & 63;
    float a = 0.0f;
#pragma unroll
    for (int o = 0; o < kOut; ++o) a = fmaf(L.W3[o][j], L.dy[p][o], a);
    const float h = L.H2[p][j];
    const float d = a * ((1.0f - h) * (1.0f + h));
    L.D2[p][j] = d;
    L.D2T[j][p] = d;
  }
  __syncthreads();
  // dW2, db2
  {
    const int j0 = 4 * (tid >> 4);
#pragma unroll 4
    for (int p = 0; p < kTile; ++p) {
      const float4 d = *reinterpret_cast<const float4*>(&L.D2[p][j0]);
      const float4 h = *reinterpret_cast<const float4*>(&L.H1[p][q0]);
      const float dv[4] = {d.x, d.y, d.z, d.w}, hv[4] = {h.x, h.y, h.z, h.w};
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) G.W2[r][c] = fmaf(dv[r], hv[c], G.W2[r][c]);
    }
  }
  if (tid < kH) {
    float g = 0.0f;
#pragma unroll 8
    for (int p = 0; p < kTile; ++p) g += L.D2[p][tid];
    G.b2 += g;
  }
  // dz1 = (W2^T dz2) (1 - h1^2), in H2's place (H2 was last read before the barrier above)
  {
    float a[kRP][4];
#pragma unroll
    for (int r = 0; r < kRP; ++r)
#pragma unroll
      for (int c = 0; c < 4; ++c) a[r][c] = 0.0f;
#pragma unroll 16
    for (int j = 0; j < kH; ++j) {
      const float4 w = *reinterpret_cast<const float4*>(&L.W2[j][q0]);
#pragma unroll
      for (int r = 0; r < kRP; ++r) {
        const float d = L.D2T[j][r0 + r];
        a[r][0] = fmaf(w.x, d, a[r][0]);
        a[r][1] = fmaf(w.y, d, a[r][1]);
        a[r][2] = fmaf(w.z, d, a[r][2]);
        a[r][3] = fmaf(w.w, d, a[r][3]);
      }
    }
#pragma unroll
    for (int r = 0; r < kRP; ++r)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float h = L.H1[r0 + r][q0 + c];
        L.H2[r0 + r][q0 + c] = a[r][c] * ((1.0f - h) * (1.0f + h));
      }
  }
  __syncthreads();
  // dW1, db1
  if (tid < 2 * kH) {
    const int k = tid & 63;
    float g = 0.0f;
    if (tid < kH) {
#pragma unroll 8
      for (int p = 0; p < kTile; ++p) g = fmaf(L.H2[p][k], L.x[p], g);
    } else {
#pragma unroll 8
      for (int p = 0; p < kTile; ++p) g += L.H2[p][k];
    }
    G.l1 += g;
  }
  __syncthreads();
}

// Gradient of the whole data set for the parameters in L: blocks take
// tiles b, b + G, ...; per-block partial gradients go to partial[b][*] (rows
// of kMlpStride) and partial losses to ploss[b].
__device__ __forceinline__ void block_grad(MlpLds& L, const MlpArgs& A) {
  const int tid = threadIdx.x;
  MlpAcc G{};
  const int64_t n_tiles = (A.n + kTile - 1) / kTile;
  for (int64_t tl = blockIdx.x; tl < n_tiles; tl += gridDim.x)
    tile_grad(L, A.x, A.t, A.mask, A.n, tl * kTile, A.inv_cnt, G);
  float* out = A.partial + (size_t)blockIdx.x * kMlpStride;
  const int j0 = 4 * (tid >> 4), k0 = 4 * (tid & 15);
#pragma unroll
  for (int r = 0; r < 4; ++r)
    *reinterpret_cast<float4*>(&out[OFF_W2 + (j0 + r) * kH + k0]) =
        make_float4(G.W2[r][0], G.W2[r][1], G.W2[r][2], G.W2[r][3]);
  out[OFF_W3 + tid] = G.W3[0];
  if (tid < kOut * kH - 256)
    out[OFF_W3 + 256 + tid] = G.W3[1];
  else if (tid - (kOut * kH - 256) < kOut)
    out[OFF_B3 + tid - (kOut * kH - 256)] = G.b3;
  if (tid < kH) out[OFF_B2 + tid] = G.b2;
  if (tid < 2 * kH) out[(tid < kH ? OFF_W1 : OFF_B1 - kH) + tid] = G.l1;
  // loss: a fixed tree over the wave, then the waves in turn
  float s = G.loss;
  for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d, 64);
  if ((tid & 63) == 0) L.red[tid >> 6] = s;
  __syncthreads();
  if (tid == 0) A.ploss[blockIdx.x] = (L.red[0] + L.red[1]) + (L.red[2] + L.red[3]);
}

// Whole block: the sum over the nb partial gradients of the parameters
// [first, first + per), per = 64, 128 or 256: thread tid (and 256 / per row
// groups side by side, combined in order) returns parameter first + tid of the
// first `per` threads.
__device__ __forceinline__ float reduce_rows(const float* partial, int nb, int first, int per,
                                             float* red) {
  const int tid = threadIdx.x, c = tid & (per - 1), grp = tid / per, groups = 256 / per;
  const int i = first + c;
  float g = 0.0f;
  if (i < kMlpParams) {
#pragma unroll 8
    for (int b = grp; b < nb; b += groups) g += partial[(size_t)b * kMlpStride + i];
  }
  __syncthreads();
  red[tid] = g;
  __syncthreads();
  float s = red[c];
  for (int k = 1; k < groups; ++k) s += red[k * per + c];
  return s;
}

// Parameters a block reduces at a time: with enough blocks a few rows groups
// share the rows of one parameter, so that fewer loads wait on each other.
__device__ __forceinline__ int reduce_width(int blocks) {
  return blocks * 64 >= kMlpParams ? 64 : (blocks * 128 >= kMlpParams ? 128 : 256);
}

__global__ __launch_bounds__(256) void k_mlp_grad(MlpArgs A) {
  __shared__ MlpLds L;
  load_params(L, A.params);
  __syncthreads();
  block_grad(L, A);
}

// Fixed-order reduction of the per-block partials.
__global__ __launch_bounds__(256) void k_mlp_reduce(const float* __restrict__ partial, const float* __restrict__ ploss,
                                                    int nb, float* __restrict__ grad, float* __restrict__ loss) {
  __shared__ float red[256];
  const int first = blockIdx.x * 64;
  const float g = reduce_rows(partial, nb, first, 64, red);
  if (threadIdx.x < 64 && first + (int)threadIdx.x < kMlpParams) grad[first + threadIdx.x] = g;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    float s = 0.0f;
    for (int b = 0; b < nb; ++b) s += ploss[b];
    *loss = s;
  }
}

// Every epoch: gradient (all blocks), fixed-order reduction and Adam update
// (the parameters dealt over the blocks), then the blocks reload the
// parameters.  Two grid barriers per epoch; the last block, which has the
// fewest parameters, sums the loss.
__global__ __launch_bounds__(256) void k_mlp_train(MlpArgs A) {
  __shared__ MlpLds L;
  __shared__ uint32_t s_pub[kBarWords];
  __shared__ float s_rate[3];
  uint32_t gen = 0;
  const int per = reduce_width((int)gridDim.x);
  for (int e = 0; e < A.epochs; ++e) {
    load_params(L, A.params);
    if (threadIdx.x == 255) {
      s_rate[0] =
          (float)(A.lr_min + 0.5 * (A.lr0 - A.lr_min) * (1.0 + cos(3.14159265358979323846 * e / A.epochs)));
      s_rate[1] = 1.0f / (1.0f - powf(A.beta1, (float)(e + 1)));
      s_rate[2] = 1.0f / (1.0f - powf(A.beta2, (float)(e + 1)));
    }
    __syncthreads();
    block_grad(L, A);
    grid_barrier(A.bar, gen, s_pub, [](uint32_t*) {});
    const float lr = s_rate[0], c1 = s_rate[1], c2 = s_rate[2];
    for (int first = (int)blockIdx.x * per; first < kMlpParams; first += (int)gridDim.x * per) {
      const int i = first + (int)threadIdx.x;
      const bool mine = (int)threadIdx.x < per && i < kMlpParams;
      const float m0 = mine ? A.m[i] : 0.0f, v0 = mine ? A.v[i] : 0.0f, p0 = mine ? A.params[i] : 0.0f;
      const float g = reduce_rows(A.partial, (int)gridDim.x, first, per, L.red);
      if (mine) {
        const float m = A.beta1 * m0 + (1.0f - A.beta1) * g;
        const float v = A.beta2 * v0 + (1.0f - A.beta2) * g * g;
        A.m[i] = m;
        A.v[i] = v;
        A.params[i] = p0 - lr * (m * c1) / (sqrtf(v * c2) + A.eps);
      }
    }
    if (blockIdx.x == gridDim.x - 1 && A.loss_hist) {  // the block with the fewest parameters
      float s = 0.0f;
      for (int b = (int)threadIdx.x; b < (int)gridDim.x; b += 256) s += A.ploss[b];
      for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d, 64);
      __syncthreads();
      if ((threadIdx.x & 63) == 0) L.red[threadIdx.x >> 6] = s;
      __syncthreads();
      if (threadIdx.x == 0) A.loss_hist[e] = ((L.red[0] + L.red[1]) + (L.red[2] + L.red[3])) * A.inv_cnt;
    }
    grid_barrier(A.bar, gen, s_pub, [](uint32_t*) {});
  }
}

// ---------------------------------------------------------------------------
// Inference.
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;

// Logistic function of t, with t given as -t log2(e) (the factor lives in the
// weights and biases that produce it): 1 / (1 + 2^-t log2 e), one exponential
// and one reciprocal; 0 and 1 at the ends.
__device__ __forceinline__ float logistic_l2(float neg_t_log2e) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(neg_t_log2e));
}

// The hidden layers use tanh(z) = 2 s - 1 with s = logistic(2 z): the next
// layer takes s as its input, with its weights doubled (exact in bfloat16, so
// the matrix operands are the weights themselves and the doubling is applied
// to the product) and its bias reduced by the row sum of its bfloat16 weights.
// Each activation is then one multiply-add, one exponential, one add and one
// reciprocal; s, not tanh(z), is what is rounded to bfloat16.
constexpr float kM2L2E = -2.0f * 1.4426950408889634f;  // -2 log2(e)

constexpr int kMaskLds = 4096;

// Operand fragments in LDS: for MFMA k-step s and lane l, 8 bf16 values.
struct InferLds {
  bf16x8 A2[2][4][64];  // W2: M-block m (output features 32m..), k-step s (inputs 16s + 8 (l/32) + q)
  bf16x8 A3[4][64];     // W3 padded to 32 rows; k-step s, q -> feature 32 (s/2) + 8 (2 (s%2) + q/4) + 4 (l/32) + q%4
  float a1[64], c1[64];  // layer 1: -2 log2(e) (W1, b1)
  float c2[64];          // layer 2: -2 log2(e) (b2 - row sums of bf16 W2)
  float y_scale[8], y_off[8];  // output: 2 sd_y, (b3 - row sums of bf16 W3) sd_y + mu_y
  uint8_t mask[kMaskLds];      // the fallback mask per cell, when it has at most kMaskLds cells
};

// The tiles of one wave, 32 points each: lanes l and l + 32 both work on
// point l of a tile (the two halves of the MFMA operands), and each writes its
// half of the outputs.  MASK_LDS: the fallback mask sits in LDS (otherwise it
// is read from global memory); the two cases are separate instantiations so
// that each read is a plain LDS or global load, never a generic one, whose wait
// would also wait for the field read ahead for the next tile.  The table rows
// of the outputs that fall back are read before the next tile's field and
// before the network, so that their latency overlaps the network and waiting
// for them does not wait for that prefetch.
template <bool MASK_LDS>
__device__ __forceinline__ void infer_tiles(const InferArgs& A, const InferLds& L, int lane, int64_t wave,
                                            int64_t nwave) {
  const int half = lane >> 5, col = lane & 31;
  const int64_t stride = nwave * 32;
  // the field of the lane's point in the wave's next tile, read one
  // iteration ahead (an index clamped into the array, so that the load needs
  // no branch)
  float en_next = A.EN[min(wave * 32 + col, A.n - 1)];
  for (int64_t p0 = wave * 32; p0 < A.n; p0 += stride) {
    const int64_t p = p0 + col;
    const bool valid = p < A.n;
    const float EN = valid ? en_next : 1.0f;
    const float lnEN = logf(EN);
    const float xs = (lnEN - A.mu_x) * A.inv_sd_x;
    // bit o set: output o of this point's cell takes the table
    unsigned fbm = 0u;
    float tf = 0.0f, ta[4] = {0.0f, 0.0f, 0.0f, 0.0f}, tb[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (A.n_cells > 0) {
      const int cell = min(max((int)floorf((lnEN - A.cell_lo) * A.inv_cell_w), 0), A.n_cells - 1);
      fbm = (unsigned)(MASK_LDS ? L.mask[cell] : A.fb_mask[cell]) & kAllOut;
      if (fbm) {
        const float u = fminf(fmaxf((lnEN - A.tab_lo) * A.inv_tab_w, 0.0f), (float)(A.n_nodes - 1));
        const float fl = fminf(floorf(u), (float)(A.n_nodes - 2));
        tf = u - fl;
        // this lane's outputs 4 half + j of the nodes on either side
        const float* row = A.table + (size_t)(int)fl * kOut + 4 * half;
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (4 * half + j < kOut) {
            ta[j] = row[j];
            tb[j] = row[kOut + j];
          }
      }
    }
    en_next = A.EN[min(p + stride, A.n - 1)];
    floatx16 c3;
    for (int r = 0; r < 16; ++r) c3[r] = 0.0f;
    // The perceptron runs unless every output of every point of the wave
    // falls back to the table (the condition is wave-uniform, as the matrix
    // instructions need).
    if (__ballot(valid && fbm != kAllOut) != 0) {
      // layer 2: C2[m] = W2[32m.., :] s1 over 4 k-steps of 16
      floatx16 c2[2];
      for (int m = 0; m < 2; ++m)
        for (int r = 0; r < 16; ++r) c2[m][r] = 0.0f;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        bf16x8 b;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int k = 16 * s + 8 * half + q;
          b[q] = (__bf16)logistic_l2(fmaf(L.a1[k], xs, L.c1[k]));
        }
        c2[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(L.A2[0][s][lane], b, c2[0], 0, 0, 0);
        c2[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(L.A2[1][s][lane], b, c2[1], 0, 0, 0);
      }
      // activation of layer 2 (z = 2 C2 + b2 - row sum); rows of C2 held by
      // this lane: 8 i + 4 half + j (i = reg / 4, j = reg % 4)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int m = s >> 1;
        bf16x8 b;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int i = 2 * (s & 1) + (q >> 2), j = q & 3;
          const int row = 8 * i + 4 * half + j;
          b[q] = (__bf16)logistic_l2(fmaf(c2[m][4 * i + j], 2.0f * kM2L2E, L.c2[32 * m + row]));
        }
        c3 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(L.A3[s][lane], b, c3, 0, 0, 0);
      }
    }
    if (!valid) continue;
    // outputs: rows 4 half + j (j < 4) of C3 are outputs 0..3 (half 0) and 4..7 (half 1)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int o = 4 * half + j;
      if (o >= kOut) break;
      float y = fmaf(c3[j], L.y_scale[o], L.y_off[o]);
      if ((fbm >> o) & 1u) y = fmaf(tf, tb[j] - ta[j], ta[j]);
      A.out[(size_t)o * A.n + p] = y;
    }
  }
}

// Five waves per SIMD (92 registers, no spills): left to itself the compiler
// gives the table rows held across the network registers of their own (103)
// and the kernel would drop to four.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5))) void k_mlp_infer(InferArgs A) {
  __shared__ InferLds L;
  const int tid = threadIdx.x;
  const float* P = A.params;
  for (int i = tid; i < 2 * 4 * 64; i += 256) {
    const int m = i >> 8, s = (i >> 6) & 3, l = i & 63;
    bf16x8 v;
    for (int q = 0; q < 8; ++q) {
      const int o = 32 * m + (l & 31), k = 16 * s + 8 * (l >> 5) + q;
      v[q] = (__bf16)P[OFF_W2 + o * kH + k];
    }
    L.A2[m][s][l] = v;
  }
  for (int i = tid; i < 4 * 64; i += 256) {
    const int s = i >> 6, l = i & 63;
    bf16x8 v;
    for (int q = 0; q < 8; ++q) {
      const int o = l & 31;
      const int f = 32 * (s >> 1) + 8 * (2 * (s & 1) + (q >> 2)) + 4 * (l >> 5) + (q & 3);
      v[q] = (__bf16)(o < kOut ? P[OFF_W3 + o * kH + f] : 0.0f);
    }
    L.A3[s][l] = v;
  }
  // The row sums of the bfloat16 weights, exact in double in any order: four
  // threads a row of W2, 32 a row of W3 (one thread a row took 64 loads of 64
  // rows each one after another: 11.4 -> 10.5 us a launch at 1000 points).
  {
    const int row = tid >> 2, part = tid & 3;
    double rs = 0.0;
#pragma unroll
    for (int q = 0; q < kH / 4; ++q) rs += (double)(float)(__bf16)P[OFF_W2 + row * kH + 4 * q + part];
    rs += __shfl_xor(rs, 1);
    rs += __shfl_xor(rs, 2);
    if (part == 0) L.c2[row] = kM2L2E * (float)((double)P[OFF_B2 + row] - rs);
  }
  if (tid < 64) {
    L.a1[tid] = kM2L2E * P[OFF_W1 + tid];
    L.c1[tid] = kM2L2E * P[OFF_B1 + tid];
  }
  {
    const int row = tid >> 5, part = tid & 31;  // 8 rows, of which kOut there are
    double rs = 0.0;
    if (row < kOut)
      for (int j = part; j < kH; j += 32) rs += (double)(float)(__bf16)P[OFF_W3 + row * kH + j];
    for (int d = 1; d < 32; d <<= 1) rs += __shfl_xor(rs, d);
    if (part == 0) {
      L.y_scale[row] = row < kOut ? 2.0f * A.sd_y[row] : 0.0f;
      L.y_off[row] = row < kOut ? (float)(((double)P[OFF_B3 + row] - rs) * A.sd_y[row] + A.mu_y[row]) : 0.0f;
    }
  }
  const bool mask_lds = A.n_cells <= kMaskLds;
  if (mask_lds)
    for (int i = tid; i < A.n_cells; i += 256) L.mask[i] = A.fb_mask[i];
  __syncthreads();
  const int64_t wave = (int64_t)blockIdx.x * 4 + (tid >> 6);
  const int64_t nwave = (int64_t)gridDim.x * 4;
  if (mask_lds)
    infer_tiles<true>(A, L, tid & 63, wave, nwave);
  else
    infer_tiles<false>(A, L, tid & 63, wave, nwave);
}

// ---------------------------------------------------------------------------
hipError_t launch_mlp_grad(const MlpArgs& a, int grid, hipStream_t stream) {
  hipLaunchKernelGGL(k_mlp_grad, dim3(grid), dim3(256), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_mlp_reduce(const float* partial, const float* ploss, int nb, float* grad, float* loss,
                             hipStream_t stream) {
  hipLaunchKernelGGL(k_mlp_reduce, dim3((kMlpParams + 63) / 64), dim3(256), 0, stream, partial, ploss, nb, grad,
                     loss);
  return hipGetLastError();
}

hipError_t occupancy_mlp_train(int* blocks_per_cu) {
  return coresident_blocks((const void*)k_mlp_train, 256, 0, blocks_per_cu);
}

hipError_t launch_mlp_train(const MlpArgs& a, int grid, hipStream_t stream) {
  void* kargs[] = {(void*)&a};
  return hipLaunchCooperativeKernel((const void*)k_mlp_train, dim3(grid), dim3(256), kargs, 0, stream);
}

hipError_t launch_mlp_infer(const InferArgs& a, int grid, hipStream_t stream) {
  hipLaunchKernelGGL(k_mlp_infer, dim3(grid), dim3(256), 0, stream, a);
  return hipGetLastError();
}

}  // namespace pcmcc
