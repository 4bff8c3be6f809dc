// Learned constitutive surrogate: MLP 13 -> 128 -> 128 -> 128 -> 6 (SiLU) on gfx950.
//
// All of it is dense products, run on the FP32 matrix cores (v_mfma_f32_16x16x4f32: lane l holds
// A[l % 16][l / 16] and B[l / 16][l % 16], result entry r sits in row 4 (l / 16) + r, column l % 16).
// Four products are chained so that lane group l / 16 takes four neighbouring k: the A operand is one
// 16-byte LDS read per 16 k.
#include <mutex>

#include "fe_internal.hpp"

namespace fe {

constexpr int HID = FE_MLP_HIDDEN, NIN = FE_MLP_IN, NOUT = FE_MLP_OUT;
constexpr int OFF_W1 = 0, OFF_B1 = OFF_W1 + NIN * HID;
constexpr int OFF_W2 = OFF_B1 + HID, OFF_B2 = OFF_W2 + HID * HID;
constexpr int OFF_W3 = OFF_B2 + HID, OFF_B3 = OFF_W3 + HID * HID;
constexpr int OFF_W4 = OFF_B3 + HID, OFF_B4 = OFF_W4 + HID * NOUT;
static_assert(OFF_B4 + NOUT == FE_MLP_PARAMS, "parameter layout");

constexpr int LDA = HID + 4;    // LDS row stride in floats (16-byte rows, no bank conflicts)
constexpr int MS16 = 16;        // samples per tile

typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float sigm(float z) { return 1.0f / (1.0f + __expf(-z)); }
__device__ __forceinline__ float silu_f(float z) { return z * sigm(z); }
__device__ __forceinline__ float silu_d(float z) {
  const float s = sigm(z);
  return s * (1.0f + z * (1.0f - s));
}

// Two 16-column tiles of a 128 x 128 matrix in registers, as the B operand: w[4 kk + s][ct] is entry
// (k, col) with k = 16 kk + 4 (lane / 16) + s and col = col0 + 16 ct.
struct WeightTile {
  float w[HID / 4][2];
  // B[k][col] = W[k * HID + col]
  __device__ __forceinline__ void load(const float* __restrict__ W, int g, int col0) {
#pragma unroll
    for (int kk = 0; kk < HID / 16; ++kk)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) w[4 * kk + s][ct] = W[(16 * kk + 4 * g + s) * HID + col0 + 16 * ct];
  }
  // B[k][col] = W[col * HID + k]
  __device__ __forceinline__ void load_transposed(const float* __restrict__ W, int g, int col0) {
#pragma unroll
    for (int kk = 0; kk < HID / 16; ++kk)
#pragma unroll
      for (int ct = 0; ct < 2; ++ct)
#pragma unroll
        for (int s = 0; s < 4; ++s) w[4 * kk + s][ct] = W[(col0 + 16 * ct) * HID + 16 * kk + 4 * g + s];
  }
  // acc[t][ct] = rows 16 t .. 16 t + 15 of act (LDS) times this tile
  template <int NT> __device__ __forceinline__ void multiply(const float* act, int g, int c, v4f acc[NT][2]) const {
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t][0] = acc[t][1] = v4f{0.f, 0.f, 0.f, 0.f};
    const float* row = act + c * LDA + 4 * g;
    v4f next = *reinterpret_cast<const v4f*>(row);
#pragma unroll
    for (int m = 0; m < HID / 16 * NT; ++m) {
      const int kk = m / NT, t = m % NT, m1 = m + 1;
      const v4f a = next;
      if (m1 < HID / 16 * NT) next = *reinterpret_cast<const v4f*>(row + m1 % NT * 16 * LDA + m1 / NT * 16);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int ct = 0; ct < 2; ++ct)
          acc[t][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], w[4 * kk + s][ct], acc[t][ct], 0, 0, 0);
    }
    // issue order: each LDS read ahead of the eight products before its own (left to itself the
    // compiler reads, waits and multiplies in turn)
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
#pragma unroll
    for (int m = 0; m < HID / 16 * NT; ++m) {
      if (m + 1 < HID / 16 * NT) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);
    }
  }
};

// Values (MLP_VALUES: NT tiles of 16 samples) or values and the 6 forward-mode tangent columns
// (MLP_TANGENT: tile 0 the values of 16 samples, tile 1 + j the tangents by input j, NT = 7; MLP_TANGENT8: 8
// samples, the lower half of tile t their path 2 t, the upper half path 2 t + 1, NT = 4).  A workgroup keeps the
// two 128 x 128 weight matrices in its registers, 32 columns per wave, and walks over groups of
// samples; the activations of a group pass through one LDS buffer.  A sample's tangent rows lie in
// the same lane (or 32 lanes on) and register as its value row, and the first layer's tangents are rows of W1 times SiLU', not a product.  Bound by the matrix cores: 402 us for 100 000
// points with tangents (49 GFLOP, 322 us at the FP32 matrix rate) against 604 us with eight rows per
// sample, one of them padding, and the weights read from the caches by every wave.
constexpr int64_t FWD_BLOCKS = 512;
constexpr int64_t TANGENT8_MAX = 2048;
enum { MLP_VALUES, MLP_TANGENT, MLP_TANGENT8 };
template <int NT, int MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void mlp_fwd_kernel(
    const float* __restrict__ W, const float* __restrict__ x, float* __restrict__ y, float* __restrict__ jac,
    float* __restrict__ cache, int64_t n) {
  constexpr bool TAN = MODE != MLP_VALUES, HALF = MODE == MLP_TANGENT8;
  static_assert(MODE == MLP_VALUES || NT == (HALF ? 4 : NOUT + 1), "value and tangent rows");
  constexpr int NV = TAN ? 1 : NT;           // tiles with value rows
  constexpr int SPG = HALF ? 8 : NV * 16;    // samples per group
  constexpr int LDX = 20;
  __shared__ alignas(16) float act[NT * 16 * LDA];
  __shared__ alignas(16) float s_x[NV * 16 * LDX];
  __shared__ float s_w1[16 * HID];           // rows NIN .. 15 zero
  __shared__ float s_w4[HID * NOUT], s_b[3 * HID];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, c = lane & 15;
  const int col0 = 32 * wave + c;
  const int64_t groups = (n + SPG - 1) / SPG;
  // this lane's input of each value tile of a group (zero past the 13 inputs and past the samples)
  const auto load_x = [&](int64_t grp, float xv[NV]) {
#pragma unroll
    for (int t = 0; t < NV; ++t) {
      const int64_t gs = grp * SPG + 16 * t + (HALF ? (tid >> 4) & 7 : tid >> 4);
      xv[t] = (tid & 15) < NIN && grp < groups && gs < n ? x[gs * NIN + (tid & 15)] : 0.0f;
    }
  };
  float xv[NV];
  load_x(blockIdx.x, xv);
  WeightTile w2, w3;
  w2.load(W + OFF_W2, g, col0);
  w3.load(W + OFF_W3, g, col0);
  for (int i = tid; i < 3 * HID; i += 256) s_b[i] = W[(i < HID ? OFF_B1 : (i < 2 * HID ? OFF_B2 - HID : OFF_B3 - 2 * HID)) + i];
  for (int i = tid; i < 16 * HID; i += 256) s_w1[i] = i < NIN * HID ? W[OFF_W1 + i] : 0.0f;
  for (int i = tid; i < HID * NOUT; i += 256) s_w4[i] = W[OFF_W4 + i];

  // pre-activations z = acc + bias of a layer: cached, through SiLU (and SiLU' for the tangents) to LDS
  auto epilogue = [&](v4f acc[NT][2], int layer, int64_t s0) {
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
      const int col = col0 + 16 * ct;
#pragma unroll
      for (int t = 0; t < NV; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 16 * t + 4 * g + r;
          const bool value = !HALF || g < 2;
          const float z = (HALF ? __shfl(acc[t][ct][r], lane & 31, 64) : acc[t][ct][r]) + s_b[layer * HID + col];
          if (cache && value && s0 + row < n) cache[(s0 + row) * (3 * HID) + layer * HID + col] = z;
          float h = silu_f(z);
          if (TAN) {
            const float d = silu_d(z);
            if (HALF && !value) h = d * (layer == 0 ? s_w1[col] : acc[0][ct][r]);
#pragma unroll
            for (int j = 1; j < NT; ++j) {
              const int path = HALF ? 2 * j + (g >> 1) : j;  // (path 7 is a pad row)
              act[(16 * j + row) * LDA + col] = d * (layer == 0 ? s_w1[(path - 1) * HID + col] : acc[j][ct][r]);
            }
          }
          act[row * LDA + col] = h;
        }
    }
  };

  for (int64_t grp = blockIdx.x; grp < groups; grp += gridDim.x) {
    const int64_t s0 = grp * SPG;
#pragma unroll
    for (int t = 0; t < NV; ++t) s_x[(16 * t + (tid >> 4)) * LDX + (tid & 15)] = xv[t];
    __syncthreads();  // (and the output layer of the group before has read act)
    load_x(grp + gridDim.x, xv);
    v4f acc[NT][2];
#pragma unroll
    for (int t = 0; t < NV; ++t) {
      acc[t][0] = acc[t][1] = v4f{0.f, 0.f, 0.f, 0.f};
      const v4f a = *reinterpret_cast<const v4f*>(s_x + (16 * t + c) * LDX + 4 * g);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int ct = 0; ct < 2; ++ct)
          acc[t][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], s_w1[(4 * g + s) * HID + col0 + 16 * ct], acc[t][ct], 0, 0, 0);
    }
    epilogue(acc, 0, s0);
    __syncthreads();
    w2.multiply<NT>(act, g, c, acc);
    __syncthreads();
    epilogue(acc, 1, s0);
    __syncthreads();
    w3.multiply<NT>(act, g, c, acc);
    __syncthreads();
    epilogue(acc, 2, s0);
    __syncthreads();
    // output layer: 6 columns padded to one tile, no activation; each wave takes whole row tiles
    for (int t = wave; t < NT; t += 4) {
      v4f o = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < HID / 16; ++kk) {
        const v4f a = *reinterpret_cast<const v4f*>(act + (16 * t + c) * LDA + 16 * kk + 4 * g);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const float bv = c < NOUT ? s_w4[(16 * kk + 4 * g + s) * NOUT + c] : 0.0f;
          o = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], bv, o, 0, 0, 0);
        }
      }
      if (c < NOUT) {
        const float b4 = W[OFF_B4 + c];
        const int path = HALF ? 2 * t + (g >> 1) : (TAN ? t : 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int64_t gs = s0 + (HALF ? 4 * (g & 1) : (TAN ? 0 : 16 * t) + 4 * g) + r;
          if (gs >= n) continue;
          if (path == 0) y[gs * NOUT + c] = o[r] + b4;
          else if (path <= NOUT) jac[gs * (NOUT * NOUT) + c * NOUT + path - 1] = o[r];
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// backward pass of the mean squared error.  (1) per sample, the pre-activation
// gradients delta_l = dL/dz_l of all layers go to a workspace [n][3*128+6];
// (2) the weight gradients dWt_l[i][o] = sum_s h_{l-1}[s][i] delta_l[s][o] are
// batch-reduced products: 64 x 64 tiles, the batch split into chunks
// whose partial tiles are added with FP32 atomics (dW zeroed first).

constexpr int WSTRIDE = 3 * HID + NOUT;  // workspace row: delta1, delta2, delta3, delta4

// delta_l = silu'(z_l) * (delta_{l+1} W_{l+1}^T) for 16 samples, 32 columns per wave, the weights as B
// operands in registers.  Bound by latency (two 64 KB weight matrices and three dependent products per
// workgroup): 16 us for 4096 samples against 138 us on the vector units.
__global__ __launch_bounds__(256) void mlp_delta_kernel(const float* __restrict__ W, const float* __restrict__ cache,
                                                        const float* __restrict__ y, const float* __restrict__ t,
                                                        float* __restrict__ work, double* loss, int64_t n) {
  __shared__ alignas(16) float s_d[2][MS16 * LDA];
  __shared__ float s_d4[MS16 * 9];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, c = lane & 15;
  const int col0 = 32 * wave + c;
  const int64_t s0 = (int64_t)blockIdx.x * MS16;
  WeightTile w3, w2;
  w3.load_transposed(W + OFF_W3, g, col0);
  w2.load_transposed(W + OFF_W2, g, col0);
  float w4[2][2];
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) w4[s][ct] = 4 * s + g < NOUT ? W[OFF_W4 + (col0 + 16 * ct) * NOUT + 4 * s + g] : 0.0f;
  float z[3][2][4];
#pragma unroll
  for (int l = 0; l < 3; ++l)
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t gs = s0 + 4 * g + r;
        z[l][ct][r] = gs < n ? cache[gs * (3 * HID) + l * HID + col0 + 16 * ct] : 0.0f;
      }
  if (wave == 0) {  // delta4 and the loss: lanes (sample, output pair)
    const float scale = 2.0f / (float)n;
    double lsum = 0;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int i = lane + 64 * u, smp = i >> 3, o = i & 7;
      const int64_t gs = s0 + smp;
      float d = 0.0f;
      if (o < NOUT && gs < n) {
        const float e = y[gs * NOUT + o] - t[gs * NOUT + o];
        lsum += (double)e * (double)e;
        d = scale * e;
        work[gs * WSTRIDE + 3 * HID + o] = d;
      }
      s_d4[smp * 9 + o] = d;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) lsum += __shfl_down(lsum, off, 64);
    if (lane == 0) unsafeAtomicAdd(loss, lsum / (double)n);
  }
  __syncthreads();
  v4f acc[1][2];
  acc[0][0] = acc[0][1] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < 2; ++s)  // K = 6 padded to 8: k = 4 s + lane / 16
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
      acc[0][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(s_d4[c * 9 + 4 * s + g], w4[s][ct], acc[0][ct], 0, 0, 0);
#pragma unroll
  for (int l = 2; l >= 0; --l) {
    if (l < 2) {
      __syncthreads();
      if (l == 1) w3.multiply<1>(s_d[0], g, c, acc);
      else w2.multiply<1>(s_d[1], g, c, acc);
    }
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 4 * g + r, col = col0 + 16 * ct;
        const float d = silu_d(z[l][ct][r]) * acc[0][ct][r];
        if (l > 0) s_d[2 - l][row * LDA + col] = d;
        if (s0 + row < n) work[(s0 + row) * WSTRIDE + l * HID + col] = d;
      }
  }
}

// Weight-gradient tiles of 64 inputs x 64 outputs, the batch index as the contraction: blockIdx.y names
// (layer, input tile, output tile), 12 in all, blockIdx.x a chunk of `chunk` samples (a multiple
// of 64), chosen so that the chip is filled without adding more than 64 partial tiles per address.
// A wave holds 32 x 32 of the tile.  Bound by latency and the atomic adds: 23 us for 4096 samples
// against 109 us on the vector units with 32 x 32 tiles and chunks of 1024.
constexpr int WG_T = 64, WG_LD = WG_T + 16, WG_TILES = 12;  // (stride: the four lane groups in different banks)
constexpr int WG_CHUNK = 256, WG_MAXCHUNKS = 64;
static int64_t wgrad_chunk(int64_t n) {
  return std::max<int64_t>(WG_CHUNK, ((n + WG_MAXCHUNKS - 1) / WG_MAXCHUNKS + WG_T - 1) / WG_T * WG_T);
}

__global__ __launch_bounds__(256) void mlp_wgrad_kernel(const float* __restrict__ x, const float* __restrict__ cache,
                                                        const float* __restrict__ work, float* dW, int64_t n,
                                                        int64_t chunk) {
  __shared__ float hs[WG_T * WG_LD], ds[WG_T * WG_LD];  // [sample][column]
  const int tile = blockIdx.y;
  int layer, it, ot;
  if (tile < 2) {
    layer = 0; it = 0; ot = tile;
  } else if (tile < 10) {
    layer = 1 + (tile - 2) / 4; it = (tile - 2) % 4 / 2; ot = tile % 2;
  } else {
    layer = 3; it = tile - 10; ot = 0;
  }
  const int nin = layer == 0 ? NIN : HID, nout = layer == 3 ? NOUT : HID;
  const int woff = layer == 0 ? OFF_W1 : (layer == 1 ? OFF_W2 : (layer == 2 ? OFF_W3 : OFF_W4));
  const int boff = layer == 0 ? OFF_B1 : (layer == 1 ? OFF_B2 : (layer == 2 ? OFF_B3 : OFF_B4));
  const int doff = layer * HID;  // delta_{layer+1} column offset in the workspace
  const int64_t k0 = (int64_t)blockIdx.x * chunk, k1 = min<int64_t>(n, k0 + chunk);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, c = lane & 15;
  const int i0 = 32 * (wave >> 1), o0 = 32 * (wave & 1);
  // this lane's column of the staged blocks, samples wave, wave + 4, ..
  const int hi = it * WG_T + lane, ho = ot * WG_T + lane;
  const bool hin = hi < nin, din = ho < nout;
  const float* H = layer == 0 ? x + hi : cache + (layer - 1) * HID + hi;
  const int hstride = layer == 0 ? NIN : 3 * HID;
  const float* D = work + doff + ho;
  v4f acc[2][2];
  acc[0][0] = acc[0][1] = acc[1][0] = acc[1][1] = v4f{0.f, 0.f, 0.f, 0.f};
  float bacc = 0.f;
  for (int64_t sb = k0; sb < k1; sb += WG_T) {
    float hv[16], dv[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int64_t gs = sb + wave + 4 * u;
      hv[u] = hin && gs < k1 ? H[gs * hstride] : 0.0f;
      dv[u] = din && gs < k1 ? D[gs * WSTRIDE] : 0.0f;
    }
    __syncthreads();  // the block before has been read
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int row = wave + 4 * u;
      // (samples past the end have delta 0)
      hs[row * WG_LD + lane] = layer == 0 ? hv[u] : silu_f(hv[u]);
      ds[row * WG_LD + lane] = dv[u];
      bacc += dv[u];
    }
    __syncthreads();
#pragma unroll 4
    for (int k = 0; k < WG_T; k += 4) {
      float a[2], b[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        a[u] = hs[(k + g) * WG_LD + i0 + 16 * u + c];
        b[u] = ds[(k + g) * WG_LD + o0 + 16 * u + c];
      }
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) acc[u][v] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u], b[v], acc[u][v], 0, 0, 0);
    }
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      const int o = ot * WG_T + o0 + 16 * v + c;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = it * WG_T + i0 + 16 * u + 4 * g + r;
        if (i < nin && o < nout) unsafeAtomicAdd(dW + woff + i * nout + o, acc[u][v][r]);
      }
    }
  if (it == 0 && din) unsafeAtomicAdd(dW + boff + ho, bacc);
}

__global__ void adam_kernel(float* W, const float* dW, float* m, float* v, int64_t np, float lr, float b1, float b2,
                            float eps, float c1, float c2) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < np; i += (int64_t)gridDim.x * blockDim.x) {
    const float g = dW[i];
    const float mi = b1 * m[i] + (1.0f - b1) * g;
    const float vi = b2 * v[i] + (1.0f - b2) * g * g;
    m[i] = mi;
    v[i] = vi;
    W[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
  }
}

__global__ void zero_kernel(float* a, int64_t n, double* d) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) a[i] = 0;
  if (blockIdx.x == 0 && threadIdx.x == 0 && d) *d = 0;
}

static void launch_backward(const float* W, const float* x, const float* cache, const float* y, const float* target,
                            float* dW, double* loss, float* work, int64_t n, hipStream_t s) {
  const int64_t chunk = wgrad_chunk(n);
  hipLaunchKernelGGL(zero_kernel, dim3(64), dim3(256), 0, s, dW, (int64_t)FE_MLP_PARAMS, loss);
  hipLaunchKernelGGL(mlp_delta_kernel, dim3((unsigned)((n + MS16 - 1) / MS16)), dim3(256), 0, s, W, cache, y, target,
                     work, loss, n);
  hipLaunchKernelGGL(mlp_wgrad_kernel, dim3((unsigned)((n + chunk - 1) / chunk), WG_TILES), dim3(256), 0, s, x, cache,
                     work, dW, n, chunk);
}

}  // namespace fe

using namespace fe;

#define HIPCHK(x)                                  \
  do {                                             \
    hipError_t _e = (x);                           \
    if (_e != hipSuccess) return hip_fail(_e, #x); \
  } while (0)

extern "C" int fe_mlp_forward(const float* W, const float* x, float* y, float* jac, float* cache, int64_t n,
                              void* stream) {
  if (!W || !x || !y || n < 0) {
    set_error("fe_mlp_forward: W, x and y are required, n >= 0");
    return FE_ERR_ARG;
  }
  if (n == 0) return FE_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  // Persistent workgroups, two per CU (registers and LDS).  Groups of 8 samples while those of 16 leave half the
  // CUs without work (1000 points: 16 us against 23; 3000: 24 against 22); values alone take one tile of
  // 16 samples per group while a workgroup has one group, two above
  const auto blocks = [](int64_t groups) { return dim3((unsigned)std::min<int64_t>(groups, FWD_BLOCKS)); };
  if (jac && n <= TANGENT8_MAX)
    hipLaunchKernelGGL((mlp_fwd_kernel<4, MLP_TANGENT8>), blocks((n + 7) / 8), dim3(256), 0, s, W, x, y, jac, cache, n);
  else if (jac)
    hipLaunchKernelGGL((mlp_fwd_kernel<7, MLP_TANGENT>), blocks((n + 15) / 16), dim3(256), 0, s, W, x, y, jac, cache, n);
  else if (n <= 16 * FWD_BLOCKS)
    hipLaunchKernelGGL((mlp_fwd_kernel<1, MLP_VALUES>), blocks((n + 15) / 16), dim3(256), 0, s, W, x, y, jac, cache, n);
  else
    hipLaunchKernelGGL((mlp_fwd_kernel<2, MLP_VALUES>), blocks((n + 31) / 32), dim3(256), 0, s, W, x, y, jac, cache, n);
  HIPCHK(hipGetLastError());
  return FE_OK;
}

extern "C" int fe_mlp_backward(const float* W, const float* x, const float* cache, const float* y, const float* target,
                               float* dW, double* loss, float* work, int64_t n, void* stream) {
  if (!W || !x || !cache || !y || !target || !dW || !loss || !work || n <= 0) {
    set_error("fe_mlp_backward: all arrays are required, n > 0");
    return FE_ERR_ARG;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  launch_backward(W, x, cache, y, target, dW, loss, work, n, s);
  HIPCHK(hipGetLastError());
  return FE_OK;
}

// Workspace of fe_mlp_backward_static: the per-sample pre-activation gradients of at most
// FE_MLP_STATIC_MAX samples, in a file-scope device array (each GPU the library runs on holds its
// own copy, 12.8 MB, until the process ends).  Host code never passes the array's name to a
// kernel (on the host it is only a stand-in for the symbol): the device address is looked up
// once per device with hipGetSymbolAddress and kept in g_scratch_dev.
static __device__ __align__(256) float scratch[(size_t)FE_MLP_STATIC_MAX * WSTRIDE];

constexpr int SCRATCH_MAX_DEVICES = 64;
static std::mutex g_scratch_mu;
static float* g_scratch_dev[SCRATCH_MAX_DEVICES];

// Device address of `scratch` on the current device, or null (error recorded) on failure.
static float* scratch_on_current_device() {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) {
    hip_fail(e, "hipGetDevice");
    return nullptr;
  }
  if (dev < 0 || dev >= SCRATCH_MAX_DEVICES) {
    set_error("fe_mlp_backward_static: device index beyond the supported range");
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) {
      hip_fail(e != hipSuccess ? e : hipErrorInvalidSymbol, "hipGetSymbolAddress(scratch)");
      return nullptr;
    }
    g_scratch_dev[dev] = static_cast<float*>(ptr);
  }
  return g_scratch_dev[dev];
}

extern "C" int fe_mlp_backward_static(const float* W, const float* x, const float* cache, const float* y,
                                      const float* target, float* dW, double* loss, int64_t n, void* stream) {
  if (!W || !x || !cache || !y || !target || !dW || !loss || n <= 0) {
    set_error("fe_mlp_backward_static: all arrays are required, n > 0");
    return FE_ERR_ARG;
  }
  if (n > FE_MLP_STATIC_MAX) {
    set_error("fe_mlp_backward_static: n exceeds FE_MLP_STATIC_MAX samples (use fe_mlp_backward with a workspace)");
    return FE_ERR_ARG;
  }
  float* work = scratch_on_current_device();
  if (!work) return FE_ERR_HIP;
  // the delta kernel writes every workspace entry the weight-gradient kernel reads
  // (rows 0..n-1), so the array's contents from an earlier call never matter
  hipStream_t s = static_cast<hipStream_t>(stream);
  launch_backward(W, x, cache, y, target, dW, loss, work, n, s);
  HIPCHK(hipGetLastError());
  return FE_OK;
}

extern "C" int fe_adam_step(float* W, const float* dW, float* m, float* v, int64_t np, double lr, double beta1,
                            double beta2, double eps, int t, void* stream) {
  if (!W || !dW || !m || !v || np <= 0 || t < 1) {
    set_error("fe_adam_step: arrays required, n_param > 0, t >= 1");
    return FE_ERR_ARG;
  }
  const double c1 = 1.0 / (1.0 - std::pow(beta1, t)), c2 = 1.0 / (1.0 - std::pow(beta2, t));
  hipLaunchKernelGGL(adam_kernel, dim3((unsigned)std::min<int64_t>((np + 255) / 256, 1024)), dim3(256), 0,
                     static_cast<hipStream_t>(stream), W, dW, m, v, np, (float)lr, (float)beta1, (float)beta2,
                     (float)eps, (float)c1, (float)c2);
  HIPCHK(hipGetLastError());
  return FE_OK;
}
