// Learned per-element coarse correction: a three-layer perceptron
//   z1 = x W1^T + b1, h1 = relu(z1); z2 = h1 W2^T + b2, h2 = relu(z2);
//   o = h2 W3^T + b3  (the packed factor of the element's coarse operator)
// trained on the GPU by the kernels of this file (forward, loss and
// backward, Adam of Kingma & Ba 2015).  The paper leaves the PCG
// preconditioner open (section 4.2.2); this network is one choice of it.
//
// Precision (per network): BF16 (the default) keeps FP32 master parameters
// and BF16 copies of the weights that feed the forward layers, which run on
// MFMA (v_mfma_f32_16x16x16_bf16, FP32 accumulation) with BF16 layer
// inputs; the backward pass is FP32 (v_mfma_f32_16x16x4_f32, full FP32
// products and sums) on the same BF16-rounded weights and layer inputs as the
// forward pass.  FP32 runs the forward
// layers on VALU with the FP32 master weights and FP32 hidden activations
// (the network input stays BF16), and the backward pass on the same values:
// it differs from an exact evaluation only by FP32 rounding, which makes
// element-by-element checks of every parameter block possible.
//
// MFMA tile (16x16x16): lane l holds A[l % 16][4 (l / 16) + 0..3] and
// B[4 (l / 16) + 0..3][l % 16] (4 BF16 values each); the result C[4 (l / 16) +
// q][l % 16] is accumulator slot q.
//
// A minibatch of training (512 samples, K = 27) is 0.2 GFLOP and 3 MB: what
// bounds it is the latency of its chain of dependent kernels.  The chain is
// forward (the three layers in one launch), loss, and one launch per layer of
// the backward pass, whose weight, bias and input gradients depend on the
// same data and run side by side: 68 us a pass, against 680 us with a launch
// per product, a thread per bias (walking the batch) and a thread per sample
// in the loss.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <fstream>
#include <random>
#include <vector>

#include "common.h"
#include "sem_internal.h"

namespace sem {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// forward pass on MFMA
// ---------------------------------------------------------------------------
// o = W3 relu(W2 relu(W1 x + b1) + b2) + b3 for the rows of X [M][ldx] BF16
// (kin columns, kin % 16 == 0; W1 [128][kin], W2 [128][128], W3 [>= 16
// ceil(n_out / 16)][128] BF16, the rows beyond n_out zero).  A workgroup takes 16 rows
// through the three layers: wave w forms columns 16 w .. of both hidden
// layers (passed on through LDS in BF16) and every eighth 16-column tile of
// the output.  The weights of layer 2 and of the wave's first output tile are
// asked for before anything else.  When non-null, h1b, h2b (BF16) and h1f,
// h2f (FP32), all [M][128], receive the hidden activations for a backward
// pass.
constexpr int FW_WAVES = 8;
__global__ void __launch_bounds__(64 * FW_WAVES)
    k_forward_mfma(int M, int kin, int n_out, const uint16_t *__restrict__ X, int ldx,
                   const uint16_t *__restrict__ W1, const float *__restrict__ b1,
                   const uint16_t *__restrict__ W2, const float *__restrict__ b2,
                   const uint16_t *__restrict__ W3, const float *__restrict__ b3,
                   float *__restrict__ O, int ldo, uint16_t *__restrict__ h1b,
                   uint16_t *__restrict__ h2b, float *__restrict__ h1f,
                   float *__restrict__ h2f) {
  constexpr int H = 128, PITCH = H + 8;  // rows 4 banks apart
  __shared__ __align__(16) uint16_t lds[2][16 * PITCH];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int r = l & 15, g = l >> 4;
  const int row0 = blockIdx.x * 16;
  const int nt3 = (n_out + 15) / 16;
  auto wfrag = [&](const uint16_t *W, int tile, int ks) {
    return *reinterpret_cast<const s16x4 *>(W + (size_t)(16 * tile + r) * H + 16 * ks + 4 * g);
  };
  s16x4 w2[H / 16], w3[H / 16];
#pragma unroll
  for (int ks = 0; ks < H / 16; ++ks) w2[ks] = wfrag(W2, w, ks);
#pragma unroll
  for (int ks = 0; ks < H / 16; ++ks) w3[ks] = wfrag(W3, w < nt3 ? w : 0, ks);
  const int col = 16 * w + r;  // of the hidden layers
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  {
    const int ar = row0 + r;
    for (int k0 = 0; k0 < kin; k0 += 16) {
      s16x4 a = {0, 0, 0, 0};
      if (ar < M) a = *reinterpret_cast<const s16x4 *>(X + (size_t)ar * ldx + k0 + 4 * g);
      const s16x4 b = *reinterpret_cast<const s16x4 *>(W1 + (size_t)col * kin + k0 + 4 * g);
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, acc, 0, 0, 0);
    }
  }
  // bias, relu; to LDS and, when wanted, to memory
  auto hidden = [&](const f32x4 &v, float bias, uint16_t *L, uint16_t *hb, float *hf) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int rr = 4 * g + q;
      const float x = fmaxf(v[q] + bias, 0.0f);
      const uint16_t xb = f32_to_bf16(x);
      L[rr * PITCH + col] = xb;
      if (row0 + rr < M) {
        if (hb) hb[(size_t)(row0 + rr) * H + col] = xb;
        if (hf) hf[(size_t)(row0 + rr) * H + col] = x;
      }
    }
  };
  hidden(acc, b1[col], lds[0], h1b, h1f);
  __syncthreads();
  acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < H / 16; ++ks) {
    const s16x4 a = *reinterpret_cast<const s16x4 *>(&lds[0][r * PITCH + 16 * ks + 4 * g]);
    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, w2[ks], acc, 0, 0, 0);
  }
  hidden(acc, b2[col], lds[1], h2b, h2f);
  __syncthreads();
  s16x4 h[H / 16];
#pragma unroll
  for (int ks = 0; ks < H / 16; ++ks)
    h[ks] = *reinterpret_cast<const s16x4 *>(&lds[1][r * PITCH + 16 * ks + 4 * g]);
  for (int t = w; t < nt3; t += FW_WAVES) {
    acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < H / 16; ++ks)
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(h[ks], w3[ks], acc, 0, 0, 0);
    if (t + FW_WAVES < nt3) {  // the next tile's weights while this one is stored
#pragma unroll
      for (int ks = 0; ks < H / 16; ++ks) w3[ks] = wfrag(W3, t + FW_WAVES, ks);
    }
    const int c = 16 * t + r;
    if (c < n_out) {
      const float bias = b3[c];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = row0 + 4 * g + q;
        if (row < M) O[(size_t)row * ldo + c] = acc[q] + bias;
      }
    }
  }
}

template <class T> __device__ inline float asf(T v);
template <> __device__ inline float asf<float>(float v) { return v; }
template <> __device__ inline float asf<uint16_t>(uint16_t v) {
  return bf16_to_f32(v);
}

// ---------------------------------------------------------------------------
// forward layer on VALU, FP32 weights (the FP32 precision of a network)
// ---------------------------------------------------------------------------
// Y[m][n] = act(sum_k X[m][k] W[n][k] + b[n]) for n < N, k < K: X [M][ldx]
// (BF16 or FP32), W FP32 [N][ldw], Y FP32 [M][ldy].  16 x 16 output tiles,
// 16-wide K slices through LDS; the sum runs over k in ascending order.
template <class TX, bool RELU>
__global__ void __launch_bounds__(256)
    k_dense_f32(int M, int K, int N, const TX *__restrict__ X, int ldx,
                const float *__restrict__ W, int ldw, const float *__restrict__ b,
                float *__restrict__ Y, int ldy) {
  __shared__ float sx[16][17], sw[16][17];
  const int tm = threadIdx.x / 16, tn = threadIdx.x % 16;
  const int m = blockIdx.x * 16 + tm, n = blockIdx.y * 16 + tn;
  float acc = 0.f;
  for (int k0 = 0; k0 < K; k0 += 16) {
    const int r = threadIdx.x / 16, c = threadIdx.x % 16;
    const int mi = blockIdx.x * 16 + r, ni = blockIdx.y * 16 + r, kc = k0 + c;
    sx[r][c] = (mi < M && kc < K) ? asf<TX>(X[(size_t)mi * ldx + kc]) : 0.f;
    sw[r][c] = (ni < N && kc < K) ? W[(size_t)ni * ldw + kc] : 0.f;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) acc += sx[tm][q] * sw[tn][q];
    __syncthreads();
  }
  if (m < M && n < N) {
    float v = acc + b[n];
    if (RELU) v = fmaxf(v, 0.0f);
    Y[(size_t)m * ldy + n] = v;
  }
}

// ---------------------------------------------------------------------------
// loss of the coarse-operator factor
// ---------------------------------------------------------------------------
// The output is a lower-triangular K x K factor L (row-major packed); per
// sample, T holds y and alpha* (2K values) and the loss is the mean of
// (L L^T y - alpha*)^2; dL = g v^T + y (L^T g)^T with v = L^T y and g the
// loss gradient with respect to L L^T y.  One wave per sample, lane i the
// row (column) i of the triangular products, the factor in LDS.
constexpr int LF_WAVES = 4;
template <int K>
__global__ void __launch_bounds__(64 * LF_WAVES)
    k_loss_factor(int B, const float *__restrict__ O, int ldo,
                  const float *__restrict__ T, float *__restrict__ dO, int lddo,
                  double *__restrict__ lossp) {
  constexpr int KK = K * (K + 1) / 2;
  struct Sample {
    double dd[K];
    float o[KK], y[K], v[K], g[K], w[K];
  };
  __shared__ Sample smp[LF_WAVES];
  const int wv = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int b = blockIdx.x * LF_WAVES + wv;
  if (b >= B) return;  // a whole wave; the waves do not wait for each other
  Sample &S = smp[wv];
  const float *o = O + (size_t)b * ldo, *t = T + (size_t)b * 2 * K;
  for (int q = l; q < KK; q += 64) S.o[q] = o[q];
  const int i = l < K ? l : K - 1;  // lanes beyond K repeat the last row
  const float yi = t[i], as = t[K + i];
  S.y[i] = yi;
  wave_lds_sync();
  const int row = i * (i + 1) / 2;
  float v = 0.f;
#pragma unroll
  for (int m = 0; m < K; ++m)
    if (m >= i) v += S.o[m * (m + 1) / 2 + i] * S.y[m];
  S.v[i] = v;
  wave_lds_sync();
  float a = 0.f;
#pragma unroll
  for (int m = 0; m < K; ++m)
    if (m <= i) a += S.o[row + m] * S.v[m];
  const float d = a - as;
  S.g[i] = (float)(2.0 / ((double)B * K)) * d;
  S.dd[i] = (double)d * (double)d;
  wave_lds_sync();
  float w = 0.f;
#pragma unroll
  for (int m = 0; m < K; ++m)
    if (m >= i) w += S.o[m * (m + 1) / 2 + i] * S.g[m];
  S.w[i] = w;
  wave_lds_sync();
  for (int q = l; q < KK; q += 64) {
    // packed index q = a (a + 1) / 2 + c
    int ra = (int)((sqrtf(8.f * (float)q + 1.f) - 1.f) * 0.5f);
    ra -= ra * (ra + 1) / 2 > q;
    ra += (ra + 1) * (ra + 2) / 2 <= q;
    const int c = q - ra * (ra + 1) / 2;
    dO[(size_t)b * lddo + q] = S.g[ra] * S.v[c] + S.y[ra] * S.w[c];
  }
  double loss = 0.0;
#pragma unroll
  for (int m = 0; m < K; ++m) loss += S.dd[m];
  if (l == 0) lossp[b] = loss;
}

// ---------------------------------------------------------------------------
// backward pass of one layer (FP32 matrix instructions)
// ---------------------------------------------------------------------------
// v_mfma_f32_16x16x4_f32: lane l holds A[l % 16][l / 16] and
// B[l / 16][l % 16]; the result C[4 (l / 16) + q][l % 16] is slot q.
constexpr int BW_WAVES = 8;

template <class TX, class TW> struct LayerGrad {
  int B, N, K;                // samples, outputs, inputs of the layer
  const float *dY;            // [B][lddy], the gradient at the layer's output
  int lddy;
  const TX *X;                // [B][ldx], the layer's input
  int ldx;
  float *dW, *db, *dW2, *db2; // gradients; *2: a second copy, or null
  // the gradient at the input through its relu, K = 128 (null: none):
  // dZ = (dY W) o (Hf > 0)
  const TW *W;                // [N][128]
  const float *Hf;            // [B][128]
  float *dZ;                  // [B][128]
  // mean loss (null: none)
  const double *lossp;
  double *loss;
  double loss_count;
  int tiles_w, tiles_x;       // workgroups per kind
};

// dW[n][k] = sum_b dY[b][n] X[b][k] for 16 n and 32 k, the samples dealt to
// the eight waves four at a time and their sums added in wave order; the
// first k tile also sums dY itself (db), as one more column of ones
template <class TX, class TW>
__device__ inline void grad_w_tile(const LayerGrad<TX, TW> &p, int tile, float *red) {
  const int nk = (p.K + 31) / 32;
  const int n0 = tile / nk * 16, k0 = tile % nk * 32;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, r = l & 15, g = l >> 4;
  const bool n_ok = n0 + r < p.N, k_ok0 = k0 + r < p.K, k_ok1 = k0 + 16 + r < p.K;
  f32x4 c0 = {0.f, 0.f, 0.f, 0.f}, c1 = c0, cb = c0;
  constexpr int U = 8;
  for (int b0 = 4 * w; b0 < p.B; b0 += 4 * BW_WAVES * U) {
    float a[U], x0[U], x1[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int b = b0 + 4 * BW_WAVES * u + g;
      const bool ok = b < p.B;
      a[u] = ok && n_ok ? p.dY[(size_t)b * p.lddy + n0 + r] : 0.f;
      x0[u] = ok && k_ok0 ? asf<TX>(p.X[(size_t)b * p.ldx + k0 + r]) : 0.f;
      x1[u] = ok && k_ok1 ? asf<TX>(p.X[(size_t)b * p.ldx + k0 + 16 + r]) : 0.f;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      c0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u], x0[u], c0, 0, 0, 0);
      c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u], x1[u], c1, 0, 0, 0);
      if (k0 == 0) cb = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u], 1.f, cb, 0, 0, 0);
    }
  }
  // red[wave][3][16 rows][16 columns]
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int at = w * 768 + (4 * g + q) * 16 + r;
    red[at] = c0[q];
    red[at + 256] = c1[q];
    red[at + 512] = cb[q];
  }
  __syncthreads();
  const int t = threadIdx.x;  // 512 threads: tile t / 256, row, column
  const int n = n0 + (t & 255) / 16, k = k0 + (t / 256) * 16 + (t & 15);
  float s = 0.f;
#pragma unroll
  for (int q = 0; q < BW_WAVES; ++q) s += red[q * 768 + t];
  if (n < p.N && k < p.K) {
    p.dW[(size_t)n * p.K + k] = s;
    if (p.dW2) p.dW2[(size_t)n * p.K + k] = s;
  }
  if (k0 == 0 && t < 16 && n0 + t < p.N) {
    float sb = 0.f;
#pragma unroll
    for (int q = 0; q < BW_WAVES; ++q) sb += red[q * 768 + 512 + t * 16];
    p.db[n0 + t] = sb;
    if (p.db2) p.db2[n0 + t] = sb;
  }
}

// four consecutive values of a row of weights
__device__ inline void load4(const float *p, float (&v)[4]) {
  // (a layer's rows of parameters are only 4-byte aligned)
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = p[j];
}
__device__ inline void load4(const uint16_t *p, float (&v)[4]) {
  const s16x4 x = *reinterpret_cast<const s16x4 *>(p);
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = bf16_to_f32((uint16_t)x[j]);
}

// dZ[b][k] = (sum_n dY[b][n] W[n][k]) (Hf[b][k] > 0) for 16 b.  Wave w takes
// the columns 64 (w % 2) .. + 63 and every fourth chunk of 16 outputs n
// (w / 2 first); the four partial sums are added in order.  Within a chunk,
// slot q of lane group g takes n = 4 g + q and tile j the columns 4 r + j,
// so that a lane reads consecutive entries of its row of dY and of W (one
// column a load and every wave reading all of dY: 24 us against 12 at 512 x 378).
template <class TX, class TW>
__device__ inline void grad_x_tile(const LayerGrad<TX, TW> &p, int tile, float *red) {
  constexpr int H = 128;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, r = l & 15, g = l >> 4;
  const int b = tile * 16 + r, k0 = 64 * (w & 1) + 4 * r;
  f32x4 c[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) c[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int n0 = 16 * (w >> 1); n0 < p.N; n0 += 64) {
    float a[4], x[4][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int n = n0 + 4 * g + q;
      a[q] = n < p.N && b < p.B ? p.dY[(size_t)b * p.lddy + n] : 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) x[q][j] = 0.f;
      if (n < p.N) load4(p.W + (size_t)n * H + k0, x[q]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        c[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[q], x[q][j], c[j], 0, 0, 0);
  }
  // red[quarter][row][column]
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int j = 0; j < 4; ++j) red[(w >> 1) * 2048 + (4 * g + q) * H + k0 + j] = c[j][q];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int t = u * 64 * BW_WAVES + threadIdx.x, row = tile * 16 + t / H;
    if (row < p.B) {
      const size_t at = (size_t)row * H + t % H;
      const float s = ((red[t] + red[2048 + t]) + red[4096 + t]) + red[6144 + t];
      p.dZ[at] = p.Hf[at] > 0.f ? s : 0.f;
    }
  }
}

// workgroups [0, tiles_x) form dZ, the next tiles_w the weight gradients, one
// more (when asked for) the mean loss
template <class TX, class TW>
__global__ void __launch_bounds__(64 * BW_WAVES) k_layer_grad(LayerGrad<TX, TW> p) {
  __shared__ float red[4 * 2048];  // >= BW_WAVES * 768
  __shared__ double sm[BW_WAVES];
  const int q = blockIdx.x;
  if (q < p.tiles_x) {
    grad_x_tile(p, q, red);
  } else if (q < p.tiles_x + p.tiles_w) {
    grad_w_tile(p, q - p.tiles_x, red);
  } else {
    double a = 0.0;
    for (int m = threadIdx.x; m < p.B; m += 64 * BW_WAVES) a += p.lossp[m];
    const double s = block_sum<64 * BW_WAVES>(a, sm);
    if (threadIdx.x == 0) *p.loss = s / p.loss_count;
  }
}

__global__ void k_adam(int64_t n, float *__restrict__ th, float *__restrict__ m,
                       float *__restrict__ v, const float *__restrict__ g,
                       float lr, float b1, float b2, float eps, float c1,
                       float c2) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n) return;
  const float gq = g[q];
  const float mq = b1 * m[q] + (1.f - b1) * gq;
  const float vq = b2 * v[q] + (1.f - b2) * gq * gq;
  m[q] = mq;
  v[q] = vq;
  th[q] -= lr * (mq / c1) / (sqrtf(vq / c2) + eps);
}

// BF16 weights from the FP32 master: W1b [H][kin], W2b [H][H],
// W3b [w3rows][H] (rows >= n_out zero)
__global__ void k_refresh(int n_in, int kin, int H, int n_out, int w3rows,
                          const float *__restrict__ th, uint16_t *__restrict__ W1b,
                          uint16_t *__restrict__ W2b, uint16_t *__restrict__ W3b) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t n1 = (int64_t)H * kin, n2 = (int64_t)H * H,
                n3 = (int64_t)w3rows * H;
  const float *W1 = th, *W2 = th + (int64_t)H * n_in + H,
              *W3 = W2 + (int64_t)H * H + H;
  if (q < n1) {
    const int r = (int)(q / kin), c = (int)(q % kin);
    W1b[q] = c < n_in ? f32_to_bf16(W1[(int64_t)r * n_in + c]) : 0;
  } else if (q < n1 + n2) {
    const int64_t p = q - n1;
    W2b[p] = f32_to_bf16(W2[p]);
  } else if (q < n1 + n2 + n3) {
    const int64_t p = q - n1 - n2;
    const int r = (int)(p / H), c = (int)(p % H);
    W3b[p] = r < n_out ? f32_to_bf16(W3[(int64_t)r * H + c]) : 0;
  }
}

}  // namespace sem

// ---------------------------------------------------------------------------
// the network object
// ---------------------------------------------------------------------------
struct sem_mlp {
  int n_in = 0, H = 0, n_out = 0, kin = 0;
  int prec = SEM_BF16;      // SEM_BF16 (MFMA, BF16 weights) or SEM_FP32 (VALU)
  int w3rows = 16;          // rows of W3b: n_out, padded
  int64_t np = 0, step = 0;
  uint64_t version = 1;     // changes whenever the parameters change
  double damping = 1.0;     // scale of the correction in the preconditioner
  double ref_rate = 0.0;    // Jacobi-PCG log10 residual drop per iteration
                            // on the training problem (0: unknown)
  sem::DevBuf th, m, v, grad, W1b, W2b, W3b;
  sem::DevBuf dev_damping;  // device copy of `damping` read by the correction
                            // kernels (captured graphs see its updates)
  // training scratch, sized for `cap` samples
  int cap = 0;
  sem::DevBuf h1b, h2b, h1f, h2f, of, dO, dz2, dz1, lossp;
  double *host_loss = nullptr;  // pinned; the loss kernel writes it
  ~sem_mlp() {
    if (host_loss) (void)hipHostFree(host_loss);
  }
};

namespace sem {

void mlp_set_damping(sem_mlp *net, double d, double rate);

static int64_t mlp_np(int n_in, int H, int n_out) {
  return (int64_t)H * n_in + H + (int64_t)H * H + H + (int64_t)n_out * H + n_out;
}

void mlp_refresh(sem_mlp *net, hipStream_t s) {
  const int64_t n = (int64_t)net->H * net->kin + (int64_t)net->H * net->H +
                    (int64_t)net->w3rows * net->H;
  hipLaunchKernelGGL(k_refresh, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                     net->n_in, net->kin, net->H, net->n_out, net->w3rows,
                     net->th.as<float>(),
                     net->W1b.as<uint16_t>(), net->W2b.as<uint16_t>(),
                     net->W3b.as<uint16_t>());
  SEM_HIP(hipGetLastError());
}

sem_mlp *mlp_create(int n_in, int H, int n_out, uint64_t seed) {
  if (n_in < 1 || n_in > 4096) fail(SEM_ERR_ARG, "mlp: n_in must be in 1..4096");
  if (H != 128) fail(SEM_ERR_ARG, "mlp: hidden width must be 128");
  if (n_out < 1 || n_out > 1024) fail(SEM_ERR_ARG, "mlp: n_out must be in 1..1024");
  sem_mlp *net = new sem_mlp();
  try {
    net->n_in = n_in;
    net->H = H;
    net->n_out = n_out;
    net->kin = (n_in + 15) / 16 * 16;
    net->w3rows = (n_out + 15) / 16 * 16;
    net->np = mlp_np(n_in, H, n_out);
    net->th.alloc(net->np * 4);
    net->m.alloc(net->np * 4);
    net->v.alloc(net->np * 4);
    net->grad.alloc(net->np * 4);
    net->W1b.alloc((size_t)H * net->kin * 2);
    net->W2b.alloc((size_t)H * H * 2);
    net->W3b.alloc((size_t)net->w3rows * H * 2);
    // He initialisation (normal, std sqrt(2 / fan_in)), zero biases
    std::vector<float> th(net->np, 0.0f);
    std::mt19937_64 rng(seed);
    std::normal_distribution<double> nd(0.0, 1.0);
    int64_t k = 0;
    auto fill = [&](int rows, int cols) {
      const double sd = std::sqrt(2.0 / cols);
      for (int64_t q = 0; q < (int64_t)rows * cols; ++q) th[k++] = (float)(nd(rng) * sd);
      k += rows;  // bias
    };
    fill(H, n_in);
    fill(H, H);
    fill(n_out, H);
    SEM_HIP(hipMemcpy(net->th.p, th.data(), net->np * 4, hipMemcpyHostToDevice));
    SEM_HIP(hipMemset(net->m.p, 0, net->np * 4));
    SEM_HIP(hipMemset(net->v.p, 0, net->np * 4));
    SEM_HIP(hipHostMalloc((void **)&net->host_loss, sizeof(double), 0));
    net->dev_damping.alloc(sizeof(float));
    mlp_set_damping(net, 1.0, 0.0);
    mlp_refresh(net, nullptr);
    SEM_HIP(hipDeviceSynchronize());
  } catch (...) {
    delete net;
    throw;
  }
  return net;
}

void mlp_set_params(sem_mlp *net, const float *host, int64_t n) {
  net->version += 1;
  if (n != net->np) fail(SEM_ERR_ARG, "mlp_set_params: wrong parameter count");
  SEM_HIP(hipMemcpy(net->th.p, host, n * 4, hipMemcpyHostToDevice));
  SEM_HIP(hipMemset(net->m.p, 0, n * 4));
  SEM_HIP(hipMemset(net->v.p, 0, n * 4));
  net->step = 0;
  mlp_refresh(net, nullptr);
  SEM_HIP(hipDeviceSynchronize());
}

void mlp_get_params(const sem_mlp *net, float *host, int64_t n) {
  if (n != net->np) fail(SEM_ERR_ARG, "mlp_get_params: wrong parameter count");
  SEM_HIP(hipDeviceSynchronize());
  SEM_HIP(hipMemcpy(host, net->th.p, n * 4, hipMemcpyDeviceToHost));
}

static void ensure_scratch(sem_mlp *net, int B) {
  if (B <= net->cap) return;
  const int H = net->H;
  net->h1b.alloc((size_t)B * H * 2);
  net->h2b.alloc((size_t)B * H * 2);
  net->h1f.alloc((size_t)B * H * 4);
  net->h2f.alloc((size_t)B * H * 4);
  const int wo = net->n_out > 16 ? net->n_out : 16;
  net->of.alloc((size_t)B * wo * 4);
  net->dO.alloc((size_t)B * wo * 4);
  net->dz2.alloc((size_t)B * H * 4);
  net->dz1.alloc((size_t)B * H * 4);
  net->lossp.alloc((size_t)B * 8);
  net->cap = B;
}

// forward of B samples X [B][ldx] BF16 (ldx >= kin, padding columns zero)
// into O [B][ldo] FP32.  FP32 precision uses the FP32 scratch; keep: the
// hidden activations stay in the network's scratch for a backward pass (BF16
// precision: h1b, h2b, the next layer's inputs, and their FP32 values h1f,
// h2f)
static void forward_into(sem_mlp *net, const uint16_t *X, int ldx, int B, float *O, int ldo,
                         bool keep, hipStream_t s) {
  if (B <= 0) return;
  if (ldx < net->kin || ldx % 16 != 0)
    fail(SEM_ERR_ARG, "mlp_forward: ldx must be >= padded n_in and a multiple of 16");
  const int H = net->H;
  const float *W1 = net->th.as<float>();
  const float *b1 = W1 + (int64_t)H * net->n_in;
  const float *W2 = b1 + H;
  const float *b2 = W2 + (int64_t)H * H;
  const float *W3 = b2 + H;
  const float *b3 = W3 + (int64_t)net->n_out * H;
  if (keep || net->prec == SEM_FP32) ensure_scratch(net, B);
  if (net->prec == SEM_FP32) {
    const unsigned gm = (unsigned)((B + 15) / 16);
    float *h1f = net->h1f.as<float>(), *h2f = net->h2f.as<float>();
    hipLaunchKernelGGL((k_dense_f32<uint16_t, true>), dim3(gm, H / 16), dim3(256),
                       0, s, B, net->n_in, H, X, ldx, W1, net->n_in, b1, h1f, H);
    hipLaunchKernelGGL((k_dense_f32<float, true>), dim3(gm, H / 16), dim3(256), 0,
                       s, B, H, H, (const float *)h1f, H, W2, H, b2, h2f, H);
    hipLaunchKernelGGL((k_dense_f32<float, false>),
                       dim3(gm, (unsigned)((net->n_out + 15) / 16)), dim3(256), 0,
                       s, B, H, net->n_out, (const float *)h2f, H, W3, H, b3, O,
                       ldo);
    SEM_HIP(hipGetLastError());
    return;
  }
  // (a launch holds fewer than 2^32 threads, here 32 a sample)
  constexpr int ROWS = 1 << 26;
  auto kept = [&](auto *p, int64_t r0) { return keep ? p + r0 * H : nullptr; };
  for (int64_t r0 = 0; r0 < B; r0 += ROWS) {
    const int n = (int)std::min<int64_t>(B - r0, ROWS);
    hipLaunchKernelGGL(k_forward_mfma, dim3((unsigned)((n + 15) / 16)), dim3(64 * FW_WAVES), 0,
                       s, n, net->kin, net->n_out, X + r0 * ldx, ldx, net->W1b.as<uint16_t>(),
                       b1, net->W2b.as<uint16_t>(), b2, net->W3b.as<uint16_t>(), b3,
                       O + r0 * ldo, ldo, kept(net->h1b.as<uint16_t>(), r0),
                       kept(net->h2b.as<uint16_t>(), r0), kept(net->h1f.as<float>(), r0),
                       kept(net->h2f.as<float>(), r0));
  }
  SEM_HIP(hipGetLastError());
}

// whether an output of n floats at p lies over the samples X [B][ldx]
static bool over_input(const float *p, int64_t n, const uint16_t *X, int ldx, int B) {
  const uintptr_t a = (uintptr_t)p, x = (uintptr_t)X;
  return a < x + (uintptr_t)((int64_t)B * ldx * 2) && x < a + (uintptr_t)(n * 4);
}

void mlp_forward(sem_mlp *net, const uint16_t *X, int ldx, int B, float *O,
                 int ldo, hipStream_t s) {
  if (B <= 0 || !over_input(O, (int64_t)B * ldo, X, ldx, B))
    return forward_into(net, X, ldx, B, O, ldo, false, s);
  // in place: workgroups store their samples' outputs while others still read
  // theirs, so the outputs take the way through the scratch
  ensure_scratch(net, B);
  float *of = net->of.as<float>();
  forward_into(net, X, ldx, B, of, ldo, false, s);
  SEM_HIP(hipMemcpyAsync(O, of, (size_t)B * ldo * 4, hipMemcpyDeviceToDevice, s));
}

// Backward pass from net->dO (written by a loss kernel) into net->grad
// (flat parameter order) and, when non-null, grad, on the weights and layer
// inputs the forward pass used; returns the mean loss over B samples of
// `count` terms each.  TH: the type of the hidden layers' values and of the
// weights in the products (BF16, or FP32 for an FP32 network).
template <class TH>
static double mlp_backward(sem_mlp *net, const uint16_t *X, int ldx, int B, int count,
                           float *grad, hipStream_t s) {
  constexpr bool f32 = sizeof(TH) == 4;
  const int H = net->H;
  const int wo = net->n_out > 16 ? net->n_out : 16;
  const int64_t o1 = 0, ob1 = o1 + (int64_t)H * net->n_in, o2 = ob1 + H,
                ob2 = o2 + (int64_t)H * H, o3 = ob2 + H, ob3 = o3 + (int64_t)net->n_out * H;
  float *g = net->grad.as<float>();
  const float *th = net->th.as<float>();
  const TH *W2 = f32 ? (const TH *)(th + o2) : (const TH *)net->W2b.p;
  const TH *W3 = f32 ? (const TH *)(th + o3) : (const TH *)net->W3b.p;
  const TH *h1 = f32 ? (const TH *)net->h1f.p : (const TH *)net->h1b.p;
  const TH *h2 = f32 ? (const TH *)net->h2f.p : (const TH *)net->h2b.p;
  auto second = [&](int64_t off) { return grad ? grad + off : nullptr; };
  auto launch = [&](auto p) {
    p.B = B;
    p.tiles_w = (p.N + 15) / 16 * ((p.K + 31) / 32);
    p.tiles_x = p.dZ ? (B + 15) / 16 : 0;
    const int grid = p.tiles_x + p.tiles_w + (p.loss ? 1 : 0);
    void (*kernel)(decltype(p)) = k_layer_grad;
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(64 * BW_WAVES), 0, s, p);
  };
  LayerGrad<TH, TH> p3{};
  p3.N = net->n_out, p3.K = H;
  p3.dY = net->dO.as<float>(), p3.lddy = wo;
  p3.X = h2, p3.ldx = H;
  p3.dW = g + o3, p3.db = g + ob3, p3.dW2 = second(o3), p3.db2 = second(ob3);
  p3.W = W3, p3.Hf = net->h2f.as<float>(), p3.dZ = net->dz2.as<float>();
  p3.lossp = net->lossp.as<double>(), p3.loss = net->host_loss;
  p3.loss_count = (double)B * count;
  launch(p3);
  LayerGrad<TH, TH> p2{};
  p2.N = H, p2.K = H;
  p2.dY = net->dz2.as<float>(), p2.lddy = H;
  p2.X = h1, p2.ldx = H;
  p2.dW = g + o2, p2.db = g + ob2, p2.dW2 = second(o2), p2.db2 = second(ob2);
  p2.W = W2, p2.Hf = net->h1f.as<float>(), p2.dZ = net->dz1.as<float>();
  launch(p2);
  // layer 1 (the input X is BF16 in both precisions)
  LayerGrad<uint16_t, TH> p1{};
  p1.N = H, p1.K = net->n_in;
  p1.dY = net->dz1.as<float>(), p1.lddy = H;
  p1.X = X, p1.ldx = ldx;
  p1.dW = g + o1, p1.db = g + ob1, p1.dW2 = second(o1), p1.db2 = second(ob1);
  launch(p1);
  SEM_HIP(hipGetLastError());
  SEM_HIP(hipStreamSynchronize(s));
  return *net->host_loss;
}

// loss and gradient of the coarse-operator factor (n_out = K(K+1)/2,
// K in {1, 8, 27}); T [B][2K] holds y and alpha* per sample.  The gradient
// goes to the network's own buffer and, when non-null, to grad.
double mlp_loss_grad_factor(sem_mlp *net, const uint16_t *X, int ldx,
                            const float *T, int K, int B, float *grad,
                            hipStream_t s) {
  if (net->n_out != K * (K + 1) / 2 || (K != 1 && K != 8 && K != 27))
    fail(SEM_ERR_ARG, "mlp_loss_grad_factor: K must be 1, 8 or 27 and "
                      "n_out = K(K+1)/2");
  ensure_scratch(net, B);
  const int wo = net->n_out > 16 ? net->n_out : 16;
  // a gradient that lies over X, which the last layer's launch still reads, is
  // copied after it
  const bool over = grad && over_input(grad, net->np, X, ldx, B);
  float *copy = over ? grad : nullptr;
  if (over) grad = nullptr;
  forward_into(net, X, ldx, B, net->of.as<float>(), wo, true, s);
  const dim3 g((unsigned)((B + LF_WAVES - 1) / LF_WAVES)), t(64 * LF_WAVES);
  if (K == 1)
    hipLaunchKernelGGL(k_loss_factor<1>, g, t, 0, s, B, net->of.as<float>(), wo, T,
                       net->dO.as<float>(), wo, net->lossp.as<double>());
  else if (K == 8)
    hipLaunchKernelGGL(k_loss_factor<8>, g, t, 0, s, B, net->of.as<float>(), wo, T,
                       net->dO.as<float>(), wo, net->lossp.as<double>());
  else
    hipLaunchKernelGGL(k_loss_factor<27>, g, t, 0, s, B, net->of.as<float>(), wo, T,
                       net->dO.as<float>(), wo, net->lossp.as<double>());
  SEM_HIP(hipGetLastError());
  const double loss = net->prec == SEM_FP32
                          ? mlp_backward<float>(net, X, ldx, B, K, grad, s)
                          : mlp_backward<uint16_t>(net, X, ldx, B, K, grad, s);
  if (copy)
    SEM_HIP(hipMemcpyAsync(copy, net->grad.p, (size_t)net->np * 4, hipMemcpyDeviceToDevice, s));
  return loss;
}

uint64_t mlp_version(const sem_mlp *net) { return net->version; }

void mlp_set_precision(sem_mlp *net, int prec) {
  if (prec != SEM_BF16 && prec != SEM_FP32)
    fail(SEM_ERR_ARG, "mlp_set_precision: SEM_BF16 or SEM_FP32");
  SEM_HIP(hipDeviceSynchronize());  // no forward pass may be in flight
  net->prec = prec;
  net->version += 1;  // outputs derived from the network must be recomputed
}

int mlp_precision(const sem_mlp *net) { return net->prec; }

void mlp_adam(sem_mlp *net, const float *grad, double lr, double b1, double b2,
              double eps, hipStream_t s) {
  net->version += 1;
  net->step += 1;
  const double c1 = 1.0 - std::pow(b1, (double)net->step);
  const double c2 = 1.0 - std::pow(b2, (double)net->step);
  hipLaunchKernelGGL(k_adam, dim3((unsigned)((net->np + 255) / 256)), dim3(256), 0,
                     s, net->np, net->th.as<float>(), net->m.as<float>(),
                     net->v.as<float>(), grad ? grad : net->grad.as<float>(),
                     (float)lr, (float)b1, (float)b2, (float)eps, (float)c1,
                     (float)c2);
  SEM_HIP(hipGetLastError());
  mlp_refresh(net, s);
}

// ---------------------------------------------------------------------------
// checkpoint: header, FP32 master parameters, Adam moments, CRC-32 (IEEE
// 802.3 polynomial, reflected) of everything before it
// ---------------------------------------------------------------------------
static uint32_t crc32_update(uint32_t crc, const unsigned char *p, size_t n) {
  static uint32_t table[256];
  static bool init = false;
  if (!init) {
    for (uint32_t i = 0; i < 256; ++i) {
      uint32_t c = i;
      for (int k = 0; k < 8; ++k) c = (c & 1) ? 0xEDB88320u ^ (c >> 1) : c >> 1;
      table[i] = c;
    }
    init = true;
  }
  crc = ~crc;
  for (size_t q = 0; q < n; ++q) crc = table[(crc ^ p[q]) & 0xff] ^ (crc >> 8);
  return ~crc;
}

struct CkptHeader {
  char magic[8];  // "SEMMLP01"
  uint32_t version, n_in, H, n_out;
  uint64_t step, np;
  double damping, ref_rate;
};

void mlp_save(const sem_mlp *net, const char *path) {
  SEM_HIP(hipDeviceSynchronize());
  CkptHeader hd{};
  memcpy(hd.magic, "SEMMLP01", 8);
  hd.version = 2;
  hd.damping = net->damping;
  hd.ref_rate = net->ref_rate;
  hd.n_in = net->n_in;
  hd.H = net->H;
  hd.n_out = net->n_out;
  hd.step = (uint64_t)net->step;
  hd.np = (uint64_t)net->np;
  std::vector<float> buf(3 * net->np);
  SEM_HIP(hipMemcpy(buf.data(), net->th.p, net->np * 4, hipMemcpyDeviceToHost));
  SEM_HIP(hipMemcpy(buf.data() + net->np, net->m.p, net->np * 4,
                    hipMemcpyDeviceToHost));
  SEM_HIP(hipMemcpy(buf.data() + 2 * net->np, net->v.p, net->np * 4,
                    hipMemcpyDeviceToHost));
  uint32_t crc = crc32_update(0, (const unsigned char *)&hd, sizeof hd);
  crc = crc32_update(crc, (const unsigned char *)buf.data(), buf.size() * 4);
  std::ofstream f(path, std::ios::binary);
  if (!f) fail(SEM_ERR_ARG, "mlp_save: cannot open file");
  f.write((const char *)&hd, sizeof hd);
  f.write((const char *)buf.data(), buf.size() * 4);
  f.write((const char *)&crc, 4);
  if (!f) fail(SEM_ERR_ARG, "mlp_save: write failed");
}

sem_mlp *mlp_load(const char *path) {
  std::ifstream f(path, std::ios::binary);
  if (!f) fail(SEM_ERR_ARG, "mlp_load: cannot open file");
  CkptHeader hd{};
  f.read((char *)&hd, sizeof hd);
  if (!f || memcmp(hd.magic, "SEMMLP01", 8) != 0 || hd.version != 2)
    fail(SEM_ERR_ARG, "mlp_load: not a network checkpoint");
  if (hd.H != 128 || hd.n_in < 1 || hd.n_in > 4096 || hd.n_out < 1 ||
      hd.n_out > 1024 || hd.np != (uint64_t)mlp_np(hd.n_in, hd.H, hd.n_out) ||
      !std::isfinite(hd.damping) || !std::isfinite(hd.ref_rate))
    fail(SEM_ERR_ARG, "mlp_load: inconsistent shapes");
  std::vector<float> buf(3 * hd.np);
  f.read((char *)buf.data(), buf.size() * 4);
  uint32_t crc_file = 0;
  f.read((char *)&crc_file, 4);
  if (!f) fail(SEM_ERR_ARG, "mlp_load: truncated checkpoint");
  uint32_t crc = crc32_update(0, (const unsigned char *)&hd, sizeof hd);
  crc = crc32_update(crc, (const unsigned char *)buf.data(), buf.size() * 4);
  if (crc != crc_file) fail(SEM_ERR_ARG, "mlp_load: checksum mismatch");
  sem_mlp *net = mlp_create(hd.n_in, hd.H, hd.n_out, 0);
  try {
    SEM_HIP(hipMemcpy(net->th.p, buf.data(), hd.np * 4, hipMemcpyHostToDevice));
    SEM_HIP(hipMemcpy(net->m.p, buf.data() + hd.np, hd.np * 4,
                      hipMemcpyHostToDevice));
    SEM_HIP(hipMemcpy(net->v.p, buf.data() + 2 * hd.np, hd.np * 4,
                      hipMemcpyHostToDevice));
    net->step = (int64_t)hd.step;
    mlp_set_damping(net, hd.damping, hd.ref_rate);
    mlp_refresh(net, nullptr);
    SEM_HIP(hipDeviceSynchronize());
  } catch (...) {
    delete net;
    throw;
  }
  return net;
}

void mlp_destroy(sem_mlp *net) { delete net; }

void mlp_info(const sem_mlp *net, int *n_in, int *H, int *n_out, int64_t *np,
              int64_t *step) {
  if (n_in) *n_in = net->n_in;
  if (H) *H = net->H;
  if (n_out) *n_out = net->n_out;
  if (np) *np = net->np;
  if (step) *step = net->step;
}

int mlp_padded_inputs(const sem_mlp *net) { return net->kin; }

double mlp_damping(const sem_mlp *net) { return net->damping; }
double mlp_ref_rate(const sem_mlp *net) { return net->ref_rate; }
void mlp_set_damping(sem_mlp *net, double d, double rate) {
  net->damping = d;
  net->ref_rate = rate;
  const float f = (float)d;
  SEM_HIP(hipDeviceSynchronize());  // no solve may be reading it
  SEM_HIP(hipMemcpy(net->dev_damping.p, &f, sizeof f, hipMemcpyHostToDevice));
}

const float *mlp_damping_dev(const sem_mlp *net) {
  return net->dev_damping.as<float>();
}

}  // namespace sem
