// Document-topic encoder: a d_in -> hidden -> hidden -> k_out perceptron that
// maps a whitened document to topic proportions (GELU hidden layers, softmax
// output), standing in for the per-document simplex-constrained solve of the
// inference step, which stays as its judge and fallback.
//
//   forward : Z1 = X W1 + b1, H1 = gelu(Z1), Z2 = H1 W2 + b2, H2 = gelu(Z2),
//             Z3 = H2 W3 + b3, P = softmax(Z3)
//   backward: dZ3 = (P - T)/B, dW3 = H2^T dZ3, dZ2 = (dZ3 W3^T) gelu'(Z2),
//             dW2 = H1^T dZ2, dZ1 = (dZ2 W2^T) gelu'(Z1), dW1 = X^T dZ1,
//             db = column sums of dZ
// Products run on BF16 matrix cores (v_mfma_f32_16x16x32_bf16, FP32
// accumulation); weights are FP32 masters with BF16 copies, activations and
// dZ are rounded to BF16, pre-activations stay FP32.  gelu(z) = z Phi(z),
// Phi(z) = (1 + erf(z / sqrt 2)) / 2, from the device math library's erff and
// expf.  Training minimises the mean cross-entropy against solve outputs by
// Adam.
//
// One block takes a tile of documents through every layer, so activations
// stay on the chip.  A layer is the transposed product Z^T = W^T A^T: the
// weights are the matrix core's A operand and come straight from the caches
// in fragment order, the activations are its B operand (16 documents by 32
// consecutive features, one 16-byte LDS read).  A wave owns 32 output
// features at a time as two 16-row products; row m of product t stands for
// feature 8 (m / 4) + 4 t + m % 4 of the 32, so that the accumulators of a
// lane are 8 consecutive features of one document: one 16-byte LDS store,
// and the next layer's operand with its reduction index in natural order.
// Bound: the vector ALUs (the GELUs, two error functions' worth of code per
// hidden unit and document), then the weights' path out of the caches, which
// is why a block takes 64 documents where there are enough of them: one
// weight fragment then feeds four products.  131072 rows forward at 50 - 256 -
// 256 - 50: 90 us (265 TFLOP/s; 1635 us as four kernels per 4096 rows, the
// activations through memory).  A training step of 4096 rows: k_train 25 us,
// k_grads 9, k_update 7 (220 us as separate products and sums).
#include <algorithm>
#include <cmath>

#include "tlda_internal.h"

namespace tlda {
namespace {

constexpr int kThreads = 512, kWaves = kThreads / 64;

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t to_bf16(float f) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 b16x2 __attribute__((ext_vector_type(2)));
  const b16x2 h = __builtin_convertvector((f32x2{f, 0.f}), b16x2);
  return (uint16_t)(__builtin_bit_cast(uint32_t, h) & 0xffffu);
}
__device__ __forceinline__ uint32_t to_bf16x2(float lo, float hi) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 b16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{lo, hi}), b16x2));
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__host__ __device__ inline int pad32(int n) { return (n + 31) / 32 * 32; }

// Place of weight (k, o) (input k, output o) in the fragments of a product
// whose reduction index is k: 32 x 32 blocks, output blocks outermost; in a
// block product t, then lane (row m = feature as in the file comment, group
// q), then 8 consecutive k.
__host__ __device__ inline size_t frag_at(int k, int o, int k_pad) {
  const int oo = o & 31, kk = k & 31;
  const int t = (oo >> 2) & 1, m = 4 * (oo >> 3) + (oo & 3);
  const size_t block = (size_t)(o >> 5) * (k_pad >> 5) + (k >> 5);
  return ((block * 2 + t) * 64 + (kk >> 3) * 16 + m) * 8 + (kk & 7);
}

// The encoder's device copies of its parameters: BF16 fragments of W1, W2, W3
// (forward: reduction over the input) and of W2, W3 with input and output
// exchanged (backward), all padded to 32 by zeros, and the padded biases.
struct Frags {
  uint16_t *w1, *w2, *w3, *t2, *t3;
  float *b1, *b2, *b3;
};
inline size_t frag_halves(int D, int H, int K) {
  const size_t d = pad32(D), h = pad32(H), k = pad32(K);
  return d * h + 2 * h * h + 2 * h * k;
}
inline size_t bias_floats(int H, int K) { return 2 * (size_t)pad32(H) + pad32(K); }
inline Frags frags_of(const tlda_mlp& m) {
  const size_t d = pad32(m.d_in), h = pad32(m.hidden), k = pad32(m.k_out);
  Frags f;
  f.w1 = m.wfrag;
  f.w2 = f.w1 + d * h;
  f.w3 = f.w2 + h * h;
  f.t2 = f.w3 + h * k;
  f.t3 = f.t2 + h * h;
  f.b1 = m.bpad;
  f.b2 = f.b1 + h;
  f.b3 = f.b2 + h;
  return f;
}

// Writes parameter e's value into the copies.
__device__ inline void put_param(const Frags& f, int D, int H, int K, size_t e, float v) {
  const size_t n1 = (size_t)D * H, n2 = n1 + H, n3 = n2 + (size_t)H * H, n4 = n3 + H,
               n5 = n4 + (size_t)H * K;
  if (e < n1) {
    f.w1[frag_at((int)(e / H), (int)(e % H), pad32(D))] = to_bf16(v);
  } else if (e < n2) {
    f.b1[e - n1] = v;
  } else if (e < n3) {
    const int i = (int)((e - n2) / H), o = (int)((e - n2) % H);
    f.w2[frag_at(i, o, pad32(H))] = to_bf16(v);
    f.t2[frag_at(o, i, pad32(H))] = to_bf16(v);
  } else if (e < n4) {
    f.b2[e - n3] = v;
  } else if (e < n5) {
    const int i = (int)((e - n4) / K), o = (int)((e - n4) % K);
    f.w3[frag_at(i, o, pad32(H))] = to_bf16(v);
    f.t3[frag_at(o, i, pad32(K))] = to_bf16(v);
  } else {
    f.b3[e - n5] = v;
  }
}

__global__ void __launch_bounds__(256) k_refresh(const float* __restrict__ p, int D, int H, int K,
                                                 size_t n, Frags f) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) put_param(f, D, H, K, i, p[i]);
}

// Output features 32 tp .. 32 tp + 31 of NT x 16 documents: acc[t][n][r] of
// lane (l16, q) is feature 32 tp + 8 q + 4 t + r of document 16 n + l16.
// w: the layer's fragments, ks_n blocks of 32 inputs; act: LDS, lda halves a
// document.
template <int NT>
__device__ __forceinline__ void layer(const uint16_t* __restrict__ w, int tp, int ks_n,
                                      const uint16_t* act, int lda, int lane,
                                      floatx4 (&acc)[2][NT]) {
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[t][n] = floatx4{0.f, 0.f, 0.f, 0.f};
  const u32x4* wp = reinterpret_cast<const u32x4*>(w) + (size_t)tp * ks_n * 128 + lane;
  const uint16_t* ap = act + (lane & 15) * lda + 8 * (lane >> 4);
#pragma unroll 4
  for (int ks = 0; ks < ks_n; ++ks) {
    const u32x4 a0 = wp[ks * 128], a1 = wp[ks * 128 + 64];
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      const u32x4 b = *reinterpret_cast<const u32x4*>(ap + n * 16 * lda + ks * 32);
      acc[0][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a0),
                                                          __builtin_bit_cast(bf16x8, b),
                                                          acc[0][n], 0, 0, 0);
      acc[1][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a1),
                                                          __builtin_bit_cast(bf16x8, b),
                                                          acc[1][n], 0, 0, 0);
    }
  }
}

// The 8 values of a lane as one LDS store (v[4 t + r]).
__device__ __forceinline__ void store_act(uint16_t* act, int lda, int tp, int doc, int q,
                                          const float (&v)[8]) {
  const u32x4 h = {to_bf16x2(v[0], v[1]), to_bf16x2(v[2], v[3]), to_bf16x2(v[4], v[5]),
                   to_bf16x2(v[6], v[7])};
  *reinterpret_cast<u32x4*>(act + doc * lda + tp * 32 + 8 * q) = h;
}

__device__ __forceinline__ float phi_cdf2(float z) { return 1.0f + erff(z * 0.70710678118654752f); }

// rows x D floats from X (row-major, contiguous) to LDS documents in BF16;
// documents from `rows` on and features from D on (to Dp) are zeros.
__device__ inline void load_rows(const float* __restrict__ X, int rows, int docs, int D, int Dp,
                                 uint16_t* act, int lda) {
  for (int e = threadIdx.x; e < docs * Dp; e += kThreads) {
    const int r = e / Dp, d = e - r * Dp;
    act[r * lda + d] = r < rows && d < D ? to_bf16(X[(size_t)r * D + d]) : (uint16_t)0;
  }
}
// The same for wide inputs (rows > 0): a wave takes every kWaves-th document, with
// eight loads of a lane on their way at once, where the loop above has one.  A
// narrow network over a wide input is bound by them: 262144 rows of 1024 - 64 -
// 16 take 452 us (2.4 TB/s of X) and took 821; up to 128 inputs the loop above
// is as fast (50 - 256 - 50, 131072 rows) or faster (5 - 16 - 5 by 10%).
constexpr int kWideInput = 128;
template <int DOCS>
__device__ inline void load_wide_rows(const float* __restrict__ X, int rows, int D, int Dp,
                                      uint16_t* act, int lda) {
  constexpr int R = DOCS / kWaves, S = 8 / R;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int d0 = 0; d0 < Dp; d0 += 64 * S) {
    float v[S][R];
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const int r = min(wave + kWaves * i, rows - 1), d = min(d0 + 64 * s + lane, D - 1);
        v[s][i] = X[(size_t)r * D + d];
      }
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const int r = wave + kWaves * i, d = d0 + 64 * s + lane;
        if (d < Dp) act[r * lda + d] = r < rows && d < D ? to_bf16(v[s][i]) : (uint16_t)0;
      }
  }
}

// Softmax of the logits of one document over four lanes (j = 0 .. 3, lane j
// holding entries j, j + 4, ...): p[i] replaces z[i].  Entries l, l + 64, ..
// are added first and the 64 sums pairwise at distances 32, 16, 8, 4, 2, 1.
// Returns log sum exp.  K <= 256.
__device__ inline float softmax_row(float* z, int K, int j) {
  float mx = -INFINITY;
  for (int i = j; i < K; i += 4) mx = fmaxf(mx, z[i]);
  mx = fmaxf(mx, __shfl_xor(mx, 1, 64));
  mx = fmaxf(mx, __shfl_xor(mx, 2, 64));
  float s[16];
#pragma unroll
  for (int m = 0; m < 16; ++m) {
    s[m] = 0.f;
    for (int i = j + 4 * m; i < K; i += 64) {
      const float v = expf(z[i] - mx);
      z[i] = v;
      s[m] += v;
    }
  }
#pragma unroll
  for (int d = 8; d > 0; d >>= 1)
#pragma unroll
    for (int m = 0; m < d; ++m) s[m] += s[m + d];
  float sum = s[0];
  sum += __shfl_xor(sum, 2, 64);
  sum += __shfl_xor(sum, 1, 64);
  const float inv = 1.0f / sum;
  for (int i = j; i < K; i += 4) z[i] *= inv;
  return mx + logf(sum);
}

// theta = softmax(...) for a tile of 16 NT documents.  LDS: two activation
// buffers of 16 NT documents, each as wide as what it holds: lda halves for the
// rows of X and the second hidden layer, ldb for the first and the logits in
// FP32.  WIDE: D > kWideInput (an instance of its own: beside each other the two
// ways in cost the narrow one 0.3%).
template <int NT, bool WIDE>
__global__ void __launch_bounds__(kThreads) k_forward(const float* __restrict__ X, int64_t n_rows,
                                                      int D, int H, int K, int lda, int ldb,
                                                      Frags f, float* __restrict__ theta) {
  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
  constexpr int docs = 16 * NT;
  uint16_t* buf[2] = {lds, lds + docs * lda};
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Dp = pad32(D), Hp = pad32(H), Kp = pad32(K);
  const int64_t row0 = (int64_t)blockIdx.x * docs;
  const int rows = (int)min((int64_t)docs, n_rows - row0);
  if (WIDE)
    load_wide_rows<docs>(X + row0 * D, rows, D, Dp, buf[0], lda);
  else
    load_rows(X + row0 * D, rows, docs, D, Dp, buf[0], lda);
  __syncthreads();
#pragma unroll
  for (int l = 0; l < 2; ++l) {   // hidden layers
    const uint16_t* w = l == 0 ? f.w1 : f.w2;
    const float* bias = l == 0 ? f.b1 : f.b2;
    for (int tp = wave; tp < Hp / 32; tp += kWaves) {
      floatx4 acc[2][NT];
      layer<NT>(w, tp, (l == 0 ? Dp : Hp) / 32, buf[l], l == 0 ? lda : ldb, lane, acc);
      const float* bp = bias + tp * 32 + 8 * q;
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        float h[8];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float z = acc[t][n][r] + bp[4 * t + r];
            h[4 * t + r] = 0.5f * z * phi_cdf2(z);
          }
        store_act(buf[1 - l], l == 0 ? ldb : lda, tp, n * 16 + l16, q, h);
      }
    }
    __syncthreads();
  }
  float* logits = reinterpret_cast<float*>(buf[1]);
  const int ldl = ldb / 2;
  for (int tp = wave; tp < Kp / 32; tp += kWaves) {
    floatx4 acc[2][NT];
    layer<NT>(f.w3, tp, Hp / 32, buf[0], lda, lane, acc);
    const float* bp = f.b3 + tp * 32 + 8 * q;
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          logits[(n * 16 + l16) * ldl + tp * 32 + 8 * q + 4 * t + r] = acc[t][n][r] + bp[4 * t + r];
  }
  __syncthreads();
  if (tid < 4 * docs) softmax_row(logits + (tid >> 2) * ldl, K, tid & 3);
  __syncthreads();
  float* out = theta + row0 * K;
  for (int e = tid; e < rows * K; e += kThreads) {
    const int r = e / K;
    out[e] = logits[r * ldl + e - r * K];
  }
}

// Features of the tile's 16 documents, transposed to [feature][ld] at column
// col0: two 16-byte stores per feature.
__device__ inline void store_transposed(const uint16_t* act, int lda, int width,
                                        uint16_t* __restrict__ out, size_t ld, size_t col0) {
  for (int f = threadIdx.x; f < width; f += kThreads) {
    u32x4 v[2];
#pragma unroll
    for (int i = 0; i < 8; ++i)
      v[i >> 2][i & 3] = (uint32_t)act[2 * i * lda + f] | ((uint32_t)act[(2 * i + 1) * lda + f] << 16);
    u32x4* p = reinterpret_cast<u32x4*>(out + (size_t)f * ld + col0);
    p[0] = v[0];
    p[1] = v[1];
  }
}

// What the weight gradients read, transposed: [feature][ld], the rows of
// gradient chunk z at columns z chunk_pad .. (zeros behind its rows).
struct TrainTiles {
  uint16_t *x, *h1, *h2, *d1, *d2, *d3;
  size_t ld;
  int chunk, chunk_pad;
};

// Forward and backward of 16 documents of one gradient chunk: block (x, z)
// takes rows 16 x .. of chunk z.  The wave that computes a hidden unit's
// pre-activation also computes its dZ, in the same lane, so gelu' waits in
// registers (PP: blocks of 32 hidden units per wave).
// LDS: three activation buffers of 16 x lda halves (X, then dZ2; H1; H2, then
// dZ1), dZ3 (16 x ldk) and the logits.
template <int PP>
__global__ void __launch_bounds__(kThreads) k_train(const float* __restrict__ X,
                                                    const float* __restrict__ T, int n, int D,
                                                    int H, int K, int lda, Frags f, TrainTiles o,
                                                    float inv_b, float* __restrict__ row_loss) {
  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
  const int Dp = pad32(D), Hp = pad32(H), Kp = pad32(K);
  const int ldk = Kp + 8, ldl = Kp + 4;
  uint16_t* bx = lds;
  uint16_t* b1 = bx + 16 * lda;
  uint16_t* b2 = b1 + 16 * lda;
  uint16_t* b3 = b2 + 16 * lda;
  float* logits = reinterpret_cast<float*>(b3 + 16 * ldk);
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int in_chunk = 16 * blockIdx.x;
  const int row0 = blockIdx.y * o.chunk + in_chunk;
  const int rows = max(0, min(min(16, o.chunk - in_chunk), n - row0));
  const size_t col0 = (size_t)blockIdx.y * o.chunk_pad + in_chunk;
  float g1[PP][8], g2[PP][8];

  load_rows(X + (size_t)row0 * D, rows, 16, D, Dp, bx, lda);
  __syncthreads();
  auto hidden = [&](const uint16_t* w, const float* bias, int ks, const uint16_t* in, uint16_t* out,
                    float (&g)[PP][8]) {
#pragma unroll
    for (int pp = 0; pp < PP; ++pp) {
      const int tp = wave + pp * kWaves;
      if (tp >= Hp / 32) break;
      floatx4 acc[2][1];
      layer<1>(w, tp, ks, in, lda, lane, acc);
      const float* bp = bias + tp * 32 + 8 * q;
      float h[8];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float z = acc[t][0][r] + bp[4 * t + r];
          const float c2 = phi_cdf2(z);
          h[4 * t + r] = 0.5f * z * c2;
          g[pp][4 * t + r] = 0.5f * c2 + z * expf(-0.5f * z * z) * 0.39894228040143268f;
        }
      store_act(out, lda, tp, l16, q, h);
    }
  };
  hidden(f.w1, f.b1, Dp / 32, bx, b1, g1);
  store_transposed(bx, lda, D, o.x, o.ld, col0);
  __syncthreads();
  hidden(f.w2, f.b2, Hp / 32, b1, b2, g2);
  store_transposed(b1, lda, H, o.h1, o.ld, col0);
  __syncthreads();
  for (int tp = wave; tp < Kp / 32; tp += kWaves) {
    floatx4 acc[2][1];
    layer<1>(f.w3, tp, Hp / 32, b2, lda, lane, acc);
    const float* bp = f.b3 + tp * 32 + 8 * q;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        logits[l16 * ldl + tp * 32 + 8 * q + 4 * t + r] = acc[t][0][r] + bp[4 * t + r];
  }
  store_transposed(b2, lda, H, o.h2, o.ld, col0);
  __syncthreads();
  if (tid < 64) {   // four lanes a document: P, dZ3 = (P - T) / B and the cross-entropy
    const int doc = tid >> 2, j = tid & 3;
    const bool in = doc < rows;
    float* z = logits + doc * ldl;
    const float* t = T + (size_t)(row0 + doc) * K;
    float ce[16];   // sum t (lse - z) = sum t lse - t z, added as the softmax sum is
    float zk[16];
#pragma unroll
    for (int m = 0; m < 16; ++m) zk[m] = j + 4 * m < K ? z[j + 4 * m] : 0.f;
    float keep[3][16];
    if (K > 64) {
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int m = 0; m < 16; ++m) {
          const int i = j + 4 * m + 64 * (c + 1);
          keep[c][m] = i < K ? z[i] : 0.f;
        }
    }
    const float lse = softmax_row(z, K, j);
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      ce[m] = 0.f;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int i = j + 4 * m + 64 * c;
        if (i >= K) break;
        const float ti = in ? t[i] : 0.f;
        ce[m] += ti * (lse - (c == 0 ? zk[m] : keep[c > 0 ? c - 1 : 0][m]));
        b3[doc * ldk + i] = in ? to_bf16((z[i] - ti) * inv_b) : (uint16_t)0;
      }
    }
    for (int i = K + j; i < Kp; i += 4) b3[doc * ldk + i] = 0;
#pragma unroll
    for (int d = 8; d > 0; d >>= 1)
#pragma unroll
      for (int m = 0; m < d; ++m) ce[m] += ce[m + d];
    float s = ce[0];
    s += __shfl_xor(s, 2, 64);
    s += __shfl_xor(s, 1, 64);
    if (in && j == 0) row_loss[row0 + doc] = s;
  }
  __syncthreads();
  auto back = [&](const uint16_t* w, int ks, const uint16_t* in, int ld_in, uint16_t* out,
                  const float (&g)[PP][8]) {
#pragma unroll
    for (int pp = 0; pp < PP; ++pp) {
      const int tp = wave + pp * kWaves;
      if (tp >= Hp / 32) break;
      floatx4 acc[2][1];
      layer<1>(w, tp, ks, in, ld_in, lane, acc);
      float d[8];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) d[4 * t + r] = acc[t][0][r] * g[pp][4 * t + r];
      store_act(out, lda, tp, l16, q, d);
    }
  };
  back(f.t3, Kp / 32, b3, ldk, bx, g2);
  store_transposed(b3, ldk, K, o.d3, o.ld, col0);
  __syncthreads();
  back(f.t2, Hp / 32, bx, lda, b2, g1);
  store_transposed(bx, lda, H, o.d2, o.ld, col0);
  __syncthreads();
  store_transposed(b2, lda, H, o.d1, o.ld, col0);
}

// Gradient partials.  The first blocks take one 64 x 64 tile of dW1, dW2 or
// dW3 over one chunk of rows (a wave 32 x 32 of it; both operands are 16-byte
// pieces of the transposed tiles, straight from the caches); the others take
// 256 bias entries over 64 rows, four interleaved row sums combined at the
// end.  ws_w: [chunk][weights in parameter order without the biases], ws_b:
// [64-row chunk][b1, b2, b3].
struct GradPlan {
  int t1, t2, t3;        // 64 x 64 tiles of each weight matrix
  int splits;            // row chunks
  int bias_blocks;       // column blocks of the bias entries
  int bias_chunks;
};

__global__ void __launch_bounds__(256) k_grads(int n, int D, int H, int K, TrainTiles o, GradPlan g,
                                               float* __restrict__ ws_w, float* __restrict__ ws_b) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, q = lane >> 4;
  const int tiles = g.t1 + g.t2 + g.t3;
  int b = blockIdx.x;
  if (b >= tiles * g.splits) {
    b -= tiles * g.splits;
    const int chunk = b / g.bias_blocks, e = b % g.bias_blocks * 256 + tid;
    if (e >= 2 * H + K) return;
    const uint16_t* m = e < H ? o.d1 + (size_t)e * o.ld
                              : e < 2 * H ? o.d2 + (size_t)(e - H) * o.ld
                                          : o.d3 + (size_t)(e - 2 * H) * o.ld;
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    const int r0 = chunk * 64, r1 = min(n, r0 + 64);
    int z = r0 / o.chunk, c = r0 - z * o.chunk;
    if (c + 64 <= o.chunk && r1 - r0 == 64 && c % 8 == 0) {
      // 64 rows in a piece (16-byte aligned: chunks are padded to 32)
      const u32x4* p = reinterpret_cast<const u32x4*>(m + (size_t)z * o.chunk_pad + c);
      u32x4 v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = p[i];
#pragma unroll
      for (int i = 0; i < 32; ++i) {
        const uint32_t w = v[i >> 2][i & 3];
        s[2 * (i & 1)] += __uint_as_float(w << 16);
        s[2 * (i & 1) + 1] += __uint_as_float(w & 0xffff0000u);
      }
    } else {
      for (int r = r0; r < r1; r += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (r + u < r1) {
            s[u] += from_bf16(m[(size_t)z * o.chunk_pad + c]);
            if (++c == o.chunk) {
              c = 0;
              ++z;
            }
          }
      }
    }
    ws_b[(size_t)chunk * (2 * H + K) + e] = (s[0] + s[1]) + (s[2] + s[3]);
    return;
  }
  const int z = b / tiles;
  int t = b % tiles;
  const uint16_t *A, *B;
  int M, N;
  size_t off = (size_t)z * ((size_t)D * H + (size_t)H * H + (size_t)H * K);
  if (t < g.t1) {
    A = o.x, B = o.d1, M = D, N = H;
  } else if (t < g.t1 + g.t2) {
    t -= g.t1;
    A = o.h1, B = o.d2, M = H, N = H;
    off += (size_t)D * H;
  } else {
    t -= g.t1 + g.t2;
    A = o.h2, B = o.d3, M = H, N = K;
    off += (size_t)D * H + (size_t)H * H;
  }
  const int nt = (N + 63) / 64;
  const int m0 = t / nt * 64 + (wave >> 1) * 32, n0 = t % nt * 64 + (wave & 1) * 32;
  const size_t col = (size_t)z * o.chunk_pad + 8 * q;
  const uint16_t* ap = A + (size_t)(m0 + l16) * o.ld + col;
  const uint16_t* bp = B + (size_t)(n0 + l16) * o.ld + col;
  floatx4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto products = [&](const u32x4 (&a)[2], const u32x4 (&bb)[2]) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[i]),
                                                            __builtin_bit_cast(bf16x8, bb[j]),
                                                            acc[i][j], 0, 0, 0);
  };
  // 128 rows (the usual chunk) at a time, every operand loaded before the
  // first product: one round trip to the caches
  int k0 = 0;
  for (; k0 + 128 <= o.chunk_pad; k0 += 128) {
    u32x4 a[4][2], bb[4][2];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[u][i] = *reinterpret_cast<const u32x4*>(ap + i * 16 * o.ld + k0 + 32 * u);
        bb[u][i] = *reinterpret_cast<const u32x4*>(bp + i * 16 * o.ld + k0 + 32 * u);
      }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < 4; ++u) products(a[u], bb[u]);
  }
  for (; k0 < o.chunk_pad; k0 += 32) {
    u32x4 a[2], bb[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      a[i] = *reinterpret_cast<const u32x4*>(ap + i * 16 * o.ld + k0);
      bb[i] = *reinterpret_cast<const u32x4*>(bp + i * 16 * o.ld + k0);
    }
    products(a, bb);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int gm = m0 + i * 16 + 4 * q + r, gn = n0 + j * 16 + l16;
        if (gm < M && gn < N) ws_w[off + (size_t)gm * N + gn] = acc[i][j][r];
      }
}

// Gradient of parameter e from its partials, added in chunk order.
__device__ inline float sum_partials(const float* __restrict__ ws, int n, size_t stride) {
  constexpr int kU = 8;
  float s = 0.f;
  for (int z = 0; z < n; z += kU) {
    float v[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) v[u] = ws[(size_t)min(z + u, n - 1) * stride];
#pragma unroll
    for (int u = 0; u < kU; ++u)
      if (z + u < n) s += v[u];
  }
  return s;
}

// loss = sum of the row losses / n (fixed order, one block of 256)
__device__ inline void mean_loss(const float* __restrict__ row_loss, int n, float* out) {
  __shared__ float red[256];
  float s = 0.f;
  for (int i = threadIdx.x; i < n; i += 256) s += row_loss[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = red[0] / (float)n;
}

struct AdamArgs {
  float *p, *m, *v;
  float lr, beta1, beta2, eps, c1, c2;   // c1 = 1 - beta1^t, c2 = 1 - beta2^t
};

// Every parameter's gradient from the partials; then either the gradient
// itself (ADAM false, grads may be NULL) or one Adam step (Kingma & Ba,
// Algorithm 1), with the BF16 and padded copies following.  The last block
// takes the loss.
template <bool ADAM>
__global__ void __launch_bounds__(256) k_update(int n, int D, int H, int K, GradPlan g,
                                                const float* __restrict__ ws_w,
                                                const float* __restrict__ ws_b,
                                                const float* __restrict__ row_loss,
                                                float* __restrict__ loss, float* __restrict__ grads,
                                                AdamArgs a, Frags f) {
  if (blockIdx.x == gridDim.x - 1) {
    if (loss != nullptr) mean_loss(row_loss, n, loss);
    return;
  }
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t n1 = (size_t)D * H, n2 = n1 + H, n3 = n2 + (size_t)H * H, n4 = n3 + H,
               n5 = n4 + (size_t)H * K, n6 = n5 + K;
  if (e >= n6) return;
  // a weight's place among the weights, a bias's among the biases
  size_t w = e, bias = 0;
  bool is_bias = false;
  if (e >= n5) is_bias = true, bias = 2 * (size_t)H + (e - n5);
  else if (e >= n4) w = e - 2 * (size_t)H;
  else if (e >= n3) is_bias = true, bias = H + (e - n3);
  else if (e >= n2) w = e - H;
  else if (e >= n1) is_bias = true, bias = e - n1;
  const float gi = is_bias ? sum_partials(ws_b + bias, g.bias_chunks, 2 * (size_t)H + K)
                           : sum_partials(ws_w + w, g.splits, n6 - 2 * (size_t)H - K);
  if (!ADAM) {
    grads[e] = gi;
    return;
  }
  const float mi = a.beta1 * a.m[e] + (1.0f - a.beta1) * gi;
  const float vi = a.beta2 * a.v[e] + (1.0f - a.beta2) * gi * gi;
  a.m[e] = mi;
  a.v[e] = vi;
  const float pi = a.p[e] - a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
  a.p[e] = pi;
  put_param(f, D, H, K, e, pi);
}

// Rows are split into chunks of at least kGradChunk (at most kGradSplits), each
// with its own partial of every weight gradient.
constexpr int kGradChunk = 128, kGradSplits = 32;
struct Chunks {
  int splits, chunk, chunk_pad;
};
Chunks chunks_of(int n) {
  Chunks c;
  const int s = std::min(kGradSplits, std::max(1, n / kGradChunk));
  c.chunk = (n + s - 1) / s;
  c.splits = (n + c.chunk - 1) / c.chunk;
  c.chunk_pad = pad32(c.chunk);
  return c;
}
// columns of the transposed tiles for up to max_batch rows: a chunk's padding
// adds at most 31
size_t tile_cols(int max_batch) {
  return ((size_t)max_batch + kGradSplits * 32 + 63) / 32 * 32;
}
int pad64(int n) { return (n + 63) / 64 * 64; }

}  // namespace

// LDS of k_forward: halves a document in the two buffers, bytes of a block.
static int forward_lda(int D, int H) { return std::max(pad32(D), pad32(H)) + 8; }
static int forward_ldb(int H, int K) { return std::max(pad32(H), 2 * pad32(K)) + 8; }
static size_t forward_lds(int D, int H, int K, int docs) {
  return (size_t)docs * (forward_lda(D, H) + forward_ldb(H, K)) * sizeof(uint16_t);
}
// and of k_train
static int train_lda(int D, int H) { return std::max(pad32(D), pad32(H)) + 8; }
static size_t train_lds(int D, int H, int K) {
  return (size_t)16 * (3 * train_lda(D, H) + pad32(K) + 8) * sizeof(uint16_t) +
         16 * (pad32(K) + 4) * sizeof(float);
}
constexpr size_t kForwardLds = 80 * 1024;   // two blocks on a compute unit
static auto forward_kernel(int D, int nt) {
  if (D > kWideInput)
    return nt == 4 ? k_forward<4, true> : nt == 2 ? k_forward<2, true> : k_forward<1, true>;
  return nt == 4 ? k_forward<4, false> : nt == 2 ? k_forward<2, false> : k_forward<1, false>;
}
static auto train_kernel(int H) {
  return H <= 32 * kWaves ? k_train<1> : H <= 64 * kWaves ? k_train<2> : k_train<4>;
}

// Dynamic LDS past the default 64 KB (of the compute unit's 160) has to be
// allowed; once, when an encoder is made, for the kernels that need it (any
// encoder's need, since the permission is the kernel's).
hipError_t mlp_allow_lds(int D, int H, int K) {
  auto allow = [](const void* kernel, size_t bytes) {
    return bytes <= 64 * 1024 ? hipSuccess
                              : hipFuncSetAttribute(
                                    kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  };
  hipError_t e = hipSuccess;
  for (int nt = 1; nt <= 4 && e == hipSuccess; nt *= 2) {
    const size_t bytes = forward_lds(D, H, K, 16 * nt);
    if (nt == 1 || bytes <= kForwardLds)
      e = allow(reinterpret_cast<const void*>(forward_kernel(D, nt)), bytes);
  }
  if (e != hipSuccess) return e;
  return allow(reinterpret_cast<const void*>(train_kernel(H)), train_lds(D, H, K));
}

size_t mlp_param_count(int d_in, int hidden, int k_out) {
  return (size_t)d_in * hidden + hidden + (size_t)hidden * hidden + hidden +
         (size_t)hidden * k_out + k_out;
}

size_t mlp_frag_halves(int d_in, int hidden, int k_out) { return frag_halves(d_in, hidden, k_out); }
size_t mlp_bias_floats(int hidden, int k_out) { return bias_floats(hidden, k_out); }

size_t mlp_workspace_floats(int d_in, int hidden, int k_out, int max_batch) {
  const size_t weights = (size_t)d_in * hidden + (size_t)hidden * hidden + (size_t)hidden * k_out;
  return kGradSplits * weights + ((size_t)max_batch + 63) / 64 * (2 * (size_t)hidden + k_out);
}

size_t mlp_tile_halves(int d_in, int hidden, int k_out, int max_batch) {
  return (pad64(d_in) + 4 * (size_t)pad64(hidden) + pad64(k_out)) * tile_cols(max_batch);
}

hipError_t mlp_forward(tlda_mlp& m, const float* X, int64_t n, float* theta) {
  if (n <= 0) return hipSuccess;
  const int D = m.d_in, H = m.hidden, K = m.k_out;
  const int lda = forward_lda(D, H), ldb = forward_ldb(H, K);
  const Frags f = frags_of(m);
  // 64 documents a block while the grid still fills the 256 compute units
  // twice over and two blocks' LDS fits on one; 32 or 16 below that, or for
  // wide layers
  int nt = 1;
  if (forward_lds(D, H, K, 64) <= kForwardLds && n >= 64 * 512) nt = 4;
  else if (forward_lds(D, H, K, 32) <= kForwardLds && n >= 32 * 512) nt = 2;
  auto kernel = forward_kernel(D, nt);
  const size_t lds = forward_lds(D, H, K, 16 * nt);
  // a launch takes fewer than 2^32 work items
  const int64_t docs = 16 * nt, most = ((int64_t(1) << 32) / kThreads - 1) * docs;
  for (int64_t r = 0; r < n; r += most) {
    const int64_t rows = std::min(most, n - r);
    hipLaunchKernelGGL(kernel, dim3((unsigned)((rows + docs - 1) / docs)), dim3(kThreads), lds,
                       m.stream, X + r * D, rows, D, H, K, lda, ldb, f, theta + r * K);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Forward, backward and the gradient partials of n <= max_batch rows.
static hipError_t train_partials(tlda_mlp& m, const float* X, const float* T, int n, GradPlan& g) {
  const int D = m.d_in, H = m.hidden, K = m.k_out;
  const Chunks c = chunks_of(n);
  TrainTiles o;
  o.ld = tile_cols(m.max_batch);
  o.chunk = c.chunk;
  o.chunk_pad = c.chunk_pad;
  o.x = m.tiles;
  o.h1 = o.x + (size_t)pad64(D) * o.ld;
  o.h2 = o.h1 + (size_t)pad64(H) * o.ld;
  o.d1 = o.h2 + (size_t)pad64(H) * o.ld;
  o.d2 = o.d1 + (size_t)pad64(H) * o.ld;
  o.d3 = o.d2 + (size_t)pad64(H) * o.ld;
  const int lda = train_lda(D, H);
  const size_t lds = train_lds(D, H, K);
  const dim3 grid(c.chunk_pad / 16, c.splits);
  const Frags f = frags_of(m);
  const float inv_b = 1.0f / (float)n;
  auto kernel = train_kernel(H);
  hipLaunchKernelGGL(kernel, grid, dim3(kThreads), lds, m.stream, X, T, n, D, H, K, lda, f, o, inv_b,
                     m.row_loss);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  g.t1 = pad64(D) / 64 * (pad64(H) / 64);
  g.t2 = pad64(H) / 64 * (pad64(H) / 64);
  g.t3 = pad64(H) / 64 * (pad64(K) / 64);
  g.splits = c.splits;
  g.bias_blocks = (2 * H + K + 255) / 256;
  g.bias_chunks = (n + 63) / 64;
  const size_t weights = (size_t)D * H + (size_t)H * H + (size_t)H * K;
  hipLaunchKernelGGL(k_grads, dim3((g.t1 + g.t2 + g.t3) * g.splits + g.bias_blocks * g.bias_chunks),
                     dim3(256), 0, m.stream, n, D, H, K, o, g, m.ws, m.ws + kGradSplits * weights);
  return hipGetLastError();
}

hipError_t mlp_gradients(tlda_mlp& m, const float* X, const float* T, int n, float* grads,
                         float* loss) {
  GradPlan g;
  hipError_t e = train_partials(m, X, T, n, g);
  if (e != hipSuccess || (grads == nullptr && loss == nullptr)) return e;
  const int D = m.d_in, H = m.hidden, K = m.k_out;
  const size_t weights = (size_t)D * H + (size_t)H * H + (size_t)H * K;
  const unsigned blocks = grads != nullptr ? (unsigned)((m.n_params + 255) / 256) : 0u;
  hipLaunchKernelGGL(k_update<false>, dim3(blocks + 1), dim3(256), 0, m.stream, n, D, H, K, g, m.ws,
                     m.ws + kGradSplits * weights, m.row_loss, loss, grads, AdamArgs{}, Frags{});
  return hipGetLastError();
}

hipError_t mlp_train_step(tlda_mlp& m, const float* X, const float* T, int n, float lr, float beta1,
                          float beta2, float eps, float* loss) {
  GradPlan g;
  hipError_t e = train_partials(m, X, T, n, g);
  if (e != hipSuccess) return e;
  m.adam_t += 1;
  AdamArgs a{m.params, m.adam_m, m.adam_v, lr, beta1, beta2, eps, 0.f, 0.f};
  a.c1 = 1.0f - (float)std::pow((double)beta1, (double)m.adam_t);
  a.c2 = 1.0f - (float)std::pow((double)beta2, (double)m.adam_t);
  const int D = m.d_in, H = m.hidden, K = m.k_out;
  const size_t weights = (size_t)D * H + (size_t)H * H + (size_t)H * K;
  hipLaunchKernelGGL(k_update<true>, dim3((unsigned)((m.n_params + 255) / 256) + 1), dim3(256), 0,
                     m.stream, n, D, H, K, g, m.ws, m.ws + kGradSplits * weights, m.row_loss, loss,
                     nullptr, a, frags_of(m));
  return hipGetLastError();
}

hipError_t mlp_refresh(tlda_mlp& m) {
  const size_t n = m.n_params;
  hipLaunchKernelGGL(k_refresh, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, m.stream, m.params,
                     m.d_in, m.hidden, m.k_out, n, frags_of(m));
  return hipGetLastError();
}

}  // namespace tlda
