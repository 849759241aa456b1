// Post-processing and document-topic inference (FP64 unless noted).
//
// Unwhitening (section "Recovering the Topic Model Parameters" and Theorem 1)
// in the tight-frame reading for centred moments: with
// w_k = (1+theta)^(1/3) phi_k, the topic weight a_k is the root in (0, 1] of
// a^(1/3) |w_k|^2 + a = 1, the centred topic is nu_k = (W^T)^+ a_k^(-1/3) w_k
// with (W^T)^+ = U diag(lambda)^(1/2), and mu_k = nu_k + M1.
//
// Inference: theta_d = argmin over the simplex of |x_d - A theta|^2 with
// A = W^T (mu - M1 1^T), by projected gradient with step 1 / lambda_max(A^T A).
#include "tlda_internal.h"

namespace tlda {
namespace {

// Per topic: scale[k] = (1+theta)^(1/3) a_k^(-1/3), alpha[k] = a_k / sum a,
// lambda[k] = (1+theta) |phi_k|^3.  One block; K <= 256.  With u = a^(1/3) the
// weight's equation is f(u) = u^3 + r u - 1 = 0, f convex and increasing, so
// Newton's method comes down to the root from any start above it (min(1, 1 /
// r) is) and squares its error: 200 bisections with a cube root each took 25 us.
__global__ void __launch_bounds__(256) k_frame_weights(const float* __restrict__ Phi, int D, int K,
                                                       double theta, double* __restrict__ scale,
                                                       double* __restrict__ alpha,
                                                       double* __restrict__ lambda) {
  __shared__ double a_sh[256];
  const int k = threadIdx.x;
  double a = 0.0;
  if (k < K) {
    double n2 = 0.0;
    for (int d = 0; d < D; ++d) {
      const double v = (double)Phi[d * K + k];
      n2 += v * v;
    }
    const double c = cbrt(1.0 + theta);
    const double r = c * c * n2;   // |w_k|^2
    // (a norm past the range, or NaN, is an infinite one: the weight vanishes)
    double u = !(r < INFINITY) ? 0x1p-67 : r > 1.0 ? 1.0 / r : 1.0;
    for (int it = 0; it < 60 && r < INFINITY; ++it) {
      const double d = (u * (u * u + r) - 1.0) / (3.0 * u * u + r);
      u -= d;
      if (!(fabs(d) > 1e-16 * u)) break;
    }
    a = u * u * u;
    scale[k] = c / u;
    if (lambda != nullptr) lambda[k] = (1.0 + theta) * n2 * sqrt(n2);
  }
  a_sh[k] = a;
  __syncthreads();
  if (k < K) {
    double s = 0.0;
    for (int j = 0; j < K; ++j) s += a_sh[j];
    alpha[k] = a / s;
  }
}

// Classic recovery: lambda_k = (1+theta)|phi_k|^3, scale[k] = lambda_k / |phi_k|
// (so that mu_k = lambda_k (W^T)^+ phi_k / |phi_k|), alpha_k proportional to
// lambda_k^-2; a zero column gets scale 0 and weight 0.  One block; K <= 256.
__global__ void __launch_bounds__(256) k_classic_weights(const float* __restrict__ Phi, int D,
                                                         int K, double theta,
                                                         double* __restrict__ scale,
                                                         double* __restrict__ alpha,
                                                         double* __restrict__ lambda) {
  __shared__ double w_sh[256];
  const int k = threadIdx.x;
  double w = 0.0;
  if (k < K) {
    double n2 = 0.0;
    for (int d = 0; d < D; ++d) {
      const double v = (double)Phi[d * K + k];
      n2 += v * v;
    }
    const double lam = (1.0 + theta) * n2 * sqrt(n2);
    scale[k] = (1.0 + theta) * n2;
    w = lam > 0.0 ? 1.0 / (lam * lam) : 0.0;
    if (lambda != nullptr) lambda[k] = lam;
  }
  w_sh[k] = w;
  __syncthreads();
  if (k < K) {
    double s = 0.0;
    for (int j = 0; j < K; ++j) s += w_sh[j];
    alpha[k] = s > 0.0 ? w / s : 0.0;
  }
}

// One block per column k of Phi (D <= 256): the column is read into LDS,
// then Phi[d][k] = eig[d]^(-1/2) sum_e C[d][e] eig_prev[e]^(1/2) phi[e].
__global__ void __launch_bounds__(256) k_rebase(const double* __restrict__ C,
                                                const double* __restrict__ eig,
                                                const double* __restrict__ eig_prev, int D, int K,
                                                float* __restrict__ Phi) {
  __shared__ double col[256];
  const int k = blockIdx.x, d = threadIdx.x;
  if (d < D) col[d] = (double)Phi[d * K + k] * sqrt(eig_prev[d]);
  __syncthreads();
  if (d < D) {
    double s = 0.0;
    for (int e = 0; e < D; ++e) s += C[d * D + e] * col[e];
    Phi[d * K + k] = (float)(s / sqrt(eig[d]));
  }
}

// mu[i][k] = sum_d U[i][d] sqrt(eig[d]) phi[d][k] scale[k] + m[i] (m may be
// NULL).  A block takes a run of rows and 64 columns, one lane per column:
// sqrt(eig) phi scale is formed once per block in LDS, a row of U is read by
// all lanes at once, and the row of mu is one 512-byte write.  sums (or NULL):
// [block row][K] sums of the clipped entries, added in row order by
// k_simplex_scale.  Bound: 2 V D K flops and the writes of mu.
constexpr int kMuRows = 64;   // rows per block, 16 per wave
__global__ void __launch_bounds__(256) k_mu(const float* __restrict__ Phi,
                                            const double* __restrict__ U,
                                            const double* __restrict__ eig,
                                            const double* __restrict__ m,
                                            const double* __restrict__ scale, int V, int D, int K,
                                            double* __restrict__ mu, double* __restrict__ sums) {
  constexpr int kD = 64;   // rows of Phi at a time
  __shared__ double P[kD * 64];
  __shared__ double red[4][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int k = blockIdx.y * 64 + lane;
  const int r0 = blockIdx.x * kMuRows + wave * 16;
  const double sk = k < K ? scale[k] : 0.0;
  double s[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) s[i] = 0.0;
  for (int d0 = 0; d0 < D; d0 += kD) {
    const int nd = min(kD, D - d0);
    __syncthreads();
    for (int d = wave; d < nd; d += 4)
      P[d * 64 + lane] = k < K ? sqrt(eig[d0 + d]) * (double)Phi[(d0 + d) * K + k] : 0.0;
    __syncthreads();
    for (int d = 0; d < nd; ++d) {
      const double p = P[d * 64 + lane];
#pragma unroll
      for (int i = 0; i < 16; ++i)
        s[i] = fma(U[(size_t)min(r0 + i, V - 1) * D + d0 + d], p, s[i]);
    }
  }
  double pos = 0.0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int r = r0 + i;
    if (r < V && k < K) {
      const double v = s[i] * sk + (m != nullptr ? m[r] : 0.0);
      mu[(size_t)r * K + k] = v;
      pos += fmax(v, 0.0);
    }
  }
  if (sums == nullptr) return;
  red[wave][lane] = pos;
  __syncthreads();
  if (wave == 0 && k < K)
    sums[(size_t)blockIdx.x * K + k] =
        (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

// tot[k] = sum over the nb blocks' column sums, in a fixed order (16 phases
// combined in LDS); a column with no positive entry gets 1.
__global__ void __launch_bounds__(1024) k_simplex_total(const double* __restrict__ sums, int nb,
                                                        int K, double* __restrict__ tot) {
  __shared__ double red[16][64];
  const int lane = threadIdx.x & 63, ph = threadIdx.x >> 6;
  const int k = blockIdx.x * 64 + lane;
  double s = 0.0;
  if (k < K)
    for (int b = ph; b < nb; b += 16) s += sums[(size_t)b * K + k];
  red[ph][lane] = s;
  __syncthreads();
  if (ph == 0 && k < K) {
    for (int i = 1; i < 16; ++i) s += red[i][lane];
    tot[k] = s > 0.0 ? s : 1.0;
  }
}

// Clips negative entries and divides every column by its total.
__global__ void __launch_bounds__(256) k_simplex_scale(double* __restrict__ mu, size_t n, int K,
                                                       const double* __restrict__ tot) {
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (e < n) mu[e] = fmax(mu[e], 0.0) / tot[e % K];
}

// G32 = A^T A (K x K, FP64 sums rounded to FP32), and into Gw the smaller of
// A^T A and A A^T, whose largest eigenvalue is the same.  One thread per entry.
__global__ void __launch_bounds__(256) k_infer_G(const double* __restrict__ A, int D, int K,
                                                 double* __restrict__ Gw,
                                                 float* __restrict__ G32) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e < K * K) {
    const int j = e / K, k = e % K;
    double s = 0.0;
    for (int d = 0; d < D; ++d) s += A[d * K + j] * A[d * K + k];
    if (K <= D) Gw[e] = s;
    G32[e] = (float)s;
  }
  if (D < K && e < D * D) {
    const int i = e / D, j = e % D;
    double s = 0.0;
    for (int k = 0; k < K; ++k) s += A[i * K + k] * A[j * K + k];
    Gw[e] = s;
  }
}

// Orders this wave's LDS stores before its later LDS loads by other lanes.
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// One wave per document; lane l owns topics l, l + 64, ... (TPL per lane).
// The simplex projection finds, for each topic, its rank in decreasing order
// (ties by index) and the sum of all values ranked at or above it; the
// largest rank r whose value exceeds (prefix_r - 1) / r sets the threshold.
//
// GIVEN: the start point is read from `out` (e.g. an encoder's output on the
// simplex) instead of the uniform 1/K.
// GAP_RULE: instead of stopping when the L1 change of an iterate falls below
// tol, stop at the first iterate after min_steps steps whose duality gap for
// h(t) = |x - A t|^2 / 2, g.t - min_k g_k with g = A^T (A t - x) = G t - b, is
// at most gap_tol (it bounds h(t) - min h); rows that need more than
// min_steps steps are counted in *n_stepped.
template <int TPL, bool GIVEN, bool GAP_RULE>
__global__ void __launch_bounds__(256) k_infer(const float* __restrict__ X, int n_rows,
                                               const float* __restrict__ A32,
                                               const float* __restrict__ G32,
                                               const float* __restrict__ step32, int D, int K,
                                               int max_iter, float tol, float* __restrict__ out,
                                               float gap_tol, int min_steps,
                                               int* __restrict__ n_stepped) {
  __shared__ float xs[4][TLDA_MAX_D];
  __shared__ float ys[4][64 * TPL];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = blockIdx.x * 4 + wave;
  if (row >= n_rows) return;
  const float step = step32[0];
  for (int d = lane; d < D; d += 64) xs[wave][d] = X[(size_t)row * D + d];
  wave_sync();
  float b[TPL], t[TPL];
#pragma unroll
  for (int q = 0; q < TPL; ++q) {
    const int k = lane + 64 * q;
    float s = 0.f;
    if (k < K)
      for (int d = 0; d < D; ++d) s = fmaf(A32[d * K + k], xs[wave][d], s);
    b[q] = s;
    if (GIVEN)
      t[q] = k < K ? out[(size_t)row * K + k] : 0.f;
    else
      t[q] = k < K ? 1.0f / (float)K : 0.f;
  }
  for (int it = 0; it < max_iter; ++it) {
#pragma unroll
    for (int q = 0; q < TPL; ++q) ys[wave][lane + 64 * q] = t[q];
    wave_sync();
    float y[TPL];
    float gt = 0.f, gmin = INFINITY;
#pragma unroll
    for (int q = 0; q < TPL; ++q) {
      const int k = lane + 64 * q;
      float g = 0.f;
      if (k < K) {
        for (int j = 0; j < K; ++j) g = fmaf(G32[k * K + j], ys[wave][j], g);
        g -= b[q];
        gt = fmaf(g, t[q], gt);
        gmin = fminf(gmin, g);
      }
      y[q] = t[q] - step * g;
    }
    if (GAP_RULE) {
      for (int off = 32; off > 0; off >>= 1) {
        gt += __shfl_xor(gt, off, 64);
        gmin = fminf(gmin, __shfl_xor(gmin, off, 64));
      }
      if (it >= min_steps && gt - gmin <= gap_tol) break;   // within gap_tol of the minimum
      if (it == min_steps && lane == 0) atomicAdd(n_stepped, 1);
    }
    wave_sync();
#pragma unroll
    for (int q = 0; q < TPL; ++q) ys[wave][lane + 64 * q] = y[q];
    wave_sync();
    int best_rank = 0;
    float best_tau = 0.f;
#pragma unroll
    for (int q = 0; q < TPL; ++q) {
      const int k = lane + 64 * q;
      if (k >= K) continue;
      int rank = 0;
      float pref = 0.f;
      for (int j = 0; j < K; ++j) {
        const float v = ys[wave][j];
        if (v > y[q] || (v == y[q] && j <= k)) {
          ++rank;
          pref += v;
        }
      }
      const float tau = (pref - 1.0f) / (float)rank;
      if (y[q] - tau > 0.f && rank > best_rank) {
        best_rank = rank;
        best_tau = tau;
      }
    }
    for (int off = 32; off > 0; off >>= 1) {
      const int orank = __shfl_xor(best_rank, off, 64);
      const float otau = __shfl_xor(best_tau, off, 64);
      if (orank > best_rank) {
        best_rank = orank;
        best_tau = otau;
      }
    }
    float change = 0.f;
#pragma unroll
    for (int q = 0; q < TPL; ++q) {
      const int k = lane + 64 * q;
      const float tn = k < K ? fmaxf(y[q] - best_tau, 0.f) : 0.f;
      change += fabsf(tn - t[q]);
      t[q] = tn;
    }
    for (int off = 32; off > 0; off >>= 1) change += __shfl_xor(change, off, 64);
    wave_sync();
    if (!GAP_RULE && change < tol) break;
  }
#pragma unroll
  for (int q = 0; q < TPL; ++q) {
    const int k = lane + 64 * q;
    if (k < K) out[(size_t)row * K + k] = t[q];
  }
}

}  // namespace

size_t unwhiten_scratch_doubles(int V, int K) {
  return (size_t)((V + kMuRows - 1) / kMuRows + 2) * K;   // column sums, totals, scales
}

// mu from the scales in scratch[0 .. K), clipped and renormalised when asked.
static hipError_t launch_mu(const float* Phi, const double* U, const double* eig, const double* m,
                            int V, int D, int K, uint32_t flags, double* mu, double* scratch,
                            hipStream_t s) {
  const bool simplex = (flags & TLDA_PROJECT_SIMPLEX) != 0;
  const int nb = (V + kMuRows - 1) / kMuRows, kb = (K + 63) / 64;
  double *tot = scratch + K, *sums = tot + K;
  hipLaunchKernelGGL(k_mu, dim3(nb, kb), dim3(256), 0, s, Phi, U, eig, m, scratch, V, D, K, mu,
                     simplex ? sums : nullptr);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !simplex) return e;
  hipLaunchKernelGGL(k_simplex_total, dim3(kb), dim3(1024), 0, s, sums, nb, K, tot);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const size_t n = (size_t)V * K;
  hipLaunchKernelGGL(k_simplex_scale, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, mu, n, K,
                     tot);
  return hipGetLastError();
}

hipError_t launch_unwhiten(const float* Phi, const double* U, const double* eig, const double* m,
                           int V, int D, int K, double theta, uint32_t flags, double* mu,
                           double* alpha, double* lambda, double* scratch, hipStream_t s) {
  hipLaunchKernelGGL(k_frame_weights, dim3(1), dim3(256), 0, s, Phi, D, K, theta, scratch, alpha,
                     lambda);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_mu(Phi, U, eig, m, V, D, K, flags, mu, scratch, s);
}

hipError_t launch_rebase(const double* C, const double* eig, const double* eig_prev, int D, int K,
                         float* Phi, hipStream_t s) {
  hipLaunchKernelGGL(k_rebase, dim3(K), dim3(256), 0, s, C, eig, eig_prev, D, K, Phi);
  return hipGetLastError();
}

hipError_t launch_unwhiten_classic(const float* Phi, const double* U, const double* eig, int V,
                                   int D, int K, double theta, uint32_t flags, double* mu,
                                   double* alpha, double* lambda, double* scratch, hipStream_t s) {
  hipLaunchKernelGGL(k_classic_weights, dim3(1), dim3(256), 0, s, Phi, D, K, theta, scratch,
                     alpha, lambda);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_mu(Phi, U, eig, nullptr, V, D, K, flags, mu, scratch, s);
}

hipError_t launch_inference_setup(const double* W, const double* m, const double* mu, int V,
                                  int D, int K, double* part, double* A, double* G, float* A32,
                                  float* G32, float* step32, hipStream_t s) {
  hipError_t e = launch_project(W, m, mu, V, D, K, part, A, A32, s);
  if (e != hipSuccess) return e;
  const int n = K > D ? K : D;
  hipLaunchKernelGGL(k_infer_G, dim3((n * n + 255) / 256), dim3(256), 0, s, A, D, K, G, G32);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return launch_top_eig(G, K < D ? K : D, step32, s);
}

template <bool GIVEN, bool GAP_RULE>
hipError_t launch_infer_t(const float* X, int n_rows, const float* A32, const float* G32,
                          const float* step32, int D, int K, int max_iter, float tol, float* theta,
                          float gap_tol, int min_steps, int* n_stepped, hipStream_t s) {
  if (n_rows == 0) return hipSuccess;
  const dim3 grid((n_rows + 3) / 4);
  if (K <= 64)
    hipLaunchKernelGGL((k_infer<1, GIVEN, GAP_RULE>), grid, dim3(256), 0, s, X, n_rows, A32, G32,
                       step32, D, K, max_iter, tol, theta, gap_tol, min_steps,
                       n_stepped);
  else if (K <= 128)
    hipLaunchKernelGGL((k_infer<2, GIVEN, GAP_RULE>), grid, dim3(256), 0, s, X, n_rows, A32, G32,
                       step32, D, K, max_iter, tol, theta, gap_tol, min_steps,
                       n_stepped);
  else
    hipLaunchKernelGGL((k_infer<4, GIVEN, GAP_RULE>), grid, dim3(256), 0, s, X, n_rows, A32, G32,
                       step32, D, K, max_iter, tol, theta, gap_tol, min_steps,
                       n_stepped);
  return hipGetLastError();
}

hipError_t launch_infer(const float* X, int n_rows, const float* A32, const float* G32,
                        const float* step32, int D, int K, int max_iter, float tol,
                        float* theta, hipStream_t s) {
  return launch_infer_t<false, false>(X, n_rows, A32, G32, step32, D, K, max_iter, tol, theta,
                                      0.f, 0, nullptr, s);
}

hipError_t launch_infer_gap(const float* X, int n_rows, const float* A32, const float* G32,
                            const float* step32, int D, int K, bool given_start, float gap_tol,
                            int min_steps, int max_iter, float* theta, int* n_stepped,
                            hipStream_t s) {
  return given_start
             ? launch_infer_t<true, true>(X, n_rows, A32, G32, step32, D, K, max_iter, 0.f, theta,
                                          gap_tol, min_steps, n_stepped, s)
             : launch_infer_t<false, true>(X, n_rows, A32, G32, step32, D, K, max_iter, 0.f,
                                           theta, gap_tol, min_steps, n_stepped, s);
}

}  // namespace tlda
