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
// k_simplex_scale.  Bound: 2 V D K flops on the FP64 vector ALUs and the writes
// of mu: 46 us at V = 20000, D = K = 50, where the sums of the clipped entries
// cost 12 us in two small kernels after it (82 in a pass over mu by columns).
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

// G = A^T A (FP64 sums rounded to FP32) in the fragment order of k_infer, and
// into Gw the smaller of A^T A and A A^T, whose largest eigenvalue is the same.
// One thread per entry; entries of topics past K are zeros.
__global__ void __launch_bounds__(256) k_infer_G(const double* __restrict__ A, int D, int K,
                                                 double* __restrict__ Gw,
                                                 float* __restrict__ Gf) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  const int Kp = (K + 15) / 16 * 16;
  if (e < Kp * Kp) {
    const int j = e / Kp, k = e % Kp;
    double s = 0.0;
    if (j < K && k < K) {
      for (int d = 0; d < D; ++d) s += A[d * K + j] * A[d * K + k];
      if (K <= D) Gw[j * K + k] = s;
    }
    // row j = 16 mo + m of the product, column k = 16 mt + 4 q + r of its step (mt, r)
    const int lane = (k >> 2 & 3) * 16 + (j & 15);
    Gf[((j >> 4) * (Kp / 4) + (k >> 4) * 4 + (k & 3)) * 64 + lane] = (float)s;
  }
  if (D < K && e < D * D) {
    const int i = e / D, j = e % D;
    double s = 0.0;
    for (int k = 0; k < K; ++k) s += A[i * K + k] * A[j * K + k];
    Gw[e] = s;
  }
}

// The projected-gradient solve: 16 documents per wave, one per column of the
// FP32 matrix core's tiles (v_mfma_f32_16x16x4_f32).  Lane (l16, q) holds, for
// document l16, topics 16 mt + 4 q + r (mt < TM, r < 4) of every vector: what
// a product leaves in its accumulators, and what step (mt, r) of the next
// product takes as its B operand, if G's columns are taken in that order.  So
// t, b and the iterate never leave their registers; sums over a document's
// topics are 4 TM values in the lane and two exchanges between lane groups.
//
// The simplex projection max(y - tau, 0) solves sum max(y - tau, 0) = 1 by
// Newton's method on that convex, decreasing, piecewise linear function of
// tau: tau <- (sum of the entries above tau - 1) / (their number), started from
// the previous iterate's tau (whose support is mostly the same: two or three
// passes), until the number above stays.  From any start the sets are nested
// from then on, so an unchanged number is an unchanged set, and the last tau is
// the exact threshold of it.
//
// Documents finish at different iterations: a wave takes new ones from its
// queue when kRefill columns are free (the b = A^T x of new documents costs
// about an iteration for the whole wave).  There are kInferQueues queues, each
// with every kInferQueues-th 16 rows and every kInferQueues-th wave: one address
// takes an atomic every 14 ns, which held 300000 rows at 262 us where they had
// few iterations to do (2 topics, no iteration: 266 us with one queue, 39 with
// 16, 80 with a wave per document; 5 topics, 20 iterations: 282, 156, 1490).
//
// Bound: the vector ALUs (the projection) and the FP32 matrix cores (4 TM
// steps of TM tiles an iteration) about alike; two waves or more per SIMD
// overlap them (up to 64 topics, where G's fragments stay in registers).  65536
// documents of 50 topics, up to 200 iterations: 1.16 ms (6.5 with a lane per
// topic and the products as sums over lanes).  Past 64 topics a wave has a
// SIMD's registers to itself, does not fit them (up to 128 topics 540 bytes a
// lane in scratch memory, past that 528) and takes G from the caches in every
// iteration.  It is still the faster way: 300000 documents, 60 iterations, 65
// topics 11.1 ms (44 with a wave per document), 100 27 (63), 120 55 (72),
// 128 with D = 30 52 (122); 65536 documents, 200 iterations, 256 topics 220 ms
// (384).
//
// given: the start point is read from `out` (e.g. an encoder's output on the
// simplex) instead of the uniform 1/K.
// gap_rule: instead of stopping when the L1 change of an iterate falls below
// tol, stop at the first iterate after min_steps steps whose duality gap for
// h(t) = |x - A t|^2 / 2, g.t - min_k g_k with g = A^T (A t - x) = G t - b, is
// at most gap_tol (it bounds h(t) - min h); rows that need more than
// min_steps steps are counted in *n_stepped.
typedef float floatx4 __attribute__((ext_vector_type(4)));
constexpr int kRefill = 4;

__device__ __forceinline__ float group_sum(float v) {   // over the document's four lanes
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}
__device__ __forceinline__ int group_sum(int v) {
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}
__device__ __forceinline__ float group_min(float v) {
  v = fminf(v, __shfl_xor(v, 16, 64));
  return fminf(v, __shfl_xor(v, 32, 64));
}

template <int TM>
__global__ void __launch_bounds__(64, TM <= 4 ? 2 : 1) k_infer(
    const float* __restrict__ X, int n_rows, const float* __restrict__ A32,
    const float* __restrict__ Gf, const float* __restrict__ step32, int D, int K, int max_iter,
    float tol, float* __restrict__ out, bool given, bool gap_rule, float gap_tol, int min_steps,
    int* __restrict__ n_stepped, unsigned* __restrict__ queues) {
  constexpr bool kRegs = TM <= 4;   // G's fragments in registers
  const int lane = threadIdx.x, l16 = lane & 15, q = lane >> 4;
  const int nt = (K + 15) / 16;                        // tiles of topics (<= TM)
  const int last = min(4, K - 16 * (nt - 1));          // steps of the last tile with topics < K
  const float step = step32[0];
  const unsigned own = blockIdx.x % kInferQueues;
  unsigned* queue = queues + own * kInferQueueStride;
  // the row of this wave's queue's entry e
  auto queued = [&](unsigned e) { return e / 16 * (16 * kInferQueues) + 16 * own + e % 16; };
  float gf[kRegs ? TM * TM * 4 : 1];
  if (kRegs) {
#pragma unroll
    for (int i = 0; i < TM * TM * 4; ++i) {
      const int mo = i / (4 * TM), ks = i % (4 * TM);
      gf[i] = mo < nt && ks < 4 * nt ? Gf[(mo * 4 * nt + ks) * 64 + lane] : 0.f;
    }
  }
  float t[TM][4], b[TM][4];
#pragma unroll
  for (int m = 0; m < TM; ++m)
#pragma unroll
    for (int r = 0; r < 4; ++r) t[m][r] = b[m][r] = 0.f;
  int row = -1, it = 0, stepped = 0;
  float tau = 0.f;
  bool drained = false;
  auto topic = [&](int m, int r) { return 16 * m + 4 * q + r; };

  while (true) {
    const unsigned free = (unsigned)(__ballot(row < 0) & 0xffffull);
    const int nfree = __popc(free);
    if (nfree == 16 && drained) break;
    if (!drained && nfree >= kRefill) {
      // (unsigned: every wave's last request goes past n_rows)
      unsigned base = 0;
      if (lane == 0) base = atomicAdd(queue, (unsigned)nfree);
      base = (unsigned)__builtin_amdgcn_readfirstlane((int)base);
      drained = queued(base + nfree) >= (unsigned)n_rows;
      const unsigned mine = queued(base + __popc(free & ((1u << l16) - 1u)));
      const bool fresh = row < 0 && mine < (unsigned)n_rows;
      if (fresh) {
        row = (int)mine;
        it = 0;
        tau = -INFINITY;
      }
      if (__ballot(fresh) != 0) {
        floatx4 acc[TM];
#pragma unroll
        for (int m = 0; m < TM; ++m) acc[m] = floatx4{0.f, 0.f, 0.f, 0.f};
        const float* x = X + (size_t)(fresh ? row : 0) * D;
        for (int d0 = 0; d0 < D; d0 += 4) {
          const int d = d0 + q, dc = min(d, D - 1);
          const float xv = x[dc], xb = fresh && d < D ? xv : 0.f;
#pragma unroll
          for (int m = 0; m < TM; ++m)
            if (m < nt) {
              const float a = A32[dc * K + min(16 * m + l16, K - 1)];
              acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, xb, acc[m], 0, 0, 0);
            }
        }
        if (fresh) {
#pragma unroll
          for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const bool in = topic(m, r) < K;
              b[m][r] = in ? acc[m][r] : 0.f;
              t[m][r] = !in ? 0.f : given ? out[(size_t)row * K + topic(m, r)] : 1.0f / (float)K;
            }
        }
      }
    }
    bool done = row >= 0 && it >= max_iter;   // (at once when max_iter is 0)
    if (max_iter > 0) {
      // g = G t - b
      floatx4 acc[TM];
#pragma unroll
      for (int m = 0; m < TM; ++m) acc[m] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int mt = 0; mt < TM; ++mt) {
        if (mt >= nt) break;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (mt == nt - 1 && r >= last) break;
#pragma unroll
          for (int mo = 0; mo < TM; ++mo) {
            if (!kRegs && mo >= nt) break;
            const float a = kRegs ? gf[mo * 4 * TM + mt * 4 + r]
                                  : Gf[(mo * 4 * nt + mt * 4 + r) * 64 + lane];
            acc[mo] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, t[mt][r], acc[mo], 0, 0, 0);
          }
        }
      }
      float y[TM][4];
      float gt = 0.f, gmin = INFINITY;
#pragma unroll
      for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float g = acc[m][r] - b[m][r];
          const bool in = topic(m, r) < K;
          if (gap_rule) {
            gt = fmaf(g, t[m][r], gt);
            gmin = fminf(gmin, in ? g : INFINITY);
          }
          y[m][r] = in ? t[m][r] - step * g : -INFINITY;
        }
      if (gap_rule) {
        const bool close = group_sum(gt) - group_min(gmin) <= gap_tol;
        done = done || (row >= 0 && it >= min_steps && close);
        stepped += __popcll(__ballot(row >= 0 && it == min_steps && !done) & 0xffffull);
      }
      bool settled = row < 0 || done;
      int above = -1;
      for (int pass = 0; pass < K + 8; ++pass) {
        float s = 0.f;
        int c = 0;
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const bool a = y[m][r] > tau;
            s += a ? y[m][r] : 0.f;
            c += a ? 1 : 0;
          }
        s = group_sum(s);
        c = group_sum(c);
        settled = settled || c == above;
        above = c;
        if (__ballot(c == 0) != 0) {
          // nothing above an old tau: restart below the largest entry
          float mx = -INFINITY;
#pragma unroll
          for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) mx = fmaxf(mx, y[m][r]);
          mx = -group_min(-mx);
          // (no finite entry at all: the document's numbers are not finite)
          tau = c != 0 ? (s - 1.0f) / (float)c : mx > -INFINITY ? mx - 1.0f : 0.f;
        } else {
          tau = (s - 1.0f) / (float)c;
        }
        if (__ballot(!settled) == 0) break;
      }
      float change = 0.f;
      const bool move = row >= 0 && !done;
#pragma unroll
      for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float tn = fmaxf(y[m][r] - tau, 0.f);
          change += fabsf(tn - t[m][r]);
          t[m][r] = move ? tn : t[m][r];
        }
      if (move) ++it;
      done = done || (row >= 0 && it >= max_iter);
      if (!gap_rule && tol > 0.f) {
        const bool still = group_sum(change) < tol;
        done = done || (row >= 0 && still);
      }
    }
    if (done) {
#pragma unroll
      for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (topic(m, r) < K) out[(size_t)row * K + topic(m, r)] = t[m][r];
      row = -1;
    }
  }
  if (stepped > 0 && lane == 0) atomicAdd(n_stepped, stepped);
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
                                  float* Gf, float* step32, hipStream_t s) {
  hipError_t e = launch_project(W, m, mu, V, D, K, part, A, A32, s);
  if (e != hipSuccess) return e;
  const int n = K > D ? (K + 15) / 16 * 16 : (D + 15) / 16 * 16;
  hipLaunchKernelGGL(k_infer_G, dim3((n * n + 255) / 256), dim3(256), 0, s, A, D, K, G, Gf);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return launch_top_eig(G, K < D ? K : D, step32, s);
}

// The queues must be zero.  As many waves as the 256 compute units hold: three per
// SIMD with G in registers up to 64 topics, one past that.
static hipError_t launch_infer_k(const float* X, int n_rows, const float* A32, const float* Gf,
                                 const float* step32, int D, int K, int max_iter, float tol,
                                 float* theta, bool given, bool gap_rule, float gap_tol,
                                 int min_steps, int* n_stepped, int* queue, hipStream_t s) {
  if (n_rows == 0) return hipSuccess;
  const int waves = (n_rows + 15) / 16, most = K <= 64 ? 3072 : 1024;
  const dim3 grid(waves < most ? waves : most);
#define TLDA_INFER(tm)                                                                           \
  hipLaunchKernelGGL(k_infer<tm>, grid, dim3(64), 0, s, X, n_rows, A32, Gf, step32, D, K,        \
                     max_iter, tol, theta, given, gap_rule, gap_tol, min_steps, n_stepped,        \
                     reinterpret_cast<unsigned*>(queue))
  if (K <= 16) TLDA_INFER(1);
  else if (K <= 32) TLDA_INFER(2);
  else if (K <= 64) TLDA_INFER(4);
  else if (K <= 128) TLDA_INFER(8);
  else TLDA_INFER(16);
#undef TLDA_INFER
  return hipGetLastError();
}

hipError_t launch_infer(const float* X, int n_rows, const float* A32, const float* Gf,
                        const float* step32, int D, int K, int max_iter, float tol,
                        float* theta, int* queue, hipStream_t s) {
  return launch_infer_k(X, n_rows, A32, Gf, step32, D, K, max_iter, tol, theta, false, false, 0.f,
                        0, nullptr, queue, s);
}

hipError_t launch_infer_gap(const float* X, int n_rows, const float* A32, const float* Gf,
                            const float* step32, int D, int K, bool given_start, float gap_tol,
                            int min_steps, int max_iter, float* theta, int* n_stepped, int* queue,
                            hipStream_t s) {
  return launch_infer_k(X, n_rows, A32, Gf, step32, D, K, max_iter, 0.f, theta, given_start, true,
                        gap_tol, min_steps, n_stepped, queue, s);
}

}  // namespace tlda
