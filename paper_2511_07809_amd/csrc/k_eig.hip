// FP64 building blocks of the whitening refresh: the top-D eigenpairs of
// M2~ = (alpha0 + 1)(S2 / N - M1 M1^T) by block subspace iteration with
// Cholesky-QR orthonormalisation and a final Rayleigh-Ritz step solved by
// parallel-order cyclic Jacobi (section "Online Decomposition of the Second
// Moment": W = U diag(lambda)^(-1/2) so that W^T M2~ W = I).
#include <algorithm>

#include "tlda_internal.h"

namespace tlda {

thread_local EigEnv g_eig_env;

namespace {

// ---------------------------------------------------------------------------
// Dense FP64 GEMM on the vector ALUs (a second route to check the matrix
// cores' against): C (M x N) = A (M x Kd) B, all row-major.  64 x 64 output
// tile per 256-thread block, 4 x 4 register tile per thread, K step 16 staged
// through LDS.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_gemm64(int M, int N, int Kd, const double* __restrict__ A,
                                                int lda, const double* __restrict__ B, int ldb,
                                                double* __restrict__ C, int ldc,
                                                const int* __restrict__ pick,
                                                const double* __restrict__ B_set) {
  __shared__ double As[16][64 + 2];
  __shared__ double Bs[16][64 + 2];
  if (pick != nullptr && *pick) {
    if (B_set == nullptr) return;
    B = B_set;
  }
  const int tid = threadIdx.x;
  const int tx = tid & 15, ty = tid >> 4;
  const int row0 = blockIdx.y * 64, col0 = blockIdx.x * 64;
  double acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.0;

  for (int k0 = 0; k0 < Kd; k0 += 16) {
    // A tile: 64 rows x 16 k  ->  As[k][row]
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int idx = tid + e * 256;
      const int r = idx >> 4, kk = idx & 15;
      const int gr = row0 + r, gk = k0 + kk;
      As[kk][r] = gr < M && gk < Kd ? A[(size_t)gr * lda + gk] : 0.0;
    }
    // B tile: 16 k x 64 cols
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int idx = tid + e * 256;
      const int kk = idx >> 6, c = idx & 63;
      const int gk = k0 + kk, gc = col0 + c;
      Bs[kk][c] = (gk < Kd && gc < N) ? B[(size_t)gk * ldb + gc] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      double a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[kk][ty + 16 * i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Bs[kk][tx + 16 * j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fma(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int gr = row0 + ty + 16 * i;
    if (gr >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int gc = col0 + tx + 16 * j;
      if (gc < N) C[(size_t)gr * ldc + gc] = acc[i][j];
    }
  }
}

// ---------------------------------------------------------------------------
// Dense FP64 GEMM on the matrix cores: C (M x N) = A (M x K) B, row-major,
// v_mfma_f64_16x16x4f64 (lane l supplies A[l % 16][l / 16] and B[l / 16][l %
// 16]; accumulator register r of lane l is D[4 r + l / 16][l % 16]).
//
// Bound: the matrix cores (78.6 TFLOP/s FP64; 72 on a large library product
// here).  Block: 8 waves over a tile of 128 rows x 16 NT columns, NT <= 13, so
// that the refresh's products up to p = 208 read the V x V matrix once and
// compute no more than a tile's padding; a wave owns 16 rows and every column
// tile (one A operand feeds NT products; a 2 x NT / 2 split reads LDS less,
// which is not what bounds, and divides odd NT unevenly).  K advances 16 at a
// time through double-buffered LDS, A's slab with the reduction index
// leading, whose stride of 144 makes every operand read free of bank
// conflicts; the next slab is loaded into registers while the current one is
// multiplied (buffer loads from 32-bit offsets kept for the whole tile; rows
// of A past K are zeroed when they are stored, after the matrix work).
// SYM: A is symmetric, so its slab is read along its rows, as it lies in LDS.
// Work is dealt out in slabs: the tiles' slabs in a row, cut into gridDim.x
// equal runs, so that every compute unit ends together whatever M is.  A run
// that covers a tile writes C; the pieces of a divided tile go to ws, piece
// (block + tile), and k_dgemm_sum adds them in order.
// 20000^2 x 200: 2.70 ms, 59 TFLOP/s, and 27 us for the pieces (3.6 ms with
// narrower tiles and K in whole chunks); 20000^2 x 100: 1.5 ms, 53 TFLOP/s (1.95
// ms).  Storing the next slab before the last
// products changed neither.
// pick (or NULL): with B_set, *pick chooses the right operand (B_set where it
// is set); without it, nothing is done where it is set.
// ---------------------------------------------------------------------------
typedef double doublex4 __attribute__((ext_vector_type(4)));
constexpr int kDgBM = 128, kDgBK = 16, kDgThreads = 512, kDgMaxNT = 13;
constexpr int kDgLdA = kDgBM + 16;

struct DgPlan {
  int gx, gy, nt;         // column and row tiles, 16-column tiles per block
  int slabs;              // K slabs per tile
  int blocks;
  long long total() const { return (long long)gx * gy * slabs; }
  size_t ws() const {     // doubles of the pieces
    return blocks == gx * gy ? 0 : (size_t)(blocks + gx * gy) * kDgBM * 16 * nt;
  }
};
// One round of resident blocks: two on a CU while the sums of a tile take at
// most 112 columns (56 registers of a lane; one block above that has the CU's
// registers to itself).  Runs of at least 4 slabs; short products (K < 256: the
// block times a p x p matrix, 16 slabs at most) take whole tiles, whose pieces
// would be a read and a write of C more.
DgPlan dgemm_plan(int M, int N, int K, int num_cu) {
  DgPlan d;
  const int tiles = (N + 15) / 16;
  d.gx = (tiles + kDgMaxNT - 1) / kDgMaxNT;
  d.nt = (tiles + d.gx - 1) / d.gx;
  d.gy = (M + kDgBM - 1) / kDgBM;
  d.slabs = (K + kDgBK - 1) / kDgBK;
  const long long slots = (long long)num_cu * (d.nt <= 7 ? 2 : 1);
  const long long most = d.total() / 4 > 1 ? d.total() / 4 : 1;
  d.blocks = K < 256 ? d.gx * d.gy : (int)(slots < most ? slots : most);
  return d;
}

// Buffer descriptor of the doubles p .. end (an operand's slab starts at p; a
// lane's offset in it fits 32 bits, and reads past `end` give zero).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t slab(const double* p, const double* end) {
  const size_t bytes = (size_t)(end - p) * sizeof(double);
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(p), 0,
                                           (int)(uint32_t)(bytes < 0xfffffff0u ? bytes : 0xfffffff0u),
                                           0x00020000);
}

template <int NT, bool SYM>
__global__ void __launch_bounds__(kDgThreads, NT <= 7 ? 4 : 2) k_dgemm_mfma(
    int M, int N, int K, int gx, int slabs, long long total, const double* __restrict__ A, int lda,
    const double* __restrict__ B, int ldb, double* __restrict__ C, int ldc,
    double* __restrict__ ws, const int* __restrict__ pick, const double* __restrict__ B_set) {
  constexpr int BNC = 16 * NT, LDB_S = 16 * (NT | 1);
  constexpr int A_PER = kDgBM * kDgBK / kDgThreads;
  constexpr int B_PER = (kDgBK * BNC + kDgThreads - 1) / kDgThreads;
  __shared__ double As[2][kDgBK * kDgLdA];
  __shared__ double Bs[2][kDgBK * LDB_S];
  if (pick != nullptr && *pick) {
    if (B_set == nullptr) return;
    B = B_set;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  long long s0 = blockIdx.x * total / gridDim.x;
  const long long s1 = (blockIdx.x + 1) * total / gridDim.x;
  while (s0 < s1) {
    const int tile = (int)(s0 / slabs);
    const int kt0 = (int)(s0 - (long long)tile * slabs);
    const int kt1 = (int)min((long long)slabs, kt0 + (s1 - s0));
    s0 += kt1 - kt0;
    const int row0 = tile / gx * kDgBM, col0 = tile % gx * BNC;
    doublex4 acc[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[j] = doublex4{0.0, 0.0, 0.0, 0.0};
    double ra[A_PER], rb[B_PER];
    int oa[A_PER], ob[B_PER];
#pragma unroll
    for (int i = 0; i < A_PER; ++i) {
      const int e = tid + i * kDgThreads;
      const int r = min(SYM ? e % kDgBM : e / kDgBK, M - 1 - row0);
      const int k = SYM ? e / kDgBM : e % kDgBK;
      oa[i] = 8 * (SYM ? k * lda + r : r * lda + k);
    }
#pragma unroll
    for (int i = 0; i < B_PER; ++i) {
      const int e = min(tid + i * kDgThreads, kDgBK * BNC - 1);
      ob[i] = 8 * (e / BNC * ldb + min(e % BNC, N - 1 - col0));
    }
    auto load = [&](int k0) {
      const auto rsa = slab(SYM ? A + (size_t)k0 * lda + row0 : A + (size_t)row0 * lda + k0,
                            A + (size_t)(SYM ? K - 1 : M - 1) * lda + (SYM ? M : K));
      const auto rsb = slab(B + (size_t)k0 * ldb + col0, B + (size_t)(K - 1) * ldb + N);
#pragma unroll
      for (int i = 0; i < A_PER; ++i)
        ra[i] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rsa, oa[i], 0, 0));
#pragma unroll
      for (int i = 0; i < B_PER; ++i)
        rb[i] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rsb, ob[i], 0, 0));
    };
    auto store = [&](int buf, int k0) {
#pragma unroll
      for (int i = 0; i < A_PER; ++i) {
        const int e = tid + i * kDgThreads;
        const int r = SYM ? e % kDgBM : e / kDgBK, k = SYM ? e / kDgBM : e % kDgBK;
        As[buf][k * kDgLdA + r] = k0 + k < K ? ra[i] : 0.0;
      }
#pragma unroll
      for (int i = 0; i < B_PER; ++i) {
        const int e = tid + i * kDgThreads;
        if (e < kDgBK * BNC) Bs[buf][(e / BNC) * LDB_S + e % BNC] = rb[i];
      }
    };
    load(kt0 * kDgBK);
    store(0, kt0 * kDgBK);
    __syncthreads();
    for (int kt = kt0; kt < kt1; ++kt) {
      const int cur = (kt - kt0) & 1;
      if (kt + 1 < kt1) load((kt + 1) * kDgBK);
      const double* as = As[cur] + (lane >> 4) * kDgLdA + wave * 16 + (lane & 15);
      const double* bs = Bs[cur] + (lane >> 4) * LDB_S + (lane & 15);
#pragma unroll
      for (int ks = 0; ks < kDgBK / 4; ++ks) {
        const double a = as[4 * ks * kDgLdA];
#pragma unroll
        for (int j = 0; j < NT; ++j)
          acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, bs[4 * ks * LDB_S + j * 16], acc[j], 0,
                                                        0, 0);
      }
      if (kt + 1 < kt1) store(cur ^ 1, (kt + 1) * kDgBK);
      __syncthreads();
    }
    const bool whole = kt1 - kt0 == slabs;
    double* piece = ws + (size_t)(whole ? 0 : blockIdx.x + tile) * kDgBM * BNC;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int c = j * 16 + (lane & 15);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int rr = wave * 16 + 4 * r + (lane >> 4);
        if (!whole) piece[rr * BNC + c] = acc[j][r];
        else if (row0 + rr < M && col0 + c < N)
          C[(size_t)(row0 + rr) * ldc + col0 + c] = acc[j][r];
      }
    }
  }
}

// The divided tiles of k_dgemm_mfma: block (x, tile) adds its entries' pieces
// in block order, 8 loads in flight.
__global__ void __launch_bounds__(256) k_dgemm_sum(const double* __restrict__ ws, int M, int N,
                                                   int bnc, int gx, int slabs, int blocks,
                                                   double* __restrict__ C, int ldc,
                                                   const int* __restrict__ skip) {
  constexpr int kU = 8;
  if (skip != nullptr && *skip) return;
  const int tile = blockIdx.y;
  const long long total = (long long)gridDim.y * slabs, s = (long long)tile * slabs;
  // the block of slab s starts at or before it: b total / blocks < s + 1
  const int b0 = (int)(((s + 1) * blocks - 1) / total);
  const int b1 = (int)(((s + slabs) * blocks - 1) / total);
  if (b0 == b1) return;
  const size_t per = (size_t)kDgBM * bnc;
  const int e = blockIdx.x * 256 + threadIdx.x;          // kDgBM * bnc is a multiple of 256
  const double* p = ws + (size_t)(b0 + tile) * per + e;
  double sum = 0.0;
  for (int b = 0; b <= b1 - b0; b += kU) {
    double v[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) v[u] = p[(size_t)min(b + u, b1 - b0) * per];
#pragma unroll
    for (int u = 0; u < kU; ++u)
      if (b + u <= b1 - b0) sum += v[u];
  }
  const int row = tile / gx * kDgBM + e / bnc, col = tile % gx * bnc + e % bnc;
  if (row < M && col < N) C[(size_t)row * ldc + col] = sum;
}

template <bool SYM>
hipError_t dgemm_mfma(int M, int N, int K, const double* A, int lda, const double* B, int ldb,
                      double* C, int ldc, const int* pick, const double* B_set, hipStream_t s) {
  DgPlan d = dgemm_plan(M, N, K, g_eig_env.num_cu);
  if (d.ws() > g_eig_env.ws_doubles) d.blocks = d.gx * d.gy;
  switch (d.nt) {
#define TLDA_DG(n)                                                                                \
  case n:                                                                                         \
    hipLaunchKernelGGL((k_dgemm_mfma<n, SYM>), dim3(d.blocks), dim3(kDgThreads), 0, s, M, N, K,   \
                       d.gx, d.slabs, d.total(), A, lda, B, ldb, C, ldc, g_eig_env.ws, pick,      \
                       B_set);                                                                    \
    break;
    TLDA_DG(1) TLDA_DG(2) TLDA_DG(3) TLDA_DG(4) TLDA_DG(5) TLDA_DG(6) TLDA_DG(7) TLDA_DG(8)
    TLDA_DG(9) TLDA_DG(10) TLDA_DG(11) TLDA_DG(12) TLDA_DG(13)
#undef TLDA_DG
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || d.blocks == d.gx * d.gy) return e;
  hipLaunchKernelGGL(k_dgemm_sum, dim3(kDgBM * 16 * d.nt / 256, d.gx * d.gy), dim3(256), 0, s,
                     g_eig_env.ws, M, N, 16 * d.nt, d.gx, d.slabs, d.blocks, C, ldc,
                     B_set == nullptr ? pick : nullptr);
  return hipGetLastError();
}

// C (M x N) = A (M x Kd) B: the matrix cores, or the vector-ALU tile kernel.
// sym: A is symmetric.  pick, B_set: as for k_dgemm_mfma.
hipError_t gemm(int M, int N, int Kd, const double* A, int lda, const double* B, int ldb, double* C,
                int ldc, bool sym, const int* pick, const double* B_set, hipStream_t s) {
  if (g_eig_env.route == 0)
    return sym ? dgemm_mfma<true>(M, N, Kd, A, lda, B, ldb, C, ldc, pick, B_set, s)
               : dgemm_mfma<false>(M, N, Kd, A, lda, B, ldb, C, ldc, pick, B_set, s);
  hipLaunchKernelGGL(k_gemm64, dim3((N + 63) / 64, (M + 63) / 64), dim3(256), 0, s, M, N, Kd, A,
                     lda, B, ldb, C, ldc, pick, B_set);
  return hipGetLastError();
}

// splitmix64 (Steele, Lea & Flood 2014) as a counter-based generator for the
// refresh's start block: entry (i, c) is uniform in [-1, 1).
__device__ inline uint64_t splitmix64(uint64_t x) {
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}

__global__ void k_random_block(double* __restrict__ Q, int V, int p, uint64_t seed) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)V * p) return;
  const uint64_t r = splitmix64(seed * 0x100000001B3ull + idx);
  Q[idx] = (double)(r >> 11) * (1.0 / 9007199254740992.0) * 2.0 - 1.0;
}

// Cyclic Jacobi with the round-robin parallel ordering: in each round the
// m/2 disjoint pairs (circle method) are rotated at once, so every pair of
// indices is visited once per sweep.  A pair is rotated only while its
// off-diagonal entry is significant relative to its diagonal entries
// (|a_ij| > 1e-15 sqrt|a_ii a_jj|) and to the matrix (|a_ij| > 1e-20 |A|_F);
// a sweep without rotations ends the iteration.  A (p x p, symmetric) is
// diagonalised in place, Z accumulates the rotations, ev gets the diagonal.
// info |= 2 if 60 sweeps leave an off-diagonal mass above 1e-10 |A|_F.
__global__ void __launch_bounds__(1024) k_jacobi(double* __restrict__ A, double* __restrict__ Z,
                                                 double* __restrict__ ev, int p,
                                                 int* __restrict__ info) {
  extern __shared__ double sh[];   // c[m/2], s[m/2], pair indices, reduction scratch
  __shared__ int sh_rot;
  __shared__ double sh_norm;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int m = (p + 1) & ~1;
  const int half = m / 2;
  double* cs = sh;
  double* sn = sh + half;
  int* pi = reinterpret_cast<int*>(sh + 2 * half);
  int* pj = pi + half;
  double* red = sh + 3 * half;     // 2 * nt doubles
  for (int idx = tid; idx < p * p; idx += nt) Z[idx] = (idx / p == idx % p) ? 1.0 : 0.0;
  // Frobenius norm (invariant under the rotations)
  double tot = 0.0;
  for (int idx = tid; idx < p * p; idx += nt) tot += A[idx] * A[idx];
  red[tid] = tot;
  __syncthreads();
  for (int w = nt / 2; w > 0; w >>= 1) {
    if (tid < w) red[tid] += red[tid + w];
    __syncthreads();
  }
  if (tid == 0) sh_norm = sqrt(red[0]);
  __threadfence_block();
  __syncthreads();
  const double tiny = 1e-20 * sh_norm;
  for (int sweep = 0; sweep < 60; ++sweep) {
    if (tid == 0) sh_rot = 0;
    __syncthreads();
    for (int r = 0; r < m - 1; ++r) {
      for (int k = tid; k < half; k += nt) {
        int i, j;
        if (k == 0) { i = 0; j = 1 + r; }
        else {
          i = 1 + (r + k) % (m - 1);
          j = 1 + (r - k + (m - 1)) % (m - 1);
        }
        if (i > j) { const int t = i; i = j; j = t; }
        double c = 1.0, s = 0.0;
        if (j < p) {
          const double aij = A[(size_t)i * p + j];
          const double aii = A[(size_t)i * p + i], ajj = A[(size_t)j * p + j];
          if (fabs(aij) > tiny && fabs(aij) > 1e-15 * sqrt(fabs(aii * ajj))) {
            const double tau = (ajj - aii) / (2.0 * aij);
            const double t = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
            c = 1.0 / sqrt(1.0 + t * t);
            s = t * c;
            sh_rot = 1;
          }
        }
        pi[k] = i;
        pj[k] = j;
        cs[k] = c;
        sn[k] = s;
      }
      __syncthreads();
      // columns i, j of A and Z
      for (int idx = tid; idx < half * p; idx += nt) {
        const int k = idx / p, row = idx % p;
        const int i = pi[k], j = pj[k];
        const double s = sn[k];
        if (j >= p || s == 0.0) continue;
        const double c = cs[k];
        const double ai = A[(size_t)row * p + i], aj = A[(size_t)row * p + j];
        A[(size_t)row * p + i] = c * ai - s * aj;
        A[(size_t)row * p + j] = s * ai + c * aj;
        const double zi = Z[(size_t)row * p + i], zj = Z[(size_t)row * p + j];
        Z[(size_t)row * p + i] = c * zi - s * zj;
        Z[(size_t)row * p + j] = s * zi + c * zj;
      }
      __threadfence_block();
      __syncthreads();
      // rows i, j of A
      for (int idx = tid; idx < half * p; idx += nt) {
        const int k = idx / p, col = idx % p;
        const int i = pi[k], j = pj[k];
        const double s = sn[k];
        if (j >= p || s == 0.0) continue;
        const double c = cs[k];
        const double ai = A[(size_t)i * p + col], aj = A[(size_t)j * p + col];
        A[(size_t)i * p + col] = c * ai - s * aj;
        A[(size_t)j * p + col] = s * ai + c * aj;
      }
      __threadfence_block();
      __syncthreads();
    }
    if (sh_rot == 0) break;
    __syncthreads();
  }
  // final check of the remaining off-diagonal mass
  double off = 0.0;
  for (int idx = tid; idx < p * p; idx += nt)
    if (idx / p != idx % p) off += A[idx] * A[idx];
  red[tid] = off;
  __syncthreads();
  for (int w = nt / 2; w > 0; w >>= 1) {
    if (tid < w) red[tid] += red[tid + w];
    __syncthreads();
  }
  if (tid == 0 && sqrt(red[0]) > 1e-10 * sh_norm) atomicOr(info, 2);
  for (int i = tid; i < p; i += nt) ev[i] = A[(size_t)i * p + i];
}

// The same iteration for p <= kRotP: the packed lower triangle of A stays in
// LDS (160.8 KB at p = 200) and every rotation is written out, for
// k_jacobi_vectors to apply to Z afterwards, one row of Z per wave on its own
// compute unit; kept in one block, Z is as many LDS or L2 bytes a round again.
// Bound: LDS, half (half - 1) / 2 rotated 2 x 2 blocks a round, then the chain
// of a rotation's angle and two barriers a round.  (i, j) entry of A, i >= j,
// at i (i + 1) / 2 + j.  A thread owns the 2 x 2 blocks at the rows of pair a
// and the columns of pair b > a of the same (a, b) in every round, at most MAXB.
// rot: [sweeps][m - 1][half] rotations (c, s); *n_sweeps: sweeps that rotated.
// The rotations take 3.6 ms at p = 200 and 0.5 at p = 100, the vectors 0.29 and
// 0.1 (58 and 1.42 ms when one block kept matrix and vectors, the larger one in
// memory): a round is two barriers and one pair per thread, a serial chain.
// Past p = 200 the triangle does not fit LDS and k_jacobi keeps both in memory:
// the refresh at V = 5000, D = 100 takes 10 ms with p = 200 and 108 with 201
// (143 both before).
constexpr int kRotP = 200, kRotThreads = 1024, kMaxSweeps = 60;

__device__ __forceinline__ int tri(int i, int j) {
  const int hi = max(i, j), lo = min(i, j);
  return hi * (hi + 1) / 2 + lo;
}

// Pair k of round r of the circle method over m players.
__device__ __forceinline__ int2 circle_pair(int r, int k, int m) {
  int i, j;
  if (k == 0) {
    i = 0;
    j = 1 + r;
  } else {
    i = r + k;
    if (i >= m - 1) i -= m - 1;
    j = r - k;
    if (j < 0) j += m - 1;
    ++i;
    ++j;
  }
  return i < j ? make_int2(i, j) : make_int2(j, i);
}

// Barrier for LDS data alone: __syncthreads would also wait for the rotations
// on their way to memory, twice a round.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int MAXB>
__global__ void __launch_bounds__(kRotThreads) k_jacobi_rot(const double* __restrict__ Ag, int p,
                                                            double* __restrict__ ev,
                                                            double2* __restrict__ rot,
                                                            int* __restrict__ n_sweeps,
                                                            int* __restrict__ info) {
  extern __shared__ double A[];           // [p (p + 1) / 2]
  __shared__ double2 cs[kRotP / 2];
  __shared__ int2 pr[kRotP / 2];
  __shared__ double red[kRotThreads / 64];
  __shared__ int sh_rot;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m = (p + 1) & ~1, half = m / 2;
  auto block_sum = [&](double v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    __syncthreads();
    if (lane == 0) red[wave] = v;
    __syncthreads();
    double t = 0.0;
    for (int w = 0; w < kRotThreads / 64; ++w) t += red[w];
    return t;
  };
  // Frobenius norm (invariant under the rotations)
  double tot = 0.0;
  for (int idx = tid; idx < p * p; idx += kRotThreads) {
    const int i = idx / p, j = idx - i * p;
    if (j <= i) {
      const double v = Ag[idx];
      A[tri(i, j)] = v;
      tot += (i == j ? 1.0 : 2.0) * v * v;
    }
  }
  const double norm = sqrt(block_sum(tot));
  const double tiny = 1e-20 * norm;
  // this thread's blocks (a, b), a < b, of the half (half - 1) / 2
  int ba[MAXB], bb[MAXB];
#pragma unroll
  for (int u = 0; u < MAXB; ++u) {
    int t = tid + u * kRotThreads;
    ba[u] = -1;
    bb[u] = 0;
    if (t < half * (half - 1) / 2) {
      int b = 1;
      while (b * (b + 1) / 2 <= t) ++b;
      bb[u] = b;
      ba[u] = t - b * (b - 1) / 2;
    }
  }
  int sweep = 0;
  for (; sweep < kMaxSweeps; ++sweep) {
    if (tid == 0) sh_rot = 0;
    __syncthreads();
    for (int r = 0; r < m - 1; ++r) {
      if (tid < half) {
        const int2 ij = circle_pair(r, tid, m);
        double c = 1.0, s = 0.0;
        if (ij.y < p) {
          const int xii = tri(ij.x, ij.x), xjj = tri(ij.y, ij.y), xij = tri(ij.y, ij.x);
          const double aij = A[xij], aii = A[xii], ajj = A[xjj];
          if (fabs(aij) > tiny && aij * aij > 1e-30 * fabs(aii * ajj)) {
            // cos 2phi = |d| / h, h = sqrt(d^2 + o^2); c = cos phi, s of o's and d's signs
            const double d = ajj - aii, o = 2.0 * aij;
            const double ih = inv_sqrt(fma(d, d, o * o));
            const double c2 = fma(0.5 * fabs(d), ih, 0.5);
            const double rc = inv_sqrt(c2);
            const double hs = (d >= 0.0 ? 0.5 : -0.5) * o * ih;
            c = c2 * rc;
            s = hs * rc;
            const double t = s * rc;
            A[xii] = fma(-t, aij, aii);
            A[xjj] = fma(t, aij, ajj);
            A[xij] = 0.0;
            sh_rot = 1;
          }
        }
        pr[tid] = ij;
        cs[tid] = make_double2(c, s);
        rot[((size_t)sweep * (m - 1) + r) * half + tid] = make_double2(c, s);
      }
      lds_barrier();
      // A <- J^T A J on the block (a, b): b's columns, then a's rows.  Entries
      // at the padding index p do not exist.
#pragma unroll
      for (int u = 0; u < MAXB; ++u) {
        if (ba[u] < 0) continue;
        const double2 ra = cs[ba[u]], rb = cs[bb[u]];
        if (ra.y == 0.0 && rb.y == 0.0) continue;
        const int2 ia = pr[ba[u]], ib = pr[bb[u]];
        const bool ha = ia.y < p, hb = ib.y < p;
        const int t00 = tri(ia.x, ib.x), t01 = tri(ia.x, ib.y), t10 = tri(ia.y, ib.x),
                  t11 = tri(ia.y, ib.y);
        const double x00 = A[t00];
        const double x01 = hb ? A[t01] : 0.0, x10 = ha ? A[t10] : 0.0;
        const double x11 = ha && hb ? A[t11] : 0.0;
        const double y00 = rb.x * x00 - rb.y * x01, y01 = rb.y * x00 + rb.x * x01;
        const double y10 = rb.x * x10 - rb.y * x11, y11 = rb.y * x10 + rb.x * x11;
        A[t00] = ra.x * y00 - ra.y * y10;
        if (hb) A[t01] = ra.x * y01 - ra.y * y11;
        if (ha) A[t10] = ra.y * y00 + ra.x * y10;
        if (ha && hb) A[t11] = ra.y * y01 + ra.x * y11;
      }
      lds_barrier();
    }
    if (sh_rot == 0) break;
    __syncthreads();
  }
  // final check of the remaining off-diagonal mass
  double off = 0.0;
  for (int idx = tid; idx < p * p; idx += kRotThreads) {
    const int i = idx / p, j = idx - i * p;
    if (j < i) off += 2.0 * A[tri(i, j)] * A[tri(i, j)];
  }
  off = block_sum(off);
  if (tid == 0) {
    if (sqrt(off) > 1e-10 * norm) atomicOr(info, 2);
    *n_sweeps = sweep;
  }
  for (int i = tid; i < p; i += kRotThreads) ev[i] = A[tri(i, i)];
}

// Z = the product of k_jacobi_rot's rotations: one wave per row of Z, the row
// in LDS, lane l taking pairs l and l + 64 of every round; the next round's
// rotations are on their way while this one's are applied.
__global__ void __launch_bounds__(64) k_jacobi_vectors(const double2* __restrict__ rot,
                                                       const int* __restrict__ n_sweeps, int p,
                                                       double* __restrict__ Z) {
  __shared__ double z[kRotP + 2];
  const int lane = threadIdx.x, row = blockIdx.x;
  const int m = (p + 1) & ~1, half = m / 2;
  for (int i = lane; i < m; i += 64) z[i] = i == row ? 1.0 : 0.0;
  const int rounds = *n_sweeps * (m - 1);
  const int k0 = min(lane, half - 1), k1 = min(lane + 64, half - 1);
  constexpr int kU = 4;   // rounds of rotations in flight
  double2 q0[kU], q1[kU];
#pragma unroll
  for (int u = 0; u < kU; ++u) {
    const size_t o = (size_t)min(u, max(rounds - 1, 0)) * half;
    q0[u] = rot[o + k0];
    q1[u] = rot[o + k1];
  }
  int r = 0;
  for (int t = 0; t < rounds; t += kU) {
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const double2 c0 = q0[u], c1 = q1[u];
      const size_t o = (size_t)min(t + u + kU, rounds - 1) * half;
      q0[u] = rot[o + k0];
      q1[u] = rot[o + k1];
      if (t + u < rounds) {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (lane < half && c0.y != 0.0) {
          const int2 ij = circle_pair(r, lane, m);
          const double a = z[ij.x], b = z[ij.y];
          z[ij.x] = c0.x * a - c0.y * b;
          z[ij.y] = c0.y * a + c0.x * b;
        }
        if (lane + 64 < half && c1.y != 0.0) {
          const int2 ij = circle_pair(r, lane + 64, m);
          const double a = z[ij.x], b = z[ij.y];
          z[ij.x] = c1.x * a - c1.y * b;
          z[ij.y] = c1.y * a + c1.x * b;
        }
        if (++r == m - 1) r = 0;
      }
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
  for (int i = lane; i < p; i += 64) Z[(size_t)row * p + i] = z[i];
}

// Sorts the Ritz values in decreasing order (ties: lower index first), keeps
// the top D, and gathers the matching eigenvector columns into Zs [p][D].
__global__ void __launch_bounds__(256) k_select_top(const double* __restrict__ Z,
                                                    const double* __restrict__ ev, int p, int D,
                                                    double* __restrict__ Zs,
                                                    double* __restrict__ eigD) {
  for (int c = threadIdx.x; c < p; c += blockDim.x) {
    int rank = 0;
    const double v = ev[c];
    for (int k = 0; k < p; ++k) {
      const double w = ev[k];
      if (w > v || (w == v && k < c)) ++rank;
    }
    if (rank < D) {
      eigD[rank] = v;
      for (int r = 0; r < p; ++r) Zs[(size_t)r * D + rank] = Z[(size_t)r * p + c];
    }
  }
}

// Sign rule: the entry of largest magnitude of every column of U (V x D) is
// made positive (lowest row index on ties).  One block per column.
__global__ void __launch_bounds__(256) k_sign_fix(double* __restrict__ U, int V, int D) {
  __shared__ double bv[256];
  __shared__ int bi[256];
  const int col = blockIdx.x, tid = threadIdx.x;
  double best = -1.0;
  int besti = V;
  for (int i = tid; i < V; i += blockDim.x) {
    const double a = fabs(U[(size_t)i * D + col]);
    if (a > best) { best = a; besti = i; }
  }
  bv[tid] = best;
  bi[tid] = besti;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if (tid < w) {
      if (bv[tid + w] > bv[tid] || (bv[tid + w] == bv[tid] && bi[tid + w] < bi[tid])) {
        bv[tid] = bv[tid + w];
        bi[tid] = bi[tid + w];
      }
    }
    __syncthreads();
  }
  const bool flip = bi[0] < V && U[(size_t)bi[0] * D + col] < 0.0;
  __syncthreads();
  if (flip)
    for (int i = tid; i < V; i += blockDim.x) U[(size_t)i * D + col] = -U[(size_t)i * D + col];
}

// W = U diag(eig)^(-1/2) in FP64 and its FP32 copy with row stride Dp (zero
// padding beyond D).
__global__ void k_form_w(const double* __restrict__ U, const double* __restrict__ eig, int V, int D,
                         int Dp, double* __restrict__ W, float* __restrict__ W32) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)V * Dp) return;
  const int i = (int)(idx / Dp), d = (int)(idx % Dp);
  if (d < D) {
    const double w = U[(size_t)i * D + d] / sqrt(eig[d]);
    W[(size_t)i * D + d] = w;
    W32[idx] = (float)w;
  } else {
    W32[idx] = 0.0f;
  }
}

// mw32[d] = sum_i W[i][d] m[i] (FP64 sum, one block per column); padding zero.
__global__ void __launch_bounds__(256) k_mw(const double* __restrict__ W, const double* __restrict__ m,
                                            int V, int D, int Dp, float* __restrict__ mw32) {
  __shared__ double red[256];
  const int d = blockIdx.x, tid = threadIdx.x;
  if (d >= D) {
    if (tid == 0) mw32[d] = 0.0f;
    return;
  }
  double s = 0.0;
  for (int i = tid; i < V; i += blockDim.x) s += W[(size_t)i * D + d] * m[i];
  red[tid] = s;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if (tid < w) red[tid] += red[tid + w];
    __syncthreads();
  }
  if (tid == 0) mw32[d] = (float)red[0];
}

// For an injected W: eig[d] = 1 / |w_d|^2 and U = W diag(eig)^(1/2).
__global__ void __launch_bounds__(256) k_from_injected(const double* __restrict__ W, int V, int D,
                                                       double* __restrict__ U,
                                                       double* __restrict__ eig) {
  __shared__ double red[256];
  const int d = blockIdx.x, tid = threadIdx.x;
  double s = 0.0;
  for (int i = tid; i < V; i += blockDim.x) {
    const double w = W[(size_t)i * D + d];
    s += w * w;
  }
  red[tid] = s;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if (tid < w) red[tid] += red[tid + w];
    __syncthreads();
  }
  const double nrm2 = red[0];
  if (tid == 0) eig[d] = nrm2 > 0.0 ? 1.0 / nrm2 : 0.0;
  const double sc = nrm2 > 0.0 ? 1.0 / sqrt(nrm2) : 0.0;
  for (int i = tid; i < V; i += blockDim.x) U[(size_t)i * D + d] = W[(size_t)i * D + d] * sc;
}

inline int blocks_for(size_t n, int bs) { return (int)((n + bs - 1) / bs); }

}  // namespace

hipError_t launch_random_block(double* Q, int V, int p, uint64_t seed, hipStream_t s) {
  hipLaunchKernelGGL(k_random_block, dim3(blocks_for((size_t)V * p, 256)), dim3(256), 0, s, Q, V,
                     p, seed);
  return hipGetLastError();
}

hipError_t launch_m2_apply(const double* M2, const double* Q, double* Y, int V, int p,
                           const int* pick, const double* Q_set, hipStream_t s) {
  return gemm(V, p, V, M2, V, Q, p, Y, p, true, pick, Q_set, s);
}

size_t jacobi_scratch_doubles(int p) {
  if (p > kRotP) return 0;
  const size_t m = (p + 1) & ~1;
  return 2 * (size_t)kMaxSweeps * (m - 1) * (m / 2);
}

hipError_t launch_jacobi(double* A, double* Z, double* ev, int p, double* scratch, int* info,
                         hipStream_t s) {
  if (p <= kRotP) {
    const size_t lds = sizeof(double) * p * (p + 1) / 2;
    auto kernel = p <= 128 ? k_jacobi_rot<2> : k_jacobi_rot<5>;
    if (lds > 60 * 1024) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                               hipFuncAttributeMaxDynamicSharedMemorySize,
                                               (int)lds);
      if (e != hipSuccess) return e;
    }
    double2* rot = reinterpret_cast<double2*>(scratch);
    hipLaunchKernelGGL(kernel, dim3(1), dim3(kRotThreads), lds, s, A, p, ev, rot, info + 2, info);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_jacobi_vectors, dim3(p), dim3(64), 0, s, rot, info + 2, p, Z);
    return hipGetLastError();
  }
  const int m = (p + 1) & ~1;
  const int nt = 1024;
  const size_t shmem = sizeof(double) * (3 * (m / 2) + 2 * nt) + sizeof(int) * m;
  hipLaunchKernelGGL(k_jacobi, dim3(1), dim3(nt), shmem, s, A, Z, ev, p, info);
  return hipGetLastError();
}

hipError_t launch_block_product(const double* Q, const double* Z, double* Out, int V, int p,
                                const int* skip, hipStream_t s) {
  return gemm(V, p, p, Q, p, Z, p, Out, p, false, skip, nullptr, s);
}

hipError_t launch_ritz_vectors(const double* Q, const double* Z, const double* ev, int V, int p,
                               int D, double* U, double* eigD, hipStream_t s) {
  // Zs is placed right after eigD's D entries in caller scratch: eigD [D], Zs [p][D]
  double* Zs = eigD + D;
  hipLaunchKernelGGL(k_select_top, dim3(1), dim3(256), 0, s, Z, ev, p, D, Zs, eigD);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = gemm(V, D, p, Q, p, Zs, D, U, D, false, nullptr, nullptr, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_sign_fix, dim3(D), dim3(256), 0, s, U, V, D);
  return hipGetLastError();
}

hipError_t launch_form_whitening(const double* U, const double* eig, const double* m, int V, int D,
                                 int Dp, double* W, float* W32, float* mw32, hipStream_t s) {
  hipLaunchKernelGGL(k_form_w, dim3(blocks_for((size_t)V * Dp, 256)), dim3(256), 0, s, U, eig, V,
                     D, Dp, W, W32);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_mw, dim3(Dp), dim3(256), 0, s, W, m, V, D, Dp, mw32);
  return hipGetLastError();
}

hipError_t launch_from_injected(const double* W, int V, int D, double* U, double* eig,
                                hipStream_t s) {
  hipLaunchKernelGGL(k_from_injected, dim3(D), dim3(256), 0, s, W, V, D, U, eig);
  return hipGetLastError();
}

size_t dgemm_ws_doubles(int M, int N, int K, int num_cu) {
  return dgemm_plan(M, N, K, num_cu).ws();
}

}  // namespace tlda
