// The refresh's orthonormalisation on the FP64 matrix cores: Gram products of
// tall blocks (k_gram, below), and the Cholesky factor and triangular inverse
// of the p x p Gram matrix, G + shift I = R^T R (R upper), Binv = R^-1, so
// that Q = Y Binv is orthonormal.
//
// Factor and inverse.
// Bound: a chain of p pivots.  Each costs a reciprocal square root and a
// rank-one update; only the 16 pivots of a diagonal tile have to be taken one
// at a time, so a single wave does those in registers and everything else of
// the block step (the tile row of R, the trailing update, the inverse) is
// 16 x 16 x 16 products on v_mfma_f64_16x16x4f64.
//
// Tiles are kept in the accumulator layout of that instruction: register r of
// lane l holds entry (4 r + l / 16, l % 16), which is entry r * 64 + l of the
// row-major tile.  With the upper factor no product needs a transpose:
//   row of R  : R_kj = R_kk^-T A_kj      B operand = accumulators of A_kj
//   trailing  : A_ij -= R_ki^T R_kj      both operands = tiles as stored
//   inverse   : L^-1 (= Binv^T), block column i, Y_ii = R_ii^-T,
//               Y_ji = -R_jj^-T sum_k R_kj^T Y_ki, again both as stored
// since lane l supplies A[l % 16][4 s + l / 16] and B[4 s + l / 16][l % 16] in
// step s.  R_kk^-T is stored by columns, where entry s * 64 + l is the A
// operand.
//
// Factor and inverse at p = 100: 45 us (34 and 11), 145 before (a wave per
// column and a block-wide barrier per pivot, on the vector ALUs); at p = 200:
// 88 and 27 us, 1420 before (the matrix in memory); at p = 21: 12 us, 29 before.
// A 16-pivot step takes 4.75 us of them.
#include "tlda_internal.h"

namespace tlda {
namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));
constexpr int kTile = 16, kTileE = kTile * kTile, kMaxNb = 32;   // p <= 512

__device__ __forceinline__ int tile_at(int i, int j) { return j * (j + 1) / 2 + i; }   // i <= j

// the same tile in the order k_gram numbers them (by tile rows)
__device__ __forceinline__ int part_tile(int i, int j, int nb) {
  return i * nb - i * (i - 1) / 2 + (j - i);
}

__device__ __forceinline__ double lane_value(double v, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
  return __hiloint2double(hi, lo);
}

// Orders this wave's LDS stores before its later LDS loads by other lanes.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ doublex4 load_tile(const double* t, int lane) {
  return doublex4{t[lane], t[64 + lane], t[128 + lane], t[192 + lane]};
}
__device__ __forceinline__ void store_tile(double* t, int lane, doublex4 v) {
#pragma unroll
  for (int r = 0; r < 4; ++r) t[r * 64 + lane] = v[r];
}

// acc += op(a) b over 16 terms, operands as in the file comment
__device__ __forceinline__ doublex4 tile_mfma(doublex4 a, doublex4 b, doublex4 acc) {
#pragma unroll
  for (int s = 0; s < 4; ++s)
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], acc, 0, 0, 0);
  return acc;
}

// One wave: the Cholesky factor of the 16 x 16 tile `a` (row-major in LDS)
// and the inverse of its transpose.  Lanes 0-15 (and 32-47) hold a column of
// the tile, lanes 16-31 a column of the identity, and both take the same
// elimination, which turns the identity into R^-T.  A pivot that is not
// positive is taken as one and reported.
__device__ inline bool factor_tile(const double* a, int lane, double* r_out, double* rinvt_cols) {
  const int c = lane & 15;
  const bool ident = (lane >> 4) & 1;
  double v[kTile];
#pragma unroll
  for (int i = 0; i < kTile; ++i) v[i] = ident ? (i == c ? 1.0 : 0.0) : a[i * kTile + c];
  bool ok = true;
#pragma unroll
  for (int j = 0; j < kTile; ++j) {
    const double d = lane_value(v[j], j);
    const bool pos = d > 0.0;
    ok = ok && pos;
    const double rs = inv_sqrt(d);
    v[j] *= pos ? rs : 1.0;
    v[j] = !pos && lane == j ? 1.0 : v[j];
    // Every later row is updated here and now: left to itself the compiler
    // puts row i's updates off to pivot i, where they are a chain, and holds
    // all the multipliers in (spilled) scalar registers until then.
#pragma unroll
    for (int i = j + 1; i < kTile; ++i) {
      v[i] = fma(-lane_value(v[j], i), v[j], v[i]);
      asm volatile("" : "+v"(v[i]));
    }
  }
  wave_sync();
  if (lane < 16) {
#pragma unroll
    for (int i = 0; i < kTile; ++i) r_out[i * kTile + c] = i <= c ? v[i] : 0.0;
  } else if (lane < 32) {
#pragma unroll
    for (int i = 0; i < kTile; ++i) rinvt_cols[c * kTile + i] = v[i];
  }
  return ok;
}

// Entry (gi, gj) of the symmetric matrix padded to whole tiles by the
// identity, read from the upper triangle.
__device__ __forceinline__ double padded(const double* G, int p, int gi, int gj) {
  const int a = min(gi, gj), b = max(gi, gj);
  return b < p ? G[(size_t)a * p + b] : a == b ? 1.0 : 0.0;
}

// One wave: block column i of L^-1 = R^-T from the tiles of R and of the
// diagonal inverses, written to Binv = R^-1 (row-major, p x p; the part below
// the diagonal is left alone).  y: this column's own tiles, in LDS.  The tiles
// of R are loaded four at a time, ahead of the products that take them.
__device__ inline void inverse_column(const double* tiles, const double* dinv, int nb, int i, int p,
                                      double* y, double* Binv, int lane) {
  constexpr int kU = 4;
  const int row = lane >> 4, col = lane & 15;
  for (int j = i; j < nb; ++j) {
    doublex4 v;
    if (j == i) {
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = dinv[i * kTileE + col * kTile + 4 * r + row];
    } else {
      const doublex4 d = load_tile(dinv + j * kTileE, lane);
      doublex4 s[kU], a[kU];   // an accumulator each: consecutive products do not wait
#pragma unroll
      for (int u = 0; u < kU; ++u) s[u] = doublex4{0.0, 0.0, 0.0, 0.0};
      for (int k = i; k < j; k += kU) {
#pragma unroll
        for (int u = 0; u < kU; ++u)
          a[u] = load_tile(tiles + (size_t)tile_at(min(k + u, j - 1), j) * kTileE, lane);
#pragma unroll
        for (int u = 0; u < kU; ++u)
          if (k + u < j) s[u] = tile_mfma(a[u], load_tile(y + (k + u) * kTileE, lane), s[u]);
      }
      v = tile_mfma(d, -((s[0] + s[1]) + (s[2] + s[3])), doublex4{0.0, 0.0, 0.0, 0.0});
    }
    store_tile(y + j * kTileE, lane, v);
    wave_sync();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int gr = i * kTile + col, gc = j * kTile + 4 * r + row;
      if (gr < p && gc < p && gr <= gc) Binv[(size_t)gr * p + gc] = v[r];
    }
  }
}

// The largest nb whose nb (nb + 1) / 2 tiles are at most n.
constexpr int panel_tiles(int n) {
  int nb = 1;
  while ((nb + 1) * (nb + 2) / 2 <= n) ++nb;
  return nb;
}

// Where the diagonal of R spans less than this, the iteration goes on without
// the second Cholesky-QR pass (the cold refresh at V = 20000, p = 200 takes 263
// ms with it everywhere, 244 without it there).  Between iterations only the
// span of the block matters, which one pass leaves as it is; its columns need
// not be orthonormal, just far from dependent.  With G + s I = R^T R they come
// out with Q^T Q = I - s R^-T R^-1, off by s / sigma_min(R)^2: about 1e-4 at this
// limit with the shift s of 1e-12 of the largest diagonal entry.  (The diagonal
// of an unpivoted R only estimates its condition, so this is a rule of thumb; the
// last iteration before the projection always runs both passes.)
constexpr double kWell = 1e-4;

// The factor, tiles in registers: one block of NW waves, tile t = tile_at(i, j)
// in slot t / NW of wave t % NW (NW SLOTS >= the tile count; at most two waves
// per SIMD, so that a tile being factored fits beside them).  Nothing is
// written to memory before the last step, since every barrier would wait for
// it.  skip (or NULL): nothing to do when it is set.  well (or NULL) receives 1
// when the smallest diagonal entry of R is at least kWell of the largest.
// nz > 0: G holds the nz chunks of a Gram product's tiles (k_gram), which are
// added here in chunk order: a launch less where there are few.  INV: the block
// goes on to the inverse, its tiles in LDS.
template <int NW, int SLOTS, bool INV>
__global__ void __launch_bounds__(64 * NW) k_chol(const double* __restrict__ G, int p,
                                                  double shift_rel, double* __restrict__ tiles,
                                                  double* __restrict__ dinv,
                                                  double* __restrict__ Binv,
                                                  int* __restrict__ info,
                                                  const int* __restrict__ skip,
                                                  int* __restrict__ well, int nz) {
  constexpr int NB = panel_tiles(NW * SLOTS);
  if (skip != nullptr && *skip) return;
  // row k of R while it is applied (INV: every tile of R, kept)
  __shared__ double panel[(INV ? NB * (NB + 1) / 2 : NB) * kTileE];
  __shared__ double dcols[NB * kTileE], diag[kTileE];
  __shared__ double ybuf[INV ? NB * NB * kTileE : 1];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb = (p + kTile - 1) / kTile, nt = nb * (nb + 1) / 2;
  const int row = lane >> 4, col = lane & 15;
  doublex4 acc[SLOTS];
  int ti[SLOTS], tj[SLOTS];
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    const int t = wave + NW * s;
    ti[s] = tj[s] = -1;
    if (t < nt) {
      int j = 0;
      while ((j + 1) * (j + 2) / 2 <= t) ++j;
      tj[s] = j;
      ti[s] = t - j * (j + 1) / 2;
      if (nz > 0) {
        const double* g = G + (size_t)part_tile(ti[s], j, nb) * kTileE;
        acc[s] = doublex4{0.0, 0.0, 0.0, 0.0};
        for (int z = 0; z < nz; z += 8) {   // 8 chunks' loads in flight
          doublex4 c[8];
#pragma unroll
          for (int u = 0; u < 8; ++u)
            c[u] = load_tile(g + (size_t)min(z + u, nz - 1) * nt * kTileE, lane);
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if (z + u < nz) acc[s] += c[u];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int gi = ti[s] * kTile + 4 * r + row, gj = j * kTile + col;
          if (max(gi, gj) >= p) acc[s][r] = gi == gj ? 1.0 : 0.0;
        }
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          acc[s][r] = padded(G, p, ti[s] * kTile + 4 * r + row, j * kTile + col);
      }
    }
  }
  double mx = 0.0;
  for (int i = lane; i < p; i += 64) {
    double g = 0.0;
    if (nz > 0) {
      const double* d = G + (size_t)part_tile(i / kTile, i / kTile, nb) * kTileE + i % kTile * (kTile + 1);
      for (int z = 0; z < nz; z += 8) {
        double c[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) c[u] = d[(size_t)min(z + u, nz - 1) * nt * kTileE];
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (z + u < nz) g += c[u];
      }
    } else {
      g = G[(size_t)i * p + i];
    }
    mx = fmax(mx, g);
  }
  for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off, 64));
  const double shift = shift_rel * mx;
#pragma unroll
  for (int s = 0; s < SLOTS; ++s)
    if (ti[s] >= 0 && ti[s] == tj[s]) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (4 * r + row == col && ti[s] * kTile + col < p) acc[s][r] += shift;
    }
  bool ok = true;
  const doublex4 zero = {0.0, 0.0, 0.0, 0.0};
  for (int k = 0; k < nb; ++k) {
    if (tile_at(k, k) % NW == wave) {   // its owner factors the diagonal tile
#pragma unroll
      for (int s = 0; s < SLOTS; ++s)
        if (ti[s] == k && tj[s] == k) store_tile(diag, lane, acc[s]);
      wave_sync();
      ok = factor_tile(diag, lane, diag, dcols + k * kTileE) && ok;
      wave_sync();
#pragma unroll
      for (int s = 0; s < SLOTS; ++s)
        if (ti[s] == k && tj[s] == k) acc[s] = load_tile(diag, lane);
    }
    __syncthreads();
    // row k of R: R_kj = R_kk^-T A_kj
    const doublex4 da = load_tile(dcols + k * kTileE, lane);
#pragma unroll
    for (int s = 0; s < SLOTS; ++s)
      if (ti[s] == k && tj[s] > k) {
        acc[s] = tile_mfma(da, acc[s], zero);
        store_tile(panel + (INV ? wave + NW * s : tj[s]) * kTileE, lane, acc[s]);
      }
    __syncthreads();
    // trailing tiles: A_ij -= R_ki^T R_kj
#pragma unroll
    for (int s = 0; s < SLOTS; ++s)
      if (ti[s] > k)
        acc[s] = tile_mfma(-load_tile(panel + (INV ? tile_at(k, ti[s]) : ti[s]) * kTileE, lane),
                           load_tile(panel + (INV ? tile_at(k, tj[s]) : tj[s]) * kTileE, lane),
                           acc[s]);
  }
  if (!ok && lane == 0) atomicOr(info, 1);
  if (well != nullptr) {
    // diag is free now: the waves' smallest and largest diagonal entries
    double lo = INFINITY, hi = 0.0;
#pragma unroll
    for (int s = 0; s < SLOTS; ++s)
      if (ti[s] >= 0 && ti[s] == tj[s]) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (4 * r + row == col && ti[s] * kTile + col < p) {
            lo = fmin(lo, acc[s][r]);
            hi = fmax(hi, acc[s][r]);
          }
      }
    for (int off = 32; off > 0; off >>= 1) {
      lo = fmin(lo, __shfl_xor(lo, off, 64));
      hi = fmax(hi, __shfl_xor(hi, off, 64));
    }
    if (lane == 0) {
      diag[2 * wave] = lo;
      diag[2 * wave + 1] = hi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < NW; ++w) {
        lo = fmin(lo, diag[2 * w]);
        hi = fmax(hi, diag[2 * w + 1]);
      }
      *well = lo >= kWell * hi ? 1 : 0;
    }
  }
  if (INV) {
    for (int i = wave; i < nb; i += NW)
      inverse_column(panel, dcols, nb, i, p, ybuf + i * NB * kTileE, Binv, lane);
  } else {
#pragma unroll
    for (int s = 0; s < SLOTS; ++s)
      if (ti[s] >= 0) store_tile(tiles + (size_t)(wave + NW * s) * kTileE, lane, acc[s]);
    for (int k = wave; k < nb; k += NW)
      store_tile(dinv + k * kTileE, lane, load_tile(dcols + k * kTileE, lane));
  }
}

// The same for more tiles than fit in registers (91 at p = 208): they live in
// `tiles`, each touched by wave t % 16 alone.
__global__ void __launch_bounds__(1024) k_chol_mem(const double* __restrict__ G, int p,
                                                   double shift_rel, double* tiles, double* dinv,
                                                   int* __restrict__ info,
                                                   const int* __restrict__ skip,
                                                   int* __restrict__ well) {
  constexpr int NW = 16;
  if (skip != nullptr && *skip) return;
  __shared__ double panel[kMaxNb * kTileE];
  __shared__ double diag[kTileE], dcols[kTileE];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb = (p + kTile - 1) / kTile, nt = nb * (nb + 1) / 2;
  const int row = lane >> 4, col = lane & 15;
  double mx = 0.0;
  for (int i = lane; i < p; i += 64) mx = fmax(mx, G[(size_t)i * p + i]);
  for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off, 64));
  const double shift = shift_rel * mx;
  for (int t = wave; t < nt; t += NW) {
    int j = 0;
    while ((j + 1) * (j + 2) / 2 <= t) ++j;
    const int i = t - j * (j + 1) / 2;
    doublex4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int gi = i * kTile + 4 * r + row, gj = j * kTile + col;
      v[r] = padded(G, p, gi, gj) + (gi == gj && gi < p ? shift : 0.0);
    }
    store_tile(tiles + (size_t)t * kTileE, lane, v);
  }
  __threadfence_block();
  const doublex4 zero = {0.0, 0.0, 0.0, 0.0};
  for (int k = 0; k < nb; ++k) {
    const int tk = tile_at(k, k);
    if (tk % NW == wave) {
      store_tile(diag, lane, load_tile(tiles + (size_t)tk * kTileE, lane));
      wave_sync();
      const bool ok = factor_tile(diag, lane, tiles + (size_t)tk * kTileE, dcols);
      if (!ok && lane == 0) atomicOr(info, 1);
      wave_sync();
      store_tile(dinv + k * kTileE, lane, load_tile(dcols, lane));
    }
    __syncthreads();
    const doublex4 da = load_tile(dcols, lane);
    for (int j = k + 1; j < nb; ++j) {
      const int t = tile_at(k, j);
      if (t % NW != wave) continue;
      const doublex4 v = tile_mfma(da, load_tile(tiles + (size_t)t * kTileE, lane), zero);
      store_tile(panel + j * kTileE, lane, v);
      store_tile(tiles + (size_t)t * kTileE, lane, v);
    }
    __syncthreads();
    for (int j = k + 1; j < nb; ++j)
      for (int i = k + 1; i <= j; ++i) {
        const int t = tile_at(i, j);
        if (t % NW != wave) continue;
        double* tp = tiles + (size_t)t * kTileE;
        store_tile(tp, lane, tile_mfma(-load_tile(panel + i * kTileE, lane),
                                       load_tile(panel + j * kTileE, lane), load_tile(tp, lane)));
      }
  }
  if (well == nullptr) return;
  __threadfence_block();
  __syncthreads();
  if (wave == 0) {
    double lo = INFINITY, hi = 0.0;
    for (int j = lane; j < p; j += 64) {
      const double d = tiles[(size_t)tile_at(j / kTile, j / kTile) * kTileE + j % kTile * (kTile + 1)];
      lo = fmin(lo, d);
      hi = fmax(hi, d);
    }
    for (int off = 32; off > 0; off >>= 1) {
      lo = fmin(lo, __shfl_xor(lo, off, 64));
      hi = fmax(hi, __shfl_xor(hi, off, 64));
    }
    if (lane == 0) *well = lo >= kWell * hi ? 1 : 0;
  }
}

// One wave per block column of the inverse: independent chains, so the columns
// go to different compute units (27 us at p = 200; 123 in one block of waves).
__global__ void __launch_bounds__(64) k_tri_inverse(const double* __restrict__ tiles,
                                                    const double* __restrict__ dinv, int p,
                                                    double* __restrict__ Binv,
                                                    const int* __restrict__ skip) {
  __shared__ double y[kMaxNb * kTileE];
  if (skip != nullptr && *skip) return;
  const int nb = (p + kTile - 1) / kTile;
  inverse_column(tiles, dinv, nb, blockIdx.x, p, y, Binv, threadIdx.x);
}

// ---------------------------------------------------------------------------
// G (pa x pb) = A^T (B - m 1^T) for tall row-major blocks A (V x pa), B (V x
// pb); m [V] or NULL.  Lane l of a step over four rows v needs A[v + l / 16]
// [16 i + l % 16] and B[v + l / 16][16 j + l % 16]: 128-byte row segments
// straight from memory, no staging.  A block takes one unit of at most kGramN
// tiles of one tile row (one A operand feeds them all) and one chunk of the
// rows, its four waves every fourth group of four rows; the waves' tiles are
// added in LDS, the chunks' in chunk order by k_gram_sum, so the sum's order
// is fixed.  sym (B = A, or A^T B symmetric by construction): only tiles i <=
// j are formed, and mirrored.
// Bound: the matrix cores, 2 V p (p + 16) / 2 flops when symmetric; a wider
// unit would spill, a narrower one reads more operand bytes per product.
// V = 20000, p = 200: 48 us and 6 for the sum of the chunks (18 TFLOP/s; 150 us
// on the vector ALUs with every entry formed), p = 100: 19 and 7.
// ---------------------------------------------------------------------------
constexpr int kGramN = 7, kGramWaves = 4;

struct GramShape {
  int pa, pb;
  bool sym;
  __host__ __device__ int na() const { return (pa + kTile - 1) / kTile; }
  __host__ __device__ int nb() const { return (pb + kTile - 1) / kTile; }
  // tiles of tile row i, and the units they are dealt out in
  __host__ __device__ int len(int i) const { return sym ? nb() - i : nb(); }
  __host__ __device__ int parts(int i) const { return (len(i) + kGramN - 1) / kGramN; }
  __host__ __device__ int units() const {
    int u = 0;
    for (int i = 0; i < na(); ++i) u += parts(i);
    return u;
  }
  __host__ __device__ int tiles() const { return sym ? nb() * (nb() + 1) / 2 : na() * nb(); }
  // number of the first tile of tile row i
  __host__ __device__ int tile0(int i) const { return sym ? i * nb() - i * (i - 1) / 2 : i * nb(); }
};

__global__ void __launch_bounds__(64 * kGramWaves) k_gram(const double* __restrict__ A,
                                                          const double* __restrict__ B,
                                                          const double* __restrict__ m, int V,
                                                          GramShape g, int chunk,
                                                          double* __restrict__ part,
                                                          const int* __restrict__ skip) {
  __shared__ double red[kGramWaves - 1][kGramN * kTileE];
  if (skip != nullptr && *skip) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int i = 0, u = blockIdx.x;   // unit u of the tile rows: j0 .. j0 + n - 1 of row i
  while (u >= g.parts(i)) u -= g.parts(i++);
  const int first = u * g.len(i) / g.parts(i);
  const int n = (u + 1) * g.len(i) / g.parts(i) - first;
  const int j0 = (g.sym ? i : 0) + first;
  const int v0 = blockIdx.y * chunk, v1 = min(V, v0 + chunk);
  const int row = lane >> 4, col = lane & 15;
  const int ca = min(i * kTile + col, g.pa - 1);
  doublex4 acc[kGramN];
#pragma unroll
  for (int q = 0; q < kGramN; ++q) acc[q] = doublex4{0.0, 0.0, 0.0, 0.0};
  // Operands of the next four rows are loaded while the current ones are
  // multiplied, all from clamped addresses: columns past the last only reach
  // entries that are not stored, and rows past the chunk are taken out by a
  // zero A operand when it is used (a select at the load would wait for it).
  double a, b[kGramN], mr = 0.0;
  bool in;
  auto load = [&](int v) {
    const int r = v + row;
    in = r < v1;
    const size_t rc = (size_t)min(r, V - 1);
    a = A[rc * g.pa + ca];
    if (m != nullptr) mr = m[rc];
#pragma unroll
    for (int q = 0; q < kGramN; ++q)
      b[q] = B[rc * g.pb + min((j0 + min(q, n - 1)) * kTile + col, g.pb - 1)];
  };
  int v = v0 + 4 * wave;
  if (v < v1) load(v);
  for (; v < v1; v += 4 * kGramWaves) {
    const double ac = in ? a : 0.0;
    double bc[kGramN];
#pragma unroll
    for (int q = 0; q < kGramN; ++q) bc[q] = b[q] - mr;
    if (v + 4 * kGramWaves < v1) load(v + 4 * kGramWaves);
#pragma unroll
    for (int q = 0; q < kGramN; ++q)
      if (q < n) acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(ac, bc[q], acc[q], 0, 0, 0);
  }
  if (wave > 0) {
#pragma unroll
    for (int q = 0; q < kGramN; ++q)
      if (q < n) store_tile(red[wave - 1] + q * kTileE, lane, acc[q]);
  }
  __syncthreads();
  if (wave == 0) {
    double* out = part + ((size_t)blockIdx.y * g.tiles() + g.tile0(i) + first) * kTileE;
#pragma unroll
    for (int q = 0; q < kGramN; ++q)
      if (q < n) {
        doublex4 s = acc[q];
#pragma unroll
        for (int w = 0; w < kGramWaves - 1; ++w) s += load_tile(red[w] + q * kTileE, lane);
        store_tile(out + q * kTileE, lane, s);
      }
  }
}

// G (pa x pb) from nz chunks of tiles: four lanes per entry, lane c adding the
// c-th quarter of the chunks in chunk order, the quarters combined as
// (q0 + q1) + (q2 + q3).  A lane issues the loads of 8 chunks before adding
// them; the last batch loads from chunk indexes clamped into its quarter and
// adds only the chunks that exist.  G32: an FP32 copy, or NULL.
__global__ void __launch_bounds__(256) k_gram_sum(const double* __restrict__ part, int nz,
                                                  GramShape g, double* __restrict__ G,
                                                  float* __restrict__ G32,
                                                  const int* __restrict__ skip) {
  constexpr int kU = 8;
  if (skip != nullptr && *skip) return;
  const int e = blockIdx.x * 64 + (threadIdx.x >> 2);   // 64 entries per block: within one tile
  const int c = threadIdx.x & 3;
  const int t = e / kTileE;
  const size_t stride = (size_t)g.tiles() * kTileE;
  const int per = (nz + 3) / 4;
  const int z0 = min(c * per, nz), z1 = min(z0 + per, nz);
  double s = 0.0;
  for (int z = z0; z < z1; z += kU) {
    double v[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) v[u] = part[(size_t)min(z + u, z1 - 1) * stride + e];
#pragma unroll
    for (int u = 0; u < kU; ++u)
      if (z + u < z1) s += v[u];
  }
  s += __shfl_xor(s, 1, 64);
  s += __shfl_xor(s, 2, 64);
  int i = 0;
  while (t >= g.tile0(i + 1)) ++i;
  const int j = (g.sym ? i : 0) + t - g.tile0(i);
  const int w = e % kTileE;
  const int gi = i * kTile + w / kTile, gj = j * kTile + w % kTile;
  if (c == 0 && gi < g.pa && gj < g.pb) {
    G[(size_t)gi * g.pb + gj] = s;
    if (G32 != nullptr) G32[(size_t)gi * g.pb + gj] = (float)s;
    if (g.sym && i != j) G[(size_t)gj * g.pb + gi] = s;
  }
}

// ---------------------------------------------------------------------------
// The largest eigenvalue of a symmetric positive semidefinite n x n matrix,
// n <= 128, by repeated squaring: B <- B^2 / tr(B^2) from G / tr(G) tends to
// the projector on the top eigenspace, and tr(G B) / tr(B) is the mean of the
// eigenvalues weighted by their 2^k-th powers.  After k squarings it is short
// of the largest by less than n / (2 e 2^k) relative whatever the gaps are
// (x e^(-2^(k+1) x), summed), so 40 bound it by 5e-11, far below the FP32 step
// size it is for; usually B is a projector (tr(B^2) = 1 to rounding) after 8
// to 15, and that ends it.  One block; the tiles stay in LDS, and as B is
// symmetric its tiles serve as both operands as they are stored.  Bound: the
// chain of squarings, 30 us at n = 50 (1030 us when a whole Jacobi iteration
// gave the one eigenvalue).
// Writes step = 1 / lambda (0 when there is no positive eigenvalue).
// ---------------------------------------------------------------------------
constexpr int kTopNb = 8, kTopWaves = 8;

template <int SLOTS>
__global__ void __launch_bounds__(64 * kTopWaves) k_top_eig(const double* __restrict__ G, int n,
                                                            float* __restrict__ step) {
  constexpr int NBM = SLOTS <= 2 ? 4 : kTopNb;
  __shared__ double B[NBM * NBM * kTileE];
  __shared__ double red[kTopWaves];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row = lane >> 4, col = lane & 15;
  const int nb = (n + kTile - 1) / kTile, nt = nb * (nb + 1) / 2;
  doublex4 g[SLOTS], v[SLOTS];
  int ti[SLOTS], tj[SLOTS];
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    const int t = wave + kTopWaves * s;
    ti[s] = tj[s] = -1;
    g[s] = doublex4{0.0, 0.0, 0.0, 0.0};
    if (t < nt) {
      int j = 0;
      while ((j + 1) * (j + 2) / 2 <= t) ++j;
      tj[s] = j;
      ti[s] = t - j * (j + 1) / 2;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int gi = ti[s] * kTile + 4 * r + row, gj = j * kTile + col;
        if (gi < n && gj < n) g[s][r] = G[(size_t)gi * n + gj];
      }
    }
    v[s] = g[s];
  }
  // sum over the block of f(slot), in wave order
  auto total = [&](auto f) {
    double x = 0.0;
#pragma unroll
    for (int s = 0; s < SLOTS; ++s)
      if (ti[s] >= 0) x += f(s);
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
    __syncthreads();
    if (lane == 0) red[wave] = x;
    __syncthreads();
    double all = 0.0;
#pragma unroll
    for (int w = 0; w < kTopWaves; ++w) all += red[w];
    return all;
  };
  auto trace_part = [&](int s) {
    double x = 0.0;
    if (ti[s] == tj[s]) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (4 * r + row == col) x += v[s][r];
    }
    return x;
  };
  double tr = total(trace_part);
  double mx = 0.0;
  if (tr > 0.0) {
    for (int k = 0; k < 40; ++k) {
      const double sc = 1.0 / tr;
#pragma unroll
      for (int s = 0; s < SLOTS; ++s)
        if (ti[s] >= 0) {
          v[s] *= sc;
          store_tile(B + (ti[s] * nb + tj[s]) * kTileE, lane, v[s]);
          if (ti[s] != tj[s]) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
              B[(tj[s] * nb + ti[s]) * kTileE + col * kTile + 4 * r + row] = v[s][r];
          }
        }
      __syncthreads();
#pragma unroll
      for (int s = 0; s < SLOTS; ++s)
        if (ti[s] >= 0) {
          v[s] = doublex4{0.0, 0.0, 0.0, 0.0};
          for (int m = 0; m < nb; ++m)
            v[s] = tile_mfma(load_tile(B + (m * nb + ti[s]) * kTileE, lane),
                             load_tile(B + (m * nb + tj[s]) * kTileE, lane), v[s]);
        }
      tr = total(trace_part);
      if (!(tr < 1.0 - 1e-14)) break;
    }
    mx = total([&](int s) {
      double x = 0.0;
#pragma unroll
      for (int r = 0; r < 4; ++r) x += g[s][r] * v[s][r];
      return ti[s] == tj[s] ? x : 2.0 * x;
    }) / tr;
  }
  if (threadIdx.x == 0) *step = mx > 0.0 ? (float)(1.0 / mx) : 0.0f;
}

}  // namespace

size_t chol_scratch_doubles(int p) {
  const size_t nb = (p + kTile - 1) / kTile;
  return (nb * (nb + 1) / 2 + nb) * kTileE;
}

// Binv (p x p; its part below the diagonal must hold zeros, which stay)
// becomes R^-1 of G + shift_rel max diag(G) I = R^T R; *info |= 1 on a pivot
// that is not positive.  scratch: chol_scratch_doubles(p).  nz > 0: G is the
// chunks of k_gram (nb <= 5).
static hipError_t launch_chol_inverse(const double* G, int p, double shift_rel, double* scratch,
                                      double* Binv, int* info, const int* skip, int* well, int nz,
                                      hipStream_t s) {
  const int nb = (p + kTile - 1) / kTile;
  if (p < 1 || nb > kMaxNb) return hipErrorInvalidValue;
  double* tiles = scratch;
  double* dinv = tiles + (size_t)nb * (nb + 1) / 2 * kTileE;
#define TLDA_CHOL(nw, slots, inv)                                                             \
  hipLaunchKernelGGL((k_chol<nw, slots, inv>), dim3(1), dim3(64 * nw), 0, s, G, p, shift_rel, \
                     tiles, dinv, Binv, info, skip, well, nz)
  // Up to p = 80 the block forms the inverse as well (its 15 tiles fit LDS beside
  // their inverse, and a launch costs 2 us and more where the columns' waves on
  // other compute units would save less); up to 144 and 208 the tiles fit in 6
  // and 12 slots of eight waves, past that they stay in memory, where every step
  // of the chain waits for it.
  if (nb <= 5) {
    TLDA_CHOL(4, 4, true);
    return hipGetLastError();
  }
  if (nb <= 9) TLDA_CHOL(8, 6, false);
  else if (nb <= 13) TLDA_CHOL(8, 12, false);
  else
    hipLaunchKernelGGL(k_chol_mem, dim3(1), dim3(1024), 0, s, G, p, shift_rel, tiles, dinv, info,
                       skip, well);
#undef TLDA_CHOL
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_tri_inverse, dim3(nb), dim3(64), 0, s, tiles, dinv, p, Binv, skip);
  return hipGetLastError();
}

// Row chunks of the Gram product: enough blocks for `blocks` in all, chunks of
// at least 64 rows.
static int gram_chunks(int V, const GramShape& g, int blocks) {
  const int want = blocks / g.units(), most = (V + 63) / 64;
  return want < 1 ? 1 : want < most ? want : most;
}
// Blocks of the tall products: four a CU (four waves per SIMD) for the refresh's,
// whose tile rows are several units; two for the one projection of an inference,
// whose chunks the sum reads again and whose scratch every context keeps.
constexpr int kGramBlocks = 1024, kProjectBlocks = 512;

// The chunks alone; their number to nz.
static hipError_t launch_gram_chunks(const double* A, const double* B, const double* m, int V,
                                     const GramShape& g, int blocks, double* part, int& nz,
                                     const int* skip, hipStream_t s) {
  nz = gram_chunks(V, g, blocks);
  const int step = 4 * kGramWaves;
  const int chunk = ((V + nz - 1) / nz + step - 1) / step * step;
  nz = (V + chunk - 1) / chunk;
  hipLaunchKernelGGL(k_gram, dim3(g.units(), nz), dim3(64 * kGramWaves), 0, s, A, B, m, V, g, chunk,
                     part, skip);
  return hipGetLastError();
}

static hipError_t launch_gram_sum(const double* part, int nz, const GramShape& g, double* G,
                                  float* G32, const int* skip, hipStream_t s) {
  hipLaunchKernelGGL(k_gram_sum, dim3(g.tiles() * (kTileE / 64)), dim3(256), 0, s, part, nz, g, G,
                     G32, skip);
  return hipGetLastError();
}

size_t gram_scratch_doubles(int V, int p, bool sym) {
  const GramShape g{p, p, sym};
  return (size_t)gram_chunks(V, g, kGramBlocks) * g.tiles() * kTileE;
}
hipError_t launch_gram(const double* A, const double* B, double* G, int V, int p, bool sym,
                       double* part, hipStream_t s) {
  const GramShape g{p, p, sym};
  int nz = 0;
  const hipError_t e = launch_gram_chunks(A, B, nullptr, V, g, kGramBlocks, part, nz, nullptr, s);
  return e != hipSuccess ? e : launch_gram_sum(part, nz, g, G, nullptr, nullptr, s);
}

hipError_t launch_gram_chol(const double* A, double* G, int V, int p, double* part,
                            double shift_rel, double* scratch, double* Binv, int* info,
                            const int* skip, int* well, hipStream_t s) {
  const GramShape g{p, p, true};
  int nz = 0;
  hipError_t e = launch_gram_chunks(A, A, nullptr, V, g, kGramBlocks, part, nz, skip, s);
  if (e != hipSuccess) return e;
  // up to 16 chunks (V <= 1024) of at most 15 tiles the factorisation adds itself
  if (nz <= 16 && g.nb() <= 5)
    return launch_chol_inverse(part, p, shift_rel, scratch, Binv, info, skip, well, nz, s);
  e = launch_gram_sum(part, nz, g, G, nullptr, skip, s);
  if (e != hipSuccess) return e;
  return launch_chol_inverse(G, p, shift_rel, scratch, Binv, info, skip, well, 0, s);
}

size_t project_scratch_doubles(int V, int D, int K) {
  const GramShape g{D, K, false};
  return (size_t)gram_chunks(V, g, kProjectBlocks) * g.tiles() * kTileE;
}
hipError_t launch_project(const double* W, const double* m, const double* mu, int V, int D, int K,
                          double* part, double* A, float* A32, hipStream_t s) {
  const GramShape g{D, K, false};
  int nz = 0;
  const hipError_t e = launch_gram_chunks(W, mu, m, V, g, kProjectBlocks, part, nz, nullptr, s);
  return e != hipSuccess ? e : launch_gram_sum(part, nz, g, A, A32, nullptr, s);
}

hipError_t launch_top_eig(const double* G, int n, float* step, hipStream_t s) {
  if (n < 1 || n > kTile * kTopNb) return hipErrorInvalidValue;
  if (n <= 64) hipLaunchKernelGGL(k_top_eig<2>, dim3(1), dim3(64 * kTopWaves), 0, s, G, n, step);
  else hipLaunchKernelGGL(k_top_eig<5>, dim3(1), dim3(64 * kTopWaves), 0, s, G, n, step);
  return hipGetLastError();
}

}  // namespace tlda
