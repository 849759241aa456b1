// CP-gradient data term on the classic alpha0-corrected moments (the
// appendix's cumulants, run through the batched SGD of section "Online
// Learning of the Third Moment").  Per kept document with counts c, length L,
// l2 = 1/(L(L-1)), l3 = l2/(L-2), the piece of M3 contracted with
// (W, phi_k, phi_k) is, with y = W^T c, z_w = Phi^T W_w (row w of Z = W Phi),
// s = sum_w c_w z_w, q = sum_w c_w z_w^2, r = Phi^T (W^T M1):
//   c3 l3 (y s^2 - 2 s g - y q + 2 h) - c2 l2 (2 r (y s - g) + m_w (s^2 - q))
//   + alpha0^2 m_w r^2,        g = sum_w c_w W_w z_w,  h = sum_w c_w W_w z_w^2,
// column k taking the k-th entries of s, q, r, z (c2 = alpha0(alpha0+1)/2,
// c3 = (alpha0+1)(alpha0+2)/2, m_w = W^T M1).  Grouped by what multiplies W
// rows (y_d = sum_w c_w W_w), the batch sum divided by c3 is one reduction
// with a row per nonzero (d, w),
//   sum over nonzeros (d, w):  W_w  (x)  c_w (a_d + b_d * z_w + g_d z_w^2)
//   plus m_w (x) sum_d e_d,
// with a = l3 (s^2 - q) - 2 (c2/c3) l2 r s, b = -2 l3 s + 2 (c2/c3) l2 r,
// g_d = 2 l3 and e = -(c2/c3) l2 (s^2 - q) + (alpha0^2/c3) r^2 (zero for
// dropped documents).
//
// k_classic_z forms Z (FP32, V x Kp) and r once per step.  k_classic_cp gathers
// the Z rows of a document's words for s, q and the coefficients, turns them
// into reduction rows, and accumulates the D x K outer products with the W rows
// on FP32 matrix cores.  Each block writes its partial sum and its
// kept-document count; the shared finish kernel adds them in block order, forms the
// gradient with the penalty term and updates Phi.
#include "tlda_internal.h"

#include <type_traits>

namespace tlda {
namespace {

constexpr int kThreads = 256;
constexpr int kRing = 48;     // reduction rows that a wave keeps in LDS: 15 and 32 more, in batches
constexpr int kRing16 = 52;   // BF16: rows from one column of them to the next
constexpr int classic_ring_bytes(bool bf16) { return bf16 ? 64 * kRing16 * 2 : 64 * kRing * 4; }
// Waves per block (one block per CU): three per SIMD where a wave's sums (4 NDT
// NCT registers) and W rows (4 NDT, and as many on the way) leave 168 for all,
// else two (256).
constexpr int classic_waves(int ndt, int nct) { return ndt * (nct + 1) <= 20 ? 12 : 8; }
// What a document costs besides its nonzeros, in nonzeros: less where each of
// these is many products (131072 documents of 0 to 40 words in order of length:
// FP32 at D = K = 50 340 us with 4 and 358 with 8, BF16 246 and 220, FP32 at
// D = K = 5 216 and 177).
constexpr int classic_doc_cost(int ndt, int nct, bool bf16) {
  return bf16 || ndt * nct < 4 ? 8 : 4;
}
// Runs are cut by work, not by documents, from this many nonzeros a run on and
// where a run has more than one document.  Documents in order of length, as
// bucketed corpora have them, leave the last waves twice the mean otherwise
// (131072 documents of 0 to 40 words, D = K = 50: 564 us by documents, 340 by
// work; shuffled 337 and 309).  Finding the boundaries takes 2 to 3 us, which
// smaller batches do not get back: 16000 documents of 8 words at D = K = 20 take
// 29.9 us by work and 27.9 by documents, of 20 words 42.2 and 46.5; and with a
// document a run (2000 of 300 words) the cut by work gives some waves two, 137
// against 108.
constexpr int kWorkPerRun = 96;
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef short bf16x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf_to_f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
// FP32 -> BF16 bits, round to nearest even (hardware conversion).
__device__ __forceinline__ uint16_t f_to_bf(float f) {
  const __bf16 h = (__bf16)f;
  return __builtin_bit_cast(uint16_t, h);
}

// Elements of W and Z, the same as a register holds them, and their value.
template <bool BF>
using classic_elem = std::conditional_t<BF, uint16_t, float>;
template <bool BF>
using classic_elem_bits = std::conditional_t<BF, uint32_t, float>;
template <bool BF>
__device__ __forceinline__ float classic_value(classic_elem_bits<BF> x) {
  if constexpr (BF)
    return __uint_as_float(x << 16);
  else
    return x;
}

// The lanes of a wave exchange data through LDS: what was written before is
// visible to the others after it (a wave's LDS operations complete in order,
// so this only holds the compiler's order).
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Where the run boundaries `first` and `last` of `runs` fall, for runs of equal
// work: a document costs its nonzeros and kDocCost nonzeros more.  Boundary r is the first
// document with at least r / runs of all work before it, so neighbouring runs
// agree on it and the boundaries depend on the batch alone.  The wave asks 64
// places at a time: three rounds of loads up to 2^18 documents.
template <int kDocCost>
__device__ __forceinline__ void run_bounds(const int32_t* __restrict__ row_ptr, int n, int first,
                                           int last, int runs, int lane, int& d0, int& d1) {
  const int base = row_ptr[0];
  const long long total = row_ptr[n] - base + (long long)kDocCost * n;
  const long long t[2] = {total * first / runs, total * last / runs};
  int lo[2] = {0, 0}, hi[2] = {n, n};   // the boundary is in lo .. hi
  while (lo[0] < hi[0] || lo[1] < hi[1]) {
    int p[2], v[2], step[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      step[i] = (int)(((long long)hi[i] - lo[i] + 63) / 64);
      p[i] = (int)min((long long)lo[i] + (long long)lane * step[i], (long long)hi[i]);
      v[i] = row_ptr[p[i]];
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const unsigned long long at =
          __ballot((long long)(v[i] - base) + (long long)kDocCost * p[i] >= t[i]);
      const int k = at != 0 ? __builtin_ctzll(at) : 64;   // the first place past the boundary
      const long long l = lo[i], h = hi[i], s = step[i];
      if (k < 64) hi[i] = (int)min(h, l + k * s);
      if (k > 0) lo[i] = (int)min((long long)hi[i], l + (k - 1) * s + 1);
    }
  }
  d0 = lo[0];
  d1 = lo[1];
}

// Z[w][k] = sum_d W32[w][d] Phi[d][k] (zero for K <= k < Kp); block 0 also
// writes r[k] = sum_d mw32[d] Phi[d][k] and the copy of Phi that the finish
// kernel reads while it overwrites Phi.  Phi is staged in LDS (D*K <= 16384).
__global__ void __launch_bounds__(kThreads) k_classic_z(const float* __restrict__ W32, int V,
                                                        int D, int Dp,
                                                        const float* __restrict__ Phi, int K,
                                                        int Kp, const float* __restrict__ mw32,
                                                        float* __restrict__ Z,
                                                        float* __restrict__ r,
                                                        float* __restrict__ phi_copy) {
  extern __shared__ float ph[];
  const int tid = threadIdx.x;
  for (int e = tid; e < D * K; e += kThreads) ph[e] = Phi[e];
  __syncthreads();
  if (blockIdx.x == 0) {
    for (int e = tid; e < D * K; e += kThreads) phi_copy[e] = ph[e];
    for (int k = tid; k < Kp; k += kThreads) {
      float s = 0.f;
      if (k < K)
        for (int d = 0; d < D; ++d) s = fmaf(mw32[d], ph[d * K + k], s);
      r[k] = s;
    }
  }
  const size_t n = (size_t)V * Kp;
  for (size_t e = (size_t)blockIdx.x * kThreads + tid; e < n; e += (size_t)gridDim.x * kThreads) {
    const int w = (int)(e / Kp), k = (int)(e % Kp);
    float s = 0.f;
    if (k < K) {
      const float* wr = W32 + (size_t)w * Dp;
      for (int d = 0; d < D; ++d) s = fmaf(wr[d], ph[d * K + k], s);
    }
    Z[e] = s;
  }
}

// A wave works alone on a run of consecutive documents (by_work: runs of equal
// work, else of equal documents); no wave waits for another before the block's
// sums are added at the end.  For each document
//   phase 1: lane k takes column k.  The Z rows of the document's words, 32 at
//     a time, come straight into registers and give s, q, L and the
//     coefficients a, b, g;
//   the reduction rows c (a + b z + g z^2), rounded to BF16 where W is, are
//     formed from the same registers and put into the wave's ring of kRing rows
//     in LDS (documents of more than 32 words gather their Z rows a second time
//     for it);
//   the Z rows of the next document are asked for, and
//   phase 2: as long as the ring holds 16 rows they go through the matrix
//     cores, four at a time: B from the ring, A (the W rows) straight from
//     memory into the operand registers, 16 rows ahead of their use (BF16: all
//     16 at once).  The rows of a run are consecutive nonzeros, so this side
//     needs no document.
// Each wave keeps all NDT x NCT tiles of the D x K sum.  K > 64 is split over
// gridDim.y: the columns do not depend on each other.
//
// What bounds it: issue slots and the latency of the gathers.  131072 documents
// of 20 words at D = K = 50, V = 20000 (2.52 million nonzeros, 1.35 GB through
// L2) take 265 us among other steps (288 in a kernel trace, where each launch
// waits): the matrix cores are busy for 140 of them, the vector ALU for about 75
// (per nonzero row two offsets, two readlanes, four operations for L, s and q,
// three for the reduction row).  Tiles of 16 documents per block of
// four waves, with Z gathered twice, staged in LDS and a barrier per 16 rows,
// took 475 us.  Z rows kept in LDS between the phases took 350 us: 20 KB a wave
// leave two waves per SIMD, where a ring of 12 KB leaves three.  A 64-bit
// multiply for each row's address costs 8 us, scalar multiplies 25 us.  The W
// rows of a batch are asked for while the batch before is multiplied; holding
// its products back until all of them are asked for costs 7 us.  The wait at
// the top of the loop, where nothing is in flight that was not asked for before
// the last products, lets the next products start without waiting for the Z
// rows that are asked for just ahead of them: 40 us less.
// BF16 (contexts created with TLDA_CLASSIC | TLDA_BF16): the copy W16 of W (with
// its mean projection mw16), Z16 = bf16(W16 Phi), sums and coefficients in FP32.
// It takes 150 us, with an eighth of the matrix cores' time and half the bytes;
// staged column by column in blocks of four waves it took 330.
//
// (V <= 131072: words take 24 bits, and 32 reach all of W and Z.)
template <int NDT, int NCT, bool BF>
__global__ void __launch_bounds__(64 * classic_waves(NDT, NCT)) k_classic_cp(
    const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
    const float* __restrict__ val, int n_rows, const classic_elem<BF>* __restrict__ W, int Dp,
    const classic_elem<BF>* __restrict__ Z, int Kp, const float* __restrict__ mw,
    const float* __restrict__ r_g, int D, int K, float c2r, float a0r, int by_work,
    float* __restrict__ partial, int* __restrict__ block_counts) {
  using E = classic_elem<BF>;
  constexpr int NW = classic_waves(NDT, NCT);
  constexpr int NB = 16;    // rows per batch
  constexpr int kSums = NW * 8 * 1024;   // the block's sum at the end: eight tiles at a time
  constexpr int kRings = NW * classic_ring_bytes(BF);
  __shared__ __attribute__((aligned(16))) char ring_lds[kRings > kSums ? kRings : kSums];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, l4 = lane >> 4;
  const int k0 = blockIdx.y * 64;
  char* ring = ring_lds + wave * classic_ring_bytes(BF);
  // columns past Kp repeat the last one (they reach no output)
  const int kc = k0 + lane < Kp ? k0 + lane : Kp - 1;
  const unsigned zoff = (unsigned)(sizeof(E) * kc);
  const char* Zb = reinterpret_cast<const char*>(Z);
  const float rk = r_g[kc];
  const char* Wb = reinterpret_cast<const char*>(W);
  const unsigned woff = (unsigned)(sizeof(E) * (l16 < Dp ? l16 : Dp - 1));
  const unsigned wstride = (unsigned)(sizeof(E) * Dp), zstride = (unsigned)(sizeof(E) * Kp);

  floatx4 acc[NDT][NCT];
#pragma unroll
  for (int i = 0; i < NDT; ++i)
#pragma unroll
    for (int j = 0; j < NCT; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  float es = 0.f;
  int kept = 0;

  const int run = blockIdx.x * NW + wave, runs = gridDim.x * NW;
  int d0 = (int)((long long)n_rows * run / runs);
  int d1 = (int)((long long)n_rows * (run + 1) / runs);
  if (by_work)
    run_bounds<classic_doc_cost(NDT, NCT, BF)>(row_ptr, n_rows, run, run + 1, runs, lane, d0, d1);
  const int nz0 = __builtin_amdgcn_readfirstlane(row_ptr[d0]);
  const int nz1 = __builtin_amdgcn_readfirstlane(row_ptr[d1]);

  // ---- A side: the W rows of the next batch, the words of the one after it.
  // Four rows are one FP32 operand or, packed, four of a BF16 operand's
  // sixteen.  (The bits are kept as they come: a conversion next to a load
  // would wait for it.)
  classic_elem_bits<BF> an[4][NDT];
  int ac = 0;                 // the word of row lane % NB
  int anext = nz0 + lane % NB;
  auto load_cols = [&]() {
    ac = col_idx[anext < nz1 ? anext : nz1 - 1];
    anext += NB;
  };
  auto load_a = [&]() {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const unsigned c = (unsigned)__shfl(ac, BF ? 4 * l4 + i : 4 * i + l4, 64);
      unsigned o = __umul24(c, wstride) + woff;
      asm("" : "+v"(o));
      const E* w = reinterpret_cast<const E*>(Wb + o);
#pragma unroll
      for (int t = 0; t < NDT; ++t) an[i][t] = w[16 * t];
    }
  };
  int head = 0;     // the ring's first row not yet multiplied, a multiple of NB
  int fill = 0;     // rows from there on
  // FP32: rows of 64 columns; BF16: columns of kRing rows, two words further
  // apart (a lane's operand is four rows of a column)
  auto place = [&](int r) -> char* {
    r = r >= kRing ? r - kRing : r;
    return BF ? ring + (lane * kRing16 + r) * 2 : ring + r * 256 + 4 * lane;
  };
  auto put = [&](int r, float x) {
    if constexpr (BF)
      *reinterpret_cast<uint16_t*>(place(r)) = f_to_bf(x);
    else
      *reinterpret_cast<float*>(place(r)) = x;
  };
  auto multiply = [&]() {   // a batch
    if constexpr (BF) {
      uint2 a[NDT];
#pragma unroll
      for (int t = 0; t < NDT; ++t)
        a[t] = make_uint2(an[0][t] | an[1][t] << 16, an[2][t] | an[3][t] << 16);
      load_a();
      load_cols();
#pragma unroll
      for (int c = 0; c < NCT; ++c) {
        const bf16x4_t bb = *reinterpret_cast<const bf16x4_t*>(
            ring + ((16 * c + l16) * kRing16 + head + 4 * l4) * 2);
#pragma unroll
        for (int t = 0; t < NDT; ++t)
          acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
              __builtin_bit_cast(bf16x4_t, a[t]), bb, acc[t][c], 0, 0, 0);
      }
    } else {
      float a[4][NDT];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int t = 0; t < NDT; ++t) a[i][t] = an[i][t];
      load_a();
      load_cols();
      const char* rows = ring + head * 256 + l4 * 256 + 4 * l16;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float bb[NCT];
#pragma unroll
        for (int c = 0; c < NCT; ++c)
          bb[c] = *reinterpret_cast<const float*>(rows + 1024 * i + 64 * c);
#pragma unroll
        for (int t = 0; t < NDT; ++t)
#pragma unroll
          for (int c = 0; c < NCT; ++c)
            acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][t], bb[c], acc[t][c], 0, 0, 0);
      }
    }
    fill -= NB;
    head = head + NB == kRing ? 0 : head + NB;
  };

  // ---- B side: segments of at most 32 entries of one document ----
  int rp = 0;               // row_ptr[dbase + lane]
  int dbase = d0;
  auto load_rp = [&](int d) {
    dbase = d;
    rp = row_ptr[d + lane < d1 ? d + lane : d1];
  };
  // a segment: the document, its first entry and entries, the segment's first
  // entry; documents of more than 32 entries are passed over twice
  struct Seg {
    int d, b, n, j, pass;
    __device__ int count() const { return n - j < 32 ? n - j : 32; }
    __device__ bool last() const { return j + 32 >= n; }
    __device__ bool puts() const { return n <= 32 || pass == 1; }
  };
  auto next = [&](const Seg& x) {
    Seg y = x;
    y.j = x.j + 32;
    if (x.last()) {
      y.j = 0;
      y.pass = 1;
      if (x.puts()) {
        y.pass = 0;
        y.d = x.d + 1;
        y.n = 0;
        if (y.d < d1) {
          if (y.d + 1 - dbase > 63) load_rp(y.d);
          y.b = __builtin_amdgcn_readlane(rp, y.d - dbase);
          y.n = __builtin_amdgcn_readlane(rp, y.d + 1 - dbase) - y.b;
        }
      }
    }
    return y;
  };
  // word and count of entry `lane`
  auto load_entries = [&](const Seg& x, int& c, float& v) {
    const int count = x.count();
    c = 0;
    v = 0.f;
    if (count > 0) {
      c = col_idx[x.b + x.j + (lane < count ? lane : count - 1)];
      if (lane < count) v = val[x.b + x.j + lane];
    }
  };
  // the offsets of this segment's Z rows, the words of the next one and the one after
  int c0 = 0, c1 = 0, c2 = 0;
  float v0 = 0.f, v1 = 0.f, v2 = 0.f;
  // the Z rows at offsets c0, four at a time (those that fill the last four have
  // no count)
  classic_elem_bits<BF> z[32];
  auto load_z = [&](int count) {
#pragma unroll
    for (int c = 0; c < 8; ++c)
      if (4 * c < count) {
#pragma unroll
        for (int t = 4 * c; t < 4 * c + 4; ++t) {
          unsigned o = (unsigned)__builtin_amdgcn_readlane(c0, t) + zoff;
          asm("" : "+v"(o));   // the base stays in scalar registers
          z[t] = *reinterpret_cast<const E*>(Zb + o);
        }
      }
  };
  Seg s0{d0, nz0, 0, 0, 0}, s1, s2;
  if (nz1 > nz0) {
    load_cols();
    load_a();
    load_cols();
  }
  if (d0 < d1) {
    load_rp(d0);
    s0.n = __builtin_amdgcn_readlane(rp, 1) - nz0;
  }
  load_entries(s0, c0, v0);
  s1 = next(s0);
  load_entries(s1, c2, v2);
  c0 = (int)__umul24((unsigned)c0, zstride);
  load_z(s0.count());
  float s = 0.f, q = 0.f, L = 0.f, al = 0.f, be = 0.f, g = 0.f;
  while (s0.d < d1 || fill > 0) {
    // everything asked for has arrived: the Z rows were asked for before the
    // products below, the W rows at their start, the entries before that
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    c1 = c2;
    v1 = v2;
    s2 = next(s1);
    load_entries(s2, c2, v2);
    const int cnt = s0.count();
    if (s0.pass == 0 && s0.d < d1) {
      if (s0.j == 0) s = q = L = 0.f;
#pragma unroll
      for (int c = 0; c < 8; ++c)
        if (4 * c < cnt) {
#pragma unroll
          for (int t = 4 * c; t < 4 * c + 4; ++t) {
            const float v = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v0), t));
            const float zt = classic_value<BF>(z[t]);
            L += v;
            s = fmaf(v, zt, s);
            q = fmaf(v * zt, zt, q);
          }
        }
      if (s0.last()) {
        const bool keep = L >= 3.f;   // L is the same on every lane
        const float l2 = keep ? 1.0f / (L * (L - 1.0f)) : 0.f;
        const float l3 = keep ? l2 / (L - 2.0f) : 0.f;
        const float d2 = s * s - q;
        al = l3 * d2 - 2.0f * c2r * l2 * rk * s;
        be = -2.0f * l3 * s + 2.0f * c2r * l2 * rk;
        g = 2.0f * l3;
        if (keep) es += -c2r * l2 * d2 + a0r * rk * rk;
        kept += __builtin_amdgcn_readfirstlane(keep ? 1 : 0);
      }
    }
    if (s0.puts()) {
      const int at = head + fill;
#pragma unroll
      for (int c = 0; c < 8; ++c)
        if (4 * c < cnt) {
#pragma unroll
          for (int t = 4 * c; t < 4 * c + 4; ++t) {
            const float v = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v0), t));
            const float zt = classic_value<BF>(z[t]);
            put(at + t, v * fmaf(g * zt + be, zt, al));
          }
        }
      fill += cnt;
    }
    if (s0.d >= d1) {
      // the run's last rows: zeros up to a whole batch (no wrap: head is a
      // multiple of NB)
      for (int r = fill; r < NB; ++r) put(head + r, 0.f);
      fill = NB;
    }
    s0 = s1;
    s1 = s2;
    c0 = (int)__umul24((unsigned)c1, zstride);
    v0 = v1;
    load_z(s0.count());
    wave_fence();
    // ---- phase 2: the whole batches, two at most (kRing = 48) ----
    if (fill >= NB) {
      multiply();
      if (fill >= NB) multiply();
    }
    wave_fence();
  }

  // ---- the block's sum in wave order, m_w (x) sum e, and the kept count ----
  constexpr int RD = 8;                       // tiles per round
  __shared__ float esum[64];
  __shared__ int wave_kept[NW];
  float* lds = reinterpret_cast<float*>(ring_lds);
  __syncthreads();
  lds[tid] = es;
  if (lane == 0) wave_kept[wave] = kept;
  __syncthreads();
  if (tid < 64) {
    float x = 0.f;
    for (int w = 0; w < NW; ++w) x += lds[w * 64 + tid];
    esum[tid] = x;
  }
  float* out = partial + (size_t)blockIdx.x * D * K;
#pragma unroll
  for (int q0 = 0; q0 < NDT * NCT; q0 += RD) {
    __syncthreads();
#pragma unroll
    for (int t = q0; t < q0 + RD; ++t)
      if (t < NDT * NCT)
        *reinterpret_cast<floatx4*>(lds + ((wave * RD + t - q0) * 64 + lane) * 4) =
            acc[t / NCT][t % NCT];
    __syncthreads();
    for (int e = tid; e < RD * 256; e += 64 * NW) {
      const int t = q0 + e / 256, ln = (e >> 2) & 63;
      const int k = (t % NCT) * 16 + (ln & 15), dd = (t / NCT) * 16 + 4 * (ln >> 4) + (e & 3);
      if (t < NDT * NCT && dd < D && k0 + k < K) {
        float x = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) x += lds[w * RD * 256 + e];
        out[dd * K + k0 + k] = fmaf(mw[dd], esum[k], x);
      }
    }
  }
  if (tid == 0 && blockIdx.y == 0) {
    int x = 0;
    for (int w = 0; w < NW; ++w) x += wave_kept[w];
    block_counts[blockIdx.x] = x;
  }
}

// Z16[w][k] = bf16(sum_d W16[w][d] Phi[d][k]) (zero for K <= k < Kh); block 0
// also writes r[k] = sum_d mw16[d] Phi[d][k] and the copy of Phi.
__global__ void __launch_bounds__(kThreads) k_classic_z16(const uint16_t* __restrict__ W16, int V,
                                                          int D, int Dh,
                                                          const float* __restrict__ Phi, int K,
                                                          int Kh, const float* __restrict__ mw16,
                                                          uint16_t* __restrict__ Z16,
                                                          float* __restrict__ r,
                                                          float* __restrict__ phi_copy) {
  extern __shared__ float ph[];
  const int tid = threadIdx.x;
  for (int e = tid; e < D * K; e += kThreads) ph[e] = Phi[e];
  __syncthreads();
  if (blockIdx.x == 0) {
    for (int e = tid; e < D * K; e += kThreads) phi_copy[e] = ph[e];
    for (int k = tid; k < Kh; k += kThreads) {
      float s = 0.f;
      if (k < K)
        for (int d = 0; d < D; ++d) s = fmaf(mw16[d], ph[d * K + k], s);
      r[k] = s;
    }
  }
  const size_t n = (size_t)V * Kh;
  for (size_t e = (size_t)blockIdx.x * kThreads + tid; e < n; e += (size_t)gridDim.x * kThreads) {
    const int w = (int)(e / Kh), k = (int)(e % Kh);
    float s = 0.f;
    if (k < K) {
      const uint16_t* wr = W16 + (size_t)w * Dh;
      for (int d = 0; d < D; ++d) s = fmaf(bf_to_f(wr[d]), ph[d * K + k], s);
    }
    Z16[e] = f_to_bf(s);
  }
}

template <int NDT, int NCT, bool BF>
hipError_t launch_classic_t(const tlda_csr_batch& b, const classic_elem<BF>* W, int Dp,
                            const classic_elem<BF>* Z, int Kp, const float* mw, const float* r,
                            int D, int K, double alpha0, int nblk, float* partial,
                            int* block_counts, hipStream_t s) {
  constexpr int NW = classic_waves(NDT, NCT);
  const long long runs = (long long)nblk * NW;
  const int by_work = b.n_rows > runs && b.nnz >= kWorkPerRun * runs;
  const double c2 = alpha0 * (alpha0 + 1.0) / 2.0;
  const double c3 = (alpha0 + 1.0) * (alpha0 + 2.0) / 2.0;
  launch_main(k_classic_cp<NDT, NCT, BF>, dim3(nblk, K > 64 ? 2 : 1), dim3(64 * NW), 0, s,
              b.row_ptr, b.col_idx, b.val, b.n_rows, W, Dp, Z, Kp, mw, r, D, K, (float)(c2 / c3),
              (float)(alpha0 * alpha0 / c3), by_work, partial, block_counts);
  return hipGetLastError();
}

template <bool BF>
hipError_t launch_classic(const tlda_csr_batch& b, const classic_elem<BF>* W, int Dp,
                          const classic_elem<BF>* Z, int Kp, const float* mw, const float* r, int D,
                          int K, double alpha0, int nblk, float* partial, int* block_counts,
                          hipStream_t s) {
  const int ndt = (D + 15) / 16, nct = K > 64 ? 4 : (K + 15) / 16;
#define TLDA_CLASSIC(NDT_, NCT_)                                                              \
  if (ndt == NDT_ && nct == NCT_)                                                             \
    return launch_classic_t<NDT_, NCT_, BF>(b, W, Dp, Z, Kp, mw, r, D, K, alpha0, nblk,       \
                                            partial, block_counts, s);
#define TLDA_CLASSIC_ROW(NDT_) \
  TLDA_CLASSIC(NDT_, 1) TLDA_CLASSIC(NDT_, 2) TLDA_CLASSIC(NDT_, 3) TLDA_CLASSIC(NDT_, 4)
  TLDA_CLASSIC_ROW(1) TLDA_CLASSIC_ROW(2) TLDA_CLASSIC_ROW(3) TLDA_CLASSIC_ROW(4)
  TLDA_CLASSIC_ROW(5) TLDA_CLASSIC_ROW(6) TLDA_CLASSIC_ROW(7) TLDA_CLASSIC_ROW(8)
#undef TLDA_CLASSIC_ROW
#undef TLDA_CLASSIC
  return hipErrorInvalidValue;
}

}  // namespace

bool classic_supported(int D, int K) { return D >= 1 && D <= 128 && K >= 1 && K <= 128; }

hipError_t launch_classic_z(const float* W32, int V, int D, int Dp, const float* Phi, int K,
                            int Kp, const float* mw32, float* Z, float* r, float* phi_copy,
                            int num_cu, hipStream_t s) {
  const size_t n = (size_t)V * Kp;
  size_t grid = (n + kThreads - 1) / kThreads;
  if (grid > (size_t)num_cu * 8) grid = (size_t)num_cu * 8;
  if (grid < 1) grid = 1;
  hipLaunchKernelGGL(k_classic_z, dim3((unsigned)grid), dim3(kThreads),
                     (unsigned)(sizeof(float) * D * K), s, W32, V, D, Dp, Phi, K, Kp, mw32, Z, r,
                     phi_copy);
  return hipGetLastError();
}

hipError_t launch_classic_z16(const uint16_t* W16, int V, int D, int Dh, const float* Phi, int K,
                              int Kh, const float* mw16, uint16_t* Z16, float* r, float* phi_copy,
                              int num_cu, hipStream_t s) {
  const size_t n = (size_t)V * Kh;
  size_t grid = (n + kThreads - 1) / kThreads;
  if (grid > (size_t)num_cu * 8) grid = (size_t)num_cu * 8;
  if (grid < 1) grid = 1;
  hipLaunchKernelGGL(k_classic_z16, dim3((unsigned)grid), dim3(kThreads),
                     (unsigned)(sizeof(float) * D * K), s, W16, V, D, Dh, Phi, K, Kh, mw16, Z16,
                     r, phi_copy);
  return hipGetLastError();
}

hipError_t launch_classic_cp16(const tlda_csr_batch& b, const uint16_t* W16, int Dh,
                               const uint16_t* Z16, int Kh, const float* mw16, const float* r,
                               int D, int K, double alpha0, int nblk, float* partial,
                               int* block_counts, hipStream_t s) {
  return launch_classic<true>(b, W16, Dh, Z16, Kh, mw16, r, D, K, alpha0, nblk, partial,
                              block_counts, s);
}

int classic_blocks(int D, int K, int n_rows, int num_cu) {
  const int nw = classic_waves((D + 15) / 16, K > 64 ? 4 : (K + 15) / 16);
  const int room = K > 64 ? (num_cu + 1) / 2 : num_cu;
  const int want = (n_rows - 1) / nw + 1;
  return want < room ? want : room;
}

hipError_t launch_classic_cp(const tlda_csr_batch& b, const float* W32, int Dp, const float* Z,
                             int Kp, const float* mw32, const float* r, int D, int K,
                             double alpha0, int nblk, float* partial, int* block_counts,
                             hipStream_t s) {
  return launch_classic<false>(b, W32, Dp, Z, Kp, mw32, r, D, K, alpha0, nblk, partial,
                               block_counts, s);
}

}  // namespace tlda
