// qops.hpp -- matrix-free Q products: Kronecker (FP64 MFMA) and diag + low rank.
#pragma once
#include "common.hpp"

typedef double hq_dx4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// FP64 MFMA GEMM of the Kronecker operators, up to three terms in one
// accumulator:
//   D (M x N) = sum_t +-A_t (M x K_t, col-major, lda) op_t(B_t),
//   op(B)[k][j] = B[k + ldb j], or B[j + ldb k] when transposed.
// Output element (i, j) goes to the epilogue as vector index i + ldo j.
//
// A block owns a 16 WM x 16 WN tile of D, and each of its NW waves computes the
// whole tile over its share of K, so that an operand element is loaded once per
// block, straight into the registers of the MFMA (v_mfma_f64_16x16x4f64) that
// uses it: no LDS staging and no barrier in the loop.  (Staging the slices in
// LDS was bound by its bandwidth: 1 KB of fragment reads per 64-clock MFMA and
// wave at a 16 x 16 part, 2 x 2 waves, against 0.5 KB here at 32 x 32.)  K runs in
// blocks of 16: lane l takes k = 4 (l/16) + s at step s = 0..3, so that the four
// loads of an untransposed B use up its 128-byte lines; the loads run HQ_GRING
// blocks ahead in a ring of registers (the loop is unrolled by the ring, so
// every index is static).  The waves' tiles are added through LDS in wave order
// and the epilogue runs over the sums, consecutive threads on consecutive rows.
// Operand layout of the MFMA (measured on gfx950): lane l supplies A[l%16][l/16]
// and B[l/16][l%16]; accumulator register v of lane l holds D[l/16 + 4v][l%16].
// It is fed op(B)^T and A^T, so lane l holds rows l%16 of D.
// Split-K (PART): the K blocks of all terms are divided among `kgroups` groups
// (grid = tiles x kgroups); group g writes its partial tile to
// parts + g * M * N and k_gemm_sum adds the groups in order and runs the
// epilogue.  Deterministic either way.
// ---------------------------------------------------------------------------
#define HQ_GRING 2   // K blocks in flight
#define HQ_GBAND 4   // tile rows of a band
struct GemmOps {
  const double* A[3];
  const double* B[3];
  int lda[3], ldb[3], K[3], transb[3];
  int neg[3];   // 1: the term is subtracted
  int nt;
};
// Where op(B)(k, j) of a tile is, in bytes: a 64-bit base, uniform over the block, at
// the tile's first column j0, and a 32-bit offset of the lane for column j0 + j, j < 32,
// and k < 16.  The offset alone reaches 8 (31 ldb + 15), below 2^32 for a leading
// dimension of up to 17 million (a factor of that order would take 2,000 TB);
// with the columns from 0 it would reach 8 n, past 2^32 for a variable X of n >= 2^29.
__host__ __device__ inline long long gemm_b_base(int transb, int ldb, int j0) {
  return 8ll * (transb ? (long long)j0 : (long long)ldb * j0);
}
__host__ __device__ inline unsigned gemm_b_offset(int transb, unsigned ldb, unsigned j, unsigned k) {
  return 8u * (transb ? j + ldb * k : j * ldb + k);
}
// ONE: a block per tile (kgroups 1), of one term (1) or up to three (3).  In a loop over
// tiles the compiler forms what does not change in front of it, for all three terms, and
// a product of a block or two of K a wave is bound by the instructions up to its first
// load (16 x 16 tiles, us of an iteration of one term at d = 8, 128, 160, 256: 8.0, 11.5, 13.1,
// 15.8 in the loop, 6.9, 10.3, 11.1, 13.3 without it, 6.5, 9.8, 10.7, 13.1 for one term; the
// larger tiles have more K a wave).
template <class Epi, bool PART, int WM, int WN, int NW, bool SHORT = false, int ONE = 0>
__global__ __launch_bounds__(64 * NW) void k_dgemm(int M, int N, GemmOps op, int ldo, Epi epi,
                                                   const DevParams* __restrict__ prm, int jit, RedOut red, int kgroups,
                                                   double* __restrict__ parts) {
  constexpr int NR = Epi::NR;
  constexpr int NT = 64 * NW;
  constexpr int TM = 16 * WM, TN = 16 * WN;
  constexpr int R = HQ_GRING;
  __shared__ double tile_w[NW][TM * TN];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const int tiles_m = (M + TM - 1) / TM, tiles_n = (N + TN - 1) / TN;
  const int tiles = tiles_m * tiles_n;
  const int n0 = (op.K[0] + 15) / 16;
  constexpr bool TERMS = ONE != 1;   // up to three terms, else one
  const int n1 = TERMS && op.nt > 1 ? (op.K[1] + 15) / 16 : 0;
  const int n2 = TERMS && op.nt > 2 ? (op.K[2] + 15) / 16 : 0;
  const int total = n0 + n1 + n2;
  const int per = (total + kgroups - 1) / kgroups;
  auto pick = [&](int t, auto x0, auto x1, auto x2) { return !TERMS || t == 0 ? x0 : t == 1 ? x1 : x2; };
  Epi e = epi;
  if (!ONE) e.setup(prm, jit);
  double acc[NR > 0 ? NR : 1];
#pragma unroll
  for (int q = 0; q < (NR > 0 ? NR : 1); ++q) acc[q] = 0.0;
  auto work_item = [&](int w) {
    // Work item of this block: workgroups go to the 8 XCDs in turn, so XCD x takes
    // items w = x, x + 8, ...; they are mapped to a contiguous range of an order
    // that runs through bands of HQ_GBAND tile rows column by column, and an
    // XCD's L2 then fetches a compact part of each operand.
    int i0 = 0, j0 = 0, grp = 0;
    if (!ONE || tiles > 1) {
      const int work = tiles * kgroups, xq = work / 8, xr = work % 8, xcd = w % 8;
      const int item = xcd * xq + min(xcd, xr) + w / 8;
      const int tile = ONE ? item : item % tiles;
      grp = ONE ? 0 : item / tiles;
      const int band = tile / (HQ_GBAND * tiles_n), in_band = tile - band * HQ_GBAND * tiles_n;
      const int bh = min(HQ_GBAND, tiles_m - band * HQ_GBAND);
      i0 = (band * HQ_GBAND + in_band % bh) * TM;
      j0 = (in_band / bh) * TN;
    }
    // this wave's K blocks, [c0, c1)
    const int g0 = min(total, grp * per), gn = min(total, g0 + per) - g0;
    const int c0 = g0 + (int)((long long)gn * wv / NW), c1 = g0 + (int)((long long)gn * (wv + 1) / NW);
    // Two cursors walk the blocks, one for the loads and, R blocks behind, one
    // for the products.  Within a term a load is a uniform base that moves by a
    // block and a byte offset that stays.  The last block of a term starts at
    // K - 16, so that it reads in range, and what the block before it has taken
    // is zeroed (K < 16: a clamped index, zeroed likewise).  Rows and columns past
    // the edge are read from a clamped index and never stored.  (An offset into A
    // stays below 8 (M + 12 lda) bytes: M and lda are the order of a factor.)
    struct Cur { const char *A, *B; unsigned va[WM], vb[WN]; int t, cc, nc, K; long long sa, sb; };
    struct Frag { double a[4][WM], b[4][WN]; };
    Cur lc;
    auto load_term = [&](int t, int cc) {
      lc.t = t; lc.cc = cc;
      lc.nc = pick(t, n0, n1, n2);
      lc.K = pick(t, op.K[0], op.K[1], op.K[2]);
      const int tb = pick(t, op.transb[0], op.transb[1], op.transb[2]);
      const unsigned lda = pick(t, op.lda[0], op.lda[1], op.lda[2]), ldb = pick(t, op.ldb[0], op.ldb[1], op.ldb[2]);
      lc.sa = 8ll * lda; lc.sb = tb ? 8ll * ldb : 8;   // bytes per k
      lc.A = (const char*)pick(t, op.A[0], op.A[1], op.A[2]);
      lc.B = (const char*)pick(t, op.B[0], op.B[1], op.B[2]) + gemm_b_base(tb, ldb, j0);
#pragma unroll
      for (int m = 0; m < WM; ++m)
        lc.va[m] = 8u * ((unsigned)min(i0 + 16 * m + li, M - 1) + (SHORT ? 0u : lda * 4u * lk));
#pragma unroll
      for (int n = 0; n < WN; ++n) {
        lc.vb[n] = gemm_b_offset(tb, ldb, min(16 * n + li, N - 1 - j0), SHORT ? 0u : 4u * lk);
      }
    };
    auto load = [&](Frag& f) {
      const int k0 = max(0, min(16 * lc.cc, lc.K - 16));
      const char* const Ap = lc.A + lc.sa * k0;
      const char* const Bp = lc.B + lc.sb * k0;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        // SHORT: some K is below 16, every lane's k is clamped
        const long long k = SHORT ? min(4 * lk + s, lc.K - 1 - k0) : s;
#pragma unroll
        for (int m = 0; m < WM; ++m) f.a[s][m] = *(const double*)(Ap + lc.sa * k + lc.va[m]);
#pragma unroll
        for (int n = 0; n < WN; ++n) f.b[s][n] = *(const double*)(Bp + lc.sb * k + lc.vb[n]);
      }
      // the next block; after the last one that is loaded again, unread
      if (lc.cc + 1 < lc.nc) ++lc.cc;
      else if (TERMS && lc.t + 1 < op.nt) load_term(lc.t + 1, 0);
    };
    hq_dx4 d[WM][WN];
#pragma unroll
    for (int a = 0; a < WM; ++a)
#pragma unroll
      for (int b = 0; b < WN; ++b) d[a][b] = hq_dx4{0.0, 0.0, 0.0, 0.0};
    int mt = 0, mc = 0;   // the products' cursor: term and block of it
    auto multiply = [&](Frag& f) {
      const int K = pick(mt, op.K[0], op.K[1], op.K[2]);
      const int lo = 16 * mc - max(0, min(16 * mc, K - 16));
      if (lo > 0 || K < 16) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
          if (4 * lk + s < lo || 4 * lk + s >= K) {
#pragma unroll
            for (int m = 0; m < WM; ++m) f.a[s][m] = 0.0;
#pragma unroll
            for (int n = 0; n < WN; ++n) f.b[s][n] = 0.0;
          }
      }
      const long long sg = (long long)(pick(mt, op.neg[0], op.neg[1], op.neg[2]) ? 0x80000000u : 0u) << 32;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
#pragma unroll
        for (int n = 0; n < WN; ++n) f.b[s][n] = __longlong_as_double(__double_as_longlong(f.b[s][n]) ^ sg);
#pragma unroll
        for (int m = 0; m < WM; ++m)
#pragma unroll
          for (int n = 0; n < WN; ++n)
            d[m][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(f.b[s][n], f.a[s][m], d[m][n], 0, 0, 0);
      }
      if (mc + 1 < pick(mt, n0, n1, n2)) ++mc;
      else if (TERMS && mt + 1 < op.nt) { ++mt; mc = 0; }
    };
    auto start = [&] {
      const int t0 = !TERMS ? 0 : c0 >= n0 + n1 ? 2 : c0 >= n0 ? 1 : 0;
      mt = t0;
      mc = c0 - pick(t0, 0, n0, n0 + n1);
      load_term(mt, mc);
    };
    if (ONE && c1 - c0 <= 2) {
      // a block or two without the ring, whose last loads are issued in vain and the
      // epilogue's wait for them, and the epilogue's scalars (a memory latency and
      // divisions) while the operands arrive
      Frag f[2];
      if (c1 - c0 == 2) {
        start();
        load(f[0]);
        load(f[1]);
        e.setup(prm, jit);
        multiply(f[0]);
        multiply(f[1]);
      } else if (c1 - c0 == 1) {
        start();
        load(f[0]);
        e.setup(prm, jit);
        multiply(f[0]);
      } else {
        e.setup(prm, jit);
      }
    } else if (c0 < c1) {
      start();
      Frag f[R];
#pragma unroll
      for (int r = 0; r < R; ++r) load(f[r]);
      if (ONE) e.setup(prm, jit);
      int c = c0;
      for (; c + R <= c1; c += R) {   // no conditional load: the waits count exactly the loads they need
#pragma unroll
        for (int r = 0; r < R; ++r) {
          multiply(f[r]);
          load(f[r]);
        }
      }
#pragma unroll
      for (int r = 0; r < R - 1; ++r)
        if (c + r < c1) multiply(f[r]);
    }
    // the epilogue's rows in batches whose operands are in flight together, the
    // first batch's before the tiles are added (8 waves: half the registers)
    constexpr int NE = (TM * TN + NT - 1) / NT;   // rows of the epilogue per thread
    constexpr int NB = NW > 4 && NE > 2 ? 2 : NE;
    static_assert(NE % NB == 0, "epilogue batches");
    using EO = EpiOps<Epi>;
    typename EO::type ops[NB];
    auto row_of = [&](int q, int& gi, int& gj) {
      const int k = tid + q * NT;
      gi = i0 + k % TM; gj = j0 + k / TM;
      return k < TM * TN && gi < M && gj < N;
    };
    auto load_ops = [&](int q0) {
      if constexpr (!PART) {
#pragma unroll
        for (int q = 0; q < NB; ++q) {
          int gi, gj;
          if (row_of(q0 + q, gi, gj)) ops[q] = EO::load(e, gi + ldo * gj);
        }
      }
    };
    load_ops(0);
    // lane l holds D[16 m + l%16][16 n + l/16 + 4 v] of the tile
#pragma unroll
    for (int m = 0; m < WM; ++m)
#pragma unroll
      for (int n = 0; n < WN; ++n)
#pragma unroll
        for (int v = 0; v < 4; ++v) tile_w[wv][(16 * n + lk + 4 * v) * TM + 16 * m + li] = d[m][n][v];
    __syncthreads();
#pragma unroll
    for (int q0 = 0; q0 < NE; q0 += NB) {
      if (q0 > 0) load_ops(q0);
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        int gi, gj;
        if (row_of(q0 + q, gi, gj)) {
          double s = tile_w[0][tid + (q0 + q) * NT];
#pragma unroll
          for (int g = 1; g < NW; ++g) s += tile_w[g][tid + (q0 + q) * NT];
          if constexpr (PART) parts[(size_t)grp * M * N + gi + (size_t)M * gj] = s;
          else EO::run(e, gi + ldo * gj, s, acc, ops[q]);
        }
      }
    }
    if constexpr (!ONE) __syncthreads();   // tile_w is rewritten by the next tile
  };
  if constexpr (ONE) work_item(blockIdx.x);
  else
    for (int w = blockIdx.x; w < tiles * kgroups; w += gridDim.x) work_item(w);
  if constexpr (!PART) {
    if (red.active) block_reduce_store<NR, Epi::MAXMASK>(acc, red);
  }
}

// out(i) = sum over the kgroups partial products in group order -> epilogue
template <class Epi>
__global__ __launch_bounds__(HQ_BLOCK) void k_gemm_sum(long long count, int kgroups, const double* __restrict__ parts,
                                                       Epi epi, const DevParams* __restrict__ prm, int jit,
                                                       RedOut red) {
  constexpr int NR = Epi::NR;
  Epi e = epi;
  e.setup(prm, jit);
  double acc[NR > 0 ? NR : 1];
#pragma unroll
  for (int q = 0; q < (NR > 0 ? NR : 1); ++q) acc[q] = 0.0;
  for (long long i = (long long)blockIdx.x * HQ_BLOCK + threadIdx.x; i < count; i += (long long)gridDim.x * HQ_BLOCK) {
    double q = parts[i];
    for (int g = 1; g < kgroups; ++g) q += parts[(size_t)g * count + i];
    e((int)i, q, acc);
  }
  if (red.active) block_reduce_store<NR, Epi::MAXMASK>(acc, red);
}

// ---------------------------------------------------------------------------
// Q = diag(d) + F F^T, F n x r row-major (r <= 16).
// Stage 1: per-block partial sums of t = F^T x (slots red.slot[0..r-1]).
// Stage 2 (after the final reduction): (Q x)_i = d_i x_i + sum_k F_ik t_k.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(HQ_BLOCK) void k_lr_partial(int n, int r, const double* __restrict__ F,
                                                         const double* __restrict__ x, RedOut red) {
  double acc[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) acc[k] = 0.0;
  for (long long i = (long long)blockIdx.x * HQ_BLOCK + threadIdx.x; i < n; i += (long long)gridDim.x * HQ_BLOCK) {
    const double xi = x[i];
    const double* Fi = F + (size_t)i * r;
#pragma unroll
    for (int k = 0; k < 16; ++k)
      if (k < r) acc[k] += Fi[k] * xi;
  }
  block_reduce_store<16, 0u>(acc, red);
}

template <class Epi>
__global__ __launch_bounds__(HQ_BLOCK) void k_lr_apply(int n, int r, const double* __restrict__ dg,
                                                       const double* __restrict__ F,
                                                       const double* __restrict__ x,
                                                       const double* __restrict__ t, Epi epi,
                                                       const DevParams* __restrict__ prm, int jit, RedOut red) {
  constexpr int NR = Epi::NR;
  Epi e = epi;
  e.setup(prm, jit);
  double acc[NR > 0 ? NR : 1];
#pragma unroll
  for (int s = 0; s < (NR > 0 ? NR : 1); ++s) acc[s] = 0.0;
  double tk[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) tk[k] = (k < r) ? t[k] : 0.0;
  for (long long i = (long long)blockIdx.x * HQ_BLOCK + threadIdx.x; i < n; i += (long long)gridDim.x * HQ_BLOCK) {
    const double* Fi = F + (size_t)i * r;
    double q = dg[i] * x[i];
#pragma unroll
    for (int k = 0; k < 16; ++k)
      if (k < r) q += Fi[k] * tk[k];
    e((int)i, q, acc);
  }
  if (red.active) block_reduce_store<NR, Epi::MAXMASK>(acc, red);
}
