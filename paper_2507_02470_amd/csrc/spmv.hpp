// spmv.hpp -- CSR SpMV kernels for gfx950 with a fused per-row epilogue.
#pragma once
#include "common.hpp"

// Row-split kernel for long rows: groups of G lanes each own one row (a
// block covers HQ_BLOCK / G rows per pass); the lanes stride over the row's
// nonzeros, the group's partial sums are added by a butterfly (G <= 64) or by
// wave sums combined in LDS in wave order (G = 128, 256: one row spans 2 or 4
// waves), and the group's first lane runs the epilogue.  Rows are dealt out
// in grid-stride order, so a matrix with a few hundred long rows still
// spreads over hundreds of waves.  No atomics; the summation order depends
// only on G.
//
// Lane `lane` of a group's share of the row [b, en): entries at, at + G, ...; `left`
// is the distance from `at` to the row's end (not positive: nothing is left).  The
// counts are taken against the end, and positions in 64 bits: a row may end at any
// 32-bit position, and a step past its end must not wrap.
struct RowSpan {
  size_t at;
  int left;
  __host__ __device__ RowSpan(int b, int en, int lane) : at((size_t)b + lane), left(en - b - lane) {}
  __host__ __device__ void skip(int k) { at += k; left -= k; }
};

// Partial sum of one lane, entries k = b, b + G, ... < en of a row, eight at a time: the
// columns and values, then the gathers of a step are in flight together.  While every
// lane that is left has eight, the loads are unconditional, at fixed distances from one
// address (a clamp of each position costs more than it saves: rows of 544 on 64 lanes,
// 7,502 of them, 28.4 us clamped, 25.6 so); then a lane loads what it has, so that the end
// of a row is one step too (rows of 50 on 32 lanes, 4e4 of them, epilogue included:
// 14.7 us clamped, 15.2 one entry after the other, 13.6 so; rows of 74 on 64 lanes 33.0,
// 33.1, 31.8).  Lanes that have none left do not hold a long row up (one of 5,000 among
// rows of 5, 4 lanes a row: 107 us, 80 and 56).
template <int G, bool ALL>
__device__ __forceinline__ double row_step(const int* __restrict__ col, const double* __restrict__ val,
                                           const double* xin, const RowSpan& r, double sum) {
  constexpr int U = 8;
  const int* const cp = col + r.at;
  const double* const vp = val + r.at;
  int c[U];
  double v[U], x[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    c[u] = 0; v[u] = 0.0;
    if (ALL || u * G < r.left) { c[u] = ld_stream(cp + u * G); v[u] = ld_stream(vp + u * G); }
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    x[u] = 0.0;
    if (ALL || u * G < r.left) x[u] = xin[c[u]];
  }
#pragma unroll
  for (int u = 0; u < U; ++u) sum += v[u] * x[u];
  return sum;
}
template <int G>
__device__ __forceinline__ double row_part(const int* __restrict__ col, const double* __restrict__ val,
                                           const double* xin, RowSpan r) {
  double sum = 0.0;
  for (; r.left > 0; r.skip(8 * G)) {
    if (__all(r.left > 7 * G)) sum = row_step<G, true>(col, val, xin, r, sum);
    else sum = row_step<G, false>(col, val, xin, r, sum);
  }
  return sum;
}

template <int G, class Epi>
__global__ __launch_bounds__(HQ_BLOCK) void k_csr(int nrows, const int* __restrict__ rowptr,
                                                  const int* __restrict__ col,
                                                  const double* __restrict__ val,
                                                  const double* __restrict__ xin, Epi epi,
                                                  const DevParams* __restrict__ prm, int j, RedOut red) {
  static_assert(G >= 1 && G <= HQ_BLOCK && (HQ_BLOCK % G) == 0, "lanes per row");
  constexpr int RPB = HQ_BLOCK / G;  // rows per block per pass
  constexpr int NR = Epi::NR;
  const int gl = threadIdx.x % G;
  const int gi = threadIdx.x / G;
  Epi e = epi;
  e.setup(prm, j);
  double acc[NR > 0 ? NR : 1];
#pragma unroll
  for (int s = 0; s < (NR > 0 ? NR : 1); ++s) acc[s] = 0.0;
  for (long long r0 = (long long)blockIdx.x * RPB; r0 < nrows; r0 += (long long)gridDim.x * RPB) {
    const long long row = r0 + gi;
    double sum = 0.0;
    typename EpiOps<Epi>::type ops;
    if (row < nrows) {
      const int b = rowptr[row], en = rowptr[row + 1];
      if (gl == 0) ops = EpiOps<Epi>::load(e, (int)row);
      sum = row_part<G>(col, val, xin, RowSpan(b, en, gl));
    }
    if constexpr (G > 64) {
      __shared__ double wpart[HQ_BLOCK / HQ_WAVE];
      sum = wave_sum(sum);
      if ((threadIdx.x & (HQ_WAVE - 1)) == 0) wpart[threadIdx.x / HQ_WAVE] = sum;
      __syncthreads();
      if (gl == 0) {
        const int w0 = (gi * G) / HQ_WAVE;
        sum = wpart[w0];
#pragma unroll
        for (int w = 1; w < G / HQ_WAVE; ++w) sum += wpart[w0 + w];
      }
      __syncthreads();   // wpart is rewritten by the next pass
    } else if constexpr (G > 1) {
      sum = group_sum<G>(sum);
    }
    if (row < nrows && gl == 0) EpiOps<Epi>::run(e, (int)row, sum, acc, ops);
  }
  if (red.active) block_reduce_store<NR, Epi::MAXMASK>(acc, red);
}

// CSR-stream SpMV for short rows.  A block of HQ_BLOCK threads owns RB consecutive
// rows; their nonzeros (a contiguous range of the CSR arrays) are streamed in
// chunks with fully coalesced loads, each thread forming
// val[k] * x[col[k]] for k = c0 + tid, c0 + tid + HQ_BLOCK, ... into LDS; then
// thread t < RB adds up row t's products in CSR order (a fixed summation order)
// and runs the epilogue for that row.
// What bounds it: up to a few 1e5 rows, the chain of dependent memory latencies
// (row pointers, entries, gathers, epilogue operands), so the chain has no more
// links than these: the block's range comes by scalar loads, every entry of a
// chunk is in flight at once and then every gather (no load is conditional: the
// waits between them then count exactly; threads past the end of a chunk repeat
// its last entry), and the epilogue's operands arrive with the entries.  RB and
// the E entries a thread takes of a chunk follow the matrix (stream_shape).
#define HQ_STREAM_CHUNK 2048
template <class Epi, int RB, int E>
__global__ __launch_bounds__(HQ_BLOCK) void k_csr_stream(int nrows, const int* __restrict__ rowptr,
                                                         const int* __restrict__ col,
                                                         const double* __restrict__ val,
                                                         const double* __restrict__ xin, Epi epi,
                                                         const DevParams* __restrict__ prm, int j, RedOut red) {
  constexpr int NR = Epi::NR;
  constexpr int CH = E * HQ_BLOCK;
  __shared__ double prod[CH];
  Epi e = epi;
  e.setup(prm, j);
  double acc[NR > 0 ? NR : 1];
#pragma unroll
  for (int s = 0; s < (NR > 0 ? NR : 1); ++s) acc[s] = 0.0;
  const int t = threadIdx.x;
  const int nblk = (nrows + RB - 1) / RB;
  for (int rb = blockIdx.x; rb < nblk; rb += gridDim.x) {
    const int r0 = rb * RB, nr = min(RB, nrows - r0);
    const int kb = rowptr[r0], ke = rowptr[r0 + nr];
    const int tr = min(t, nr - 1);   // (threads past the rows repeat the last row's loads)
    const int myb = rowptr[r0 + tr], mye = t < nr ? rowptr[r0 + tr + 1] : 0;
    const typename EpiOps<Epi>::type ops = EpiOps<Epi>::load(e, r0 + tr);
    double sum = 0.0;
    for (int c0 = kb; c0 < ke; c0 += CH) {
      const int c1 = min(ke, c0 + CH);
      int ci[E];
      double v[E], x[E];
#pragma unroll
      for (int u = 0; u < E; ++u) {
        const int k = min(c0 + t + u * HQ_BLOCK, c1 - 1);
        ci[u] = ld_stream(col + k);
        v[u] = ld_stream(val + k);
      }
#pragma unroll
      for (int u = 0; u < E; ++u) x[u] = xin[ci[u]];
#pragma unroll
      for (int u = 0; u < E; ++u) prod[t + u * HQ_BLOCK] = v[u] * x[u];   // (past the end: never read)
      __syncthreads();
      const int lo = max(myb, c0), hi = min(mye, c1);
      for (int k = lo; k < hi; k += 4) {
        double q[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) q[u] = prod[min(k + u, hi - 1) - c0];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (k + u < hi) sum += q[u];
      }
      __syncthreads();
    }
    if (t < nr) EpiOps<Epi>::run(e, r0 + t, sum, acc, ops);
  }
  if (red.active) block_reduce_store<NR, Epi::MAXMASK>(acc, red);
}

// Shape of k_csr_stream, as 10 RB + E: the most rows per block that still give every
// CU a block and whose entries fit one chunk, with the smallest chunk that holds
// them, since larger ones than needed cost their loads (rows of 2, 1e6 of them: 80.6 us
// an iteration with E = 2, 81.8 with 4, 85.1 with 8; random rows of 5 and 10 entries,
// n = 2e4, m = 1e4: 4.7 us a product with 32 rows, 4.4 and 6.9 with 256).  Entries fit
// where the longest row says so, or with 5% to spare on the average (rows of equal
// length need no margin: 256 rows of 8 fill a chunk of 2,048).
// Longer rows, us an iteration of a QP with two Q products:
//  even ones: blocks of 128 rows and chunks of 2,048 where those hold them (12 on
//  average, n = 50,000, 90,000, 131,072, 262,144, 390,000: 22.6, 32.1, 41.2, 66.9, 95.9 against
//  24.4, 35.6, 41.9, 64.9, 95.2 with 256 rows in several chunks and 23.9, 34.6, 44.5, 72.9, 108
//  with 64 rows and chunks of 1,024, but 18.6 against 18.1 with those at n = 33,000), 256
//  rows in several chunks of 2,048 for many rows,
//  where the stream of the matrix is what counts (18 on average: 31.7, 45.7, 52.6, 84.6,
//  124 against 30.2, 44.7, 59.5, 107, 156 with 32 rows and chunks of 1,024);
//  uneven ones: a thread adds up a row and its block waits, so few rows a block, 64, and
//  chunks of 2,048 for the long ones (15 on average, one product, n = 131,072: up to 200
//  28.9, 32.2 with 32 rows, 37.5 with 256; up to 400 38.5, 45.5, 52.0; up to 4,000 154,
//  168, 165).
inline int stream_shape(int rows, long long nnz, int maxlen, int ncu) {
  const double avg = rows > 0 ? (double)nnz / rows : 0.0;
  const bool even = maxlen >= 0 && maxlen <= 6.0 * avg;
  const auto fits = [&](int rb, int e) {
    return (maxlen >= 0 && (long long)maxlen * rb <= HQ_BLOCK * e) || 1.05 * avg * rb <= HQ_BLOCK * e;
  };
  const long long per_cu = rows / ncu;
  if (per_cu >= 256)
    for (int e : {2, 4, 8})
      if (fits(256, e)) return 2560 + e;
  if (even && per_cu >= 768) return 2568;
  if (per_cu >= 128 && fits(128, 4)) return 1284;
  if (even && per_cu >= 192 && fits(128, 8)) return 1288;
  if (even && per_cu >= 384) return 2568;
  if (per_cu >= 64) {
    if (fits(64, 2)) return 642;
    if (!even) return 648;
    if (fits(64, 4)) return 644;
  }
  return fits(32, 2) ? 322 : 324;
}

// The stream kernel gathering from a copy of the whole input vector in LDS
// (dynamic shared memory, ncols <= HQ_XLDS_MAX entries): the gathers then cost no
// L2 requests.  Persistent blocks of BS threads (= rows per pass), so the copy is
// made once per block; chunks of 4096 products (32 KB of LDS beside the copy).
#define HQ_XLDS_MAX 14336
#define HQ_XLDS_BLOCK 1024
template <class Epi, int BS>
__global__ __launch_bounds__(BS) void k_csr_xstream(int nrows, const int* __restrict__ rowptr,
                                                    const int* __restrict__ col,
                                                    const double* __restrict__ val,
                                                    const double* __restrict__ xin, Epi epi,
                                                    const DevParams* __restrict__ prm, int j, RedOut red, int ncols) {
  constexpr int NR = Epi::NR;
  constexpr int CH = 2 * HQ_STREAM_CHUNK;
  __shared__ double prod[CH];
  __shared__ int srp[BS + 1];
  extern __shared__ double xs[];
  Epi e = epi;
  e.setup(prm, j);
  double acc[NR > 0 ? NR : 1];
#pragma unroll
  for (int s = 0; s < (NR > 0 ? NR : 1); ++s) acc[s] = 0.0;
  const int t = threadIdx.x;
  for (int i = t; i < ncols; i += BS) xs[i] = xin[i];
  __syncthreads();
  const int nblk = (nrows + BS - 1) / BS;
  for (int rb = blockIdx.x; rb < nblk; rb += gridDim.x) {
    const int r0 = rb * BS;
    const int nr = min(BS, nrows - r0);
    for (int i = t; i <= nr; i += BS) srp[i] = rowptr[r0 + i];   // nr + 1 row pointers
    __syncthreads();
    const int kb = srp[0], ke = srp[nr];
    const int myb = t < nr ? srp[t] : 0, mye = t < nr ? srp[t + 1] : 0;
    double sum = 0.0;
    for (int c0 = kb; c0 < ke; c0 += CH) {
      const int c1 = min(ke, c0 + CH);
#pragma unroll 4
      for (int k = c0 + t; k < c1; k += BS) prod[k - c0] = ld_stream(val + k) * xs[ld_stream(col + k)];
      __syncthreads();
      const int lo = max(myb, c0), hi = min(mye, c1);
      for (int k = lo; k < hi; ++k) sum += prod[k - c0];
      __syncthreads();
    }
    if (t < nr) e(r0 + t, sum, acc);
    __syncthreads();   // srp is rewritten by the next row block
  }
  if (red.active) block_reduce_store<NR, Epi::MAXMASK>(acc, red);
}

// 16-bit copy of the columns of a matrix whose input vector fits LDS, and a zero
// behind them (they are read in pairs)
__global__ void k_cols16(long long nnz, const int* __restrict__ col, unsigned short* __restrict__ c16) {
  for (long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x; k <= nnz; k += (long long)gridDim.x * blockDim.x)
    c16[k] = k < nnz ? (unsigned short)col[k] : 0;
}
typedef double hq_pair __attribute__((ext_vector_type(2), aligned(8)));   // two entries' values

// The entries of the row [b, en) in pairs that start at even positions, by their
// distance `rel` (even) from the last such position at or before b: distances do not
// wrap, wherever the row lies in the 32-bit range.
struct RowPairs {
  int b, en;
  __host__ __device__ int base() const { return b & ~1; }
  __host__ __device__ int len() const { return en - base(); }
  // position of the pair to read: the pair at rel, clamped into the row (an empty row:
  // to the entry before it)
  __host__ __device__ int at(int rel) const {
    const int last = (len() - 1) & ~1, k = base() + (rel < last ? rel : last);
    return k > 0 ? k : 0;
  }
  // whether the first and the second entry of the pair at rel are the row's
  __host__ __device__ bool first(int rel) const { return rel >= (b & 1) && rel < len(); }
  __host__ __device__ bool second(int rel) const { return rel + 1 < len(); }
};

// Row-split kernel (G <= 64 lanes per row) gathering from an LDS copy of the input
// vector (at most HQ_XLDS_MAX entries): for rows of tens to hundreds of nonzeros
// over a small vector (the Lasso's Ahat^T, p columns), where the stream kernel
// would add each long row serially.  Persistent 1024-thread blocks copy the
// vector once; each wave then takes 64 rows at a time, its 64 / G groups adjacent
// rows at each of G steps (the wave reads one contiguous stretch of the matrix;
// groups 16 rows apart cost a fifth of the bandwidth), and a shuffle at the end
// gives lane l the sum of row l for the epilogue.
// Bound by the stream of the matrix, which needs some 40 KB in flight per CU beside
// the 16 waves that the vector's copy leaves room for: 10 bytes an entry
// (16-bit columns), eight entries a lane in four pairs (16- and 4-byte loads; one
// entry a load kept the address units busy), the next row's loads issued before
// the current row is summed, the row pointers of all G rows loaded at once.
// Ahat^T of the Lasso (5e5 rows of 100 over 1e4 columns), 500 MB: 165 us with 32-bit
// columns, 140 with 16-bit ones, 107 in pairs (4.7 TB/s, the rate of a large copy);
// with the iteration's epilogue 192 + 14 us for the step behind it, 150, 121.
#define HQ_XROW_U 8
template <int G, class Epi>
__global__ __launch_bounds__(HQ_XLDS_BLOCK) void k_csr_xrow(int nrows, const int* __restrict__ rowptr,
                                                            const unsigned short* __restrict__ c16,
                                                            const double* __restrict__ val,
                                                            const double* __restrict__ xin, Epi epi,
                                                            const DevParams* __restrict__ prm, int j, RedOut red,
                                                            int ncols, int nnz) {
  static_assert(G >= 1 && G <= HQ_WAVE && (HQ_WAVE % G) == 0, "lanes per row");
  constexpr int BS = HQ_XLDS_BLOCK, WAVES = BS / HQ_WAVE, U = HQ_XROW_U;
  constexpr int NR = Epi::NR;
  extern __shared__ double xs[];
  constexpr int NG = HQ_WAVE / G;   // groups of a wave
  const int lane = threadIdx.x & (HQ_WAVE - 1), gl = lane % G, gi = lane / G;
  Epi e = epi;
  e.setup(prm, j);
  double acc[NR > 0 ? NR : 1];
#pragma unroll
  for (int s = 0; s < (NR > 0 ? NR : 1); ++s) acc[s] = 0.0;
  for (int i = threadIdx.x; i < ncols; i += BS) xs[i] = xin[i];
  __syncthreads();
  struct Row { RowPairs p; unsigned c[U / 2]; hq_pair v[U / 2]; };
  const long long chunks = ((long long)nrows + HQ_WAVE - 1) / HQ_WAVE;
  for (long long ch = (long long)blockIdx.x * WAVES + threadIdx.x / HQ_WAVE; ch < chunks;
       ch += (long long)gridDim.x * WAVES) {   // same trip count in every lane of the wave
    const int row = (int)(ch * HQ_WAVE) + lane, rc = min(row, nrows - 1);
    const int rb = rowptr[rc], re = row < nrows ? rowptr[rc + 1] : rb;
    // the first U entries per lane of the group's row of step q, in pairs k, k + 1 of
    // even k (RowPairs: what is read past the row is never used; the last entry of an
    // odd number of them is the second of its pair)
    auto fetch = [&](int q, Row& r) {
      r.p.b = __shfl(rb, q * NG + gi);
      r.p.en = __shfl(re, q * NG + gi);
#pragma unroll
      for (int u = 0; u < U / 2; ++u) {
        const int k = r.p.at(2 * gl + 2 * u * G);
        r.c[u] = __builtin_nontemporal_load((const unsigned*)(c16 + k));
        r.v[u] = __builtin_nontemporal_load((const hq_pair*)(val + min(k, nnz - 2)));
      }
    };
    double mine = 0.0;
    auto sum = [&](int q, const Row& r) {
      double s = 0.0, x[U];
#pragma unroll
      for (int u = 0; u < U / 2; ++u) { x[2 * u] = xs[r.c[u] & 0xffffu]; x[2 * u + 1] = xs[r.c[u] >> 16]; }
      const int end = nnz - 1 - r.p.base();   // of the matrix's last entry
#pragma unroll
      for (int u = 0; u < U / 2; ++u) {
        const int k = 2 * gl + 2 * u * G;
        s += (k == end ? r.v[u].y : r.v[u].x) * (r.p.first(k) ? x[2 * u] : 0.0);
        s += r.v[u].y * (r.p.second(k) ? x[2 * u + 1] : 0.0);
      }
      const double* const vr = val + r.p.base();
      const unsigned short* const cr = c16 + r.p.base();
      const unsigned len = r.p.len();
      for (unsigned k = 2 * gl + U * G; k < len; k += 2 * G) {
        s += ld_stream(vr + k) * xs[ld_stream(cr + k)];
        if (k + 1 < len) s += ld_stream(vr + k + 1) * xs[ld_stream(cr + k + 1)];
      }
      s = group_sum<G>(s);
      if (gl == q) mine = s;
    };
    Row r0, r1;
    fetch(0, r0);
    if constexpr (G == 1) {
      sum(0, r0);
    } else {
#pragma unroll 1
      for (int q = 0; q < G; q += 2) {
        fetch(q + 1, r1);
        __builtin_amdgcn_sched_barrier(0);   // the sums' waits stay behind the next loads
        sum(q, r0);
        fetch(min(q + 2, G - 1), r0);
        __builtin_amdgcn_sched_barrier(0);
        sum(q + 1, r1);
      }
    }
    mine = __shfl(mine, (lane % NG) * G + lane / NG);   // row l: step l / NG of group l % NG
    if (row < nrows) e(row, mine, acc);
  }
  if (red.active) block_reduce_store<NR, Epi::MAXMASK>(acc, red);
}

// Elementwise driver: epi(i, q_i) with a precomputed / zero q.
template <class Epi>
__global__ __launch_bounds__(HQ_BLOCK) void k_elem(int n, const double* __restrict__ q, Epi epi,
                                                   const DevParams* __restrict__ prm, int j, RedOut red) {
  constexpr int NR = Epi::NR;
  Epi e = epi;
  e.setup(prm, j);
  double acc[NR > 0 ? NR : 1];
#pragma unroll
  for (int s = 0; s < (NR > 0 ? NR : 1); ++s) acc[s] = 0.0;
  for (long long i = (long long)blockIdx.x * HQ_BLOCK + threadIdx.x; i < n;
       i += (long long)gridDim.x * HQ_BLOCK)
    e((int)i, q ? q[i] : 0.0, acc);
  if (red.active) block_reduce_store<NR, Epi::MAXMASK>(acc, red);
}
