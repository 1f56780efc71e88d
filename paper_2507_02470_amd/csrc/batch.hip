// batch.hip -- many independent HPR-QPs (Algorithm 4 + Algorithm 5 of arXiv
// 2507.02470) in persistent kernels on one MI355X.
//
// One workgroup owns one instance at a time; instances are pulled from a
// work queue ordered by size (largest first).  The instances are cut into
// size classes (n <= 256, 512, 1024, 2048) and each class runs on a kernel of
// its own shape: BS = 64, 128, 256 or 512 threads with EPT = 1, 2 or 4 entries
// each (by default 256 threads up to n = 1024 and 512 above; with autotuning,
// create times every block size that can hold a class on a sample of the
// class's instances and keeps the fastest).  The kernels in use run at once on
// their own streams.
// Thread t owns entries t + BS e, e < EPT.  An iteration is bound by the latency
// of its dependent steps (a block-wide reduction per Q product, the A and A^T
// products through LDS) and by the instructions of the reductions, not by
// bandwidth, so it touches no memory: the iterate, its images Q w and A^T y, the
// Halpern anchors and (at rank <= 10, or few entries a thread) the rows of F of
// the thread's entries are in registers, and A, A^T, c, the box and diag(d) of the
// instance are in LDS, where they fit; an instance whose A (or c, box and diag(d))
// does not fit reads them from memory.  With the state in LDS, and A, c, the box
// and diag(d) read from memory at each use, the clock stamps of an iteration at
// n = 1000, m = 21 on 256 threads (one workgroup per CU) were z/x step 3,250 cycles,
// Q xhat 3,600, A v and y step 8,670, A^T 5,660, Q d 4,780, Halpern 2,380.  200
// iterations with the power methods took 2.78 ms there and take 1.27 ms now; 4,096
// instances of n = 50..2000: 38.3 ms then, 20.3 ms now.
// The whole method runs on the device in FP64: power method for lambda_A and
// lambda_Q, the sigma0 rule, the iteration, the merit R~, the stopping test, the
// restart criteria of Section 3.2 and the golden-section sigma update of
// Algorithm 5 (thread 0, broadcast through LDS).  No host round trip until every
// instance is done.
#include "hprqp.h"
#include "common.hpp"

#include <algorithm>
#include <chrono>
#include <map>
#include <tuple>
#include <type_traits>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

namespace hq {
extern thread_local std::string g_err;
}

#define HB_NMAX 2048                                  // largest n
#define HB_EPT 4                                      // most entries per thread
#define HB_NCLASS 4                                    // size classes: n <= 256, 512, 1024, 2048
#define HB_MMAX 64
#define HB_RMAX 16
#define HB_APIECE 256                                  // nonzeros of A per wave work item (A in memory)
#define HB_LPIECE 64                                   // and per group of 16 lanes (A in LDS)
#define HB_LNNZ 12000                                 // most nonzeros of A in LDS

// Shape of a kernel: BS threads for n <= BS EPT.
template <int BS, int EPT>
struct BCfg {
  static_assert((BS == 64 || BS == 128 || BS == 256 || BS == 512) && (EPT == 1 || EPT == 2 || EPT == 4), "shapes");
  static constexpr int WAVES = BS / 64;
  static constexpr int NMAX = BS * EPT;
  // pieces of A at most: a row has at most n nonzeros (checked at create); in
  // LDS, 64 rows and at most 12,000 nonzeros
  static constexpr int PMAX = HB_MMAX * ((NMAX + HB_APIECE - 1) / HB_APIECE) > 256
                                  ? HB_MMAX * ((NMAX + HB_APIECE - 1) / HB_APIECE) : 256;
  // launch bound, waves per SIMD.  Two leave 256 registers a thread, which EPT = 4
  // needs (F alone takes 80) and which 512 threads have in any case; what four and
  // three leave (128, 168) holds the iteration at EPT = 1 and 2.
  static constexpr int MIN_WAVES = EPT == 4 || (EPT == 2 && BS == 512) ? 2 : EPT == 2 ? 3 : 4;
  // most dynamic LDS of a block: PER_CU blocks (as many as the registers allow, fewer
  // for small blocks, whose instances are small) share the 160 KB of a CU, 8 KB
  // of each share stay for the static part
  static constexpr int PER_CU = BS == 512 ? (EPT == 1 ? 2 : 1) : EPT == 4 ? (BS == 256 ? 2 : 4) : EPT == 2 ? 3 : 4;
  static constexpr int DYN_LDS = (160 / PER_CU - 8) * 1024;
};

struct BInst {
  int n, m, r;
  int pad;
  const double *c, *L, *U, *l, *u, *dg, *F;
  const int *arp, *aci;
  const double* aval;
  const int *trp, *tci;   // A^T (n x m) CSR, rows ordered by row of A
  const int* tperm;       // position in A of every entry of A^T
  const double* tval;
  const double* FT;       // F with rows padded to the kernel's rank RM (entries k >= r zero)
  long long off_n, off_m;
  long long annz;         // nonzeros of A
};

struct BOpts {
  double tol;
  long long max_iter;
  int check_every;
  double sigma0, lamA, lamQ;
  double alpha1, alpha2, alpha3;
  int enable_restart, enable_sigma_update;
  // time limit: wall-clock ticks (wall_clock64) since *t0, the stamp taken
  // on the stream just before the solve kernels; 0: none
  long long time_ticks;
  const long long* t0;
};

struct BInfo {
  int term, restarts;
  long long iters;
  double sigma, sigma0, lamA, lamQ, eta_p, eta_d, eta_gap, pobj, dobj, R_last;
};

// ---------------------------------------------------------------------------
// LDS of one instance
// ---------------------------------------------------------------------------
#define HB_RED 18   // most values reduced at once

// What the checks keep between them and hand out (thread 0 writes it).
struct BState {
  double sigma, sQ, inv, kappa, sA;   // sigma, sigma lambda_Q, 1 / (1 + sQ), sigma / (1 + sQ), sigma lambda_A
  double lamA, lamQ, binf, cinf, sigma0;
  double alpha3, R0ref, Rr0, Rprev, R;
  double eta_p, eta_d, eta_gap, pobj, dobj;
  double th[5];                       // the thetas of Algorithm 5: y, w, q, 2, 3
  int term, restart;
  __device__ void derive() { sQ = sigma * lamQ; inv = 1.0 / (1.0 + sQ); kappa = sigma / (1.0 + sQ); sA = sigma * lamA; }
};

template <int BS, int EPT>
struct BShared {
  static constexpr int NMAX = BCfg<BS, EPT>::NMAX, PMAX = BCfg<BS, EPT>::PMAX;
  alignas(16) double red[2][HB_RED][BCfg<BS, EPT>::WAVES];   // wave partials, two buffers used in turn
  double y[HB_MMAX], ya[HB_MMAX], yb[HB_MMAX], l[HB_MMAX], u[HB_MMAX];
  union {
    double yn[HB_MMAX];              // y^{t+1} (Halpern) until the check is done
    double pw[HB_MMAX];              // power method vector (length m), before the iterations
  };
  // A products: row r of A is cut into pieces; piece q belongs to row prow[q]
  // and pieces pstart[r] .. pstart[r+1]-1 to row r
  unsigned char prow[PMAX];          // (m <= 64)
  int pstart[HB_MMAX + 1];
  int arp[HB_MMAX + 1];              // row pointers of A
  int np;
  BState T;
  int inst;
  BOpts opt;                         // the options, for the out-of-line check decision
};

// The instance's arrays in the dynamic LDS, in this order: vm[nm] (a vector
// shared by the block, nm = BS EPT), part (sums of the pieces of A), then, where they fit
// into `cap` bytes, the values of A, c, L, U and diag(d) (nm each, zeros
// past n), the entries of A^T (position in A
// << 8 | row) and the 16-bit columns of A.
struct BPlan {
  int part;             // pieces of A at most
  bool a_in, clu_in;    // A and A^T; c, L, U and diag(d)
  size_t bytes;
};
__host__ __device__ inline BPlan batch_plan(int nm, int n, int m, long long annz, size_t cap) {
  BPlan P;
  const size_t pa = (size_t)(annz / HB_LPIECE + m), pm = (size_t)m * ((n + HB_APIECE - 1) / HB_APIECE);
  const size_t in = 8 * (nm + pa) + 14 * (size_t)annz;
  P.a_in = annz <= HB_LNNZ && in <= cap;
  P.part = (int)(P.a_in ? pa : pm);
  P.bytes = P.a_in ? in : 8 * (nm + pm);
  P.clu_in = P.bytes + 32 * (size_t)nm <= cap;
  if (P.clu_in) P.bytes += 32 * (size_t)nm;
  return P;
}
struct BLds {
  double *vm, *part, *av, *c, *L, *U, *dg;
  unsigned short* ac;
  unsigned* tq;
  bool a_in, clu_in;
};

// DPP move of a double (both 32-bit halves with the same control); lanes
// without a source read 0, the identity of the sums and of the maxima of
// non-negative values reduced here.
template <int CTRL, int ROWMASK = 0xf>
__device__ __forceinline__ double dpp_mov(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, ROWMASK, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWMASK, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Value of lane l of a wave, in scalar registers (l wave-uniform).
__device__ __forceinline__ double readlane_d(double x, int l) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), l);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Wave reduction with DPP (fixed pattern: quad swaps, row shifts by 4 and 8,
// row broadcasts 15 and 31); the result is exact in lane 63 only.
template <bool MX>
__device__ __forceinline__ double wave_reduce63(double v) {
  auto op = [](double a, double b) { return MX ? fmax(a, b) : a + b; };
  v = op(v, dpp_mov<0xb1>(v));          // quad_perm [1,0,3,2]
  v = op(v, dpp_mov<0x4e>(v));          // quad_perm [2,3,0,1]
  v = op(v, dpp_mov<0x114>(v));         // row_shr:4
  v = op(v, dpp_mov<0x118>(v));         // row_shr:8
  v = op(v, dpp_mov<0x142, 0xa>(v));    // row_bcast:15
  v = op(v, dpp_mov<0x143, 0xc>(v));    // row_bcast:31
  return v;
}

// Sum over the 16 lanes of a row of lanes (rotations; every lane gets it)
__device__ __forceinline__ double row16_sum(double v) {
  v += dpp_mov<0x128>(v);   // row_ror:8
  v += dpp_mov<0x124>(v);
  v += dpp_mov<0x122>(v);
  v += dpp_mov<0x121>(v);
  return v;
}

// Combines the wave partials S.red[par][s][0..W) of K values after the barrier:
// lanes W s .. W s + W - 1 hold value s, a fixed butterfly, and the result is
// read from lane W s into scalar registers (max where bit s of MAXMASK is set).
template <int K, unsigned MAXMASK, int BS, int EPT>
__device__ __forceinline__ void combine(BShared<BS, EPT>& S, int& par, double (&v)[K]) {
  constexpr int W = BCfg<BS, EPT>::WAVES;   // partials per value
  static_assert(K <= HB_RED && (W == 1 || W == 2 || W == 4 || W == 8), "reduction layout");
  const int lane = threadIdx.x & 63;
  constexpr int VP = 64 / W;   // values combined per pass
#pragma unroll
  for (int s0 = 0; s0 < K; s0 += VP) {
    const int s = s0 + lane / W, w = lane % W;
    const bool mx = MAXMASK != 0u && ((MAXMASK >> (s & 31)) & 1u);
    double x = S.red[par][s < K ? s : 0][w];   // (lanes past K: read, never used)
#pragma unroll
    for (int off = 1; off < W; off <<= 1) {
      // partner lane l ^ off: DPP quad permutations for 1 and 2, a shuffle for 4
      const double y = off == 1 ? dpp_mov<0xb1>(x) : off == 2 ? dpp_mov<0x4e>(x) : __shfl_xor(x, off);
      x = mx ? fmax(x, y) : x + y;
    }
    // every lane of group q holds value q: broadcast it from the group's first lane
#pragma unroll
    for (int q = s0; q < K && q < s0 + VP; ++q) v[q] = readlane_d(x, (q - s0) * W);
  }
  par ^= 1;
}

// Block-wide reduction of K values (sum, or max where bit s of MAXMASK is
// set; maxima only of non-negative values) with one barrier: DPP wave
// reductions, lane 63 of each wave stores its partials, combine().  Fixed
// order, deterministic.  The two partial buffers alternate between calls, so a
// buffer is rewritten only after every thread has passed the barrier of the
// call in between.
template <unsigned MAXMASK, int K, int BS, int EPT>
__device__ __forceinline__ void bred(BShared<BS, EPT>& S, int& par, double (&v)[K]) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int s = 0; s < K; ++s) {
    const double x = ((MAXMASK >> s) & 1u) ? wave_reduce63<true>(v[s]) : wave_reduce63<false>(v[s]);
    if (lane == 63) S.red[par][s][wv] = x;
  }
  __syncthreads();
  combine<K, MAXMASK>(S, par, v);
}

// a += b with the halves (rows of 16 lanes) of the two interchanged: lanes
// 0-31 (even rows) of the result hold sums of a, the others sums of b.
template <int ROWS>
__device__ __forceinline__ double swap_add(double a, double b) {
  const unsigned long long x = (unsigned long long)__double_as_longlong(a), y = (unsigned long long)__double_as_longlong(b);
  typedef unsigned v2 __attribute__((ext_vector_type(2)));
  v2 lo, hi;
  if constexpr (ROWS == 32) {
    lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
    hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  } else {
    lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
    hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  }
  const double p = __longlong_as_double((long long)(((unsigned long long)hi.x << 32) | lo.x));
  const double q = __longlong_as_double((long long)(((unsigned long long)hi.y << 32) | lo.y));
  return p + q;
}

// Block-wide sums of K values, one barrier.  Two lane swaps leave four values
// in one register (one per row of 16 lanes), whose rows are then added by
// rotations: 6 instructions per value and wave where a reduction of each value
// over the 64 lanes takes 18, and those are most of what a Q product issues.
// Fixed order, deterministic; buffers as for bred().
template <int K, int BS, int EPT>
__device__ __forceinline__ void bsum(BShared<BS, EPT>& S, int& par, double (&v)[K]) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  constexpr int H = (K + 1) / 2, Q = (H + 1) / 2;
  double h[H];
#pragma unroll
  for (int i = 0; i < H; ++i) h[i] = swap_add<32>(v[2 * i], 2 * i + 1 < K ? v[2 * i + 1] : 0.0);
#pragma unroll
  for (int j = 0; j < Q; ++j) {
    // rows 0..3 hold values 4 j + 0, 2, 1, 3
    double x = swap_add<16>(h[2 * j], 2 * j + 1 < H ? h[2 * j + 1] : 0.0);
    x = row16_sum(x);
    const int row = lane >> 4, s = 4 * j + ((row & 1) << 1 | row >> 1);
    if ((lane & 15) == 0 && s < K) S.red[par][s][wv] = x;
  }
  __syncthreads();
  combine<K, 0u>(S, par, v);
}

// ---------------------------------------------------------------------------
// the per-instance operator pieces
// ---------------------------------------------------------------------------
// Load of element i of an instance array.  The arrays are in global memory
// but their pointers are read from memory, so plain indexing would give
// generic (flat) loads, which every wait for an LDS access also waits for.
template <class T>
__device__ __forceinline__ T gld(const T* p, long long i) {
  return ((const __attribute__((address_space(1))) T*)p)[i];
}
__device__ __forceinline__ double2 gld(const double2* p, long long i) {
  typedef double v2 __attribute__((ext_vector_type(2)));
  const v2 v = ((const __attribute__((address_space(1))) v2*)p)[i];
  return double2{v.x, v.y};
}

template <int RM, int BS, int EPT>
struct Elem {
  int n, m;
  const double* FT;       // F with rows padded to RM: F(i, k) = FT[i RM + k], zero for k >= r
  const double *c, *L, *U, *dg;
  int tid;                // threadIdx.x, refreshed through an empty asm statement every iteration
  __device__ bool valid(int e) const { return tid + e * BS < n; }
  __device__ int idx(int e) const { return tid + e * BS; }
  // The wave that holds the entries of the vectors of length m (thread row < m).
  // The condition is uniform and its lanes past m compute on zeros: where a
  // divergent branch rejoins with F and the state filling the registers, the
  // compiler has placed a spill before the other lanes were switched on again,
  // which lost their copy of F.
  __device__ bool rows_wave() const { return __builtin_amdgcn_readfirstlane(tid) < HB_MMAX; }
  // Addresses derived from the thread index are then recomputed in every
  // iteration instead of being hoisted out of the solve loop, where they
  // would outnumber the registers and be spilled.
  __device__ void refresh() {
    int t = (int)threadIdx.x;
    asm volatile("" : "+v"(t));
    tid = t;
  }
};

// The rows of F that a thread owns, read from the library's copy of F with
// rows padded to RM entries (16-byte loads at fixed offsets from one address
// per entry).  REG: loaded once into registers, so that the products of the
// iteration read nothing from memory.  Otherwise read at every product.
template <int RM, int EPT, bool REG>
struct QRows {
  static constexpr bool regs = REG;
  double f[REG ? EPT : 1][REG ? RM : 2];
  // (the base address passes through an empty asm statement so that the
  // compiler cannot move the loads above the point of the call, which would
  // keep the copy live across a check)
  template <int BS>
  __device__ void load(const Elem<RM, BS, EPT>& E) {
    if constexpr (REG) {
      const double* FT = E.FT;
      asm volatile("" : "+s"(FT));
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const bool ok = E.valid(e);
        const double2* fr = reinterpret_cast<const double2*>(FT + (size_t)(ok ? E.idx(e) : 0) * RM);
#pragma unroll
        for (int k = 0; k < RM / 2; ++k) {
          const double2 v = gld(fr, k);
          f[e][2 * k] = ok ? v.x : 0.0;
          f[e][2 * k + 1] = ok ? v.y : 0.0;
        }
      }
    }
  }
  template <int BS>
  __device__ __forceinline__ double2 row2(const Elem<RM, BS, EPT>& E, int e, int k) const {
    if constexpr (REG) return double2{f[e][2 * k], f[e][2 * k + 1]};
    else return gld(reinterpret_cast<const double2*>(E.FT + (size_t)(E.valid(e) ? E.idx(e) : 0) * RM), k);
  }
};

// c, L, U and diag(d) of the thread's entries (zeros past n)
template <int RM, int BS, int EPT>
__device__ __forceinline__ void load_clu(const BLds& D, const Elem<RM, BS, EPT>& E, double (&c)[EPT], double (&L)[EPT],
                                         double (&U)[EPT]) {
  if (__builtin_expect(D.clu_in, 1)) {
#pragma unroll
    for (int e = 0; e < EPT; ++e) { c[e] = D.c[E.idx(e)]; L[e] = D.L[E.idx(e)]; U[e] = D.U[E.idx(e)]; }
  } else {
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const bool ok = E.valid(e);
      const int i = ok ? E.idx(e) : 0;
      const double ci = gld(E.c, i), Li = gld(E.L, i), Ui = gld(E.U, i);
      c[e] = ok ? ci : 0.0; L[e] = ok ? Li : 0.0; U[e] = ok ? Ui : 0.0;
    }
  }
}
template <int RM, int BS, int EPT>
__device__ __forceinline__ void load_dg(const BLds& D, const Elem<RM, BS, EPT>& E, double (&dg)[EPT]) {
  if (__builtin_expect(D.clu_in, 1)) {
#pragma unroll
    for (int e = 0; e < EPT; ++e) dg[e] = D.dg[E.idx(e)];
  } else {
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const double v = gld(E.dg, E.valid(e) ? E.idx(e) : 0);
      dg[e] = E.valid(e) ? v : 0.0;
    }
  }
}

// q = Q p = diag(d) p + F (F^T p); p is 0 past n (there the rows in registers
// are zeros, and row 0 is read from memory)
template <int RM, bool REG, int BS, int EPT>
__device__ __forceinline__ void q_apply(BShared<BS, EPT>& S, int& par, const BLds& D, const Elem<RM, BS, EPT>& E,
                                        const QRows<RM, EPT, REG>& Fq, const double (&p)[EPT], double (&q)[EPT]) {
  static_assert(RM % 2 == 0, "rows are read in pairs");
  double t[RM];
#pragma unroll
  for (int k = 0; k < RM; ++k) t[k] = 0.0;
#pragma unroll
  for (int e = 0; e < EPT; ++e)
#pragma unroll
    for (int k = 0; k < RM / 2; ++k) {
      const double2 v = Fq.row2(E, e, k);
      t[2 * k] += v.x * p[e];
      t[2 * k + 1] += v.y * p[e];
    }
  bsum<RM>(S, par, t);
  double dg[EPT];
  load_dg(D, E, dg);
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    double s = dg[e] * p[e];
#pragma unroll
    for (int k = 0; k < RM / 2; ++k) {
      const double2 v = Fq.row2(E, e, k);
      s += v.x * t[2 * k];
      s += v.y * t[2 * k + 1];
    }
    q[e] = REG || E.valid(e) ? s : 0.0;
  }
}

// Pieces of the rows of A for a_apply, of `piece` nonzeros (thread 0, once per instance).
template <int BS, int EPT>
__device__ void a_pieces(BShared<BS, EPT>& S, const BInst& I, int piece) {
  int q = 0;
  for (int r = 0; r < I.m; ++r) {
    S.pstart[r] = q;
    S.arp[r] = I.arp[r];
    const int len = I.arp[r + 1] - I.arp[r];
    for (int c = 0; c * piece < len; ++c) S.prow[q++] = (unsigned char)r;
  }
  for (int r = I.m; r <= HB_MMAX; ++r) S.pstart[r] = q;
  S.arp[I.m] = I.m > 0 ? I.arp[I.m] : 0;
  S.np = q;
}

// (A p)_row for thread row < m (0 for the other threads), p staged through
// D.vm.  The waves share the pieces of all rows (a dense row does not serialise
// on one wave); thread row < m then adds its row's pieces in order.
template <int RM, int BS, int EPT>
__device__ __forceinline__ double a_apply(BShared<BS, EPT>& S, const BLds& D, const Elem<RM, BS, EPT>& E,
                                          const BInst& I, const double (&p)[EPT]) {
  constexpr int WAVES = BCfg<BS, EPT>::WAVES;
#pragma unroll
  for (int e = 0; e < EPT; ++e) D.vm[E.idx(e)] = p[e];
  __syncthreads();
  if (__builtin_expect(D.a_in, 1)) {
    // 16 lanes per piece, four entries a lane
    const int l = E.tid & 15;
    for (int q = E.tid >> 4; q < S.np; q += BS / 16) {
      const int row = S.prow[q], b = S.arp[row] + (q - S.pstart[row]) * HB_LPIECE;
      const int en = min(S.arp[row + 1], b + HB_LPIECE);
      double v[4], x[4];
      int c[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = min(b + l + 16 * u, en - 1);
        v[u] = D.av[k];
        c[u] = D.ac[k];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = D.vm[c[u]];
      double s = 0.0;
#pragma unroll
      for (int u = 0; u < 4; ++u) s += v[u] * (b + l + 16 * u < en ? x[u] : 0.0);
      s = row16_sum(s);
      if (l == 0) D.part[q] = s;
    }
  } else {
    // a wave takes pieces q0 and q0 + WAVES together (loads of both in
    // flight); each piece's sum is formed as for one piece at a time
    const int lane = E.tid & 63, wv = __builtin_amdgcn_readfirstlane(E.tid >> 6), np = S.np;
    constexpr int U = HB_APIECE / 64;
    const double* aval = I.aval;
    const int* aci = I.aci;
    asm volatile("" : "+s"(aval), "+s"(aci));   // (no addresses kept for this path)
    for (int q0 = wv; q0 < np; q0 += 2 * WAVES) {
      double av[2][U];
      int ac[2][U], left[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int q = min(q0 + h * WAVES, np - 1), row = S.prow[q];
        const int b = S.arp[row] + (q - S.pstart[row]) * HB_APIECE + lane, e = min(S.arp[row + 1], b - lane + HB_APIECE);
        left[h] = e - b;   // entry u is the piece's if 64 u < left
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int k = min(b + 64 * u, e - 1);
          av[h][u] = gld(aval, k);
          ac[h][u] = gld(aci, k);
        }
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        double s = 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u) s += av[h][u] * (64 * u < left[h] ? D.vm[ac[h][u]] : 0.0);
        s = wave_reduce63<false>(s);   // exact in lane 63
        const int q = q0 + h * WAVES;
        if (lane == 63 && q < np) D.part[q] = s;
      }
    }
  }
  __syncthreads();
  double s = 0.0;
  if (E.rows_wave()) {
    const int q1 = S.pstart[E.tid + 1];
    for (int q = S.pstart[E.tid]; q < q1; q += 8) {
      double t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) t[u] = D.part[min(q + u, q1 - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += q + u < q1 ? t[u] : 0.0;
    }
  }
  return s;
}

// g = A^T yv (yv in LDS, length m); tb/te: the entries' ranges in A^T,
// loaded once per instance.  The thread's entries advance together,
// two or three nonzeros per step, so that their loads are in flight at the same
// time (each entry's sum still runs over its nonzeros in order).
template <int RM, int BS, int EPT>
__device__ __forceinline__ void at_apply(const BLds& D, const Elem<RM, BS, EPT>& E, const BInst& I,
                                         const int (&tb)[EPT], const int (&te)[EPT], const double* yv,
                                         double (&g)[EPT]) {
  int len = 0;
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    g[e] = 0.0;
    len = max(len, te[e] - tb[e]);
  }
  constexpr int J = EPT == 4 ? 2 : 3;   // (three more nonzeros of four entries would spill)
  if (__builtin_expect(D.a_in, 1)) {
    for (int j = 0; j < len; j += J) {
      unsigned c[EPT][J];
#pragma unroll
      for (int e = 0; e < EPT; ++e)
#pragma unroll
        for (int u = 0; u < J; ++u) c[e][u] = D.tq[max(min(tb[e] + j + u, te[e] - 1), 0)];   // (past the end: read, never used)
      double v[EPT][J], yq[EPT][J];
#pragma unroll
      for (int e = 0; e < EPT; ++e)
#pragma unroll
        for (int u = 0; u < J; ++u) { v[e][u] = D.av[c[e][u] >> 8]; yq[e][u] = yv[c[e][u] & 255u]; }
#pragma unroll
      for (int e = 0; e < EPT; ++e)
#pragma unroll
        for (int u = 0; u < J; ++u) g[e] += v[e][u] * (tb[e] + j + u < te[e] ? yq[e][u] : 0.0);
    }
    return;
  }
  const double* tval = I.tval;
  const int* tci = I.tci;
  asm volatile("" : "+s"(tval), "+s"(tci));   // (no addresses kept for this path)
  for (int j = 0; j < len; j += J) {
    double v[EPT][J];
    int c[EPT][J];
#pragma unroll
    for (int e = 0; e < EPT; ++e)
#pragma unroll
      for (int u = 0; u < J; ++u) {
        const int k = max(min(tb[e] + j + u, te[e] - 1), 0);
        v[e][u] = gld(tval, k);
        c[e][u] = gld(tci, k);
      }
#pragma unroll
    for (int e = 0; e < EPT; ++e)
#pragma unroll
      for (int u = 0; u < J; ++u) g[e] += v[e][u] * (tb[e] + j + u < te[e] ? yv[c[e][u]] : 0.0);
  }
}

__device__ double golden_sigma_dev(double th1, double th2, double th3, double lamQ) {
  const double hi = sqrt(th2 / th1);
  if (th3 <= 0.0 || lamQ <= 0.0) return hi;
  const double lo = sqrt(th2 / (th1 + th3 / lamQ));
  double a = log(lo), b = log(hi);
  const double gr = 0.5 * (sqrt(5.0) - 1.0);
  const double stop = log1p(1e-12);
  for (int it = 0; it < 200 && (b - a) > stop; ++it) {
    const double p = b - gr * (b - a), q = a + gr * (b - a);
    const double sp = exp(p), sq = exp(q);
    const double slope = th1 - th2 / (sp * sq) + th3 * (sp + sq + lamQ * sp * sq) / ((1.0 + lamQ * sp) * (1.0 + lamQ * sq));
    if (slope > 0.0) b = q;
    else a = p;
  }
  return exp(0.5 * (a + b));
}

// Stopping test, restart criteria (Section 3.2) and the sigma update of
// Algorithm 5 at a check; thread 0 only, results in S.T.  Kept out of
// line: it runs once per check and its golden section needs registers the
// iteration does not.
template <int BS, int EPT>
__device__ __noinline__ void check_decision(BShared<BS, EPT>& S, long long t, long long k) {
  // (read from the LDS copy: a reference to the kernel argument itself would
  // make the compiler keep a copy of it in scratch memory)
  const BOpts& o = S.opt;
  BState& T = S.T;
  const double R = T.R;
  const double kkt = fmax(T.eta_p, fmax(T.eta_d, T.eta_gap));
  int tm = -1, rs = 0;
  if (isnan(kkt) || isnan(R)) tm = HPRQP_NUMERICAL;
  else if (kkt <= o.tol) tm = HPRQP_SOLVED;
  else if (k >= o.max_iter) tm = HPRQP_MAX_ITER;
  else if (o.time_ticks > 0 && (long long)(wall_clock64() - *o.t0) >= o.time_ticks) tm = HPRQP_TIME_LIMIT;
  else if (o.enable_restart) {
    const bool c1 = R <= o.alpha1 * T.Rr0;                                    // eq:restart_1
    const bool c2 = T.Rprev >= 0.0 && R <= o.alpha2 * T.Rr0 && R > T.Rprev;   // eq:restart_2
    const bool c3 = (double)t >= T.alpha3 * (double)k;                        // eq:restart_3
    rs = c1 || c2 || c3;
  }
  if (tm < 0 && rs) {
    if (T.R0ref < 0.0) T.R0ref = R;
    const double ratio = R / T.R0ref;
    if (o.enable_sigma_update) {
      // Algorithm 5
      double th1 = T.lamA * T.th[0] + T.lamQ * T.th[1] - 2.0 * T.th[2];
      double th2 = T.th[3], th3 = T.th[4];
      th1 = fmax(th1, 1e-12); th2 = fmax(th2, 1e-12); th3 = fmax(th3, 0.0);
      const double snew = golden_sigma_dev(th1, th2, th3, T.lamQ);
      const double beta = exp(-ratio);
      T.sigma = exp(beta * log(snew) + (1.0 - beta) * log(T.sigma));
      T.derive();
    }
    if (ratio <= 0.1) T.alpha3 = 0.2;
  }
  T.Rprev = R;
  T.term = tm; T.restart = rs;
}

// ---------------------------------------------------------------------------
// persistent kernel (RM: largest rank of F handled, F rows padded with zeros)
// ---------------------------------------------------------------------------
template <int RM, int BS, int EPT>
__global__ __launch_bounds__(BS, (BCfg<BS, EPT>::MIN_WAVES)) void k_batch_solve(
    const BInst* __restrict__ insts, const int* __restrict__ order, int count, int* __restrict__ queue, BOpts o,
    const double* __restrict__ y0, const double* __restrict__ w0, const double* __restrict__ x0,
    double* __restrict__ yo, double* __restrict__ zo, double* __restrict__ wo, double* __restrict__ xo,
    BInfo* __restrict__ infos, double* __restrict__ hbuf, int lds) {
  constexpr int NM = BCfg<BS, EPT>::NMAX;
  __shared__ BShared<BS, EPT> S;
  extern __shared__ double dyn[];
  int par = 0;
  if (threadIdx.x == 0) S.opt = o;   // read after the queue's barriers below
  // the block's check buffer: xbar, wbar, Q wbar, A^T ybar, zbar (entries owned per thread)
  double* const Hx = hbuf + (size_t)blockIdx.x * 5 * NM;
  double* const Hw = Hx + NM;
  double* const HQw = Hx + 2 * NM;
  double* const Hg = Hx + 3 * NM;
  double* const Hz = Hx + 4 * NM;
  for (;;) {
    if (threadIdx.x == 0) S.inst = atomicAdd(queue, 1);
    __syncthreads();
    const int qi = S.inst;
    __syncthreads();
    if (qi >= count) break;                        // every wave leaves together
    const int ii = order[qi];
    const BInst I = insts[ii];
    Elem<RM, BS, EPT> E;
    E.n = I.n; E.m = I.m; E.FT = I.FT;
    E.c = I.c; E.L = I.L; E.U = I.U; E.dg = I.dg;
    E.refresh();
    const int n = I.n, m = I.m;
    int tid = E.tid;
    if (E.rows_wave()) { S.l[tid] = tid < m ? I.l[tid] : 0.0; S.u[tid] = tid < m ? I.u[tid] : 0.0; }
    BLds D;
    {
      const BPlan P = batch_plan(NM, n, m, I.annz, (size_t)lds);
      D.a_in = P.a_in; D.clu_in = P.clu_in;
      D.vm = dyn; D.part = D.vm + NM; D.av = D.part + P.part;
      const int nz = P.a_in ? (int)I.annz : 0;
      D.c = D.av + nz; D.L = D.c + NM; D.U = D.L + NM; D.dg = D.U + NM;
      D.tq = (unsigned*)(P.clu_in ? D.dg + NM : D.c);
      D.ac = (unsigned short*)(D.tq + nz);
      for (int q = tid; q < nz; q += BS) {
        D.av[q] = gld(I.aval, q); D.ac[q] = (unsigned short)gld(I.aci, q);
        D.tq[q] = (unsigned)gld(I.tperm, q) << 8 | (unsigned)gld(I.tci, q);
      }
      if (P.clu_in)
        for (int q = tid; q < NM; q += BS) {
          const bool ok = q < n;
          D.c[q] = ok ? gld(I.c, q) : 0.0; D.L[q] = ok ? gld(I.L, q) : 0.0;
          D.U[q] = ok ? gld(I.U, q) : 0.0; D.dg[q] = ok ? gld(I.dg, q) : 0.0;
        }
    }
    if (tid == 0) a_pieces(S, I, D.a_in ? HB_LPIECE : HB_APIECE);
    QRows<RM, EPT, false> Fg;   // F from memory: checks (rare)
    int tb[EPT], te[EPT];       // A^T ranges of the thread's entries (empty when invalid)
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const int i = E.idx(e);
      tb[e] = i < n ? gld(I.trp, i) : 0;
      te[e] = i < n ? gld(I.trp, i + 1) : 0;
    }
    // F in registers for the power method and the iteration; not live across a
    // check, which reads F from memory and loads this copy again when it is done
    QRows<RM, EPT, (RM <= 10 || EPT <= 2)> Fq;
    Fq.load(E);
    __syncthreads();

    // ---- lambda_Q: power method on Q from the all-ones start (Section 4.1) ----
    double lamQ = o.lamQ, lamA = o.lamA;
    if (!(lamQ > 0.0)) {
      // One reduction per product: with t = F^T p at hand, q = Q p is formed
      // entry by entry and F^T q, <p, q> and <q, q> are summed together; the
      // next t is F^T q / ||q||.
      double pv[EPT], t[RM], dg[EPT];
      const double s0 = 1.0 / sqrt((double)n);
#pragma unroll
      for (int k = 0; k < RM; ++k) t[k] = 0.0;
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        pv[e] = E.valid(e) ? s0 : 0.0;
#pragma unroll
        for (int k = 0; k < RM / 2; ++k) {
          const double2 f = Fq.row2(E, e, k);
          t[2 * k] += f.x * pv[e];
          t[2 * k + 1] += f.y * pv[e];
        }
      }
      bsum<RM>(S, par, t);
      load_dg(D, E, dg);
      double lam = 0.0, lam_old = 0.0;
      for (int it = 1; it <= 5000; ++it) {
        double rr[RM + 2];
#pragma unroll
        for (int k = 0; k < RM + 2; ++k) rr[k] = 0.0;
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
          double f[RM];
          double qe = dg[e] * pv[e];
#pragma unroll
          for (int k = 0; k < RM / 2; ++k) {
            const double2 v = Fq.row2(E, e, k);
            f[2 * k] = v.x; f[2 * k + 1] = v.y;
            qe += v.x * t[2 * k];
            qe += v.y * t[2 * k + 1];
          }
          if (!Fq.regs) qe = E.valid(e) ? qe : 0.0;
#pragma unroll
          for (int k = 0; k < RM; ++k) rr[k] += f[k] * qe;
          rr[RM] += pv[e] * qe; rr[RM + 1] += qe * qe;
          pv[e] = qe;
        }
        bsum<RM + 2>(S, par, rr);
        lam = rr[RM];
        if (rr[RM + 1] == 0.0) break;
        if (it > 1 && fabs(lam - lam_old) <= 1e-6 * fabs(lam)) break;
        lam_old = lam;
        const double sc = 1.0 / sqrt(rr[RM + 1]);
#pragma unroll
        for (int e = 0; e < EPT; ++e) pv[e] *= sc;
#pragma unroll
        for (int k = 0; k < RM; ++k) t[k] = rr[k] * sc;
      }
      lamQ = 1.01 * lam;
    }
    // ---- lambda_A: power method on A A^T from the all-ones start ----
    if (!(lamA > 0.0) && m > 0) {
      double pv[EPT];
      if (tid < m) S.pw[tid] = 1.0 / sqrt((double)m);
      __syncthreads();
      double lam = 0.0, lam_old = 0.0;
      for (int it = 1; it <= 5000; ++it) {
        at_apply(D, E, I, tb, te, S.pw, pv);          // u = A^T v
        const double au = a_apply(S, D, E, I, pv);    // w = A u (row tid)
        double rr[2] = {0.0, 0.0};
        if (tid < m) { rr[0] = S.pw[tid] * au; rr[1] = au * au; }
        bsum<2>(S, par, rr);
        lam = rr[0];
        if (rr[1] == 0.0) break;
        if (it > 1 && fabs(lam - lam_old) <= 1e-6 * fabs(lam)) break;
        lam_old = lam;
        if (tid < m) S.pw[tid] = au / sqrt(rr[1]);
        __syncthreads();
      }
      lamA = 1.01 * lam;
    }
    // ---- sigma0 = ||b|| / ||c|| (Section 4.1); ||b||_inf, ||c||_inf ----
    double nrm[4] = {0.0, 0.0, 0.0, 0.0};
    if (tid < m) {
      const double a = isinf(S.l[tid]) ? 0.0 : fabs(S.l[tid]), b = isinf(S.u[tid]) ? 0.0 : fabs(S.u[tid]);
      const double bi = fmax(a, b);
      nrm[0] = bi * bi; nrm[1] = bi;
    }
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const double ce = E.valid(e) ? gld(E.c, E.idx(e)) : 0.0;
      nrm[2] += ce * ce; nrm[3] = fmax(nrm[3], fabs(ce));
    }
    bred<0xAu>(S, par, nrm);
    // the state of the checks (thread 0 alone writes it, between barriers)
    if (tid == 0) {
      const double nb = sqrt(nrm[0]), nc = sqrt(nrm[2]);
      BState& T = S.T;
      T.binf = nrm[1]; T.cinf = nrm[3];
      if (o.sigma0 > 0.0) T.sigma = o.sigma0;
      else if (nb >= 1e-16 && nb <= 1e16 && nc >= 1e-16 && nc <= 1e16) T.sigma = nb / nc;
      else T.sigma = 1.0;
      T.sigma0 = T.sigma;
      T.lamA = lamA; T.lamQ = lamQ;
      T.alpha3 = o.alpha3; T.R0ref = -1.0; T.Rr0 = -1.0; T.Rprev = -1.0; T.R = 0.0;
      T.eta_p = T.eta_d = T.eta_gap = T.pobj = T.dobj = 0.0;
      T.derive();
    }

    // ---- state: origin or warm start ----
    // iterate u^{r,t} = (x, w) of the thread's entries with the images Q w and
    // A^T y kept by linearity, and the Halpern anchors u^{r,0} with theirs
    double xs[EPT], ws[EPT], Qws[EPT], ATys[EPT], xa[EPT], wa[EPT], Qwa[EPT], ATya[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const int i = E.idx(e);
      const bool ok = i < n;
      xs[e] = (ok && x0) ? x0[I.off_n + i] : 0.0;
      ws[e] = (ok && w0) ? w0[I.off_n + i] : 0.0;
    }
    if (E.rows_wave()) S.y[tid] = y0 && tid < m ? y0[I.off_m + tid] : 0.0;
    __syncthreads();
    // sigma and its derived values, uniform; they change at checks only
    double sigma = readlane_d(S.T.sigma, 0), sQ = readlane_d(S.T.sQ, 0), inv = readlane_d(S.T.inv, 0);
    double kappa = readlane_d(S.T.kappa, 0), sA = readlane_d(S.T.sA, 0);
    long long k = 0, t = 0;
    int r = 0, term = -1, left = o.check_every;   // iterations up to the next check
    bool new_epoch = true;
    while (term < 0) {
      E.refresh();
      tid = E.tid;
      if (__builtin_expect(new_epoch, 0)) {
        // anchor u^{r,0} = u; exact A^T y and Q w
        if (E.rows_wave()) S.ya[tid] = S.y[tid];
        __syncthreads();
        at_apply(D, E, I, tb, te, S.y, ATys);
        q_apply(S, par, D, E, Fq, ws, Qws);
#pragma unroll
        for (int e = 0; e < EPT; ++e) { xa[e] = xs[e]; wa[e] = ws[e]; Qwa[e] = Qws[e]; ATya[e] = ATys[e]; }
        t = 0;
        new_epoch = false;
      }
      const double rho = 1.0 / (double)(t + 2);
      left -= 1;
      const bool is_check = left == 0 || k + 1 >= o.max_iter;
      const bool want_r = (t == 0) || is_check;
      // z/x step ("update-z", "update-x"); zbar itself is formed at checks only
      // (everything past n is and stays zero)
      double xh[EPT], xb[EPT];
      {
        double ce[EPT], Le[EPT], Ue[EPT];
        load_clu(D, E, ce, Le, Ue);
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
          const double rz = xs[e] + sigma * (-Qws[e] + ATys[e] - ce[e]);
          xb[e] = clampd(rz, Le[e], Ue[e]);
          xh[e] = 2.0 * xb[e] - xs[e];
        }
      }
      // Q xhat, v = xhat + kappa (Qw - Q xhat)
      double q1[EPT];
      q_apply(S, par, D, E, Fq, xh, q1);
      // y step ("update-y") and its Halpern update
      double dy2 = 0.0, th_y = 0.0;
      if (m > 0) {
        double v[EPT];
#pragma unroll
        for (int e = 0; e < EPT; ++e) v[e] = xh[e] + kappa * (Qws[e] - q1[e]);
        const double av = a_apply(S, D, E, I, v);
        if (E.rows_wave()) {
          const double yi = S.y[tid], yai = S.ya[tid];
          const double rr = av - sA * yi;
          const double ybv = (clampd(rr, S.l[tid], S.u[tid]) - rr) / sA;
          S.yb[tid] = ybv;
          dy2 = tid < m ? (yi - ybv) * (yi - ybv) : 0.0;
          th_y = tid < m ? (ybv - yai) * (ybv - yai) : 0.0;
          S.yn[tid] = rho * yai + (1.0 - rho) * (2.0 * ybv - yi);   // Halpern y+ (applied below)
        }
        __syncthreads();
      }
      // g = A^T ybar, d = A^T(ybar - y)
      double d[EPT], g[EPT];
      at_apply(D, E, I, tb, te, S.yb, g);
#pragma unroll
      for (int e = 0; e < EPT; ++e) d[e] = m > 0 ? g[e] - ATys[e] : 0.0;
      double q2[EPT];
      q_apply(S, par, D, E, Fq, d, q2);
      // wbar ("update-w") and Q wbar
      double wb[EPT], Qwb[EPT];
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        asm volatile("" : "+v"(xb[e]));   // xhat again, from xbar: not kept over the second product
        wb[e] = (sQ * ws[e] + (2.0 * xb[e] - xs[e])) * inv + kappa * d[e];
        Qwb[e] = (sQ * Qws[e] + q1[e]) * inv + kappa * q2[e];
      }
      // merit R~ = ||u - ubar||_M (theta decomposition of the metric of Algorithm 3)
      if (__builtin_expect(want_r, 0)) {
        double s7[7] = {dy2, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
          const double dw = ws[e] - wb[e], Qdw = Qws[e] - Qwb[e], ATdy = -d[e], QATdy = -q2[e];
          const double dx = xs[e] - xb[e];
          s7[1] += dw * Qdw; s7[2] += Qdw * ATdy; s7[3] += dx * dx;
          s7[4] += ATdy * QATdy; s7[5] += ATdy * dx; s7[6] += Qdw * dx;
        }
        bsum<7>(S, par, s7);
        if (tid == 0) {
          const double th1 = S.T.lamA * s7[0] + S.T.lamQ * s7[1] - 2.0 * s7[2];
          const double m2 = sigma * th1 + s7[3] / sigma + sigma * sigma * s7[4] / (1.0 + sQ) + 2.0 * (s7[5] - s7[6]);
          const double R = sqrt(m2 > 0.0 ? m2 : 0.0);
          S.T.R = R;
          if (t == 0) { S.T.Rr0 = R; S.T.Rprev = -1.0; }
        }
      }
      t += 1; k += 1;
      if (__builtin_expect(!is_check, 1)) {
        // Halpern step: u^{r,t+1} = rho u^{r,0} + (1 - rho)(2 ubar - u)
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
          xs[e] = rho * xa[e] + (1.0 - rho) * (2.0 * xb[e] - xs[e]);
          ws[e] = rho * wa[e] + (1.0 - rho) * (2.0 * wb[e] - ws[e]);
          Qws[e] = rho * Qwa[e] + (1.0 - rho) * (2.0 * Qwb[e] - Qws[e]);
          ATys[e] = m > 0 ? rho * ATya[e] + (1.0 - rho) * (2.0 * g[e] - ATys[e]) : 0.0;
        }
        // (read by this thread alone until the barrier of a new epoch; the next
        // y step's LDS writes are two barriers behind the readers of this one's)
        if (E.rows_wave()) S.y[tid] = S.yn[tid];
        continue;
      }

      // ---- check iteration (every check_every iterations): the bar values go
      // to the block's buffer H so that the registers of the loop above are
      // free for the stopping test and Algorithm 5
      left = o.check_every;
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const int i = E.idx(e);
        Hx[i] = xb[e]; Hw[i] = wb[e]; HQw[i] = Qwb[e]; Hg[i] = g[e];
      }
      // theta~ of Algorithm 5: D = ubar - u^{r,0}; e = A^T (ybar - y_a) = g - ATy_a
      {
        double th[5] = {th_y, 0, 0, 0, 0};
        double ev[EPT], Qe[EPT];
#pragma unroll
        for (int e = 0; e < EPT; ++e) ev[e] = m > 0 ? Hg[E.idx(e)] - ATya[e] : 0.0;
        q_apply(S, par, D, E, Fg, ev, Qe);
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
          const int i = E.idx(e);
          const double Dw = Hw[i] - wa[e], QDw = HQw[i] - Qwa[e];
          const double Dx = Hx[i] - xa[e];
          th[1] += Dw * QDw; th[2] += QDw * ev[e]; th[3] += Dx * Dx; th[4] += ev[e] * Qe[e];
        }
        bsum<5>(S, par, th);
        if (tid == 0)
#pragma unroll
          for (int q = 0; q < 5; ++q) S.T.th[q] = th[q];
      }
      // stopping quantities at (ybar, zbar, xbar) (Section 4.1), with
      // zbar = (xbar - r_z) / sigma formed here
      {
        double res[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
        double xbv[EPT], Qx[EPT];
#pragma unroll
        for (int e = 0; e < EPT; ++e) xbv[e] = Hx[E.idx(e)];
        q_apply(S, par, D, E, Fg, xbv, Qx);
        const double ax = m > 0 ? a_apply(S, D, E, I, xbv) : 0.0;   // (A xbar)_tid
        // res: 0 max|Ax-PiK|, 1 max|Ax|, 2 sum(l y+ + u y-), 3 #inf, 4 max|dual|, 5 max|g|, 6 max|Qx|,
        //      7 <x,Qx>, 8 <c,x>, 9 sum(L z+ + U z-) (+ #inf folded into 3)
        if (tid < m) {
          const double li = S.l[tid], ui = S.u[tid], yv = S.yb[tid];
          res[0] = fabs(ax - clampd(ax, li, ui));
          res[1] = fabs(ax);
          if (yv > 0.0) { if (isinf(li)) res[3] += 1.0; else res[2] += li * yv; }
          else if (yv < 0.0) { if (isinf(ui)) res[3] += 1.0; else res[2] += ui * yv; }
        }
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
          if (!E.valid(e)) continue;
          const int i = E.idx(e);
          const double ce = gld(E.c, i), Le = gld(E.L, i), Ue = gld(E.U, i), ge = Hg[i];
          const double rz = xs[e] + sigma * (-Qws[e] + ATys[e] - ce);
          const double zbe = (xbv[e] - rz) / sigma;
          Hz[i] = zbe;
          res[4] = fmax(res[4], fabs(-Qx[e] + ge + zbe - ce));
          res[5] = fmax(res[5], fabs(ge));
          res[6] = fmax(res[6], fabs(Qx[e]));
          res[7] += xbv[e] * Qx[e];
          res[8] += ce * xbv[e];
          if (zbe > 0.0) { if (isinf(Le)) res[3] += 1.0; else res[9] += Le * zbe; }
          else if (zbe < 0.0) { if (isinf(Ue)) res[3] += 1.0; else res[9] += Ue * zbe; }
        }
        bred<0x73u>(S, par, res);               // maxes: 0, 1, 4, 5, 6
        // decisions (thread 0, FP64), broadcast through LDS
        if (tid == 0) {
          BState& T = S.T;
          T.eta_p = m > 0 ? res[0] / (1.0 + fmax(T.binf, res[1])) : 0.0;
          T.eta_d = res[4] / (1.0 + fmax(T.cinf, fmax(res[5], res[6])));
          T.pobj = 0.5 * res[7] + res[8];
          if (res[3] > 0.0) { T.dobj = -INFINITY; T.eta_gap = INFINITY; }
          else {
            T.dobj = -0.5 * res[7] + res[2] + res[9];
            T.eta_gap = fabs(T.pobj - T.dobj) / (1.0 + fmax(fabs(T.pobj), fabs(T.dobj)));
          }
          check_decision(S, t, k);
        }
      }
      __syncthreads();
      term = S.T.term;
      const int restart = S.T.restart;
      const double rho1 = rho;
      sigma = readlane_d(S.T.sigma, 0); sQ = readlane_d(S.T.sQ, 0); inv = readlane_d(S.T.inv, 0);
      kappa = readlane_d(S.T.kappa, 0); sA = readlane_d(S.T.sA, 0);
      __syncthreads();
      if (term >= 0) {
        // output ubar of the last iteration (Algorithm 4, "Output")
        for (int e = 0; e < EPT; ++e) {
          const int i = E.idx(e);
          if (i < n) {
            xo[I.off_n + i] = Hx[i];
            zo[I.off_n + i] = Hz[i];
            wo[I.off_n + i] = Hw[i];
          }
        }
        break;
      }
      if (restart) {
        // u^{r+1,0} = ubar
#pragma unroll
        for (int e = 0; e < EPT; ++e) { xs[e] = Hx[E.idx(e)]; ws[e] = Hw[E.idx(e)]; }
        if (E.rows_wave()) S.y[tid] = S.yb[tid];
        r += 1;
        new_epoch = true;
      } else {
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
          const int i = E.idx(e);
          xs[e] = rho1 * xa[e] + (1.0 - rho1) * (2.0 * Hx[i] - xs[e]);
          ws[e] = rho1 * wa[e] + (1.0 - rho1) * (2.0 * Hw[i] - ws[e]);
          Qws[e] = rho1 * Qwa[e] + (1.0 - rho1) * (2.0 * HQw[i] - Qws[e]);
          ATys[e] = m > 0 ? rho1 * ATya[e] + (1.0 - rho1) * (2.0 * Hg[i] - ATys[e]) : 0.0;
        }
        if (E.rows_wave()) S.y[tid] = S.yn[tid];
      }
      __syncthreads();
      Fq.load(E);
    }
    if (tid < m) yo[I.off_m + tid] = S.yb[tid];
    if (tid == 0) {
      const BState& T = S.T;
      BInfo f;
      f.term = term; f.restarts = r; f.iters = k; f.sigma = T.sigma; f.sigma0 = T.sigma0;
      f.lamA = T.lamA; f.lamQ = T.lamQ; f.eta_p = T.eta_p; f.eta_d = T.eta_d; f.eta_gap = T.eta_gap;
      f.pobj = T.pobj; f.dobj = T.dobj; f.R_last = T.R;
      infos[ii] = f;
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// setup kernels
// ---------------------------------------------------------------------------
// per-instance validation: bit 0 bounds / non-finite data, bit 1 CSR structure
__global__ void k_batch_validate(const BInst* __restrict__ insts, int count, int* __restrict__ flags) {
  const int ii = blockIdx.x;
  if (ii >= count) return;
  const BInst I = insts[ii];
  __shared__ int sflag;
  if (threadIdx.x == 0) sflag = 0;
  __syncthreads();
  int f = 0;
  for (int i = threadIdx.x; i < I.n; i += blockDim.x) {
    if (!(I.L[i] <= I.U[i]) || I.L[i] == INFINITY || I.U[i] == -INFINITY || !isfinite(I.c[i]) || !isfinite(I.dg[i]))
      f |= 1;
    for (int k = 0; k < I.r; ++k)
      if (!isfinite(I.F[(size_t)i * I.r + k])) f |= 1;
  }
  for (int i = threadIdx.x; i < I.m; i += blockDim.x) {
    if (!(I.l[i] <= I.u[i]) || I.l[i] == INFINITY || I.u[i] == -INFINITY) f |= 1;
    const int b = I.arp[i], e = I.arp[i + 1];
    if ((i == 0 && b != 0) || b < 0 || e < b || (long long)e > I.annz || (i == I.m - 1 && e != I.annz) || e - b > I.n)
      f |= 2;
  }
  if (f) atomicOr(&sflag, f);
  __syncthreads();
  // columns, only once every row pointer lies in [0, nnz]
  if ((sflag & 2) == 0 && I.m > 0) {
    const int nnz = I.arp[I.m];
    int g = 0;
    for (int k = threadIdx.x; k < nnz; k += blockDim.x)
      if (I.aci[k] < 0 || I.aci[k] >= I.n || !isfinite(I.aval[k])) g |= 2;
    if (g) atomicOr(&sflag, g);
  }
  __syncthreads();
  if (threadIdx.x == 0) flags[ii] = sflag;
}

// A^T of one instance per block (rows of A^T ordered by row of A): LDS
// histogram, then one thread scans and scatters in CSR order (deterministic).
__global__ void k_batch_transpose(const BInst* __restrict__ insts, const int* __restrict__ rep, int nrep,
                                  int* __restrict__ trp_all, int* __restrict__ tci_all, int* __restrict__ tperm_all,
                                  double* __restrict__ tval_all, const long long* __restrict__ toff) {
  const int q = blockIdx.x;
  if (q >= nrep) return;
  const BInst I = insts[rep[q]];
  __shared__ int cnt[HB_NMAX + 1];
  for (int i = threadIdx.x; i <= I.n; i += blockDim.x) cnt[i] = 0;
  __syncthreads();
  const int nnz = I.m > 0 ? I.arp[I.m] : 0;
  for (int k = threadIdx.x; k < nnz; k += blockDim.x) atomicAdd(&cnt[I.aci[k] + 1], 1);
  __syncthreads();
  int* trp = trp_all + toff[2 * q];
  int* tci = tci_all + toff[2 * q + 1];
  int* tpm = tperm_all + toff[2 * q + 1];
  double* tv = tval_all + toff[2 * q + 1];
  if (threadIdx.x == 0) {
    for (int i = 0; i < I.n; ++i) cnt[i + 1] += cnt[i];
    for (int i = 0; i <= I.n; ++i) trp[i] = cnt[i];
    for (int row = 0; row < I.m; ++row)
      for (int k = I.arp[row]; k < I.arp[row + 1]; ++k) {
        const int p = cnt[I.aci[k]]++;
        tci[p] = row;
        tpm[p] = k;
        tv[p] = I.aval[k];
      }
  }
}

// F of every instance with rows padded to the kernel's rank RM:
// FT[i RM + k] = F(i, k) for k < r, 0 for r <= k < RM
// (one block per distinct copy: rep lists one instance of each)
__global__ void k_batch_ft(const BInst* __restrict__ insts, const int* __restrict__ rep, int nrep, int RM,
                           double* __restrict__ ft_all, const long long* __restrict__ ft_off) {
  if ((int)blockIdx.x >= nrep) return;
  const int ii = rep[blockIdx.x];
  const BInst I = insts[ii];
  double* ft = ft_all + ft_off[ii];
  const long long tot = (long long)RM * I.n;
  for (long long q = threadIdx.x; q < tot; q += blockDim.x) {
    const int i = (int)(q / RM), k = (int)(q % RM);
    ft[q] = k < I.r ? I.F[(size_t)i * I.r + k] : 0.0;
  }
}

__global__ void k_zero_ints(int* p, int k) {
  if ((int)threadIdx.x < k) p[threadIdx.x] = 0;
}

// the time-limit stamp of a solve
__global__ void k_stamp(long long* t0) {
  if (threadIdx.x == 0) *t0 = (long long)wall_clock64();
}

// ||Q(w - x)||_inf of every instance at its returned point, Q = diag(d) + F F^T
// (the diagnostic of the shadow w_Q of Proposition 2.4): one workgroup per
// instance, t = F^T (w - x) and the maximum by fixed-order reductions
#define HB_QWX_BS 256
__global__ __launch_bounds__(HB_QWX_BS) void k_batch_qwx(const BInst* __restrict__ insts, int count,
                                                          const double* __restrict__ w, const double* __restrict__ x,
                                                          double* __restrict__ out) {
  constexpr int NW = HB_QWX_BS / 64;
  __shared__ double part[16][NW];
  __shared__ double t[16];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int ii = blockIdx.x; ii < count; ii += gridDim.x) {
    const BInst I = insts[ii];
    const double* wi = w + I.off_n;
    const double* xi = x + I.off_n;
    double acc[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) acc[k] = 0.0;
    for (int i = threadIdx.x; i < I.n; i += HB_QWX_BS) {
      const double d = wi[i] - xi[i];
#pragma unroll
      for (int k = 0; k < 16; ++k)
        if (k < I.r) acc[k] += I.F[(size_t)i * I.r + k] * d;
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const double v = wave_sum(acc[k]);
      if (lane == 0) part[k][wv] = v;
    }
    __syncthreads();
    if (threadIdx.x < 16) {
      double v = 0.0;
      for (int q = 0; q < NW; ++q) v += part[threadIdx.x][q];
      t[threadIdx.x] = v;
    }
    __syncthreads();
    double mx = 0.0;
    for (int i = threadIdx.x; i < I.n; i += HB_QWX_BS) {
      double q = I.dg[i] * (wi[i] - xi[i]);
      for (int k = 0; k < I.r; ++k) q += I.F[(size_t)i * I.r + k] * t[k];
      mx = fmax(mx, fabs(q));
    }
    mx = wave_max(mx);
    if (lane == 0) part[0][wv] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
      double v = part[0][0];
      for (int q = 1; q < NW; ++q) v = fmax(v, part[0][q]);
      out[ii] = v;
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// The solve kernels by rank (10 or 16), threads per workgroup and entries per thread.
typedef void (*BKernel)(const BInst*, const int*, int, int*, BOpts, const double*, const double*, const double*,
                        double*, double*, double*, double*, BInfo*, double*, int);
struct BShape {
  BKernel k;
  int bs, ept, cap;   // cap: most dynamic LDS
};
template <int RM, int BS, int EPT>
constexpr BShape bshape() { return {k_batch_solve<RM, BS, EPT>, BS, EPT, BCfg<BS, EPT>::DYN_LDS}; }

struct hprqp_batch {
  int count = 0;
  hipStream_t st = nullptr, own_st = nullptr;
  BOpts o{};
  BInst* d_insts = nullptr;
  int* d_order = nullptr;
  int* d_queue = nullptr;
  int* d_flags = nullptr;
  BInfo* d_infos = nullptr;
  double* d_qwx = nullptr;     // ||Q(w - x)||_inf per instance
  long long* d_t0 = nullptr;   // time-limit stamp
  int *trp = nullptr, *tci = nullptr, *tperm = nullptr;
  double* tval = nullptr;
  long long* d_toff = nullptr;
  int* d_rep = nullptr;
  double* ft = nullptr;        // F of every instance, rows padded to rank_max
  long long* d_ftoff = nullptr;
  int* d_ftrep = nullptr;      // one instance per distinct F
  // one persistent kernel per shape in use: kernel k takes the instances
  // d_order[first, first + cnt) (largest first), on its own stream (kernel 0 on
  // the batch stream); d_queue holds one counter per kernel
  struct Kern {
    const BShape* sh = nullptr;
    int first = 0, cnt = 0, grid = 0;
    size_t lds = 0;            // dynamic LDS
    double* hbuf = nullptr;    // per-block check buffers
    hipStream_t st = nullptr;  // created by the library for kernels 1..
    hipEvent_t ev_join = nullptr;
  } kern[HB_NCLASS];
  int nkern = 0;
  std::vector<int> order_default;   // d_order as built at create
  hipEvent_t ev_fork = nullptr;
  // size classes n <= 256 << c: instances, block size, and (autotuned) the
  // mean kernel time per instance-iteration of each candidate block size
  int class_cnt[HB_NCLASS] = {0, 0, 0, 0};
  int class_bs[HB_NCLASS] = {0, 0, 0, 0};
  double class_us[HB_NCLASS][HB_NCLASS] = {};   // [class][log2(bs / 64)], 0: not timed
  int tuned = 0;
  long long total_n = 0, total_m = 0;
  int rank_max = 0;       // 10 or 16: the kernel instantiation used
  double last_kernel_s = 0.0;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  ~hprqp_batch() {
    void* ps[] = {d_insts, d_order, d_queue, d_flags,   d_infos, trp,     tci,     tperm,
                  tval,    d_toff,  d_rep,   ft,        d_ftoff, d_ftrep, d_qwx,   d_t0};
    for (void* p : ps)
      if (p) hipFree(p);
    for (auto& k : kern) {
      if (k.hbuf) hipFree(k.hbuf);
      if (k.ev_join) hipEventDestroy(k.ev_join);
      if (k.st) hipStreamDestroy(k.st);
    }
    if (e0) hipEventDestroy(e0);
    if (e1) hipEventDestroy(e1);
    if (ev_fork) hipEventDestroy(ev_fork);
    if (own_st) hipStreamDestroy(own_st);
  }
};

namespace {
struct BErr {
  hprqp_status st;
  std::string msg;
};
[[noreturn]] void bfail(hprqp_status st, const std::string& m) { throw BErr{st, m}; }
void bcheck(hipError_t e, const char* what) {
  if (e != hipSuccess) {
    if (e == hipErrorOutOfMemory) bfail(HPRQP_ERR_OOM, std::string(what) + ": out of device memory");
    bfail(HPRQP_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
  }
}
#define HBC(x) bcheck((x), #x)

template <int RM>
const BShape& batch_shape_of(int bs, int ept) {
  static const BShape all[] = {bshape<RM, 64, 4>(),  bshape<RM, 128, 4>(), bshape<RM, 128, 2>(),
                               bshape<RM, 256, 4>(), bshape<RM, 256, 2>(), bshape<RM, 256, 1>(),
                               bshape<RM, 512, 4>(), bshape<RM, 512, 2>(), bshape<RM, 512, 1>()};
  for (const BShape& s : all)
    if (s.bs == bs && s.ept == ept) return s;
  bfail(HPRQP_ERR_HIP, "no batch kernel of this shape");
}
// Size class c (n <= 256 << c) on bs threads: the fewest entries per thread that hold it.
const BShape& batch_shape(int rank, int bs, int c) {
  const int ept = std::max(1, (256 << c) / bs);
  return rank == 10 ? batch_shape_of<10>(bs, ept) : batch_shape_of<16>(bs, ept);
}

// Dynamic LDS of a kernel for the instances `ids`: the largest plan of any.
size_t batch_lds(const BShape& sh, const std::vector<BInst>& hi, const std::vector<int>& ids) {
  size_t need = 0;
  for (int i : ids) need = std::max(need, batch_plan(sh.bs * sh.ept, hi[i].n, hi[i].m, hi[i].annz, (size_t)sh.cap).bytes);
  return (need + 15) / 16 * 16;
}

// Workgroups resident on the device at once.
int batch_resident(const BShape& sh, size_t lds, int ncu) {
  HBC(hipFuncSetAttribute((const void*)sh.k, hipFuncAttributeMaxDynamicSharedMemorySize, sh.cap));
  int per_cu = 0;
  HBC(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)sh.k, sh.bs, lds));
  return ncu * std::max(per_cu, 1);
}

// Launch of a persistent solve kernel.
void batch_launch(const BShape& sh, size_t lds, hipStream_t s, int grid, const BInst* insts, const int* order, int cnt,
                  int* queue, const BOpts& o, const double* y0, const double* w0, const double* x0, double* y,
                  double* z, double* w, double* x, BInfo* infos, double* hbuf) {
  sh.k<<<grid, sh.bs, lds, s>>>(insts, order, cnt, queue, o, y0, w0, x0, y, z, w, x, infos, hbuf, (int)lds);
  HBC(hipGetLastError());
}

// The batched solver's shape autotuner.  For every size class with at least
// 8 instances, each block size that can hold the class (n <= 4 bs) is timed
// on a sample of the class's instances -- evenly spaced over the class, at
// most eight per compute unit, enough to fill the device -- running
// exactly 100 iterations per instance (tolerance 0, lambda's fixed at 1, so
// no power method) into scratch outputs; the default block size is kept
// unless another is at least 5% faster (near ties would otherwise flip
// between runs).  Only the speed is measured: the shapes do not change
// what is computed beyond the order of the block reductions.
void autotune_batch(hprqp_batch* b, const std::vector<BInst>& hi, const std::vector<int> (&cls)[HB_NCLASS], int ncu) {
  BOpts o = b->o;
  o.tol = 0.0; o.max_iter = 100; o.check_every = 100; o.lamA = 1.0; o.lamQ = 1.0; o.sigma0 = 1.0;
  o.time_ticks = 0;
  const long long tn = std::max(1ll, b->total_n), tm = std::max(1ll, b->total_m);
  double *sy = nullptr, *sz = nullptr, *sw = nullptr, *sx = nullptr, *hb = nullptr;
  int *sorder = nullptr, *squeue = nullptr;
  BInfo* sinfo = nullptr;
  hipEvent_t t0 = nullptr, t1 = nullptr;
  const auto cleanup = [&] {
    for (void* p : {(void*)sy, (void*)sz, (void*)sw, (void*)sx, (void*)hb, (void*)sorder, (void*)squeue, (void*)sinfo})
      if (p) hipFree(p);
    if (t0) hipEventDestroy(t0);
    if (t1) hipEventDestroy(t1);
  };
  try {
    HBC(hipMalloc(&sy, tm * sizeof(double)));
    HBC(hipMalloc(&sz, tn * sizeof(double)));
    HBC(hipMalloc(&sw, tn * sizeof(double)));
    HBC(hipMalloc(&sx, tn * sizeof(double)));
    HBC(hipMalloc(&sinfo, b->count * sizeof(BInfo)));
    HBC(hipMalloc(&squeue, sizeof(int)));
    HBC(hipMalloc(&sorder, b->count * sizeof(int)));
    HBC(hipEventCreate(&t0));
    HBC(hipEventCreate(&t1));
    size_t hb_cap = 0;
    for (int c = 0; c < HB_NCLASS; ++c) {
      const int cnt = (int)cls[c].size();
      if (cnt < 8) continue;
      const int want = std::min(cnt, 8 * ncu);
      std::vector<int> sample;
      for (int q = 0; q < want; ++q) sample.push_back(cls[c][(size_t)q * cnt / want]);
      HBC(hipMemcpyAsync(sorder, sample.data(), sample.size() * sizeof(int), hipMemcpyHostToDevice, b->st));
      double best = 0.0;
      int best_bs = b->class_bs[c];
      for (int lb = 0; lb < HB_NCLASS; ++lb) {
        const int bs = 64 << lb;
        if (HB_EPT * bs < (256 << c)) continue;    // cannot hold the class
        const BShape& sh = batch_shape(b->rank_max, bs, c);
        const size_t lds = batch_lds(sh, hi, sample);
        const int grid = std::max(1, std::min(want, batch_resident(sh, lds, ncu)));
        const size_t need = (size_t)grid * 5 * sh.ept * bs;
        if (need > hb_cap) {
          if (hb) HBC(hipFree(hb));
          hb = nullptr;
          HBC(hipMalloc(&hb, need * sizeof(double)));
          hb_cap = need;
        }
        float ms = 0.f;
        for (int rep = 0; rep < 2; ++rep) {   // the first launch loads the code
          k_zero_ints<<<1, 64, 0, b->st>>>(squeue, 1);
          HBC(hipEventRecord(t0, b->st));
          batch_launch(sh, lds, b->st, grid, b->d_insts, sorder, (int)sample.size(), squeue, o, nullptr, nullptr,
                       nullptr, sy, sz, sw, sx, sinfo, hb);
          HBC(hipEventRecord(t1, b->st));
          HBC(hipEventSynchronize(t1));
          HBC(hipEventElapsedTime(&ms, t0, t1));
        }
        const double us = 1e3 * ms / (100.0 * sample.size());   // per instance-iteration
        b->class_us[c][lb] = us;
        if (bs == b->class_bs[c]) best = best > 0.0 ? std::min(best, us) : us;
      }
      // the fastest, unless within 5% of the default
      double dflt = 0.0;
      for (int lb = 0; lb < HB_NCLASS; ++lb)
        if ((64 << lb) == b->class_bs[c]) dflt = b->class_us[c][lb];
      double bu = dflt;
      for (int lb = 0; lb < HB_NCLASS; ++lb) {
        const double us = b->class_us[c][lb];
        if (us > 0.0 && us < 0.95 * dflt && us < bu) { bu = us; best_bs = 64 << lb; }
      }
      b->class_bs[c] = best_bs;
      (void)best;
    }
    b->tuned = 1;
  } catch (...) {
    cleanup();
    throw;
  }
  cleanup();
}

void batch_create_impl(int count, const hprqp_problem* probs, const hprqp_options* opt, hipStream_t st,
                       hprqp_batch** out) {
  if (count <= 0 || !probs || !opt || !out) bfail(HPRQP_ERR_ARG, "bad arguments");
  if (opt->check_every <= 0 || opt->max_iter <= 0 || !(opt->tol >= 0.0)) bfail(HPRQP_ERR_ARG, "bad options");
  auto* b = new hprqp_batch();
  try {
    b->count = count;
    if (!st) {
      HBC(hipStreamCreateWithFlags(&b->own_st, hipStreamNonBlocking));
      HBC(hipDeviceSynchronize());
      st = b->own_st;
    }
    b->st = st;
    b->o.tol = opt->tol; b->o.max_iter = opt->max_iter; b->o.check_every = opt->check_every;
    b->o.sigma0 = opt->sigma0; b->o.lamA = opt->lambda_A; b->o.lamQ = opt->lambda_Q;
    b->o.alpha1 = opt->alpha1; b->o.alpha2 = opt->alpha2; b->o.alpha3 = opt->alpha3;
    b->o.enable_restart = opt->enable_restart; b->o.enable_sigma_update = opt->enable_sigma_update;
    if (!(opt->time_limit_s >= 0.0)) bfail(HPRQP_ERR_ARG, "time_limit_s must be >= 0");
    if (opt->time_limit_s > 0.0) {
      int dev = 0, khz = 0;
      HBC(hipGetDevice(&dev));
      HBC(hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev));
      if (khz <= 0) bfail(HPRQP_ERR_HIP, "device reports no wall-clock rate");
      const double ticks = std::ceil(opt->time_limit_s * 1e3 * (double)khz);
      b->o.time_ticks = ticks >= 9e18 ? (long long)9e18 : std::max(1ll, (long long)ticks);
    }
    std::vector<BInst> hi(count);
    // unique A matrices (instances may share one) -> one A^T each
    std::vector<int> rep_of(count);
    std::vector<int> reps;
    std::map<std::tuple<const void*, const void*, const void*, int, int>, int> rep_index;
    std::vector<long long> toff;
    long long tn = 0, tz = 0;
    for (int i = 0; i < count; ++i) {
      const hprqp_problem& P = probs[i];
      if (P.qkind != HPRQP_Q_LOWRANK) bfail(HPRQP_ERR_UNSUPPORTED, "batched solve supports qkind HPRQP_Q_LOWRANK only");
      if (P.l1_weight != 0.0) bfail(HPRQP_ERR_UNSUPPORTED, "batched solve supports phi = box indicator only (l1_weight 0)");
      if (P.n <= 0 || P.n > HB_NMAX || P.m < 0 || P.m > HB_MMAX || P.lr_rank < 0 || P.lr_rank > HB_RMAX)
        bfail(HPRQP_ERR_UNSUPPORTED, "batched solve needs 0 < n <= 2048, 0 <= m <= 64, lr_rank <= 16 (instance " +
                                         std::to_string(i) + ")");
      if (!P.c || !P.L || !P.U || !P.lr_d || (P.lr_rank > 0 && !P.lr_F) ||
          (P.m > 0 && (!P.l || !P.u || !P.a_rowptr || (P.a_nnz > 0 && (!P.a_col || !P.a_val)))))
        bfail(HPRQP_ERR_ARG, "missing array in instance " + std::to_string(i));
      BInst& I = hi[i];
      std::memset(&I, 0, sizeof(I));
      I.n = P.n; I.m = P.m; I.r = P.lr_rank;
      I.c = P.c; I.L = P.L; I.U = P.U; I.l = P.l; I.u = P.u; I.dg = P.lr_d; I.F = P.lr_F;
      I.arp = P.a_rowptr; I.aci = P.a_col; I.aval = P.a_val;
      I.off_n = b->total_n; I.off_m = b->total_m;
      I.annz = P.m > 0 ? P.a_nnz : 0;
      if (P.a_nnz < 0 || P.a_nnz > (1ll << 30)) bfail(HPRQP_ERR_SHAPE, "bad a_nnz in instance " + std::to_string(i));
      b->total_n += P.n; b->total_m += P.m;
      const auto akey = std::make_tuple((const void*)P.a_rowptr, (const void*)P.a_col, (const void*)P.a_val, P.n, P.m);
      const auto it = rep_index.find(akey);
      int found = it == rep_index.end() ? -1 : it->second;
      if (found < 0) {
        found = (int)reps.size();
        rep_index.emplace(akey, found);
        reps.push_back(i);
        toff.push_back(tn);
        toff.push_back(tz);
        tn += P.n + 1;
        tz += std::max<long long>(P.a_nnz, 0);
      }
      rep_of[i] = found;
    }
    HBC(hipMalloc(&b->trp, std::max<long long>(tn, 1) * sizeof(int)));
    HBC(hipMalloc(&b->tci, std::max<long long>(tz, 1) * sizeof(int)));
    HBC(hipMalloc(&b->tperm, std::max<long long>(tz, 1) * sizeof(int)));
    HBC(hipMalloc(&b->tval, std::max<long long>(tz, 1) * sizeof(double)));
    for (int i = 0; i < count; ++i) {
      const int q = rep_of[i];
      hi[i].trp = b->trp + toff[2 * q];
      hi[i].tci = b->tci + toff[2 * q + 1];
      hi[i].tperm = b->tperm + toff[2 * q + 1];
      hi[i].tval = b->tval + toff[2 * q + 1];
    }
    // padded copy of F: rank class of the kernel (10 or 16)
    int maxr = 0;
    for (int i = 0; i < count; ++i) maxr = std::max(maxr, hi[i].r);
    b->rank_max = maxr <= 10 ? 10 : 16;
    // (one padded copy per distinct F: instances that share F share the copy)
    std::vector<long long> ftoff(count);
    std::map<std::tuple<const double*, int, int>, long long> ft_index;
    std::vector<int> ft_rep;
    long long tf = 0;
    for (int i = 0; i < count; ++i) {
      const auto key = std::make_tuple(hi[i].F, hi[i].n, hi[i].r);
      const auto it = ft_index.find(key);
      if (it != ft_index.end()) { ftoff[i] = it->second; continue; }
      ftoff[i] = tf;
      ft_index.emplace(key, tf);
      ft_rep.push_back(i);
      tf += (long long)b->rank_max * hi[i].n;
    }
    HBC(hipMalloc(&b->ft, std::max<long long>(tf, 1) * sizeof(double)));
    HBC(hipMalloc(&b->d_ftoff, count * sizeof(long long)));
    HBC(hipMemcpyAsync(b->d_ftoff, ftoff.data(), count * sizeof(long long), hipMemcpyHostToDevice, st));
    for (int i = 0; i < count; ++i) hi[i].FT = b->ft + ftoff[i];
    HBC(hipMalloc(&b->d_insts, count * sizeof(BInst)));
    HBC(hipMemcpyAsync(b->d_insts, hi.data(), count * sizeof(BInst), hipMemcpyHostToDevice, st));
    HBC(hipMalloc(&b->d_flags, count * sizeof(int)));
    HBC(hipMemsetAsync(b->d_flags, 0, count * sizeof(int), st));
    k_batch_validate<<<count, 256, 0, st>>>(b->d_insts, count, b->d_flags);
    std::vector<int> flags(count);
    HBC(hipMemcpyAsync(flags.data(), b->d_flags, count * sizeof(int), hipMemcpyDeviceToHost, st));
    HBC(hipStreamSynchronize(st));
    for (int i = 0; i < count; ++i) {
      if (flags[i] & 2) bfail(HPRQP_ERR_SHAPE, "CSR structure of A invalid in instance " + std::to_string(i));
      if (flags[i] & 1) bfail(HPRQP_ERR_BOUNDS, "invalid bounds or non-finite data in instance " + std::to_string(i));
    }
    HBC(hipMalloc(&b->d_rep, reps.size() * sizeof(int)));
    HBC(hipMalloc(&b->d_toff, toff.size() * sizeof(long long)));
    HBC(hipMemcpyAsync(b->d_rep, reps.data(), reps.size() * sizeof(int), hipMemcpyHostToDevice, st));
    HBC(hipMemcpyAsync(b->d_toff, toff.data(), toff.size() * sizeof(long long), hipMemcpyHostToDevice, st));
    k_batch_transpose<<<(int)reps.size(), 256, 0, st>>>(b->d_insts, b->d_rep, (int)reps.size(), b->trp, b->tci,
                                                         b->tperm, b->tval, b->d_toff);
    HBC(hipMalloc(&b->d_ftrep, ft_rep.size() * sizeof(int)));
    HBC(hipMemcpyAsync(b->d_ftrep, ft_rep.data(), ft_rep.size() * sizeof(int), hipMemcpyHostToDevice, st));
    k_batch_ft<<<(int)ft_rep.size(), 256, 0, st>>>(b->d_insts, b->d_ftrep, (int)ft_rep.size(), b->rank_max, b->ft,
                                                   b->d_ftoff);
    // largest instances first
    std::vector<int> order(count);
    for (int i = 0; i < count; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](int a, int c) { return hi[a].n > hi[c].n; });
    HBC(hipMalloc(&b->d_order, count * sizeof(int)));
    HBC(hipMalloc(&b->d_queue, HB_NCLASS * sizeof(int)));
    HBC(hipMalloc(&b->d_infos, count * sizeof(BInfo)));
    HBC(hipEventCreate(&b->e0));
    HBC(hipEventCreate(&b->e1));
    HBC(hipMalloc(&b->d_qwx, count * sizeof(double)));
    HBC(hipMalloc(&b->d_t0, sizeof(long long)));
    b->o.t0 = b->d_t0;
    int dev = 0, ncu = 0;
    HBC(hipGetDevice(&dev));
    HBC(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
    // size classes: class c holds the instances with 256 << (c - 1) < n <= 256 << c
    std::vector<int> cls_order[HB_NCLASS];
    for (int i : order) {
      int c = 0;
      while (hi[i].n > (256 << c)) ++c;
      cls_order[c].push_back(i);
    }
    for (int c = 0; c < HB_NCLASS; ++c) {
      b->class_cnt[c] = (int)cls_order[c].size();
      b->class_bs[c] = c == HB_NCLASS - 1 ? 512 : 256;     // default shapes
    }
    const int bt = opt->batch_threads;
    if (bt != 0 && bt != 64 && bt != 128 && bt != 256 && bt != 512)
      bfail(HPRQP_ERR_ARG, "batch_threads must be 0, 64, 128, 256 or 512");
    if (bt != 0) {
      for (int c = 0; c < HB_NCLASS; ++c)
        if (HB_EPT * bt >= (256 << c)) b->class_bs[c] = bt;
    } else if (opt->spmv_autotune == 1) {
      autotune_batch(b, hi, cls_order, ncu);
    }
    // one kernel per shape in use, its instances largest first
    std::vector<int> korder;
    b->nkern = 0;
    const BShape* cls_sh[HB_NCLASS];
    for (int c = 0; c < HB_NCLASS; ++c) cls_sh[c] = &batch_shape(b->rank_max, b->class_bs[c], c);
    for (int c0 = HB_NCLASS - 1; c0 >= 0; --c0) {
      if (c0 + 1 < HB_NCLASS && cls_sh[c0] == cls_sh[c0 + 1]) continue;   // (equal shapes are neighbours)
      std::vector<int> mine;
      for (int c = c0; c >= 0 && cls_sh[c] == cls_sh[c0]; --c)
        mine.insert(mine.end(), cls_order[c].begin(), cls_order[c].end());
      if (mine.empty()) continue;
      hprqp_batch::Kern& K = b->kern[b->nkern];
      K.sh = cls_sh[c0];
      K.first = (int)korder.size();
      K.cnt = (int)mine.size();
      K.lds = batch_lds(*K.sh, hi, mine);
      K.grid = std::max(1, std::min(K.cnt, batch_resident(*K.sh, K.lds, ncu)));
      HBC(hipMalloc(&K.hbuf, (size_t)K.grid * 5 * K.sh->ept * K.sh->bs * sizeof(double)));
      if (b->nkern > 0) {
        HBC(hipStreamCreateWithFlags(&K.st, hipStreamNonBlocking));
        HBC(hipEventCreateWithFlags(&K.ev_join, hipEventDisableTiming));
      }
      korder.insert(korder.end(), mine.begin(), mine.end());
      ++b->nkern;
    }
    if (b->nkern > 1) HBC(hipEventCreateWithFlags(&b->ev_fork, hipEventDisableTiming));
    b->order_default = korder;
    HBC(hipMemcpyAsync(b->d_order, korder.data(), count * sizeof(int), hipMemcpyHostToDevice, st));
    HBC(hipStreamSynchronize(st));
    *out = b;
  } catch (...) {
    delete b;
    throw;
  }
}

void solve_batch_impl(hprqp_batch* b, const double* y0, const double* w0, const double* x0, double* y, double* z,
                      double* w, double* x, hprqp_info* infos) {
  if (!b || !z || !w || !x || (b->total_m > 0 && !y)) bfail(HPRQP_ERR_ARG, "NULL argument");
  if (b->own_st) HBC(hipDeviceSynchronize());
  k_zero_ints<<<1, 64, 0, b->st>>>(b->d_queue, HB_NCLASS);
  HBC(hipEventRecord(b->e0, b->st));
  k_stamp<<<1, 64, 0, b->st>>>(b->d_t0);
  // one launch per shape in use, kernels 1.. on their own streams
  if (b->nkern > 1) HBC(hipEventRecord(b->ev_fork, b->st));
  for (int k = 0; k < b->nkern; ++k) {
    const hprqp_batch::Kern& K = b->kern[k];
    hipStream_t s = k == 0 ? b->st : K.st;
    if (k > 0) HBC(hipStreamWaitEvent(s, b->ev_fork, 0));
    batch_launch(*K.sh, K.lds, s, K.grid, b->d_insts, b->d_order + K.first, K.cnt, b->d_queue + k, b->o, y0, w0, x0, y,
                 z, w, x, b->d_infos, K.hbuf);
    if (k > 0) HBC(hipEventRecord(K.ev_join, s));
  }
  for (int k = 1; k < b->nkern; ++k) HBC(hipStreamWaitEvent(b->st, b->kern[k].ev_join, 0));
  HBC(hipEventRecord(b->e1, b->st));
  k_batch_qwx<<<std::min(b->count, 4096), HB_QWX_BS, 0, b->st>>>(b->d_insts, b->count, w, x, b->d_qwx);
  HBC(hipGetLastError());
  std::vector<BInfo> hi(b->count);
  std::vector<double> hq(b->count);
  HBC(hipMemcpyAsync(hi.data(), b->d_infos, b->count * sizeof(BInfo), hipMemcpyDeviceToHost, b->st));
  HBC(hipMemcpyAsync(hq.data(), b->d_qwx, b->count * sizeof(double), hipMemcpyDeviceToHost, b->st));
  HBC(hipStreamSynchronize(b->st));
  float ms = 0.f;
  HBC(hipEventElapsedTime(&ms, b->e0, b->e1));
  b->last_kernel_s = ms * 1e-3;
  if (infos)
    for (int i = 0; i < b->count; ++i) {
      hprqp_info& f = infos[i];
      std::memset(&f, 0, sizeof(f));
      f.term = hi[i].term; f.iters = hi[i].iters; f.restarts = hi[i].restarts;
      f.sigma = hi[i].sigma; f.sigma0 = hi[i].sigma0; f.lambda_A = hi[i].lamA; f.lambda_Q = hi[i].lamQ;
      f.eta_p = hi[i].eta_p; f.eta_d = hi[i].eta_d; f.eta_gap = hi[i].eta_gap;
      f.pobj = hi[i].pobj; f.dobj = hi[i].dobj; f.R_last = hi[i].R_last;
      f.qwx_gap = hq[i];
    }
}
}  // namespace

#define HB_GUARD(...)                 \
  try {                               \
    hq::g_err.clear();                \
    __VA_ARGS__;                      \
    return HPRQP_OK;                  \
  } catch (const BErr& e) {           \
    hq::g_err = e.msg;                \
    return e.st;                      \
  } catch (const std::exception& e) { \
    hq::g_err = e.what();             \
    return HPRQP_ERR_HIP;             \
  }

extern "C" {

hprqp_status hprqp_batch_create(int32_t count, const hprqp_problem* probs, const hprqp_options* opt,
                                hipStream_t stream, hprqp_batch** out) {
  HB_GUARD(batch_create_impl(count, probs, opt, stream, out));
}

hprqp_status hprqp_solve_batch(hprqp_batch* b, const double* y0, const double* w0, const double* x0, double* y,
                               double* z, double* w, double* x, hprqp_info* infos_host) {
  HB_GUARD(solve_batch_impl(b, y0, w0, x0, y, z, w, x, infos_host));
}


hprqp_status hprqp_batch_shapes(hprqp_batch* b, int32_t* class_count_host, int32_t* class_threads_host,
                                double* class_us_host) {
  HB_GUARD(if (!b) bfail(HPRQP_ERR_ARG, "NULL batch");
           for (int c = 0; c < HB_NCLASS; ++c) {
             if (class_count_host) class_count_host[c] = b->class_cnt[c];
             if (class_threads_host) class_threads_host[c] = b->class_bs[c];
             for (int lb = 0; lb < HB_NCLASS; ++lb)
               if (class_us_host) class_us_host[c * HB_NCLASS + lb] = b->class_us[c][lb];
           });
}

hprqp_status hprqp_batch_set_priority(hprqp_batch* b, const float* priority) {
  HB_GUARD(if (!b) bfail(HPRQP_ERR_ARG, "NULL batch");
           std::vector<int> ord = b->order_default;
           if (priority) {
             std::vector<float> pr(b->count);
             HBC(hipMemcpyAsync(pr.data(), priority, b->count * sizeof(float), hipMemcpyDeviceToHost, b->st));
             HBC(hipStreamSynchronize(b->st));
             for (float& v : pr)
               if (!std::isfinite(v)) v = -INFINITY;     // no usable prediction: last
             // each kernel's queue: highest priority first, ties in the default order
             for (int k = 0; k < b->nkern; ++k) {
               auto first = ord.begin() + b->kern[k].first;
               std::stable_sort(first, first + b->kern[k].cnt, [&](int a, int c) { return pr[a] > pr[c]; });
             }
           }
           HBC(hipMemcpyAsync(b->d_order, ord.data(), b->count * sizeof(int), hipMemcpyHostToDevice, b->st));
           HBC(hipStreamSynchronize(b->st)));
}

double hprqp_batch_last_kernel_s(hprqp_batch* b) { return b ? b->last_kernel_s : 0.0; }

void hprqp_batch_destroy(hprqp_batch* b) { delete b; }

}  // extern "C"
