// small.hpp -- one workgroup runs a whole check segment of HPR-QP
// (Algorithm 4, Tseg iterations and the check) for a small problem.
//
// At n, m of a few hundred the four products of an iteration are a few
// microseconds of work each, and the per-launch cost of a graph node
// (~7 us) is what an iteration costs.  Here the products are phases of one
// 1024-thread workgroup separated by barriers: each phase runs the same
// fused epilogue as the multi-block kernels (so the arithmetic is that of
// the four-launch path; the iterations of a staged segment that need no
// reductions and no outputs run it from registers, small_fast), rows are taken by groups of G lanes (butterfly sum
// in a fixed order), and the reductions of a phase go through the block
// reduction into the same slots, with one partial per slot.  When the
// matrices and every vector of the iteration fit (dynamic LDS, up to
// HQ_SMALL_LDS bytes; STAGED), they are copied into LDS at the start of the
// segment and the written vectors back at its end, so every gather is an LDS
// access; otherwise they stay in global memory.  The staged kernel derives
// every pointer from the LDS base only (never a global fallback), so the
// compiler addresses them as LDS (ds_read/ds_write) instead of generic flat
// accesses, which go through the vector-memory path and are counted by both
// wait counters.  Explicit Q (CSR) or Q = 0 only.
#pragma once
#include "common.hpp"
#include "epilogues.hpp"
#include "epilogues_primal.hpp"

#ifndef HQ_SMALL_BS
#define HQ_SMALL_BS 1024
#endif
#define HQ_SMALL_LDS (150 * 1024)

struct SmallMat {
  int rows;
  const int* rp;     // nullptr: the zero matrix (q = 0 for every row)
  const int* ci;
  const double* v;
};

// vectors of the iteration, by index
enum : int {
  SV_L, SV_U, SV_C, SV_LB, SV_UB, SV_IE, SV_ID,                 // read only
  SV_YA, SV_WA, SV_XA, SV_ATYA, SV_QWA, SV_PTA,                  // read only during a segment
  SV_Y, SV_YBAR, SV_W, SV_X, SV_ATY, SV_QW, SV_XH, SV_V, SV_Q1, SV_D, SV_G, SV_E, SV_XB, SV_ZB, SV_WBAR,
  SV_QWBAR, SV_XBO, SV_ZBO,                                      // written
  SV_PE, SV_PAX, SV_PDY, SV_PT, SV_PTB, SV_PDT,                  // written (primal methods only)
  SV_COUNT,
  SV_FIRST_WRITTEN = SV_Y
};

struct SmallArgs {
  SmallMat A, AT, Q;
  int n, m;
  double* vec[SV_COUNT];      // global arrays (nullptr: absent)
  int vlen[SV_COUNT];
  double l1;
  double* partials;
  int* counts;
  const DevParams* prm;
  // LDS staging (lds_bytes = 0: none): byte offsets of the vectors and of the
  // matrices' row pointers, columns and values
  int lds_bytes;              // (every vector is followed by a zero, the operand of missing entries)
  int voff[SV_COUNT];
  int moff[3][3];             // [A, AT, Q][rp, ci, v]
};

// q_i = (M x)_i for every row, then epi(i, q_i); block reduction of the
// epilogue's accumulators; a barrier makes the epilogue's stores visible to
// the next phase.  KEEP: the compiler may keep addresses formed from the thread index
// from one phase to the next.  Where the registers hold them that is faster (the
// primal methods, n = 200: 3.78 us an iteration recomputed, 3.63 kept); where they do not
// they would be spilled.
template <int G, bool KEEP = false, class Epi>
__device__ __forceinline__ void small_phase(const SmallMat& M, const double* __restrict__ x, Epi e,
                                            const DevParams* __restrict__ prm, int j, const RedOut& red) {
  constexpr int NR = Epi::NR;
  e.setup(prm, j);
  double acc[NR > 0 ? NR : 1];
#pragma unroll
  for (int s = 0; s < (NR > 0 ? NR : 1); ++s) acc[s] = 0.0;
  int tid = (int)threadIdx.x;
  if constexpr (!KEEP) asm volatile("" : "+v"(tid));
  const int gl = tid % G, gi = tid / G;
  for (int row = gi; row < M.rows; row += HQ_SMALL_BS / G) {
    double sum = 0.0;
    if (M.rp) {
      const int b = M.rp[row], en = M.rp[row + 1];
#pragma unroll 4
      for (int k = b + gl; k < en; k += G) sum += M.v[k] * x[M.ci[k]];
    }
    sum = group_sum<G>(sum);   // (a group's lanes share a row: active together)
    if (gl == 0) e(row, sum, acc);
  }
  if (red.active) block_reduce_store<NR, Epi::MAXMASK, true>(acc, red);
  __syncthreads();
}

__device__ __forceinline__ RedOut small_red(const SmallArgs& a, int s0, int s1 = -1, int s2 = -1) {
  RedOut r;
  r.partials = a.partials;
  r.counts = a.counts;
  for (int s = 0; s < 16; ++s) r.slot[s] = -1;
  r.slot[0] = (int8_t)s0; r.slot[1] = (int8_t)s1; r.slot[2] = (int8_t)s2;
  r.active = s0 >= 0 || s1 >= 0 || s2 >= 0;
  return r;
}

template <class T>
__device__ __forceinline__ void small_copy(T* __restrict__ dst, const T* __restrict__ src, int count) {
  for (int i = threadIdx.x; i < count; i += HQ_SMALL_BS) dst[i] = src[i];
}

// The arrays the phases use: LDS copies when staged (copied in here), else
// the global ones.  (Loops over the arrays are unrolled so that V and mats
// stay in registers.)  BATCHED: the vectors are copied eleven at a time and followed by
// a zero, the operand of small_fast's missing entries.  Copied one by one they leave the
// kernel with fewer scalars spilled over its phases: 3.54 us an iteration of the
// primal methods at n = 200, 3.63 batched.
template <bool STAGED, bool BATCHED>
__device__ __forceinline__ void small_stage_in(const SmallArgs& a, unsigned char* lds, double* (&V)[SV_COUNT],
                                               SmallMat (&mats)[3]) {
#pragma unroll
  for (int s = 0; s < SV_COUNT; ++s) V[s] = STAGED ? nullptr : a.vec[s];
  if constexpr (STAGED && !BATCHED) {
#pragma unroll
    for (int s = 0; s < SV_COUNT; ++s)
      if (a.vec[s]) {
        double* p = (double*)(lds + a.voff[s]);
        small_copy(p, a.vec[s], a.vlen[s]);
        V[s] = p;
      }
  }
  if constexpr (STAGED && BATCHED) {
    // the loads of eleven vectors in flight together
    constexpr int NB = 11;
#pragma unroll
    for (int s0 = 0; s0 < SV_COUNT; s0 += NB) {
      double first[NB];
#pragma unroll
      for (int q = 0; q < NB && s0 + q < SV_COUNT; ++q) {
        const int s = s0 + q, n = a.vlen[s];
        first[q] = a.vec[s] && n > 0 ? a.vec[s][min((int)threadIdx.x, n - 1)] : 0.0;
      }
#pragma unroll
      for (int q = 0; q < NB && s0 + q < SV_COUNT; ++q) {
        const int s = s0 + q, n = a.vlen[s];
        if (!a.vec[s]) continue;
        double* p = (double*)(lds + a.voff[s]);
        if ((int)threadIdx.x <= n) p[threadIdx.x] = (int)threadIdx.x < n ? first[q] : 0.0;
        for (int i = threadIdx.x + HQ_SMALL_BS; i <= n; i += HQ_SMALL_BS) p[i] = i < n ? a.vec[s][i] : 0.0;
        V[s] = p;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if (STAGED) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      SmallMat& M = mats[q];
      const SmallMat Mg = M;   // the arrays in global memory (rp == nullptr: the zero matrix)
      M.rp = nullptr; M.ci = nullptr; M.v = nullptr;
      if (Mg.rp) {
        int* rp = (int*)(lds + a.moff[q][0]);
        int* ci = (int*)(lds + a.moff[q][1]);
        double* v = (double*)(lds + a.moff[q][2]);
        small_copy(rp, Mg.rp, Mg.rows + 1);
        __syncthreads();   // the row pointers give the number of nonzeros
        const int nnz = rp[Mg.rows];
        small_copy(ci, Mg.ci, nnz);
        small_copy(v, Mg.v, nnz);
        M.rp = rp; M.ci = ci; M.v = v;
      }
    }
    __syncthreads();
  }
}

// the written vectors back to global memory at the end of a staged segment
template <bool STAGED>
__device__ __forceinline__ void small_stage_out(const SmallArgs& a, double* const (&V)[SV_COUNT]) {
  if (STAGED) {
#pragma unroll
    for (int s = SV_FIRST_WRITTEN; s < SV_COUNT; ++s)
      if (a.vec[s]) small_copy(a.vec[s], V[s], a.vlen[s]);
  }
}

// The entries of one matrix that a lane of a row's group multiplies: k = b + gl,
// b + gl + G, ...; the first K of them in registers (missing ones: 0 times the
// zero behind the vector), further ones read from LDS.
template <int G, int K>
struct SmallRow {
  typedef const __attribute__((address_space(3))) double* lds_ptr;
  double v[K];
  lds_ptr p[K];   // where the entry's operand is in the vector x
  int k0, en;
  __device__ __forceinline__ void load(const SmallMat& M, int row, const double* x, int pad) {
    const bool on = M.rp != nullptr && row < M.rows;
    const int b = on ? M.rp[row] : 0;
    en = on ? M.rp[row + 1] : 0;
    k0 = b + (int)(threadIdx.x % G);
#pragma unroll
    for (int u = 0; u < K; ++u) {
      const int k = k0 + G * u;
      int c = pad;
      v[u] = 0.0;
      if (M.rp) {
        const int kk = k < en ? k : 0;
        const double val = M.v[kk];
        const int ci = M.ci[kk];
        v[u] = k < en ? val : 0.0;
        c = k < en ? ci : pad;
      }
      p[u] = (lds_ptr)(x + c);
    }
    k0 += G * K;
  }
  // the sum of small_phase, in its order, with the vector `delta` entries behind x
  __device__ __forceinline__ double dot(const SmallMat& M, int delta, const double* __restrict__ xd) const {
    double t[K], sum = 0.0;
#pragma unroll
    for (int u = 0; u < K; ++u) t[u] = *(p[u] + delta);
#pragma unroll
    for (int u = 0; u < K; ++u) sum += v[u] * t[u];
    for (int k = k0; k < en; k += G) sum += M.v[k] * xd[M.ci[k]];
    return group_sum<G>(sum);
  }
};

// Iterations j0 <= j < j1 of a staged segment, none of them with reductions or
// with outputs for a check.  The phases above are bound by latency: a row
// pointer, an entry and a gather read from LDS in turn, then the row's operands,
// and two or three divisions of scalars that all 16 waves repeat.  Here a group
// keeps its row's matrix entries, state, anchors, c and box in registers (the
// lanes of a group hold copies), the scalars of the epoch are formed once, and
// only the four vectors that the next product gathers go through LDS.  The
// arithmetic is that of the epilogues EpiQ1, EpiY, EpiAT and EpiQ2 on the same
// sums, so the iterates are the same to the last bit.  n = 200, m = 100, 4,900
// nonzeros of Q, a segment of 100 iterations: about 600 us in phases alone, 294 us
// with these (copies in and out included).  What is left is the LDS reads of the
// gathers (260 wave reads for the two Q products) and the instructions of 16 waves.
// Every register counts at 1024 threads: operands of the loop in scratch memory
// cost more than the loop's own work (337 us with seven of them).
__device__ __forceinline__ double uniform(double x) {   // a value equal in all lanes, in scalar registers
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readfirstlane((int)(b & 0xffffffffll)), hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
#define HQ_SMALL_KQ 10
#define HQ_SMALL_KA 4
#define HQ_SMALL_KT 2
template <int G>
__device__ __forceinline__ void small_fast(const SmallArgs& a, double* const (&V)[SV_COUNT], const SmallMat& A,
                                           const SmallMat& AT, const SmallMat& Q, const DevParams* prm, int j0, int j1) {
  const int row = threadIdx.x / G;
  const bool own = threadIdx.x % G == 0, okn = row < a.n, okm = row < a.m;
  const int i = okn ? row : 0, im = okm ? row : 0;
  SmallRow<G, HQ_SMALL_KQ> rQ;
  SmallRow<G, HQ_SMALL_KA> rA;
  SmallRow<G, HQ_SMALL_KT> rT;
  rQ.load(Q, row, V[SV_XH], a.n);
  rA.load(A, row, V[SV_V], a.n);
  rT.load(AT, row, V[SV_YBAR], a.m);
  double xh = V[SV_XH][i], w = V[SV_W][i], Qw = V[SV_QW][i], ATy = V[SV_ATY][i];
  const double wa = V[SV_WA][i], Qwa = V[SV_QWA][i], xa = V[SV_XA][i], ATya = V[SV_ATYA][i];
  const bool rows = a.m > 0;
  double y = 0.0, ya = 0.0, l = 0.0, u = 0.0, d = rows ? 0.0 : V[SV_D][i];
  if (rows) { y = V[SV_Y][im]; ya = V[SV_YA][im]; l = V[SV_L][im]; u = V[SV_U][im]; }
  IterScalars s;
  s.load(prm, j0);
  const double sigma = uniform(s.sigma), sQ = uniform(s.sQ), kappa = uniform(s.kappa), sA = uniform(s.sA);
  const double inv = uniform(s.inv), sl1 = uniform(s.sigma * a.l1);
  const int64_t t0 = prm->t0;
  // the waves without rows of A sit its phase out; the last wave, which has the
  // fewest rows, divides for the next iteration's rho
  const int row0 = __builtin_amdgcn_readfirstlane(row);
  const bool wave_m = row0 < a.m, last = __builtin_amdgcn_readfirstlane((int)threadIdx.x) == HQ_SMALL_BS - HQ_WAVE;
  __shared__ double srho[2];
  if (last) srho[j0 & 1] = 1.0 / (double)(t0 + j0 + 2);
  __syncthreads();
  for (int j = j0; j < j1; ++j) {
    const double rho = srho[j & 1];
    if (last) srho[(j + 1) & 1] = 1.0 / (double)(t0 + j + 3);
    const double q1 = rQ.dot(Q, 0, V[SV_XH]);
    if (rows) {
      if (own && okn) V[SV_V][row] = __builtin_fma(kappa, Qw - q1, xh);
      __syncthreads();
      if (wave_m) {
        const double q = rA.dot(A, 0, V[SV_V]);
        const double r = y_arg(q, sA, y);
        const double yb = (clampd(r, l, u) - r) / sA;
        if (own && okm) V[SV_YBAR][row] = yb;
        y = halpern(rho, ya, reflect(yb, y));
      }
      __syncthreads();
      const double g = rT.dot(AT, 0, V[SV_YBAR]);
      d = g - ATy;
      ATy = halpern(rho, ATya, reflect(g, ATy));
      if (own && okn) V[SV_D][row] = d;
    }
    __syncthreads();   // (without rows: every group has read xh)
    int delta = (a.voff[SV_D] - a.voff[SV_XH]) / 8;
    asm volatile("" : "+s"(delta));   // (the sums are formed again: a second set of addresses would spill)
    const double q2 = rows ? rQ.dot(Q, delta, V[SV_D]) : 0.0;
    const double wb = w_bar(sQ, w, xh, inv, kappa, d);
    const double Qwb = w_bar(sQ, Qw, q1, inv, kappa, q2);
    const double xn = halpern(rho, xa, xh);
    w = halpern(rho, wa, reflect(wb, w));
    Qw = halpern(rho, Qwa, reflect(Qwb, Qw));
    const double rz = z_arg(xn, sigma, Qw, ATy, V[SV_C][i]);   // (c, L and U stay in LDS: 128 registers)
    const double xbn = prox_phi(rz, sl1, V[SV_LB][i], V[SV_UB][i]);
    xh = reflect(xbn, xn);
    if (own && okn) V[SV_XH][row] = xh;
    __syncthreads();
  }
  if (own && okn) { V[SV_W][row] = w; V[SV_QW][row] = Qw; V[SV_ATY][row] = ATy; }
  if (own && okm) V[SV_Y][row] = y;
  __syncthreads();
}

// one iteration as phases (all forms: merit, check)
template <int G, bool KEEP = false>
__device__ __forceinline__ void small_iteration(const SmallArgs& a, double* const (&V)[SV_COUNT], const SmallMat& A,
                                                const SmallMat& AT, const SmallMat& Q, const DevParams* prm, int j,
                                                int Tseg) {
  const RedOut none = small_red(a, -1);
  const bool check = (j == Tseg - 1);
  const int rgroup = check ? SL_RC : (j == 0 ? SL_RF : -1);
  const bool want_r = rgroup >= 0;
  const bool xb_next = j >= Tseg - 2;
  // a3: q1 = Q xhat, v
  small_phase<G, KEEP>(Q, V[SV_XH], EpiQ1{V[SV_XH], V[SV_QW], V[SV_V], V[SV_Q1], 0.0}, prm, j, none);
  if (a.m > 0) {
    // a4: A v, ybar, y+
    small_phase<G, KEEP>(A, V[SV_V], EpiY{V[SV_L], V[SV_U], V[SV_YA], V[SV_Y], V[SV_YBAR], want_r, check, 0.0, 0.0},
                   prm, j, small_red(a, want_r ? rgroup : -1, check ? SL_TH : -1));
    // a5: A^T ybar, d, A^T y+
    small_phase<G, KEEP>(AT, V[SV_YBAR], EpiAT{V[SV_ATY], V[SV_ATYA], V[SV_D], V[SV_G], V[SV_E], check, 0.0}, prm, j,
                   none);
  }
  if (check) {
    if (a.m > 0) {
      RedOut r = none;
      for (int s = 0; s < 4; ++s) r.slot[s] = (int8_t)(SL_RA + s);
      r.active = 1;
      small_phase<G, KEEP>(A, V[SV_XB], EpiResA{V[SV_L], V[SV_U], V[SV_YBAR], V[SV_IE]}, prm, j, r);
    }
    RedOut r = none;
    for (int s = 0; s < 7; ++s) r.slot[s] = (int8_t)(SL_RQ + s);
    r.active = 1;
    small_phase<G, KEEP>(Q, V[SV_XB],
                   EpiResQ{V[SV_XB], V[SV_ZB], a.m > 0 ? V[SV_G] : nullptr, V[SV_C], V[SV_LB], V[SV_UB], V[SV_XBO],
                           V[SV_ZBO], V[SV_ID], a.l1},
                   prm, j, r);
  }
  // a6: Q d, wbar, Halpern, next z/x step
  EpiQ2 e6;
  e6.xh = V[SV_XH]; e6.w = V[SV_W]; e6.Qw = V[SV_QW]; e6.XB = V[SV_XB]; e6.ZB = V[SV_ZB];
  e6.q1 = V[SV_Q1]; e6.d = V[SV_D]; e6.wa = V[SV_WA]; e6.Qwa = V[SV_QWA]; e6.xa = V[SV_XA]; e6.ATy = V[SV_ATY];
  e6.c = V[SV_C]; e6.L = V[SV_LB]; e6.U = V[SV_UB]; e6.e = V[SV_E];
  e6.wbar = V[SV_WBAR]; e6.qwbar = V[SV_QWBAR]; e6.x = V[SV_X]; e6.xbar_out = V[SV_XBO];
  e6.want_r = want_r; e6.check = check; e6.xb_next = xb_next; e6.trace = 0;
  e6.l1 = a.l1;
  RedOut r6 = none;
  if (want_r)
    for (int s = 0; s < 6; ++s) r6.slot[s] = (int8_t)(rgroup + 1 + s);
  if (check)
    for (int s = 0; s < 3; ++s) r6.slot[6 + s] = (int8_t)(SL_TH + 1 + s);
  r6.active = want_r || check;
  const SmallMat Qd{a.n, a.m > 0 ? Q.rp : nullptr, a.m > 0 ? Q.ci : nullptr, a.m > 0 ? Q.v : nullptr};
  small_phase<G, KEEP>(Qd, V[SV_D], e6, prm, j, r6);
  if (check && a.m > 0 && Q.rp) small_phase<G, KEEP>(Q, V[SV_E], EpiTheta3{V[SV_E]}, prm, j, small_red(a, SL_TH + 4));
}

// The staged segment's copies of its arguments and scalars, in LDS.
struct SmallShared {
  SmallArgs a;
  DevParams prm;
};
__device__ __forceinline__ SmallShared& small_shared() {
  __shared__ SmallShared s;
  return s;
}
template <class T>
__device__ __forceinline__ T* uniform_ptr(T* p) {
  return (T*)__double_as_longlong(uniform(__longlong_as_double((long long)p)));
}

// The same out of line for a staged segment, whose iterations between checks run
// from registers (small_fast): inlined, its addresses and reduction slots would
// be kept over them and push their operands into scratch memory.
template <int G>
__device__ __noinline__ void small_staged_iteration(int j, int Tseg) {
  extern __shared__ __align__(16) unsigned char small_lds[];
  const SmallArgs& sa = small_shared().a;
  SmallArgs a;   // (only what the phases read)
  a.n = __builtin_amdgcn_readfirstlane(sa.n); a.m = __builtin_amdgcn_readfirstlane(sa.m);
  a.l1 = uniform(sa.l1);
  a.partials = uniform_ptr(sa.partials); a.counts = uniform_ptr(sa.counts);
  j = __builtin_amdgcn_readfirstlane(j); Tseg = __builtin_amdgcn_readfirstlane(Tseg);
  double* V[SV_COUNT];
#pragma unroll
  for (int s = 0; s < SV_COUNT; ++s) {
    const int off = __builtin_amdgcn_readfirstlane(sa.vec[s] ? sa.voff[s] : -1);
    V[s] = off >= 0 ? (double*)(small_lds + off) : nullptr;
  }
  SmallMat mats[3];
  const SmallMat gm[3] = {sa.A, sa.AT, sa.Q};
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const bool on = __builtin_amdgcn_readfirstlane(gm[q].rp != nullptr) != 0;
    mats[q].rows = __builtin_amdgcn_readfirstlane(gm[q].rows);
    const int o0 = __builtin_amdgcn_readfirstlane(sa.moff[q][0]), o1 = __builtin_amdgcn_readfirstlane(sa.moff[q][1]),
              o2 = __builtin_amdgcn_readfirstlane(sa.moff[q][2]);
    mats[q].rp = on ? (const int*)(small_lds + o0) : nullptr;
    mats[q].ci = on ? (const int*)(small_lds + o1) : nullptr;
    mats[q].v = on ? (const double*)(small_lds + o2) : nullptr;
  }
  small_iteration<G>(a, V, mats[0], mats[1], mats[2], &small_shared().prm, j, Tseg);
}

// Iterations from which a staged segment runs those between its checks from registers
// (FAST), n G <= 1024: setting that up and its three iterations out of line take 10 us more
// than phases inlined, an iteration from registers 2.1 us less (n = 60, segments
// of 1, 3, 20 and 100 iterations: 30, 43, 111, 429 us in phases, 36, 54, 89, 239 so).
// Larger staged problems have no such iterations, and are faster out of line.
#define HQ_SMALL_FAST_FROM 8
template <int G, bool STAGED, bool FAST = STAGED>
__global__ __launch_bounds__(HQ_SMALL_BS) void k_small_segment(SmallArgs a, int Tseg) {
  extern __shared__ __align__(16) unsigned char small_lds[];
  double* V[SV_COUNT];
  SmallMat mats[3] = {a.A, a.AT, a.Q};
  small_stage_in<STAGED, FAST>(a, small_lds, V, mats);
  // the segment's scalars (sigma, lambda's, t0) are read by every phase: keep a copy in LDS
  SmallShared& S = small_shared();
  if (threadIdx.x == 0) {
    S.prm = *a.prm;
    if (FAST) S.a = a;
  }
  __syncthreads();
  if constexpr (FAST) {
    for (int j = 0; j < Tseg; ++j) {
      // all but the first iteration (merit) and the last two (outputs of the check)
      if (j == 1 && Tseg > 3 && (long long)max(a.n, a.m) * G <= HQ_SMALL_BS) {
        small_fast<G>(a, V, mats[0], mats[1], mats[2], &S.prm, j, Tseg - 2);
        j = Tseg - 2;
      }
      small_staged_iteration<G>(j, Tseg);
    }
  } else {
    for (int j = 0; j < Tseg; ++j) small_iteration<G, STAGED>(a, V, mats[0], mats[1], mats[2], &S.prm, j, Tseg);
  }
  small_stage_out<STAGED>(a, V);
}

// HPR on the primal reformulations (Algorithms 6 and 7 of the appendix,
// meth = 1, 2): the products of an iteration as phases, in the order and with
// the epilogues of the multi-launch path.
template <int G, bool STAGED>
__global__ __launch_bounds__(HQ_SMALL_BS) void k_small_primal(SmallArgs a, int Tseg, int meth) {
  extern __shared__ __align__(16) unsigned char small_lds[];
  double* V[SV_COUNT];
  SmallMat mats[3] = {a.A, a.AT, a.Q};
  small_stage_in<STAGED, false>(a, small_lds, V, mats);
  __shared__ DevParams sprm;
  if (threadIdx.x == 0) sprm = *a.prm;
  __syncthreads();
  const DevParams* prm = &sprm;
  const SmallMat& A = mats[0];
  const SmallMat& AT = mats[1];
  const SmallMat& Q = mats[2];
  const RedOut none = small_red(a, -1);
  const SmallMat zero_n{a.n, nullptr, nullptr, nullptr};
  const bool rows = a.m > 0;
  for (int j = 0; j < Tseg; ++j) {
    const bool check = (j == Tseg - 1);
    const int rgroup = check ? SL_RC : (j == 0 ? SL_RF : -1);
    const bool want_r = rgroup >= 0;
    const int store_bar = want_r || check;
    const auto at = [&](int off) { return want_r ? rgroup + off : -1; };
    // Q x (Algorithm 6) or Q v with the v/t-step (Algorithm 7)
    if (meth == 1) {
      small_phase<G, true>(Q, V[SV_X], EpiStore{V[SV_Q1]}, prm, j, none);
    } else {
      small_phase<G, true>(Q, V[SV_W],
                     EpiP2V{V[SV_W], V[SV_X], V[SV_PTA], V[SV_PT], V[SV_WBAR], V[SV_V], V[SV_QW], V[SV_E], V[SV_PDT],
                            V[SV_PTB], want_r, check},
                     prm, j, small_red(a, at(1), at(4), check ? SL_TH + 2 : -1));
    }
    // A x with the s/y-step
    if (rows)
      small_phase<G, true>(A, V[SV_X],
                     EpiPY{V[SV_L], V[SV_U], V[SV_YA], V[SV_Y], V[SV_YBAR], V[SV_PE], V[SV_PAX], V[SV_PDY], want_r,
                           check, store_bar},
                     prm, j, small_red(a, at(3), check ? SL_TH + 1 : -1));
    // A^T (2 ybar - y) with the x-step
    // (a value, not a reference to one of two locals: that would keep both in scratch)
    const SmallMat ATx{a.n, rows ? AT.rp : nullptr, rows ? AT.ci : nullptr, rows ? AT.v : nullptr};
    if (meth == 1) {
      small_phase<G, true>(ATx, V[SV_PE],
                     EpiP1X{V[SV_Q1], V[SV_C], V[SV_LB], V[SV_UB], V[SV_XA], V[SV_X], V[SV_XB], V[SV_ZB], V[SV_D],
                            want_r, check, store_bar, a.l1},
                     prm, j, small_red(a, at(0), check ? SL_TH : -1));
    } else {
      small_phase<G, true>(ATx, V[SV_PE],
                     EpiP2X{V[SV_V], V[SV_C], V[SV_LB], V[SV_UB], V[SV_XA], V[SV_WA], V[SV_WBAR], V[SV_PDT], V[SV_X],
                            V[SV_W], V[SV_XB], V[SV_ZB], V[SV_D], want_r, check, store_bar, a.l1},
                     prm, j, small_red(a, at(0), at(5), check ? SL_TH : -1));
    }
    if (want_r) {
      // <A dx, dy> and <dx, Q dx> (Algorithm 6) or <dv, Q dv> (Algorithm 7)
      if (rows) small_phase<G, true>(A, V[SV_XB], EpiMeritA{V[SV_PAX], V[SV_PDY]}, prm, j, small_red(a, rgroup + 2));
      if (meth == 1) small_phase<G, true>(Q, V[SV_XB], EpiMeritQ{V[SV_Q1], V[SV_D]}, prm, j, small_red(a, rgroup + 1));
      else small_phase<G, true>(Q, V[SV_WBAR], EpiMeritQ{V[SV_QW], V[SV_E]}, prm, j, small_red(a, rgroup + 6));
    }
    if (check) {
      // stopping quantities at (ybar, zbar, xbar): A^T ybar, A xbar, Q xbar
      if (rows) {
        small_phase<G, true>(AT, V[SV_YBAR], EpiStore{V[SV_G]}, prm, j, none);
        RedOut r = none;
        for (int s = 0; s < 4; ++s) r.slot[s] = (int8_t)(SL_RA + s);
        r.active = 1;
        small_phase<G, true>(A, V[SV_XB], EpiResA{V[SV_L], V[SV_U], V[SV_YBAR], V[SV_IE]}, prm, j, r);
      }
      RedOut r = none;
      for (int s = 0; s < 7; ++s) r.slot[s] = (int8_t)(SL_RQ + s);
      r.active = 1;
      small_phase<G, true>(Q, V[SV_XB],
                     EpiResQ{V[SV_XB], V[SV_ZB], rows ? V[SV_G] : nullptr, V[SV_C], V[SV_LB], V[SV_UB], V[SV_XBO],
                             V[SV_ZBO], V[SV_ID], a.l1},
                     prm, j, r);
    }
  }
  small_stage_out<STAGED>(a, V);
}
