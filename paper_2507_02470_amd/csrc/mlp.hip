// mlp.hip -- the warm-start surrogate: a 3-layer GELU MLP trained and run
// with hand-written BF16 MFMA GEMMs (FP32 accumulate) on gfx950.
//
// Every GEMM is C[M x N] = A[M x K] * B[K x N] with both operands stored so
// that K is the contiguous dimension (the library keeps transposed BF16
// copies of weights, activations and gradients, with every leading
// dimension padded to a multiple of 8 and zero-filled), which lets each
// lane fetch its 8 consecutive K values of a v_mfma_f32_32x32x16_bf16
// operand with one 16-byte load.
//
// A training step's arithmetic is a few microseconds on this chip; what it costs
// is launches and the latency chain of each.  So every elementwise step
// (standardization, bias, GELU, loss gradient, GELU', the BF16 copies and their
// transposes) runs in the epilogue of the GEMM that produces its operand, the K
// splits of a GEMM are waves of one block, and GEMMs that do not depend on each
// other share a launch: 7 launches for loss_grad and 1 for Adam (35 before;
// batch 256, 1021-512-512-2022, the whole step: 270 -> 98 us).
#include "hprqp_mlp.h"
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <string>
#include <utility>
#include <vector>

namespace hq {
extern thread_local std::string g_err;
}

typedef __bf16 hm_bf16x8 __attribute__((ext_vector_type(8)));
typedef float hm_f32x16 __attribute__((ext_vector_type(16)));
typedef uint16_t hm_u16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ uint16_t f2bf(float f) {
  const __bf16 b = (__bf16)f;   // round to nearest even
  return __builtin_bit_cast(uint16_t, b);
}
__device__ __forceinline__ float bf2f(uint16_t u) { return __builtin_bit_cast(float, (uint32_t)u << 16); }

static inline int rup8(int v) { return (v + 7) & ~7; }

__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_d(float z) {
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * 0.39894228040143268f * expf(-0.5f * z * z);
}

// ---------------------------------------------------------------------------
// The plain GEMM entry point (any strides).  Block = 4 waves in a 2 x 2 arrangement, each wave a 32 x 32 tile of
// C (one 32x32x16 MFMA per K step of 16).  Operand layout of the MFMA
// (measured on gfx950): lane l holds A[l%32][8(l/32) + e] and
// B[8(l/32) + e][l%32], e = 0..7; accumulator register v of lane l holds
// C[8(v/4) + 4(l/32) + v%4][l%32].
// A(i, k) = A[i*a_rs + k*a_cs], B(k, j) = B[k*b_rs + j*b_cs]; when a_cs == 1
// (resp. b_rs == 1) and the row start is 16-byte aligned the 8 values come
// from one vector load.
// Split K: blockIdx.z takes the K range [z kper, (z + 1) kper) (kper a
// multiple of 16) and writes its partial tile to W[z] (M x N, dense); a
// second kernel adds the partials in the order z = 0, 1, ... (deterministic).
// Without a split (W == nullptr) the tile goes to C directly.
// ---------------------------------------------------------------------------
#define HM_KUNROLL 8
__global__ __launch_bounds__(256) void k_gemm_bf16(int M, int N, int K, int kper, const uint16_t* __restrict__ A,
                                                  long long a_rs, long long a_cs, const uint16_t* __restrict__ B,
                                                  long long b_rs, long long b_cs, float* __restrict__ C, long long ldc,
                                                  int accumulate, float* __restrict__ W) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int li = lane & 31, lh = lane >> 5;
  const int i0 = blockIdx.x * 64 + (wv & 1) * 32;
  const int j0 = blockIdx.y * 64 + (wv >> 1) * 32;
  const int ia = i0 + li, jb = j0 + li;
  const int kbeg = blockIdx.z * kper, kend = min(K, kbeg + kper);
  const bool a_vec = (a_cs == 1) && ((a_rs & 7) == 0) && ((((uintptr_t)A) & 15) == 0);
  const bool b_vec = (b_rs == 1) && ((b_cs & 7) == 0) && ((((uintptr_t)B) & 15) == 0);
  hm_f32x16 acc = {};
  auto frag_a = [&](int kb) {
    hm_u16x8 au;
    if (a_vec && ia < M && kb + 8 <= kend) {
      au = *reinterpret_cast<const hm_u16x8*>(A + (long long)ia * a_rs + kb);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        au[e] = (ia < M && kb + e < kend) ? A[(long long)ia * a_rs + (long long)(kb + e) * a_cs] : 0;
    }
    return au;
  };
  auto frag_b = [&](int kb) {
    hm_u16x8 bu;
    if (b_vec && jb < N && kb + 8 <= kend) {
      bu = *reinterpret_cast<const hm_u16x8*>(B + (long long)jb * b_cs + kb);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        bu[e] = (jb < N && kb + e < kend) ? B[(long long)(kb + e) * b_rs + (long long)jb * b_cs] : 0;
    }
    return bu;
  };
  // software pipeline: the fragments of the next HM_KUNROLL k-steps are
  // loaded before the MFMAs of the current ones, so their latency overlaps
  // the matrix-core work instead of stalling it
  hm_u16x8 au[HM_KUNROLL], bu[HM_KUNROLL];
#pragma unroll
  for (int u = 0; u < HM_KUNROLL; ++u) {
    const int kb = kbeg + 16 * u + 8 * lh;
    au[u] = frag_a(kb);
    bu[u] = frag_b(kb);
  }
  for (int k0 = kbeg; k0 < kend; k0 += 16 * HM_KUNROLL) {
    const int k1 = k0 + 16 * HM_KUNROLL;
    hm_u16x8 an[HM_KUNROLL], bn[HM_KUNROLL];
    if (k1 < kend) {
#pragma unroll
      for (int u = 0; u < HM_KUNROLL; ++u) {
        const int kb = k1 + 16 * u + 8 * lh;
        an[u] = frag_a(kb);
        bn[u] = frag_b(kb);
      }
    }
#pragma unroll
    for (int u = 0; u < HM_KUNROLL; ++u)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(hm_bf16x8, au[u]),
                                                    __builtin_bit_cast(hm_bf16x8, bu[u]), acc, 0, 0, 0);
    if (k1 < kend) {
#pragma unroll
      for (int u = 0; u < HM_KUNROLL; ++u) {
        au[u] = an[u];
        bu[u] = bn[u];
      }
    }
  }
  float* const Wz = W ? W + (size_t)blockIdx.z * M * N : nullptr;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int row = i0 + 8 * (v >> 2) + 4 * lh + (v & 3);
    const int col = j0 + li;
    if (row < M && col < N) {
      if (Wz) Wz[(size_t)row * N + col] = acc[v];
      else C[(long long)row * ldc + col] = accumulate ? C[(long long)row * ldc + col] + acc[v] : acc[v];
    }
  }
}

// C (+)= sum over z = 0..S-1 of W[z] (M x N each), in that order
__global__ void k_splitk_reduce(int M, int N, int S, const float* __restrict__ W, float* __restrict__ C, long long ldc,
                                int accumulate) {
  const long long total = (long long)M * N;
  for (long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (long long)gridDim.x * blockDim.x) {
    float sum = W[t];
    for (int z = 1; z < S; ++z) sum += W[(size_t)z * total + t];
    float* p = C + (t / N) * ldc + t % N;
    *p = accumulate ? *p + sum : sum;
  }
}

// ---------------------------------------------------------------------------
// The network's GEMMs.  A job is C (M x N) = A B^T over K-contiguous operands
// (A[i lda + k], B[j ldb + k], K and both ld multiples of 8) in 32 x 32 tiles;
// S waves of a block share a tile's K (slices of whole 16-steps, as many as
// gemm_splits gives), their partial tiles are added through LDS in slice order,
// and the job's epilogue runs on the sums.  A block of NW waves takes NW / S
// tiles; a launch takes up to two jobs and the column sums of one bias gradient.
// At these sizes (a 512 x 512 output is 256 tiles) a launch is bound by its chain
// of latencies: few k-steps a wave, all of its loads in flight at once.
// ---------------------------------------------------------------------------
enum { HM_HIDDEN, HM_OUT, HM_BACK, HM_WGRAD };
struct MlpJob {
  int kind = HM_WGRAD;
  int M = 0, N = 0, K = 0, S = 1, kper = 0, tiles_m = 0, tiles = 0, blocks = 0;
  const uint16_t *A = nullptr, *B = nullptr;
  int lda = 0, ldb = 0;
  // epilogue, by kind:
  //  HIDDEN  Z = sum + bias; act = BF16(GELU(Z)), actT its transpose
  //  OUT     Z = sum + bias (standardized output); user = out_mean + out_sd Z;
  //          or the warm start; or the loss and its gradient dY (gf, act, actT)
  //  BACK    dA = sum; gf = dA GELU'(Z), act and actT its BF16 copies
  //  WGRAD   C = sum, C2 too if given
  float *C = nullptr, *C2 = nullptr, *Z = nullptr, *gf = nullptr;
  uint16_t *act = nullptr, *actT = nullptr;
  const float* bias = nullptr;
  int ld = 0, ldt = 0;    // leading dimensions of C / Z / gf / act, and of actT (rows M .. ldt - 1 are zeroed)
};
struct MlpOut {           // the OUT epilogue's data
  const float *mean = nullptr, *sd = nullptr, *istd = nullptr;
  float* user = nullptr;                                   // batch x N
  const double *L = nullptr, *U = nullptr;                 // warm start (w0 given)
  double *y0 = nullptr, *w0 = nullptr, *x0 = nullptr;
  int* bad = nullptr;
  float* score = nullptr;
  int n = 0, m = 0;
  const float *T = nullptr, *w = nullptr;                  // loss (T given)
  float* Tstd = nullptr;
  double* partial = nullptr;                               // one per block
};
struct ColSum { const float* dZ = nullptr; float *db = nullptr, *db2 = nullptr; int B = 0, N = 0, ld = 0, blocks = 0; };
struct MlpLaunch { MlpJob job[2]; MlpOut out; ColSum cs; };

#define HM_PITCH 33
#define HM_SLAB 64     // K of a slab: one 128-byte line of every row
#define HM_RING 3      // slabs in flight

// Partial tile of a wave: MFMAs over the k-steps of [kbeg, kend), in order.  A
// slab of 32 rows x 64 k of each operand is loaded line by line (8 rows a load, 16
// bytes a lane; loading MFMA fragments directly touches 32 lines a load, and
// eight waves then refetch every line four times through the L1), passes
// through the wave's own LDS, its 16-byte chunks swizzled by row so that neither
// side has bank conflicts, and is read back as fragments.  Loads run HM_RING
// slabs ahead.
__device__ __forceinline__ hm_f32x16 mlp_tile(const MlpJob& J, int i0, int j0, int kbeg, int kend, hm_u16x8* lds) {
  const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5, lr = lane >> 3, lc = lane & 7;
  const uint16_t *Ar[4], *Br[4];   // the lane's rows (past the edge: clamped, not stored)
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    Ar[q] = J.A + (long long)min(i0 + lr + 8 * q, J.M - 1) * J.lda;
    Br[q] = J.B + (long long)min(j0 + lr + 8 * q, J.N - 1) * J.ldb;
  }
  hm_f32x16 acc = {};
  hm_u16x8 a[HM_RING][4], b[HM_RING][4];
  auto load = [&](int s, int k0) {
    const int kb = min(k0 + 8 * lc, kend - 8);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      a[s][q] = *reinterpret_cast<const hm_u16x8*>(Ar[q] + kb);
      b[s][q] = *reinterpret_cast<const hm_u16x8*>(Br[q] + kb);
    }
  };
  // a lane reads what other lanes of its wave wrote, and they write again: LDS
  // accesses keep their order across this (no instruction comes of it: a wave's
  // LDS operations complete in order)
  auto exchange = [&] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  auto mul = [&](int s, int k0) {
    exchange();   // (here, and not behind the reads: the loads of a later slab may pass them)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      lds[(lr + 8 * q) * 8 + (lc ^ lr)] = a[s][q];
      lds[256 + (lr + 8 * q) * 8 + (lc ^ lr)] = b[s][q];
    }
    exchange();
    hm_u16x8 fa[4], fb[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      fa[u] = lds[li * 8 + ((2 * u + lh) ^ (li & 7))];
      fb[u] = lds[256 + li * 8 + ((2 * u + lh) ^ (li & 7))];
    }
    const bool part = k0 + HM_SLAB > kend;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (part) {
        if (k0 + 16 * u >= kend) break;
        if (k0 + 16 * u + 8 >= kend && lh) { fa[u] = hm_u16x8{}; fb[u] = hm_u16x8{}; }   // half a step left
      }
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(hm_bf16x8, fa[u]),
                                                    __builtin_bit_cast(hm_bf16x8, fb[u]), acc, 0, 0, 0);
    }
  };
  // (a slab past the end is the last entries again, unused)
#pragma unroll
  for (int s = 0; s < HM_RING; ++s)
    if (kbeg + s * HM_SLAB < kend) load(s, kbeg + s * HM_SLAB);
  int k0 = kbeg;
  for (; k0 + HM_RING * HM_SLAB < kend; k0 += HM_RING * HM_SLAB) {
#pragma unroll
    for (int s = 0; s < HM_RING; ++s) {
      mul(s, k0 + s * HM_SLAB);
      load(s, k0 + (s + HM_RING) * HM_SLAB);
    }
  }
#pragma unroll
  for (int s = 0; s < HM_RING; ++s)
    if (k0 + s * HM_SLAB < kend) mul(s, k0 + s * HM_SLAB);
  return acc;
}

template <int NW>
__global__ __launch_bounds__(64 * NW) void k_mlp_gemm(MlpLaunch p) {
  // the waves' operand slabs, then the partial tiles and the tiles to transpose
  __shared__ hm_u16x8 slab[NW][512];
  static_assert(sizeof(slab[0]) >= 32 * HM_PITCH * sizeof(float) + 32 * (HM_PITCH + 1) * sizeof(uint16_t), "reuse");
  float (*const part)[32 * HM_PITCH] = reinterpret_cast<float (*)[32 * HM_PITCH]>(&slab[0][0]);
  uint16_t (*const tr)[32 * (HM_PITCH + 1)] = reinterpret_cast<uint16_t (*)[32 * (HM_PITCH + 1)]>(part + NW);
  const int t = threadIdx.x, lane = t & 63;
  int blk = blockIdx.x;
  if (blk >= p.job[0].blocks + p.job[1].blocks) {
    // db[j] = sum_b dZ[b][j]: 8 NW columns a block, thread (g, c) summing rows g,
    // g + 8, ... of its column in FP64, the 8 sums of a column added in order
    constexpr int CW = 8 * NW;
    double* const ps = reinterpret_cast<double*>(&slab[0][0]);
    const int c = t % CW, g = t / CW, j = (blk - p.job[0].blocks - p.job[1].blocks) * CW + c;
    double s = 0.0;
    if (j < p.cs.N) {
#pragma unroll 8
      for (int b = g; b < p.cs.B; b += 8) s += p.cs.dZ[(long long)b * p.cs.ld + j];
    }
    ps[g * CW + c] = s;
    __syncthreads();
    if (g == 0 && j < p.cs.N) {
      double r = ps[c];
#pragma unroll
      for (int q = 1; q < 8; ++q) r += ps[q * CW + c];
      p.cs.db[j] = (float)r;
      if (p.cs.db2) p.cs.db2[j] = (float)r;
    }
    return;
  }
  const bool second = blk >= p.job[0].blocks;
  if (second) blk -= p.job[0].blocks;
  const MlpJob& J = p.job[second ? 1 : 0];
  const int S = J.S, wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int tt = wv / S, tile = blk * (NW / S) + tt;   // the wave's tile, in its products and its epilogue
  const int i0 = (tile % J.tiles_m) * 32, j0 = (tile / J.tiles_m) * 32;
  // epilogue: 64 S threads per tile, thread tl taking column tl % 32 of rows
  // tl / 32, tl / 32 + 2 S, ...: its operands are loaded before the products
  const int P = 64 * S, tl = t - tt * P, c = tl & 31, col = j0 + c;
  const bool cin = tile < J.tiles && col < J.N;
  const MlpOut& o = p.out;
  const bool lossy = J.kind == HM_OUT && o.T != nullptr;
  float cb = 0.0f, cm = 0.0f, cs = 0.0f, ci = 0.0f, cw = 1.0f, er[16];
  double cL = 0.0, cU = 0.0;
  if (cin && J.bias) cb = J.bias[col];
  if (cin && J.kind == HM_OUT) {
    cm = o.mean[col]; cs = o.sd[col]; ci = o.istd[col];
    if (o.w) cw = o.w[col];
    if (o.w0 && col >= o.m + o.n && col < o.m + 2 * o.n) { cL = o.L[col - o.m - o.n]; cU = o.U[col - o.m - o.n]; }
  }
  const float* const ex = lossy ? o.T : J.kind == HM_BACK ? J.Z : nullptr;   // one operand per element
  const long long ex_ld = lossy ? J.N : J.ld;
#pragma unroll
  for (int q = 0; q < 16; ++q)
    if (ex && q * P < 1024) {
      const int row = i0 + ((tl + q * P) >> 5);
      er[q] = cin && row < J.M ? ex[row * ex_ld + col] : 0.0f;
    }
  {
    const int z = wv % S, kbeg = z * J.kper, kend = min(J.K, kbeg + J.kper);
    const bool work = tile < J.tiles && kbeg < kend;
    hm_f32x16 acc = {};
    if (work) acc = mlp_tile(J, i0, j0, kbeg, kend, slab[wv]);
    __syncthreads();   // the slabs' memory holds the partial tiles now
    if (work) {
      const int li = lane & 31, lh = lane >> 5;
#pragma unroll
      for (int v = 0; v < 16; ++v) part[wv][(8 * (v >> 2) + 4 * lh + (v & 3)) * HM_PITCH + li] = acc[v];
    }
  }
  __syncthreads();
  const int nz = (J.K + J.kper - 1) / J.kper;
  const double scale = lossy ? 1.0 / ((double)J.M * (double)J.N) : 0.0;
  const float gscale = (float)(2.0 * scale);
  double lacc = 0.0;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    if (q * P >= 1024) break;
    const int r = (tl + q * P) >> 5, row = i0 + r;
    uint16_t hb = 0;
    if (cin && row < J.M) {
      float v = part[tt * S][r * HM_PITCH + c];
      for (int z = 1; z < nz; ++z) v += part[tt * S + z][r * HM_PITCH + c];
      const long long at = (long long)row * J.ld + col;
      switch (J.kind) {
        case HM_HIDDEN: {
          v += cb;
          J.Z[at] = v;
          hb = f2bf(gelu(v));
          J.act[at] = hb;
          break;
        }
        case HM_OUT: {
          v += cb;
          J.Z[at] = v;
          if (o.user) o.user[(long long)row * J.N + col] = __builtin_fmaf(cs, v, cm);
          if (o.w0) {
            // prediction [y (m); z (n); w (n) (; ell)] -> FP64 start; z is not read by the iteration
            const float f = __builtin_fmaf(cs, v, cm);
            const int m = o.m, n = o.n, j = col - m - n;
            if (col < m) {
              if (!isfinite(f)) atomicOr(o.bad + row, 1);
              o.y0[(long long)row * m + col] = (double)f;
            } else if (j >= 0 && j < n) {
              if (!isfinite(f)) atomicOr(o.bad + row, 1);
              o.w0[(long long)row * n + j] = (double)f;
              o.x0[(long long)row * n + j] = fmin(fmax((double)f, cL), cU);
            } else if (j == n && o.score) {
              o.score[row] = f;
            }
          }
          if (lossy) {
            // weighted MSE: dY = 2 w (Y - T) / (B N).  The standardized target is
            // rounded before the difference (the empty asm keeps them apart).
            float ts = (er[q] - cm) * ci;
            asm volatile("" : "+v"(ts));
            o.Tstd[(long long)row * J.N + col] = ts;
            const float d = v - ts;
            lacc += (double)cw * (double)d * (double)d;
            const float g = gscale * cw * d;
            J.gf[at] = g;
            hb = f2bf(g);
            J.act[at] = hb;
          }
          break;
        }
        case HM_BACK: {
          J.C[at] = v;
          const float g = v * gelu_d(er[q]);
          J.gf[at] = g;
          hb = f2bf(g);
          J.act[at] = hb;
          break;
        }
        default: {
          J.C[at] = v;
          if (J.C2) J.C2[at] = v;
        }
      }
    }
    if (J.actT) tr[tt][c * (HM_PITCH + 1) + r] = hb;
  }
  if (J.actT) {
    __syncthreads();
    if (tile < J.tiles)
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        if (q * P >= 1024) break;
        const int cc = (tl + q * P) >> 5, r = tl & 31;
        if (j0 + cc < J.N && i0 + r < J.ldt)
          J.actT[(long long)(j0 + cc) * J.ldt + i0 + r] = tr[tt][cc * (HM_PITCH + 1) + r];
      }
  }
  if (lossy) {
    double* const ps = reinterpret_cast<double*>(&slab[0][0]);
    for (int off = 32; off; off >>= 1) lacc += __shfl_xor(lacc, off);
    __syncthreads();
    if (lane == 0) ps[wv] = lacc;
    __syncthreads();
    if (t == 0) {
      double s = ps[0];
      for (int w = 1; w < NW; ++w) s += ps[w];
      o.partial[blk] = s * scale;
    }
  }
}

// Network input: Xb (rows x cols_p, BF16) <- (X - mean) * inv_std, zero padding,
// and its transpose Xt (cols_p x rows_p) if given; clears `bad` (rows) if given.
// A block takes 32 x 32 tiles of its 32 columns: one, up to the 65,535 blocks a second
// grid dimension holds (2.1 million samples), then every 65,535th.
#define HM_INPUT_ROWS 65535
__global__ __launch_bounds__(256) void k_mlp_input(int rows, int rows_p, int cols, int cols_p, const float* __restrict__ X,
                                                   const float* __restrict__ mean, const float* __restrict__ inv_std,
                                                   uint16_t* __restrict__ Xb, uint16_t* __restrict__ Xt,
                                                   int* __restrict__ bad) {
  __shared__ uint16_t tile[32][33];
  const int c0 = blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8 threads
  const int c = c0 + tx;
  const float mu = c < cols ? mean[c] : 0.0f, is = c < cols ? inv_std[c] : 0.0f;
  for (int r0 = blockIdx.y * 32;;) {
#pragma unroll
    for (int y = ty; y < 32; y += 8) {
      const int r = r0 + y;
      uint16_t u = 0;
      if (r < rows && c < cols) u = f2bf((X[(long long)r * cols + c] - mu) * is);
      if (r < rows && c < cols_p) Xb[(long long)r * cols_p + c] = u;
      if (Xt) tile[y][tx] = u;
    }
    if (bad && blockIdx.x == 0 && threadIdx.x < 32 && r0 + (int)threadIdx.x < rows) bad[r0 + threadIdx.x] = 0;
    if (Xt) {
      __syncthreads();
#pragma unroll
      for (int y = ty; y < 32; y += 8)
        if (c0 + y < cols_p && r0 + tx < rows_p) Xt[(long long)(c0 + y) * rows_p + r0 + tx] = tile[tx][y];
    }
    if (rows_p - r0 <= 32 * HM_INPUT_ROWS) return;
    r0 += 32 * HM_INPUT_ROWS;
    if (Xt) __syncthreads();   // (the next tile)
  }
}

// Samples whose predicted y or w is not finite start from the origin (the
// cold start of Algorithm 4): bad[s] = 1
__global__ __launch_bounds__(256) void k_warm_fix(int n, int m, const int* __restrict__ bad, double* __restrict__ y0,
                                                  double* __restrict__ w0, double* __restrict__ x0) {
  const long long s = blockIdx.x;
  if (!bad[s]) return;
  for (int i = threadIdx.x; i < m; i += blockDim.x) y0[s * m + i] = 0.0;
  for (int j = threadIdx.x; j < n; j += blockDim.x) { w0[s * n + j] = 0.0; x0[s * n + j] = 0.0; }
}

// out (rows x cols, FP32) <- a stage tensor with leading dimension ld, FP32
// or BF16 bits (exact widening)
__global__ void k_export(int rows, int cols, long long ld, const float* __restrict__ f32,
                         const uint16_t* __restrict__ b16, float* __restrict__ out) {
  const long long total = (long long)rows * cols;
  for (long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (long long)gridDim.x * blockDim.x) {
    const long long r = t / cols, c = t % cols;
    out[t] = f32 ? f32[r * ld + c] : __uint_as_float((unsigned)b16[r * ld + c] << 16);
  }
}

// Column statistics of a (rows x cols) FP32 matrix for the standardization:
// per column, the sum (pass 0) or the sum of squared deviations from `mean`
// (pass 1) over a chunk of rows into part[chunk][col], FP64, rows in order.
#define HM_STAT_ROWS 1024
__global__ void k_col_stats(long long rows, int cols, const float* __restrict__ X, const double* __restrict__ mean,
                            double* __restrict__ part) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= cols) return;
  const long long r0 = (long long)blockIdx.y * HM_STAT_ROWS, r1 = min(rows, r0 + HM_STAT_ROWS);
  double s = 0.0;
  for (long long r = r0; r < r1; ++r) {
    const double v = X[r * cols + j];
    s += mean ? (v - mean[j]) * (v - mean[j]) : v;
  }
  part[(long long)blockIdx.y * cols + j] = s;
}
// out[j] = sum of the chunks' partials in chunk order, divided by `div`
// (sqrt of it when `root`): the mean (div = rows) or the standard deviation
// (div = rows - 1)
__global__ void k_col_finish(int chunks, int cols, const double* __restrict__ part, double div, int root,
                             double* __restrict__ out64, float* __restrict__ out32) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= cols) return;
  double s = 0.0;
  for (int c = 0; c < chunks; ++c) s += part[(long long)c * cols + j];
  s /= div;
  if (root) s = sqrt(s);
  out64[j] = s;
  out32[j] = (float)s;
}

// Network input of family members: X[s] = [c_s (n); u_s (m)] in FP32
__global__ void k_family_features(int batch, int n, int m, const double* __restrict__ c, const double* __restrict__ u,
                                  float* __restrict__ X) {
  const long long total = (long long)batch * (n + m);
  for (long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (long long)gridDim.x * blockDim.x) {
    const long long s = t / (n + m);
    const int k = (int)(t % (n + m));
    X[t] = (float)(k < n ? c[s * n + k] : u[s * m + (k - n)]);
  }
}
// Training targets of family members: T[s] = [y_s (m); z_s (n); w_s (n)] in
// FP32, and with iters given a last column log(max(iters_s, 1)) (the length of
// the solve that produced the member's solution)
__global__ void k_family_targets(int batch, int n, int m, const double* __restrict__ y, const double* __restrict__ z,
                                 const double* __restrict__ w, const long long* __restrict__ iters,
                                 float* __restrict__ T) {
  const int no = m + 2 * n + (iters ? 1 : 0);
  const long long total = (long long)batch * no;
  for (long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (long long)gridDim.x * blockDim.x) {
    const long long s = t / no;
    const int k = (int)(t % no);
    T[t] = k < m ? (float)y[s * m + k]
         : k < m + n ? (float)z[s * n + (k - m)]
         : k < m + 2 * n ? (float)w[s * n + (k - m - n)]
         : (float)log((double)(iters[s] > 1 ? iters[s] : 1));
  }
}

__device__ __forceinline__ float adam_step(float& p, float g, float& m, float& v, float lr, float b1, float b2,
                                           float eps, float c1, float c2) {
  const float mi = b1 * m + (1.0f - b1) * g;
  const float vi = b2 * v + (1.0f - b2) * g * g;
  m = mi; v = vi;
  p -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  return p;
}

// One Adam step on every parameter, and the BF16 copies of the weights, Wb
// (rows x cols_p) and its transpose Wt (cols x rows_p), from the tile just
// updated.  Blocks take the 32 x 32 tiles of the three weight matrices, then the
// biases.  (The copies' padding is zero from creation.)  step = 0: the copies only.
struct AdamArgs {
  float *p, *m, *v;
  const float* g;
  long long off_W[3], off_b[3];
  int rows[3], cols[3], rows_p[3], cols_p[3], tiles[3];
  uint16_t *Wb[3], *Wt[3];
  float lr, b1, b2, eps, c1, c2;
  int step;
};
__global__ __launch_bounds__(256) void k_adam(AdamArgs a) {
  __shared__ uint16_t tile[32][33];
  int blk = blockIdx.x;
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    if (blk < a.tiles[l]) {
      const int tn = (a.cols[l] + 31) / 32, c0 = (blk % tn) * 32, r0 = (blk / tn) * 32;
      const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
      const int c = c0 + tx;
      float pv[4], gv[4], mv[4], vv[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = r0 + ty + 8 * q;
        if (r < a.rows[l] && c < a.cols[l]) {
          const long long i = a.off_W[l] + (long long)r * a.cols[l] + c;
          pv[q] = a.p[i];
          if (a.step) { gv[q] = a.g[i]; mv[q] = a.m[i]; vv[q] = a.v[i]; }
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = r0 + ty + 8 * q;
        if (r < a.rows[l] && c < a.cols[l]) {
          const long long i = a.off_W[l] + (long long)r * a.cols[l] + c;
          if (a.step) {
            a.p[i] = adam_step(pv[q], gv[q], mv[q], vv[q], a.lr, a.b1, a.b2, a.eps, a.c1, a.c2);
            a.m[i] = mv[q]; a.v[i] = vv[q];
          }
          const uint16_t u = f2bf(pv[q]);
          a.Wb[l][(long long)r * a.cols_p[l] + c] = u;
          tile[ty + 8 * q][tx] = u;
        }
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int cc = c0 + ty + 8 * q, r = r0 + tx;
        if (cc < a.cols[l] && r < a.rows[l]) a.Wt[l][(long long)cc * a.rows_p[l] + r] = tile[tx][ty + 8 * q];
      }
      return;
    }
    blk -= a.tiles[l];
  }
  if (!a.step) return;
  // biases, one after the other in thread order
  long long k = (long long)blk * 256 + threadIdx.x;
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    if (k < a.rows[l]) {
      const long long i = a.off_b[l] + k;
      float pv = a.p[i], mv = a.m[i], vv = a.v[i];
      a.p[i] = adam_step(pv, a.g[i], mv, vv, a.lr, a.b1, a.b2, a.eps, a.c1, a.c2);
      a.m[i] = mv; a.v[i] = vv;
      return;
    }
    k -= a.rows[l];
  }
}

// ---------------------------------------------------------------------------
// network object
// ---------------------------------------------------------------------------
struct hprqp_mlp {
  int d[4];          // n_in, h1, h2, n_out
  int dp[4];         // padded to multiples of 8
  int maxb, maxbp;
  hipStream_t st = nullptr, own_st = nullptr;
  long long np = 0;
  long long off_W[3], off_b[3];
  float *P = nullptr, *G = nullptr, *Mm = nullptr, *Vv = nullptr;   // params, grad, Adam moments
  long long adam_t = 0;
  uint16_t *Wb[3] = {}, *Wt[3] = {};
  uint16_t *Xb = nullptr, *Xt = nullptr, *A1b = nullptr, *A1t = nullptr, *A2b = nullptr, *A2t = nullptr;
  float *Z1 = nullptr, *Z2 = nullptr, *Y = nullptr;
  float *dYf = nullptr, *dA2 = nullptr, *dZ2f = nullptr, *dA1 = nullptr, *dZ1f = nullptr;
  uint16_t *dYb = nullptr, *dYt = nullptr, *dZ2b = nullptr, *dZ2t = nullptr, *dZ1b = nullptr, *dZ1t = nullptr;
  double* loss_part = nullptr;  // pinned host memory: the loss of each block of the output layer
  int ncu = 0;
  // input / output standardization (set by hprqp_mlp_set_scaling; identity by default)
  float *in_mean = nullptr, *in_istd = nullptr, *out_mean = nullptr, *out_sd = nullptr, *out_istd = nullptr;
  float* Tstd = nullptr;
  std::vector<void*> owned;
  hipEvent_t ev[4] = {};
  int nev = 0;
  double last_flop = 0.0;
  int last_batch = 0;   // batch of the last forward / loss_grad
  ~hprqp_mlp() {
    for (void* p : owned) hipFree(p);
    for (auto e : ev)
      if (e) hipEventDestroy(e);
    if (loss_part) hipHostFree(loss_part);
    if (own_st) hipStreamDestroy(own_st);
  }
};

namespace {
struct MErr {
  hprqp_status st;
  std::string msg;
};
[[noreturn]] void mfail(hprqp_status st, const std::string& m) { throw MErr{st, m}; }
void mcheck(hipError_t e, const char* w) {
  if (e != hipSuccess) {
    if (e == hipErrorOutOfMemory) mfail(HPRQP_ERR_OOM, std::string(w) + ": out of device memory");
    mfail(HPRQP_ERR_HIP, std::string(w) + ": " + hipGetErrorString(e));
  }
}
#define HMC(x) mcheck((x), #x)

// The handle's device arrays: asked for one by one, then taken (zeroed) from one
// allocation
struct Arena {
  std::vector<std::pair<void**, size_t>> want;
  size_t bytes = 0;
  template <class T>
  void add(T*& p, size_t count) {
    want.emplace_back((void**)&p, bytes);
    bytes += (std::max<size_t>(count, 1) * sizeof(T) + 255) / 256 * 256;
  }
  void take(hprqp_mlp& n) {
    void* base = nullptr;
    HMC(hipMalloc(&base, bytes));
    n.owned.push_back(base);
    HMC(hipMemsetAsync(base, 0, bytes, n.st));
    for (auto& w : want) *w.first = (char*)base + w.second;
  }
};

int eg(long long work) {
  long long g = (work + 255) / 256;
  return (int)std::max(1LL, std::min(g, 4096LL));
}

// K splits of a network GEMM, waves of the block that has the tile: doubled while the
// launch holds fewer than 4 waves per CU (a wave per 32 x 32 tile and split, counted in
// fours) and each split keeps at least 4 k-steps of 16.  The network's GEMMs are small: a
// 512 x 512 output is 256 tiles, a wave a CU, too few to hide the operand loads.
int gemm_splits(int M, int N, int K, int ncu) {
  const long long waves = 4LL * ((M + 63) / 64) * ((N + 63) / 64);
  const int ksteps = (K + 15) / 16;
  int S = 1;
  while (S < 8 && waves * S < 4LL * ncu && ksteps >= 8 * S) S *= 2;
  return S;
}

// C (+)= A B with S K-splits (S > 1: the partials go through ws, which holds
// at least S M N floats)
void gemm_split(hipStream_t st, int M, int N, int K, const uint16_t* A, long long a_rs, long long a_cs,
                const uint16_t* B, long long b_rs, long long b_cs, float* C, long long ldc, int acc, int S, float* ws) {
  const int ksteps = (K + 15) / 16;
  if (S < 1) S = 1;
  const int kper = 16 * ((ksteps + S - 1) / S);
  const int Se = kper > 0 ? (K + kper - 1) / kper : 1;
  if (Se <= 1) {
    dim3 grid((M + 63) / 64, (N + 63) / 64, 1);
    k_gemm_bf16<<<grid, 256, 0, st>>>(M, N, K, std::max(kper, 16), A, a_rs, a_cs, B, b_rs, b_cs, C, ldc, acc, nullptr);
    return;
  }
  dim3 grid((M + 63) / 64, (N + 63) / 64, Se);
  k_gemm_bf16<<<grid, 256, 0, st>>>(M, N, K, kper, A, a_rs, a_cs, B, b_rs, b_cs, C, ldc, acc, ws);
  k_splitk_reduce<<<eg((long long)M * N), 256, 0, st>>>(M, N, Se, ws, C, ldc, acc);
}

// a job of the network: operands and shape; the caller fills in the epilogue
MlpJob job(const hprqp_mlp& n, int kind, int M, int N, int K, const uint16_t* A, int lda, const uint16_t* B, int ldb) {
  MlpJob J;
  J.kind = kind; J.M = M; J.N = N; J.K = K;
  J.A = A; J.lda = lda; J.B = B; J.ldb = ldb;
  J.S = gemm_splits(M, N, K, n.ncu);
  J.kper = 16 * (((K + 15) / 16 + J.S - 1) / J.S);
  J.tiles_m = (M + 31) / 32;
  J.tiles = J.tiles_m * ((N + 31) / 32);
  return J;
}
ColSum colsum(int B, int N, const float* dZ, int ld, float* db, float* db2) {
  ColSum c;
  c.B = B; c.N = N; c.dZ = dZ; c.ld = ld; c.db = db; c.db2 = db2;
  return c;
}
// Waves per block: 8 where a tile's K is shared by 8, else 4 (more blocks: the
// output layer at batch 512 is 1024 tiles).  Returns the first job's blocks.
int launch(hprqp_mlp& n, MlpLaunch p) {
  const int NW = p.job[0].S == 8 || p.job[1].S == 8 ? 8 : 4;
  for (MlpJob& J : p.job) J.blocks = (J.tiles * J.S + NW - 1) / NW;
  p.cs.blocks = (p.cs.N + 8 * NW - 1) / (8 * NW);
  const int grid = p.job[0].blocks + p.job[1].blocks + p.cs.blocks;
  if (NW == 8) k_mlp_gemm<8><<<grid, 512, 0, n.st>>>(p);
  else k_mlp_gemm<4><<<grid, 256, 0, n.st>>>(p);
  return p.job[0].blocks;
}

AdamArgs adam_args(hprqp_mlp& n) {
  AdamArgs a{};
  a.p = n.P; a.m = n.Mm; a.v = n.Vv; a.g = n.G;
  for (int l = 0; l < 3; ++l) {
    a.off_W[l] = n.off_W[l]; a.off_b[l] = n.off_b[l];
    a.rows[l] = n.d[l + 1]; a.cols[l] = n.d[l]; a.rows_p[l] = n.dp[l + 1]; a.cols_p[l] = n.dp[l];
    a.tiles[l] = ((a.rows[l] + 31) / 32) * ((a.cols[l] + 31) / 32);
    a.Wb[l] = n.Wb[l]; a.Wt[l] = n.Wt[l];
  }
  return a;
}
void refresh_weights(hprqp_mlp& n) {
  const AdamArgs a = adam_args(n);
  k_adam<<<a.tiles[0] + a.tiles[1] + a.tiles[2], 256, 0, n.st>>>(a);
}

void create_impl(const int32_t dims[4], int32_t max_batch, const float* params_host, hipStream_t st, hprqp_mlp** out) {
  if (!dims || !out || max_batch <= 0) mfail(HPRQP_ERR_ARG, "bad arguments");
  for (int i = 0; i < 4; ++i)
    if (dims[i] <= 0 || dims[i] > (1 << 16)) mfail(HPRQP_ERR_SHAPE, "layer sizes must be in [1, 65536]");
  auto* n = new hprqp_mlp();
  try {
    if (!st) {
      HMC(hipStreamCreateWithFlags(&n->own_st, hipStreamNonBlocking));
      HMC(hipDeviceSynchronize());
      st = n->own_st;
    }
    n->st = st;
    for (int i = 0; i < 4; ++i) { n->d[i] = dims[i]; n->dp[i] = rup8(dims[i]); }
    n->maxb = max_batch;
    n->maxbp = rup8(max_batch);
    long long o = 0;
    for (int l = 0; l < 3; ++l) {
      n->off_W[l] = o; o += (long long)n->d[l + 1] * n->d[l];
      n->off_b[l] = o; o += n->d[l + 1];
    }
    n->np = o;
    Arena mem;
    mem.add(n->P, o);
    mem.add(n->G, o);
    mem.add(n->Mm, o);
    mem.add(n->Vv, o);
    for (int l = 0; l < 3; ++l) {
      mem.add(n->Wb[l], (size_t)n->dp[l + 1] * n->dp[l]);
      mem.add(n->Wt[l], (size_t)n->dp[l + 1] * n->dp[l]);
    }
    const size_t B = n->maxbp;
    mem.add(n->Xb, B * n->dp[0]);
    mem.add(n->Xt, B * n->dp[0]);
    mem.add(n->A1b, B * n->dp[1]);
    mem.add(n->A1t, B * n->dp[1]);
    mem.add(n->A2b, B * n->dp[2]);
    mem.add(n->A2t, B * n->dp[2]);
    mem.add(n->Z1, B * n->dp[1]);
    mem.add(n->Z2, B * n->dp[2]);
    mem.add(n->Y, B * n->dp[3]);
    mem.add(n->dYf, B * n->dp[3]);
    mem.add(n->dYb, B * n->dp[3]);
    mem.add(n->dYt, B * n->dp[3]);
    mem.add(n->dA2, B * n->dp[2]);
    mem.add(n->dZ2f, B * n->dp[2]);
    mem.add(n->dZ2b, B * n->dp[2]);
    mem.add(n->dZ2t, B * n->dp[2]);
    mem.add(n->dA1, B * n->dp[1]);
    mem.add(n->dZ1f, B * n->dp[1]);
    mem.add(n->dZ1b, B * n->dp[1]);
    mem.add(n->dZ1t, B * n->dp[1]);
    {
      int dev = 0;
      HMC(hipGetDevice(&dev));
      HMC(hipDeviceGetAttribute(&n->ncu, hipDeviceAttributeMultiprocessorCount, dev));
      // at most one block per tile of the output layer
      const size_t most = ((B + 31) / 32) * ((size_t)(n->d[3] + 31) / 32);
      HMC(hipHostMalloc((void**)&n->loss_part, most * sizeof(double), hipHostMallocDefault));
    }
    mem.add(n->in_mean, n->d[0]);
    mem.add(n->in_istd, n->d[0]);
    mem.add(n->out_mean, n->d[3]);
    mem.add(n->out_sd, n->d[3]);
    mem.add(n->out_istd, n->d[3]);
    mem.add(n->Tstd, (size_t)n->maxb * n->d[3]);
    mem.take(*n);
    if (params_host) HMC(hipMemcpyAsync(n->P, params_host, o * sizeof(float), hipMemcpyHostToDevice, st));
    {
      std::vector<float> ones(std::max(n->d[0], n->d[3]), 1.0f);
      HMC(hipMemcpyAsync(n->in_istd, ones.data(), n->d[0] * sizeof(float), hipMemcpyHostToDevice, st));
      HMC(hipMemcpyAsync(n->out_sd, ones.data(), n->d[3] * sizeof(float), hipMemcpyHostToDevice, st));
      HMC(hipMemcpyAsync(n->out_istd, ones.data(), n->d[3] * sizeof(float), hipMemcpyHostToDevice, st));
      HMC(hipStreamSynchronize(st));
    }
    for (auto& e : n->ev) HMC(hipEventCreate(&e));
    refresh_weights(*n);
    HMC(hipStreamSynchronize(st));
    *out = n;
  } catch (...) {
    delete n;
    throw;
  }
}

void mark(hprqp_mlp& n) { HMC(hipEventRecord(n.ev[n.nev++], n.st)); }

// Forward pass; `out`: what the output layer's epilogue makes of its result.
// train: the transposed copies and the loss (its partials in n.loss_part, one per
// block of the returned count).
int forward_impl(hprqp_mlp& n, int B, const float* X, const MlpOut& out) {
  if (B <= 0 || B > n.maxb || !X) mfail(HPRQP_ERR_ARG, "batch out of range or NULL input");
  n.last_batch = B;
  const bool train = out.T != nullptr;
  const int in = n.d[0], h1 = n.d[1], h2 = n.d[2], no = n.d[3];
  const int inp = n.dp[0], h1p = n.dp[1], h2p = n.dp[2], outp = n.dp[3];
  const int Bp = rup8(B);
  k_mlp_input<<<dim3((inp + 31) / 32, std::min((Bp + 31) / 32, HM_INPUT_ROWS)), 256, 0, n.st>>>(
      B, Bp, in, inp, X, n.in_mean, n.in_istd, n.Xb, train ? n.Xt : nullptr, out.bad);
  n.nev = 0;
  mark(n);
  auto hidden = [&](MlpJob J, float* Z, uint16_t* act, uint16_t* actT, const float* bias, int ld) {
    J.Z = Z; J.act = act; J.actT = train ? actT : nullptr; J.bias = bias; J.ld = ld; J.ldt = Bp;
    MlpLaunch p;
    p.job[0] = J;
    launch(n, p);
  };
  hidden(job(n, HM_HIDDEN, B, h1, inp, n.Xb, inp, n.Wb[0], inp), n.Z1, n.A1b, n.A1t, n.P + n.off_b[0], h1p);
  hidden(job(n, HM_HIDDEN, B, h2, h1p, n.A1b, h1p, n.Wb[1], h1p), n.Z2, n.A2b, n.A2t, n.P + n.off_b[1], h2p);
  MlpLaunch p;
  p.out = out;
  p.out.mean = n.out_mean; p.out.sd = n.out_sd; p.out.istd = n.out_istd;
  p.out.Tstd = n.Tstd;
  p.out.partial = n.loss_part;
  MlpJob J = job(n, HM_OUT, B, no, h2p, n.A2b, h2p, n.Wb[2], h2p);
  J.Z = n.Y; J.bias = n.P + n.off_b[2]; J.ld = outp;
  J.gf = n.dYf; J.act = n.dYb; J.actT = train ? n.dYt : nullptr; J.ldt = Bp;
  p.job[0] = J;
  const int parts = launch(n, p);
  mark(n);
  n.last_flop = 2.0 * B * ((double)inp * h1 + (double)h1p * h2 + (double)h2p * no);
  return parts;
}

// Warm starts of `count` samples in chunks of the network's batch: every chunk's
// launches are queued behind the last one's (they share its buffers, in the order of
// the stream), one wait at the end.  With a wait a chunk, 2,048 samples in chunks of
// 256 took 0.46 ms; with one, 0.33 ms.
void warm_impl(hprqp_mlp* n, int count, int most, const float* X, int qn, int qm, const double* L, const double* U,
               double* y0, double* w0, double* x0, int32_t* bad, float* score) {
  if (!n || !L || !U || !w0 || !x0 || !bad || (qm > 0 && !y0)) mfail(HPRQP_ERR_ARG, "NULL argument");
  if (qn <= 0 || qm < 0 || (qm + 2 * qn != n->d[3] && qm + 2 * qn + 1 != n->d[3]))
    mfail(HPRQP_ERR_SHAPE, "n_out must equal m + 2 n or m + 2 n + 1");
  if (score && qm + 2 * qn + 1 != n->d[3]) mfail(HPRQP_ERR_SHAPE, "score needs n_out = m + 2 n + 1");
  if (count <= 0 || count > most || !X) mfail(HPRQP_ERR_ARG, "batch out of range or NULL input");
  for (long long s = 0; s < count; s += n->maxb) {
    const int B = (int)std::min<long long>(n->maxb, count - s);
    MlpOut out;
    out.L = L; out.U = U; out.n = qn; out.m = qm;
    out.y0 = y0 ? y0 + s * qm : nullptr; out.w0 = w0 + s * qn; out.x0 = x0 + s * qn;
    out.bad = bad + s; out.score = score ? score + s : nullptr;
    forward_impl(*n, B, X + s * n->d[0], out);
    k_warm_fix<<<B, 256, 0, n->st>>>(qn, qm, out.bad, out.y0, out.w0, out.x0);
  }
  HMC(hipGetLastError());
  HMC(hipStreamSynchronize(n->st));
}

void loss_grad_impl(hprqp_mlp& n, int B, const float* X, const float* T, const float* w, float* loss_host,
                    float* grad) {
  if (!T) mfail(HPRQP_ERR_ARG, "NULL targets");
  MlpOut out;
  out.T = T; out.w = w;
  const int parts = forward_impl(n, B, X, out);
  const int in = n.d[0], h1 = n.d[1], h2 = n.d[2], no = n.d[3];
  const int h1p = n.dp[1], h2p = n.dp[2], outp = n.dp[3];
  const int Bp = rup8(B);
  const double fwd_flop = n.last_flop;
  float* const G = n.G;
  // a weight gradient (K = batch) into G and the caller's copy
  auto wgrad = [&](int l, int M, int N, const uint16_t* At, const uint16_t* Bt) {
    MlpJob J = job(n, HM_WGRAD, M, N, Bp, At, Bp, Bt, Bp);
    J.C = G + n.off_W[l]; J.C2 = grad ? grad + n.off_W[l] : nullptr; J.ld = N;
    return J;
  };
  auto back = [&](MlpJob J, float* dA, const float* Z, float* gf, uint16_t* act, uint16_t* actT, int ld) {
    J.C = dA; J.Z = const_cast<float*>(Z); J.gf = gf; J.act = act; J.actT = actT; J.ld = ld; J.ldt = Bp;
    return J;
  };
  auto bsum = [&](int l, int N, const float* dZ, int ld) {
    return colsum(B, N, dZ, ld, G + n.off_b[l], grad ? grad + n.off_b[l] : nullptr);
  };
  mark(n);
  MlpLaunch p;
  // dA2 = dY W3, dZ2 = dA2 GELU'(Z2); dW3 = dY^T A2, db3
  p.job[0] = back(job(n, HM_BACK, B, h2, outp, n.dYb, outp, n.Wt[2], outp), n.dA2, n.Z2, n.dZ2f, n.dZ2b, n.dZ2t, h2p);
  p.job[1] = wgrad(2, no, h2, n.dYt, n.A2t);
  p.cs = bsum(2, no, n.dYf, outp);
  launch(n, p);
  // dA1 = dZ2 W2, dZ1 = dA1 GELU'(Z1); dW2 = dZ2^T A1, db2
  p.job[0] = back(job(n, HM_BACK, B, h1, h2p, n.dZ2b, h2p, n.Wt[1], h2p), n.dA1, n.Z1, n.dZ1f, n.dZ1b, n.dZ1t, h1p);
  p.job[1] = wgrad(1, h2, h1, n.dZ2t, n.A1t);
  p.cs = bsum(1, h2, n.dZ2f, h2p);
  launch(n, p);
  // dW1 = dZ1^T X, db1
  p.job[0] = wgrad(0, h1, in, n.dZ1t, n.Xt);
  p.job[1] = MlpJob{};
  p.cs = bsum(0, h1, n.dZ1f, h1p);
  launch(n, p);
  mark(n);
  n.last_flop = fwd_flop + 2.0 * ((double)no * h2 * Bp + (double)B * h2 * outp + (double)h2 * h1 * Bp +
                                  (double)B * h1 * h2p + (double)h1 * in * Bp);
  HMC(hipGetLastError());
  HMC(hipStreamSynchronize(n.st));
  double L = 0.0;
  for (int q = 0; q < parts; ++q) L += n.loss_part[q];
  if (loss_host) *loss_host = (float)L;
}

}  // namespace

// mean and standard deviation (divisor rows - 1) of every column of X
// (rows x cols, device, FP32), FP64 on the device, into mean64/sd64 (device)
// and the host arrays mean_h/sd_h
void col_moments(hipStream_t st, long long rows, int cols, const float* X, float* mean_h, float* sd_h) {
  const int chunks = (int)((rows + HM_STAT_ROWS - 1) / HM_STAT_ROWS);
  double *part = nullptr, *mean = nullptr, *sd = nullptr;
  float* f32 = nullptr;
  const auto done = [&] {
    for (void* p : {(void*)part, (void*)mean, (void*)sd, (void*)f32})
      if (p) hipFree(p);
  };
  try {
    HMC(hipMalloc(&part, (size_t)chunks * cols * sizeof(double)));
    HMC(hipMalloc(&mean, cols * sizeof(double)));
    HMC(hipMalloc(&sd, cols * sizeof(double)));
    HMC(hipMalloc(&f32, cols * sizeof(float)));
    const dim3 g((cols + 255) / 256, chunks);
    k_col_stats<<<g, 256, 0, st>>>(rows, cols, X, nullptr, part);
    k_col_finish<<<(cols + 255) / 256, 256, 0, st>>>(chunks, cols, part, (double)rows, 0, mean, f32);
    HMC(hipMemcpyAsync(mean_h, f32, cols * sizeof(float), hipMemcpyDeviceToHost, st));
    k_col_stats<<<g, 256, 0, st>>>(rows, cols, X, mean, part);
    k_col_finish<<<(cols + 255) / 256, 256, 0, st>>>(chunks, cols, part, (double)std::max(1ll, rows - 1), 1, sd, f32);
    HMC(hipMemcpyAsync(sd_h, f32, cols * sizeof(float), hipMemcpyDeviceToHost, st));
    HMC(hipStreamSynchronize(st));
  } catch (...) {
    done();
    throw;
  }
  done();
}

#define HM_GUARD(...)                 \
  try {                               \
    hq::g_err.clear();                \
    __VA_ARGS__;                      \
    return HPRQP_OK;                  \
  } catch (const MErr& e) {           \
    hq::g_err = e.msg;                \
    return e.st;                      \
  } catch (const std::exception& e) { \
    hq::g_err = e.what();             \
    return HPRQP_ERR_HIP;             \
  }

extern "C" {

hprqp_status hprqp_mlp_create(const int32_t dims[4], int32_t max_batch, const float* params_host, hipStream_t stream,
                              hprqp_mlp** out) {
  HM_GUARD(create_impl(dims, max_batch, params_host, stream, out));
}

int64_t hprqp_mlp_num_params(const hprqp_mlp* n) { return n ? n->np : 0; }

hprqp_status hprqp_mlp_forward(hprqp_mlp* n, int32_t batch, const float* X, float* Y) {
  HM_GUARD(if (!n || !Y) mfail(HPRQP_ERR_ARG, "NULL argument"); MlpOut out; out.user = Y;
           forward_impl(*n, batch, X, out); HMC(hipGetLastError()); HMC(hipStreamSynchronize(n->st)));
}

hprqp_status hprqp_mlp_set_scaling(hprqp_mlp* n, const float* in_mean, const float* in_std, const float* out_mean,
                                   const float* out_std) {
  HM_GUARD(
      if (!n || !in_mean || !in_std || !out_mean || !out_std) mfail(HPRQP_ERR_ARG, "NULL argument");
      std::vector<float> ii(n->d[0]), oi(n->d[3]);
      for (int i = 0; i < n->d[0]; ++i) ii[i] = in_std[i] > 1e-12f ? 1.0f / in_std[i] : 0.0f;
      for (int i = 0; i < n->d[3]; ++i) oi[i] = out_std[i] > 1e-12f ? 1.0f / out_std[i] : 0.0f;
      HMC(hipMemcpyAsync(n->in_mean, in_mean, n->d[0] * sizeof(float), hipMemcpyHostToDevice, n->st));
      HMC(hipMemcpyAsync(n->in_istd, ii.data(), n->d[0] * sizeof(float), hipMemcpyHostToDevice, n->st));
      HMC(hipMemcpyAsync(n->out_mean, out_mean, n->d[3] * sizeof(float), hipMemcpyHostToDevice, n->st));
      HMC(hipMemcpyAsync(n->out_sd, out_std, n->d[3] * sizeof(float), hipMemcpyHostToDevice, n->st));
      HMC(hipMemcpyAsync(n->out_istd, oi.data(), n->d[3] * sizeof(float), hipMemcpyHostToDevice, n->st));
      HMC(hipStreamSynchronize(n->st)));
}

hprqp_status hprqp_mlp_warm_start(hprqp_mlp* n, int32_t batch, const float* X, int32_t qn, int32_t qm, const double* L,
                                  const double* U, double* y0, double* w0, double* x0, int32_t* bad, float* score) {
  HM_GUARD(warm_impl(n, batch, n ? n->maxb : 0, X, qn, qm, L, U, y0, w0, x0, bad, score));
}

hprqp_status hprqp_mlp_warm_starts(hprqp_mlp* n, int32_t count, const float* X, int32_t qn, int32_t qm, const double* L,
                                   const double* U, double* y0, double* w0, double* x0, int32_t* bad, float* score) {
  HM_GUARD(warm_impl(n, count, INT32_MAX, X, qn, qm, L, U, y0, w0, x0, bad, score));
}

hprqp_status hprqp_mlp_fit_scaling(hprqp_mlp* n, int64_t rows, const float* X, const float* T, float* stats_host) {
  HM_GUARD(
      if (!n || !X || !T) mfail(HPRQP_ERR_ARG, "NULL argument");
      if (rows < 2) mfail(HPRQP_ERR_SHAPE, "at least two samples are needed");
      std::vector<float> xm(n->d[0]), xs(n->d[0]), tm(n->d[3]), ts(n->d[3]);
      col_moments(n->st, rows, n->d[0], X, xm.data(), xs.data());
      col_moments(n->st, rows, n->d[3], T, tm.data(), ts.data());
      if (stats_host) {
        float* o = stats_host;
        for (int i = 0; i < n->d[0]; ++i) { o[i] = xm[i]; o[n->d[0] + i] = xs[i]; }
        o += 2 * n->d[0];
        for (int i = 0; i < n->d[3]; ++i) { o[i] = tm[i]; o[n->d[3] + i] = ts[i]; }
      }
      const hprqp_status st = hprqp_mlp_set_scaling(n, xm.data(), xs.data(), tm.data(), ts.data());
      if (st != HPRQP_OK) mfail(st, hq::g_err));
}

hprqp_status hprqp_mlp_intermediate(hprqp_mlp* n, int32_t which, float* out, int32_t* rows_host, int32_t* cols_host) {
  HM_GUARD(
      if (!n) mfail(HPRQP_ERR_ARG, "NULL handle");
      const int B = n->last_batch;
      const int in = n->d[0], h1 = n->d[1], h2 = n->d[2], o = n->d[3];
      const int inp = n->dp[0], h1p = n->dp[1], h2p = n->dp[2], op = n->dp[3];
      struct Src { int cols; long long ld; const float* f; const uint16_t* b; };
      Src s{};
      switch (which) {
        case 0: s = {in, inp, nullptr, n->Xb}; break;
        case 1: s = {h1, h1p, n->Z1, nullptr}; break;
        case 2: s = {h1, h1p, nullptr, n->A1b}; break;
        case 3: s = {h2, h2p, n->Z2, nullptr}; break;
        case 4: s = {h2, h2p, nullptr, n->A2b}; break;
        case 5: s = {o, op, n->Y, nullptr}; break;
        case 6: s = {o, op, n->dYf, nullptr}; break;
        case 7: s = {o, op, nullptr, n->dYb}; break;
        case 8: s = {h2, h2p, n->dA2, nullptr}; break;
        case 9: s = {h2, h2p, n->dZ2f, nullptr}; break;
        case 10: s = {h2, h2p, nullptr, n->dZ2b}; break;
        case 11: s = {h1, h1p, n->dA1, nullptr}; break;
        case 12: s = {h1, h1p, n->dZ1f, nullptr}; break;
        case 13: s = {h1, h1p, nullptr, n->dZ1b}; break;
        case 14: s = {o, o, n->Tstd, nullptr}; break;
        default: mfail(HPRQP_ERR_ARG, "which must be in [0, 14]");
      }
      if (rows_host) *rows_host = B;
      if (cols_host) *cols_host = s.cols;
      if (out && B > 0) {
        k_export<<<eg((long long)B * s.cols), 256, 0, n->st>>>(B, s.cols, s.ld, s.f, s.b, out);
        HMC(hipGetLastError());
      }
      HMC(hipStreamSynchronize(n->st)));
}

hprqp_status hprqp_family_features(int32_t batch, int32_t n, int32_t m, const double* c, const double* u, float* X,
                                   hipStream_t stream) {
  HM_GUARD(if (batch < 0 || n <= 0 || m < 0 || !c || !X || (m > 0 && !u)) mfail(HPRQP_ERR_ARG, "bad arguments");
           if (batch > 0) k_family_features<<<eg((long long)batch * (n + m)), 256, 0, stream>>>(batch, n, m, c, u, X);
           HMC(hipGetLastError()); HMC(hipStreamSynchronize(stream)));
}

hprqp_status hprqp_family_targets(int32_t batch, int32_t n, int32_t m, const double* y, const double* z,
                                  const double* w, const int64_t* iters, float* T, hipStream_t stream) {
  HM_GUARD(if (batch < 0 || n <= 0 || m < 0 || !z || !w || !T || (m > 0 && !y)) mfail(HPRQP_ERR_ARG, "bad arguments");
           if (batch > 0)
             k_family_targets<<<eg((long long)batch * (m + 2 * n + 1)), 256, 0, stream>>>(
                 batch, n, m, y, z, w, reinterpret_cast<const long long*>(iters), T);
           HMC(hipGetLastError()); HMC(hipStreamSynchronize(stream)));
}

hprqp_status hprqp_mlp_loss_grad(hprqp_mlp* n, int32_t batch, const float* X, const float* T, const float* out_w,
                                 float* loss_host, float* grad) {
  HM_GUARD(if (!n) mfail(HPRQP_ERR_ARG, "NULL handle"); loss_grad_impl(*n, batch, X, T, out_w, loss_host, grad));
}

hprqp_status hprqp_mlp_adam(hprqp_mlp* n, float lr, float beta1, float beta2, float eps) {
  HM_GUARD(if (!n) mfail(HPRQP_ERR_ARG, "NULL handle"); n->adam_t += 1;
           const float c1 = 1.0f - std::pow(beta1, (float)n->adam_t);
           const float c2 = 1.0f - std::pow(beta2, (float)n->adam_t);
           AdamArgs a = adam_args(*n); a.step = 1;
           a.lr = lr; a.b1 = beta1; a.b2 = beta2; a.eps = eps; a.c1 = c1; a.c2 = c2;
           const int nb = n->d[1] + n->d[2] + n->d[3];
           k_adam<<<a.tiles[0] + a.tiles[1] + a.tiles[2] + (nb + 255) / 256, 256, 0, n->st>>>(a));
}

hprqp_status hprqp_mlp_get_params(hprqp_mlp* n, float* params_host) {
  HM_GUARD(if (!n || !params_host) mfail(HPRQP_ERR_ARG, "NULL argument");
           HMC(hipMemcpyAsync(params_host, n->P, n->np * sizeof(float), hipMemcpyDeviceToHost, n->st));
           HMC(hipStreamSynchronize(n->st)));
}

hprqp_status hprqp_mlp_set_params(hprqp_mlp* n, const float* params_host) {
  HM_GUARD(if (!n || !params_host) mfail(HPRQP_ERR_ARG, "NULL argument");
           HMC(hipMemcpyAsync(n->P, params_host, n->np * sizeof(float), hipMemcpyHostToDevice, n->st));
           refresh_weights(*n); HMC(hipStreamSynchronize(n->st)));
}

hprqp_status hprqp_mlp_gemm_stats(hprqp_mlp* n, double* ms_host, double* flop_host) {
  HM_GUARD(if (!n) mfail(HPRQP_ERR_ARG, "NULL handle"); HMC(hipStreamSynchronize(n->st)); double ms = 0.0;
           // GEMM intervals: forward (ev0-1); backward (ev2-3) if present
           for (int i = 0; i + 1 < n->nev; i += 2) {
             float t = 0.f;
             HMC(hipEventElapsedTime(&t, n->ev[i], n->ev[i + 1]));
             ms += t;
           } if (ms_host) *ms_host = ms;
           if (flop_host) *flop_host = n->last_flop);
}

void hprqp_mlp_destroy(hprqp_mlp* n) { delete n; }

hprqp_status hprqp_gemm_bf16(int32_t M, int32_t N, int32_t K, const uint16_t* A, int64_t a_rs, int64_t a_cs,
                             const uint16_t* B, int64_t b_rs, int64_t b_cs, float* C, int64_t ldc, int32_t accumulate,
                             int32_t split_k, float* workspace, hipStream_t stream) {
  HM_GUARD(if (M < 0 || N < 0 || K < 0 || !A || !B || !C) mfail(HPRQP_ERR_ARG, "bad GEMM arguments");
           if (split_k < 1 || split_k > 64) mfail(HPRQP_ERR_ARG, "split_k must be in [1, 64]");
           if (split_k > 1 && !workspace) mfail(HPRQP_ERR_ARG, "split_k > 1 needs a workspace of split_k M N floats");
           if (M > 0 && N > 0)
             gemm_split(stream, M, N, K, A, a_rs, a_cs, B, b_rs, b_cs, C, ldc, accumulate, split_k, workspace);
           HMC(hipGetLastError()); HMC(hipStreamSynchronize(stream)));
}

}  // extern "C"
