// Host-side check of the operand addresses of the Kronecker GEMM (csrc/qops.hpp):
// the base and offset functions that the kernel calls, for the untransposed operand
// X (s x p) and the transposed factor (p x p), against 64-bit arithmetic at sizes up
// to the largest n that a problem can have.  Built host-only (no kernel runs, no GPU
// needed).  Prints "OK" and exits 0 on success.
#include <algorithm>
#include <cstdio>
#include "qops.hpp"

static long long failures = 0;

// every lane's address in the tile at column j0, for the K blocks at k0 = 0 and at the end
static void check_tile(int transb, int ld, int N, int K, int tn, int j0) {
  const long long base = gemm_b_base(transb, ld, j0);
  const long long sb = transb ? 8ll * ld : 8ll;   // bytes per k
  for (int k0 : {0, std::max(0, K - 16)})
    for (int j = 0; j < tn; ++j)
      for (int k = 0; k < std::min(16, K); ++k) {
        const int jt = std::min(j, N - 1 - j0);
        const long long got = base + sb * (k0 + k % 4) + (long long)gemm_b_offset(transb, ld, jt, k & ~3);
        const long long J = j0 + jt, Kk = k0 + k;
        const long long want = 8ll * (transb ? J + (long long)ld * Kk : Kk + (long long)ld * J);
        if (got != want && ++failures <= 10)
          std::printf("transb %d ld %d N %d j0 %d j %d k %lld: %lld, not %lld\n", transb, ld, N, j0, j, Kk, got, want);
      }
}

int main() {
  // (s, p): s p = n below 2^31; 190,000 is the largest order of a factor in 288 GB
  const int sizes[][2] = {{1, 1}, {3, 40}, {300, 290}, {16384, 32767}, {16384, 32768}, {23170, 23170}, {23171, 23171},
                          {8192, 65536}, {65536, 8192}, {46340, 46340}, {11302, 190000}, {190000, 11302}};
  for (const auto& sp : sizes) {
    const int s = sp[0], p = sp[1];
    for (int tn : {16, 32}) {
      const int tiles = (p + tn - 1) / tn;
      for (int t = 0; t < tiles; t += std::max(1, tiles / 37)) {
        check_tile(0, s, p, s, tn, t * tn);
        check_tile(1, p, p, p, tn, t * tn);
      }
      check_tile(0, s, p, s, tn, (tiles - 1) * tn);
      check_tile(1, p, p, p, tn, (tiles - 1) * tn);
    }
  }
  std::printf(failures ? "FAILED (%lld)\n" : "OK\n", failures);
  return failures != 0;
}
