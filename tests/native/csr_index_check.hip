// Host-side check of the positions that the row-split products read (csrc/spmv.hpp):
// the position functions that the kernels call, stepped as the kernels step them, over
// rows that begin and end anywhere in the 32-bit range, up to its very end.  Every
// entry of a row is taken once, nothing outside of it is used, and what is read in
// place of a missing entry lies in the matrix.  Built host-only (no kernel runs, no
// GPU needed).  Prints "OK" and exits 0 on success.
#include <cstdio>
#include <algorithm>
#include <vector>
#include "spmv.hpp"

static long long failures = 0;
#define CHECK(c, ...)                                          \
  do {                                                         \
    if (!(c) && ++failures <= 20) { std::printf(__VA_ARGS__); std::printf("\n"); } \
  } while (0)

// k_csr: G lanes, steps of four entries a lane
static void check_split(long long b, long long en, int G) {
  std::vector<int> taken(en - b, 0);
  for (int lane = 0; lane < G; ++lane) {
    RowSpan r((int)b, (int)en, lane);
    for (int step = 0; r.left > 0; ++step) {
      if (step > 3 + (int)((en - b) / G)) { CHECK(false, "no end: b %lld en %lld G %d", b, en, G); break; }
      for (int u = 0; u < 4; ++u) {
        const long long kk = (long long)(r.at + std::min(u * G, r.left - 1));
        CHECK(kk >= b && kk < en, "read %lld of [%lld, %lld) G %d", kk, b, en, G);
        if (u * G < r.left && kk >= b && kk < en) ++taken[kk - b];
      }
      r.skip(4 * G);
    }
  }
  for (long long k = b; k < en; ++k) CHECK(taken[k - b] == 1, "entry %lld of [%lld, %lld) taken %d times, G %d", k, b, en, taken[k - b], G);
}

// k_csr_xrow: pairs, four of them a lane in flight, then the rest; nnz entries in all
static void check_pairs(long long b, long long en, int G, long long nnz) {
  const RowPairs p{(int)b, (int)en};
  std::vector<int> taken(en - b, 0);
  auto take = [&](long long k) { CHECK(k >= b && k < en, "used %lld of [%lld, %lld) G %d", k, b, en, G); if (k >= b && k < en) ++taken[k - b]; };
  for (int lane = 0; lane < G; ++lane) {
    for (int u = 0; u < HQ_XROW_U / 2; ++u) {
      const int rel = 2 * lane + 2 * u * G;
      const long long k = p.at(rel);
      CHECK(k >= 0 && k < nnz, "read %lld of %lld: [%lld, %lld) G %d", k, nnz, b, en, G);
      if (p.first(rel)) { CHECK(k == p.base() + (long long)rel, "pair at %lld", k); take(k); }
      if (p.second(rel)) { CHECK(k == p.base() + (long long)rel, "pair at %lld", k); take(k + 1); }
    }
    for (unsigned rel = 2 * lane + HQ_XROW_U * G; rel < (unsigned)p.len(); rel += 2 * G) {
      take((long long)p.base() + rel);
      if (rel + 1 < (unsigned)p.len()) take((long long)p.base() + rel + 1);
    }
  }
  for (long long k = b; k < en; ++k) CHECK(taken[k - b] == 1, "entry %lld of [%lld, %lld) taken %d times, G %d (pairs)", k, b, en, taken[k - b], G);
}

int main() {
  const long long top = (1ll << 31) - 1;
  for (int G = 1; G <= HQ_BLOCK; G *= 2)
    for (long long gap : {0ll, 1ll, 2ll, 63ll, 64ll, 255ll, 256ll, 500ll, 511ll, 512ll, 1023ll, 1024ll, 2048ll, top - 5000})
      for (int len : {0, 1, 2, 3, 5, 8, 31, 64, 65, 74, 257, 511, 512, 513, 1024, 1300, 4096}) {
        const long long en = top - gap, b = en - len;
        check_split(b, en, G);
        if (G <= HQ_WAVE) check_pairs(b, en, G, top - gap + (gap < 5 ? gap : 5));
      }
  for (int G = 1; G <= HQ_WAVE; G *= 2)
    for (int b : {0, 1, 2, 3})
      for (int len : {0, 1, 2, 3, 9, 64, 600}) {
        if (b + len < 2) continue;   // (the pairs need two entries)
        check_pairs(b, b + len, G, b + len);
      }
  std::printf(failures ? "FAILED (%lld)\n" : "OK\n", failures);
  return failures != 0;
}
