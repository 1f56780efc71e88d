// Host-side check of the shape of the stream product and of the positions that the
// row-split products read (csrc/spmv.hpp):
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

// k_csr: G lanes, steps of eight entries a lane
static void check_split(long long b, long long en, int G) {
  std::vector<int> taken(en - b, 0);
  for (int lane = 0; lane < G; ++lane) {
    RowSpan r((int)b, (int)en, lane);
    for (int step = 0; r.left > 0; ++step) {
      if (step > 3 + (int)((en - b) / G)) { CHECK(false, "no end: b %lld en %lld G %d", b, en, G); break; }
      for (int u = 0; u < 8; ++u) {
        if (u * G >= r.left) continue;
        const long long kk = (long long)(r.at + u * G);
        CHECK(kk >= b && kk < en, "read %lld of [%lld, %lld) G %d", kk, b, en, G);
        if (kk >= b && kk < en) ++taken[kk - b];
      }
      r.skip(8 * G);
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

// shape of the stream product: rows per block and entries a thread, of those built
static void check_shapes() {
  const int ncu = 256;
  auto want = [&](int rows, long long nnz, int maxlen, int shape) {
    const int got = stream_shape(rows, nnz, maxlen, ncu);
    CHECK(got == shape, "stream_shape(%d, %lld, %d) = %d, not %d", rows, nnz, maxlen, got, shape);
  };
  // rows of equal length take the smallest chunk that holds them
  want(90000, 180000, 2, 2562);      // (the assignment rows of A^T)
  want(65536, 4 * 65536ll, 4, 2564);
  want(65536, 8 * 65536ll, 8, 2568);
  want(32768, 8 * 32768ll, 8, 1284);
  want(16384, 16 * 16384ll, 16, 644);
  want(5000, 16 * 5000ll, 16, 322);
  // lengths that vary, or are not known, leave 5%
  want(90000, 180000, 9, 2564);
  want(90000, 180000, -1, 2564);
  want(1000000, 2500000, 12, 2564);
  // even rows of 8 to 32: many of them in several chunks of 256 rows, fewer in small blocks
  want(98304, 98304 * 17ll, 40, 2568);
  want(98303, 98303 * 17ll, 40, 324);
  want(390000, 390000 * 31ll, 60, 2568);
  want(98303, 98303 * 12ll, 30, 1288);
  want(49152, 49152 * 12ll, 30, 1288);
  want(49151, 49151 * 12ll, 30, 644);
  want(196607, 196607 * 12ll, 30, 1288);
  want(196608, 196608 * 12ll, 30, 2568);
  // uneven ones in blocks of 64
  want(390000, 390000 * 15ll, 90, 2568);
  want(390000, 390000 * 15ll, 91, 648);
  want(16384, 16384 * 15ll, 91, 648);
  want(16383, 16383 * 15ll, 91, 322);
  want(390000, 390000 * 17ll, -1, 648);
  // a longest row of any size does not wrap
  want(98303, 98303 * 12ll, 2147483647, 648);
  for (long long rows : {0ll, 1ll, 31ll, 8191ll, 8192ll, 16384ll, 32768ll, 65535ll, 65536ll, 98304ll, 5000000ll, 67000000ll})
    for (int avg = 0; avg <= 32; ++avg) {
      const int shape = stream_shape((int)rows, rows * avg, -1, ncu);
      bool built = false;
      for (int s : {322, 324, 642, 644, 648, 1284, 1288, 2562, 2564, 2568}) built |= s == shape;
      CHECK(built, "stream_shape(%lld, avg %d) = %d: no such kernel", rows, avg, shape);
    }
}

int main() {
  check_shapes();
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
