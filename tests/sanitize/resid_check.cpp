// Host check of the split of a CSR matrix's rows among the slots of the
// residual kernel (layout.hpp): every row once, in order, and no slot with more
// work than its share and one row; and of its batches of nonzeros.
#include <algorithm>
#include <climits>
#include <cstdio>
#include <random>
#include <vector>

#include "layout.hpp"

static int failures = 0;
#define CHECK(c)                                              \
  do {                                                        \
    if (!(c)) {                                               \
      std::printf("line %d: %s\n", __LINE__, #c);             \
      ++failures;                                             \
    }                                                         \
  } while (0)

static void split(const std::vector<int>& rp, int64_t nslot) {
  const int64_t n = (int64_t)rp.size() - 1, nnz = rp[n];
  int64_t longest = 0;
  for (int64_t r = 0; r < n; ++r) longest = std::max<int64_t>(longest, rp[r + 1] - rp[r]);
  const int64_t total = rks::resid_key(nnz, n), share = (total + nslot - 1) / nslot;
  int64_t next = 0;
  for (int64_t s = 0; s < nslot; ++s) {
    const int64_t r0 = rks::resid_row_at(rp.data(), n, std::min(total, s * share));
    const int64_t r1 = rks::resid_row_at(rp.data(), n, std::min(total, (s + 1) * share));
    CHECK(r0 == next && r0 <= r1 && r1 <= n);
    CHECK(rks::resid_key(rp[r1], r1) - rks::resid_key(rp[r0], r0) <= share + longest + rks::kResidRowCost);
    next = r1;
  }
  CHECK(next == n);
}

// The last entries of the largest matrix: every entry once, none past the end.
static void batches(uint32_t e0, uint32_t et, uint32_t u) {
  uint32_t next = e0;
  for (uint32_t e = e0; e < et; e += u)
    for (uint32_t q = 0; q < u; ++q) {
      const uint32_t eq = rks::batch_entry(e, q, et);
      CHECK(eq >= e0 && eq < et);
      if (e + q < et) CHECK(eq == next++);
    }
  CHECK(next == et);
}

int main() {
  for (int len = 1; len < 40; ++len)
    for (int et : {40, INT_MAX - 7, INT_MAX}) batches(et - len, et, 8);
  std::mt19937 g(7);
  for (int64_t n : {4, 64, 1031, 40000})
    for (int kind = 0; kind < 5; ++kind) {
      std::vector<int> rp(n + 1, 0);
      for (int64_t r = 0; r < n; ++r) {
        int len = (int)(g() % 30);
        if (kind == 1) len = 0;                              // no nonzeros
        if (kind == 2 && r >= n / 2) len = 0;                // a run of empty rows at the end
        if (kind == 3 && r >= n / 8 && r < n - 2) len = 0;   // inside
        if (kind == 4 && r != n / 3) len = 0;                // one row
        rp[r + 1] = rp[r] + len;
      }
      for (int64_t nslot : {32, 256, 65536}) split(rp, nslot);
    }
  std::printf("ok: %d failures\n", failures);
  return failures != 0;
}
