// Walks the index arithmetic of the golden-label scan for many shapes and
// aborts on the first access that leaves its buffer: slices of the logits,
// list entries and headers in the row bitmaps, the row kernel's slots.
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>

#include <random>
#include <vector>

#include "golden_geometry.h"

using namespace lsa;

#define CHECK(c)                                                                                   \
  do {                                                                                             \
    if (!(c)) {                                                                                    \
      printf("n=%lld first=%lld slice=%d: %s\n", (long long)g_n, (long long)g_first, g_slice, #c); \
      exit(1);                                                                                     \
    }                                                                                              \
  } while (0)

static int64_t g_n, g_first;
static int g_slice;

// One row of n entries at logit `first` of a sequence that starts at seq_first,
// in a buffer of `total` logits.
static void check_row(int64_t n, int64_t seq_first, int64_t first, int64_t total, bool every_load) {
  const GoldenSlices gs = golden_slices(n, seq_first);
  const int ns = gs.slices, words = (int)((n + 31) / 32), sw = slice_words(words, ns), cap = slice_cap(words, ns);
  g_n = n, g_first = first, g_slice = -1;
  CHECK(ns >= 1 && sw * ns <= words);
  CHECK(cap >= 1 && cap <= kSliceListMax && cap * ns <= kGoldenSlots);
  CHECK(kOpenWord < sw && kOpenWord >= kSliceHead);  // no slice's header
  CHECK(kSliceHead + cap + (cap + 1) / 2 <= sw);     // header, values, 16-bit entry numbers
  int end = 0;
  for (int sl = 0; sl < ns; ++sl) {
    g_slice = sl;
    const ScanSlice s = scan_slice(first, (int)n, gs.slice_vecs, sl);
    const int64_t at = first - s.lead + 4 * (int64_t)s.v0;
    CHECK(s.v0 == end && s.v1 > s.v0 && s.v1 - s.v0 <= kGoldenSliceVecs);  // no gap, no overlap
    end = s.v1;
    CHECK(at >= 0 && at % 4 == 0);
    CHECK(s.have >= 0 && s.have <= s.v1 - s.v0 && s.have >= s.v1 - s.v0 - 1);
    CHECK(at + 4 * (int64_t)s.have <= first + n && first + n <= total);
    // a load is inside the row's buffer or past its records, where it returns 0
    const int64_t records = 16 * (int64_t)s.have;
    const int loads = kGoldenSliceVecs / kGoldenScanThreads;
    int64_t seen = 0;
    for (int j = 0; j < loads; ++j)
      for (int t = 0; t < kGoldenScanThreads; t += every_load ? 1 : kGoldenScanThreads - 1) {
        const int64_t off = scan_offset(t, j);
        CHECK(off >= 0 && off + 16 <= 16 * (int64_t)kGoldenSliceVecs);
        CHECK(off % 16 == 0 && (off + 16 <= records || off >= records));
        CHECK(off >= records || at + off / 4 + 4 <= total);
        seen += off < records;
      }
    if (every_load) CHECK(seen == s.have);
    // the entries of the float4 that reaches past the row's end
    const int64_t left = n + s.lead - 4 * ((int64_t)s.v0 + s.have);
    if (s.have < s.v1 - s.v0) {
      CHECK(sl == ns - 1 && left >= 1 && left <= 3);
      CHECK(at + 4 * (int64_t)s.have + left == first + n);
    }
    // entry numbers: 16 bits, and the row's own entries
    const int64_t last = 4 * (int64_t)(s.v1 - s.v0) - 1;
    CHECK(last < 65536 && scan_offset(kGoldenScanThreads - 1, loads - 1) / 4 + 3 < 65536);
    const uint32_t id0 = sl == 0 ? (uint32_t)s.lead : 0u;
    CHECK(slice_entry((uint32_t)sl, gs.slice_vecs, id0, s.lead) == (uint32_t)(4 * s.v0 + (int)id0 - s.lead));
    const int64_t top = sl == ns - 1 ? n - 1 : 4 * (int64_t)s.v1 - s.lead - 1;
    CHECK(slice_entry((uint32_t)sl, gs.slice_vecs, (uint32_t)(top + s.lead - 4 * (int64_t)s.v0), s.lead) == (uint32_t)top);
    CHECK(top < n);
  }
  g_slice = -1;
  CHECK(end == (n + (first & 3) + 3) / 4);  // the whole row
  const uint32_t inv = slot_inverse((uint32_t)cap);
  for (uint32_t f = 0; f < (uint32_t)kGoldenSlots; ++f) CHECK(slot_slice(f, inv) == f / (uint32_t)cap);
}

int main() {
  std::mt19937_64 rng(5);
  long rows = 0;
  auto sequence = [&](int64_t n, int64_t seq_first, int64_t n_rows, int64_t total, bool every_load) {
    if (golden_slices(n, seq_first).slices == 0) return;
    for (int64_t r = 0; r < 4 && r < n_rows; ++r, ++rows) check_row(n, seq_first, seq_first + r * n, total, every_load);
    check_row(n, seq_first, seq_first + (n_rows - 1) * n, total, every_load);
  };
  // every length up to five slices, at every start within a float4
  for (int64_t n = kGoldenDirectMax + 1; n <= 5 * 16384 + 70; n += n < 17000 ? 1 : 13)
    for (int64_t first = 0; first < 4; ++first) sequence(n, first, 5, first + 5 * n, n < 16500 || n % 509 == 0);
  // lengths around every whole number of slices, up to the longest
  for (int64_t k = 1; k <= 256; ++k)
    for (int64_t d = -9; d <= 9; ++d) {
      const int64_t n = k * 16384 + d;
      if (n <= 4194304) sequence(n, (int64_t)(rng() % 8), 3, 8 + 3 * n, false);
    }
  // ragged batches laid out as the plan does
  for (int it = 0; it < 3000; ++it) {
    const int batch = 1 + (int)(rng() % 64);
    const int64_t n_rows = (1 + (int64_t)(rng() % 64)) * (1 + (int64_t)(rng() % 63));
    std::vector<int64_t> n(batch);
    int64_t entries = 0;
    for (auto& x : n) {
      x = 1 + (int64_t)(rng() % (1ull << (rng() % 23)));
      entries += x;
    }
    int64_t off = 0;
    for (const auto x : n) {
      sequence(x, n_rows * off, n_rows, n_rows * entries, false);
      off += x;
    }
  }
  printf("ok: %ld rows\n", rows);
  return 0;
}
