// Index arithmetic of the golden-label scan as plain constexpr functions, which
// the host's plan, the kernels and the CPU tests (built without HIP) share.
#ifndef LSA_GOLDEN_GEOMETRY_H_
#define LSA_GOLDEN_GEOMETRY_H_

#include <stdint.h>

namespace lsa {

// Rows of up to kGoldenDirectMax entries are held in one workgroup's registers
// (kGoldenHeld per thread) and decided there.  A longer row is scanned first, in
// slices of up to kGoldenSliceVecs float4s (16,384 entries), which leave their
// largest entries to the row kernel: up to kGoldenListMax candidates.  1,344
// rows, us a call, peaked / flat logits, held against scanned: 2,500 entries
// 29 / 33, 54 / 79; 8,192 36 / 52, 39 / 91; 16,384 48 / 74, 45 / 116; with 48
// entries per thread (two workgroups per CU) 24,000 75 / 112, 56 / 134.  Past
// 16,384 peaked rows lose more held than flat ones gain.  Against three passes over
// every row, peaked rows of 16,385 and 24,000 entries take 53 / 87 and 56 / 102 us,
// flat ones 118 to 125 / 100 and 134 to 147 / 126, with p = 1 102 / 91 and 112 / 113;
// from 32,768 entries on none takes longer.
constexpr int kGoldenHeld = 32;
constexpr int kGoldenDirectMax = 512 * kGoldenHeld;
constexpr int kGoldenListMax = 2048;
constexpr int kGoldenSliceVecs = 4096;
constexpr int kGoldenScanThreads = 512;
constexpr int64_t kGoldenScanGrid = 1 << 22;  // slices of one launch
static_assert(kGoldenScanGrid * kGoldenScanThreads < (int64_t(1) << 32), "threads of a grid");
constexpr int kSliceListMax = 340;  // entries a slice lists at most
constexpr int kGoldenSlots = 3072;  // listed entries of a row the row kernel takes in

// What the scan leaves of a slice, in 32-bit words at the slice's share of the
// row's bitmap: the maximum m (float), the threshold key, the sum of the other
// entries' weights 2^(x c - m c) (float), the number of listed entries, then
// `cap` values and `cap` 16-bit entry numbers within the slice.
constexpr int kSliceHead = 4;
// Word of the row's bitmap that marks a scanned row the row kernel leaves open;
// it holds a list entry of the first slice until then.
constexpr int kOpenWord = kSliceHead;

constexpr int least(int a, int b) { return a < b ? a : b; }

// Slices of a row of n entries whose sequence starts at logit `first`, 0 where
// the exact kernel takes the whole row: slices of equal length in float4s; a row
// that may start inside a float4 spans one more.
struct GoldenSlices {
  int32_t slices, slice_vecs;
};
constexpr GoldenSlices golden_slices(int64_t n, int64_t first) {
  if (n <= kGoldenDirectMax) return {0, 0};
  const int64_t vecs = n % 4 == 0 && first % 4 == 0 ? n / 4 : (n + 6) / 4;
  const int64_t ns = (vecs + kGoldenSliceVecs - 1) / kGoldenSliceVecs;
  return {(int32_t)ns, (int32_t)((vecs + ns - 1) / ns)};
}

// The slice's words of the row's bitmap and how many entries it can list, the
// same for every slice of a row.
constexpr int slice_words(int words, int ns) { return words / ns; }
constexpr int slice_cap(int words, int ns) {
  return least((slice_words(words, ns) - kSliceHead) * 2 / 3, least(kGoldenSlots / ns, kSliceListMax));
}

// Slice sl of the row that starts at logit `first`: float4 v of the row holds
// its entries 4 v - lead .. + 3 and sits at logit first - lead + 4 v, a multiple
// of 4; the slice takes float4s v0 .. v1 - 1, of which the first `have` lie
// within the row (the next one, if any, reaches past its end).
struct ScanSlice {
  int lead, v0, v1, have;
};
constexpr ScanSlice scan_slice(int64_t first, int n, int slice_vecs, int sl) {
  const int lead = (int)(first & 3), v0 = sl * slice_vecs;
  const int v1 = least(v0 + slice_vecs, (n + lead + 3) >> 2);
  return {lead, v0, v1, least(v1, (n + lead) / 4) - v0};
}
// Byte offset within the slice of float4 j of thread tid.
constexpr int scan_offset(int tid, int j) { return 16 * (tid + kGoldenScanThreads * j); }

// Slot f of a row kernel's list is entry f % cap of slice f / cap; the division
// by multiplication is exact for f < 2^16.
constexpr uint32_t slot_inverse(uint32_t cap) { return (0xFFFFFFFFu + (uint64_t)cap) / cap; }
constexpr uint32_t slot_slice(uint32_t f, uint32_t inverse) { return (uint32_t)(((uint64_t)f * inverse) >> 32); }
// Entry of the row that entry `id` of slice s stands for.
constexpr uint32_t slice_entry(uint32_t s, int slice_vecs, uint32_t id, int lead) {
  return 4u * s * (uint32_t)slice_vecs + id - (uint32_t)lead;
}

// Scale of a slice's sum: the weight of entry x is 2^(x c + off) with c =
// kSliceLog2e and off = -m c, each rounded to float32 (m: the slice's maximum).
constexpr float kSliceLog2e = 1.44269502f;
constexpr float slice_off(float m) { return m == -__builtin_inff() ? 0.f : -(m * kSliceLog2e); }

// How far a slice's sum R of n weights e^-d (d: the distance below the slice's
// maximum m; M is the row's) may be from the exact masses of the same entries,
// relative to R, beyond which the exact masses only lose their floor.  Entry by
// entry the errors are at most
//   1.34e-8 |x|            c against log2 e (|x| <= |m| + d), in the exponent
//   6e-8 d                 the rounding of the exponent, at most d / log 2 in size
//   2.4e-7                 the hardware's exponential
//   5.4e-7                 nine roundings of the float32 sums
//   6e-8 (d + M - m + 4)   the exact method itself
// and the mean of d over the weights is at most mean_d = log(n / R), its value
// when all of them are equal.  (Entries further than 87 below m have no weight.)
// The first is an error e of the exponent, a factor of up to exp(e) <= 1 + e + e^2
// for e < 1; logits of 10^7 reach 0.14, and past e = 1 the sum says nothing.
constexpr double slice_error(double m, double M, double mean_d) {
  const double e = 1.4e-8 * (m < 0.0 ? -m : m) + 1.5e-7 * mean_d + 6e-8 * (M - m) + 1.1e-6;
  return e < 1.0 ? e + e * e : __builtin_inf();
}

// Whether no entry of a slice has any mass: every one lies more than 64 below
// the row's maximum M, where the fixed exponential is 0 (as are the masses from
// 27.8 on).  Slices masked with a large negative number, the type's lowest one
// among them, whose sum may be infinite or not a number.
constexpr bool slice_weightless(double m, double M) { return M - m > 64.0; }

}  // namespace lsa

#endif  // LSA_GOLDEN_GEOMETRY_H_
